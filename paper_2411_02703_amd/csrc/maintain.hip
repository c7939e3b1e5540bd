// Map maintenance on the GPU (LVI-GS Section III-C): opacity pruning.  The delay buffer of Section III-C exists
// so that freshly initialised Gaussians are not removed "before they can be observed" once their opacity has
// dropped to the prunable threshold; this is the removal itself: every Gaussian whose opacity sigmoid(logit)
// lies below the threshold is dropped, and the survivors' parameters and Adam moments are compacted to the
// front of the output arrays in their original order.
//
// Work: one flag per Gaussian, an exclusive scan of the flags (the library's scan), then a gather of every kept
// row of the fifteen arrays (five parameter groups x params, m, v; see copy_rows).  HBM-bound: 3 (44 + 12K) bytes
// read and at most as many written per Gaussian.
#include "common.h"

namespace {

// keep[i] = (opacity logit >= thr): the decision is a float comparison of the logit with the threshold's logit
// (computed once on the host), so it is exact and identical wherever it is evaluated.
__global__ void k_prune_flags(const float* __restrict__ opac, int64_t n, float thr, int32_t* __restrict__ keep) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) keep[i] = opac[i] >= thr ? 1 : 0;
}

struct Rows {
  const float* in[15];
  float* out[15];
  int len[15];  // floats per Gaussian
};

Rows rows_of(const gs_params& p, const gs_params& m, const gs_params& v, const gs_params& op, const gs_params& om,
             const gs_params& ov) {
  const int K3 = 3 * (p.sh_degree + 1) * (p.sh_degree + 1);
  Rows r;
  const gs_params* src[3] = {&p, &m, &v};
  const gs_params* dst[3] = {&op, &om, &ov};
  for (int k = 0; k < 3; ++k) {
    r.in[5 * k + 0] = src[k]->means;      r.out[5 * k + 0] = dst[k]->means;      r.len[5 * k + 0] = 3;
    r.in[5 * k + 1] = src[k]->log_scales; r.out[5 * k + 1] = dst[k]->log_scales; r.len[5 * k + 1] = 3;
    r.in[5 * k + 2] = src[k]->quats;      r.out[5 * k + 2] = dst[k]->quats;      r.len[5 * k + 2] = 4;
    r.in[5 * k + 3] = src[k]->opacity;    r.out[5 * k + 3] = dst[k]->opacity;    r.len[5 * k + 3] = 1;
    r.in[5 * k + 4] = src[k]->sh;         r.out[5 * k + 4] = dst[k]->sh;         r.len[5 * k + 4] = K3;
  }
  return r;
}

// A block copies the rows src[0, m) (in LDS, at most 256) of five arrays to the consecutive rows from row0 on, and blockIdx.y selects
// parameters or moments.  What bounds it is HBM: reads and writes run element by element over the block's output, which
// is contiguous, up to four loads a thread in flight, in 16-byte words where both arrays' rows are made of them.  The row
// of a word is e / units by a multiplication (a 64-bit division per element had made the copy of 1M Gaussians of degree
// 3 VALU-bound: 514 us pruned, 576 us permuted).
constexpr int kRowBlock = 256;

// Rows a block copies: some 4 k words of an array set, and few where there are few Gaussians.  Prune of 1M at 64, 128 and
// 256 rows: degree 0 163, 129, 92 us; degree 2 217, 202, 208; degree 3 282, 297, 310.  Of 6 k of degree 0 22.7, 22.9, 23.1,
// of 12 k 23.0, 23.2, 23.5, of 24 k 24.3, 23.8, 24.0, of 40 k 26.1, 25.0, 24.8 (the reorder's random reads hardly differ).
inline int rows_per_block(int64_t n, int sh_degree) {
  return n < (int64_t(1) << 14) || sh_degree >= 3 ? 64 : sh_degree == 2 ? 128 : 256;
}

template <int B, class T>
__device__ __forceinline__ void copy_batch(const T* __restrict__ in, T* __restrict__ out, int e, int units, uint32_t inv,
                                           const int32_t* src) {
  T v[B];
#pragma unroll
  for (int i = 0; i < B; ++i) {
    const int r = (int)((uint32_t)(e + i * kRowBlock) * inv >> 22);
    v[i] = in[(int64_t)src[r] * units + (e + i * kRowBlock - r * units)];
  }
#pragma unroll
  for (int i = 0; i < B; ++i) out[e + i * kRowBlock] = v[i];
}

template <class T>
__device__ __forceinline__ void copy_units(const T* __restrict__ in, T* __restrict__ out, int64_t row0, int m, int units,
                                           const int32_t* src) {
  // e / units = (e inv) >> 22 for e < 256 units, units <= 75: e (inv units - 2^22) < 2^22 and e inv < 2^31
  const uint32_t inv = ((1u << 22) + (uint32_t)units - 1) / (uint32_t)units;
  const int total = m * units;
  out += row0 * units;
  int e = threadIdx.x;
  for (; e + 3 * kRowBlock < total; e += 4 * kRowBlock) copy_batch<4>(in, out, e, units, inv, src);
  if (e + 2 * kRowBlock < total) {
    copy_batch<3>(in, out, e, units, inv, src);
    e += 3 * kRowBlock;
  }
  for (; e < total; e += kRowBlock) copy_batch<1>(in, out, e, units, inv, src);
}

__device__ __forceinline__ void copy_rows(const Rows& r, int64_t row0, int m, const int32_t* src) {
#pragma unroll
  for (int k = 4; k >= 0; --k) {
    const int a = 5 * blockIdx.y + k, len = r.len[a];
    const float* in = r.in[a];
    float* out = r.out[a];
    if (len % 4 == 0 && ((reinterpret_cast<uintptr_t>(in) | reinterpret_cast<uintptr_t>(out)) & 15) == 0)
      copy_units(reinterpret_cast<const float4*>(in), reinterpret_cast<float4*>(out), row0, m, len / 4, src);
    else
      copy_units(in, out, row0, m, len, src);
  }
}

// Block b lists the kept ones of its `rows` Gaussians; their output rows are consecutive.  The last one writes the total.
__global__ __launch_bounds__(kRowBlock) void k_prune_gather(const Rows r, int64_t n, int rows,
                                                            const int32_t* __restrict__ keep,
                                                            const int32_t* __restrict__ off,
                                                            int64_t* __restrict__ n_kept) {
  __shared__ int32_t src[kRowBlock];
  const int64_t g0 = (int64_t)blockIdx.x * rows, g = g0 + threadIdx.x, last = min(g0 + rows, n) - 1;
  const int32_t row0 = off[g0];
  if (g <= last && keep[g]) src[off[g] - row0] = (int32_t)g;
  if (last == n - 1 && blockIdx.y == 0 && threadIdx.x == 0) n_kept[0] = (int64_t)off[last] + keep[last];
  __syncthreads();
  copy_rows(r, row0, off[last] + keep[last] - row0, src);
}

}  // namespace

namespace gs_launch {

size_t prune_scratch_ints(int64_t n) { return 2 * (size_t)((n + 63) / 64 * 64) + scan_scratch_ints(n); }

hipError_t prune(const gs_params& p, const gs_params& m, const gs_params& v, float thr_logit, const gs_params& op,
                 const gs_params& om, const gs_params& ov, int64_t* n_kept, int32_t* scratch, hipStream_t st) {
  const int64_t n = p.n;
  const size_t na = (size_t)((n + 63) / 64 * 64);
  int32_t* keep = scratch;
  int32_t* off = scratch + na;
  int32_t* scan_scr = scratch + 2 * na;
  const unsigned blocks = (unsigned)((n + 255) / 256);
  k_prune_flags<<<blocks, 256, 0, st>>>(p.opacity, n, thr_logit, keep);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  if ((e = scan_exclusive(keep, off, n, scan_scr, st)) != hipSuccess) return e;
  const int rows = rows_per_block(n, p.sh_degree);
  k_prune_gather<<<dim3((unsigned)((n + rows - 1) / rows), 3), kRowBlock, 0, st>>>(rows_of(p, m, v, op, om, ov), n, rows,
                                                                                  keep, off, n_kept);
  return hipGetLastError();
}

}  // namespace gs_launch

// ------------------------------------------------------------------ spatial order
// Gaussians ordered along a Z-order (Morton) curve of their means: neighbouring Gaussians then sit in neighbouring
// rows, so the threads of one wave see nearly the same views in projection and its backward, records gathered by a
// tile come from nearby memory, and emission writes longer runs.  Each coordinate is quantised to 21 bits over
// the means' bounding box, q = min(2^21 - 1, floor((x - lo) * s)) with s = (2^21 - 1) / max(hi - lo, 1e-30) (FP32,
// no contraction), and the three are interleaved (x in bit 3k, y in 3k + 1, z in 3k + 2).  A stable radix sort
// of the codes gives the permutation; rows of parameters and moments are gathered through it.
namespace {

__device__ __forceinline__ uint32_t ordered_bits(float x) {
  const uint32_t u = __float_as_uint(x);
  return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}
__device__ __forceinline__ float from_ordered(uint32_t o) {
  return __uint_as_float((o & 0x80000000u) ? (o & 0x7fffffffu) : ~o);
}

// Few blocks (kBoxBlocks), each reduced in LDS before its six atomics: they all meet in one cache line, about 5 ns each
// (with six per wave of 2048 blocks the box of 1M means took 560 us).
constexpr int kBoxBlocks = 128;
constexpr int kBoxThreads = 1024;

__global__ __launch_bounds__(kBoxThreads) void k_bbox(const float* __restrict__ means, int64_t n,
                                                      uint32_t* __restrict__ box) {
  __shared__ uint32_t sh[6][kBoxThreads / 64];
  uint32_t b[6] = {~0u, ~0u, ~0u, 0u, 0u, 0u};
#pragma unroll 4
  for (int64_t g = (int64_t)blockIdx.x * kBoxThreads + threadIdx.x; g < n; g += (int64_t)gridDim.x * kBoxThreads)
    for (int k = 0; k < 3; ++k) {
      const uint32_t o = ordered_bits(means[3 * g + k]);
      b[k] = min(b[k], o);
      b[3 + k] = max(b[3 + k], o);
    }
  for (int k = 0; k < 6; ++k) {
    for (int s = 32; s >= 1; s >>= 1) {
      const uint32_t o = (uint32_t)__shfl_xor((int)b[k], s);
      b[k] = k < 3 ? min(b[k], o) : max(b[k], o);
    }
    if ((threadIdx.x & 63) == 0) sh[k][threadIdx.x >> 6] = b[k];
  }
  __syncthreads();
  if (threadIdx.x < 6) {
    const int k = threadIdx.x;
    uint32_t x = sh[k][0];
    for (int w = 1; w < kBoxThreads / 64; ++w) x = k < 3 ? min(x, sh[k][w]) : max(x, sh[k][w]);
    if (k < 3) atomicMin(box + k, x);
    else atomicMax(box + k, x);
  }
}

__device__ __forceinline__ uint64_t spread3(uint32_t v) {
  uint64_t x = v & 0x1fffffu;
  x = (x | (x << 32)) & 0x1f00000000ffffull;
  x = (x | (x << 16)) & 0x1f0000ff0000ffull;
  x = (x | (x << 8)) & 0x100f00f00f00f00full;
  x = (x | (x << 4)) & 0x10c30c30c30c30c3ull;
  x = (x | (x << 2)) & 0x1249249249249249ull;
  return x;
}

__global__ void k_morton(const float* __restrict__ means, int64_t n, const uint32_t* __restrict__ box,
                         uint64_t* __restrict__ keys, int32_t* __restrict__ vals) {
#pragma clang fp contract(off)
  const int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (g >= n) return;
  uint64_t code = 0;
  for (int k = 0; k < 3; ++k) {
    const float lo = from_ordered(box[k]), hi = from_ordered(box[3 + k]);
    const float s = 2097151.0f / fmaxf(hi - lo, 1e-30f);
    const float t = (means[3 * g + k] - lo) * s;
    const uint32_t q = (uint32_t)fminf(floorf(t), 2097151.0f);
    code |= spread3(q) << k;
  }
  keys[g] = code;
  vals[g] = (int32_t)g;
}

// out row k = in row perm[k]
__global__ __launch_bounds__(kRowBlock) void k_permute(const Rows r, int64_t n, int rows,
                                                       const int32_t* __restrict__ perm) {
  __shared__ int32_t src[kRowBlock];
  const int64_t k0 = (int64_t)blockIdx.x * rows;
  const int m = (int)min((int64_t)rows, n - k0);
  if ((int)threadIdx.x < m) src[threadIdx.x] = perm[k0 + threadIdx.x];
  __syncthreads();
  copy_rows(r, k0, m, src);
}

}  // namespace

namespace gs_launch {

// scratch: keys x2 (u64) + vals x2 + box + sort scratch
size_t order_scratch_ints(int64_t n) {
  const size_t a = (size_t)((n + 63) / 64 * 64);
  return 2 * 2 * a + 2 * a + 64 + sort_scratch_ints(n);
}

hipError_t spatial_order(const gs_params& p, const gs_params& m, const gs_params& v, const gs_params& op,
                         const gs_params& om, const gs_params& ov, int32_t* perm_out, int32_t* scratch,
                         hipStream_t st) {
  const int64_t n = p.n;
  const size_t a = (size_t)((n + 63) / 64 * 64);
  auto* k0 = reinterpret_cast<uint64_t*>(scratch);
  auto* k1 = reinterpret_cast<uint64_t*>(scratch + 2 * a);
  int32_t* v0 = scratch + 4 * a;
  int32_t* v1 = scratch + 5 * a;
  auto* box = reinterpret_cast<uint32_t*>(scratch + 6 * a);
  int32_t* sort_scr = scratch + 6 * a + 64;
  hipError_t e = fill_i32(reinterpret_cast<int32_t*>(box), -1, 3, st);  // lo = all ones
  if (e != hipSuccess) return e;
  if ((e = fill_i32(reinterpret_cast<int32_t*>(box) + 3, 0, 3, st)) != hipSuccess) return e;
  int64_t nb = (n + kBoxThreads - 1) / kBoxThreads;
  if (nb > kBoxBlocks) nb = kBoxBlocks;
  k_bbox<<<(unsigned)nb, kBoxThreads, 0, st>>>(p.means, n, box);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  k_morton<<<(unsigned)((n + 255) / 256), 256, 0, st>>>(p.means, n, box, k0, v0);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  if ((e = sort_pairs(k0, v0, k1, v1, n, nullptr, n, 64, sort_scr, st)) != hipSuccess) return e;  // back in v0
  const int rows = rows_per_block(n, p.sh_degree);
  k_permute<<<dim3((unsigned)((n + rows - 1) / rows), 3), kRowBlock, 0, st>>>(rows_of(p, m, v, op, om, ov), n, rows, v0);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  if (perm_out) return hipMemcpyAsync(perm_out, v0, (size_t)n * 4, hipMemcpyDeviceToDevice, st);
  return hipSuccess;
}

}  // namespace gs_launch
