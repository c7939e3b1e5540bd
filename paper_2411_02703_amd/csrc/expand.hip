// Map expansion on the GPU (LVI-GS Sections III-A, III-C, III-E): a keyframe's colourised LiDAR points become new
// Gaussians.
//   1. Visibility filter (Sec. III-C, eq. Vp): a point is projected into the keyframe (the projection's FP32
//      operation order) and kept where the visibility rendered from the current map is still at most tau_alpha
//      (the map does not yet explain that pixel); points outside the image or behind the near plane are kept.
//   2. Voxel deduplication and density cap (Sec. III-A): points live in voxels of a fixed size; a point is
//      accepted while its voxel holds fewer than `cap` points, counting the map's Gaussians and this batch's
//      earlier points (input order).  The points' keys are sorted (the library's stable radix sort), so each point's
//      rank in its voxel comes from a binary search; the map's Gaussians find their voxel's run of points by another
//      and are counted there (only voxels that hold points matter).
//   3. Initialisation (Sec. III-E): mean = the point, log-scales = log sqrt of the mean squared distance to its 3
//      nearest accepted neighbours (>= 1e-7), identity rotation, opacity logit = inverse sigmoid of the initial
//      opacity, SH degree-0 coefficients from the colour, higher bands 0, Adam moments 0.  The neighbours come
//      from a uniform grid over the accepted points (sorted cell keys, ring search with an exact stopping rule:
//      after ring k every unvisited point is at least k cell sizes away), sixteen lanes a point; a point whose third
//      neighbour is not settled within kMaxRing rings is searched by brute force, a wave per point.
// Accepted points are appended after the n_old existing Gaussians in their input order.
#include <algorithm>

#include "common.h"

namespace {

constexpr uint64_t kInvalid = ~0ull;
constexpr int kBias = 1 << 20;  // voxel / cell coordinates are packed as 21-bit fields (|index| < 2^20)
constexpr int kMaxRing = 3;
constexpr float kY0 = 0.28209479177387814f;

__device__ __forceinline__ bool cell_of(float x, float y, float z, float inv, float size, int c[3]) {
  // floor(x / size) with the IEEE division (the comparison value is the same everywhere)
  const float q[3] = {x / size, y / size, z / size};
  (void)inv;
  for (int k = 0; k < 3; ++k) {
    const float f = floorf(q[k]);
    if (!(f > -(float)kBias && f < (float)kBias)) return false;
    c[k] = (int)f;
  }
  return true;
}

__device__ __forceinline__ uint64_t pack(const int c[3]) {
  return (uint64_t)(c[0] + kBias) | ((uint64_t)(c[1] + kBias) << 21) | ((uint64_t)(c[2] + kBias) << 42);
}

// First index in sorted keys[0, n) whose key is >= k.
__device__ __forceinline__ int64_t lower_bound(const uint64_t* __restrict__ keys, int64_t n, uint64_t k) {
  int64_t lo = 0, hi = n;
  while (lo < hi) {
    const int64_t mid = (lo + hi) >> 1;
    if (keys[mid] < k) lo = mid + 1; else hi = mid;
  }
  return lo;
}

struct ExpandCam {
  float R[9], T[3], fx, fy, cx, cy;
  int W, H;
};

// 1. visibility filter and voxel keys of the new points (kInvalid: filtered out or outside the key range)
__global__ void k_point_keys(const float* __restrict__ pts, int64_t M, ExpandCam c, const float* __restrict__ vis,
                             float tau, float near_z, float voxel, uint64_t* __restrict__ keys,
                             int32_t* __restrict__ vals) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= M) return;
  const float x = pts[3 * i], y = pts[3 * i + 1], z = pts[3 * i + 2];
  bool pass = true;
  float t[3];
  for (int r = 0; r < 3; ++r)
    t[r] = __builtin_fmaf(c.R[3 * r + 2], z, __builtin_fmaf(c.R[3 * r + 1], y, __builtin_fmaf(c.R[3 * r], x, c.T[r])));
  if (t[2] >= near_z) {
    const float u = __builtin_fmaf(c.fx, t[0] / t[2], c.cx), v = __builtin_fmaf(c.fy, t[1] / t[2], c.cy);
    if (u >= 0.f && u < (float)c.W && v >= 0.f && v < (float)c.H) pass = vis[(int64_t)(int)v * c.W + (int)u] <= tau;
  }
  int cc[3];
  keys[i] = pass && cell_of(x, y, z, 0.f, voxel, cc) ? pack(cc) : kInvalid;
  vals[i] = (int32_t)i;
}

// The map's Gaussians per point voxel, counted at the voxel's first sorted point.  Latency-bound: a binary search over
// the points' keys per Gaussian (they fit the L2), kTop levels of it in LDS.  (Sorting the keys of 1M Gaussians instead
// took 24 launches and 350 us.)  Counts stop at the cap, beyond which they change nothing, and a wave whose lanes share
// a voxel adds once, so that a crowded voxel does not become a queue of atomics.
constexpr int kTop = 1024;

__global__ __launch_bounds__(256) void k_map_count(const float* __restrict__ means, int64_t N, float voxel,
                                                   const uint64_t* __restrict__ pk, int M, int cap,
                                                   int32_t* __restrict__ have) {
  __shared__ uint64_t top[kTop];  // top[i] = the last key of the i-th of kTop stretches of `step` keys
  const int step = (M + kTop - 1) / kTop;
  for (int i = threadIdx.x; i < kTop; i += 256) {
    const int64_t e = (int64_t)(i + 1) * step - 1;
    top[i] = e < M ? pk[e] : kInvalid;
  }
  __syncthreads();
  for (int64_t j = (int64_t)blockIdx.x * 256 + threadIdx.x; j < N; j += (int64_t)gridDim.x * 256) {
    int cc[3], at = -1;
    if (cell_of(means[3 * j], means[3 * j + 1], means[3 * j + 2], 0.f, voxel, cc)) {
      const uint64_t k = pack(cc);
      int b = 0;  // the first stretch whose last key is >= k (valid keys are below kInvalid)
      for (int h = kTop / 2; h >= 1; h >>= 1) b += top[b + h - 1] < k ? h : 0;
      int lo = min(b * step, M), hi = min(lo + step, M);
      while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if (pk[mid] < k) lo = mid + 1; else hi = mid;
      }
      if (lo < M && pk[lo] == k && have[lo] < cap) at = lo;
    }
    const uint64_t need = __ballot(at >= 0);
    if (need) {
      const int lead = __builtin_ctzll(need), first = __shfl(at, lead);
      const uint64_t same = __ballot(at == first);
      if (at == first) {
        if ((int)__lane_id() == lead) atomicAdd(have + at, (int)__popcll(same));
      } else if (at >= 0) {
        atomicAdd(have + at, 1);
      }
    }
  }
}

// 2. acceptance: rank of the point in its voxel (sorted, stable) plus the map's count there, against the cap
__global__ void k_accept(const uint64_t* __restrict__ pk, const int32_t* __restrict__ pv, int64_t M,
                         const int32_t* __restrict__ have, int cap, int32_t* __restrict__ accept) {
  const int64_t s = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (s >= M) return;
  const uint64_t k = pk[s];
  int ok = 0;
  if (k != kInvalid) {
    const int64_t first = lower_bound(pk, s, k);
    ok = have[first] + (s - first) < cap;
  }
  accept[pv[s]] = ok;
}

// 3a. grid cell keys of the accepted points, compacted to their output order, and their number
__global__ void k_cell_keys(const float* __restrict__ pts, const int32_t* __restrict__ accept,
                            const int32_t* __restrict__ off, int64_t M, float cell, uint64_t* __restrict__ keys,
                            int32_t* __restrict__ vals, int32_t* __restrict__ count, int64_t* __restrict__ n_added) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i == M - 1) {
    count[0] = off[i] + accept[i];
    n_added[0] = count[0];
  }
  if (i >= M || !accept[i]) return;
  int cc[3];
  const bool ok = cell_of(pts[3 * i], pts[3 * i + 1], pts[3 * i + 2], 0.f, cell, cc);
  keys[off[i]] = ok ? pack(cc) : kInvalid;
  vals[off[i]] = (int32_t)i;
}

__device__ __forceinline__ void push3(float d, float b[3]) {
  if (d < b[2]) {
    b[2] = d;
    if (b[2] < b[1]) { const float t = b[1]; b[1] = b[2]; b[2] = t; }
    if (b[1] < b[0]) { const float t = b[0]; b[0] = b[1]; b[1] = t; }
  }
}

__device__ __forceinline__ float spacing_log_scale(const float b[3]) {
  int found = 0;
  float sum = 0.f;
  for (int k = 0; k < 3; ++k)
    if (b[k] < INFINITY) { sum += b[k]; ++found; }
  const float d2 = fmaxf(found ? sum / (float)found : 0.f, 1e-7f);
  return 0.5f * logf(d2);
}

// The sorted accepted points' positions, so that a cell's points are read in one run.
__global__ void k_sorted_points(const float* __restrict__ pts, const int32_t* __restrict__ cv,
                                const int32_t* __restrict__ count, float4* __restrict__ sp) {
  const int64_t s = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (s >= count[0]) return;
  const int64_t i = cv[s];
  sp[s] = make_float4(pts[3 * i], pts[3 * i + 1], pts[3 * i + 2], __int_as_float((int)i));
}

// The smallest three of `lanes` (a power of two) neighbouring lanes' sorted triples, in every one of them: three rounds
// of a minimum, whose lowest holder drops it.
template <int LANES>
__device__ __forceinline__ void merge3(float b[3]) {
  float best[3];
  const int lane = __lane_id();
  const uint64_t group = LANES == 64 ? ~0ull : ((1ull << (LANES & 63)) - 1) << (lane & ~(LANES - 1));
  for (int r = 0; r < 3; ++r) {
    float m = b[0];
    for (int sh = LANES / 2; sh >= 1; sh >>= 1) m = fminf(m, __shfl_xor(m, sh));
    best[r] = m;
    const uint64_t hold = __ballot(b[0] == m && m < INFINITY) & group;
    if (hold && lane == __builtin_ctzll(hold)) {
      b[0] = b[1];
      b[1] = b[2];
      b[2] = INFINITY;
    }
  }
  for (int k = 0; k < 3; ++k) b[k] = best[k];
}

// 3b. ring search over the sorted cells; the log-scale goes to the new Gaussian's row, unsettled points to a list.
// Latency-bound: kKnnLanes lanes share a point, each taking rows of cells along x, which are one run of the sorted keys
// (x is the key's lowest field): one binary search a row, where a search per cell, all by one thread, took 765 us for
// 100k points.  Rings 0 and 1 go together (ring 0 settles only a point with three copies, which ring 1 cannot change);
// in a later ring the rows inside the ring before are left with their two end cells.
constexpr int kKnnLanes = 16;

__device__ __forceinline__ void search_run(const float4* __restrict__ sp, const uint64_t* __restrict__ ck, int64_t A,
                                           uint64_t from, uint64_t to, int64_t s, float4 p, float b[3]) {
  for (int64_t j = lower_bound(ck, A, from); j < A && ck[j] <= to; ++j) {
    if (j == s) continue;
    const float4 q = sp[j];
    const float ex = q.x - p.x, ey = q.y - p.y, ez = q.z - p.z;
    push3(ex * ex + ey * ey + ez * ez, b);
  }
}

__global__ __launch_bounds__(256) void k_knn(const float4* __restrict__ sp, const uint64_t* __restrict__ ck,
                                             const int32_t* __restrict__ count, float cell,
                                             const int32_t* __restrict__ off, float* __restrict__ out_ls,
                                             int32_t* __restrict__ brute, int32_t* __restrict__ n_brute) {
  const int64_t A = count[0];
  const int64_t s = (((int64_t)blockIdx.y * gridDim.x + blockIdx.x) * blockDim.x + threadIdx.x) / kKnnLanes;
  const int sub = threadIdx.x % kKnnLanes;
  if (s >= A) return;  // (the whole group)
  const float4 p = sp[s];
  int c0[3];
  const bool in_range = cell_of(p.x, p.y, p.z, 0.f, cell, c0);
  float b[3] = {INFINITY, INFINITY, INFINITY};
  for (int ring = 1; in_range && ring <= kMaxRing; ++ring) {
    const int side = 2 * ring + 1;
    const int x0 = max(c0[0] - ring, 1 - kBias), x1 = min(c0[0] + ring, kBias - 1);
    float mine[3] = {INFINITY, INFINITY, INFINITY};
    for (int row = sub; row < side * side; row += kKnnLanes) {
      const int dy = row % side - ring, dz = row / side - ring;
      const int y = c0[1] + dy, z = c0[2] + dz;
      if (abs(y) >= kBias || abs(z) >= kBias) continue;
      const int l[3] = {x0, y, z}, h[3] = {x1, y, z};
      if (ring == 1 || max(abs(dy), abs(dz)) == ring) {
        search_run(sp, ck, A, pack(l), pack(h), s, p, mine);
      } else {  // the ends only, where they are in the key range
        if (c0[0] - ring == x0) search_run(sp, ck, A, pack(l), pack(l), s, p, mine);
        if (c0[0] + ring == x1) search_run(sp, ck, A, pack(h), pack(h), s, p, mine);
      }
    }
    merge3<kKnnLanes>(mine);
    for (int k = 0; k < 3; ++k) push3(mine[k], b);
    const float reach = (float)ring * cell;
    if (b[2] <= reach * reach) {
      if (sub < 3) out_ls[3 * (int64_t)off[__float_as_int(p.w)] + sub] = spacing_log_scale(b);
      return;
    }
  }
  if (sub == 0) brute[atomicAdd(n_brute, 1)] = (int)s;
}

// 3c. brute force for the unsettled points: a wave per point over every accepted point, then a wave reduction
__global__ __launch_bounds__(256) void k_knn_brute(const float4* __restrict__ sp, const int32_t* __restrict__ count,
                                                   const int32_t* __restrict__ brute,
                                                   const int32_t* __restrict__ n_brute,
                                                   const int32_t* __restrict__ off, float* __restrict__ out_ls) {
  const int64_t A = count[0];
  const int lane = threadIdx.x & 63;
  const int64_t wave = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6;
  const int64_t n_waves = ((int64_t)gridDim.x * blockDim.x) >> 6;
  for (int64_t w = wave; w < n_brute[0]; w += n_waves) {
    const int64_t s = brute[w];
    const float4 p = sp[s];
    float b[3] = {INFINITY, INFINITY, INFINITY};
#pragma unroll 4
    for (int64_t j = lane; j < A; j += 64) {
      const float4 q = sp[j];
      const float ex = q.x - p.x, ey = q.y - p.y, ez = q.z - p.z;
      push3(j == s ? INFINITY : ex * ex + ey * ey + ez * ez, b);
    }
    merge3<64>(b);
    if (lane == 0) {
      const float ls = spacing_log_scale(b);
      float* o = out_ls + 3 * (int64_t)off[__float_as_int(p.w)];
      o[0] = o[1] = o[2] = ls;
    }
  }
}

// 3d. the other parameters and zero moments of every new Gaussian
struct NewRows {
  float* means; float* quats; float* opac; float* sh;
  float* m[5]; float* v[5];  // means, log_scales, quats, opacity, sh of the moments
};

// Rows [0, m) of an array from row g0 on are zeroed, or set by f(row, element); contiguous over the block.
template <class F>
__device__ __forceinline__ void write_rows(float* __restrict__ a, int64_t g0, int m, int len, F f) {
  a += g0 * len;
  for (int e = threadIdx.x; e < m * len; e += 256) a[e] = f(e / len, e % len);
}

// A block's accepted points fill consecutive rows; it writes them array by array (a thread per point writing its own
// rows made every store a line of its own).  blockIdx.y: parameters, first and second moments.
__global__ __launch_bounds__(256) void k_expand_write(const float* __restrict__ pts, const float* __restrict__ rgb,
                                                      const int32_t* __restrict__ accept,
                                                      const int32_t* __restrict__ off, int64_t M, int64_t n_old, int K3,
                                                      float logit, NewRows r) {
  __shared__ int32_t src[256];
  const int64_t i0 = (int64_t)blockIdx.x * 256, i = i0 + threadIdx.x, last = min(i0 + 256, M) - 1;
  const int32_t first = off[i0];
  const int m = off[last] + accept[last] - first;
  const int64_t g0 = n_old + first;
  if (blockIdx.y) {
    float* const* d = blockIdx.y == 1 ? r.m : r.v;
    const auto zero = [](int, int) { return 0.f; };
    write_rows(d[0], g0, m, 3, zero);
    write_rows(d[1], g0, m, 3, zero);
    write_rows(d[2], g0, m, 4, zero);
    write_rows(d[3], g0, m, 1, zero);
    write_rows(d[4], g0, m, K3, zero);
    return;
  }
  if (i < M && accept[i]) src[off[i] - first] = (int32_t)i;
  __syncthreads();
  write_rows(r.means, g0, m, 3, [&](int p, int k) { return pts[3 * (int64_t)src[p] + k]; });
  write_rows(r.quats, g0, m, 4, [](int, int k) { return k == 0 ? 1.f : 0.f; });
  write_rows(r.opac, g0, m, 1, [&](int, int) { return logit; });
  write_rows(r.sh, g0, m, K3, [&](int p, int k) { return k < 3 ? (rgb[3 * (int64_t)src[p] + k] - 0.5f) / kY0 : 0.f; });
}

}  // namespace

namespace gs_launch {

// Scratch layout (int32 units, 64-aligned pieces): point keys/vals x2, sorted positions, accept, off, brute list (before
// it the map's counts per voxel), counters, sort scratch (reused by the two sorts), scan scratch.
struct ExpandLayout {
  size_t pk0, pk1, pv0, pv1, sp, acc, off, brute, cnt, sort, scan, total;
};

static size_t a64(size_t x) { return (x + 63) / 64 * 64; }

static ExpandLayout expand_layout(int64_t M) {
  ExpandLayout L;
  size_t o = 0;
  const size_t m2 = a64(2 * (size_t)M);
  L.pk0 = o; o += m2; L.pk1 = o; o += m2; L.pv0 = o; o += a64(M); L.pv1 = o; o += a64(M);
  L.sp = o; o += a64(4 * (size_t)M + 4);  // (room to start at a multiple of 16 bytes)
  L.acc = o; o += a64(M); L.off = o; o += a64(M); L.brute = o; o += a64(M); L.cnt = o; o += 64;
  L.sort = o; o += a64(sort_scratch_ints(M > 0 ? M : 1));
  L.scan = o; o += a64(scan_scratch_ints(M > 0 ? M : 1));
  L.total = o;
  return L;
}

size_t expand_scratch_ints(int64_t M) { return expand_layout(M).total; }

hipError_t expand(const gs_params& p, const gs_params& m, const gs_params& v, int64_t n_old, const float* pts,
                  const float* rgb, int64_t M, const gs_camera& cam, const float* vis, float tau, float near_z,
                  float voxel, int cap, float cell, float init_logit, int64_t* n_added, int32_t* scratch,
                  hipStream_t st) {
  const ExpandLayout L = expand_layout(M);
  auto u64 = [&](size_t o) { return reinterpret_cast<uint64_t*>(scratch + o); };
  int32_t* cnt = scratch + L.cnt;
  hipError_t e = fill_i32(cnt, 0, 64, st);
  if (e != hipSuccess) return e;
  ExpandCam c;
  for (int k = 0; k < 9; ++k) c.R[k] = cam.R[k];
  for (int k = 0; k < 3; ++k) c.T[k] = cam.T[k];
  c.fx = cam.fx; c.fy = cam.fy; c.cx = cam.cx; c.cy = cam.cy; c.W = cam.width; c.H = cam.height;
  const unsigned bm = (unsigned)((M + 255) / 256);
  int32_t* have = scratch + L.brute;
  if ((e = fill_i32(have, 0, M, st)) != hipSuccess) return e;
  // 1. filter + voxel keys, sorted (stable: input order inside a voxel)
  k_point_keys<<<bm, 256, 0, st>>>(pts, M, c, vis, tau, near_z, voxel, u64(L.pk0), scratch + L.pv0);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  if ((e = sort_pairs(u64(L.pk0), scratch + L.pv0, u64(L.pk1), scratch + L.pv1, M, nullptr, M, 64,
                      scratch + L.sort, st)) != hipSuccess)
    return e;  // 8 passes: the sorted pairs are back in the first buffers
  if (n_old > 0) {
    const int64_t bn = (n_old + 255) / 256;
    k_map_count<<<(unsigned)(bn < 2048 ? bn : 2048), 256, 0, st>>>(p.means, n_old, voxel, u64(L.pk0), (int)M, cap, have);
    if ((e = hipGetLastError()) != hipSuccess) return e;
  }
  // 2. acceptance, and the output order
  k_accept<<<bm, 256, 0, st>>>(u64(L.pk0), scratch + L.pv0, M, have, cap, scratch + L.acc);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  if ((e = scan_exclusive(scratch + L.acc, scratch + L.off, M, scratch + L.scan, st)) != hipSuccess) return e;
  // 3. cells of the accepted points (sorted, sized by M, counted on the device), spacing, the new rows
  k_cell_keys<<<bm, 256, 0, st>>>(pts, scratch + L.acc, scratch + L.off, M, cell, u64(L.pk1), scratch + L.pv1, cnt,
                                  n_added);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  if ((e = sort_pairs(u64(L.pk1), scratch + L.pv1, u64(L.pk0), scratch + L.pv0, M, cnt, M, 64, scratch + L.sort,
                      st)) != hipSuccess)
    return e;
  float* ls_new = p.log_scales + 3 * n_old;
  auto* sp = reinterpret_cast<float4*>((reinterpret_cast<uintptr_t>(scratch + L.sp) + 15) & ~(uintptr_t)15);
  k_sorted_points<<<bm, 256, 0, st>>>(pts, scratch + L.pv1, cnt, sp);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  // (a dimension of a grid has less than 2^32 threads; 2^28 points take more)
  const int64_t bk = (M * kKnnLanes + 255) / 256, bx = std::min<int64_t>(bk, 1 << 23);
  k_knn<<<dim3((unsigned)bx, (unsigned)((bk + bx - 1) / bx)), 256, 0, st>>>(sp, u64(L.pk1), cnt, cell, scratch + L.off,
                                                                            ls_new, scratch + L.brute, cnt + 1);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  k_knn_brute<<<256, 256, 0, st>>>(sp, cnt, scratch + L.brute, cnt + 1, scratch + L.off, ls_new);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  NewRows r;
  r.means = p.means; r.quats = p.quats; r.opac = p.opacity; r.sh = p.sh;
  const gs_params* mv[2] = {&m, &v};
  for (int k = 0; k < 2; ++k) {
    float** d = k == 0 ? r.m : r.v;
    d[0] = mv[k]->means; d[1] = mv[k]->log_scales; d[2] = mv[k]->quats; d[3] = mv[k]->opacity; d[4] = mv[k]->sh;
  }
  const int K3 = 3 * (p.sh_degree + 1) * (p.sh_degree + 1);
  k_expand_write<<<dim3(bm, 3), 256, 0, st>>>(pts, rgb, scratch + L.acc, scratch + L.off, M, n_old, K3, init_logit, r);
  return hipGetLastError();
}

}  // namespace gs_launch
