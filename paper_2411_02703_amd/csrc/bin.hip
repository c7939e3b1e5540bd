// Tile binning (integer work, bit-exact by construction).  The order inside a tile is ascending depth bits, ties
// by record index, so the sorted order is unique.  Two stable LSD radix sorts (8-bit digits) reach it:
//   1. the visible records, listed wave by wave and view by view (Gaussians ascending inside a view), are sorted
//      by their 32-bit depth bits (4 passes over the records, not the instances);
//   2. the records are emitted in that order, each as its run of tile instances (key = global tile id, value =
//      record id), and the instances are sorted by tile (2 passes at up to 65,536 tiles).
// A stable sort by tile of a depth-ordered sequence is the (tile, depth, record) order; ties in depth keep
// ascending Gaussian index inside a view (the records of one view are listed in Gaussian order), and records
// of different views never share a tile.  The sorted value of an instance is its record id.
//
// The compositing backward stores each instance's partial derivatives at a slot of its own, laid out Gaussian by
// Gaussian (the exclusive scan of the per-Gaussian instance counts), views ascending inside a Gaussian, a
// record's tiles row by row: each record's first slot is written here, in Gaussian order, so that the projection
// backward reads one contiguous run per Gaussian.
#include "common.h"
#include "chain.h"

namespace {

constexpr int kScanThreads = 256;
constexpr int kScanItems = 16;
constexpr int kScanTile = kScanThreads * kScanItems;  // 4096

// Exclusive scan of 256 values, one per thread; returns the exclusive prefix, *total = sum.
__device__ __forceinline__ int block_scan_256(int x, int* sh_wave, int* total) {
  const int lane = __lane_id(), wave = threadIdx.x >> 6;
  int incl = x;
  for (int d = 1; d < 64; d <<= 1) {
    const int y = __shfl_up(incl, d);
    if (lane >= d) incl += y;
  }
  if (lane == 63) sh_wave[wave] = incl;
  __syncthreads();
  int base = 0;
  for (int w = 0; w < wave; ++w) base += sh_wave[w];
  *total = sh_wave[0] + sh_wave[1] + sh_wave[2] + sh_wave[3];
  __syncthreads();
  return base + incl - x;
}

// Each block scans kScanTile consecutive items (exclusive) and writes its total.
__global__ __launch_bounds__(kScanThreads) void k_scan_tile(const int32_t* in, int32_t* out, int64_t n,
                                                            int32_t* sums) {
  __shared__ int sh_wave[4];
  const int64_t base = (int64_t)blockIdx.x * kScanTile + (int64_t)threadIdx.x * kScanItems;
  // a thread's 16 items as four 16-byte loads and stores when they are all in range and the arrays are aligned
  const bool vec = base + kScanItems <= n &&
                   ((reinterpret_cast<uintptr_t>(in) | reinterpret_cast<uintptr_t>(out)) & 15) == 0;
  int v[kScanItems];
  if (vec) {
    const int4* p = reinterpret_cast<const int4*>(in + base);
#pragma unroll
    for (int q = 0; q < kScanItems / 4; ++q) {
      const int4 x = p[q];
      v[4 * q] = x.x;
      v[4 * q + 1] = x.y;
      v[4 * q + 2] = x.z;
      v[4 * q + 3] = x.w;
    }
  } else {
#pragma unroll
    for (int i = 0; i < kScanItems; ++i) {
      const int64_t idx = base + i;
      v[i] = idx < n ? in[idx] : 0;
    }
  }
  int acc = 0;
#pragma unroll
  for (int i = 0; i < kScanItems; ++i) acc += v[i];
  int total;
  int run = block_scan_256(acc, sh_wave, &total);
  int o[kScanItems];
#pragma unroll
  for (int i = 0; i < kScanItems; ++i) {
    o[i] = run;
    run += v[i];
  }
  if (vec) {
    int4* p = reinterpret_cast<int4*>(out + base);
#pragma unroll
    for (int q = 0; q < kScanItems / 4; ++q) p[q] = make_int4(o[4 * q], o[4 * q + 1], o[4 * q + 2], o[4 * q + 3]);
  } else {
#pragma unroll
    for (int i = 0; i < kScanItems; ++i) {
      const int64_t idx = base + i;
      if (idx < n) out[idx] = o[i];
    }
  }
  if (threadIdx.x == 0) sums[blockIdx.x] = total;
}

__global__ __launch_bounds__(kScanThreads) void k_scan_add(int32_t* out, int64_t n, const int32_t* sums) {
  const int64_t base = (int64_t)blockIdx.x * kScanTile;
  const int add = sums[blockIdx.x];
  for (int i = threadIdx.x; i < kScanTile; i += kScanThreads) {
    const int64_t idx = base + i;
    if (idx < n) out[idx] += add;
  }
}

__global__ void k_fill_i32(int32_t* __restrict__ p, int32_t v, int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = v;
}
// Two int32 ranges set to v in one launch: [p, p + n) and [q, q + m).
__global__ void k_fill2_i32(int32_t* __restrict__ p, int64_t n, int32_t* __restrict__ q, int64_t m, int32_t v) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = v;
  if (i < m) q[i] = v;
}
__global__ void k_fill_f32(float* __restrict__ p, float v, int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = v;
}

__device__ __forceinline__ int64_t sort_count(const int32_t* count_dev, int64_t n_sized, int64_t cap) {
  if (count_dev == nullptr) return n_sized;
  const int64_t c = count_dev[0];
  return c < cap ? c : cap;
}

// Radix sort, one launch per 8-bit digit: k_sort_digits counts every digit of every key in one read; each pass then
// finds its blocks' positions by a chained scan (a block publishes its digit counts, adds up those of the blocks before
// it and publishes the sums).  With a histogram pass and a scan pass per digit in place of the chain, which cost two
// launches and a read of the keys each, the six passes of a keyframe step (0.75 M records, 1.5 M instances) took 234 us
// and those of a 24-view step (3.3 M and 21.6 M) 730; now 180 and 491, 21 and 67 of them for the digits.
//
// Words of a sort that must be zero before its first launch: digit counts and a ticket per pass.  The counts are kept
// in kCopies copies, since the blocks' adds to one cache line queue (about 5 ns each).
constexpr int kCopies = 8;
constexpr int kSortZero32 = kCopies * 4 * 256 + 64, kSortZero64 = kCopies * 8 * 256 + 64;

using gsk::kWhole;  // (chain.h describes the states)
__device__ __forceinline__ void put_state(uint32_t* p, uint32_t v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ uint32_t get_state(const uint32_t* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

constexpr int kDigitThreads = 256;
constexpr int kDigitItems = 8;
constexpr int kDigitBlocks = 1024;

// Keys per tile of the passes, by the number of keys (known on the device only).  Small sorts want many short blocks,
// large ones long runs in the output and few states: with 2048 and 8192 keys a tile a pass of 2 k keys takes 5.2 and
// 9.7 us, of 100 k 64-bit keys 7.3 and 11.9, of 270 k 22.8 and 21.3, of 0.75 M 39 and 30, of 1.5 M 52 and 40.  64-bit keys
// have 4096 a tile as long as that is at most a tile per CU (256): eight passes over 530 k, 1 M and 1.5 M take 126, 155 and
// 209 us with 4096 and 147, 168 and 181 with 8192 (156, 173 and 200 with a histogram and a scan per digit, which two passes
// over 1.5 M still do as fast: 49 against 51).  32-bit ones gain nothing: a keyframe step 1576 us with 8192, 1582 with 4096.
constexpr int kSortThreads = 1024;
constexpr int kSmallItems = 2, kMidItems = 4, kLargeItems = 8;
constexpr int64_t kSmallSort = int64_t(1) << 19, kMidSort = int64_t(1) << 20;
template <class KeyT>
__host__ __device__ inline int sort_tile(int64_t n) {
  const bool mid = sizeof(KeyT) == 8 && n <= kMidSort;
  return kSortThreads * (n <= kSmallSort ? kSmallItems : mid ? kMidItems : kLargeItems);
}

// (The first pass's states are cleared here.)
template <class KeyT>
__global__ __launch_bounds__(kDigitThreads) void k_sort_digits(const KeyT* __restrict__ keys,
                                                               const int32_t* __restrict__ count_dev, int64_t n_sized,
                                                               int64_t cap, int passes,
                                                               int32_t* __restrict__ digits,
                                                               uint32_t* __restrict__ state) {
  __shared__ int h[(int)sizeof(KeyT)][256];
  const int64_t n = sort_count(count_dev, n_sized, cap);
  const int tile = sort_tile<KeyT>(n);
  const int64_t words = (n + tile - 1) / tile * 256;
  for (int64_t i = (int64_t)blockIdx.x * kDigitThreads + threadIdx.x; i < words; i += (int64_t)gridDim.x * kDigitThreads)
    state[i] = 0;
  constexpr int kStep = kDigitThreads * kDigitItems;
  if ((int64_t)blockIdx.x * kStep >= n) return;
  for (int p = 0; p < passes; ++p) h[p][threadIdx.x] = 0;
  __syncthreads();
  for (int64_t base = (int64_t)blockIdx.x * kStep; base < n; base += (int64_t)gridDim.x * kStep) {
    KeyT key[kDigitItems];
#pragma unroll
    for (int i = 0; i < kDigitItems; ++i) {
      const int64_t idx = base + i * kDigitThreads + threadIdx.x;
      key[i] = idx < n ? keys[idx] : KeyT(0);
    }
#pragma unroll
    for (int i = 0; i < kDigitItems; ++i) {
      const bool valid = base + i * kDigitThreads + threadIdx.x < n;
      const uint64_t vb = __ballot(valid);
      if (vb == 0) break;
      const int lead = __builtin_ctzll(vb);
      for (int p = 0; p < passes; ++p) {
        // the first lane's digit is counted once for the wave: high digits agree in most lanes, and adds of many
        // lanes to one address are taken one by one
        const int d = (int)((key[i] >> (8 * p)) & 255u);
        const int d0 = __builtin_amdgcn_readlane(d, lead);
        const uint64_t same = __ballot(valid && d == d0);
        if (valid && d != d0) atomicAdd(&h[p][d], 1);
        if ((int)__lane_id() == lead) atomicAdd(&h[p][d0], (int)__popcll(same));
      }
    }
  }
  __syncthreads();
  for (int p = 0; p < passes; ++p) {
    const int c = h[p][threadIdx.x];
    if (c) atomicAdd(digits + 256 * ((blockIdx.x % kCopies) * passes + p) + threadIdx.x, c);
  }
}

// Stable scatter of one 8-bit digit.  Tiles are taken in the order of a ticket counter, so that every tile before a
// running block's belongs to a block that runs or has finished: the waits below end, because a block publishes its own
// counts before it waits (and where another sort meddles, after kChainLooks looks, with every place in range).  Each wave ranks its keys (ITEMS rounds of 64) with ballot-based digit matching, the block
// orders them in LDS (digit-major, stable), adds up the earlier tiles' counts (a digit per thread, kLook tiles' words in
// flight) and writes runs to their global places, first keys, then values through the same LDS.  state: this pass's
// states, cleared before; next: the following pass's, cleared here.
constexpr int kLook = 8;

template <class KeyT>
struct SortStage {
  KeyT key[kSortThreads * kLargeItems];
  uint16_t cnt[kSortThreads / 64][256];
  int32_t ofs[256];
  int wave[2][4];
  int tile;
};

// The wave's keys (ITEMS rounds of 64 from i0, valid below nvalid) ranked among its keys of the same digit, by ballots;
// cnt (zero before) ends as the wave's count of each digit.
template <int ITEMS, class KeyT>
__device__ __forceinline__ void rank_digit(const KeyT* key, int i0, int nvalid, int shift, uint16_t* cnt, int* pos) {
  const uint64_t lt = gsk::lanemask_lt();
#pragma unroll
  for (int k = 0; k < ITEMS; ++k) {
    const bool valid = i0 + k * 64 < nvalid;
    const int d = (int)((key[k] >> shift) & 255u);
    uint64_t peers = __ballot(valid);
#pragma unroll
    for (int b = 0; b < 8; ++b) {
      const bool bit = (d >> b) & 1;
      const uint64_t bb = __ballot(bit);
      peers &= bit ? bb : ~bb;
    }
    const int rank = __popcll(peers & lt);
    int before = 0;
    if (valid) before = cnt[d];
    pos[k] = before + rank;
    __builtin_amdgcn_wave_barrier();
    if (valid && rank == 0) cnt[d] = (uint16_t)(before + __popcll(peers));
    __builtin_amdgcn_wave_barrier();
  }
}

template <class KeyT, int ITEMS>
__device__ __forceinline__ void scatter_tile(SortStage<KeyT>& s, const KeyT* __restrict__ kin,
                                             const int32_t* __restrict__ vin, KeyT* __restrict__ kout,
                                             int32_t* __restrict__ vout, int64_t n, int pass, int dc, uint32_t* state,
                                             uint32_t* next) {
  constexpr int THREADS = kSortThreads, TILE = THREADS * ITEMS, WAVES = THREADS / 64;
  KeyT* sk = s.key;
  int32_t* sv = reinterpret_cast<int32_t*>(s.key);
  auto& wcnt = s.cnt;
  auto& gofs = s.ofs;
  auto& sh_wave = s.wave;
  const int tid = threadIdx.x, wave = tid >> 6, lane = __lane_id(), shift = 8 * pass;
  const int tile = s.tile;
  const int64_t base = (int64_t)tile * TILE;
  const int nvalid = (int)min((int64_t)TILE, n - base);
  kin += base;
  vin += base;
  const int i0 = wave * 64 * ITEMS + lane;
  KeyT key[ITEMS];
  int pos[ITEMS];
#pragma unroll
  for (int k = 0; k < ITEMS; ++k) {
    const bool valid = i0 + k * 64 < nvalid;
    key[k] = valid ? kin[i0 + k * 64] : KeyT(0);
  }
  rank_digit<ITEMS>(key, i0, nvalid, shift, wcnt[wave], pos);
  __syncthreads();
  // digit tid: the tile's count is published, the waves' first places in the tile and the digit's first place overall
  uint32_t* my_state = state + (int64_t)tile * 256 + tid;
  int total = 0, in_c = 0, in_d = 0;
  if (tid < 256) {
#pragma unroll
    for (int w = 0; w < WAVES; ++w) total += wcnt[w][tid];
    put_state(my_state, tile == 0 ? kWhole | (uint32_t)total : (uint32_t)total + 1u);
    next[(int64_t)tile * 256 + tid] = 0;
    int t;
    in_c = gsk::wave_excl_scan(total, t);
    if (lane == 0) sh_wave[0][wave] = t;
    in_d = gsk::wave_excl_scan(dc, t);
    if (lane == 0) sh_wave[1][wave] = t;
  }
  __syncthreads();
  if (tid < 256) {
    for (int w = 0; w < wave; ++w) {
      in_c += sh_wave[0][w];
      in_d += sh_wave[1][w];
    }
    int run = in_c;
#pragma unroll
    for (int w = 0; w < WAVES; ++w) {
      const int c = wcnt[w][tid];
      wcnt[w][tid] = (uint16_t)run;
      run += c;
    }
  }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < ITEMS; ++k) {
    if (i0 + k * 64 < nvalid) {
      pos[k] += wcnt[wave][(int)((key[k] >> shift) & 255u)];
      sk[pos[k]] = key[k];
    }
  }
  int32_t val[ITEMS];  // (here, so that the loads' time passes in the waits below)
#pragma unroll
  for (int k = 0; k < ITEMS; ++k) val[k] = i0 + k * 64 < nvalid ? vin[i0 + k * 64] : 0;
  if (tid < 256) {
    uint32_t before = 0;
    if (tile > 0) {
      before = gsk::keys_before<kLook>(tile, gsk::kChainLooks,
                                       [&](int j) { return get_state(state + (int64_t)j * 256 + tid); });
      put_state(my_state, kWhole | (before + (uint32_t)total));
    }
    gofs[tid] = in_d + (int)before - in_c;
  }
  __syncthreads();
  int out[ITEMS];
#pragma unroll
  for (int k = 0; k < ITEMS; ++k) {
    const int p = k * THREADS + tid;
    if (p < nvalid) {
      const KeyT kk = sk[p];
      out[k] = (int)gsk::key_place((uint32_t)gofs[(int)((kk >> shift) & 255u)], p, (uint32_t)n);
      kout[out[k]] = kk;
    }
  }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < ITEMS; ++k)
    if (i0 + k * 64 < nvalid) sv[pos[k]] = val[k];
  __syncthreads();
#pragma unroll
  for (int k = 0; k < ITEMS; ++k) {
    const int p = k * THREADS + tid;
    if (p < nvalid) vout[out[k]] = sv[p];
  }
}

template <class KeyT>
__global__ __launch_bounds__(kSortThreads, sizeof(KeyT) == 4 ? 8 : 4) void k_sort_scatter(
    const KeyT* __restrict__ kin, const int32_t* __restrict__ vin, KeyT* __restrict__ kout, int32_t* __restrict__ vout,
    const int32_t* __restrict__ count_dev, int64_t n_sized, int64_t cap, int pass, int passes, int32_t* digits,
    uint32_t* state, uint32_t* next) {
  __shared__ SortStage<KeyT> s;
  const int64_t n = sort_count(count_dev, n_sized, cap);
  if ((int64_t)blockIdx.x * sort_tile<KeyT>(n) >= n) return;  // (as many blocks as tiles go on)
  const int tid = threadIdx.x;
  if (tid == 0) {  // (the minimum: where another sort meddles with the tickets, the tile is one of this sort's all the same)
    const uint32_t ticket = (uint32_t)atomicAdd(digits + kCopies * 256 * passes + pass, 1);
    s.tile = (int)min(ticket, (uint32_t)((n - 1) / sort_tile<KeyT>(n)));
  }
  for (int i = tid; i < kSortThreads / 64 * 256; i += kSortThreads) (&s.cnt[0][0])[i] = 0;
  int dc = 0;  // the digit's keys
  if (tid < 256) {
#pragma unroll
    for (int i = 0; i < kCopies; ++i) dc += digits[256 * (i * passes + pass) + tid];
  }
  __syncthreads();
  if (n <= kSmallSort)
    scatter_tile<KeyT, kSmallItems>(s, kin, vin, kout, vout, n, pass, dc, state, next);
  else if (sizeof(KeyT) == 8 && n <= kMidSort)
    scatter_tile<KeyT, kMidItems>(s, kin, vin, kout, vout, n, pass, dc, state, next);
  else
    scatter_tile<KeyT, kLargeItems>(s, kin, vin, kout, vout, n, pass, dc, state, next);
}

// A sort of at most kBlockSort keys: every pass in one block, through its LDS, where the launches of a kernel per pass were
// the cost.  Four passes over 300 keys take 17 us here and 31 in launches of their own, over 2000 21 and 35, over 6000 39
// and 41, over 8192 41 and 41 (and a capacity is seldom full).  Input and output may be the same arrays.
constexpr int kBlockSort = kSortThreads * kLargeItems;

template <class KeyT>
struct BlockStage {
  KeyT key[kBlockSort];
  int32_t val[kBlockSort];
  uint16_t cnt[kSortThreads / 64][256];
  int wave[4];
};

template <class KeyT, int ITEMS>
__device__ __forceinline__ void sort_block(BlockStage<KeyT>& s, const KeyT* kin, const int32_t* vin, KeyT* kout,
                                           int32_t* vout, int n, int passes) {
  constexpr int WAVES = kSortThreads / 64;
  const int tid = threadIdx.x, wave = tid >> 6, i0 = wave * 64 * ITEMS + __lane_id();
  KeyT key[ITEMS];
  int32_t val[ITEMS];
  int pos[ITEMS];
#pragma unroll
  for (int k = 0; k < ITEMS; ++k) {
    const bool valid = i0 + k * 64 < n;
    key[k] = valid ? kin[i0 + k * 64] : KeyT(0);
    val[k] = valid ? vin[i0 + k * 64] : 0;
  }
  for (int p = 0; p < passes; ++p) {
    const int shift = 8 * p;
    for (int i = tid; i < WAVES * 256; i += kSortThreads) (&s.cnt[0][0])[i] = 0;
    __syncthreads();
    rank_digit<ITEMS>(key, i0, n, shift, s.cnt[wave], pos);
    __syncthreads();
    int first = 0;
    if (tid < 256) {
      int total = 0, t;
#pragma unroll
      for (int w = 0; w < WAVES; ++w) total += s.cnt[w][tid];
      first = gsk::wave_excl_scan(total, t);
      if (__lane_id() == 0) s.wave[wave] = t;
    }
    __syncthreads();
    if (tid < 256) {
      for (int w = 0; w < wave; ++w) first += s.wave[w];
#pragma unroll
      for (int w = 0; w < WAVES; ++w) {
        const int c = s.cnt[w][tid];
        s.cnt[w][tid] = (uint16_t)first;
        first += c;
      }
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < ITEMS; ++k) {
      if (i0 + k * 64 < n) {
        const int q = s.cnt[wave][(int)((key[k] >> shift) & 255u)] + pos[k];
        s.key[q] = key[k];
        s.val[q] = val[k];
      }
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < ITEMS; ++k) {
      if (i0 + k * 64 < n) {
        key[k] = s.key[i0 + k * 64];
        val[k] = s.val[i0 + k * 64];
      }
    }
  }
#pragma unroll
  for (int k = 0; k < ITEMS; ++k) {
    if (i0 + k * 64 < n) {
      kout[i0 + k * 64] = key[k];
      vout[i0 + k * 64] = val[k];
    }
  }
}

template <class KeyT>
__global__ __launch_bounds__(kSortThreads) void k_sort_block(const KeyT* kin, const int32_t* vin, KeyT* kout,
                                                             int32_t* vout, const int32_t* __restrict__ count_dev,
                                                             int64_t n_sized, int64_t cap, int passes) {
  __shared__ BlockStage<KeyT> s;
  const int n = (int)sort_count(count_dev, n_sized, cap);
  if (n <= kSortThreads) sort_block<KeyT, 1>(s, kin, vin, kout, vout, n, passes);
  else if (n <= 2 * kSortThreads) sort_block<KeyT, 2>(s, kin, vin, kout, vout, n, passes);
  else if (n <= 4 * kSortThreads) sort_block<KeyT, 4>(s, kin, vin, kout, vout, n, passes);
  else sort_block<KeyT, 8>(s, kin, vin, kout, vout, n, passes);
}

// ------------------------------------------------------------------ the record list and the emission
// Visible records listed wave by wave (64 consecutive Gaussians), view by view inside a wave, Gaussians ascending
// inside a view: key = depth bits, value = record id.  The count
// R goes to counters[kRecCount] (entries past the record capacity are not written; R > capacity implies more
// instances than the instance capacity, which the instance total flags).
constexpr int kRecCount = 196;
// The instance total: the end of the exclusive scan of the per-Gaussian instance counts (the full count even
// when the record list itself overflowed), set by the record list's first thread.
constexpr int kInstSum = 197;

// Running sums over blocks of 256 items (Gaussians, sorted records) without a scan: the kernel that forms the items'
// counts leaves each block's total and adds it to the total of its group of kGroup blocks; a block of the consumer sums
// the groups and then the blocks before it, a wave by itself.  (Scans of the items took three launches, 14 us, each.)
constexpr int kGroup = gsk::kTotalsGroup;

// part_before only loads, so that a caller can have its own loads in flight beside them before it sums the lanes.
__device__ __forceinline__ int64_t part_before(const int32_t* __restrict__ blocks,
                                               const unsigned long long* __restrict__ groups, int64_t b) {
  const int lane = __lane_id();
  const int64_t grp = b / kGroup;
  int64_t x = lane < (int)(b % kGroup) ? blocks[grp * kGroup + lane] : 0;
  for (int64_t i0 = 0; i0 < grp; i0 += 256) {  // four loads in flight
    unsigned long long v[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) v[k] = i0 + 64 * k + lane < grp ? groups[i0 + 64 * k + lane] : 0;
    x += (int64_t)((v[0] + v[1]) + (v[2] + v[3]));
  }
  return x;
}

__device__ __forceinline__ int rect_area(const short4 rc) { return (rc.y - rc.x + 1) * (rc.w - rc.z + 1); }

// ... and each visible record's first partial slot.  The instances of a wave's 64 Gaussians occupy one run of
// slots from inst_first[g0] (g0 the wave's first Gaussian), laid out in the record list's order: view by view,
// Gaussians ascending within a view; so the projection backward, which takes the views together, reads each
// view's partials of the wave as one contiguous run.  Wide records (more than kWideRecord tiles) are appended
// to big_rec (count in counters[kBigCount], one atomic per block: they queue at about 5 ns each, 30 us of a view
// whose every wave held some; the list order is not fixed, which nothing depends on).
constexpr int kBigCount = 198;
constexpr int kFrameCounters = 256;  // the frame's counters; behind them the two sorts' zeroed words

//
// With many views the reads of rectangles and depths, 8 and 4 bytes a visible record in rows of n, set the time:
// kViewBatch views' reads are in flight together.
constexpr int kViewBatch = 4;
constexpr int kWideList = 1024;

__global__ __launch_bounds__(256) void k_record_list(const uint64_t* __restrict__ vis_mask,
                                                    const int32_t* __restrict__ n_rec,
                                                    const int32_t* __restrict__ n_inst, gsk::Totals tot,
                                                    int32_t* __restrict__ first, int32_t* __restrict__ inst_first,
                                                    const short4* __restrict__ rect,
                                                    const uint32_t* __restrict__ zbits, int V, int64_t n, int64_t rcap,
                                                    uint32_t* __restrict__ rkeys, int32_t* __restrict__ rvals,
                                                    int32_t* __restrict__ rec_slot, int32_t* __restrict__ big_rec,
                                                    int32_t* __restrict__ counters, int64_t capacity) {
  __shared__ int s_rec[4], s_inst[4];
  __shared__ int32_t s_wide[kWideList];
  __shared__ int s_wides, s_wide_at;
  const int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int wave = threadIdx.x >> 6;
  if (threadIdx.x == 0) s_wides = 0;
  const bool here = g < n;
  const uint64_t m = here ? vis_mask[g] : 0ull;
  const int my_rec = here ? n_rec[g] : 0, my_inst = here ? n_inst[g] : 0;
  int64_t c = part_before(tot.rec, tot.rec_group, blockIdx.x);
  int64_t inst_base = part_before(tot.inst, tot.inst_group, blockIdx.x);
  int wave_rec, wave_inst;
  const int rec_ex = gsk::wave_excl_scan(my_rec, wave_rec), inst_ex = gsk::wave_excl_scan(my_inst, wave_inst);
  if (__lane_id() == 0) {
    s_rec[wave] = wave_rec;
    s_inst[wave] = wave_inst;
  }
  c = gsk::wave_sum64(c);
  inst_base = gsk::wave_sum64(inst_base);
  __syncthreads();
  for (int w = 0; w < wave; ++w) {
    c += s_rec[w];
    inst_base += s_inst[w];
  }
  if (here) {
    first[g] = (int32_t)c + rec_ex;
    inst_first[g] = (int32_t)inst_base + inst_ex;
  }
  if (g == n - 1) {
    // the record count R, and counters[0] = the instance total (the full count) with the overflow flag if it is above
    // the capacity
    const int64_t total = inst_base + inst_ex + my_inst;
    counters[kRecCount] = (int32_t)c + rec_ex + my_rec;
    counters[kInstSum] = (int32_t)total;
    counters[0] = (int32_t)total;
    if (total > capacity) atomicOr(counters + 1, GS_FLAG_INSTANCE_OVERFLOW);
  }
  // The wave's records start where its first Gaussian's do and are listed view by view, each view's records in lane
  // (Gaussian) order, so that every read and write of a view is one coalesced run.  Within a view the list keeps
  // ascending Gaussian index, which is all the depth sort's tie rule needs (records of different views never share a
  // tile).
  int32_t slot_c = (int32_t)inst_base;
  const uint64_t lt = gsk::lanemask_lt();
  for (int v0 = 0; v0 < V; v0 += kViewBatch) {
    if (__ballot((m >> v0) != 0) == 0) break;
    short4 rcs[kViewBatch];
    uint32_t zs[kViewBatch];
#pragma unroll
    for (int i = 0; i < kViewBatch; ++i) {
      const bool vis = v0 + i < V && (m >> (v0 + i)) & 1ull;
      const int64_t r = (int64_t)(v0 + i) * n + g;
      rcs[i] = make_short4(0, -1, 0, -1);
      zs[i] = 0;
      if (vis) {
        rcs[i] = rect[r];
        zs[i] = zbits[r];
      }
    }
#pragma unroll
    for (int i = 0; i < kViewBatch; ++i) {
      const bool vis = v0 + i < V && (m >> (v0 + i)) & 1ull;
      const uint64_t vb = __ballot(vis);
      if (vb == 0) continue;
      const int64_t pos = c + __popcll(vb & lt);
      c += __popcll(vb);
      const int64_t r = (int64_t)(v0 + i) * n + g;
      const int area = rect_area(rcs[i]);  // (0 for the empty rectangle)
      int view_total;
      const int before = gsk::wave_excl_scan(area, view_total);
      const int32_t slot = slot_c + before;
      slot_c += view_total;
      if (!vis) continue;
      if (pos < rcap) {
        rkeys[pos] = zs[i];
        rvals[pos] = (int32_t)r;
      }
      rec_slot[r] = slot;
      const bool wide = area > gsk::kWideRecord;
      const uint64_t wb = __ballot(wide);
      if (wb) {
        const int lead = __builtin_ctzll(wb);
        int base = 0;
        if (__lane_id() == lead) base = atomicAdd(&s_wides, __popcll(wb));
        base = __builtin_amdgcn_readlane(base, lead);
        const int at = base + __popcll(wb & lt);
        if (wide && at < kWideList) {
          s_wide[at] = (int32_t)r;
        } else if (wide) {  // (more of them than the block's list holds)
          const int bpos = atomicAdd(counters + kBigCount, 1);
          if (bpos < rcap) big_rec[bpos] = (int32_t)r;
        }
      }
    }
  }
  __syncthreads();
  const int wides = min(s_wides, kWideList);
  if (wides == 0) return;
  if (threadIdx.x == 0) s_wide_at = atomicAdd(counters + kBigCount, wides);
  __syncthreads();
  for (int i = threadIdx.x; i < wides; i += 256)
    if (s_wide_at + i < rcap) big_rec[s_wide_at + i] = s_wide[i];
}

// The tile rectangle of each depth-sorted record, in sorted order (tx0 | tx1 << 16 in rx[j], ty0 | ty1 << 16 in ry[j]) so
// that the emission reads it in coalesced runs, and the totals of their instance counts.
__global__ __launch_bounds__(256) void k_record_counts(const int32_t* __restrict__ rvals,
                                                       const short4* __restrict__ rect,
                                                       const int32_t* __restrict__ counters, int64_t rcap,
                                                       uint32_t* __restrict__ rx, uint32_t* __restrict__ ry,
                                                       int32_t* __restrict__ blocks,
                                                       unsigned long long* __restrict__ groups,
                                                       int32_t* __restrict__ waves) {
  __shared__ int s_cnt[4];
  const int64_t R = sort_count(counters + kRecCount, rcap, rcap);
  for (int64_t b = blockIdx.x; b * 256 < R; b += gridDim.x) {
    const int64_t j = b * 256 + threadIdx.x;
    int cnt = 0;
    if (j < R) {
      const short4 rc = rect[rvals[j]];
      cnt = rect_area(rc);
      rx[j] = (uint32_t)(uint16_t)rc.x | ((uint32_t)(uint16_t)rc.y << 16);
      ry[j] = (uint32_t)(uint16_t)rc.z | ((uint32_t)(uint16_t)rc.w << 16);
    }
    gsk::leave_totals<1>({cnt}, s_cnt, {blocks}, {groups}, b);
    if (threadIdx.x < 4) {  // and where each wave's records start in the block, so that the emission's waves are by themselves
      int before = 0;
      for (int w = 0; w < (int)threadIdx.x; ++w) before += s_cnt[w];
      waves[4 * b + threadIdx.x] = before;
    }
  }
}

// Records with more tiles than this are emitted by a whole wave, a tile per lane.
constexpr int kSolo = gsk::kWideRecord;

__device__ __forceinline__ int64_t read_lane64(int64_t x, int l) {
  const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)x, l);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)((uint64_t)x >> 32), l);
  return (int64_t)(((uint64_t)hi << 32) | lo);
}

// One thread per depth-sorted record: its run of instances (tiles row by row) starts at the sum of the counts before it;
// key = global tile id, value = record id.  Records with more than kSolo tiles are written by the whole wave, a tile per lane.  The
// runs of a wave's records are consecutive, so the other records are first laid out
// in a per-wave LDS window of kEmitWin instances and then stored by the wave in coalesced runs, a window at a
// time; positions of wide records in a window are marked empty and skipped by the copy.
constexpr int kEmitWin = 512;
constexpr uint32_t kEmitEmpty = 0xffffffffu;  // no tile id takes this value

__global__ __launch_bounds__(256) void k_emit(const int32_t* __restrict__ rvals, const int32_t* __restrict__ blocks,
                                             const unsigned long long* __restrict__ groups,
                                             const int32_t* __restrict__ waves, const uint32_t* __restrict__ rx,
                                             const uint32_t* __restrict__ ry,
                                             const gs_camera* __restrict__ cams,
                                             int V, int64_t n, const int32_t* __restrict__ counters, int64_t rcap,
                                             int64_t capacity, uint32_t* __restrict__ keys,
                                             int32_t* __restrict__ vals) {
  __shared__ uint32_t wkey[4][kEmitWin];
  __shared__ int32_t wval[4][kEmitWin];
  const int64_t R = sort_count(counters + kRecCount, rcap, rcap);
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  for (int64_t blk = blockIdx.x; blk * 256 < R; blk += gridDim.x) {
    const int64_t j = blk * 256 + threadIdx.x;
    const bool here = j < R;
    const int64_t jj = here ? j : R - 1;
    const int64_t r = rvals[jj];
    const uint32_t x = rx[jj], y = ry[jj];
    const int64_t part = part_before(blocks, groups, blk);
    const int start = waves[4 * blk + wv];
    short4 rc = make_short4(0, -1, 0, -1);
    int toff = 0, tx_n = 1;
    if (here) {
      rc = make_short4((short)(x & 0xffffu), (short)(x >> 16), (short)(y & 0xffffu), (short)(y >> 16));
      const int v = (int)((uint32_t)r / (uint32_t)n);  // r < 2^31
      toff = cams[v].tile_offset;
      tx_n = cams[v].tiles_x;
    }
    const int w = rc.y - rc.x + 1, cnt = here ? w * (rc.w - rc.z + 1) : 0;
    int wave_cnt;
    const int64_t o = gsk::wave_sum64(part) + start + gsk::wave_excl_scan(cnt, wave_cnt);
    const uint64_t present = __ballot(here);
    if (present == 0) continue;  // the same in every lane of the wave
    uint64_t big = __ballot(cnt > kSolo);
    // the wave's instances are [lo, hi): the records of lanes 0 .. last are consecutive in the sorted list
    const int last = 63 - __builtin_clzll(present);
    const int64_t lo = read_lane64(o, 0), hi = read_lane64(o + cnt, last);
    uint32_t* wk = wkey[wv];
    int32_t* wvv = wval[wv];
    const bool direct = hi - lo > 64 * kSolo;  // mostly wide records' runs: more windows to walk than to fill
    if (direct && here && cnt <= kSolo) {
      int id = toff + rc.z * tx_n + rc.x, x = 0;
      for (int64_t q = o; q < min(o + cnt, capacity); ++q) {
        keys[q] = (uint32_t)id;
        vals[q] = (int32_t)r;
        ++id;
        if (++x == w) {
          x = 0;
          id += tx_n - w;
        }
      }
    }
    for (int64_t win = lo; win < hi && !direct; win += kEmitWin) {
      if (big) {
        for (int i = lane; i < kEmitWin; i += 64) wk[i] = kEmitEmpty;
      }
      if (here && cnt <= kSolo) {
        const int64_t k0 = max(o, win) - o, k1 = min(o + cnt, win + kEmitWin) - o;
        if (k0 < k1) {
          int ty = rc.z + (int)k0 / w, tx = rc.x + (int)k0 % w;
          for (int64_t k = k0; k < k1; ++k) {
            const int i = (int)(o + k - win);
            wk[i] = (uint32_t)(toff + ty * tx_n + tx);
            wvv[i] = (int32_t)r;
            if (++tx > rc.y) {
              tx = rc.x;
              ++ty;
            }
          }
        }
      }
      __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "workgroup");  // the wave's LDS writes land before its reads
      const int m = (int)min<int64_t>(kEmitWin, hi - win);
      for (int i = lane; i < m; i += 64) {
        const uint32_t kk = wk[i];
        const int64_t q = win + i;
        if (kk != kEmitEmpty && q < capacity) {
          keys[q] = kk;
          vals[q] = wvv[i];
        }
      }
      __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "workgroup");  // and its reads before the next window's writes
    }
    // wide records, a tile per lane: lane k's first tile, then 64 tiles on, which is dq rows and dr tiles (no division in
    // the loop: the nearest records are the widest and meet in a few waves, whose time is the kernel's)
    const int dq = 64 / max(w, 1), dr = 64 - dq * w;
    const float inv_w = 1.f / (float)max(w, 1);
    while (big) {
      const int L = __builtin_ctzll(big);
      big &= big - 1;
      const int64_t oL = read_lane64(o, L);
      const int rL = __builtin_amdgcn_readlane((int)r, L);
      const int cL = __builtin_amdgcn_readlane(cnt, L), wL = __builtin_amdgcn_readlane(w, L);
      const int x0 = __builtin_amdgcn_readlane((int)rc.x, L), y0 = __builtin_amdgcn_readlane((int)rc.z, L);
      const int toL = __builtin_amdgcn_readlane(toff, L), txL = __builtin_amdgcn_readlane(tx_n, L);
      const int dqL = __builtin_amdgcn_readlane(dq, L), drL = __builtin_amdgcn_readlane(dr, L);
      const float invL = gsk::read_lane(inv_w, L);
      const int row = (int)(((float)lane + 0.5f) * invL);  // lane / wL (half a tile from every whole row)
      int x = lane - row * wL;
      int id = toL + (y0 + row) * txL + x0 + x;
      const int m = (int)max<int64_t>(0, min<int64_t>(cL, capacity - oL));
      uint32_t* kq = keys + oL;
      int32_t* vq = vals + oL;
      const int step = dqL * txL + drL, wrap = txL - wL;
      for (int k = lane; k < m; k += 64) {
        kq[k] = (uint32_t)id;
        vq[k] = rL;
        x += drL;
        id += step;
        if (x >= wL) {
          x -= wL;
          id += wrap;
        }
      }
    }
  }
}

__global__ __launch_bounds__(256) void k_ranges(const uint32_t* __restrict__ keys, const int32_t* __restrict__ count_dev,
                                                int64_t n_sized, int64_t cap, int2* __restrict__ range) {
  const int64_t n = sort_count(count_dev, n_sized, cap);
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256) {
    const uint32_t t = keys[i];
    if (i == 0 || keys[i - 1] != t) range[t].x = (int)i;
    if (i == n - 1 || keys[i + 1] != t) range[t].y = (int)(i + 1);
  }
}

// Compositing schedule: tiles in descending order of their list length, bucketed by floor(log2(len + 1))
// (32 buckets, longest first; the order inside a bucket does not matter).  Tiles longer than the segment
// length (split into depth segments by the fused backward) all go to bucket 0, so they lead the schedule.
__device__ __forceinline__ int len_bucket(const int2* range, int t, int seg_len) {
  const int len = range[t].y - range[t].x;
  if (seg_len > 0 && len > seg_len) return 0;
  return __clz((unsigned)len + 1u);  // 31 - floor(log2(len + 1)): longer lists get smaller bucket ids
}

__global__ __launch_bounds__(256) void k_sched_hist(const int2* __restrict__ range, int n_tiles, int seg_len,
                                                    int32_t* __restrict__ bucket_cnt) {
  __shared__ int h[32];
  if (threadIdx.x < 32) h[threadIdx.x] = 0;
  __syncthreads();
  const int t = blockIdx.x * blockDim.x + threadIdx.x;
  if (t < n_tiles) atomicAdd(&h[len_bucket(range, t, seg_len)], 1);
  __syncthreads();
  if (threadIdx.x < 32 && h[threadIdx.x]) atomicAdd(bucket_cnt + threadIdx.x, h[threadIdx.x]);
}

__global__ void k_sched_scan(const int32_t* __restrict__ bucket_cnt, int32_t* __restrict__ bucket_off) {
  if (threadIdx.x != 0) return;
  int run = 0;
  for (int b = 0; b < 32; ++b) {
    bucket_off[b] = run;
    run += bucket_cnt[b];
  }
}

__global__ __launch_bounds__(256) void k_sched_scatter(const int2* __restrict__ range, int n_tiles, int seg_len,
                                                       int32_t* __restrict__ bucket_off, int32_t* __restrict__ order) {
  __shared__ int h[32], base[32];
  if (threadIdx.x < 32) h[threadIdx.x] = 0;
  __syncthreads();
  const int t = blockIdx.x * blockDim.x + threadIdx.x;
  int b = 0, rank = 0;
  if (t < n_tiles) {
    b = len_bucket(range, t, seg_len);
    rank = atomicAdd(&h[b], 1);
  }
  __syncthreads();
  if (threadIdx.x < 32 && h[threadIdx.x]) base[threadIdx.x] = atomicAdd(bucket_off + threadIdx.x, h[threadIdx.x]);
  __syncthreads();
  if (t < n_tiles) order[base[b] + rank] = t;
}

// Work items of the fused backward, in schedule order: one per tile, or one per depth segment of a tile
// longer than seg_len (those lead the schedule, so their segments take item indices 0 .. slots - 1, which
// are also their segment-state slots).
__global__ __launch_bounds__(256) void k_seg_count(const int2* __restrict__ range, const int32_t* __restrict__ order,
                                                   int n_tiles, int seg_len, int32_t* __restrict__ seg_count) {
  const int p = blockIdx.x * blockDim.x + threadIdx.x;
  if (p >= n_tiles) return;
  const int2 r = range[order[p]];
  const int len = r.y - r.x;
  seg_count[p] = len > seg_len ? (len + seg_len - 1) / seg_len : 1;
}

__global__ __launch_bounds__(256) void k_seg_emit(const int32_t* __restrict__ order, int n_tiles,
                                                  const int32_t* __restrict__ seg_count,
                                                  const int32_t* __restrict__ seg_first, int4* __restrict__ items,
                                                  int32_t* __restrict__ counters) {
  const int p = blockIdx.x * blockDim.x + threadIdx.x;
  if (p == 0) {
    const int nl = counters[128];  // bucket 0: split tiles
    counters[194] = nl;
    counters[193] = nl > 0 ? seg_first[nl - 1] + seg_count[nl - 1] : 0;
    counters[192] = seg_first[n_tiles - 1] + seg_count[n_tiles - 1];
  }
  if (p >= n_tiles) return;
  const int n = seg_count[p], first = seg_first[p], t = order[p];
  for (int k = 0; k < n; ++k) items[first + k] = make_int4(t, k, n > 1 ? first : -1, p);
}

// Frames of at most kSchedOneBlock tiles: the schedule and the work items in one workgroup, each phase a loop
// over the tiles between barriers (bucket histogram; its scan; the scatter into schedule order, which also
// stores each position's segment count; the scan of the segment counts with the items), in place of the seven
// launches above, whose fixed cost dominates there.  The results are those of the launches above (the order
// inside a bucket is again that of the LDS atomics).  Without segments (seg_len <= 0) only the schedule.
constexpr int kSchedOneBlock = 16384;

__global__ __launch_bounds__(1024) void k_schedule_small(const int2* __restrict__ range, int n_tiles, int seg_len,
                                                         int32_t* __restrict__ order, int32_t* __restrict__ seg_count,
                                                         int32_t* __restrict__ seg_first, int4* __restrict__ items,
                                                         int32_t* __restrict__ counters) {
  __shared__ int h[32], base[32], wsum[16];
  const int tid = threadIdx.x, lane = __lane_id(), wave = tid >> 6;
  if (tid < 32) h[tid] = 0;
  __syncthreads();
  // each thread's list lengths, loaded once (all loads in flight together) and kept for the scatter
  constexpr int kPer = kSchedOneBlock / 1024;
  int lens[kPer];
#pragma unroll
  for (int j = 0; j < kPer; ++j) {
    const int t = j * 1024 + tid;
    lens[j] = t < n_tiles ? range[t].y - range[t].x : -1;
  }
  auto bucket = [&](int len) { return len < 0 ? 32 : (seg_len > 0 && len > seg_len ? 0 : __clz((unsigned)len + 1u)); };
  // the LDS atomics are taken once per distinct bucket of a wave (a wave's tiles fall into a few buckets, and
  // atomics of many lanes on one address serialise)
#pragma unroll
  for (int j = 0; j < kPer; ++j) {
    if (j * 1024 >= n_tiles) break;
    const int b = bucket(lens[j]);
    for (uint64_t rest = __builtin_amdgcn_ballot_w64(b < 32); rest;) {
      const int lb = __builtin_amdgcn_readlane(b, __builtin_ctzll(rest));
      const uint64_t m = __builtin_amdgcn_ballot_w64(b == lb);
      if (lane == 0) atomicAdd(&h[lb], __popcll(m));
      rest &= ~m;
    }
  }
  __syncthreads();
  if (tid == 0) {
    int run = 0;
    for (int b = 0; b < 32; ++b) {
      base[b] = run;
      counters[128 + b] = h[b];
      run += h[b];
      counters[160 + b] = run;
    }
  }
  __syncthreads();
  const uint64_t lt = gsk::lanemask_lt();
#pragma unroll
  for (int j = 0; j < kPer; ++j) {
    if (j * 1024 >= n_tiles) break;
    const int t = j * 1024 + tid, len = lens[j], b = bucket(len);
    int pos = 0;
    for (uint64_t rest = __builtin_amdgcn_ballot_w64(b < 32); rest;) {
      const int lb = __builtin_amdgcn_readlane(b, __builtin_ctzll(rest));
      const uint64_t m = __builtin_amdgcn_ballot_w64(b == lb);
      int at = 0;
      if (lane == 0) at = atomicAdd(&base[lb], __popcll(m));
      at = __builtin_amdgcn_readlane(at, 0);
      if (b == lb) pos = at + __popcll(m & lt);
      rest &= ~m;
    }
    if (b < 32) {
      order[pos] = t;
      if (seg_len > 0) seg_count[pos] = len > seg_len ? (len + seg_len - 1) / seg_len : 1;
    }
  }
  if (seg_len <= 0) return;
  __syncthreads();  // order and seg_count of this workgroup visible to all its threads
  const int nl = h[0];
  int carry = 0;
  for (int c0 = 0; c0 < n_tiles; c0 += 4096) {  // four consecutive positions per thread
    const int p0 = c0 + 4 * tid;
    int cnt[4], til[4], sum = 0;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      cnt[j] = p0 + j < n_tiles ? seg_count[p0 + j] : 0;
      til[j] = p0 + j < n_tiles ? order[p0 + j] : 0;
      sum += cnt[j];
    }
    int wt;
    const int ex = gsk::wave_excl_scan(sum, wt);
    if (lane == 0) wsum[wave] = wt;
    __syncthreads();
    int before = 0, chunk = 0;
    for (int w = 0; w < 16; ++w) {
      before += w < wave ? wsum[w] : 0;
      chunk += wsum[w];
    }
    int first = carry + before + ex;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int p = p0 + j, n = cnt[j];
      if (p < n_tiles) {
        seg_first[p] = first;
        for (int k = 0; k < n; ++k) items[first + k] = make_int4(til[j], k, n > 1 ? first : -1, p);
        if (p == nl - 1) counters[193] = first + n;
      }
      first += n;
    }
    carry += chunk;
    __syncthreads();  // wsum is rewritten by the next chunk
  }
  if (tid == 0) {
    counters[194] = nl;
    if (nl == 0) counters[193] = 0;
    counters[192] = carry;
  }
}

inline int64_t cdiv(int64_t a, int64_t b) { return (a + b - 1) / b; }
// Blocks of 256 threads over items whose number only the device knows, which may be far below the capacity: every block
// costs about 0.3 ns to start and end (25 us for a capacity of 24 M), so they stride over the items from here on.
inline unsigned strided_blocks(int64_t cap) { return (unsigned)std::min<int64_t>(cdiv(cap, 256), 4096); }
inline int64_t align64(int64_t a) { return (a + 63) & ~int64_t(63); }

}  // namespace

namespace gs_launch {

size_t scan_scratch_ints(int64_t n) {
  size_t total = 0;
  while (n > 1) {
    n = cdiv(n, kScanTile);
    total += (size_t)align64(n);
  }
  return total + 64;
}

hipError_t scan_exclusive(const int32_t* in, int32_t* out, int64_t n, int32_t* scratch, hipStream_t st) {
  if (n <= 0) return hipSuccess;
  const int64_t nb = cdiv(n, kScanTile);
  int32_t* sums = scratch;
  k_scan_tile<<<(unsigned)nb, kScanThreads, 0, st>>>(in, out, n, sums);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  if (nb > 1) {
    e = scan_exclusive(sums, sums, nb, scratch + align64(nb), st);
    if (e != hipSuccess) return e;
    k_scan_add<<<(unsigned)nb, kScanThreads, 0, st>>>(out, n, sums);
    return hipGetLastError();
  }
  return hipSuccess;
}

hipError_t fill_i32(int32_t* p, int32_t v, int64_t n, hipStream_t st) {
  if (n <= 0) return hipSuccess;
  k_fill_i32<<<(unsigned)cdiv(n, 256), 256, 0, st>>>(p, v, n);
  return hipGetLastError();
}

hipError_t fill_f32(float* p, float v, int64_t n, hipStream_t st) {
  if (n <= 0) return hipSuccess;
  k_fill_f32<<<(unsigned)cdiv(n, 256), 256, 0, st>>>(p, v, n);
  return hipGetLastError();
}

// Tiles of a sort of up to n keys, and its two passes' states.  (The 4096-key tiles of 64-bit keys are at most as many as
// the 2048-key ones of kSmallSort.)
static int64_t sort_blocks(int64_t n) {
  if (n < 1) n = 1;
  const int64_t few = n < kSmallSort ? n : kSmallSort;
  const int64_t small = cdiv(few, kSortThreads * kSmallItems), large = cdiv(n, kSortThreads * kLargeItems);
  return small > large ? small : large;
}
static size_t state_ints(int64_t n) { return 512 * (size_t)sort_blocks(n); }

size_t sort_scratch_ints(int64_t n) { return (size_t)kSortZero64 + state_ints(n); }
size_t frame_sort_scratch_ints(int64_t n) { return state_ints(n); }

// zeroed: the words described at kSortZero32 / 64, zero; states: state_ints(n_sized).
template <class KeyT>
static hipError_t sort_impl(KeyT* k0, int32_t* v0, KeyT* k1, int32_t* v1, int64_t n_sized, const int32_t* count_dev,
                            int64_t cap, int key_bits, int32_t* zeroed, int32_t* states, hipStream_t st) {
  if (n_sized <= 0) return hipSuccess;
  const int passes = (key_bits + 7) / 8;
  if (n_sized <= kBlockSort) {
    k_sort_block<KeyT><<<1, kSortThreads, 0, st>>>(k0, v0, passes & 1 ? k1 : k0, passes & 1 ? v1 : v0, count_dev, n_sized,
                                                   cap, passes);
    return hipGetLastError();
  }
  const int64_t nb = sort_blocks(n_sized);
  uint32_t* state[2] = {reinterpret_cast<uint32_t*>(states), reinterpret_cast<uint32_t*>(states) + 256 * nb};
  const int64_t db = cdiv(n_sized, kDigitThreads * kDigitItems);
  k_sort_digits<KeyT><<<(unsigned)(db < kDigitBlocks ? db : kDigitBlocks), kDigitThreads, 0, st>>>(
      k0, count_dev, n_sized, cap, passes, zeroed, state[0]);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  KeyT* kb[2] = {k0, k1};
  int32_t* vb[2] = {v0, v1};
  for (int p = 0; p < passes; ++p) {
    const int src = p & 1, dst = src ^ 1;
    k_sort_scatter<KeyT><<<(unsigned)nb, kSortThreads, 0, st>>>(kb[src], vb[src], kb[dst], vb[dst], count_dev, n_sized,
                                                                cap, p, passes, zeroed, state[src], state[dst]);
    if ((e = hipGetLastError()) != hipSuccess) return e;
  }
  return hipSuccess;
}

hipError_t sort_pairs(uint64_t* k0, int32_t* v0, uint64_t* k1, int32_t* v1, int64_t n_sized, const int32_t* count_dev,
                      int64_t cap, int key_bits, int32_t* scratch, hipStream_t st) {
  hipError_t e = fill_i32(scratch, 0, kSortZero64, st);
  if (e != hipSuccess) return e;
  return sort_impl<uint64_t>(k0, v0, k1, v1, n_sized, count_dev, cap, key_bits, scratch, scratch + kSortZero64, st);
}

hipError_t sort_by_tile(const gs_frame& f, int64_t n_sized, const int32_t* count_dev, hipStream_t st) {
  return sort_impl<uint32_t>(f.keys[0], f.vals[0], f.keys[1], f.vals[1], n_sized, count_dev, f.capacity, f.key_bits,
                             f.counters + kFrameCounters + kSortZero32, f.scratch, st);
}

// Behind the frame's counters: the words of its two sorts, the emission's group totals (both cleared by binning), the
// projection's group totals (cleared by it), and the block totals.
constexpr int kGroupItems = 256 * kGroup;

struct EmitTotals {
  int32_t *blocks, *waves;
  unsigned long long* groups;
};
gsk::Totals project_totals(const gs_frame& f);
static EmitTotals emit_totals(const gs_frame& f) {
  EmitTotals t;
  t.groups = reinterpret_cast<unsigned long long*>(f.counters + kFrameCounters + 2 * kSortZero32);
  const gsk::Totals p = project_totals(f);
  t.blocks = p.inst + align64(cdiv(f.n, 256));
  t.waves = t.blocks + align64(cdiv(f.rec_cap, 256));
  return t;
}
gsk::Totals project_totals(const gs_frame& f) {
  gsk::Totals t;
  const int64_t groups = cdiv(f.n, kGroupItems);
  t.rec_group = reinterpret_cast<unsigned long long*>(f.counters + kFrameCounters + 2 * kSortZero32) +
                cdiv(f.rec_cap, kGroupItems);
  t.inst_group = t.rec_group + groups;
  t.rec = reinterpret_cast<int32_t*>(t.inst_group + groups);
  t.inst = t.rec + align64(cdiv(f.n, 256));
  return t;
}

size_t counter_ints(int64_t n, int64_t rec_cap) {
  return (size_t)(kFrameCounters + 2 * kSortZero32 + 2 * (cdiv(rec_cap, kGroupItems) + 2 * cdiv(n, kGroupItems)) +
                  2 * align64(cdiv(n, 256)) + 5 * align64(cdiv(rec_cap, 256)));
}

hipError_t clear_project(const gs_frame& f, hipStream_t st) {
  const int64_t m = 4 * cdiv(f.n, kGroupItems);
  k_fill2_i32<<<(unsigned)cdiv(m, 256), 256, 0, st>>>(f.counters, 2,
                                                      reinterpret_cast<int32_t*>(project_totals(f).rec_group), m, 0);
  return hipGetLastError();
}

// Binning up to the instance total: the records' first partial slots, the record list sorted by depth (record ids
// in rvals[0]), each sorted record's tile rectangle (rkeys[0], rkeys[1]) and the totals of their instance counts, the
// instance total and the overflow flag.
hipError_t bin_records(const gs_frame& f, hipStream_t st) {
  const int64_t rcap = f.rec_cap;
  // the tile ranges; and of the counters the schedule's buckets and all behind them, the two sorts' words and the
  // emission's group totals
  constexpr int kFirst = 128;
  const int64_t nr = 2 * (int64_t)f.n_tiles;
  const int64_t nc = kFrameCounters - kFirst + 2 * kSortZero32 + 2 * cdiv(rcap, kGroupItems);
  k_fill2_i32<<<(unsigned)cdiv(nr > nc ? nr : nc, 256), 256, 0, st>>>(f.tile_range, nr, f.counters + kFirst, nc, 0);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  k_record_list<<<(unsigned)cdiv(f.n, 256), 256, 0, st>>>(f.vis_mask, f.n_rec, f.n_inst, project_totals(f), f.rec_first,
                                                          f.inst_first, reinterpret_cast<const short4*>(f.rect), f.zbits,
                                                          f.n_views, f.n, rcap, f.rkeys[0], f.rvals[0], f.rec_slot,
                                                          f.big_rec, f.counters, f.capacity);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  if ((e = sort_impl<uint32_t>(f.rkeys[0], f.rvals[0], f.rkeys[1], f.rvals[1], rcap, f.counters + kRecCount, rcap, 32,
                               f.counters + kFrameCounters, f.scratch, st)) != hipSuccess)
    return e;  // 4 passes: the sorted records are back in rkeys[0] / rvals[0]
  // the sorted rectangles take the depth keys' buffers, which are no longer needed
  const EmitTotals t = emit_totals(f);
  k_record_counts<<<strided_blocks(rcap), 256, 0, st>>>(f.rvals[0], reinterpret_cast<const short4*>(f.rect),
                                                             f.counters, rcap, f.rkeys[0], f.rkeys[1], t.blocks,
                                                             t.groups, t.waves);
  return hipGetLastError();
}

hipError_t emit(const gs_frame& f, hipStream_t st) {
  const EmitTotals t = emit_totals(f);
  k_emit<<<strided_blocks(f.rec_cap), 256, 0, st>>>(f.rvals[0], t.blocks, t.groups, t.waves, f.rkeys[0], f.rkeys[1], f.cams,
                                                         f.n_views, f.n, f.counters, f.rec_cap, f.capacity, f.keys[0],
                                                         f.vals[0]);
  return hipGetLastError();
}

// The longest-first schedule; its 32 bucket counts (counters[128..160)) were cleared by bin_records.
hipError_t tile_schedule(const gs_frame& f, hipStream_t st) {
  int32_t* cnt = f.counters + 128;
  int32_t* off = f.counters + 160;
  hipError_t e = hipSuccess;
  const auto* rng = reinterpret_cast<const int2*>(f.tile_range);
  if (f.n_tiles <= kSchedOneBlock) {  // with the work items
    k_schedule_small<<<1, 1024, 0, st>>>(rng, f.n_tiles, f.seg_len, f.tile_order, f.seg_count, f.seg_first,
                                         reinterpret_cast<int4*>(f.items), f.counters);
    return hipGetLastError();
  }
  const unsigned nb = (unsigned)cdiv(f.n_tiles, 256);
  k_sched_hist<<<nb, 256, 0, st>>>(rng, f.n_tiles, f.seg_len, cnt);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  k_sched_scan<<<1, 64, 0, st>>>(cnt, off);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  k_sched_scatter<<<nb, 256, 0, st>>>(rng, f.n_tiles, f.seg_len, off, f.tile_order);
  return hipGetLastError();
}

hipError_t work_items(const gs_frame& f, hipStream_t st) {
  if (f.seg_len <= 0 || f.n_tiles <= kSchedOneBlock) return hipSuccess;  // small frames: by tile_schedule
  const auto* rng = reinterpret_cast<const int2*>(f.tile_range);
  const unsigned nb = (unsigned)cdiv(f.n_tiles, 256);
  k_seg_count<<<nb, 256, 0, st>>>(rng, f.tile_order, f.n_tiles, f.seg_len, f.seg_count);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  if ((e = scan_exclusive(f.seg_count, f.seg_first, f.n_tiles, f.scratch, st)) != hipSuccess) return e;
  k_seg_emit<<<nb, 256, 0, st>>>(f.tile_order, f.n_tiles, f.seg_count, f.seg_first, reinterpret_cast<int4*>(f.items),
                                 f.counters);
  return hipGetLastError();
}

// Tile ranges (cleared by bin_records).
hipError_t ranges(const gs_frame& f, const uint32_t* keys, int64_t n_sized, const int32_t* count_dev,
                  hipStream_t st) {
  if (n_sized <= 0) return hipSuccess;
  k_ranges<<<strided_blocks(n_sized), 256, 0, st>>>(keys, count_dev, n_sized, f.capacity,
                                                         reinterpret_cast<int2*>(f.tile_range));
  return hipGetLastError();
}

}  // namespace gs_launch
