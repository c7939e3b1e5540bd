// Internal device helpers of libgs (HIP, gfx950).  Not part of the public ABI.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "../../include/libgs.h"

namespace gsk {

constexpr int kWave = 64;
// Partial sums of the SSIM term (its loss_out[1 .. kLossSlots]).
constexpr int kLossSlots = 32;

// Frames of at least this many tiles run the forward of the backward's whole tiles in the kernel of the segments'
// sums (at six waves a SIMD instead of four) and keep its result in a state slot per work item; smaller frames, which
// leave the chip partly idle and wait for their longest tile, run it in the backward's kernel.  A training step with the
// forward in the sums' kernel and in the backward's: 252 tiles of 16x16 with 13 records 100 and 94 us, 1008 with 32 146
// and 141, 2028 with 56 212 and 207; a keyframe of 6.7 k tiles 1585 and 1604, odd views of 32x8 tiles 466 and 480, one
// active view of 24 1357 and 1366; 24 views of 16x8 tiles 6240 and 6225.  Frames of random Gaussians lie within 2% either
// way up to 200 k tiles (16x16 above 200 records a tile gain, 16x8 and 8x8 lose).
constexpr int kWholeTiles = 2048;

// Slots of a frame's segment state (none where lists are never split, seg_cap = 0: k_render_bwd keeps no state).
inline int seg_slots(int n_tiles, int seg_cap) {
  return seg_cap > 0 && n_tiles >= kWholeTiles ? n_tiles + seg_cap : seg_cap;
}

// Options as the kernels see them (passed by value).
struct DevOpts {
  float near_z, lowpass, alpha_min, alpha_max, t_min;
  float bg[3];
  int tile_w, tile_h;
};

inline DevOpts dev_opts(const gs_opts& o) {
  DevOpts d;
  d.near_z = o.near_z;
  d.lowpass = o.lowpass;
  d.alpha_min = o.alpha_min;
  d.alpha_max = o.alpha_max;
  d.t_min = o.t_min;
  d.bg[0] = o.bg[0];
  d.bg[1] = o.bg[1];
  d.bg[2] = o.bg[2];
  d.tile_w = o.tile_w;
  d.tile_h = o.tile_h;
  return d;
}

// ------------------------------------------------------------------ wave primitives
__device__ __forceinline__ uint64_t ballot(bool p) { return __ballot(p); }

__device__ __forceinline__ int lane_id() { return __lane_id(); }

__device__ __forceinline__ uint64_t lanemask_lt() {
  const int l = __lane_id();
  return l == 0 ? 0ull : (~0ull >> (64 - l));
}

// n plus the number of set bits of m below this lane.
__device__ __forceinline__ int rank_in(uint64_t m, int n) {
  return (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, (uint32_t)n));
}

// DPP move of a float with control CTRL; lanes without a valid source (bound_ctrl) or in a masked row read 0.
// bound_ctrl lets the move fold into the consuming add (v_add_f32_dpp).
template <int CTRL, int ROW_MASK = 0xf>
__device__ __forceinline__ float dpp_f(float x) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), CTRL, ROW_MASK, 0xf, true));
}

// Sum over the 64 lanes of a wave; the total lands in lane 63.  Six DPP adds:
// pairs, quads, half rows, rows (mirrors), then row broadcasts 15 and 31 across rows.
__device__ __forceinline__ float wave_sum_last(float x) {
  x += dpp_f<0xB1>(x);        // quad_perm [1,0,3,2]
  x += dpp_f<0x4E>(x);        // quad_perm [2,3,0,1]
  x += dpp_f<0x141>(x);       // row_half_mirror
  x += dpp_f<0x140>(x);       // row_mirror
  x += dpp_f<0x142, 0xa>(x);  // row_bcast:15 into rows 1 and 3
  x += dpp_f<0x143, 0xc>(x);  // row_bcast:31 into rows 2 and 3
  return x;
}

// A value known to be the same in every lane, moved to scalar registers.
__device__ __forceinline__ uint64_t uniform64(uint64_t v) {
  const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v);
  const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
  return ((uint64_t)hi << 32) | lo;
}

// The value of the lane n before in its row of 16 (0 from outside the row), or of lane 15 of the row before (rows 1 and
// 3), or of lane 31 (rows 2 and 3): the steps of a scan over the wave.  (In registers; a __shfl_up costs an LDS trip.)
template <int CTRL, int ROWS = 0xf>
__device__ __forceinline__ int dpp_or_zero(int x) {
  return __builtin_amdgcn_update_dpp(0, x, CTRL, ROWS, 0xf, ROWS == 0xf);
}
// Exclusive prefix sum over the 64 lanes (lane order) of a non-negative int; total = the wave's sum.  Called with every
// lane of the wave active.
__device__ __forceinline__ int wave_excl_scan(int x, int& total) {
  int incl = x;
  incl += dpp_or_zero<0x111>(incl);
  incl += dpp_or_zero<0x112>(incl);
  incl += dpp_or_zero<0x114>(incl);
  incl += dpp_or_zero<0x118>(incl);
  incl += dpp_or_zero<0x142, 0xa>(incl);
  incl += dpp_or_zero<0x143, 0xc>(incl);
  total = __builtin_amdgcn_readlane(incl, 63);
  return incl - x;
}

template <int CTRL, int ROWS = 0xf>
__device__ __forceinline__ int64_t dpp_or_zero64(int64_t x) {
  const uint32_t lo = (uint32_t)dpp_or_zero<CTRL, ROWS>((int)(uint32_t)x);
  const uint32_t hi = (uint32_t)dpp_or_zero<CTRL, ROWS>((int)(uint32_t)((uint64_t)x >> 32));
  return (int64_t)(((uint64_t)hi << 32) | lo);
}
__device__ __forceinline__ int64_t wave_sum64(int64_t x) {
  x += dpp_or_zero64<0x111>(x);
  x += dpp_or_zero64<0x112>(x);
  x += dpp_or_zero64<0x114>(x);
  x += dpp_or_zero64<0x118>(x);
  x += dpp_or_zero64<0x142, 0xa>(x);
  x += dpp_or_zero64<0x143, 0xc>(x);
  const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)x, 63);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)((uint64_t)x >> 32), 63);
  return (int64_t)(((uint64_t)hi << 32) | lo);
}

// Totals of a count per Gaussian over the blocks of 256 threads that form them, and over groups of kTotalsGroup blocks.
constexpr int kTotalsGroup = 64;
struct Totals {
  int32_t *rec, *inst;                            // visible records and instances of a block
  unsigned long long *rec_group, *inst_group;     // ... of a group, added up (cleared before)
};
// Called by every thread of a block of 256 with N counts of the 256 items `block`; shared: 4 N ints.
template <class T, int N>
struct Few {
  T v[N];
};
template <int N>
__device__ __forceinline__ void leave_totals(Few<int, N> x, int* shared, Few<int32_t*, N> blocks,
                                             Few<unsigned long long*, N> groups, int64_t block) {
  __syncthreads();  // (a block that comes here again has read its last totals)
#pragma unroll
  for (int i = 0; i < N; ++i) {
    int total;
    wave_excl_scan(x.v[i], total);
    if (__lane_id() == 0) shared[4 * i + (threadIdx.x >> 6)] = total;
  }
  __syncthreads();
  if ((int)threadIdx.x < N) {
#pragma unroll
    for (int i = 0; i < N; ++i) {
      if ((int)threadIdx.x != i) continue;
      const int all = shared[4 * i] + shared[4 * i + 1] + shared[4 * i + 2] + shared[4 * i + 3];
      blocks.v[i][block] = all;
      if (all) atomicAdd(groups.v[i] + block / kTotalsGroup, (unsigned long long)all);
    }
  }
}

__device__ __forceinline__ float read_lane(float x, int l) {
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), l));
}

// Records with more tile instances than this are wide: binning emits them a tile per lane of a wave and lists
// them (frame counters[198], big_rec), and their instance partials are summed by a wave per record before the
// projection backward, which then reads one pre-summed partial for them.
constexpr int kWideRecord = 32;

// Hardware float atomic add without return (global_atomic_add_f32).
__device__ __forceinline__ void atomic_add_f32(float* p, float v) { unsafeAtomicAdd(p, v); }

// View of a global tile: largest v with tile_offset <= tile (n_views <= 64; every lane of the wave asks for the same
// tile).  Past a few views the lanes read an offset each: a scalar loop waits for one load after the other.
__device__ __forceinline__ int view_of_tile(const gs_camera* __restrict__ cams, int n_views, int tile) {
  if (n_views > 4) {
    const int l = lane_id();
    return __popcll(ballot(l < n_views && cams[l < n_views ? l : 0].tile_offset <= tile)) - 1;
  }
  int v = 0;
  for (int i = 1; i < n_views; ++i)
    if (cams[i].tile_offset <= tile) v = i;
  return v;
}

__device__ __forceinline__ float sgnf(float x) { return x > 0.f ? 1.f : (x < 0.f ? -1.f : 0.f); }

// Unless *skip_flags has the overflow bit (the frame's gradients are then undefined): step <- step + 1;
// bias = {1 - beta1^step, sqrt(1 - beta2^step)} (computed in double), bias[2] = 0.  Otherwise bias[2] = 1 and
// nothing else changes; the update kernels then leave every parameter and moment as it is.
struct AdamPrep {
  int64_t* step = nullptr;
  float* bias = nullptr;
  float b1 = 0.f, b2 = 0.f;
  const int32_t* skip_flags = nullptr;
};
__device__ __forceinline__ void adam_prep_step(const AdamPrep& a) {
  if (a.skip_flags && (a.skip_flags[0] & GS_FLAG_INSTANCE_OVERFLOW)) {
    a.bias[2] = 1.f;
    return;
  }
  const int64_t t = a.step[0] + 1;
  a.step[0] = t;
  a.bias[0] = (float)(1.0 - pow((double)a.b1, (double)t));
  a.bias[1] = (float)sqrt(1.0 - pow((double)a.b2, (double)t));
  a.bias[2] = 0.f;
}

// loss[0] = sum of part[0, n), by one workgroup (every thread calls it; a power of two of waves, at most 16).
struct LossSum {
  const float* part = nullptr;
  int n = 0;
  float* loss = nullptr;
};
__device__ __forceinline__ void sum_losses(const LossSum& l, float* shared) {
  const int threads = (int)blockDim.x;
  float v = 0.f;
  for (int i = threadIdx.x; i < l.n; i += threads * 8) {
    float x[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) x[k] = i + k * threads < l.n ? l.part[i + k * threads] : 0.f;
    v += ((x[0] + x[1]) + (x[2] + x[3])) + ((x[4] + x[5]) + (x[6] + x[7]));
  }
  v = wave_sum_last(v);
  if ((threadIdx.x & 63) == 63) shared[threadIdx.x >> 6] = v;
  __syncthreads();
  if (threadIdx.x == 0) {
    float sum = shared[0];
    for (int w = 1; w < threads / 64; ++w) sum += shared[w];
    l.loss[0] = sum;
  }
}

}  // namespace gsk

// ------------------------------------------------------------------ host launchers (one per file)
namespace gs_launch {
hipError_t project(const gs_params& p, const gs_frame& f, const gs_opts& o, hipStream_t s);
// Projection backward; with ls.part the loss is summed in passing (see loss_total).
hipError_t project_bwd(const gs_params& p, const gs_frame& f, const gs_opts& o, const gs_params& g,
                       const gsk::LossSum& ls, hipStream_t s);
size_t scan_scratch_ints(int64_t n);
// Exclusive scan of in[0, n) into out (in place allowed).
hipError_t scan_exclusive(const int32_t* in, int32_t* out, int64_t n, int32_t* scratch, hipStream_t s);
hipError_t fill_i32(int32_t* p, int32_t v, int64_t n, hipStream_t s);
hipError_t fill_f32(float* p, float v, int64_t n, hipStream_t s);
// Binning up to the instance total: the records' first partial slots, visible records sorted by depth, their
// rectangles and the totals of their instance counts, counters[0] = instances (overflow flagged).
hipError_t bin_records(const gs_frame& f, hipStream_t s);
hipError_t emit(const gs_frame& f, hipStream_t s);
size_t sort_scratch_ints(int64_t n);
// the instances by tile; bin_records has cleared this sort's words behind the counters
hipError_t sort_by_tile(const gs_frame& f, int64_t n_sized, const int32_t* count_dev, hipStream_t s);
size_t frame_sort_scratch_ints(int64_t n);  // of a frame's sorts, whose zeroed words lie behind the counters
size_t counter_ints(int64_t n, int64_t rec_cap);  // the frame's counters and the words behind them
gsk::Totals project_totals(const gs_frame& f);
hipError_t clear_project(const gs_frame& f, hipStream_t s);  // counters[0..1] and the totals that the projection adds to
hipError_t sort_pairs(uint64_t* k0, int32_t* v0, uint64_t* k1, int32_t* v1, int64_t n_sized,
                      const int32_t* count_dev, int64_t cap, int key_bits, int32_t* scratch, hipStream_t s);
hipError_t ranges(const gs_frame& f, const uint32_t* keys, int64_t n_sized, const int32_t* count_dev, hipStream_t s);
hipError_t tile_schedule(const gs_frame& f, hipStream_t s);
hipError_t work_items(const gs_frame& f, hipStream_t s);
hipError_t render_fwd(const gs_frame& f, const gs_opts& o, const gs_images& out, hipStream_t s);
hipError_t count_pairs(const gs_frame& f, const gs_opts& o, unsigned long long* counts, hipStream_t s);
hipError_t count_valid(const gs_frame& f, const float* tgt_depth, int64_t max_pixels, hipStream_t s);
// frame loss[0] = sum of the tiles' losses that render_bwd left (tile_losses)
gsk::LossSum tile_losses(const gs_frame& f);
hipError_t loss_total(const gs_frame& f, hipStream_t s);
hipError_t render_bwd(const gs_frame& f, const gs_opts& o, const gs_images* fwd, const gs_loss& l,
                      hipStream_t s);
hipError_t adam(const gs_params& p, const gs_params& g, const gs_params& m, const gs_params& v,
                const gs_adam& a, hipStream_t s);
// SSIM term of the photometric loss: gradient written to g_rgb, value to loss[0] (loss holds 1 + kLossSlots).
hipError_t ssim(const gs_camera* cams_host, const gs_camera* cams_dev, int n_views, const float* rgb,
                const float* tgt, float lambda, float* g_rgb, float* loss, hipStream_t s);
// Opacity pruning: keep flags, their scan and the gather of every kept row (scratch: prune_scratch_ints(n)).
size_t prune_scratch_ints(int64_t n);
hipError_t prune(const gs_params& p, const gs_params& m, const gs_params& v, float thr_logit, const gs_params& op,
                 const gs_params& om, const gs_params& ov, int64_t* n_kept, int32_t* scratch, hipStream_t s);
// Map expansion: filter, voxel cap, neighbour spacing and the new rows (scratch: expand_scratch_ints(M)).
size_t expand_scratch_ints(int64_t M);
hipError_t expand(const gs_params& p, const gs_params& m, const gs_params& v, int64_t n_old, const float* pts,
                  const float* rgb, int64_t M, const gs_camera& cam, const float* vis, float tau, float near_z,
                  float voxel, int cap, float cell, float init_logit, int64_t* n_added, int32_t* scratch,
                  hipStream_t s);
// Spatial (Morton) order: out row k = in row perm[k] for params, m, v (scratch: order_scratch_ints(n)).
size_t order_scratch_ints(int64_t n);
hipError_t spatial_order(const gs_params& p, const gs_params& m, const gs_params& v, const gs_params& op,
                         const gs_params& om, const gs_params& ov, int32_t* perm_out, int32_t* scratch,
                         hipStream_t s);
// Projection backward fused with Adam: params, m, v updated in place; the gradient is written to grads_out
// when it is non-NULL.  The step's count and bias corrections are advanced in passing.
hipError_t project_bwd_adam(const gs_params& p, const gs_frame& f, const gs_opts& o, const gs_params& m,
                            const gs_params& v, const gs_adam& a, const gs_params* grads_out, const gsk::LossSum& ls,
                            hipStream_t s);
}  // namespace gs_launch
