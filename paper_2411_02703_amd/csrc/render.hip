// Per-tile front-to-back compositing of colour, depth and visibility (LVI-GS Section III-B,
// eqs. Cp, Dp, Vp with the alpha of eq. alpha) and its backward.
//
// One workgroup per tile (or depth segment of a long one).  The tile is split into 8x8 sub-tiles of four 4x4-pixel
// blocks.  The tile's depth-sorted list is staged in rounds of a record or two per thread into LDS; the records of the
// next round are fetched into registers while the current one is composited.  Each staged record carries its exact
// pixel rectangle (every pixel outside it has alpha < exp(-1/2)/255, so it would be skipped anyway), and sets its
// bit in the mask of every block its ellipse meets; from the masks each wave counts off the blocks' lists.  Small
// blocks waste few lanes on records that cover part of a sub-tile (coarse pyramid levels hold many sub-pixel
// Gaussians), and a record is skipped only where it cannot contribute, so the result does not depend on them.
//
// The forward gives a lane a pixel: one wave per sub-tile, whose four blocks walk their lists in lock-step, one record
// per step and block, read from LDS by broadcast.  The backward gives a wave one block at a time, its lanes sixteen
// records by four pixel rows (backward_round).
//
// The backward goes through the list in the same front-to-back order as the forward.  With the forward's final
// values C, D, V of a pixel and its upstream gradient g, the gradient of alpha_i is
//   dL/dalpha_i = T_i q_i - (S - P_i) / (1 - alpha_i),   q_i = g . (c_i, d_i, 1),
//   S = g . (C, D, V),  P_i = sum_{j <= i} alpha_j T_j q_j,
// i.e. what lies behind record i is S - P_i.  No per-pixel state is stored between the forward and the
// backward (the fused variant recomputes C, D, V with a first sweep), and the skip / stop decisions are re-evaluated
// with the forward's arithmetic: the same alphas, and transmittances multiplied in the same order.  Per-record partial
// derivatives are summed in LDS and stored as the partials of the tile's instances once per round.
#include "common.h"

namespace {

using gsk::DevOpts;

// A tile's geometry: 8x8 sub-tiles, one wave each, walked as four 4x4-pixel blocks.
template <int TW, int TH, int DEPTH_, int BATCH_ = TW * TH * DEPTH_>
struct Geo {
  static constexpr int SX = TW / 8;            // sub-tiles across
  static constexpr int SY = TH / 8;            // sub-tiles down
  static constexpr int NW = SX * SY;           // waves per tile
  static constexpr int NT = 64 * NW;           // threads = pixels of the tile
  static constexpr int DEPTH = DEPTH_;         // records staged per thread
  static constexpr int BATCH = BATCH_;         // records staged per round (fewer than NT: by the first threads)
  static constexpr int MC = BATCH / 32;        // 32-bit mask words per block
  static constexpr int NB = 4 * NW;            // blocks per tile
  static_assert(TW % 8 == 0 && TH % 8 == 0 && NW >= 1 && NW <= 4, "tile shape");
  static_assert(DEPTH == 1 || DEPTH == 2, "batch depth");
  static_assert(BATCH <= NT * DEPTH && BATCH % 64 == 0, "records per round");
};

// The backward's geometry: rounds of 128 records whatever the forward uses.  Each wave sums its records' gradients
// in its own LDS rows (40 bytes a record), which set the round's size: 128 leaves four waves a SIMD at every tile
// shape (three at 16x16 and 32x8 where the forward stages two records a thread, whose round shares the block's LDS).
template <int TW, int TH>
using BGeo = Geo<TW, TH, 1, (TW * TH >= 128 ? 128 : 64)>;

// The forward's workgroup state: one round of staged records.  Slot BATCH of the records is an empty one (opacity 0):
// it contributes nowhere, and pads the blocks' lists.
template <class G>
struct Stage {
  float4 A[G::BATCH + 1], B[G::BATCH + 1], C[G::BATCH + 1];
  uint64_t odd[G::BATCH / 64];                    // staged records that need the whole of eval_pair (see scatter)
  alignas(16) uint32_t bm[G::MC][G::NB];          // per block: staged records that can reach it
  alignas(16) uint16_t list[G::NW][4][G::BATCH + 16];  // per block: those records in order, as byte offsets of A
  int alive[G::NW];                               // per wave: a pixel is still live
};

// The backward's workgroup state: the staged round, its records' gradient sums, and the state of the tile's pixels
// (blocks of 4x4 pixels, sixteen consecutive entries a block, row by row).  The last slot of the records and of the
// sums is for lanes without a record.
template <class G>
struct BwdStage {
  float4 A[G::BATCH + 1], B[G::BATCH + 1];
  float2 C[G::BATCH + 1];                      // green, blue
  uint64_t odd[G::BATCH / 64];                 // as in Stage
  alignas(16) uint32_t bm[G::MC][G::NB];
  int alive[G::NW];
  int next;                                    // the next block of the tile that no wave has taken
  alignas(16) float acc8[G::NW][G::BATCH + 1][8];  // per wave: each record's sums 0, 4, 1, 5, 2, 6, 3, 7 (flush_grads)
  alignas(16) float acc2[G::NW][G::BATCH + 1][2];  // and 8, 9
  alignas(16) uint8_t list[G::NW][G::BATCH + 48];  // per wave: the staged records of the block it works on, in order
  alignas(16) float T[G::NT];                  // transmittance so far (0: pixel outside the image or ended before)
  alignas(16) float R[G::NT];                  // S - P: the upstream-weighted sum of what still lies behind
  alignas(16) float g[4][G::NT], gv[G::NT];    // upstream gradient: red, green, blue, depth; visibility
};

struct TileCtx {
  int view, W, H, tx0, ty0;  // view and tile origin (pixels)
  int px, py;                // this lane's pixel
  int wave, lane;
  int64_t pix_off;
  float weight;
  bool inside;               // pixel inside the image
};

// Geometry of this thread's pixel in global tile `tile`.
template <class G>
__device__ __forceinline__ void tile_at(const gs_camera* __restrict__ cams, int V, int tile, TileCtx& t) {
  t.view = gsk::view_of_tile(cams, V, tile);
  const gs_camera& c = cams[t.view];
  const int lt = tile - c.tile_offset;
  const int tyi = lt / c.tiles_x, txi = lt - tyi * c.tiles_x;
  t.wave = threadIdx.x >> 6;
  t.lane = threadIdx.x & 63;
  t.W = c.width;
  t.H = c.height;
  t.tx0 = txi * (8 * G::SX);
  t.ty0 = tyi * (8 * G::SY);
  // lanes of a block are consecutive; blocks of a wave in row-major order over its sub-tile
  const int r = t.lane >> 4, p = t.lane & 15;
  t.px = t.tx0 + (t.wave % G::SX) * 8 + (r & 1) * 4 + (p & 3);
  t.py = t.ty0 + (t.wave / G::SX) * 8 + (r >> 1) * 4 + (p >> 2);
  t.pix_off = c.pixel_offset;
  t.weight = fmaxf(c.loss_weight, 0.f);  // an inactive view (weight < 0) adds nothing to the loss
  t.inside = t.px < t.W && t.py < t.H;
}

// Workgroup b composites tile order[b]: tiles in descending order of list length, so the longest start first.
template <class G>
__device__ __forceinline__ bool tile_setup(const gs_camera* __restrict__ cams, int V, int n_tiles,
                                           const int32_t* __restrict__ order, TileCtx& t, int& tile) {
  if ((int)blockIdx.x >= n_tiles) return false;
  tile = order[blockIdx.x];
  tile_at<G>(cams, V, tile, t);
  return true;
}

// One record at one pixel: returns false if skipped (power > 0 or alpha < alpha_min).  The operation
// sequence is fixed (contraction off, explicit fma) so that every kernel and every tile shape computes the
// same bits for the same (record, pixel) pair.  Everything is computed whatever the outcome (no branch: in a
// lock-step walk some lane of the wave nearly always takes every path, and the branches only add exec-mask
// work); G and alpha are meaningful only where the result is true.
// WHOLE = false leaves out what cannot happen for a record that is not odd (see scatter): a positive power and an
// alpha above alpha_max.  The bits are the same; on this chip a compare, a minimum and a select each cost as much
// as two multiplications.
template <bool WHOLE>
__device__ __forceinline__ bool eval_pair(const float4& A, const float4& B, float fx, float fy, const DevOpts& op,
                                          float& alpha, bool& clamped, float& dx, float& dy) {
#pragma clang fp contract(off)
  dx = A.x - fx;
  dy = A.y - fy;
  const float adx2 = (B.x * dx) * dx;
  const float quad = __builtin_fmaf(B.z * dy, dy, adx2);  // a dx^2 + c dy^2
  const float bxy = (B.y * dx) * dy;
  const float power = __builtin_fmaf(-0.5f, quad, -bxy);  // -(a dx^2 + c dy^2)/2 - b dx dy
  alpha = A.w * __expf(power);
  if (!WHOLE) {
    clamped = false;
    return alpha >= op.alpha_min;
  }
  clamped = alpha > op.alpha_max;
  alpha = fminf(alpha, op.alpha_max);  // the same value as clamped ? alpha_max : alpha (alpha is finite)
  return !(power > 0.f) && alpha >= op.alpha_min;
}

// The pixel rectangle in a record's last two words.
__device__ __forceinline__ void unpack_rect(float rect_x, float rect_y, int& x0, int& x1, int& y0, int& y1) {
  const int a = __float_as_int(rect_x), b = __float_as_int(rect_y);
  x0 = a & 0xffff;
  x1 = (int)((unsigned)a >> 16);
  y0 = b & 0xffff;
  y1 = (int)((unsigned)b >> 16);
}

// Records of the tile list in flight, per thread: the round held in registers (ids r, data A, B, C) and the ids of
// the round after it (rn).
// Loads are unconditional (past the end of the list its last record is read again: never used, but valid data), so
// nothing waits on them until the round is written to LDS.
template <int DEPTH>
__device__ __forceinline__ void fetch_records(const float4* __restrict__ rec, const int (&r)[DEPTH],
                                              float4 (&A)[DEPTH], float4 (&B)[DEPTH], float4 (&C)[DEPTH]) {
#pragma unroll
  for (int k = 0; k < DEPTH; ++k) {
    const float4* p = rec + 3 * (int64_t)r[k];
    A[k] = p[0];
    B[k] = p[1];
    C[k] = p[2];
  }
}

template <class G, int DEPTH>
__device__ __forceinline__ void fetch_ids(const int32_t* __restrict__ vals, int first, int end, int (&ids)[DEPTH]) {
#pragma unroll
  for (int k = 0; k < DEPTH; ++k) {
    const int i = min(first + k * G::NT + (int)threadIdx.x, end - 1);
    ids[k] = i >= 0 ? vals[i] : 0;
  }
}

// Write the round held in registers into LDS, then start fetching the round after it (its ids were fetched
// one round earlier) and the ids of the round after that.
template <class G, int DEPTH>
__device__ __forceinline__ void stage_round(Stage<G>& s, const float4* __restrict__ rec,
                                            const int32_t* __restrict__ vals, int b0, int end, int (&r)[DEPTH],
                                            int (&rn)[DEPTH], float4 (&A)[DEPTH], float4 (&B)[DEPTH],
                                            float4 (&C)[DEPTH]) {
#pragma unroll
  for (int k = 0; k < DEPTH; ++k) {
    const int j = k * G::NT + (int)threadIdx.x;
    s.A[j] = A[k];
    s.B[j] = B[k];
    s.C[j] = C[k];
    r[k] = rn[k];
  }
  fetch_records<DEPTH>(rec, r, A, B, C);
  fetch_ids<G, DEPTH>(vals, b0 + 2 * G::BATCH, end, rn);
}

// End of a round: every wave publishes whether it still has a live pixel, then the workgroup meets.  Returns
// whether any pixel of the tile is live (the same answer in every thread).
template <class G, class St>
__device__ __forceinline__ bool round_barrier(St& s, const TileCtx& t, bool live) {
  const bool wl = __builtin_amdgcn_ballot_w64(live) != 0;
  if (t.lane == 0) s.alive[t.wave] = wl;
  __syncthreads();
  bool any = false;
#pragma unroll
  for (int w = 0; w < G::NW; ++w) any |= s.alive[w] != 0;
  return any;
}

// Clear the block masks.
template <class G, class St>
__device__ __forceinline__ void clear_masks(St& s) {
  for (int i = threadIdx.x; i < G::MC * G::NB; i += G::NT) (&s.bm[0][0])[i] = 0u;
}

// Set a staged record (slot j of the round) in the masks of the blocks it can reach.  Blocks are numbered
// wave-major (the wave's sub-tile, then row-major inside it).  Returns whether the record is odd: its conic so
// thin that the FP32 power might come out positive, or its opacity close enough to alpha_max to be clamped.  (With
// det > 1e-3 a c, |b dx dy| stays below 0.9995 of half of a dx^2 + c dy^2, so the power is negative by far more
// than its rounding; and exp of it is at most 1.)
//
// A record passes the skip test at a pixel only where alpha = o G >= alpha_min, i.e. inside its ellipse
// q(d) = a dx^2 + 2 b dx dy + c dy^2 <= k = 2 ln(o / alpha_min).  For each pixel row of the record's rectangle
// the ellipse meets the row's line of pixel centres in an x-interval
//   [(-b dy - sqrt(a k - det dy^2)) / a, (-b dy + sqrt(a k - det dy^2)) / a],   det = a c - b^2,
// and a block is marked iff one of its rows holds a pixel centre in that interval (the union over the block's
// rows is taken as one interval, a superset).  k is widened by 1% + 0.01: with det > 1e-3 a c (else the whole
// rectangle is kept) the FP32 power of the walk is within 0.1% of q, so no pair the walk would accept is
// pruned and the result does not change (the hardware square root and logarithm used here err by a few ulp,
// far inside that widening).
template <class G>
__device__ __forceinline__ bool scatter(uint32_t (*bm)[G::NB], int j, const float4& A, const float4& B, float rect_x,
                                        float rect_y, const TileCtx& t, const DevOpts& op) {
  constexpr int GX = 2 * G::SX, GY = 2 * G::SY;  // blocks across and down the tile
  const float ca = B.x, cb = B.y, cc = B.z;
  const float det = ca * cc - cb * cb;
  const bool cull = det > 1e-3f * ca * cc;  // else the whole rectangle is kept
  const bool odd = !cull || A.w > 0.999f * op.alpha_max;
  int x0, x1, y0, y1;
  unpack_rect(rect_x, rect_y, x0, x1, y0, y1);
  const int gx0 = max(x0 - t.tx0, 0) >> 2, gx1 = min(x1 - t.tx0, 8 * G::SX - 1) >> 2;
  const int gy0 = max(y0 - t.ty0, 0) >> 2, gy1 = min(y1 - t.ty0, 8 * G::SY - 1) >> 2;
  if (x1 < t.tx0 || y1 < t.ty0 || gx0 >= GX || gy0 >= GY) return odd;
  const float kq = 2.f * __logf(A.w / op.alpha_min) * 1.01f + 0.01f;
  const float inv_a = 1.f / ca, ak = ca * kq;
  const uint32_t bit = 1u << (j & 31);
  const int wd = j >> 5;
  for (int gy = gy0; gy <= gy1; ++gy) {
    int cx0 = gx0, cx1 = gx1;
    if (cull) {
      // pixel rows of this block row inside the record's rectangle
      const int r0 = max(t.ty0 + gy * 4, y0), r1 = min(t.ty0 + gy * 4 + 3, y1);
      int lo = 1 << 30, hi = -(1 << 30);
      for (int yy = r0; yy <= r1; ++yy) {
        const float dy = (float)yy + 0.5f - A.y;
        const float disc = ak - det * dy * dy;
        if (disc < 0.f) continue;
        const float sq = __builtin_amdgcn_sqrtf(disc);  // the hardware root (~1 ulp): k is widened far more
        // pixel columns whose centres px + 0.5 lie in [A.x + xl, A.x + xr]
        const float xl = A.x + (-cb * dy - sq) * inv_a - 0.5f, xr = A.x + (-cb * dy + sq) * inv_a - 0.5f;
        lo = min(lo, (int)ceilf(fminf(fmaxf(xl, -1.f), 65536.f)));
        hi = max(hi, (int)floorf(fminf(fmaxf(xr, -1.f), 65536.f)));
      }
      if (lo > hi) continue;
      cx0 = max(gx0, (max(lo, t.tx0) - t.tx0) >> 2);
      cx1 = min(gx1, (hi - t.tx0) >> 2);
      if (hi < t.tx0) continue;
    }
    for (int gx = cx0; gx <= cx1; ++gx) atomicOr(&bm[wd][((gy >> 1) * G::SX + (gx >> 1)) * 4 + (gy & 1) * 2 + (gx & 1)], bit);
  }
  return odd;
}

// One record of the forward at this lane's pixel.  STOP applies the stop rule: a pixel ends before the pair that would
// take T below t_min, and keeps its T with the sign set, which fails every later comparison with t_min.
template <bool STOP, bool WHOLE>
__device__ __forceinline__ void forward_step(const float4& A, const float4& B, const float2& C, float fx, float fy,
                                             const DevOpts& op, float& T, float& Cr, float& Cg, float& Cb, float& D,
                                             float& Vs) {
#pragma clang fp contract(off)
  float alpha, dx, dy;
  bool cl;
  const bool ok = eval_pair<WHOLE>(A, B, fx, fy, op, alpha, cl, dx, dy);
  // a pair that does not contribute adds w = 0 and multiplies T by 1 (colours, depth and T are finite and the sums
  // non-negative, so every sum keeps its bits)
  const float am = ok ? alpha : 0.f;
  float w = am * T;
  const float Tn = T * (1.f - am);
  if (STOP) {
    const bool go = Tn >= op.t_min;
    w = go ? w : 0.f;
    T = go ? Tn : -fabsf(T);
  } else {
    T = Tn;
  }
  Cr = __builtin_fmaf(w, B.w, Cr);
  Cg = __builtin_fmaf(w, C.x, Cg);
  Cb = __builtin_fmaf(w, C.y, Cb);
  D = __builtin_fmaf(w, A.z, D);
  Vs = Vs + w;
}

// Steps of one round: the wave's four blocks (a 16-lane row each) walk their lists in lock-step, one record per step
// and block, read from LDS by broadcast one step ahead.  Shorter lists end in the empty record.  n is even.
template <class G, bool STOP, bool WHOLE>
__device__ __forceinline__ void forward_round(const Stage<G>& s, const uint16_t* list, int n, float fx, float fy,
                                              const DevOpts& op, float& T, float& Cr, float& Cg, float& Cb, float& D,
                                              float& Vs) {
  auto get = [&](uint32_t o, float4& A, float4& B, float2& C) {
    A = *reinterpret_cast<const float4*>(reinterpret_cast<const char*>(s.A) + o);
    B = *reinterpret_cast<const float4*>(reinterpret_cast<const char*>(s.B) + o);
    C = *reinterpret_cast<const float2*>(reinterpret_cast<const char*>(s.C) + o);
  };
  float4 A0, B0, A1, B1;
  float2 C0, C1;
  get(list[0], A0, B0, C0);
  uint32_t o1 = list[1], o0 = list[2];
#pragma unroll 1
  for (int p = 0; p < n; p += 2) {
    get(o1, A1, B1, C1);
    o1 = list[p + 3];
    forward_step<STOP, WHOLE>(A0, B0, C0, fx, fy, op, T, Cr, Cg, Cb, D, Vs);
    get(o0, A0, B0, C0);
    o0 = list[p + 4];
    forward_step<STOP, WHOLE>(A1, B1, C1, fx, fy, op, T, Cr, Cg, Cb, D, Vs);
    if (STOP && __builtin_amdgcn_ballot_w64(T >= op.t_min) == 0) break;  // every pixel of the wave has ended
  }
}

// Forward walk of records [rg.x, rg.y) for this lane's pixel from transmittance T (in/out), adding to the
// partial sums: rounds of staged records (with the next round in flight), each wave walking its blocks' lists.  STOP
// applies the stop rule; without it the walk multiplies on (the transmittance product of a depth segment).
template <class G, bool STOP>
__device__ __forceinline__ void forward_walk(Stage<G>& s, const float4* __restrict__ rec,
                                             const int32_t* __restrict__ vals, int2 rg, const TileCtx& t,
                                             const DevOpts& op, bool live, float& T, float& Cr, float& Cg, float& Cb,
                                             float& D, float& Vs) {
  constexpr int DEPTH = G::DEPTH;
  const float fx = (float)t.px + 0.5f, fy = (float)t.py + 0.5f;
  if (STOP && !live) T = -T;
  int fr[DEPTH], frn[DEPTH];
  float4 fA[DEPTH], fB[DEPTH], fC[DEPTH];
  fetch_ids<G, DEPTH>(vals, rg.x, rg.y, fr);
  fetch_ids<G, DEPTH>(vals, rg.x + G::BATCH, rg.y, frn);
  fetch_records<DEPTH>(rec, fr, fA, fB, fC);
  if (threadIdx.x == 0) s.A[G::BATCH] = s.B[G::BATCH] = s.C[G::BATCH] = make_float4(0.f, 0.f, 0.f, 0.f);
  uint16_t(*list)[G::BATCH + 16] = s.list[t.wave];
  for (int b0 = rg.x;; b0 += G::BATCH) {
    if (!(round_barrier<G>(s, t, STOP ? T >= op.t_min : live) && b0 < rg.y)) break;
    clear_masks<G>(s);
    stage_round<G, DEPTH>(s, rec, vals, b0, rg.y, fr, frn, fA, fB, fC);
    // every entry of the lists past their ends is the empty record
    for (int i = t.lane; i < 4 * (G::BATCH + 16) / 8; i += 64) {
      constexpr uint32_t e = G::BATCH * 16 * 0x10001u;
      reinterpret_cast<uint4*>(list)[i] = make_uint4(e, e, e, e);
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < DEPTH; ++k) {
      const int j = k * G::NT + (int)threadIdx.x;
      bool odd = false;
      if (b0 + j < rg.y) odd = scatter<G>(s.bm, j, s.A[j], s.B[j], s.C[j].z, s.C[j].w, t, op);
      const uint64_t m = __builtin_amdgcn_ballot_w64(odd);
      if (t.lane == 0) s.odd[j >> 6] = m;
    }
    __syncthreads();
    int n[4] = {0, 0, 0, 0};
    uint64_t odd = 0;
#pragma unroll
    for (int h = 0; h < G::BATCH / 64; ++h) {
      const uint4 w4 = *reinterpret_cast<const uint4*>(&s.bm[2 * h + (t.lane >> 5)][4 * t.wave]);
      const uint32_t wb[4] = {w4.x, w4.y, w4.z, w4.w};
      uint64_t all = 0;
#pragma unroll
      for (int b = 0; b < 4; ++b) {
        const bool bit = (wb[b] >> (t.lane & 31)) & 1u;
        const uint64_t m = __builtin_amdgcn_ballot_w64(bit);
        if (bit) list[b][gsk::rank_in(m, n[b])] = (uint16_t)((64 * h + t.lane) * 16);
        n[b] += __popcll(m);
        all |= m;
      }
      odd |= all & gsk::uniform64(s.odd[h]);
    }
    const int steps = (max(max(n[0], n[1]), max(n[2], n[3])) + 1) & ~1;
    if (steps == 0) continue;
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");  // the lists are read by this wave's other lanes only
    const uint16_t* mine = list[t.lane >> 4];
    if (odd)
      forward_round<G, STOP, true>(s, mine, steps, fx, fy, op, T, Cr, Cg, Cb, D, Vs);
    else
      forward_round<G, STOP, false>(s, mine, steps, fx, fy, op, T, Cr, Cg, Cb, D, Vs);
  }
  if (STOP) T = fabsf(T);
}

// Forward sweep of one whole tile for this lane's pixel (forward kernel and fused backward).
template <class G>
__device__ __forceinline__ void forward_sweep(Stage<G>& s, const float4* __restrict__ rec,
                                              const int32_t* __restrict__ vals, int2 rg, const TileCtx& t,
                                              const DevOpts& op, float& T, float& Cr, float& Cg, float& Cb,
                                              float& D, float& Vs) {
  T = 1.f;
  Cr = Cg = Cb = D = Vs = 0.f;
  forward_walk<G, true>(s, rec, vals, rg, t, op, t.inside, T, Cr, Cg, Cb, D, Vs);
}

// Final values of this lane's pixel (background behind transmittance T) into the planar images.
__device__ __forceinline__ void write_pixel(const TileCtx& t, const DevOpts& op, float T, float Cr, float Cg, float Cb,
                                            float D, float Vs, float* __restrict__ out_rgb,
                                            float* __restrict__ out_depth, float* __restrict__ out_vis) {
  if (!t.inside) return;
  const int64_t P = (int64_t)t.W * t.H;
  const int64_t i = (int64_t)t.py * t.W + t.px;
  out_rgb[3 * t.pix_off + i] = __builtin_fmaf(T, op.bg[0], Cr);
  out_rgb[3 * t.pix_off + P + i] = __builtin_fmaf(T, op.bg[1], Cg);
  out_rgb[3 * t.pix_off + 2 * P + i] = __builtin_fmaf(T, op.bg[2], Cb);
  out_depth[t.pix_off + i] = D;
  out_vis[t.pix_off + i] = Vs;
}

template <int TW, int TH, int DEPTH>
__global__ __launch_bounds__(TW * TH, 6) void k_render_fwd(const float4* __restrict__ rec,
                                                        const int32_t* __restrict__ vals,
                                                        const int2* __restrict__ range,
                                                        const gs_camera* __restrict__ cams, int V, int n_tiles,
                                                        const int32_t* __restrict__ order, DevOpts op,
                                                        float* __restrict__ out_rgb, float* __restrict__ out_depth,
                                                        float* __restrict__ out_vis) {
  using G = Geo<TW, TH, DEPTH>;
  __shared__ Stage<G> s;
  TileCtx t;
  int tile;
  if (!tile_setup<G>(cams, V, n_tiles, order, t, tile)) return;
  float T, Cr, Cg, Cb, D, Vs;
  forward_sweep<G>(s, rec, vals, range[tile], t, op, T, Cr, Cg, Cb, D, Vs);
  write_pixel(t, op, T, Cr, Cg, Cb, D, Vs, out_rgb, out_depth, out_vis);
}

struct BwdArgs {
  const float* fwd_rgb;
  const float* fwd_depth;
  const float* fwd_vis;
  const float* g_rgb;
  const float* g_depth;
  const float* g_vis;
  const float* tgt_rgb;
  const float* tgt_depth;
  const int32_t* n_valid;  // per view
  float lambda_d;
  float lambda_ssim;  // loss mode: the L1 colour term takes 1 - lambda_ssim; g_rgb (if given) is added
  float* ipart;              // [slot][12]: instance partials, each record's instances one run
  const int32_t* rec_slot;   // first slot of each record; a record's tiles follow row by row
  int64_t capacity;          // slots stored (a slot at or past it belongs to an overflowed frame)
  float* loss_part;          // [n_tiles]: each tile's loss, by schedule position
};

// Depth segments of the fused backward (see k_bwd_sums).
struct SegArgs {
  const int4* items;        // {tile, segment, first slot of the tile or -1, schedule position}
  const int32_t* counters;  // [192] items, [193] slots of split tiles, [194] split tiles
  const int32_t* order;
  const int32_t* seg_count;
  const int32_t* seg_first;
  float* seg;               // [slot][6][NT]
  float* split;             // [split tile][12][NT]
  int len;                  // records per segment
  bool whole;               // k_bwd_sums runs the forward of whole tiles too
};

// What the upstream gradient of this lane's pixel is formed from: the targets (loss mode) or the image gradients.  Read
// before the forward sweep, which hides the loads.
struct Upstream {
  float r = 0.f, g = 0.f, b = 0.f, d = 0.f, v = 0.f;  // loss mode: target colour and depth; else the gradient
  float xr = 0.f, xg = 0.f, xb = 0.f;                 // loss mode: the gradient of a further colour term (gs_ssim's)
};

template <bool LOSS>
__device__ __forceinline__ Upstream load_upstream(const TileCtx& t, const BwdArgs& a) {
  Upstream u;
  if (!t.inside) return u;
  const int64_t P = (int64_t)t.W * t.H;
  const int64_t pi = (int64_t)t.py * t.W + t.px, ci = 3 * t.pix_off + pi, di = t.pix_off + pi;
  if (LOSS) {
    u.r = a.tgt_rgb[ci];
    u.g = a.tgt_rgb[ci + P];
    u.b = a.tgt_rgb[ci + 2 * P];
    u.d = a.tgt_depth[di];
    if (a.g_rgb) {
      u.xr = a.g_rgb[ci];
      u.xg = a.g_rgb[ci + P];
      u.xb = a.g_rgb[ci + 2 * P];
    }
  } else {
    if (a.g_rgb) {
      u.r = a.g_rgb[ci];
      u.g = a.g_rgb[ci + P];
      u.b = a.g_rgb[ci + 2 * P];
    }
    if (a.g_depth) u.d = a.g_depth[di];
    if (a.g_vis) u.v = a.g_vis[di];
  }
  return u;
}

// Upstream gradient of this pixel from its final values: the L1 loss gradient (eqs. Lc, Ld, L) or the
// given image gradients.  Adds the pixel's loss to loss_acc.
template <bool LOSS>
__device__ __forceinline__ void pixel_upstream(const TileCtx& t, const BwdArgs& a, const Upstream& u, float Cf, float Gf,
                                               float Bf, float Df, float& gr, float& gg, float& gb, float& gd,
                                               float& gv, float& loss_acc) {
  if (!LOSS) {
    gr = u.r;
    gg = u.g;
    gb = u.b;
    gd = u.d;
    gv = u.v;
    return;
  }
  gr = gg = gb = gd = gv = 0.f;
  if (!t.inside) return;
  const float wrgb = t.weight * (1.f - a.lambda_ssim) / (3.f * (float)((int64_t)t.W * t.H));
  const int M = a.n_valid[t.view];
  const float wd = M > 0 ? t.weight * a.lambda_d / (float)M : 0.f;
  const float er = Cf - u.r, eg = Gf - u.g, eb = Bf - u.b;
  gr = wrgb * gsk::sgnf(er) + u.xr;
  gg = wrgb * gsk::sgnf(eg) + u.xg;
  gb = wrgb * gsk::sgnf(eb) + u.xb;
  loss_acc += wrgb * (fabsf(er) + fabsf(eg) + fabsf(eb));
  if (u.d > 0.f) {
    const float ed = Df - u.d;
    gd = wd * gsk::sgnf(ed);
    loss_acc += wd * fabsf(ed);
  }
}

// Stores the workgroup's loss as that of the tile at schedule position `at` (every thread must call it).  Plain stores,
// added up by sum_losses: atomics into one or two cache lines take about 5 ns each whichever words they hit, which
// had made frames of many short tiles wait for them (22 k tiles: 123 us).
template <class G>
__device__ __forceinline__ void store_loss(const TileCtx& t, const BwdArgs& a, int at, float loss_acc) {
  __shared__ float part[G::NW];
  const float ls = gsk::wave_sum_last(loss_acc);
  if (t.lane == 63) part[t.wave] = ls;
  __syncthreads();
  if (threadIdx.x == 0) {
    float sum = part[0];
#pragma unroll
    for (int w = 1; w < G::NW; ++w) sum += part[w];
    a.loss_part[at] = sum;
  }
}

__global__ __launch_bounds__(1024) void k_loss_total(gsk::LossSum l) {
  __shared__ float wsum[16];
  gsk::sum_losses(l, wsum);
}

// Partial slot of the instance of a record (first slot and pixel rectangle) in the tile at pixel origin (tx0, ty0): the
// record's first slot plus the tile's index in the record's tile rectangle, row by row (the emission order).
template <class G>
__device__ __forceinline__ int inst_slot(int first, float rect_x, float rect_y, const TileCtx& t) {
  constexpr int TWp = 8 * G::SX, THp = 8 * G::SY;
  int x0, x1, y0, y1;
  unpack_rect(rect_x, rect_y, x0, x1, y0, y1);
  const int rx0 = x0 / TWp, rx1 = x1 / TWp, ry0 = y0 / THp;
  return first + (t.ty0 / THp - ry0) * (rx1 - rx0 + 1) + (t.tx0 / TWp - rx0);
}

// Store the LDS sums of this thread's staged record (slot j of the round) as the partial of its instance at slot q.
// The sums are, over the record's contributing pixels (d = mean - pixel centre,
// dq = dL/dalpha alpha):
//   dq, dq dx, dq dy, dq dx^2, dq dx dy, dq dy^2, w g_r, w g_g, w g_b, w g_d;
// with the conic (a, b, c) of the record, power = -(a dx^2 + c dy^2)/2 - b dx dy and alpha = o exp(power) give
//   dL/dmean = -(a S_x + b S_y, b S_x + c S_y),  dL/d(a, b, c) = -(S_xx / 2, S_xy, S_yy / 2),  dL/do = S / o.
// Plain stores: every instance has exactly one writer (its tile or depth segment), so nothing is accumulated
// in HBM.
template <class G>
__device__ __forceinline__ void flush_grads(BwdStage<G>& s, int j, int q, float* __restrict__ ipart,
                                            int64_t capacity) {
  float v[10];
#pragma unroll
  for (int w = 0; w < G::NW; ++w) {
    const float4* p = reinterpret_cast<const float4*>(s.acc8[w][j]);
    const float4 x = p[0], y = p[1];
    const float2 z = *reinterpret_cast<const float2*>(s.acc2[w][j]);
    const float u[10] = {x.x, x.z, y.x, y.z, x.y, x.w, y.y, y.w, z.x, z.y};
#pragma unroll
    for (int i = 0; i < 10; ++i) v[i] = w ? v[i] + u[i] : u[i];
  }
  if (q < 0 || q >= capacity) return;
  const float4 B = s.B[j];
  float4* dst = reinterpret_cast<float4*>(ipart) + 3 * (int64_t)q;
  dst[0] = make_float4(-(B.x * v[1] + B.y * v[2]), -(B.y * v[1] + B.z * v[2]), -0.5f * v[3], -v[4]);
  dst[1] = make_float4(-0.5f * v[5], v[0] / s.A[j].w, v[6], v[7]);
  dst[2] = make_float4(v[8], v[9], 0.f, 0.f);
}

// Zero partials for the instances [b0, end) that the walk never staged (every pixel ended before them).
template <class G>
__device__ __forceinline__ void zero_grads(const float4* __restrict__ rec, const int32_t* __restrict__ vals,
                                           const TileCtx& t, float* __restrict__ ipart,
                                           const int32_t* __restrict__ rec_slot, int64_t capacity, int b0, int end) {
  const float4 z = make_float4(0.f, 0.f, 0.f, 0.f);
  for (int p = b0 + (int)threadIdx.x; p < end; p += G::NT) {
    const int64_t r = vals[p];
    const float4 C = rec[3 * r + 2];
    const int q = inst_slot<G>(rec_slot[r], C.z, C.w, t);
    if (q < 0 || q >= capacity) continue;
    float4* dst = reinterpret_cast<float4*>(ipart) + 3 * (int64_t)q;
    dst[0] = z;
    dst[1] = z;
    dst[2] = z;
  }
}

using f32x4 = __attribute__((ext_vector_type(4))) float;

// Products over each 16-lane row, left to right, of four independent values: lane l ends with
// (((x_0 om_1) om_2) ...) om_l, rounded after every factor as the forward's walk rounds it.  Every step multiplies lane
// l - 1's value by om_l; lane 0 has no source and, in the DPP form without bound_ctrl, keeps its value, and after step s
// lanes up to s hold their final product, which further steps form again.  (The four instructions of a step alternate, so
// every DPP read comes at least three instructions after the write of its register.)
#define GS_ROW_STEP                                                       \
  "v_mul_f32_dpp %0, %0, %4 row_shr:1 row_mask:0xf bank_mask:0xf\n\t" \
  "v_mul_f32_dpp %1, %1, %5 row_shr:1 row_mask:0xf bank_mask:0xf\n\t" \
  "v_mul_f32_dpp %2, %2, %6 row_shr:1 row_mask:0xf bank_mask:0xf\n\t" \
  "v_mul_f32_dpp %3, %3, %7 row_shr:1 row_mask:0xf bank_mask:0xf\n\t"
__device__ __forceinline__ void row_products(float (&x)[4], const float (&om)[4]) {
  asm("s_nop 1\n\t" GS_ROW_STEP GS_ROW_STEP GS_ROW_STEP GS_ROW_STEP GS_ROW_STEP GS_ROW_STEP GS_ROW_STEP GS_ROW_STEP
          GS_ROW_STEP GS_ROW_STEP GS_ROW_STEP GS_ROW_STEP GS_ROW_STEP GS_ROW_STEP GS_ROW_STEP "s_nop 1"
      : "+v"(x[0]), "+v"(x[1]), "+v"(x[2]), "+v"(x[3])
      : "v"(om[0]), "v"(om[1]), "v"(om[2]), "v"(om[3]));
}
#undef GS_ROW_STEP

// Sums over the four 16-lane rows of the wave, spread over the rows: rows 0, 1, 2, 3 get the sum of a, b, c, d.
__device__ __forceinline__ float row_reduce4(float a, float b, float c, float d) {
  auto half = [](float x, float y) {  // rows 0, 1: x over the wave's halves, rows 2, 3: y
    const auto p = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(y), false, false);
    return __uint_as_float(p[0]) + __uint_as_float(p[1]);
  };
  const float x = half(a, c), y = half(b, d);
  const auto p = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(y), false, false);
  return __uint_as_float(p[0]) + __uint_as_float(p[1]);
}

// The same of two values: rows 0 and 1 get the sum of a, rows 2 and 3 that of b.
__device__ __forceinline__ float row_reduce2(float a, float b) {
  auto p = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
  const uint32_t x = __float_as_uint(__uint_as_float(p[0]) + __uint_as_float(p[1]));
  p = __builtin_amdgcn_permlane16_swap(x, x, false, false);
  return __uint_as_float(p[0]) + __uint_as_float(p[1]);
}

// Whether a pixel of the block is still live (a lane holds four of them; T >= 0, so its bits compare like integers).
__device__ __forceinline__ bool any_live(const f32x4& T, const DevOpts& op) {
  const int m = max(max(__float_as_int(T[0]), __float_as_int(T[1])), max(__float_as_int(T[2]), __float_as_int(T[3])));
  return __builtin_amdgcn_ballot_w64(__int_as_float(m) >= op.t_min) != 0;
}

// One staged round of the backward: the waves take the tile's 4x4 blocks in turn, each block with all 64 lanes: lane
// l holds record l % 16 of sixteen records of the block's list and the four pixels of the block's row l / 16.
//   * The list: the wave counts off the block's mask into an index list, so that sixteen lanes always hold sixteen
//     records that reach the block, however sparse the mask; the last sixteen are filled up with the empty record,
//     whose opacity is 0.
//   * Transmittances: with om = 1 - alpha (1 for a pair that does not contribute), the transmittance behind a record is
//     the pixel's T times om over the lanes up to its own, multiplied left to right as in the forward, so that every
//     weight w and every stop has the forward's bits.  The gradient needs S less the weights in front of a record, and a
//     weight that differs from the one in S leaves its difference behind: with a scan in four steps, which multiplies in
//     another order and takes 3 to 5% less of a step, the error of dL/dalpha over lists of 4 to 200 records was 0.95 to
//     1.08 times that of a walk pair by pair, and 4.6 times at 200 equal alphas, where the roundings of the one order
//     all go one way; as it is 0.88 to 1.01 times (a float32 model of both sweeps against 64 bits).  A pair counts while
//     T (1 - alpha) >= t_min; that product never rises along the list, so nothing after the stop counts either.  S - P is
//     the pixel's R less a scan of sums over the lanes.
//   * Matrix cores, in FP32, where a contraction uses most of their tile: q = g . (c, d, 1) of all sixteen pixels and
//     records is one 16x16x4 product (channels as the inner index), and the sums of w g over a lane's four pixels
//     are four 4x4x1 products (sixteen of them side by side, each of four channels and four records).
//   * A record's ten sums over the block's rows are reduced and spread over the rows (ten values by eight lane swaps),
//     and added to the wave's own LDS sums by plain reads and writes, once per sixteen records: LDS float atomics
//     take about two cycles a lane and had kept the LDS busy for 85% of the kernel's time.
//   * A pair that does not contribute has alpha = w = 0 and adds 0 times what its pixel's upstream gradient gives, which
//     is 0 as long as that is finite.  A block with a pixel whose gradient is not, or is so large that a product of it
//     might not be (far), leaves such pairs out instead: what is not finite reaches the records that contribute at its
//     pixel, no others.
// Returns whether a pixel of the blocks that this wave took is still live.
// What bounds it is issue.
constexpr float kFarGradient = 1e18f;

template <class G, bool VIS, bool WHOLE>
__device__ __forceinline__ void backward_block(BwdStage<G>& s, const TileCtx& t, const DevOpts& op, int blk,
                                               const uint8_t* list, int n, bool far, f32x4& T) {
  const int r = t.lane & 15, k = t.lane >> 4, p0 = blk * 16, sub = blk >> 2;
  f32x4 R = *reinterpret_cast<const f32x4*>(&s.R[p0 + 4 * k]);
  f32x4 gv = {0.f, 0.f, 0.f, 0.f};
  if (VIS) gv = *reinterpret_cast<const f32x4*>(&s.gv[p0 + 4 * k]);
  const float gq = s.g[k][p0 + r];
  const f32x4 gw = *reinterpret_cast<const f32x4*>(&s.g[t.lane & 3][p0 + 4 * k]);
  // this lane's channel of a record (the inner index of q): red, green, blue, depth
  const float* chan = k == 0 ? &s.B[0].w : k == 1 ? &s.C[0].x : k == 2 ? &s.C[0].y : &s.A[0].z;
  const int chan_shift = k == 1 || k == 2 ? 1 : 2;
  const float fx0 = (float)(t.tx0 + (sub % G::SX) * 8 + (blk & 1) * 4) + 0.5f;
  const float fy = (float)(t.ty0 + (sub / G::SX) * 8 + (blk & 2) * 2 + k) + 0.5f;
  // the records of the next sixteen are read while these are worked on
  int j = list[r], jn = list[16 + r];
  float4 A = s.A[j], B = s.B[j];
  float ch = chan[j << chan_shift];
#pragma unroll 1
  for (int c = 0; c < n; c += 16) {
    float2* sum8 = reinterpret_cast<float2*>(&s.acc8[t.wave][j][2 * k]);
    float* sum2 = &s.acc2[t.wave][j][k >> 1];
    const float2 old8 = *sum8;
    const float old2 = *sum2;
    const f32x4 q = __builtin_amdgcn_mfma_f32_16x16x4f32(gq, ch, gv, 0, 0, 0);
    float am[4], om[4], x[4], Tn[4], dx[4], dy = 0.f;
    bool clamped[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      float alpha;
      const bool ok = eval_pair<WHOLE>(A, B, fx0 + (float)i, fy, op, alpha, clamped[i], dx[i], dy);
      am[i] = ok ? alpha : 0.f;
      om[i] = 1.f - am[i];
      Tn[i] = T[i] * om[i];
    }
    j = jn;
    jn = list[c + 32 + r];
    A = s.A[j];
    B = s.B[j];
    ch = chan[j << chan_shift];
    row_products(Tn, om);
    float w[4], pre[4], s0, sx, sxx;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
#pragma clang fp contract(off)
      // in front of the record: the record before's, the pixel's T in front of the first
      x[i] = __int_as_float(__builtin_amdgcn_update_dpp(__float_as_int(T[i]), __float_as_int(Tn[i]), 0x111, 0xf, 0xf,
                                                        false));
      if (!(Tn[i] >= op.t_min)) am[i] = 0.f;
      T[i] = gsk::dpp_f<0x15F>(Tn[i]);  // row_newbcast: the last lane's
      w[i] = am[i] * x[i];
      pre[i] = w[i] * q[i];
      pre[i] += gsk::dpp_f<0x111>(pre[i]);  // row_shr:1
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) pre[i] += gsk::dpp_f<0x112>(pre[i]);
#pragma unroll
    for (int i = 0; i < 4; ++i) pre[i] += gsk::dpp_f<0x114>(pre[i]);
#pragma unroll
    for (int i = 0; i < 4; ++i) pre[i] += gsk::dpp_f<0x118>(pre[i]);
    f32x4 col = {0.f, 0.f, 0.f, 0.f};
    if (WHOLE && far) {
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        const f32x4 gc = *reinterpret_cast<const f32x4*>(&s.g[c][p0 + 4 * k]);
#pragma unroll
        for (int i = 0; i < 4; ++i) col[c] += am[i] > 0.f ? gc[i] * w[i] : 0.f;
      }
    } else {
#pragma unroll
      for (int i = 0; i < 4; ++i) col = __builtin_amdgcn_mfma_f32_4x4x1f32(gw[i], w[i], col, 0, 0, 0);
    }
    float dalpha[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const float Rn = R[i] - pre[i];
      R[i] = gsk::dpp_f<0x15F>(Rn);
      dalpha[i] = x[i] * q[i] - Rn * __builtin_amdgcn_rcpf(om[i]);
      if (WHOLE && clamped[i]) am[i] = 0.f;  // a clamped alpha passes no gradient
    }
    if (WHOLE && far) {
#pragma unroll
      for (int i = 0; i < 4; ++i) dalpha[i] = am[i] > 0.f ? dalpha[i] : 0.f;
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const float dq = am[i] * dalpha[i];
      const float dqx = dq * dx[i];
      s0 = i ? s0 + dq : dq;
      sx = i ? sx + dqx : dqx;
      sxx = i ? __builtin_fmaf(dqx, dx[i], sxx) : dqx * dx[i];
    }
    const float sy = s0 * dy;
    const float v0 = row_reduce4(s0, sx, sy, sxx), v1 = row_reduce4(sx * dy, sy * dy, col[0], col[1]);
    const float v2 = row_reduce2(col[2], col[3]);
    *sum8 = make_float2(old8.x + v0, old8.y + v1);
    *sum2 = old2 + v2;
    if (!any_live(T, op)) break;
  }
  if (r == 0) {
    *reinterpret_cast<f32x4*>(&s.T[p0 + 4 * k]) = T;
    *reinterpret_cast<f32x4*>(&s.R[p0 + 4 * k]) = R;
  }
}

template <class G, bool VIS>
__device__ __forceinline__ bool backward_round(BwdStage<G>& s, const TileCtx& t, const DevOpts& op) {
  uint8_t* list = s.list[t.wave];
  uint64_t odd[G::BATCH / 64];
#pragma unroll
  for (int h = 0; h < G::BATCH / 64; ++h) odd[h] = gsk::uniform64(s.odd[h]);
  bool any = false;
  int blk = t.wave;
#pragma unroll 1
  for (; blk < G::NB; blk = __builtin_amdgcn_readfirstlane(t.lane == 0 ? atomicAdd(&s.next, 1) : 0)) {
    f32x4 T = *reinterpret_cast<const f32x4*>(&s.T[blk * 16 + 4 * (t.lane >> 4)]);
    if (!any_live(T, op)) continue;
    const int px = blk * 16 + (t.lane & 15);
    bool far = !(fabsf(s.g[t.lane >> 4][px]) < kFarGradient && fabsf(s.R[px]) < kFarGradient);
    if (VIS) far |= !(fabsf(s.gv[px]) < kFarGradient);
    far = __builtin_amdgcn_ballot_w64(far) != 0;
    int n = 0;
    uint64_t whole = 0;
#pragma unroll
    for (int h = 0; h < G::BATCH / 64; ++h) {
      const bool bit = (s.bm[2 * h + (t.lane >> 5)][blk] >> (t.lane & 31)) & 1u;
      const uint64_t m = __builtin_amdgcn_ballot_w64(bit);
      if (bit) list[gsk::rank_in(m, n)] = (uint8_t)(64 * h + t.lane);
      n += __popcll(m);
      whole |= m & odd[h];
    }
    if (n == 0) {
      any = true;
      continue;
    }
    if (t.lane < 16) list[n + t.lane] = (uint8_t)G::BATCH;  // the empty record
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");  // the list is read by other lanes of this wave only
    if (whole || far)
      backward_block<G, VIS, true>(s, t, op, blk, list, n, far, T);
    else
      backward_block<G, VIS, false>(s, t, op, blk, list, n, false, T);
    any |= any_live(T, op);
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
  }
  return any;
}

// Backward of records [rg.x, rg.y), front to back, from this lane's pixel's transmittance T and prefix P (its state
// at rg.x), with upstream gradient g and S = g . (C, D, V) of the final values.  Per-record partial derivatives are
// summed in LDS and stored as the instances' partials once per round; instances after the walk's end get zero
// partials.  VIS: the visibility has an upstream gradient of its own (never in loss mode).
template <class G, bool VIS>
__device__ __forceinline__ void backward_walk(BwdStage<G>& s, const float4* __restrict__ rec,
                                              const int32_t* __restrict__ vals, int2 rg, const TileCtx& t,
                                              const DevOpts& op, bool live, float T, float Pp, float gr, float gg,
                                              float gb, float gd, float gv, float S, const BwdArgs& a) {
  static_assert(G::DEPTH == 1 && G::BATCH < 256, "a record per thread, 8-bit lists");
  if (rg.x >= rg.y) return;  // the same in every thread of the workgroup
  // this thread's record of the round in flight, the id of the next round's, and the instance slot of the staged one
  // (the threads past BATCH stage nothing)
  const bool stager = G::NT == G::BATCH || (int)threadIdx.x < G::BATCH;
  const int jt = threadIdx.x;
  int fr[1], frn[1], first = 0;
  float4 fA[1], fB[1], fC[1];
  int slot = 0;
  if (stager) {
    fetch_ids<G, 1>(vals, rg.x, rg.y, fr);
    fetch_ids<G, 1>(vals, rg.x + G::BATCH, rg.y, frn);
    fetch_records<1>(rec, fr, fA, fB, fC);
    first = a.rec_slot[fr[0]];
  }
  {
    const int p = threadIdx.x;  // sixteen lanes hold a block, row by row
    s.T[p] = live ? T : 0.f;
    s.R[p] = S - Pp;
    if (VIS) s.gv[p] = gv;
    s.g[0][p] = gr;
    s.g[1][p] = gg;
    s.g[2][p] = gb;
    s.g[3][p] = gd;
  }
  // entries past a list's end are read ahead: they stay valid slots
  if (t.lane < (G::BATCH + 48) / 4) reinterpret_cast<uint32_t*>(s.list[t.wave])[t.lane] = 0;
  if (threadIdx.x == 0) {
    s.A[G::BATCH] = s.B[G::BATCH] = make_float4(0.f, 0.f, 0.f, 0.f);
    s.C[G::BATCH] = make_float2(0.f, 0.f);
  }
  for (int b0 = rg.x;; b0 += G::BATCH) {
    const bool go = round_barrier<G>(s, t, live) && b0 < rg.y;
    if (b0 != rg.x && stager && b0 - G::BATCH + jt < rg.y) flush_grads<G>(s, jt, slot, a.ipart, a.capacity);
    if (!go) {
      zero_grads<G>(rec, vals, t, a.ipart, a.rec_slot, a.capacity, b0, rg.y);
      break;
    }
    clear_masks<G>(s);
    if (threadIdx.x == 0) s.next = G::NW;
    const float4 A = fA[0], B = fB[0], C = fC[0];
    if (stager) {
      s.A[jt] = A;
      s.B[jt] = B;
      s.C[jt] = make_float2(C.x, C.y);
      if (b0 + jt < rg.y) {
#pragma unroll
        for (int w = 0; w < G::NW; ++w) {
          float4* p = reinterpret_cast<float4*>(s.acc8[w][jt]);
          p[0] = p[1] = make_float4(0.f, 0.f, 0.f, 0.f);
          *reinterpret_cast<float2*>(s.acc2[w][jt]) = make_float2(0.f, 0.f);
        }
      }
      slot = inst_slot<G>(first, C.z, C.w, t);
      fr[0] = frn[0];
      fetch_records<1>(rec, fr, fA, fB, fC);
      first = a.rec_slot[fr[0]];
      fetch_ids<G, 1>(vals, b0 + 2 * G::BATCH, rg.y, frn);
    }
    __syncthreads();
    if (stager) {
      const bool odd = b0 + jt < rg.y && scatter<G>(s.bm, jt, A, B, C.z, C.w, t, op);
      const uint64_t m = __builtin_amdgcn_ballot_w64(odd);
      if (t.lane == 0) s.odd[jt >> 6] = m;
    }
    __syncthreads();
    live = backward_round<G, VIS>(s, t, op);
  }
}

// Upstream gradient g and S = g . (C, D, V) of this lane's pixel of a whole tile, from the forward images or a forward
// sweep.  at: the tile's schedule position.
template <class G, bool HAVE_FWD, bool LOSS>
__device__ __forceinline__ void tile_upstream(Stage<G>& s, const float4* __restrict__ rec,
                                              const int32_t* __restrict__ vals, int2 rg, const TileCtx& t,
                                              const DevOpts& op, const BwdArgs& a, int at, float& gr, float& gg,
                                              float& gb, float& gd, float& gv, float& S) {
  float Cf = 0.f, Gf = 0.f, Bf = 0.f, Df = 0.f, Vf = 0.f;
  const Upstream u = load_upstream<LOSS>(t, a);
  if (HAVE_FWD) {
    if (t.inside) {
      const int64_t P = (int64_t)t.W * t.H;
      const int64_t pi = (int64_t)t.py * t.W + t.px;
      Cf = a.fwd_rgb[3 * t.pix_off + pi];
      Gf = a.fwd_rgb[3 * t.pix_off + P + pi];
      Bf = a.fwd_rgb[3 * t.pix_off + 2 * P + pi];
      Df = a.fwd_depth[t.pix_off + pi];
      Vf = a.fwd_vis[t.pix_off + pi];
    }
  } else {
    float T;
    forward_sweep<G>(s, rec, vals, rg, t, op, T, Cf, Gf, Bf, Df, Vf);
    Cf = __builtin_fmaf(T, op.bg[0], Cf);
    Gf = __builtin_fmaf(T, op.bg[1], Gf);
    Bf = __builtin_fmaf(T, op.bg[2], Bf);
  }
  float loss_acc = 0.f;
  pixel_upstream<LOSS>(t, a, u, Cf, Gf, Bf, Df, gr, gg, gb, gd, gv, loss_acc);
  S = gr * Cf + gg * Gf + gb * Bf + gd * Df + gv * Vf;
  if (LOSS) store_loss<G>(t, a, at, loss_acc);
  __syncthreads();  // every wave is done with the forward's records: the backward's state takes their place
}

constexpr size_t max_size(size_t a, size_t b) { return a > b ? a : b; }

// A kernel's LDS block as one of the structures that take turns in it.
template <class S>
__device__ __forceinline__ S& lds_as(char* buf) {
  return *reinterpret_cast<S*>(buf);
}

template <int TW, int TH, int DEPTH, bool HAVE_FWD, bool LOSS>
__global__ __launch_bounds__(TW * TH, 4) void k_render_bwd(const float4* __restrict__ rec,
                                                        const int32_t* __restrict__ vals,
                                                        const int2* __restrict__ range,
                                                        const gs_camera* __restrict__ cams, int V, int n_tiles,
                                                        const int32_t* __restrict__ order, DevOpts op, BwdArgs a) {
  using G = Geo<TW, TH, DEPTH>;
  using GB = BGeo<TW, TH>;
  __shared__ alignas(16) char buf[max_size(sizeof(BwdStage<GB>), sizeof(Stage<G>))];
  TileCtx t;
  int tile;
  if (!tile_setup<G>(cams, V, n_tiles, order, t, tile)) return;
  const int2 rg = range[tile];
  float gr, gg, gb, gd, gv, S;
  tile_upstream<G, HAVE_FWD, LOSS>(lds_as<Stage<G>>(buf), rec, vals, rg, t, op, a, blockIdx.x, gr, gg, gb, gd,
                                          gv, S);
  backward_walk<GB, !LOSS>(lds_as<BwdStage<GB>>(buf), rec, vals, rg, t, op, t.inside, 1.f, 0.f, gr, gg, gb, gd, gv, S, a);
}

// ---------------------------------------------------------------------------------------------------------
// Fused backward with depth segments.  A tile list longer than L records is split into segments of L,
// each its own workgroup, so the few huge tiles of coarse pyramid levels no longer serialise the launch.
// Compositing is a product of transmittances, so per pixel:
//   1. each segment k walks its records from T = 1 without the stop rule: its transmittance product T_k and
//      local sums (C, D, V)_k (k_bwd_sums, alongside the unsplit tiles);
//   2. T_start,k = T_0 T_1 ... T_{k-1} (left to right); the pixel's last live segment k* is the
//      last with T_start,k >= t_min, and only there can the stop rule end the walk: that segment is walked
//      again from T_start,k* with the stop rule (k_seg_stop; not where the forward images are given);
//   3. the final values are sum_{k<k*} T_start,k (C, D, V)_k plus segment k*'s stopped sums plus the
//      background; from them the upstream gradient g, S and each segment's start state (T_start,k,
//      P_start,k = g . sum_{j<k} contribution_j) (k_seg_combine);
//   4. each live segment runs the backward walk from its start state (k_bwd_main).
// The result equals the unsplit walk up to FP32 rounding of the transmittance product (the association of
// the product differs), which can move a stop decision that lies within that rounding of t_min.
template <class G>
__device__ __forceinline__ int2 segment_range(int2 rg, int k, int L) {
  const int lo = rg.x + k * L;
  return make_int2(lo, min(rg.y, lo + L));
}

// Step 1 for one depth segment: its transmittance product and local sums, from T = 1 without the stop rule.
template <class G>
__device__ __forceinline__ void segment_sums(Stage<G>& s, const float4* __restrict__ rec,
                                             const int32_t* __restrict__ vals, int2 rg, int4 it, const TileCtx& t,
                                             const DevOpts& op, const SegArgs& g) {
  float T = 1.f, Cr = 0.f, Cg = 0.f, Cb = 0.f, D = 0.f, Vs = 0.f;
  forward_walk<G, false>(s, rec, vals, segment_range<G>(rg, it.y, g.len), t, op, t.inside, T, Cr, Cg, Cb, D,
                                Vs);
  float* o = g.seg + (size_t)(it.z + it.y) * 6 * G::NT + threadIdx.x;
  o[0 * G::NT] = T;
  o[1 * G::NT] = Cr;
  o[2 * G::NT] = Cg;
  o[3 * G::NT] = Cb;
  o[4 * G::NT] = D;
  o[5 * G::NT] = Vs;
}

// The work items of a launch: one per workgroup (item blockIdx.x while it is below count), or with PERSIST a
// grid sized to what the GPU holds at once, whose workgroups take items in schedule order from the counter
// *ctr (zeroed before the launch) until count is reached; every workgroup then leaves the loop.
template <bool PERSIST, class Body>
__device__ __forceinline__ void for_items(int count, int32_t* ctr, Body body) {
  if constexpr (!PERSIST) {
    if ((int)blockIdx.x < count) body((int)blockIdx.x);
  } else {
    __shared__ int s_item;
    while (true) {
      __syncthreads();  // the previous item's LDS is no longer read
      if (threadIdx.x == 0) s_item = atomicAdd(ctr, 1);
      __syncthreads();
      const int b = s_item;
      if (b >= count) return;
      body(b);
    }
  }
}

// A whole tile of 1 to kOwnForward - 1 records has its forward in the backward's block instead of k_bwd_sums: the sums
// that k_bwd_sums leaves behind (20 B written and read per pixel) cost as much as a very short list's sweep, which the
// backward's kernel runs at two thirds of the waves.  Steps with the line at 2, 8 and 32: 14.8 k tiles of 32x8 with some
// 23 records each 521, 525 and 538 us; 29.7 k of 16x8 with 21 522, 525 and 539; 24 views 6.31, 6.32 and 6.33 ms.
constexpr int kOwnForward = 8;

// Step 1 of the backward: segments of the split tiles run segment_sums; whole tiles run the forward sweep up to the
// upstream gradient and leave it (g and S, six floats a pixel) in the segment state's slot of their work item (with
// forward images, and in small frames, k_bwd_main forms it itself).  A kernel of its own, since the forward's walk
// needs 80 of the backward's 128 registers and half of its LDS (21.6 of 34 KB at 16x16 and 32x8, 8.7 of 19.6 at 16x8, 3.8
// of 7.2 at 8x8): six waves a SIMD instead of four (kWholeTiles has what that is worth).  With two records a thread (50.8
// KB, the staged records in scratch) three, which is why that never wins.
template <int TW, int TH, int DEPTH, bool HAVE_FWD, bool LOSS, bool PERSIST = false>
__global__ __launch_bounds__(TW * TH, 6) void k_bwd_sums(const float4* __restrict__ rec, const int32_t* __restrict__ vals,
                                                      const int2* __restrict__ range,
                                                      const gs_camera* __restrict__ cams, int V, DevOpts op,
                                                      BwdArgs a, SegArgs g, int32_t* ctr) {
  using G = Geo<TW, TH, DEPTH>;
  __shared__ Stage<G> s;
  for_items<PERSIST>(!HAVE_FWD && g.whole ? g.counters[192] : g.counters[193], ctr, [&](int b) {
    const int4 it = g.items[b];
    TileCtx t;
    tile_at<G>(cams, V, it.x, t);
    if (it.z >= 0) {
      segment_sums<G>(s, rec, vals, range[it.x], it, t, op, g);
    } else if (const int2 rg = range[it.x]; !HAVE_FWD && (rg.x >= rg.y || rg.y - rg.x >= kOwnForward)) {
      float v[6];
      tile_upstream<G, false, LOSS>(s, rec, vals, rg, t, op, a, it.w, v[0], v[1], v[2], v[3], v[4], v[5]);
      if (rg.x >= rg.y) return;  // an empty tile: its loss is in
      float* o = g.seg + (size_t)b * 6 * G::NT + threadIdx.x;
#pragma unroll
      for (int i = 0; i < 6; ++i)
        if (!(LOSS && i == 4)) o[i * G::NT] = v[i];  // (the visibility's is 0 in loss mode)
    }
  });
}

// Forward over the work items: whole tiles are composited and written; segments of split tiles run step 1.
template <int TW, int TH, int DEPTH>
__global__ __launch_bounds__(TW * TH, 6) void k_fwd_main(const float4* __restrict__ rec, const int32_t* __restrict__ vals,
                                                      const int2* __restrict__ range,
                                                      const gs_camera* __restrict__ cams, int V, DevOpts op,
                                                      SegArgs g, float* __restrict__ out_rgb,
                                                      float* __restrict__ out_depth, float* __restrict__ out_vis) {
  using G = Geo<TW, TH, DEPTH>;
  __shared__ Stage<G> s;
  if ((int)blockIdx.x >= g.counters[192]) return;
  const int4 it = g.items[blockIdx.x];
  TileCtx t;
  tile_at<G>(cams, V, it.x, t);
  const int2 rg = range[it.x];
  if (it.z >= 0) {
    segment_sums<G>(s, rec, vals, rg, it, t, op, g);
    return;
  }
  float T, Cr, Cg, Cb, D, Vs;
  forward_sweep<G>(s, rec, vals, rg, t, op, T, Cr, Cg, Cb, D, Vs);
  write_pixel(t, op, T, Cr, Cg, Cb, D, Vs, out_rgb, out_depth, out_vis);
}

// Segments of a split tile whose loads the combine steps keep in flight together (a tile may have a hundred
// segments, and the running products make each pixel's pass serial).
constexpr int kSegBatch = 4;
constexpr int kPrefixBatch = 16;

// Step 2: the last live segment of each pixel walks again, from its start transmittance and with the stop rule.  Every
// segment forms its own start transmittances (a pass of its own over them took 5 us in frames without a split tile and
// 23 us in one of 10 k).
template <int TW, int TH, int DEPTH, bool PERSIST = false>
__global__ __launch_bounds__(TW * TH, 6) void k_seg_stop(const float4* __restrict__ rec, const int32_t* __restrict__ vals,
                                                      const int2* __restrict__ range,
                                                      const gs_camera* __restrict__ cams, int V, DevOpts op,
                                                      SegArgs g, int32_t* ctr) {
  using G = Geo<TW, TH, DEPTH>;
  __shared__ Stage<G> s;
  for_items<PERSIST>(g.counters[193], ctr, [&](int b) {
    const int4 it = g.items[b];
    TileCtx t;
    tile_at<G>(cams, V, it.x, t);
    const int2 rg = range[it.x];
    const int n = (rg.y - rg.x + g.len - 1) / g.len;
    // start transmittances of this segment and the next: the products of the segments before them, left to right
    // (a dead pixel stays dead, so the wave stops reading once all of its pixels are)
    const float* sp = g.seg + (size_t)it.z * 6 * G::NT + threadIdx.x;
    float Ts = 1.f, Te = 1.f;
    for (int k0 = 0; k0 <= it.y; k0 += kPrefixBatch) {
      if (!__builtin_amdgcn_ballot_w64(Te >= op.t_min)) {
        Ts = Te;
        break;
      }
      float v[kPrefixBatch];
#pragma unroll
      for (int i = 0; i < kPrefixBatch; ++i) v[i] = sp[(size_t)min(k0 + i, it.y) * 6 * G::NT];
#pragma unroll
      for (int i = 0; i < kPrefixBatch; ++i) {
        if (k0 + i > it.y) break;
        Ts = Te;
        Te = Ts * v[i];
      }
    }
    const bool last = t.inside && Ts >= op.t_min && (it.y == n - 1 || Te < op.t_min);
    if (!__syncthreads_or(last)) return;
    float T = Ts, Cr = 0.f, Cg = 0.f, Cb = 0.f, D = 0.f, Vs = 0.f;
    forward_walk<G, true>(s, rec, vals, segment_range<G>(rg, it.y, g.len), t, op, last, T, Cr, Cg, Cb, D, Vs);
    if (last) {
      float* o = g.split + (size_t)it.w * 12 * G::NT + threadIdx.x;
      o[0 * G::NT] = T;
      o[1 * G::NT] = Cr;
      o[2 * G::NT] = Cg;
      o[3 * G::NT] = Cb;
      o[4 * G::NT] = D;
      o[5 * G::NT] = Vs;
    }
  });
}

// Step 3, first half: the pixel's last live segment ks (the last whose start transmittance, the product of the
// segments before it, is at least t_min) and its final sums (C, D, V) and transmittance.  One pass: while the start
// transmittance of segment k is at least t_min, k is the candidate and the weighted sum of the segments
// before it is kept aside; the sums are formed in segment order.  SUMS = false: only ks.
template <class G, bool SUMS>
__device__ __forceinline__ void split_final(const float* sp, const float* xp, int n, const TileCtx& t,
                                            const DevOpts& op, int& ks, float& Tf, float& Cr, float& Cg, float& Cb,
                                            float& D, float& Vs) {
  constexpr size_t SS = 6 * G::NT;
  constexpr int BATCH = SUMS ? kSegBatch : kPrefixBatch, W = SUMS ? 6 : 1;
  ks = 0;
  bool more = true;
  float Ts = 1.f, Rr = 0.f, Rg = 0.f, Rb = 0.f, RD = 0.f, RV = 0.f;  // weighted sums of the segments before k
  Cr = Cg = Cb = D = Vs = 0.f;
  for (int k0 = 0; k0 < n && more; k0 += BATCH) {
    float v[BATCH][W];
#pragma unroll
    for (int i = 0; i < BATCH; ++i) {
      const float* q = sp + (size_t)min(k0 + i, n - 1) * SS;
#pragma unroll
      for (int c = 0; c < W; ++c) v[i][c] = q[c * G::NT];
    }
#pragma unroll
    for (int i = 0; i < BATCH; ++i) {
      if (k0 + i < n && Ts >= op.t_min) {
        ks = k0 + i;
        if constexpr (SUMS) {
          Cr = Rr;
          Cg = Rg;
          Cb = Rb;
          D = RD;
          Vs = RV;
          Rr = __builtin_fmaf(Ts, v[i][1], Rr);
          Rg = __builtin_fmaf(Ts, v[i][2], Rg);
          Rb = __builtin_fmaf(Ts, v[i][3], Rb);
          RD = __builtin_fmaf(Ts, v[i][4], RD);
          RV = __builtin_fmaf(Ts, v[i][5], RV);
        }
        Ts *= v[i][0];
      } else {
        more = false;
      }
    }
  }
  Tf = 1.f;
  if (SUMS && t.inside) {
    Tf = xp[0];
    Cr += xp[1 * G::NT];
    Cg += xp[2 * G::NT];
    Cb += xp[3 * G::NT];
    D += xp[4 * G::NT];
    Vs += xp[5 * G::NT];
  }
}

// Forward of split tiles, step 3: write the final values.
template <int TW, int TH>
__global__ __launch_bounds__(TW * TH) void k_seg_fwd_out(const gs_camera* __restrict__ cams, int V, DevOpts op,
                                                         SegArgs g, float* __restrict__ out_rgb,
                                                         float* __restrict__ out_depth, float* __restrict__ out_vis) {
  using G = Geo<TW, TH, 1>;
  const int l = blockIdx.x;
  if (l >= g.counters[194]) return;
  TileCtx t;
  tile_at<G>(cams, V, g.order[l], t);
  const float* sp = g.seg + (size_t)g.seg_first[l] * 6 * G::NT + threadIdx.x;
  const float* xp = g.split + (size_t)l * 12 * G::NT + threadIdx.x;
  int ks;
  float T, Cr, Cg, Cb, D, Vs;
  split_final<G, true>(sp, xp, g.seg_count[l], t, op, ks, T, Cr, Cg, Cb, D, Vs);
  write_pixel(t, op, T, Cr, Cg, Cb, D, Vs, out_rgb, out_depth, out_vis);
}

// Backward of split tiles, step 3: final values (or the forward images, which spare step 2), upstream gradient, S and
// the start state (T_start, P_start) of every segment; T_start = 0 marks a segment after the pixel's end.
template <int TW, int TH, bool HAVE_FWD, bool LOSS>
__global__ __launch_bounds__(TW * TH) void k_seg_combine(const gs_camera* __restrict__ cams, int V, DevOpts op,
                                                         BwdArgs a, SegArgs g) {
  using G = Geo<TW, TH, 1>;
  const int l = blockIdx.x;
  if (l >= g.counters[194]) return;
  const int n = g.seg_count[l];
  TileCtx t;
  tile_at<G>(cams, V, g.order[l], t);
  float* sp = g.seg + (size_t)g.seg_first[l] * 6 * G::NT + threadIdx.x;
  float* xp = g.split + (size_t)l * 12 * G::NT + threadIdx.x;
  constexpr size_t SS = 6 * G::NT;
  int ks;
  float Tf, Cr, Cg, Cb, D, Vs;
  const Upstream u = load_upstream<LOSS>(t, a);
  split_final<G, !HAVE_FWD>(sp, xp, n, t, op, ks, Tf, Cr, Cg, Cb, D, Vs);
  float Cf = __builtin_fmaf(Tf, op.bg[0], Cr), Gf = __builtin_fmaf(Tf, op.bg[1], Cg);
  float Bf = __builtin_fmaf(Tf, op.bg[2], Cb), Df = D, Vf = Vs;
  if (HAVE_FWD && t.inside) {
    const int64_t P = (int64_t)t.W * t.H;
    const int64_t pi = (int64_t)t.py * t.W + t.px;
    Cf = a.fwd_rgb[3 * t.pix_off + pi];
    Gf = a.fwd_rgb[3 * t.pix_off + P + pi];
    Bf = a.fwd_rgb[3 * t.pix_off + 2 * P + pi];
    Df = a.fwd_depth[t.pix_off + pi];
    Vf = a.fwd_vis[t.pix_off + pi];
  }
  float gr, gg, gb, gd, gv, loss_acc = 0.f;
  pixel_upstream<LOSS>(t, a, u, Cf, Gf, Bf, Df, gr, gg, gb, gd, gv, loss_acc);
  const float S = gr * Cf + gg * Gf + gb * Bf + gd * Df + gv * Vf;
  if (LOSS) store_loss<G>(t, a, l, loss_acc);
  float Pr = 0.f, Tr = 1.f;
  for (int k0 = 0; k0 < n; k0 += kSegBatch) {
    // segments up to ks are read (batched); later ones only get T_start = 0
    float v[kSegBatch][6];
#pragma unroll
    for (int i = 0; i < kSegBatch; ++i) {
      const float* q = sp + (size_t)min(k0 + i, n - 1) * SS;
#pragma unroll
      for (int c = 0; c < 6; ++c) v[i][c] = k0 + i <= ks ? q[c * G::NT] : 0.f;
    }
#pragma unroll
    for (int i = 0; i < kSegBatch; ++i) {
      const int k = k0 + i;
      if (k >= n) break;
      float* q = sp + (size_t)k * SS;
      const float Ts = Tr;
      const float dot =
          k < ks ? Ts * (gr * v[i][1] + gg * v[i][2] + gb * v[i][3] + gd * v[i][4] + gv * v[i][5]) : 0.f;
      q[0] = k <= ks ? Ts : 0.f;
      q[1 * G::NT] = Pr;
      Pr += dot;
      Tr *= v[i][0];
    }
  }
  xp[6 * G::NT] = gr;
  xp[7 * G::NT] = gg;
  xp[8 * G::NT] = gb;
  xp[9 * G::NT] = gd;
  xp[10 * G::NT] = gv;
  xp[11 * G::NT] = S;
}

// Step 4, and the whole tiles: segments run the backward walk from their start state, whole tiles from the upstream
// gradient that k_bwd_sums left or that they form here.
template <int TW, int TH, int DEPTH, bool HAVE_FWD, bool LOSS, bool PERSIST = false>
__global__ __launch_bounds__(TW * TH, 4) void k_bwd_main(const float4* __restrict__ rec,
                                                         const int32_t* __restrict__ vals,
                                                         const int2* __restrict__ range,
                                                         const gs_camera* __restrict__ cams, int V, DevOpts op,
                                                         BwdArgs a, SegArgs g, int32_t* ctr) {
  using G = Geo<TW, TH, DEPTH>;
  using GB = BGeo<TW, TH>;
  __shared__ alignas(16) char buf[max_size(sizeof(BwdStage<GB>), sizeof(Stage<G>))];
  BwdStage<GB>& s = lds_as<BwdStage<GB>>(buf);
  for_items<PERSIST>(g.counters[192], ctr, [&](int b) {
    const int4 it = g.items[b];
    int2 rg = range[it.x];
    if (!HAVE_FWD && g.whole && rg.x >= rg.y) return;  // an empty tile, done by k_bwd_sums
    TileCtx t;
    tile_at<G>(cams, V, it.x, t);
    bool live = t.inside;
    float T = 1.f, P = 0.f, gr, gg, gb, gd, gv, S;
    if (it.z < 0 && !HAVE_FWD && g.whole && rg.y - rg.x >= kOwnForward) {
      const float* v = g.seg + (size_t)b * 6 * G::NT + threadIdx.x;
      gr = v[0 * G::NT];
      gg = v[1 * G::NT];
      gb = v[2 * G::NT];
      gd = v[3 * G::NT];
      gv = LOSS ? 0.f : v[4 * G::NT];
      S = v[5 * G::NT];
    } else if (it.z < 0) {
      tile_upstream<G, HAVE_FWD, LOSS>(lds_as<Stage<G>>(buf), rec, vals, rg, t, op, a, it.w, gr, gg, gb, gd, gv,
                                              S);
    } else {
      const float* sp = g.seg + (size_t)(it.z + it.y) * 6 * G::NT + threadIdx.x;
      const float* xp = g.split + (size_t)it.w * 12 * G::NT + threadIdx.x;
      T = sp[0];
      P = sp[1 * G::NT];
      live = live && T >= op.t_min;
      gr = xp[6 * G::NT];
      gg = xp[7 * G::NT];
      gb = xp[8 * G::NT];
      gd = xp[9 * G::NT];
      gv = xp[10 * G::NT];
      S = xp[11 * G::NT];
      rg = segment_range<G>(rg, it.y, g.len);
    }
    backward_walk<GB, !LOSS>(s, rec, vals, rg, t, op, live, T, P, gr, gg, gb, gd, gv, S, a);
  });
}

// Work counts of the forward: pairs evaluated (pixel inside the record's pixel rectangle, up to the
// pixel's stop) and pairs contributing.  Independent of the tile shape; diagnostic.
template <int TW, int TH>
__global__ __launch_bounds__(TW * TH) void k_count_pairs(const float4* __restrict__ rec,
                                                         const int32_t* __restrict__ vals,
                                                         const int2* __restrict__ range,
                                                         const gs_camera* __restrict__ cams, int V, int n_tiles,
                                                         const int32_t* __restrict__ order, DevOpts op,
                                                         unsigned long long* __restrict__ counts) {
  using G = Geo<TW, TH, 1>;
  __shared__ Stage<G> s;
  TileCtx t;
  int tile;
  if (!tile_setup<G>(cams, V, n_tiles, order, t, tile)) return;
  const int2 rg = range[tile];
  bool live = t.inside;
  const float fx = (float)t.px + 0.5f, fy = (float)t.py + 0.5f;
  float T = 1.f;
  unsigned long long ev = 0, co = 0;
  for (int b0 = rg.x; b0 < rg.y; b0 += G::BATCH) {
    if (!__syncthreads_or(live)) break;
    const int nb = min(G::BATCH, rg.y - b0);
    if ((int)threadIdx.x < nb) {
      const int r = vals[b0 + threadIdx.x];
      s.A[threadIdx.x] = rec[3 * (int64_t)r];
      s.B[threadIdx.x] = rec[3 * (int64_t)r + 1];
      s.C[threadIdx.x] = rec[3 * (int64_t)r + 2];
    }
    __syncthreads();
    for (int j = 0; j < nb && live; ++j) {
      int x0, x1, y0, y1;
      unpack_rect(s.C[j].z, s.C[j].w, x0, x1, y0, y1);
      if (t.px < x0 || t.px > x1 || t.py < y0 || t.py > y1) continue;
      ++ev;
      float alpha, dx, dy;
      bool cl;
      if (!eval_pair<true>(s.A[j], s.B[j], fx, fy, op, alpha, cl, dx, dy)) continue;
      const float Tn = T * (1.f - alpha);
      if (Tn < op.t_min) {
        live = false;
        continue;
      }
      ++co;
      T = Tn;
    }
  }
  // one atomic per wave (sums over the lanes first)
  for (int d = 32; d >= 1; d >>= 1) {
    ev += __shfl_xor(ev, d);
    co += __shfl_xor(co, d);
  }
  if (t.lane == 0) {
    atomicAdd(counts, ev);
    atomicAdd(counts + 1, co);
  }
}

// Valid LiDAR-depth pixels per view: grid-stride per view, one atomic per block.
// (Blocks of 1024 threads: the blocks' atomics on one cache line queue at about 5 ns each, 19 of 26 us over 24 views in
// blocks of 256.)
constexpr int kValidThreads = 1024;

__global__ __launch_bounds__(kValidThreads) void k_count_valid(const float* __restrict__ tgt_depth,
                                                     const gs_camera* __restrict__ cams,
                                                     int32_t* __restrict__ n_valid) {
  __shared__ int sh;
  if (threadIdx.x == 0) sh = 0;
  __syncthreads();
  const int v = blockIdx.y;
  const gs_camera& c = cams[v];
  const int64_t P = (int64_t)c.width * c.height;
  int cnt = 0;
  // eight independent loads in flight per thread and pass
  const int64_t step = (int64_t)gridDim.x * blockDim.x * 8;
  for (int64_t b = (int64_t)blockIdx.x * blockDim.x * 8 + threadIdx.x; b < P; b += step) {
    float d[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      const int64_t i = b + k * (int64_t)blockDim.x;
      d[k] = i < P ? tgt_depth[c.pixel_offset + i] : 0.f;
    }
#pragma unroll
    for (int k = 0; k < 8; ++k) cnt += d[k] > 0.f;
  }
  for (int d = 32; d >= 1; d >>= 1) cnt += __shfl_xor(cnt, d);
  if ((threadIdx.x & 63) == 0) atomicAdd(&sh, cnt);
  __syncthreads();
  if (threadIdx.x == 0 && sh) atomicAdd(n_valid + v, sh);
}

SegArgs seg_args(const gs_frame& f) {
  SegArgs g;
  g.items = reinterpret_cast<const int4*>(f.items);
  g.counters = f.counters;
  g.order = f.tile_order;
  g.seg_count = f.seg_count;
  g.seg_first = f.seg_first;
  g.seg = f.seg;
  g.split = f.split;
  g.len = f.seg_len;
  g.whole = f.n_tiles >= gsk::kWholeTiles;
  return g;
}

// Workgroups of a persistent launch: what the GPU holds at once (compute units x resident workgroups of the
// kernel per unit), at most cap.
template <class K>
int resident_grid(K kernel, int block, int64_t cap) {
  int dev = 0, cus = 0, occ = 0;
  if (hipGetDevice(&dev) != hipSuccess ||
      hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus < 1)
    cus = 256;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&occ, kernel, block, 0) != hipSuccess || occ < 1) occ = 1;
  const int64_t g = (int64_t)cus * occ;
  return (int)(g < cap ? g : (cap > 0 ? cap : 1));
}

template <int TW, int TH, int DEPTH>
hipError_t launch_fwd(const gs_frame& f, const DevOpts& op, const gs_images& out, hipStream_t st) {
  const int sorted = f.sort_passes & 1;
  const auto* rec = reinterpret_cast<const float4*>(f.rec);
  const auto* rng = reinterpret_cast<const int2*>(f.tile_range);
  const int bs = TW * TH;
  if (f.seg_len > 0) {
    // long lists split into depth segments
    const SegArgs g = seg_args(f);
    k_fwd_main<TW, TH, DEPTH><<<f.item_cap, bs, 0, st>>>(rec, f.vals[sorted], rng, f.cams, f.n_views, op, g, out.rgb,
                                                          out.depth, out.vis);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    k_seg_stop<TW, TH, DEPTH><<<f.seg_cap, bs, 0, st>>>(rec, f.vals[sorted], rng, f.cams, f.n_views, op, g,
                                                            nullptr);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    k_seg_fwd_out<TW, TH><<<f.long_cap, bs, 0, st>>>(f.cams, f.n_views, op, g, out.rgb, out.depth, out.vis);
    return hipGetLastError();
  }
  k_render_fwd<TW, TH, DEPTH><<<f.n_tiles, bs, 0, st>>>(rec, f.vals[sorted], rng, f.cams, f.n_views, f.n_tiles,
                                                        f.tile_order, op, out.rgb, out.depth, out.vis);
  return hipGetLastError();
}

template <int TW, int TH, int DEPTH, bool HAVE_FWD, bool LOSS>
hipError_t launch_split_bwd(const gs_frame& f, const DevOpts& op, const BwdArgs& a, bool persist, hipStream_t st) {
  const int sorted = f.sort_passes & 1;
  const auto* rec = reinterpret_cast<const float4*>(f.rec);
  const auto* rng = reinterpret_cast<const int2*>(f.tile_range);
  const int32_t* vals = f.vals[sorted];
  const int bs = TW * TH;
  const SegArgs g = seg_args(f);
  hipError_t e;
  // persistent: the three walking kernels take their items from counters[199..201]
  int32_t* ctr = f.counters + 199;
  if (persist) {
    if ((e = gs_launch::fill_i32(ctr, 0, 3, st)) != hipSuccess) return e;
    auto* kf = k_bwd_sums<TW, TH, DEPTH, HAVE_FWD, LOSS, true>;
    kf<<<resident_grid(kf, bs, !HAVE_FWD && g.whole ? f.item_cap : f.seg_cap), bs, 0, st>>>(
        rec, vals, rng, f.cams, f.n_views, op, a, g, ctr);
  } else {
    k_bwd_sums<TW, TH, DEPTH, HAVE_FWD, LOSS><<<!HAVE_FWD && g.whole ? f.item_cap : f.seg_cap, bs, 0, st>>>(
        rec, vals, rng, f.cams, f.n_views, op, a, g, nullptr);
  }
  if ((e = hipGetLastError()) != hipSuccess) return e;
  if (HAVE_FWD) {
    // the final values are given: only the segments' start states are left to form
  } else if (persist) {
    auto* ks = k_seg_stop<TW, TH, DEPTH, true>;
    ks<<<resident_grid(ks, bs, f.seg_cap), bs, 0, st>>>(rec, vals, rng, f.cams, f.n_views, op, g, ctr + 1);
  } else {
    k_seg_stop<TW, TH, DEPTH><<<f.seg_cap, bs, 0, st>>>(rec, vals, rng, f.cams, f.n_views, op, g, nullptr);
  }
  if ((e = hipGetLastError()) != hipSuccess) return e;
  k_seg_combine<TW, TH, HAVE_FWD, LOSS><<<f.long_cap, bs, 0, st>>>(f.cams, f.n_views, op, a, g);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  if (persist) {
    auto* kb = k_bwd_main<TW, TH, DEPTH, HAVE_FWD, LOSS, true>;
    kb<<<resident_grid(kb, bs, f.item_cap), bs, 0, st>>>(rec, vals, rng, f.cams, f.n_views, op, a, g, ctr + 2);
  } else {
    k_bwd_main<TW, TH, DEPTH, HAVE_FWD, LOSS><<<f.item_cap, bs, 0, st>>>(rec, vals, rng, f.cams, f.n_views, op, a,
                                                                            g, nullptr);
  }
  return hipGetLastError();
}

template <int TW, int TH, int DEPTH>
hipError_t launch_bwd(const gs_frame& f, const DevOpts& op, bool have_fwd, bool loss, const BwdArgs& a, bool persist,
                      hipStream_t st) {
  if (f.seg_len > 0) {
    // long lists split into depth segments
    if (have_fwd && loss) return launch_split_bwd<TW, TH, DEPTH, true, true>(f, op, a, persist, st);
    if (have_fwd) return launch_split_bwd<TW, TH, DEPTH, true, false>(f, op, a, persist, st);
    if (loss) return launch_split_bwd<TW, TH, DEPTH, false, true>(f, op, a, persist, st);
    return launch_split_bwd<TW, TH, DEPTH, false, false>(f, op, a, persist, st);
  }
  const int sorted = f.sort_passes & 1;
  const auto* rec = reinterpret_cast<const float4*>(f.rec);
  const auto* rng = reinterpret_cast<const int2*>(f.tile_range);
  const int nb = f.n_tiles, bs = TW * TH;
  const int32_t* vals = f.vals[sorted];
  if (have_fwd && loss)
    k_render_bwd<TW, TH, DEPTH, true, true><<<nb, bs, 0, st>>>(rec, vals, rng, f.cams, f.n_views, nb, f.tile_order,
                                                               op, a);
  else if (have_fwd)
    k_render_bwd<TW, TH, DEPTH, true, false><<<nb, bs, 0, st>>>(rec, vals, rng, f.cams, f.n_views, nb,
                                                                f.tile_order, op, a);
  else if (loss)
    k_render_bwd<TW, TH, DEPTH, false, true><<<nb, bs, 0, st>>>(rec, vals, rng, f.cams, f.n_views, nb,
                                                                f.tile_order, op, a);
  else
    k_render_bwd<TW, TH, DEPTH, false, false><<<nb, bs, 0, st>>>(rec, vals, rng, f.cams, f.n_views, nb,
                                                                 f.tile_order, op, a);
  return hipGetLastError();
}

template <int TW, int TH>
hipError_t launch_count(const gs_frame& f, const DevOpts& op, unsigned long long* counts, hipStream_t st) {
  const int sorted = f.sort_passes & 1;
  k_count_pairs<TW, TH><<<f.n_tiles, TW * TH, 0, st>>>(
      reinterpret_cast<const float4*>(f.rec), f.vals[sorted], reinterpret_cast<const int2*>(f.tile_range), f.cams,
      f.n_views, f.n_tiles, f.tile_order, op, counts);
  return hipGetLastError();
}

}  // namespace

namespace gs_launch {

// Tile shape (one wave per 8x8 sub-tile) and records staged per thread by the forward (o.batch_depth; 0 means 1).
#define GS_TILE_DISPATCH_D(FN, TW, TH, ...)                        \
  do {                                                             \
    if (o.batch_depth == 2) return FN<TW, TH, 2>(__VA_ARGS__);     \
    return FN<TW, TH, 1>(__VA_ARGS__);                             \
  } while (0)
#define GS_TILE_DISPATCH(FN, ...)                                                      \
  do {                                                                                 \
    if (o.tile_w == 16 && o.tile_h == 16) GS_TILE_DISPATCH_D(FN, 16, 16, __VA_ARGS__); \
    if (o.tile_w == 16 && o.tile_h == 8) GS_TILE_DISPATCH_D(FN, 16, 8, __VA_ARGS__);   \
    if (o.tile_w == 8 && o.tile_h == 8) GS_TILE_DISPATCH_D(FN, 8, 8, __VA_ARGS__);     \
    if (o.tile_w == 32 && o.tile_h == 8) GS_TILE_DISPATCH_D(FN, 32, 8, __VA_ARGS__);   \
    return hipErrorInvalidValue;                                                       \
  } while (0)

hipError_t render_fwd(const gs_frame& f, const gs_opts& o, const gs_images& out, hipStream_t st) {
  const DevOpts op = gsk::dev_opts(o);
  GS_TILE_DISPATCH(launch_fwd, f, op, out, st);
}

hipError_t count_pairs(const gs_frame& f, const gs_opts& o, unsigned long long* counts, hipStream_t st) {
  const DevOpts op = gsk::dev_opts(o);
  if (o.tile_w == 16 && o.tile_h == 16) return launch_count<16, 16>(f, op, counts, st);
  if (o.tile_w == 16 && o.tile_h == 8) return launch_count<16, 8>(f, op, counts, st);
  if (o.tile_w == 8 && o.tile_h == 8) return launch_count<8, 8>(f, op, counts, st);
  if (o.tile_w == 32 && o.tile_h == 8) return launch_count<32, 8>(f, op, counts, st);
  return hipErrorInvalidValue;
}

// Where the backward keeps each tile's loss: n_tiles floats behind the segment state.
static float* loss_parts(const gs_frame& f) {
  return f.seg + (size_t)gsk::seg_slots(f.n_tiles, f.seg_cap) * 6 * f.tile_w * f.tile_h;
}

gsk::LossSum tile_losses(const gs_frame& f) { return {loss_parts(f), f.n_tiles, f.loss}; }

hipError_t loss_total(const gs_frame& f, hipStream_t st) {
  k_loss_total<<<1, 1024, 0, st>>>(tile_losses(f));
  return hipGetLastError();
}

hipError_t count_valid(const gs_frame& f, const float* tgt_depth, int64_t max_pixels, hipStream_t st) {
  hipError_t e = fill_i32(f.counters + 2, 0, f.n_views, st);
  if (e != hipSuccess) return e;
  // eight loads a thread, or up to 32 where the views together make more than 128 blocks anyway
  int64_t bx = (max_pixels + kValidThreads * 32 - 1) / (kValidThreads * 32);
  const int64_t wide = (max_pixels + kValidThreads * 8 - 1) / (kValidThreads * 8), most = 128 / f.n_views;
  if (bx < most) bx = wide < most ? wide : most;
  if (bx < 1) bx = 1;
  dim3 grid((unsigned)bx, (unsigned)f.n_views);
  k_count_valid<<<grid, kValidThreads, 0, st>>>(tgt_depth, f.cams, f.counters + 2);
  return hipGetLastError();
}

hipError_t render_bwd(const gs_frame& f, const gs_opts& o, const gs_images* fwd, const gs_loss& l, hipStream_t st) {
  const DevOpts op = gsk::dev_opts(o);
  BwdArgs a;
  a.fwd_rgb = fwd ? fwd->rgb : nullptr;
  a.fwd_depth = fwd ? fwd->depth : nullptr;
  a.fwd_vis = fwd ? fwd->vis : nullptr;
  a.g_rgb = l.g_rgb;
  a.g_depth = l.g_depth;
  a.g_vis = l.g_vis;
  a.tgt_rgb = l.tgt_rgb;
  a.tgt_depth = l.tgt_depth;
  a.n_valid = f.counters + 2;
  a.lambda_d = l.lambda_d;
  a.lambda_ssim = l.lambda_ssim;
  a.ipart = f.ipart;
  a.rec_slot = f.rec_slot;
  a.capacity = f.capacity;
  a.loss_part = loss_parts(f);
  const bool loss = l.tgt_rgb != nullptr;
  GS_TILE_DISPATCH(launch_bwd, f, op, fwd != nullptr, loss, a, o.persistent != 0, st);
}

}  // namespace gs_launch
