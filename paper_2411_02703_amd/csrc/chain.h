// The look-back of the radix sort's chained scan (bin.hip), free of device code so that a host program can run it too.
#pragma once

#include <stdint.h>

#if defined(__HIPCC__)
#define GS_HD __host__ __device__ inline __attribute__((always_inline))
#define GS_UNROLL _Pragma("unroll")
#else
#define GS_HD inline
#define GS_UNROLL
#endif

namespace gsk {

// A tile's state for one digit: 0 so far absent, 1 + the count of its keys, or with the top bit the count of its and all
// earlier tiles' keys (below 2^31, as the sizes are).  Written and read whole, so that no other ordering is needed.
constexpr uint32_t kWhole = 0x80000000u;

// Looks at the states before a tile, LOOK of them each, after which it gives up.  The tiles before a running one belong to
// blocks that run or have finished, so a wait takes microseconds and a sum over 2^31 keys 2^15 looks; only two sorts at a
// time on the same state words (which callers have to keep apart) can take away a state that is waited for.  Such a tile
// goes on with a wrong count after about a second: the order is lost, but the kernel ends.
constexpr int kChainLooks = 1 << 20;

// Keys of one digit in the tiles before `tile` > 0: their states (load(j): tile j's) added up from the last one back to
// the first that holds a whole sum (tile 0's always does), LOOK of them in flight.
template <int LOOK, class Load>
GS_HD uint32_t keys_before(int tile, int looks, Load load) {
  uint32_t before = 0;
  int j = tile - 1;
  for (int look = 0; look < looks; ++look) {
    uint32_t v[LOOK];
    GS_UNROLL for (int i = 0; i < LOOK; ++i) v[i] = load(j - i > 0 ? j - i : 0);
    bool done = false;
    GS_UNROLL for (int i = 0; i < LOOK; ++i) {
      if (done || v[i] == 0) break;  // (absent so far: read again from here)
      done = (v[i] & kWhole) != 0;
      before += done ? v[i] & ~kWhole : v[i] - 1u;
      --j;
    }
    if (done) break;
  }
  return before;
}

// The place of a tile's p-th key in the output of n, `first` being its digit's first place less the tile's keys of lower
// digits.  Below n whatever the counts that it is formed from.
GS_HD uint32_t key_place(uint32_t first, int p, uint32_t n) {
  const uint32_t at = first + (uint32_t)p;
  return at < n ? at : n - 1u;
}

}  // namespace gsk
