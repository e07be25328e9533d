// The look-back of a chained scan (Merrill and Garland's single-pass prefix
// scan with decoupled look-back, 2016): what lies before a tile, from the words
// that the tiles before it publish.
#pragma once

#ifdef __HIPCC__
#include <hip/hip_runtime.h>
#define G4D_CHAIN_FN __device__ __forceinline__
#else
#define G4D_CHAIN_FN inline  // (for the host test of the waits)
#endif
#include <stdint.h>

namespace g4d {

// A tile's word: nothing yet (0), its own count, or the sum up to and with it.
constexpr uint32_t kChainCount = 1u << 30, kChainSum = 2u << 30, kChainMask = kChainCount - 1u;
constexpr int kChainWindow = 8;  // earlier tiles read at once
// Readings in a row without a new word after which a tile stops waiting, about half
// a second of them. Earlier tiles publish within microseconds; a word never
// comes only if other work writes the same words meanwhile (calls that must not
// overlap do). The sum is then wrong, and every wait still ends.
constexpr uint32_t kChainPolls = 1u << 18;

// The sum of the tiles before `tile`; load(t) reads tile t's word.
template <typename Load>
G4D_CHAIN_FN uint32_t chain_sum_before(int tile, uint32_t polls, const Load& load) {
  uint32_t sum = 0, idle = 0;
  int j = tile - 1;
  while (j >= 0) {
    uint32_t w[kChainWindow];
#pragma unroll
    for (int i = 0; i < kChainWindow; ++i) w[i] = j - i >= 0 ? load(j - i) : kChainSum;
    int step = 0;
    bool open = true;
#pragma unroll
    for (int i = 0; i < kChainWindow; ++i) {
      open = open && w[i] != 0u;
      if (open) {
        sum += w[i] & kChainMask;
        step = (w[i] & kChainSum) ? j + 1 : i + 1;
        open = !(w[i] & kChainSum);
      }
    }
    j -= step;
    idle = step ? 0u : idle + 1u;
    if (idle >= polls) break;
  }
  return sum;
}

}  // namespace g4d
