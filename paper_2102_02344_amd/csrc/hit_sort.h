// Argmax positions of one sample's channels sorted by point.
#pragma once
#include "common.h"

namespace hfta {

constexpr int HIT_THREADS = 1024;

// Argmax positions of one (model, sample) sorted by point, ties in channel order: key = point << 10 | channel (Co <= 1024,
// L < 2^21: checked on the host); bitonic, a key per thread, exchanged by shuffles inside a wavefront and through LDS
// across (10 of the 55 exchanges, where a barrier each took 15 us).  P: Co rounded up to a power of two.
// toff[tile] = first sorted position whose point lies in 128-point tile `tile` or later.
__device__ __forceinline__ void sort_hits(const int32_t* idx, int64_t idx_stride, const float* s, uint32_t* skey, float* sval, int* toff,
                                          int Co, int L, uint32_t (&sh)[2][HIT_THREADS], int P, int tiles) {
  const int t = threadIdx.x;
  uint32_t key = 0xffffffffu;
  if (t < Co) {
    const int hit = min(max(idx[t * idx_stride], 0), L - 1);
    key = ((uint32_t)hit << 10) | (uint32_t)t;
  }
  int buf = 0;
  for (int k = 2; k <= P; k <<= 1)
    for (int j = k >> 1; j > 0; j >>= 1) {
      uint32_t o;
      if (j < 64) {
        o = (uint32_t)__shfl_xor((int)key, j, 64);
      } else {                                               // the other buffer was last read before the last barrier
        sh[buf][t] = key;
        __syncthreads();
        o = sh[buf][t ^ j];
        buf ^= 1;
      }
      key = ((t & j) == 0) == ((t & k) == 0) ? min(key, o) : max(key, o);
    }
  sh[buf][t] = key;
  __syncthreads();
  if (t < Co) {
    skey[t] = key;
    sval[t] = s[key & 1023u];
  }
  for (int k = t; k <= Co; k += HIT_THREADS) {
    const int cur = k < Co ? (int)(sh[buf][k] >> 17) : tiles;
    const int prev = k > 0 ? (int)(sh[buf][k - 1] >> 17) : -1;
    for (int tl = prev + 1; tl <= cur; ++tl) toff[tl] = k;
  }
}

}  // namespace hfta
