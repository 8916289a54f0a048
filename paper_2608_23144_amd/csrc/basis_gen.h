// The seeded draws of GenBasis(s, C, P), Eq. (2), shared by the kernels that
// build basis tables (device code only).
#pragma once

#include "awsrc_internal.h"

namespace awsrc {

// Position of the m-th zero bit (0-based) among the low `width` bits of w.
__device__ __forceinline__ int nth_zero(uint64_t w, int m, int width) {
  uint64_t z = ~w;
  if (width < 64) z &= (1ull << width) - 1ull;
  int pos = 0;
#pragma unroll
  for (int half = 32; half >= 1; half >>= 1) {
    const uint64_t lowmask = (1ull << half) - 1ull;
    const int cnt = __popcll(z & lowmask);
    if (m >= cnt) { m -= cnt; z >>= half; pos += half; }
  }
  return pos;
}

// Bit j of the result is parity(j & c) for j = 64*w .. 64*w + 63: the XOR of
// the patterns "bit b of j" over the set bits b of c.
__device__ __forceinline__ uint64_t hadamard_neg_word(int c, int w) {
  const uint64_t pat[6] = {0xAAAAAAAAAAAAAAAAull, 0xCCCCCCCCCCCCCCCCull, 0xF0F0F0F0F0F0F0F0ull,
                           0xFF00FF00FF00FF00ull, 0xFFFF0000FFFF0000ull, 0xFFFFFFFF00000000ull};
  uint64_t x = 0ull;
#pragma unroll
  for (int b = 0; b < 6; ++b)
    if ((c >> b) & 1) x ^= pat[b];
  if (((c >> 6) & 1) && w == 1) x = ~x;
  return x;
}

// Column p of a seed (counter base `base`, nw sign words): the draw's m-th
// smallest column not drawn yet; marks it in used.
__device__ __forceinline__ int draw_column(uint64_t key, uint64_t base, int nw, int C, int p, uint64_t (&used)[2]) {
  const uint64_t v = splitmix64(key, base + (uint64_t)(nw + p));
  const int m = (int)(((v >> 32) * (uint64_t)(C - p)) >> 32);  // Lemire multiply-shift into [0, C-p)
  const uint64_t valid0 = C < 64 ? (1ull << C) - 1ull : ~0ull;
  const int w0 = C < 64 ? C : 64;
  const int z0 = w0 - __popcll(used[0] & valid0);
  int c;
  if (m < z0) c = nth_zero(used[0], m, w0);
  else c = 64 + nth_zero(used[1], m - z0, 64);
  used[c >> 6] |= 1ull << (c & 63);
  return c;
}

}  // namespace awsrc
