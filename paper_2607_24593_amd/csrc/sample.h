// Which part of a row held in registers the resident select samples
// (select.hip).
#pragma once

#include <hip/hip_runtime.h>

namespace pivot {

// A workgroup of `waves` (a power of two up to 16) waves holds a row as vn
// vectors per thread; block v * waves + w of 64 vectors, in row order, is wave
// w's v-th.  Each wave samples one of its blocks: this is wave w's vector v,
// such that the waves' blocks are one out of every vn consecutive ones.  (A
// choice of v by w alone, such as w mod vn, favours a part of the row wherever
// vn does not divide waves, and misses the rest where vn is larger: scores that
// drift along the row then mislead the sample.)
//   Block i vn + y + o of stratum i: with d = gcd(vn, waves), the blocks i vn
// fall on waves/d different waves, d turns of them, and each turn takes another
// y in [0, d); o centres them.  The y of consecutive turns lie on either side of
// the middle (0, d - 1, 1, d - 2, ...), so that they don't drift along the row
// themselves.  Solved here for i, given the wave.
__host__ __device__ inline int sampled_vector(int w, int waves, int vn) {
  const int lw = 31 - __builtin_clz((unsigned)waves), lv = __builtin_ctz((unsigned)vn);
  const int ld = lv < lw ? lv : lw, d = 1 << ld;
  const int o = (vn - d) / 2, x = (w - o) & (waves - 1), y = x & (d - 1);
  const int turn = 2 * y < d ? 2 * y : 2 * (d - 1 - y) + 1;
  const int u = vn >> ld, inv = u * (2 - u * u);  // u inv = 1 modulo 16 where u is odd (else waves/d = 1)
  const int i = turn * (waves >> ld) + (((x >> ld) * inv) & ((waves >> ld) - 1));
  return (i * vn + y + o) >> lw;
}

}  // namespace pivot
