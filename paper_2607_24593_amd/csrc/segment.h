// The key segment of a scoring launch (score.hip): host code, chosen before
// every launch from the launch's row blocks.
#pragma once

#include <algorithm>
#include <cmath>

#include "device_common.h"

namespace pivot {

// A workgroup's prologue (row tile, gates, scales, first keys), as the number
// of keys whose scoring takes as long on a busy CU.  In keys mode each of the
// four waves loads the whole tile of R rows and scores a quarter of the keys.
constexpr int prologue_keys(bool keys_mode, bool fp8, int rows_per_wave) {
  return !keys_mode ? 224 : (fp8 ? 150 : 300) * rows_per_wave;
}

// An idle workgroup's place in the grid, in the same unit (a decode call of 64
// sequences, 20 rows each, of which three have dense rows: 223 us without this
// term, whose dense launch took segments of 64, 184 with it).
constexpr double kIdleKeys = 15.0;

// Blocks above which a launch's workgroups are estimated instead of counted.
constexpr int kCountedBlocks = 256;

// The segment length with the shortest estimated time, up to max_seg: four
// lengths to an octave in keys mode, multiples of 256 in rows mode, from 128
// (64 in rows mode); with paged keys a power of two of at least 128, so that a
// segment starts on a page boundary or lies inside one page.
//   A grid of at most 256 workgroups puts one on a CU and takes as long as the
// longest.  Past that two share a CU and each takes twice as long, also when
// the others are idle (a ragged batch's grid is a rectangle; its idle ones end
// at once but have taken a CU's turn: 15 fp8 sequences of 1.5K-7K keys, four
// rows each, take 15.2 us in segments of 512, a grid of 210, and 19.9 in 384,
// where 175 are busy of 285).  A launch of more ends between two estimates,
// whose mean is taken: whole rounds of 256 average workgroups, and the CUs'
// even share plus most of a workgroup.
//   prologue_keys and the mean are fitted to 476 launches (keys mode 1 to 15
// rows a sequence, rows mode 16 to 32768; 1 to 64 sequences of 500-400000 keys,
// even and ragged, paged and not) timed at each length: the choice takes 1.2%
// (keys mode) and 3.6% (rows mode) more than each launch's best on the mean,
// where halving max_seg while a launch has fewer than 2048 workgroups takes 17%
// and 11%, and an estimate that counts busy workgroups only, with one prologue
// for every tile, 12% and 7%.  Us a launch, best / choice / halving: fp8, 35
// sequences of 8K-79K keys, four rows, paged, 75 / 75 / 88; 64 of 500-100000,
// four rows, 119 / 119 / 119; bf16, 33 of 2.5K-7K, 16 rows, 50 / 52 / 62.
//   Host time for 64 sequences of two blocks 1.4 us, for 64 packed runs of 500
// blocks 1.3.
inline int score_segment(const SeqTable& st, const RowSpace& rs0, const RowSpace* rs1, int rb, int rows_per_wave,
                         int max_seg, bool keys_mode, bool fp8, bool paged) {
  const double load = prologue_keys(keys_mode, fp8, rows_per_wave);
  double keys[kCountedBlocks];  // keys of each row block, while there are few
  double total = 0.0, longest = 0.0;
  bool counted = true;
  int64_t n_blocks = 0, grid_rows[2] = {0, 0}, grid_keys[2] = {0, 0};
  for (int u = 0; u < (rs1 ? 2 : 1); ++u) {
    const RowSpace& rs = u ? *rs1 : rs0;
    for (int b = 0; b < st.n; ++b) {
      const int cnt =
          rs.kind == kProxyRows ? (int)(((int64_t)st.n_rows[b] + rs.step - 1) / rs.step) : st.n_rows[b];
      int hi = std::min(rs.i1, cnt), lo = rs.i0;
      if (rs.kind == kDenseRows) hi = std::min(hi, st.dense_rows[b]);
      if (rs.kind == kProxyRows) lo = std::max(lo, st.first_proxy[b]);
      if (hi <= lo) continue;
      // a block scans the keys of its last row; the last block's last row is hi - 1
      const int64_t p0 = (int64_t)st.q_pos0[b] - rs.shift + 1, last = p0 + (int64_t)(hi - 1) * rs.step;
      const int64_t b0 = (lo - rs.i0) / rb, b1 = (hi - 1 - rs.i0) / rb;
      if (last <= 0) continue;
      grid_keys[u] = std::max(grid_keys[u], last);
      longest = std::max(longest, (double)last);
      if (counted && n_blocks + (b1 - b0 + 1) <= kCountedBlocks) {
        for (int64_t k = b0; k <= b1; ++k) {
          const int64_t x = p0 + (std::min<int64_t>(rs.i0 + (k + 1) * rb, hi) - 1) * rs.step;
          if (x <= 0) continue;  // no key in reach
          keys[n_blocks++] = (double)x;
          total += (double)x;
        }
        continue;
      }
      counted = false;
      const int64_t d = (int64_t)rb * rs.step;
      const int64_t n = std::min<int64_t>(b1 - b0 + 1, d > 0 ? (last - 1) / d + 1 : INT64_MAX);
      n_blocks += n;
      total += (double)n * ((double)last - 0.5 * (double)(n - 1) * (double)d);
    }
    grid_rows[u] = (int64_t)st.n * ((rs.i1 - rs.i0 + rb - 1) / rb);
  }
  int best = max_seg;
  double best_cost = 0.0;
  auto shorter = [&](int seg) {
    if (paged || (!keys_mode && seg <= 256)) return seg / 2;
    return seg - (keys_mode ? std::max(64, (int)(1u << (31 - __builtin_clz((unsigned)seg - 1))) / 4) : 256);
  };
  for (int seg = max_seg; seg >= (paged || keys_mode ? 128 : 64); seg = shorter(seg)) {
    const double per = 1.0 / seg;
    // rows mode: a last segment of a few keys takes next to nothing
    const int64_t least = keys_mode ? 0 : seg / 16;
    double wgs = total * per + 0.5 * (double)n_blocks;
    if (counted) {  // (x - 0.5) / seg lies at least 0.5 / seg from a whole number: exact
      int sum = 0;
      for (int64_t i = 0; i < n_blocks; ++i) sum += (int)(std::max(0.0, keys[i] - 0.5 - (double)least) * per);
      wgs = (double)(sum + n_blocks);
    }
    auto segs = [&](int64_t n) { return n > 0 ? (std::max<int64_t>(n - least, 1) + seg - 1) / seg : 0; };
    const int64_t grid = grid_rows[0] * segs(grid_keys[0]) + grid_rows[1] * segs(grid_keys[1]);
    const double wg = load + std::min((double)seg, longest);
    double cost = wg;
    if (wgs > 256.0 || grid > (keys_mode ? 256 : 264)) {  // (rows mode: the last few rarely meet a long one)
      const double rounds = std::max(2.0, std::ceil(wgs / 256.0)) * (load + total / std::max(wgs, 1.0));
      cost = 0.5 * (rounds + (wgs * load + total) / 256.0 + (keys_mode ? 0.75 : 0.5) * wg) +
             kIdleKeys / 256.0 * std::max(0.0, (double)grid - wgs);
    }
    if (seg == max_seg || cost < best_cost) {
      best = seg;
      best_cost = cost;
    }
  }
  return best;
}

}  // namespace pivot
