// Per-row top-m selection over score rows of fp32, or of bf16 (the rows the
// fp8 path writes; every bf16 value widens exactly to the fp32 it selects
// on), for the TopK of Sec. 3.1 and of Eqs. 6-7, one workgroup per row:
//   rows of at most 32768 scores (131072 bf16 or 65536 fp32 ones when a launch
//     has at most 256 rows, as in decode): topk_resident_kernel, the whole row
//     in registers (but for two shapes of fp32 launches, topk_launch);
//   other rows: 512 threads streaming the row (topk_rows16_kernel for bf16,
//     topk_rows_kernel), or, for a launch of at most 256 rows given scratch,
//     the split select described below.
//
// Long rows (n >= kSampleMinLen) are read once when the expected number of
// compacted keys fits in LDS:
//   1 sample   every stride-th 256-byte chunk of the row (at most 8192
//              fp32 or 16384 bf16 scores) is held in registers; two histogram passes over the
//              sample (top 12, then next 8 key bits) find a 20-bit prefix
//              `thr` such that at least ts sampled keys have prefix >= thr,
//              where ts is the sample's expected share of m plus four
//              standard deviations;
//   2 compact  one pass over the row appends every key with prefix >= thr to
//              LDS (at most CAP: 4096 for m <= 2048, else 8000; each wave
//              fills its own CAP / waves entries, slots from a ballot prefix)
//              (a row whose ts, scaled to the whole row, would fill more
//              than 80% of CAP skips the sample and takes the two-pass path);
//   3 select   if the pass found at least m keys (and no wave more than its
//              share of CAP),
//              they include every key >= the m-th largest of the row, ties
//              included, so block_select() over them is exact; otherwise the
//              row takes the two-pass path below.
// Few long rows (decode) with a scratch buffer: step 1 runs in
// topk_thr_kernel (one workgroup per row writes the row's threshold), step 2
// in topk_slice_kernel on P workgroups per row (each compacts 1/P of the row
// into scratch), step 3 in topk_merge_kernel, which gathers the row's
// compacted keys into LDS; one workgroup per row could not pull its row fast
// enough on its own.
// Other rows: two_level_select() (block_select.h) over the row in global
// memory: pass 1 builds a 4096-bin histogram of the top 12 key bits, pass 2
// emits the keys above the threshold bin and compacts that bin into LDS, where
// the remaining bits are resolved (ties: lower position); a threshold bin that
// overflows LDS (e.g. many equal scores) selects directly over the row.
// A row with no more than m valid entries returns all of them, then -1.
#include <algorithm>
#include <climits>
#include <cstring>

#include "block_select.h"
#include "launch.h"
#include "sample.h"

namespace pivot {

constexpr int kSelThreads = 512;
constexpr int kSelThreadsWide = 1024;  // few long rows: one workgroup per row must pull the row alone
constexpr int kWideMaxRows = kSplitMaxRows;  // "few": at most one row per CU
// LDS candidates: 16 KiB histogram + 32 KiB -> three workgroups per CU, or
// + 62.5 KiB -> two
constexpr int kSelCapSmall = 4096;
constexpr int kSelCapLarge = 8000;
constexpr int kSelCap16 = 7680;  // bf16 rows: 6-byte candidates, three 512-thread workgroups per CU
constexpr int kSampleMinLen = kSplitMinKeys;  // shorter rows take the two-pass path
constexpr int kChunk4 = 16;           // float4 per sampled chunk (256 bytes)
constexpr int kSampleChunks = 128;    // at most 8192 sampled scores
// split select: scratch entries per row over its P slices (each slice may hold
// twice its even share of the merge capacity), P in [kSplitMinP, kSplitMaxP]
constexpr int kSplitThreads = 256;
constexpr int kSplitSlots = 2 * kSelCapLarge;
constexpr int kSplitMinP = 4, kSplitMaxP = 16;
constexpr int kSplitPerMax = kSplitSlots / kSplitMinP;
constexpr int kSplitTargetBlocks = 1024;
// Largest m of the resident select: the sample's threshold then keeps at most
// 80% of its candidate buffer (kSelCap16) for every row length it takes.
constexpr int kResidentMaxM = 4608;

// Elements of a score row (fp32 or bf16, E), visited with 16-byte vector
// loads (U in flight per thread) when aligned.
template <int T, int U, class E>
struct RowSource {
  using SV = ScoreVec<E>;
  static constexpr int N = SV::N;
  const E* row;
  int count;
  template <class F>
  __device__ __forceinline__ void visit(F f) const {
    const int tid = threadIdx.x;
    if ((reinterpret_cast<uintptr_t>(row) & 15u) == 0) {
      const int nv = count / N;
      const uint4* r16 = reinterpret_cast<const uint4*>(row);
      auto each = [&](const uint4& a, int i) {
        float v[N];
        SV::unpack(a, v);
#pragma unroll
        for (int j = 0; j < N; ++j) f(float_key(v[j]), N * i + j);
      };
      int i = tid;
      for (; i + (U - 1) * T < nv; i += U * T) {
        uint4 a[U];
#pragma unroll
        for (int u = 0; u < U; ++u) a[u] = r16[i + u * T];
#pragma unroll
        for (int u = 0; u < U; ++u) each(a[u], i + u * T);
      }
      for (; i < nv; i += T) each(r16[i], i);
      for (int e = N * nv + tid; e < count; e += T) f(float_key(SV::one(row, e)), e);
    } else {
      for (int e = tid; e < count; e += T) f(float_key(SV::one(row, e)), e);
    }
  }
};

// The sampled keys (positions are not needed): V 16-byte vectors of N
// scores per thread.
template <int V, int N>
struct SampleSource {
  uint32_t key[N * V];
  bool ok[V];
  template <class F>
  __device__ __forceinline__ void visit(F f) const {
#pragma unroll
    for (int v = 0; v < V; ++v)
      if (ok[v]) {
#pragma unroll
        for (int j = 0; j < N; ++j) f(key[N * v + j], 0);
      }
  }
};

// 20-bit key prefix of the ts-th largest sampled key (ts <= sampled count);
// hist: 4096 bins of LDS.
template <int T, class Src>
__device__ uint32_t sample_prefix(const Src& src, uint32_t ts, uint32_t* hist, SelectShared& sh) {
  const int tid = threadIdx.x;
  for (int k = tid; k < 4096; k += T) hist[k] = 0;
  __syncthreads();
  src.visit([&](uint32_t key, int32_t) { atomicAdd(&hist[key >> 20], 1u); });
  __syncthreads();
  find_digit<T, true, 4096>(hist, sh, ts);
  const uint32_t d1 = sh.digit, rem = ts - sh.before;
  __syncthreads();
  for (int k = tid; k < 256; k += T) hist[k] = 0;
  __syncthreads();
  src.visit([&](uint32_t key, int32_t) {
    if ((key >> 20) == d1) atomicAdd(&hist[(key >> 12) & 255u], 1u);
  });
  __syncthreads();
  find_digit<T, true, 256>(hist, sh, rem);
  const uint32_t thr = (d1 << 8) | sh.digit;
  __syncthreads();
  return thr;
}

// A key near the ts-th largest sampled key (ts <= sampled count), from one
// pass over the top 12 key bits: the place of the ts-th key inside its bin (an
// eighth of an octave) is taken in proportion to its rank there.  The tail's
// density falls by less than half over such a bin, so the count above the
// result is a few per cent of the bin off, well inside the four standard
// deviations that ts allows for.
template <int T, class Src>
__device__ __forceinline__ uint32_t sample_base(const Src& src, uint32_t ts, uint32_t* hist, SelectShared& sh) {
  const int tid = threadIdx.x;
  for (int k = tid; k < 4096; k += T) hist[k] = 0;
  __syncthreads();
  src.visit([&](uint32_t key, int32_t) { atomicAdd(&hist[key >> 20], 1u); });
  __syncthreads();
  find_digit<T, true, 4096>(hist, sh, ts);
  const float below = (float)(sh.equal - (ts - sh.before)) / (float)sh.equal;  // in [0, 1)
  return (sh.digit << 20) + min((uint32_t)(below * 0x1p20f), 0xFFFFFu);
}

// Steps 1 of the one-read path for a long aligned row: false (before any
// load) when the expected compacted count ts n / s would not leave room for
// its spread in CAP entries; else the threshold score fthr (every key with
// prefix >= thr compares >= fthr as a float).  Uniform over the workgroup.
template <int T, int CAP, class E>
__device__ bool sample_threshold(const E* row, int n, int m, uint32_t* hist, SelectShared& sel, float& fthr) {
  using SVec = ScoreVec<E>;
  constexpr int N = SVec::N;
  constexpr int SV = kSampleChunks * kChunk4 / T;  // sampled 16-byte vectors per thread
  const int tid = threadIdx.x;
  const int nch = n / (N * kChunk4);
  const int stride = max(16, (nch + kSampleChunks - 1) / kSampleChunks);
  const int sch = (nch + stride - 1) / stride;  // chunks 0, stride, 2 stride, ... < nch
  const int s = sch * N * kChunk4;
  const float rm = (float)s * (float)m / (float)n;
  const uint32_t ts = (uint32_t)ceilf(rm + 4.0f * sqrtf(rm)) + 1u;
  if (!(ts < (uint32_t)s && (float)ts * (float)n <= 0.8f * (float)CAP * (float)s)) return false;
  const uint4* r16 = reinterpret_cast<const uint4*>(row);
  SampleSource<SV, N> smp;
#pragma unroll
  for (int v = 0; v < SV; ++v) {
    const int qi = tid + T * v;
    smp.ok[v] = qi < sch * kChunk4;
    const uint4 a = smp.ok[v] ? r16[(int64_t)(qi / kChunk4) * stride * kChunk4 + qi % kChunk4] : make_uint4(0u, 0u, 0u, 0u);
    float x[N];
    SVec::unpack(a, x);
#pragma unroll
    for (int j = 0; j < N; ++j) smp.key[N * v + j] = float_key(x[j]);
  }
  const uint32_t thr = sample_prefix<T>(smp, ts, hist, sel);
  // key >> 12 >= thr  <=>  score >= the smallest score with that prefix
  // (the key map is monotone; -0 and +0 share a key and compare equal)
  fthr = key_float(thr << 12);
  return true;
}

// Step 2 of the one-read path: wave w appends the keys >= fthr it reads to
// its own segment [w SEG, (w + 1) SEG) of (ckey, cpos), a ballot prefix
// giving each lane its slot (no LDS atomics in the stream), then the segments
// are packed to the front.  The loops are uniform over the wave, so the
// running count stays the same in every lane.  Returns the number of keys, or
// CAP + 1 when a segment overflowed.  Aligned rows only.  KT: the stored key,
// the order-preserving uint32 key, or its upper half for bf16 rows (whose
// keys have 16 significant bits, key16_expand() restores them).
template <int T, int U, int CAP, class E, class KT = uint32_t>
__device__ __forceinline__ int stream_compact(const E* row, int n, float fthr, KT* ckey, int32_t* cpos,
                                              int32_t* wcnt) {
  using SV = ScoreVec<E>;
  constexpr int N = SV::N;
  constexpr int NW = T / 64, SEG = CAP / NW, R = (SEG + 63) / 64;
  constexpr int KSHIFT = 32 - 8 * (int)sizeof(KT);
  const int tid = threadIdx.x, lane = tid & 63;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  KT* mk = ckey + wv * SEG;
  int32_t* mp = cpos + wv * SEG;
  int wc = 0;
  auto take = [&](bool valid, float v, int pos) {
    const bool t = valid && v >= fthr;
    const uint64_t bal = __ballot(t);
    if (bal) {
      const int slot =
          wc + (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(bal >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)bal, 0u));
      if (t && slot < SEG) {
        mk[slot] = (KT)(float_key(v) >> KSHIFT);
        mp[slot] = pos;
      }
      wc += (int)__popcll((unsigned long long)bal);
    }
  };
  const int nv = n / N;
  const uint4* r16 = reinterpret_cast<const uint4*>(row);
  int base = 0;
  for (; base + U * T <= nv; base += U * T) {
    uint4 a[U];
#pragma unroll
    for (int u = 0; u < U; ++u) a[u] = r16[base + u * T + tid];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      float x[N];
      SV::unpack(a[u], x);
      const int p = N * (base + u * T + tid);
#pragma unroll
      for (int j = 0; j < N; ++j) take(true, x[j], p + j);
    }
  }
  for (; base < nv; base += T) {
    const int q = base + tid;
    const bool ok = q < nv;
    float x[N];
    SV::unpack(ok ? r16[q] : make_uint4(0u, 0u, 0u, 0u), x);
#pragma unroll
    for (int j = 0; j < N; ++j) take(ok, x[j], N * q + j);
  }
  if (N * nv < n) {  // the n mod N tail
    const int e = N * nv + tid;
    const bool ok = e < n;
    take(ok, ok ? SV::one(row, e) : 0.f, e);
  }
  if (lane == 0) wcnt[wv] = wc;
  __syncthreads();
  int pre = 0, tot = 0;
  bool over = false;
#pragma unroll
  for (int w = 0; w < NW; ++w) {
    const int c = wcnt[w];
    pre += w < wv ? c : 0;
    tot += c;
    over |= c > SEG;
  }
  if (over) return CAP + 1;
  // a segment moves left onto space other waves may still be reading:
  // through registers, with a barrier in between
  KT kk[R];
  int32_t pp[R];
#pragma unroll
  for (int j = 0; j < R; ++j) {
    const int e = lane + 64 * j;
    if (e < wc) {
      kk[j] = mk[e];
      pp[j] = mp[e];
    }
  }
  __syncthreads();
#pragma unroll
  for (int j = 0; j < R; ++j) {
    const int e = lane + 64 * j;
    if (e < wc) {
      ckey[pre + e] = kk[j];
      cpos[pre + e] = pp[j];
    }
  }
  __syncthreads();
  return tot;
}

// Where row (b, i)'s indices go (OutDesc).
struct RowDest {
  int32_t* base;
  int64_t dest0;
  int ndest;
  int ld;
  __device__ RowDest(const OutDesc& od, const SeqTable& st, int b, int i) : base(od.base), ld(od.ld) {
    if (od.fan_g == 0) {
      dest0 = (int64_t)(od.groups ? st.grp0[b] : st.row0[b]) + i;
      ndest = 1;
    } else {
      dest0 = (int64_t)st.row0[b] + (int64_t)i * od.fan_g;
      ndest = min(od.fan_g, st.n_rows[b] - i * od.fan_g);
    }
  }
  __device__ __forceinline__ void operator()(int p, int32_t v) const {
    for (int u = 0; u < ndest; ++u) base[(dest0 + u) * ld + p] = v;
  }
};

// SAMPLE: the launch holds rows long enough for the one-read path (a launch
// of short rows only takes the kernel without it, which keeps the two-pass
// loops as lean as they compile alone).  Register budget: as many 512-thread
// workgroups per CU as LDS allows (three for CAP 4096, else two).
template <int CAP, int T, bool SAMPLE, class E>
__global__ __launch_bounds__(T) __attribute__((amdgpu_waves_per_eu(CAP == kSelCapSmall && T == kSelThreads ? 6 : 4)))
void topk_rows_kernel(const E* __restrict__ scores, int64_t ld, SeqTable st, RowSpace rs, OutDesc od) {
  // 16-byte row loads in flight per thread (the same bytes for bf16 rows,
  // whose vectors hold twice as many scores)
  constexpr int U = T == kSelThreads ? 4 : 8;
  __shared__ TwoLevelShared<CAP> sh;
  const int nrows = rs.i1 - rs.i0;
  const int b = blockIdx.x / nrows;
  const int i = rs.i0 + blockIdx.x % nrows;
  if (!row_active(st, rs, b, i)) return;
  const int tid = threadIdx.x;
  const int64_t n64 = row_limit(st, rs, b, i) + 1;
  const int n = (int)max((int64_t)0, n64);
  const E* row = scores + ((int64_t)b * nrows + (i - rs.i0)) * ld;
  const int m = od.m;
  const RowDest put(od, st, b, i);
  if (n <= m) {
    for (int p = tid; p < m; p += T) put(p, p < n ? p : -1);
    return;
  }
  if (tid == 0) sh.sel.emitted = 0;
  RowSource<T, U, E> src{row, n};
  const bool aligned = (reinterpret_cast<uintptr_t>(row) & 15u) == 0;
  float fthr;
  if (SAMPLE && n >= kSampleMinLen && aligned) {
    if (sample_threshold<T, CAP>(row, n, m, sh.hist, sh.sel, fthr)) {
      __shared__ int32_t wcnt[T / 64];
      const int found = stream_compact<T, U, CAP>(row, n, fthr, sh.ckey, sh.cpos, wcnt);
      if (found >= m && found <= CAP) {
        ArraySource<T> cand{sh.ckey, sh.cpos, found};
        // the sample's histogram is free: it serves the bucket pass and its list
        if (!bucket_select<T>(cand, (uint32_t)m, sh.hist, sh.hist, reinterpret_cast<int32_t*>(sh.hist + kBucketList),
                              &sh.lcount, sh.sel, put))
          block_select<T, false>(cand, (uint32_t)m, sh.sel, put);
        return;
      }
    }
  }
  two_level_select<T>(src, (uint32_t)m, sh, put);
}

// The order-preserving key of a bf16 score from its upper half: the lower
// half of a bf16 value's fp32 key is 0 for +0 and positive values, 0xFFFF for
// negative ones (float_key complements them).
__device__ __forceinline__ uint32_t key16_expand(uint32_t k16) {
  return (k16 << 16) | ((k16 & 0x8000u) ? 0u : 0xFFFFu);
}

// Elements e = tid, tid + THREADS, ... < count of (16-bit key, position) arrays.
template <int THREADS>
struct ArraySource16 {
  const uint16_t* key;
  const int32_t* pos;
  int count;
  template <class F>
  __device__ __forceinline__ void visit(F f) const {
    for (int e = threadIdx.x; e < count; e += THREADS) f(key16_expand(key[e]), pos[e]);
  }
};

// Members of one tied value (equal keys): positions only.
template <int THREADS>
struct TieSource {
  const int32_t* pos;
  int count;
  template <class F>
  __device__ __forceinline__ void visit(F f) const {
    for (int e = threadIdx.x; e < count; e += THREADS) f(0u, pos[e]);
  }
};

// The candidates of stream_compact16 in place: wave w's wcnt[w] entries
// start at w * SEG; element e of the concatenation lies in the segment whose
// prefix count it reaches.
template <int THREADS, int NW, int SEG>
struct SegSource16 {
  const uint16_t* key;
  const int32_t* pos;
  int pre[NW + 1];  // prefix counts of the segments
  __device__ SegSource16(const uint16_t* k, const int32_t* p, const int32_t* wcnt) : key(k), pos(p) {
    pre[0] = 0;  // uniform: scalar registers
#pragma unroll
    for (int w = 0; w < NW; ++w) pre[w + 1] = __builtin_amdgcn_readfirstlane(pre[w] + wcnt[w]);
  }
  __device__ __forceinline__ int count() const { return pre[NW]; }
  __device__ __forceinline__ int index(int e) const {
    int w = 0, base = 0;  // compares, not an indexed read (which would put pre[] in scratch)
#pragma unroll
    for (int k = 1; k < NW; ++k)
      if (e >= pre[k]) {
        w = k;
        base = pre[k];
      }
    return w * SEG + (e - base);
  }
  template <class F>
  __device__ __forceinline__ void visit(F f) const {
    for (int e = threadIdx.x; e < pre[NW]; e += THREADS) {
      const int i = index(e);
      f(key16_expand(key[i]), pos[i]);
    }
  }
};

// LDS of topk_rows16_kernel: one region serves, in turn, the sampling
// histogram (4096 words), the candidates (16-bit keys and int32 positions,
// CAP each) with the exact select's histogram (kNB16 words), or, for a row
// that falls back, the two-level select's buffers (TwoLevelShared<CAP2>).
constexpr int kNB16 = 1024;
template <int CAP>
struct Rows16Lds {
  static constexpr int KEY_BYTES = (2 * CAP + 15) / 16 * 16;
  static constexpr int POS_BYTES = 4 * CAP;
  static constexpr int MAIN = KEY_BYTES + POS_BYTES + 4 * kNB16;
  static constexpr int CAP2 = ((MAIN - (int)sizeof(TwoLevelShared<0>)) / 8) / 64 * 64;
  static constexpr int RAW = MAIN > 4 * 4096 ? MAIN : 4 * 4096;
  static_assert((int)sizeof(TwoLevelShared<CAP2>) <= RAW, "fallback fits the region");
};

// The 16-bit order-preserving keys of the two bf16 scores of a word
// (key16_expand(k) == float_key(score)), without branches: a half with its
// sign bit set is complemented, any other gets its sign bit set; -0 (0x8000)
// then lands on 0x7FFF, one below +0's key 0x8000, and is moved up to it.
__device__ __forceinline__ uint32_t key16_pair(uint32_t w) {
  const uint32_t t = (w >> 15) & 0x00010001u;  // the sign of each half in its bit 0
  const uint32_t k = w ^ (t * 0x7FFFu | 0x80008000u);
  return k + (((k & 0xFFFFu) == 0x7FFFu ? 1u : 0u) | ((k >> 16) == 0x7FFFu ? 0x10000u : 0u));
}

// The 16-bit order key of one bf16 value (key16_pair of one half).
__device__ __forceinline__ uint32_t key16_one(uint32_t h) {
  const uint32_t k = h ^ ((h & 0x8000u) ? 0xFFFFu : 0x8000u);
  return k + (k == 0x7FFFu ? 1u : 0u);
}

// The sampled keys of bf16 rows, packed two per register: V 16-byte vectors
// per thread.
template <int V>
struct SampleSource16 {
  uint32_t pk[4 * V];
  bool ok[V];
  template <class F>
  __device__ __forceinline__ void visit(F f) const {
#pragma unroll
    for (int v = 0; v < V; ++v)
      if (ok[v]) {
#pragma unroll
        for (int j = 0; j < 8; ++j) f(key16_expand((pk[4 * v + j / 2] >> (16 * (j & 1))) & 0xFFFFu), 0);
      }
  }
};

// sample_threshold for bf16 rows with the sample held as packed 16-bit keys, in
// 256-byte chunks: at first SCH of them (32, 4096 scores, for the large
// candidate buffer, where the count above the threshold spreads by ~8% of m at
// 131072 scores inside the room CAP leaves; 64 for the small one, m <= 2048,
// whose room is tighter), doubled up to 128 while the expected count does not
// fit.  Rows of over 250000 scores need that: with 4096 samples they went to
// the two-pass select, 950 us a launch of 2040 rows of 245760-262144 instead of 250.
// base16 receives the 16-bit key below which no kept key lies, fthr its score.
template <int T, int CAP, int SCH>
__device__ bool sample_threshold16(const bf16_t* row, int n, int m, uint32_t* hist, SelectShared& sel, float& fthr,
                                   uint32_t& base16) {
  constexpr int N = 8, MAX = 128;
  constexpr int SV = MAX * kChunk4 / T;  // sampled 16-byte vectors per thread, at most
  const int tid = threadIdx.x;
  const int nch = n / (N * kChunk4);
  int stride = 0, sch = 0;
  uint32_t ts = 0;
  bool fits = false;
#pragma unroll 1
  for (int most = SCH; most <= MAX && !fits; most *= 2) {
    stride = max(16, (nch + most - 1) / most);
    sch = (nch + stride - 1) / stride;
    const int s = sch * N * kChunk4;
    const float rm = (float)s * (float)m / (float)n;
    ts = (uint32_t)ceilf(rm + 4.0f * sqrtf(rm)) + 1u;
    fits = ts < (uint32_t)s && (float)ts * (float)n <= 0.8f * (float)CAP * (float)s;
  }
  if (!fits) return false;
  const uint4* r16 = reinterpret_cast<const uint4*>(row);
  SampleSource16<SV> smp;
#pragma unroll
  for (int v = 0; v < SV; ++v) {
    const int qi = tid + T * v;
    smp.ok[v] = qi < sch * kChunk4;
    const uint4 a = smp.ok[v] ? r16[(int64_t)(qi / kChunk4) * stride * kChunk4 + qi % kChunk4] : make_uint4(0u, 0u, 0u, 0u);
    smp.pk[4 * v + 0] = key16_pair(a.x);
    smp.pk[4 * v + 1] = key16_pair(a.y);
    smp.pk[4 * v + 2] = key16_pair(a.z);
    smp.pk[4 * v + 3] = key16_pair(a.w);
  }
  base16 = sample_base<T>(smp, ts, hist, sel) >> 16;
  fthr = key_float(key16_expand(base16));
  return true;
}

// Step 2 for bf16 rows: stream_compact storing 16-bit keys, with the next U
// vectors' loads issued before the current ones are examined, and every kept
// key counted in `hist` (kNB16 words, zeroed by the caller) at its distance
// above the threshold, bin min(k16 - base16, kNB16 - 1): below the top bin,
// one bin per bf16 value.  The waves' segments stay where they are (counts in
// wcnt; SegSource16 reads them in place).
template <int T, int U, int CAP>
__device__ __forceinline__ int stream_compact16(const bf16_t* row, int n, float fthr, uint32_t base16,
                                                uint16_t* ckey, int32_t* cpos, uint32_t* hist, int32_t* wcnt) {
  static_assert(8 * U <= 32, "one 32-bit mask per batch");
  using SV = ScoreVec<bf16_t>;
  constexpr int N = SV::N;
  constexpr int NW = T / 64, SEG = CAP / NW;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  uint16_t* mk = ckey + wv * SEG;
  int32_t* mp = cpos + wv * SEG;
  int wc = 0;  // keys this wave has kept (the same in every lane)
  // Appends the kept scores of a batch (bit 8 u + j of `bits`: score j of the
  // lane's vector u, which is vector q0 + u T of the row): a wave prefix sum
  // of the lanes' counts gives each lane its first slot, then every lane
  // writes its own keys, vector by vector, a loop over its set bits (rarely
  // more than two per vector).
  auto append = [&](const uint4 (&a)[U], uint32_t bits, int q0) {
    const uint32_t cnt = (uint32_t)__popc(bits);
    const uint32_t incl = wave_incl_sum(cnt);
    int slot = wc + (int)(incl - cnt);
    wc += __builtin_amdgcn_readlane((int)incl, 63);
#pragma unroll
    for (int u = 0; u < U; ++u) {  // a static vector index: its words stay in registers
      uint32_t mu = (bits >> (N * u)) & 0xFFu;
      const uint64_t lo = ((uint64_t)a[u].y << 32) | a[u].x, hi = ((uint64_t)a[u].w << 32) | a[u].z;
      while (mu) {
        const int j = __builtin_ctz(mu);
        mu &= mu - 1;
        const uint32_t h = (uint32_t)(((j & 4) ? hi : lo) >> (16 * (j & 3))) & 0xFFFFu;
        const uint32_t k16 = key16_one(h);
        atomicAdd(&hist[min(k16 - base16, (uint32_t)(kNB16 - 1))], 1u);
        if (slot < SEG) {
          mk[slot] = (uint16_t)k16;
          mp[slot] = N * (q0 + u * T) + j;
        }
        ++slot;
      }
    }
  };
  auto mask_of = [&](const uint4& a, int u) {
    float x[N];
    SV::unpack(a, x);
    uint32_t bits = 0;
#pragma unroll
    for (int j = 0; j < N; ++j) bits |= (x[j] >= fthr ? 1u : 0u) << (N * u + j);
    return bits;
  };
  const int nv = n / N;
  const uint4* r16 = reinterpret_cast<const uint4*>(row);
  int base = 0;
  for (; base + U * T <= nv; base += U * T) {
    uint4 a[U];
#pragma unroll
    for (int u = 0; u < U; ++u) a[u] = r16[base + u * T + tid];
    uint32_t bits = 0;
#pragma unroll
    for (int u = 0; u < U; ++u) bits |= mask_of(a[u], u);
    append(a, bits, base + tid);
  }
  for (; base < nv; base += T) {  // fewer than U T vectors left: one per lane
    const int q = base + tid;
    uint4 a[U];
#pragma unroll
    for (int u = 0; u < U; ++u) a[u] = make_uint4(0u, 0u, 0u, 0u);
    if (q < nv) a[0] = r16[q];
    append(a, q < nv ? mask_of(a[0], 0) : 0u, q);
  }
  if (N * nv < n) {  // the n mod N tail: score e is element e mod N of vector e / N
    const int e = N * nv + tid;
    const bool ok = e < n;
    const int j = e & (N - 1);
    const uint32_t h = ok ? (uint32_t)row[e] : 0u;
    const uint32_t w = (j & 1) ? (h << 16) : h;
    uint4 a[U];
#pragma unroll
    for (int u = 0; u < U; ++u) a[u] = make_uint4(0u, 0u, 0u, 0u);
    a[0] = make_uint4((j >> 1) == 0 ? w : 0u, (j >> 1) == 1 ? w : 0u, (j >> 1) == 2 ? w : 0u, (j >> 1) == 3 ? w : 0u);
    const bool t = ok && __uint_as_float(h << 16) >= fthr;
    append(a, t ? (1u << j) : 0u, e / N);
  }
  if (lane == 0) wcnt[wv] = wc;
  __syncthreads();
  int tot = 0;
  bool over = false;
#pragma unroll
  for (int w = 0; w < NW; ++w) {
    tot += wcnt[w];
    over |= wcnt[w] > SEG;
  }
  return over ? CAP + 1 : tot;
}

// The `rem` lowest of the in_b positions listed in LDS (members of one value).
template <int T, class Put>
__device__ __forceinline__ void take_tied(const int32_t* lpos, uint32_t in_b, uint32_t rem, SelectShared& sh,
                                          Put put) {
  const int tid = threadIdx.x;
  if (in_b <= (uint32_t)kBucketList) {  // rank each tied member by its position, G threads to a member
    constexpr int G = T / kBucketList;
    static_assert(G >= 1 && (G & (G - 1)) == 0 && G <= 64, "threads per tied member");
    const int t = tid / G, part = tid % G;
    const bool mine = t < (int)in_b;
    const int32_t p = mine ? lpos[t] : 0;
    const int span = ((int)in_b + G - 1) / G, u1 = min((int)in_b, (part + 1) * span);
    uint32_t r = 0;
    int u = part * span;
    for (; u + 8 <= u1; u += 8) {
      int32_t x[8];
#pragma unroll
      for (int j = 0; j < 8; ++j) x[j] = lpos[u + j];
#pragma unroll
      for (int j = 0; j < 8; ++j) r += (uint32_t)(x[j] < p);
    }
    for (; u < u1; ++u) r += (uint32_t)(lpos[u] < p);
#pragma unroll
    for (int o = 1; o < G; o <<= 1) r += __shfl_xor(r, o, 64);
    wave_append(mine && part == 0 && r < rem, &sh.emitted, [&](int slot) { put(slot, p); });
    __syncthreads();
  } else {  // many ties: a radix select on their positions (the keys are equal)
    const TieSource<T> ties{lpos, (int)in_b};
    block_select<T, false>(ties, rem, sh, put);
  }
}

// Step 3 for bf16 rows, from the histogram the compaction built: b* = the bin
// holding the m-th largest key; every candidate in a higher bin is taken, and
// bin b* (below the top bin) holds one bf16 value, so its members tie and the
// lowest positions among them complete the set.  Returns false, having
// emitted nothing, when b* is the top bin or holds more than kNB16
// members.  lpos: kNB16 LDS words (may alias hist).
template <int T, class Src, class Put>
__device__ bool select16(const Src& cand, uint32_t base16, uint32_t m, uint32_t* hist, int32_t* lpos,
                         int32_t* lcount, SelectShared& sh, Put put) {
  const int tid = threadIdx.x;
  find_digit<T, true, kNB16>(hist, sh, m);  // ends with a barrier
  const uint32_t bsel = sh.digit, rem = m - sh.before, in_b = sh.equal;
  if (bsel == (uint32_t)(kNB16 - 1) || in_b > (uint32_t)kNB16) return false;
  if (tid == 0) *lcount = 0;
  __syncthreads();
  cand.visit([&](uint32_t key, int32_t p) {
    const uint32_t d = min((key >> 16) - base16, (uint32_t)(kNB16 - 1));
    wave_append(d > bsel, &sh.emitted, [&](int slot) { put(slot, p); });
    if (d == bsel) lpos[atomicAdd(lcount, 1)] = p;
  });
  __syncthreads();
  take_tied<T>(lpos, in_b, rem, sh, put);
  return true;
}

// topk_rows_kernel's one-read path for bf16 score rows (fp8 inputs) of a
// launch holding rows of 16384+ scores: candidates take 6 bytes (16-bit key,
// int32 position) instead of 8, and the sampling histogram, the candidates
// and the row fallback share one LDS region (they are never live together),
// so three 512-thread workgroups fit a CU instead of two.
template <int CAP, int T>
__global__ __launch_bounds__(T) __attribute__((amdgpu_waves_per_eu(6)))
void topk_rows16_kernel(const bf16_t* __restrict__ scores, int64_t ld, SeqTable st, RowSpace rs, OutDesc od) {
  using Lds = Rows16Lds<CAP>;
  constexpr int U = 4;
  __shared__ __attribute__((aligned(16))) uint8_t raw[Lds::RAW];
  __shared__ SelectShared sel;
  __shared__ int32_t lcount;
  __shared__ int32_t wcnt[T / 64];
  const int nrows = rs.i1 - rs.i0;
  const int b = blockIdx.x / nrows;
  const int i = rs.i0 + blockIdx.x % nrows;
  if (!row_active(st, rs, b, i)) return;
  const int tid = threadIdx.x;
  const int n = (int)max((int64_t)0, row_limit(st, rs, b, i) + 1);
  const bf16_t* row = scores + ((int64_t)b * nrows + (i - rs.i0)) * ld;
  const int m = od.m;
  const RowDest put(od, st, b, i);
  if (n <= m) {
    for (int p = tid; p < m; p += T) put(p, p < n ? p : -1);
    return;
  }
  if (tid == 0) sel.emitted = 0;
  const bool aligned = (reinterpret_cast<uintptr_t>(row) & 15u) == 0;
  uint16_t* ckey = reinterpret_cast<uint16_t*>(raw);
  int32_t* cpos = reinterpret_cast<int32_t*>(raw + Lds::KEY_BYTES);
  uint32_t* hist = reinterpret_cast<uint32_t*>(raw + Lds::KEY_BYTES + Lds::POS_BYTES);
  for (int k = tid; k < kNB16; k += T) hist[k] = 0;  // outside the sampling histogram's words
  float fthr;
  uint32_t base16;
  if (n >= kSampleMinLen && aligned &&
      sample_threshold16<T, CAP, CAP == kSelCapSmall ? 64 : 32>(row, n, m, reinterpret_cast<uint32_t*>(raw), sel,
                                                               fthr, base16)) {
    int found;
#pragma unroll 1
    for (;;) {
      found = stream_compact16<T, U, CAP>(row, n, fthr, base16, ckey, cpos, hist, wcnt);
      if (found >= m || (base16 & 15u) == 0) break;
      // where many scores are equal, those of the threshold's bin may all lie at
      // its lower edge
      base16 &= ~15u;
      fthr = key_float(key16_expand(base16));
      __syncthreads();
      for (int k = tid; k < kNB16; k += T) hist[k] = 0;
      __syncthreads();
    }
    if (found >= m && found <= CAP) {
      const SegSource16<T, T / 64, CAP / (T / 64)> cand(ckey, cpos, wcnt);
      if (select16<T>(cand, base16, (uint32_t)m, hist, reinterpret_cast<int32_t*>(hist), &lcount, sel, put))
        return;
      if (!bucket_select<T, kNB16>(cand, (uint32_t)m, hist, hist, reinterpret_cast<int32_t*>(hist + kBucketList),
                                   &lcount, sel, put))
        block_select<T, false>(cand, (uint32_t)m, sel, put);
      return;
    }
  }
  TwoLevelShared<Lds::CAP2>& fb = *reinterpret_cast<TwoLevelShared<Lds::CAP2>*>(raw);
  __syncthreads();  // the region's previous use has ended in every wave
  if (tid == 0) fb.sel.emitted = 0;
  RowSource<T, U, bf16_t> src{row, n};
  two_level_select<T>(src, (uint32_t)m, fb, put);
}

// ---- rows held in registers ----
// Order keys of the resident select: larger score, larger key; -0 and +0 share
// one; NaNs rank by sign as in float_key; 0 is no score's key.  They are
// float_key (of a bf16 score its upper half) except that every negative
// score's key is one higher, which merges the zeros without a compare.  bf16
// words convert two scores at a time with packed 16-bit operations.
template <class E>
struct OrderKey;
template <>
struct OrderKey<bf16_t> {
  static constexpr int kShift = 0;  // histogram bins of one value each
  typedef short s2 __attribute__((ext_vector_type(2)));
  __device__ static __forceinline__ uint32_t convert(uint32_t w) {
    const s2 t = __builtin_bit_cast(s2, w) >> (short)15;
    const uint32_t k = w ^ (__builtin_bit_cast(uint32_t, t) | 0x80008000u);
    return __builtin_bit_cast(uint32_t, (s2)(__builtin_bit_cast(s2, k) - t));
  }
  __device__ static __forceinline__ uint32_t one(bf16_t h) { return convert(h) & 0xFFFFu; }
  __device__ static __forceinline__ uint32_t at(const uint4& a, int j) {
    const uint32_t w = j < 2 ? a.x : j < 4 ? a.y : j < 6 ? a.z : a.w;
    return (j & 1) ? w >> 16 : w & 0xFFFFu;
  }
  // key j >= thr without extracting an upper half
  __device__ static __forceinline__ bool reaches(const uint4& a, int j, uint32_t thr) {
    const uint32_t w = j < 2 ? a.x : j < 4 ? a.y : j < 6 ? a.z : a.w;
    return (j & 1) ? w >= (thr << 16) : (uint16_t)w >= (uint16_t)thr;
  }
  __device__ static __forceinline__ bool any_reaches(const uint4& a, uint32_t thr) {
    typedef unsigned short u2 __attribute__((ext_vector_type(2)));
    const u2 x = __builtin_elementwise_max(__builtin_bit_cast(u2, a.x), __builtin_bit_cast(u2, a.y));
    const u2 y = __builtin_elementwise_max(__builtin_bit_cast(u2, a.z), __builtin_bit_cast(u2, a.w));
    const uint32_t k = __builtin_bit_cast(uint32_t, __builtin_elementwise_max(x, y));
    return max(k >> 16, k & 0xFFFFu) >= thr;
  }
  __device__ static __forceinline__ uint32_t wide(uint32_t k) { return k << 16; }
  __device__ static __forceinline__ uint32_t narrow(uint32_t k) { return k >> 16; }
  __device__ static __forceinline__ uint32_t as_float_key(uint32_t k) {
    return (k & 0x8000u) ? k << 16 : ((k - 1u) << 16) | 0xFFFFu;
  }
};
template <>
struct OrderKey<float> {
  static constexpr int kShift = 12;  // 1024 bins: half an octave above the threshold
  __device__ static __forceinline__ uint32_t convert(uint32_t w) {
    const uint32_t t = (uint32_t)((int32_t)w >> 31);
    return (w ^ (t | 0x80000000u)) - t;
  }
  __device__ static __forceinline__ uint32_t one(float f) { return convert(__float_as_uint(f)); }
  __device__ static __forceinline__ uint32_t at(const uint4& a, int j) {
    return j == 0 ? a.x : j == 1 ? a.y : j == 2 ? a.z : a.w;
  }
  __device__ static __forceinline__ bool reaches(const uint4& a, int j, uint32_t thr) { return at(a, j) >= thr; }
  __device__ static __forceinline__ bool any_reaches(const uint4& a, uint32_t thr) {
    return max(max(a.x, a.y), max(a.z, a.w)) >= thr;
  }
  __device__ static __forceinline__ uint32_t wide(uint32_t k) { return k; }
  __device__ static __forceinline__ uint32_t narrow(uint32_t k) { return k; }
  __device__ static __forceinline__ uint32_t as_float_key(uint32_t k) { return k - 1u + (k >> 31); }
};

// One vector of order keys per thread, for sample_prefix.
template <class E>
struct ResidentSample {
  uint4 a;
  bool ok;
  template <class F>
  __device__ __forceinline__ void visit(F f) const {
    if (ok) {
#pragma unroll
      for (int j = 0; j < ScoreVec<E>::N; ++j) f(OrderKey<E>::wide(OrderKey<E>::at(a, j)), 0);
    }
  }
};

// A candidate of the resident select in LDS: one word, the key's distance above
// the threshold over the position, for bf16 rows of at most 65536 scores, else
// the key and the position.
template <class E, bool WORD>
struct Candidate {
  using W = uint2;
  __device__ static __forceinline__ W pack(uint32_t key, uint32_t, int32_t pos) {
    return make_uint2(key, (uint32_t)pos);
  }
  __device__ static __forceinline__ uint32_t above(W w, uint32_t base) { return w.x - base; }
  __device__ static __forceinline__ int32_t pos(W w) { return (int32_t)w.y; }
};
template <>
struct Candidate<bf16_t, true> {
  using W = uint32_t;
  __device__ static __forceinline__ W pack(uint32_t key, uint32_t base, int32_t pos) {
    return ((key - base) << 16) | (uint32_t)pos;
  }
  __device__ static __forceinline__ uint32_t above(W w, uint32_t) { return w >> 16; }
  __device__ static __forceinline__ int32_t pos(W w) { return (int32_t)(w & 0xFFFFu); }
};

// Three sums over the workgroup, in every thread.  Calls alternate between two
// sets of words, so each needs one barrier.
struct Three {
  uint32_t a, b, c;
};
template <int T>
__device__ __forceinline__ Three block_sums(Three x, uint32_t (&sums)[2][3][T / 64], int& turn) {
  const int lane = threadIdx.x & 63, wave = (int)(threadIdx.x >> 6);
  const Three s{wave_incl_sum(x.a), wave_incl_sum(x.b), wave_incl_sum(x.c)};
  if (lane == 63) {
    sums[turn][0][wave] = s.a;
    sums[turn][1][wave] = s.b;
    sums[turn][2][wave] = s.c;
  }
  __syncthreads();
  // a row of 16 lanes to each sum
  uint32_t y = lane < 48 && (lane & 15) < T / 64 ? sums[turn][lane >> 4][lane & 15] : 0u;
  turn ^= 1;
  y += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)y, 0x111, 0xF, 0xF, true);  // row_shr:1, 2, 4, 8
  y += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)y, 0x112, 0xF, 0xF, true);
  y += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)y, 0x114, 0xF, 0xF, true);
  y += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)y, 0x118, 0xF, 0xF, true);
  return {(uint32_t)__builtin_amdgcn_readlane((int)y, 15), (uint32_t)__builtin_amdgcn_readlane((int)y, 31),
          (uint32_t)__builtin_amdgcn_readlane((int)y, 47)};
}

// The candidates of a row, for bisect_select and (visit) bucket_select.
template <int T, class E, bool WORD>
struct CandSearch {
  using C = Candidate<E, WORD>;
  const typename C::W* w;
  uint32_t base;
  int count;
  uint32_t tied;
  template <class F>
  __device__ __forceinline__ void each(F f) const {
    for (int e = threadIdx.x; e < count; e += T) f(base + C::above(w[e], base), C::pos(w[e]));
  }
  template <class F>
  __device__ __forceinline__ void visit(F f) const {
    each([&](uint32_t key, int32_t pos) { f(OrderKey<E>::as_float_key(key), pos); });
  }
  __device__ __forceinline__ Three at_least(uint32_t k1, uint32_t k2, uint32_t k3) const {
    Three n{0, 0, 0};
    each([&](uint32_t key, int32_t) {
      n.a += (uint32_t)(key >= k1);
      n.b += (uint32_t)(key >= k2);
      n.c += (uint32_t)(key >= k3);
    });
    return n;
  }
  __device__ __forceinline__ void tie(uint32_t k) { tied = k; }
  __device__ __forceinline__ Three ties_to(int p1, int p2, int p3) const {
    Three n{0, 0, 0};
    each([&](uint32_t key, int32_t pos) {
      n.a += (uint32_t)(key == tied && pos <= p1);
      n.b += (uint32_t)(key == tied && pos <= p2);
      n.c += (uint32_t)(key == tied && pos <= p3);
    });
    return n;
  }
  __device__ __forceinline__ uint32_t take(uint32_t k, int last) {
    uint32_t n = 0;
    each([&](uint32_t key, int32_t pos) { n += (uint32_t)(key > k || (key == k && pos <= last)); });
    return n;
  }
  template <class Put>
  __device__ __forceinline__ void emit(uint32_t k, int last, int slot, Put put) const {
    each([&](uint32_t key, int32_t pos) {
      if (key > k || (key == k && pos <= last)) put(slot++, pos);
    });
  }
};

// A row in registers, for bisect_select: V vectors of order keys per thread (vn
// in use, the others and those past the row's end 0), from the score `head` on,
// and one key more (tkey, of score te) in the first threads.
template <int T, int V, class E>
struct RowSearch {
  using OK = OrderKey<E>;
  static constexpr int N = ScoreVec<E>::N, WORDS = (V * N + 31) / 32;
  uint4 a[V];
  int vn, head;
  uint32_t tkey;
  int te;
  uint32_t mask[WORDS];  // this thread's tied, then its taken scores
  bool tmask;
  template <class F>
  __device__ __forceinline__ void each(F f) const {
#pragma unroll
    for (int v = 0; v < V; ++v)
      if (v < vn) {
#pragma unroll
        for (int j = 0; j < N; ++j) f(OK::at(a[v], j), head + N * (v * T + (int)threadIdx.x) + j);
      }
    f(tkey, te);
  }
  __device__ __forceinline__ Three at_least(uint32_t k1, uint32_t k2, uint32_t k3) const {
    Three n{(uint32_t)(tkey >= k1), (uint32_t)(tkey >= k2), (uint32_t)(tkey >= k3)};
#pragma unroll
    for (int v = 0; v < V; ++v)
      if (v < vn) {
#pragma unroll
        for (int j = 0; j < N; ++j) {
          n.a += (uint32_t)OK::reaches(a[v], j, k1);
          n.b += (uint32_t)OK::reaches(a[v], j, k2);
          n.c += (uint32_t)OK::reaches(a[v], j, k3);
        }
      }
    return n;
  }
  template <class F>
  __device__ __forceinline__ void mark(F f) {
#pragma unroll
    for (int u = 0; u < WORDS; ++u) mask[u] = 0;
#pragma unroll
    for (int v = 0; v < V; ++v)
      if (v < vn) {
        const int p0 = head + N * (v * T + (int)threadIdx.x);
#pragma unroll
        for (int j = 0; j < N; ++j) mask[(v * N + j) / 32] |= (uint32_t)f(OK::at(a[v], j), p0 + j) << ((v * N + j) % 32);
      }
    tmask = f(tkey, te);
  }
  __device__ __forceinline__ void tie(uint32_t k) {
    mark([&](uint32_t key, int) { return key == k; });
  }
  // ties at most at position `last`: a prefix of the mask
  __device__ __forceinline__ uint32_t ties_to(int last) const {
    const int x = last - head - N * (int)threadIdx.x;
    const int upto = x < 0 ? 0 : N * (x / (N * T)) + min(N, x % (N * T) + 1);
    uint32_t n = (uint32_t)(tmask && te <= last);
#pragma unroll
    for (int u = 0; u < WORDS; ++u) {
      const int bits = min(max(upto - 32 * u, 0), 32);
      n += (uint32_t)__popc(mask[u] & (uint32_t)((1ull << bits) - 1ull));
    }
    return n;
  }
  __device__ __forceinline__ Three ties_to(int p1, int p2, int p3) const {
    return {ties_to(p1), ties_to(p2), ties_to(p3)};
  }
  __device__ __forceinline__ uint32_t take(uint32_t k, int last) {
    mark([&](uint32_t key, int pos) { return key > k || (key == k && pos <= last); });
    uint32_t n = (uint32_t)tmask;
#pragma unroll
    for (int u = 0; u < WORDS; ++u) n += (uint32_t)__popc(mask[u]);
    return n;
  }
  template <class Put>
  __device__ __forceinline__ void emit(uint32_t, int, int slot, Put put) const {
#pragma unroll
    for (int u = 0; u < WORDS; ++u)
      for (uint32_t x = mask[u]; x != 0; x &= x - 1) {
        const int at = 32 * u + __ffs((int)x) - 1;
        put(slot++, head + N * (at / N * T + (int)threadIdx.x) + at % N);
      }
    if (tmask) put(slot, te);
  }
};

// Exact top-m of a source whose keys are counted, not sorted: cuts the range
// [lo, hi] of the m-th largest key in four by three counts at a time, then,
// among keys equal to it, the range of the last position taken.  At the start
// c_lo keys are >= lo (at least m), c_hi above hi (fewer than m); n bounds the
// positions.  The first cuts narrow the range to keys that occur and try its
// ends, which decides at once where many keys are equal.  At most 3 + 16 cuts
// for the key and 9 for the position, each a few instructions per key and a
// barrier or two: its time hardly depends on how the keys are distributed, where
// histograms of equal keys serialise on one LDS word.
template <int T, class Src, class Put>
__device__ __forceinline__ void bisect_select(Src& src, uint32_t lo, uint32_t c_lo, uint32_t hi, uint32_t c_hi,
                                              uint32_t m, int n, uint32_t (&sums)[2][3][T / 64], SelectShared& sh,
                                              Put put) {
  int turn = 0;
  for (int cut = 0; lo < hi && c_lo != m; ++cut) {
    uint32_t k1, k2, k3;  // lo < k1 <= k2 <= k3 <= hi
    if (cut < 3) {
      uint32_t kmin = ~0u, kmax = 0u;
      src.each([&](uint32_t key, int32_t) {
        if (key >= lo) kmin = min(kmin, key);
        if (key <= hi) kmax = max(kmax, key);
      });
      block_pair_reduce<T, true>(kmin, kmax, sh);
      lo = kmin;
      hi = kmax;
      if (lo == hi) break;
      k1 = lo + 1;
      k2 = lo + (hi - lo + 1) / 2;
      k3 = hi;
    } else {
      const uint32_t range = hi - lo;
      k1 = lo + (range >> 2) + 1;
      k2 = lo + (range >> 1) + 1;
      k3 = hi - (range >> 2);
    }
    const Three c = block_sums<T>(src.at_least(k1, k2, k3), sums, turn);
    if (c.c >= m) {
      lo = k3;
      c_lo = c.c;
    } else if (c.b >= m) {
      lo = k2;
      c_lo = c.b;
      hi = k3 - 1;
      c_hi = c.c;
    } else if (c.a >= m) {
      lo = k1;
      c_lo = c.a;
      hi = k2 - 1;
      c_hi = c.b;
    } else {
      hi = k1 - 1;
      c_hi = c.a;
    }
  }
  int last = n;
  if (c_lo != m) {  // more keys equal the m-th than are taken: those of the lowest positions
    const uint32_t rem = m - c_hi;
    src.tie(lo);
    int p0 = 0, p1 = n - 1;  // the rem-th tie lies in [p0, p1]
    while (p0 < p1) {
      const int range = p1 - p0, q1 = p0 + (range >> 2), q2 = p0 + (range >> 1), q3 = p1 - 1 - (range >> 2);
      const Three c = block_sums<T>(src.ties_to(q1, q2, q3), sums, turn);
      if (c.a >= rem) {
        p1 = q1;
      } else if (c.b >= rem) {
        p0 = q1 + 1;
        p1 = q2;
      } else if (c.c >= rem) {
        p0 = q2 + 1;
        p1 = q3;
      } else {
        p0 = q3 + 1;
      }
    }
    last = p0;
  }
  const uint32_t mine = src.take(lo, last), sum = wave_incl_sum(mine);
  int slot = 0;
  if ((threadIdx.x & 63) == 63) slot = atomicAdd(&sh.emitted, (int)sum);
  src.emit(lo, last, __builtin_amdgcn_readlane(slot, 63) + (int)(sum - mine), put);
}

// A set of rows of a resident select launch; blocks [0, blocks0) take the
// first, the others the second (the proxies' rows and the guardrail's).
template <class E>
struct SelectRows {
  const E* scores;
  int64_t ld;
  RowSpace rs;
  OutDesc od;
};

// Rows of at most T V N scores (N = 8 bf16 or 4 fp32 to a 16-byte vector): one
// workgroup per row requests all of it at once, V vectors per thread.
//   1 threshold  one vector per wave and lane is the sample, 1/vn of the row
//                (vn vectors in use), a block of 64 vectors out of every vn
//                (sampled_vector, sample_base).  One vector per thread is the
//                whole row: its threshold is the m-th key's bin;
//   2 compact    the keys >= the threshold go to LDS with their positions, a
//                ballot per score and one LDS atomic per wave and vector;
//   3 select     a histogram of their distance above the threshold gives the
//                bin with the m-th key; every candidate above it is taken, and
//                its members are ranked by (key, position).
// Outside those rules the select goes on with bucket_select (the m-th key lies
// past the histogram) or bisect_select: over the candidates where the bin is too
// long, over the row, loaded again, where the threshold kept fewer than m or
// more than CAP keys.  So every row is exact.
// FILTER, for long rows in decode or with a small m, whose threads hold many
// vectors of which few reach the threshold: step 2 first lists the vectors with
// a key that does (a packed maximum and one ballot per vector), and examines
// only those, dealt evenly to the threads and read again (from L2).
// What bounds it: the fixed phases' latency and LDS operations, not the bytes
// (a row is a few tens of KiB per CU), so a candidate is one LDS word, and the
// histogram is built from the candidates rather than score by score; rows of
// that word leave four 512-thread workgroups to a CU.  Measured against the
// kernels these rows took before (two passes over the row, a sampled pass, or
// three launches splitting few long rows): 7168 bf16 rows of 4096-32768 scores
// 312 -> 150 us, 500 fp32 rows of 20011 (odd stride) 44 -> 20 us, 32 bf16 rows
// of 131071 32 -> 25 us, 24 of 5003-70001 30 -> 16 us.  Past its limits the
// row does not fit the registers of one workgroup.
template <int T, int V, int CAP, class E, bool FILTER>
__global__ __launch_bounds__(T) __attribute__((amdgpu_waves_per_eu(T == 512 && V * (int)sizeof(E) <= 16 ? 8 : 4)))
void topk_resident_kernel(SelectRows<E> set0, SelectRows<E> set1, int blocks0, SeqTable st) {
  using OK = OrderKey<E>;
  constexpr int N = ScoreVec<E>::N;
  constexpr bool WORD = sizeof(E) == 2 && T * V * N <= 65536;
  using C = Candidate<E, WORD>;
  constexpr int CAND_BYTES = ((int)sizeof(typename C::W) * (CAP + 1) + 15) / 16 * 16;  // one slot takes the overflow
  constexpr int LDS = CAND_BYTES + 4 * kNB16;
  static_assert(CAND_BYTES >= 4 * 4096, "the sampling histogram lies within the candidates");
  __shared__ __attribute__((aligned(16))) uint8_t raw[LDS];
  __shared__ uint16_t vlist[FILTER ? T * V : 1];  // vectors with a key that reaches the threshold
  __shared__ SelectShared sel;
  __shared__ uint32_t sums[2][3][T / 64];
  __shared__ int32_t lcount, kept, listed;
  const bool second = (int)blockIdx.x >= blocks0;
  const E* const scores = second ? set1.scores : set0.scores;
  const int64_t ld = second ? set1.ld : set0.ld;
  const RowSpace rs = second ? set1.rs : set0.rs;
  const OutDesc od = second ? set1.od : set0.od;
  const int bx = (int)blockIdx.x - (second ? blocks0 : 0);
  const int nrows = rs.i1 - rs.i0;
  const int b = bx / nrows;
  const int i = rs.i0 + bx % nrows;
  if (!row_active(st, rs, b, i)) return;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int n = __builtin_amdgcn_readfirstlane((int)max((int64_t)0, row_limit(st, rs, b, i) + 1));
  const E* row = scores + ((int64_t)b * nrows + (i - rs.i0)) * ld;
  const int m = od.m;
  const RowDest put(od, st, b, i);
  if (n <= m) {
    for (int p = tid; p < m; p += T) put(p, p < n ? p : -1);
    return;
  }
  typename C::W* cand = reinterpret_cast<typename C::W*>(raw);
  uint32_t* hist = reinterpret_cast<uint32_t*>(raw + CAND_BYTES);
  // the first `head` scores lie before a 16-byte boundary
  const int head = min(n, (int)((-reinterpret_cast<uintptr_t>(row) & 15u) / sizeof(E)));
  const int nv = (n - head) / N, vn = (nv + T - 1) / T;  // full vectors, and those of a thread
  const uint4* r16 = reinterpret_cast<const uint4*>(row + head);
  if (tid == 0) {
    sel.emitted = 0;
    kept = 0;
    listed = 0;
  }
  // the scores before the first vector and after the last: one each for the first threads
  const int te = tid < head ? tid : tid + N * nv;
  const uint32_t tkey = te < n && tid < 2 * N ? OK::one(row[te]) : 0u;
  auto convert = [](uint4 x, bool in) {
    return make_uint4(in ? OK::convert(x.x) : 0u, in ? OK::convert(x.y) : 0u, in ? OK::convert(x.z) : 0u,
                      in ? OK::convert(x.w) : 0u);
  };
  auto load_row = [&](uint4 (&a)[V]) {
#pragma unroll
    for (int v = 0; v < V; ++v) {
      a[v] = make_uint4(0u, 0u, 0u, 0u);
      if (v < vn && v * T + tid < nv) a[v] = r16[v * T + tid];
    }
#pragma unroll
    for (int v = 0; v < V; ++v)
      if (v < vn) a[v] = convert(a[v], v * T + tid < nv);
  };
  // what the threshold leaves to bisect_select over the row: c_lo keys >= lo, c_hi above hi
  constexpr uint32_t kTop = sizeof(E) == 2 ? 0xFFFFu : ~0u;
  uint32_t lo = 1, c_lo = (uint32_t)n, hi = kTop, c_hi = 0;
  if (vn >= 1) {
    uint4 a[V];
    load_row(a);
    // lane w: the vector that wave w samples, and the sampled vectors up to it
    const int turn = sampled_vector(lane & (T / 64 - 1), T / 64, vn);
    const uint32_t sampled =
        wave_incl_sum(lane < T / 64 ? (uint32_t)max(0, min(64, nv - (turn * T + 64 * lane))) : 0u);
    const int s = N * __builtin_amdgcn_readlane((int)sampled, 63);
    const int pick = __builtin_amdgcn_readlane(turn, wave);
    // expected sample rank of the m-th key plus four standard deviations
    const float rm = (float)s * (float)m / (float)n;
    const uint32_t ts = vn == 1 ? (uint32_t)m : (uint32_t)ceilf(rm + 4.0f * sqrtf(rm)) + 1u;
    const bool all = ts >= (uint32_t)s && n <= CAP;  // nearly every score is wanted: keep them all
    uint32_t base = 1u;
    bool ok = all;
    if (!all && ts < (uint32_t)s && (float)ts * (float)n <= 0.8f * (float)CAP * (float)s) {
      ResidentSample<E> smp;
      smp.a = a[0];
#pragma unroll
      for (int v = 1; v < V; ++v) {
        int at = v;  // opaque, or the chain becomes an indexed read of a[] in scratch memory
        asm volatile("" : "+s"(at));
        if (at == pick) smp.a = a[v];
      }
      smp.ok = pick * T + tid < nv;
      base = sample_base<T>(smp, ts, reinterpret_cast<uint32_t*>(raw), sel);
      if (vn == 1) base &= 0xFFF00000u;
      base = max(OK::narrow(base), 1u);
      ok = true;
    }
    if (ok) {
      for (int k = tid; k < kNB16; k += T) hist[k] = 0;
      __syncthreads();  // kept is set, and the sampling histogram's words are free
      // the keys >= base of vector `x`, whose first position is p0
      auto compact = [&](const uint4& x, int p0) {
        uint64_t bal[N];
        int total = 0;
#pragma unroll
        for (int j = 0; j < N; ++j) {
          bal[j] = __ballot(OK::reaches(x, j, base));
          total += (int)__popcll((unsigned long long)bal[j]);
        }
        if (total == 0) return;  // uniform over the wave
        int slot0 = 0;
        if (lane == 0) slot0 = atomicAdd(&kept, total);
        slot0 = __builtin_amdgcn_readfirstlane(slot0);
#pragma unroll
        for (int j = 0; j < N; ++j) {
          const int slot = (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(bal[j] >> 32),
                                                          __builtin_amdgcn_mbcnt_lo((uint32_t)bal[j], (uint32_t)slot0));
          if (OK::reaches(x, j, base)) cand[min(slot, CAP)] = C::pack(OK::at(x, j), base, p0 + j);
          slot0 += (int)__popcll((unsigned long long)bal[j]);
        }
      };
      if constexpr (FILTER) {
#pragma unroll
        for (int v = 0; v < V; ++v)
          if (v < vn) {
            const bool t = OK::any_reaches(a[v], base);
            const uint64_t bal = __ballot(t);
            if (bal == 0) continue;  // uniform over the wave
            int slot0 = 0;
            if (lane == 0) slot0 = atomicAdd(&listed, (int)__popcll((unsigned long long)bal));
            slot0 = __builtin_amdgcn_readfirstlane(slot0);
            const int slot = (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(bal >> 32),
                                                            __builtin_amdgcn_mbcnt_lo((uint32_t)bal, (uint32_t)slot0));
            if (t) vlist[slot] = (uint16_t)(v * T + tid);
          }
        __syncthreads();
        const int nl = __builtin_amdgcn_readfirstlane(listed);
        constexpr int U = 4;  // vectors in flight per thread
        for (int l0 = 0; l0 < nl; l0 += U * T) {
          uint4 x[U];
          int q[U];
#pragma unroll
          for (int u = 0; u < U; ++u) {
            const int l = l0 + u * T + tid;
            q[u] = l < nl ? (int)vlist[l] : -1;
            x[u] = make_uint4(0u, 0u, 0u, 0u);
            if (q[u] >= 0) x[u] = r16[q[u]];
          }
#pragma unroll
          for (int u = 0; u < U; ++u)
            if (l0 + u * T < nl) compact(convert(x[u], q[u] >= 0), head + N * q[u]);
        }
      } else {
#pragma unroll
        for (int v = 0; v < V; ++v)
          if (v < vn) compact(a[v], head + N * (v * T + tid));
      }
      if (wave == 0)
        wave_append(tkey >= base, &kept, [&](int slot) { cand[min(slot, CAP)] = C::pack(tkey, base, te); });
      __syncthreads();
      const int found = kept;
      if (found >= m && found <= CAP) {
        auto bin = [&](typename C::W w) { return min(C::above(w, base) >> OK::kShift, (uint32_t)(kNB16 - 1)); };
        // the last bin takes every key past the histogram (half of a row whose
        // threshold is negative): counted by ballot, not by adds to one word
        int far = 0;
        for (int e = tid; e < found; e += T) {
          const uint32_t d = bin(cand[e]);
          const bool past = d == (uint32_t)(kNB16 - 1);
          far += (int)__popcll((unsigned long long)__ballot(past));
          if (!past) atomicAdd(&hist[d], 1u);
        }
        if (lane == 0 && far > 0) atomicAdd(&hist[kNB16 - 1], (uint32_t)far);
        __syncthreads();
        find_digit<T, true, kNB16>(hist, sel, (uint32_t)m);
        const uint32_t bsel = sel.digit, rem = (uint32_t)m - sel.before, in_b = sel.equal;
        if (bsel != (uint32_t)(kNB16 - 1) && in_b <= (uint32_t)kBucketList) {
          uint32_t* lkey = hist;  // free once the bin is known
          int32_t* lpos = reinterpret_cast<int32_t*>(hist) + (sizeof(E) == 2 ? 0 : kBucketList);
          if (tid == 0) lcount = 0;
          __syncthreads();
          // a wave reserves the slots of all it takes with one atomic
          int mine = 0;
          for (int e = tid; e - lane < found; e += T)
            mine += (int)__popcll((unsigned long long)__ballot(e < found && bin(cand[min(e, CAP)]) > bsel));
          int slot0 = 0;
          if (lane == 0) slot0 = atomicAdd(&sel.emitted, mine);
          slot0 = __builtin_amdgcn_readfirstlane(slot0);
          for (int e = tid; e - lane < found; e += T) {
            const typename C::W w = cand[min(e, CAP)];
            const uint32_t d = bin(w);
            const bool in = e < found, take = in && d > bsel;
            const uint64_t bal = __ballot(take);
            const int slot = (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(bal >> 32),
                                                            __builtin_amdgcn_mbcnt_lo((uint32_t)bal, (uint32_t)slot0));
            if (take) put(slot, C::pos(w));
            slot0 += (int)__popcll((unsigned long long)bal);
            if (in && d == bsel) {
              const int c = atomicAdd(&lcount, 1);
              if constexpr (sizeof(E) != 2) lkey[c] = base + C::above(w, base);
              lpos[c] = C::pos(w);
            }
          }
          __syncthreads();
          if constexpr (sizeof(E) == 2)
            take_tied<T>(lpos, in_b, rem, sel, put);  // one value: lowest positions
          else
            rank_listed<T>(in_b, rem, lkey, lpos, sel, put);
          return;
        }
        CandSearch<T, E, WORD> src{cand, base, found, 0u};
        if (bsel == (uint32_t)(kNB16 - 1)) {  // past the histogram: one over the candidates' values
          const uint32_t before = sel.before;
          __syncthreads();
          if (bucket_select<T, kNB16>(src, (uint32_t)m, hist, hist, reinterpret_cast<int32_t*>(hist + kBucketList),
                                      &lcount, sel, put))
            return;
          bisect_select<T>(src, base + (bsel << OK::kShift), before + in_b, kTop, before, (uint32_t)m, n, sums, sel,
                           put);
          return;
        }
        const uint32_t first = base + (bsel << OK::kShift), past = (1u << OK::kShift) - 1u;
        const uint32_t top = kTop - first < past ? kTop : first + past;
        bisect_select<T>(src, first, sel.before + in_b, top, sel.before, (uint32_t)m, n, sums, sel, put);
        return;
      }
      if (found < m) {
        hi = base - 1;
        c_hi = (uint32_t)found;
      } else {
        lo = base;
        c_lo = (uint32_t)found;
      }
    }
  }
  RowSearch<T, V, E> src;
  load_row(src.a);
  src.vn = vn;
  src.head = head;
  src.tkey = tkey;
  src.te = te;
  __syncthreads();  // sel.emitted is set
  bisect_select<T>(src, lo, c_lo, hi, c_hi, (uint32_t)m, n, sums, sel, put);
}

// Split select, step 1: workgroup r writes row r's threshold score to
// thr[r], or NaN when the row takes the two-pass path (n <= m, short or
// unaligned row, sample declined).
template <int CAP, int T, class E>
__global__ __launch_bounds__(T) void topk_thr_kernel(const E* __restrict__ scores, int64_t ld, SeqTable st,
                                                     RowSpace rs, int m, float* __restrict__ thr) {
  __shared__ uint32_t hist[4096];
  __shared__ SelectShared sel;
  const int nrows = rs.i1 - rs.i0;
  const int r = blockIdx.x;
  const int b = r / nrows;
  const int i = rs.i0 + r % nrows;
  if (!row_active(st, rs, b, i)) return;
  const int n = (int)max((int64_t)0, row_limit(st, rs, b, i) + 1);
  const E* row = scores + ((int64_t)b * nrows + (i - rs.i0)) * ld;
  const bool aligned = (reinterpret_cast<uintptr_t>(row) & 15u) == 0;
  float fthr;
  if (n <= m || n < kSampleMinLen || !aligned || !sample_threshold<T, CAP>(row, n, m, hist, sel, fthr))
    fthr = __builtin_nanf("");
  if (threadIdx.x == 0) thr[r] = fthr;
}

// Split select, step 2: workgroup (r, s) compacts the keys >= thr[r] among
// 16-byte vectors [s per_v, (s+1) per_v) of row r (the last slice also takes
// the n mod N tail) into LDS and writes them to cand[(r P + s) per ..] with
// their count in cnt[r P + s]: -1 when the row takes the two-pass path
// (thr[r] is NaN), -2 when the slice held more than `per` keys.
template <class E>
__global__ __launch_bounds__(kSplitThreads) void topk_slice_kernel(const E* __restrict__ scores, int64_t ld,
                                                                   SeqTable st, RowSpace rs, int P, int per,
                                                                   const float* __restrict__ thr,
                                                                   uint2* __restrict__ cand,
                                                                   int32_t* __restrict__ cnt) {
  using SV = ScoreVec<E>;
  constexpr int N = SV::N;
  constexpr int T = kSplitThreads, U = 8;  // 16-byte loads in flight per thread
  __shared__ uint2 lc[kSplitPerMax];
  __shared__ int32_t nc;
  const int nrows = rs.i1 - rs.i0;
  const int r = blockIdx.x, slice = blockIdx.y;
  const int b = r / nrows;
  const int i = rs.i0 + r % nrows;
  if (!row_active(st, rs, b, i)) return;
  const int tid = threadIdx.x;
  const int n = (int)max((int64_t)0, row_limit(st, rs, b, i) + 1);
  const E* row = scores + ((int64_t)b * nrows + (i - rs.i0)) * ld;
  int32_t* my_cnt = cnt + (int64_t)r * P + slice;
  const float fthr = thr[r];
  if (__builtin_isnan(fthr)) {
    if (tid == 0) *my_cnt = -1;
    return;
  }
  if (tid == 0) nc = 0;
  __syncthreads();
  auto take = [&](float v, int pos) {
    if (v >= fthr) {
      const int c = atomicAdd(&nc, 1);
      if (c < per) lc[c] = make_uint2(float_key(v), (uint32_t)pos);
    }
  };
  const int nv = n / N;
  const int per_v = (nv + P - 1) / P;
  const int a_v = slice * per_v, e_v = min(nv, a_v + per_v);
  const uint4* r16 = reinterpret_cast<const uint4*>(row);
  int q = a_v + tid;
  for (; q + (U - 1) * T < e_v; q += U * T) {
    uint4 x[U];
#pragma unroll
    for (int u = 0; u < U; ++u) x[u] = r16[q + u * T];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      float v[N];
      SV::unpack(x[u], v);
      const int p = N * (q + u * T);
#pragma unroll
      for (int j = 0; j < N; ++j) take(v[j], p + j);
    }
  }
  for (; q < e_v; q += T) {
    float v[N];
    SV::unpack(r16[q], v);
#pragma unroll
    for (int j = 0; j < N; ++j) take(v[j], N * q + j);
  }
  if (slice == P - 1)
    for (int e = N * nv + tid; e < n; e += T) take(SV::one(row, e), e);
  __syncthreads();
  const int c = nc;
  if (tid == 0) *my_cnt = c <= per ? c : -2;
  if (c <= per) {
    uint2* dst = cand + ((int64_t)r * P + slice) * per;
    for (int e = tid; e < c; e += T) dst[e] = lc[e];
  }
}

// Split select, step 3: one workgroup per row gathers the keys its slices
// compacted (when every slice kept its keys and they number m .. CAP) into
// LDS and selects exactly over them; any other row takes the two-pass path.
template <int CAP, int T, class E>
__global__ __launch_bounds__(T) void topk_merge_kernel(const E* __restrict__ scores, int64_t ld, SeqTable st,
                                                       RowSpace rs, OutDesc od, int P, int per,
                                                       const uint2* __restrict__ cand,
                                                       const int32_t* __restrict__ cnt) {
  constexpr int U = 8 * (int)sizeof(E) / 4;  // 16-byte loads in flight (fallback path)
  constexpr int V = (CAP + T - 1) / T;  // gathered keys per thread
  __shared__ TwoLevelShared<CAP> sh;
  __shared__ int32_t pre[kSplitMaxP + 1];
  const int nrows = rs.i1 - rs.i0;
  const int r = blockIdx.x;
  const int b = r / nrows;
  const int i = rs.i0 + r % nrows;
  if (!row_active(st, rs, b, i)) return;
  const int tid = threadIdx.x;
  const int n = (int)max((int64_t)0, row_limit(st, rs, b, i) + 1);
  const E* row = scores + ((int64_t)b * nrows + (i - rs.i0)) * ld;
  const int m = od.m;
  const RowDest put(od, st, b, i);
  if (n <= m) {
    for (int p = tid; p < m; p += T) put(p, p < n ? p : -1);
    return;
  }
  if (tid < 64) {  // the slices' counts, one per lane, and their prefix sums
    const int c = tid < P ? cnt[(int64_t)r * P + tid] : 0;
    int incl = max(c, 0);
#pragma unroll
    for (int o = 1; o < kSplitMaxP; o <<= 1) {
      const int t = __shfl_up(incl, o, 64);
      if (tid >= o) incl += t;
    }
    const bool ok = __ballot(tid < P && c < 0) == 0;
    if (tid < P) pre[tid] = incl - max(c, 0);
    const int tot = __shfl(incl, P - 1, 64);
    if (tid == 0) {
      pre[P] = ok ? tot : -1;
      sh.sel.emitted = 0;
    }
  }
  __syncthreads();
  const int total = pre[P];
  if (total >= m && total <= CAP) {
    // every thread fetches its (at most V) keys at once, then stores them;
    // an element's slice comes from the prefix sums held in registers
    int pr[kSplitMaxP];
#pragma unroll
    for (int k = 0; k < kSplitMaxP; ++k) pr[k] = k < P ? pre[k] : 0x7FFFFFFF;
    uint2 v[V];
#pragma unroll
    for (int j = 0; j < V; ++j) {
      const int e = tid + j * T;
      v[j] = make_uint2(0u, 0u);
      if (e < total) {
        int s = 0, base = 0;
#pragma unroll
        for (int k = 1; k < kSplitMaxP; ++k)
          if (e >= pr[k]) {
            s = k;
            base = pr[k];
          }
        v[j] = cand[((int64_t)r * P + s) * per + (e - base)];
      }
    }
#pragma unroll
    for (int j = 0; j < V; ++j) {
      const int e = tid + j * T;
      if (e < total) {
        sh.ckey[e] = v[j].x;
        sh.cpos[e] = (int32_t)v[j].y;
      }
    }
    __syncthreads();
    ArraySource<T> src{sh.ckey, sh.cpos, total};
    if (!bucket_select<T>(src, (uint32_t)m, sh.hist, sh.hist, reinterpret_cast<int32_t*>(sh.hist + kBucketList),
                          &sh.lcount, sh.sel, put))
      block_select<T, false>(src, (uint32_t)m, sh.sel, put);
    return;
  }
  RowSource<T, U, E> src{row, n};
  two_level_select<T>(src, (uint32_t)m, sh, put);
}

size_t split_scratch_bytes(int64_t rows) {
  return (size_t)rows * ((size_t)kSplitSlots * sizeof(uint2) + (size_t)kSplitMaxP * sizeof(int32_t) + sizeof(float));
}

// Smallest limit of an active row of rs (limits grow with the row index).
static int64_t min_limit(const SeqTable& st, const RowSpace& rs) {
  int64_t lim = INT64_MAX;
  for (int b = 0; b < st.n; ++b) {
    const int cnt = rs.kind == kProxyRows ? (st.n_rows[b] + rs.step - 1) / rs.step : st.n_rows[b];
    int hi = std::min(rs.i1, cnt), lo = rs.i0;
    if (rs.kind == kDenseRows) hi = std::min(hi, st.dense_rows[b]);
    if (rs.kind == kProxyRows) lo = std::max(lo, st.first_proxy[b]);
    if (hi > lo) lim = std::min(lim, (int64_t)st.q_pos0[b] + (int64_t)lo * rs.step - rs.shift);
  }
  return lim;
}

// Scores of a row that a 512-thread workgroup holds: 8 (bf16) or 16 (fp32) vectors a thread.
constexpr int64_t kResident = 32768;

// `blocks` rows of `set`, then `more_blocks` of `more`.
template <int T, int V, bool FILTER, class E>
static hipError_t resident_launch(const SelectRows<E>& set, const SelectRows<E>* more, int blocks, int more_blocks,
                                  const SeqTable& st, hipStream_t stream) {
  const SelectRows<E>& second = more ? *more : set;
  const dim3 grid((unsigned)(blocks + more_blocks));
  if (std::max(set.od.m, second.od.m) <= kSelCapSmall / 2)
    hipLaunchKernelGGL((topk_resident_kernel<T, V, kSelCapSmall, E, FILTER>), grid, dim3(T), 0, stream, set, second,
                       blocks, st);
  else
    hipLaunchKernelGGL((topk_resident_kernel<T, V, kSelCap16, E, FILTER>), grid, dim3(T), 0, stream, set, second,
                       blocks, st);
  return hipGetLastError();
}

// Rows of at most kResident scores.  Of long ones few vectors hold a kept key
// when m is small: FILTER.  Us a launch of rows of 32768 without and with it:
// 600 bf16 rows, m = 100, 18.6 and 15.3 (the streaming kernel 16.7), m = 1024,
// 22.4 and 19.8, m = 2048, 24.5 and 23.8; 3000 of 24001, m = 1024, 53.5 and
// 53.5, m = 2048, 59 and 63; 600 fp32 rows, m = 100, 29.1 and 26.3 (26.4),
// m = 512, 30.7 and 29.2, m = 2048, 34.6 and 38.3.
template <class E>
static hipError_t resident_512(const SelectRows<E>& set, const SelectRows<E>* more, int blocks, int more_blocks,
                               int64_t lim_max, const SeqTable& st, hipStream_t stream) {
  constexpr int V = 32 / ScoreVec<E>::N * 2;  // vectors of a thread that make kResident
  const SelectRows<E>& second = more ? *more : set;
  if (lim_max + 1 > kResident / 2 && std::max(set.od.m, second.od.m) <= (sizeof(E) == 2 ? 1024 : 512)) {
    hipLaunchKernelGGL((topk_resident_kernel<kSelThreads, V, kSelCapSmall, E, true>),
                       dim3((unsigned)(blocks + more_blocks)), dim3(kSelThreads), 0, stream, set, second, blocks, st);
    return hipGetLastError();
  }
  if constexpr (sizeof(E) == 4)
    if (lim_max + 1 <= kResident / 2)
      return resident_launch<kSelThreads, V / 2, false, E>(set, more, blocks, more_blocks, st, stream);
  return resident_launch<kSelThreads, V, false, E>(set, more, blocks, more_blocks, st, stream);
}

bool topk_both_ok(bool, const SeqTable& st, const TopkRows& a, const TopkRows& b) {
  const int64_t rows = (int64_t)st.n * ((a.rs.i1 - a.rs.i0) + (b.rs.i1 - b.rs.i0));
  return rows > kWideMaxRows && rows <= 0x7FFFFFFF && a.od.m <= kResidentMaxM && b.od.m <= kResidentMaxM &&
         std::max(a.lim_max, b.lim_max) + 1 <= kResident;
}

template <class E>
static hipError_t topk_both(const SeqTable& st, const TopkRows& a, const TopkRows& b, hipStream_t stream) {
  const SelectRows<E> s0{static_cast<const E*>(a.scores), a.ld, a.rs, a.od};
  const SelectRows<E> s1{static_cast<const E*>(b.scores), b.ld, b.rs, b.od};
  return resident_512<E>(s0, &s1, st.n * (a.rs.i1 - a.rs.i0), st.n * (b.rs.i1 - b.rs.i0),
                      std::max(a.lim_max, b.lim_max), st, stream);
}

hipError_t launch_topk_both(bool scores_bf16, const SeqTable& st, const TopkRows& a, const TopkRows& b,
                            hipStream_t stream) {
  return scores_bf16 ? topk_both<bf16_t>(st, a, b, stream) : topk_both<float>(st, a, b, stream);
}

template <class E>
static hipError_t topk_launch(const E* scores, int64_t ld, const SeqTable& st, const RowSpace& rs,
                              const OutDesc& od, int64_t lim_max, void* scratch, size_t scratch_bytes,
                              hipStream_t stream) {
  const int nrows = rs.i1 - rs.i0;
  if (nrows <= 0 || st.n <= 0) return hipSuccess;
  const int64_t blocks = (int64_t)st.n * nrows;
  if (blocks > 0x7FFFFFFF) return hipErrorInvalidConfiguration;
  constexpr int N = ScoreVec<E>::N;
  // fp32 rows of which half and more are wanted: their candidates leave two
  // resident workgroups to a CU, and the two-pass select, which keeps only the
  // boundary bin's, takes less (m = 4096, us a launch, resident and two-pass: 600
  // rows of 6000 scores 24.6 and 20.7, 3000 of 8192 82 and 73, of 10240 87 and 90).
  const bool mostly = sizeof(E) == 4 && blocks > kWideMaxRows && od.m > kSelCapSmall / 2 && lim_max + 1 <= 2 * od.m;
  // fp32 rows past 16384 scores leave two resident workgroups to a CU, the
  // streaming kernel three: for 513 to 768 rows two rounds against one (m = 2048,
  // 600 rows of 32768 34.6 and 30.9, 768 37.0 and 34.0, 512 25.6 and 25.5, 900
  // 41.1 and 44.9).
  const bool one_round = sizeof(E) == 4 && blocks > 2 * 256 && blocks <= 3 * 256 && od.m <= kSelCapSmall / 2 &&
                         lim_max + 1 > kResident / 2 && ld % N == 0 && reinterpret_cast<uintptr_t>(scores) % 16 == 0 &&
                         min_limit(st, rs) + 1 >= kSampleMinLen;
  if (od.m <= kResidentMaxM && !mostly && !one_round) {
    const SelectRows<E> set{scores, ld, rs, od};
    // few rows (decode): a wide workgroup holds up to 131072 bf16 or 65536 fp32
    // scores, 16 vectors a thread.  Shorter rows take a kernel of fewer: the
    // vectors past a row's end are skipped one branch at a time, and of rows
    // this short most vectors hold a kept key, so a list of them (FILTER) costs
    // more than it saves.  Us a launch of one row, 16 vectors and this choice:
    // fp32, 6000 scores 9.3 and 7.5 (m = 2048), 16384 10.4 and 9.1, 32768 12.0
    // and 11.3; bf16 decode steps (one request, Refine) of 6001 keys 33.6 and
    // 31.6, 24000 37.0 and 35.2, 65536 41.0 and 40.5.  200 rows gain as much.
    if (blocks <= kWideMaxRows) {
      constexpr int64_t W = (int64_t)kSelThreadsWide * N;  // scores of one vector a thread
      const int64_t len = lim_max + 1;
      if (len <= 2 * W) return resident_launch<kSelThreadsWide, 2, false, E>(set, nullptr, (int)blocks, 0, st, stream);
      if (len <= 4 * W) return resident_launch<kSelThreadsWide, 4, false, E>(set, nullptr, (int)blocks, 0, st, stream);
      if (len <= 8 * W) return resident_launch<kSelThreadsWide, 8, true, E>(set, nullptr, (int)blocks, 0, st, stream);
      if (len <= 16 * W) return resident_launch<kSelThreadsWide, 16, true, E>(set, nullptr, (int)blocks, 0, st, stream);
    }
    if (lim_max + 1 <= kResident) return resident_512<E>(set, nullptr, (int)blocks, 0, lim_max, st, stream);
    // one sequence whose rows grow past that: its shorter rows on their own
    if (st.n == 1 && rs.step > 0) {
      const int64_t p0 = (int64_t)st.q_pos0[0] - rs.shift;
      const int64_t first = (kResident - 1 - p0) / rs.step + 1;  // first row longer than kResident
      if (first - rs.i0 >= kWideMaxRows && first < rs.i1) {
        RowSpace lo = rs, hi = rs;
        lo.i1 = hi.i0 = (int32_t)first;
        const int64_t lim_lo = std::min<int64_t>(lim_max, p0 + (first - 1) * rs.step);
        const hipError_t e = topk_launch(scores, ld, st, lo, od, lim_lo, scratch, scratch_bytes, stream);
        if (e != hipSuccess) return e;
        return topk_launch(scores + (first - rs.i0) * ld, ld, st, hi, od, lim_max, scratch, scratch_bytes, stream);
      }
    }
  }
  if (blocks <= kWideMaxRows && lim_max + 1 >= kSampleMinLen && scratch &&
      scratch_bytes >= split_scratch_bytes(blocks)) {
    // few long rows: P slice workgroups per row, then one merge workgroup
    const int P = (int)std::max<int64_t>(kSplitMinP, std::min<int64_t>(kSplitMaxP, kSplitTargetBlocks / blocks));
    const int per = kSplitSlots / P;
    uint2* cand = reinterpret_cast<uint2*>(scratch);
    int32_t* cnt = reinterpret_cast<int32_t*>(cand + (size_t)blocks * kSplitSlots);
    float* thr = reinterpret_cast<float*>(cnt + (size_t)blocks * kSplitMaxP);
    const dim3 sgrid((unsigned)blocks, (unsigned)P);
    const bool small = od.m <= kSelCapSmall / 2;
    if (small)
      hipLaunchKernelGGL((topk_thr_kernel<kSelCapSmall, kSelThreadsWide, E>), dim3((unsigned)blocks),
                         dim3(kSelThreadsWide), 0, stream, scores, ld, st, rs, od.m, thr);
    else
      hipLaunchKernelGGL((topk_thr_kernel<kSelCapLarge, kSelThreadsWide, E>), dim3((unsigned)blocks),
                         dim3(kSelThreadsWide), 0, stream, scores, ld, st, rs, od.m, thr);
    hipLaunchKernelGGL(topk_slice_kernel<E>, sgrid, dim3(kSplitThreads), 0, stream, scores, ld, st, rs, P, per, thr,
                       cand, cnt);
    if (small)
      hipLaunchKernelGGL((topk_merge_kernel<kSelCapSmall, kSelThreadsWide, E>), dim3((unsigned)blocks),
                         dim3(kSelThreadsWide), 0, stream, scores, ld, st, rs, od, P, per, cand, cnt);
    else
      hipLaunchKernelGGL((topk_merge_kernel<kSelCapLarge, kSelThreadsWide, E>), dim3((unsigned)blocks),
                         dim3(kSelThreadsWide), 0, stream, scores, ld, st, rs, od, P, per, cand, cnt);
    return hipGetLastError();
  }
  if (blocks <= kWideMaxRows && lim_max + 1 >= kSampleMinLen) {
    // few long rows (decode): one wide workgroup per row
    if (od.m <= kSelCapSmall / 2)
      hipLaunchKernelGGL((topk_rows_kernel<kSelCapSmall, kSelThreadsWide, true, E>), dim3((unsigned)blocks),
                         dim3(kSelThreadsWide), 0, stream, scores, ld, st, rs, od);
    else
      hipLaunchKernelGGL((topk_rows_kernel<kSelCapLarge, kSelThreadsWide, true, E>), dim3((unsigned)blocks),
                         dim3(kSelThreadsWide), 0, stream, scores, ld, st, rs, od);
    return hipGetLastError();
  }
  const bool small = od.m <= kSelCapSmall / 2, sample = lim_max + 1 >= kSampleMinLen;
  const dim3 grid((unsigned)blocks), block(kSelThreads);
  if constexpr (sizeof(E) == 2) {  // bf16 rows: 6-byte candidates, three workgroups per CU
    // only when every row takes the sampled path (a short row would fall back
    // to a two-level select with the smaller buffer the shared region leaves)
    if (sample && min_limit(st, rs) + 1 >= kSampleMinLen) {
      if (small)
        hipLaunchKernelGGL((topk_rows16_kernel<kSelCapSmall, kSelThreads>), grid, block, 0, stream, scores, ld, st,
                           rs, od);
      else
        hipLaunchKernelGGL((topk_rows16_kernel<kSelCap16, kSelThreads>), grid, block, 0, stream, scores, ld, st, rs,
                           od);
      return hipGetLastError();
    }
  }
  if (small && sample)
    hipLaunchKernelGGL((topk_rows_kernel<kSelCapSmall, kSelThreads, true, E>), grid, block, 0, stream, scores, ld, st, rs,
                       od);
  else if (sample)
    hipLaunchKernelGGL((topk_rows_kernel<kSelCapLarge, kSelThreads, true, E>), grid, block, 0, stream, scores, ld, st, rs,
                       od);
  else
    hipLaunchKernelGGL((topk_rows_kernel<kSelCapLarge, kSelThreads, false, E>), grid, block, 0, stream, scores, ld, st,
                       rs, od);
  return hipGetLastError();
}

hipError_t launch_topk(const void* scores, bool scores_bf16, int64_t ld, const SeqTable& st, const RowSpace& rs,
                       const OutDesc& od, int64_t lim_max, void* scratch, size_t scratch_bytes,
                       hipStream_t stream) {
  if (scores_bf16)
    return topk_launch(static_cast<const bf16_t*>(scores), ld, st, rs, od, lim_max, scratch, scratch_bytes, stream);
  return topk_launch(static_cast<const float*>(scores), ld, st, rs, od, lim_max, scratch, scratch_bytes, stream);
}

__global__ void fill_guardrail_kernel(int32_t* base, int width, SeqTable st, int j0, int32_t value) {
  const int j = j0 + blockIdx.x, b = blockIdx.y;
  if (b >= st.n || j >= st.first_proxy[b]) return;
  int32_t* row = base + ((int64_t)st.grp0[b] + j) * width;
  for (int e = threadIdx.x; e < width; e += blockDim.x) row[e] = value;
}

hipError_t launch_fill_guardrail(int32_t* base, int width, const SeqTable& st, int j0, int j1, int32_t value,
                                 hipStream_t stream) {
  if (j1 <= j0 || st.n <= 0) return hipSuccess;
  hipLaunchKernelGGL(fill_guardrail_kernel, dim3((unsigned)(j1 - j0), (unsigned)st.n), dim3(256), 0, stream, base,
                     width, st, j0, value);
  return hipGetLastError();
}

struct CopyDst {
  int32_t* p[kMaxCopyDst];
  int32_t n;
};

// Grid-stride copy of src[0, n) to every destination; vec: every pointer is
// 16-byte aligned, so the bulk moves as int4.
__global__ __launch_bounds__(256) void copy_fanout_kernel(const int32_t* __restrict__ src, CopyDst dst, int64_t n,
                                                          int vec) {
  const int64_t step = (int64_t)gridDim.x * blockDim.x;
  const int64_t i0 = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  int64_t tail = 0;
  if (vec) {
    const int64_t n4 = n / 4;
    const int4* s4 = reinterpret_cast<const int4*>(src);
    for (int64_t j = i0; j < n4; j += step) {
      const int4 v = s4[j];
      for (int d = 0; d < dst.n; ++d) reinterpret_cast<int4*>(dst.p[d])[j] = v;
    }
    tail = 4 * n4;
  }
  for (int64_t e = tail + i0; e < n; e += step) {
    const int32_t v = src[e];
    for (int d = 0; d < dst.n; ++d) dst.p[d][e] = v;
  }
}

hipError_t launch_copy_fanout(const int32_t* src, int32_t* const* dst, int n_dst, int64_t n, hipStream_t stream) {
  if (n <= 0 || n_dst <= 0) return hipSuccess;
  if (n_dst > kMaxCopyDst) return hipErrorInvalidValue;
  CopyDst cd;
  memset(&cd, 0, sizeof cd);
  cd.n = n_dst;
  bool vec = (reinterpret_cast<uintptr_t>(src) & 15u) == 0;
  for (int d = 0; d < n_dst; ++d) {
    cd.p[d] = dst[d];
    vec = vec && (reinterpret_cast<uintptr_t>(dst[d]) & 15u) == 0;
  }
  const int64_t units = vec ? std::max<int64_t>(n / 4, 1) : n;
  const int64_t blocks = std::min<int64_t>((units + 255) / 256, 4096);
  hipLaunchKernelGGL(copy_fanout_kernel, dim3((unsigned)blocks), dim3(256), 0, stream, src, cd, n, (int)vec);
  return hipGetLastError();
}

}  // namespace pivot
