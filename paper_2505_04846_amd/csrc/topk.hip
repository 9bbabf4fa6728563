// Exact top-k of each row of an fp32 score matrix, ordered (score desc, index asc).
//
// One 1024-thread workgroup per row, keyed by the order-preserving uint32 map of the score and,
// to break ties by lower index, the 64-bit key (score key << 32) | ~index (unique per row).
//
// Fast path (one pass over the row):
//   1. Sample.  About one score in 64 (up to 16384), in evenly spaced runs of 8 entries; a bound
//      t that about `want` sample keys reach (want chosen so that the expected number of row
//      entries at or above t lies well inside [k, kCap], see below).
//   2. Stream.  Every entry with key >= t is appended to an LDS candidate list (kCap entries).
//      If t is too high (fewer than k candidates) or the list overflows, the row takes the slow
//      path.  Otherwise the candidates contain the top-k: any other entry is below t and at
//      least k candidates are at or above it.
//   3. Select.  A bound that at least k and few more candidates reach, ties at the k-th score cut
//      by index; what reaches it is sorted and the first k written out.
// Rows of at most kCap entries are loaded whole and go straight to step 3.  Few long rows are
// streamed by several workgroups each (topk_slices_kernel, which leaves each slice's candidates in
// a scratch buffer) and selected by one (topk_merge_kernel).
//
// Bounds are found by histograms of 2048 bins spread over the keys' actual range (select_bound),
// narrowed to the bin that holds the wanted entry until few enough entries are left.  Digits of
// fixed place would not do: scores of one row share their exponent, so the first eight bits put
// every candidate into two or three bins, whose atomics serialise.
//
// Slow path (any row, exact): the same narrowing over the row in global memory, then a gather of
// the entries above the k-th key and of the lowest-index entries equal to it, and the same sort.
#include "common.h"
#include "kernels.h"

namespace hpr {

namespace {

constexpr int kThreads = 1024;
constexpr int kWaves = kThreads / kWave;
constexpr int kMaxK = 1024;
constexpr int kCap = 8192;      // LDS candidate list (keys and indices: 64 KiB)
constexpr int kRun = 8;         // sample: runs of 8 entries (two vectors), one run in 512 entries
constexpr int kMaxRuns = 2 * kCap / kRun;  // at most 2048 of them (16384 keys)
constexpr int kUnroll = 8;      // 16-byte loads in flight per thread while streaming
constexpr int kBinBits = 11;
constexpr int kBins = 1 << kBinBits;  // two per thread
constexpr uint32_t kWindow = 1u << 25;

// LDS of a workgroup (72 KiB: two fit a CU).
struct TopkShared {
  // candidate scores (as they came), then indices; during the sample, its keys
  uint32_t cbuf[2 * kCap];
  union {  // the histogram while a bound is searched, then the winners
    unsigned long long sk[kMaxK];
    uint32_t hist[kBins];
  };
  uint32_t wave_cnt[kWaves];
  uint32_t sh[4];
  uint32_t n_cand, lo, hi;
};

__device__ __forceinline__ unsigned long long key64(uint32_t key, uint32_t idx) {
  return ((unsigned long long)key << 32) | (unsigned long long)(~idx);
}

// A bound and how many entries lie above the range it stands for and inside it.
struct Bound {
  uint32_t key, above, in;
};

// Suffix sums over the workgroup's threads: the values c of this thread and all after it (and the
// total).  One barrier inside; s.wave_cnt may be rewritten after the next one.
__device__ __forceinline__ uint32_t count_from(uint32_t c, TopkShared& s, uint32_t& total) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const uint32_t y = __shfl_down(c, o);
    if (lane + o < 64) c += y;
  }
  if (lane == 0) s.wave_cnt[wave] = c;
  __syncthreads();
  total = 0;
#pragma unroll
  for (int w = 0; w < kWaves; ++w) {
    const uint32_t x = s.wave_cnt[w];
    c += w > wave ? x : 0u;
    total += x;
  }
  return c;
}

// Among the entries i < m with get(i, key) true and key in [lo, hi] (at least `want` of them, 1 <=
// want): a bound that at least `want` reach, lowered no further than to the lower edge of the
// histogram bin that holds the want-th largest.  Narrowed until at most `most` entries reach it
// (above + in <= most) or, with EXACT or when ties keep it from that, until it is the want-th
// largest key itself (in: the entries equal to it).  At most four passes: one over the window where
// the wanted entry lies below it, then 11 bits of the rest each (three for 32).
template <bool EXACT, class Get>
__device__ __forceinline__ Bound select_bound(Get get, int64_t m, uint32_t want, uint32_t most, uint32_t lo,
                              uint32_t hi, TopkShared& s) {
  const int tid = threadIdx.x;
  uint32_t above = 0;
  // The first pass looks at the top 2^25 keys only (four octaves below the largest score): bins
  // spread over all of a row whose scores straddle zero would hold an eighth of an octave each.
  uint32_t base = lo;
  if (hi - lo > kWindow) lo = hi - kWindow;
  for (;;) {
    const uint32_t range = hi - lo;
    const int bits = range ? 32 - __clz(range) : 0;
    const int shift = bits > kBinBits ? bits - kBinBits : 0;
    s.hist[tid] = 0;
    s.hist[tid + kThreads] = 0;
    __syncthreads();
    for (int64_t i = tid; i < m; i += kThreads) {
      uint32_t key;
      if (get(i, key) && key >= lo && key <= hi) atomicAdd(&s.hist[(key - lo) >> shift], 1u);
    }
    __syncthreads();
    const uint32_t h0 = s.hist[2 * tid], h1 = s.hist[2 * tid + 1];
    uint32_t total;
    const uint32_t incl = above + count_from(h0 + h1, s, total);
    total += above;
    if (total < want) {  // uniform: the wanted entry lies below the window
      above = total;
      hi = lo - 1;
      lo = base;
      __syncthreads();  // wave_cnt is rewritten by the next pass
      continue;
    }
    const uint32_t excl = incl - (h0 + h1);
    if (excl < want && want <= incl) {  // the want-th largest is in one of this thread's bins
      const bool upper = want <= excl + h1;
      s.sh[0] = 2 * tid + (upper ? 1 : 0);
      s.sh[1] = upper ? excl : excl + h1;
      s.sh[2] = upper ? h1 : h0;
    }
    __syncthreads();
    above = s.sh[1];
    const uint32_t in = s.sh[2];
    lo += s.sh[0] << shift;
    const uint32_t span = (1u << shift) - 1u;
    hi = hi - lo < span ? hi : lo + span;
    if (shift == 0 || (!EXACT && above + in <= most)) return {lo, above, in};
  }
}

// Block-wide minimum and maximum of the threads' keys into s.lo and s.hi (set up by the caller
// before a barrier: s.lo = ~0, s.hi = 0); complete after the next barrier.
__device__ __forceinline__ void merge_range(uint32_t mn, uint32_t mx, TopkShared& s) {
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) {
    const uint32_t a = __shfl_xor(mn, o), b = __shfl_xor(mx, o);
    mn = a < mn ? a : mn;
    mx = b > mx ? b : mx;
  }
  if ((threadIdx.x & 63) == 0) {
    atomicMin(&s.lo, mn);
    atomicMax(&s.hi, mx);
  }
}

// The winners left in s.sk: n 64-bit keys, k <= n <= P, P a power of two in [64, 1024], their score
// keys in [lo, hi].
struct Winners {
  uint32_t n, P, lo, hi;
};

// Sorts the winners, largest first, and writes the first k as (score, index) of row `row`.
// A key's place is the number of keys above it.  Up to 128 keys, eight threads count for each.
// Above, 2048 bins over [lo, hi]: the keys of the bins above, then the larger ones among the few
// of its own bin; if a bin holds more than kCrowd keys, a bitonic network over one key per thread
// (k = 1000: 2 us against 8 for the network, whose 55 exchanges are 64 bits wide).
__device__ __forceinline__ void sort_and_write(TopkShared& s, const Winners& w, uint32_t k,
                                               int64_t row, float* out_s, int64_t* out_i) {
  const uint32_t n = w.n, P = w.P, lo = w.lo, hi = w.hi;
  const uint32_t tid = threadIdx.x;
  constexpr uint32_t kCrowd = 24;
  __syncthreads();
  unsigned long long v;
  uint32_t at;
  bool mine;
  if (n <= 128) {
    const uint32_t e = tid >> 3;
    mine = e < n;
    v = mine ? s.sk[e] : 0ull;
    at = 0;
    if (mine)
      for (uint32_t j = tid & 7; j < n; j += 8) at += s.sk[j] > v ? 1u : 0u;
#pragma unroll
    for (int o = 1; o < 8; o <<= 1) at += __shfl_xor(at, o);
    mine = mine && (tid & 7) == 0;
  } else {
    uint32_t* hist = s.cbuf;  // the candidates are no longer needed
    unsigned long long* binned = reinterpret_cast<unsigned long long*>(s.cbuf + kBins);
    mine = tid < n;
    v = mine ? s.sk[tid] : 0ull;  // 0: below every real key
    hist[tid] = 0;
    hist[tid + kThreads] = 0;
    __syncthreads();
    const int bits = hi > lo ? 32 - __clz(hi - lo) : 0;
    const int shift = bits > kBinBits ? bits - kBinBits : 0;
    const uint32_t bin = mine ? ((uint32_t)(v >> 32) - lo) >> shift & (kBins - 1) : 0u;
    const uint32_t nth = mine ? atomicAdd(&hist[bin], 1u) : 0u;
    if (!__syncthreads_or(nth >= kCrowd)) {
      const uint32_t h0 = hist[2 * tid], h1 = hist[2 * tid + 1];
      uint32_t total;
      const uint32_t above = count_from(h0 + h1, s, total) - (h0 + h1);
      hist[2 * tid + 1] = above | h1 << 16;  // (at most 1024 of each)
      hist[2 * tid] = (above + h1) | h0 << 16;
      __syncthreads();
      const uint32_t first = hist[bin] & 0xffffu, count = hist[bin] >> 16;
      if (mine) binned[first + nth] = v;
      __syncthreads();
      at = first;
      if (mine)
        for (uint32_t j = 0; j < count; ++j) at += binned[first + j] > v ? 1u : 0u;
    } else {
      for (uint32_t size = 2; size <= P; size <<= 1) {
        for (uint32_t stride = size >> 1; stride > 0; stride >>= 1) {
          unsigned long long o = 0;
          if (stride >= 64) {
            __syncthreads();
            if (tid < P) s.sk[tid] = v;
            __syncthreads();
            if (tid < P) o = s.sk[tid ^ stride];
          } else {
            o = __shfl_xor(v, (int)stride);
          }
          const bool larger = ((tid & stride) == 0) == ((tid & size) == 0);
          v = (o > v) == larger ? o : v;
        }
      }
      at = tid;
    }
  }
  if (mine && at < k) {
    out_s[row * k + at] = key_score((uint32_t)(v >> 32));
    out_i[row * k + at] = (int64_t)(uint32_t)~(uint32_t)v;
  }
}

// Step 3: the winners among the m candidates of s.cbuf (k <= m <= kCap; s.lo <= every key <= s.hi).
__device__ __forceinline__ Winners select_winners(TopkShared& s, uint32_t m, uint32_t k) {
  const uint32_t tid = threadIdx.x;
  const float* cval = reinterpret_cast<const float*>(s.cbuf);
  const uint32_t* cidx = s.cbuf + kCap;
  uint32_t P = 64;
  while (P < k) P <<= 1;
  auto key_of = [&](int64_t i, uint32_t& key) {
    key = score_key(cval[i]);
    return true;
  };
  const uint32_t hi = s.hi;
  const Bound b = select_bound<false>(key_of, m, k, P, s.lo, hi, s);
  uint32_t tie = 0;  // of the entries equal to b.key, those with ~index >= tie
  uint32_t n = b.above + b.in;
  if (n > P) {  // uniform: more entries equal to the k-th key than there is room for
    auto tie_of = [&](int64_t i, uint32_t& key) {
      key = ~cidx[i];
      return score_key(cval[i]) == b.key;
    };
    tie = select_bound<true>(tie_of, m, k - b.above, 0, 0u, ~0u, s).key;
    n = k;
  }
  if (tid == 0) s.n_cand = 0;
  __syncthreads();
  for (uint32_t i = tid; i < m; i += kThreads) {
    const uint32_t key = score_key(cval[i]);
    if (key > b.key || (key == b.key && ~cidx[i] >= tie)) {
      const uint32_t p = atomicAdd(&s.n_cand, 1u);
      if (p < kMaxK) s.sk[p] = key64(key, cidx[i]);
    }
  }
  return {n, P, b.key, hi};
}

// The row's aligned part: whole 16-byte vectors from the first 16-byte boundary.
struct RowVec {
  const f32x4* v;
  int64_t head, nv;
};
__device__ __forceinline__ RowVec row_vec(const float* x, int64_t n) {
  RowVec r;
  r.head = (int64_t)((16u - (uint32_t)(reinterpret_cast<uintptr_t>(x) & 15u)) & 15u) / 4;
  r.nv = (n - r.head) / 4;  // n > kCap > head
  r.v = reinterpret_cast<const f32x4*>(x + r.head);
  return r;
}

// Step 1: nr runs of kRun entries, run r starting at vector r * nv / nr of the row's aligned part
// (nv >= 2 nr, so runs do not overlap); about one entry in 64 is sampled, at most kMaxRuns runs.
// The bound is one that about want sample keys reach (up to an eighth more): about want * n / ns row
// entries do, with a relative spread of about 1 / sqrt(want).  Aimed at 8 k entries, between 1024 and
// 4096: at 4096 want is 64 and the spread 512, so k <= 1024 and kCap are six standard deviations away;
// at 1024 want is 16, and fewer than k <= 128 or more than kCap entries as unlikely.  On rows longer
// than 2^20 the sample is thinner while want is at least 16: about n / 1024 entries reach the bound,
// so the list overflows often past 5 million and nearly always past 8.4 million.
// The runs are shorter than want because neighbours score alike: a paper's chunks lie together, and
// where one paper outscores the rest, its entries in the sample are those of the runs inside it.  With
// runs of 64 and want = 16, a run inside a paper of 64 to 400 chunks put the bound so high that fewer
// than k = 100 of them reached it, and the row took the slow path: 64 queries, each with such a paper
// of 200 chunks among 1,000,000 rows, took 1520 us instead of 66.  Runs of 8 can only do so where
// want / 8 of them fit, in a cluster of more than k entries.
__device__ __forceinline__ uint32_t sample_bound(const RowVec& r, int64_t n, int k, TopkShared& s) {
  const int tid = threadIdx.x;
  constexpr int kVec = kRun / 4, kPer = 64 * kRun;
  const int nr = (n + kPer - 1) / kPer < kMaxRuns ? (int)((n + kPer - 1) / kPer) : kMaxRuns;
  const int ns = kRun * nr;
  if (tid == 0) {
    s.lo = ~0u;
    s.hi = 0u;
  }
  __syncthreads();
  uint32_t mn = ~0u, mx = 0u;
  for (int u = tid; u < kVec * nr; u += kThreads) {
    const f32x4 v = r.v[(int64_t)(u / kVec) * r.nv / nr + u % kVec];
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      const uint32_t key = score_key(v[c]);
      s.cbuf[4 * u + c] = key;
      mn = key < mn ? key : mn;
      mx = key > mx ? key : mx;
    }
  }
  merge_range(mn, mx, s);
  __syncthreads();
  const int aim = 8 * k < 1024 ? 1024 : 8 * k > 4096 ? 4096 : 8 * k;
  int64_t want = (int64_t)ceil((double)aim * ns / (double)n);
  want = want > 64 ? 64 : (want < 16 ? 16 : want);
  auto key_of = [&](int64_t i, uint32_t& key) {
    key = s.cbuf[i];
    return true;
  };
  return select_bound<false>(key_of, ns, (uint32_t)want, (uint32_t)(want + want / 8), s.lo, s.hi,
                             s)
      .key;
}

// Step 2 over the vectors [j0, j1) of the row, and with `ends` the few entries before and after
// them: appends the entries with key >= t to s.cbuf, counts them in s.n_cand and their keys' range
// in s.lo, s.hi (complete after the next barrier).
__device__ __forceinline__ void stream_candidates(const float* x, int64_t n, const RowVec& r, int64_t j0,
                                  int64_t j1, bool ends, uint32_t t, TopkShared& s) {
  const int tid = threadIdx.x, lane = tid & 63;
  float* cval = reinterpret_cast<float*>(s.cbuf);
  uint32_t* cidx = s.cbuf + kCap;
  __syncthreads();  // the sample's last reads of cbuf and of the range are done
  if (tid == 0) {
    s.n_cand = 0;
    s.lo = t;
    s.hi = t;
  }
  __syncthreads();
  // Among numbers v >= tf is score_key(v) >= t.  A NaN's key lies above or below every number's, by
  // its sign: a row that holds one takes the slow path, which compares keys only.
  const float tf = key_score(t);
  float mx = tf;
  bool nan = false;
  if (ends) {
    const int64_t tail = r.head + 4 * r.nv;
    const int64_t i = tid < r.head ? tid : tail + tid - r.head;
    if (i < n && !(x[i] < tf)) {
      const uint32_t p = atomicAdd(&s.n_cand, 1u);
      if (p < (uint32_t)kCap) {
        cval[p] = x[i];
        cidx[p] = (uint32_t)i;
      }
      mx = x[i];
      nan = x[i] != x[i];
    }
  }
  // Per wave and half batch: the ballots of its 16 x 64 tests, held in scalar registers, whose count
  // reserves the wave's places in the list with one atomic; only the tests that some lane passed
  // are visited again, and what they write is the entry as it came and a 32-bit index.  A workgroup
  // alone on its CU is bound by these vector instructions (see topk_rows_kernel).
  constexpr int kHalf = kUnroll / 2;
  for (int64_t base = j0; base < j1; base += (int64_t)kThreads * kUnroll) {
    f32x4 v[kUnroll];
#pragma unroll
    for (int u = 0; u < kUnroll; ++u) {
      const int64_t j = base + (int64_t)u * kThreads + tid;
      // streaming (non-temporal) loads: the row is read once, and keeping it out of L2
      // measured 10 % faster (0.382 -> 0.345 ms for 1,024 rows of 500,000)
      v[u] = j < j1 ? __builtin_nontemporal_load(r.v + j) : f32x4{0.f, 0.f, 0.f, 0.f};
    }
    const uint32_t i0 = (uint32_t)(r.head + 4 * (base + tid));
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      uint64_t pass[4 * kHalf];
      uint32_t count = 0;
#pragma unroll
      for (int u = 0; u < kHalf; ++u) {
        const uint64_t in = __ballot(base + (int64_t)(h * kHalf + u) * kThreads + tid < j1);
#pragma unroll
        for (int c = 0; c < 4; ++c) {
          pass[4 * u + c] = __ballot(!(v[h * kHalf + u][c] < tf)) & in;
          count += (uint32_t)__popcll(pass[4 * u + c]);
        }
      }
      if (count == 0) continue;  // wave-uniform
      uint32_t p = 0;
      if (lane == 0) p = atomicAdd(&s.n_cand, count);
      p = __builtin_amdgcn_readfirstlane(p);
      if (p + count > (uint32_t)kCap) continue;  // the row takes the slow path: nothing to keep
#pragma unroll
      for (int u = 0; u < kHalf; ++u) {
#pragma unroll
        for (int c = 0; c < 4; ++c) {
          const uint64_t m = pass[4 * u + c];
          if (m == 0) continue;
          if ((m >> lane) & 1ull) {
            const uint32_t at = __builtin_amdgcn_mbcnt_hi(
                (uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, p));
            cval[at] = v[h * kHalf + u][c];
            cidx[at] = i0 + (uint32_t)(4 * kThreads * (h * kHalf + u) + c);
            mx = fmaxf(mx, v[h * kHalf + u][c]);
            nan = nan || v[h * kHalf + u][c] != v[h * kHalf + u][c];
          }
          p += (uint32_t)__popcll(m);
        }
      }
    }
  }
  if (__any(nan) && lane == 0) atomicMax(&s.n_cand, (uint32_t)kCap + 1u);
  merge_range(t, score_key(mx), s);
}

// Slow path: exact select over the row in global memory.
__device__ __forceinline__ Winners slow_row(const float* x, int64_t n, uint32_t k,
                                            TopkShared& s) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  auto key_of = [&](int64_t i, uint32_t& key) {
    key = score_key(x[i]);
    return true;
  };
  const Bound b = select_bound<true>(key_of, n, k, 0, 0u, ~0u, s);
  const uint32_t K = b.key, n_gt = b.above, need_eq = k - n_gt;
  if (tid == 0) s.n_cand = 0;
  __syncthreads();
  uint32_t eq_base = 0;
  for (int64_t base = 0; base < n; base += kThreads) {
    const int64_t i = base + tid;
    bool gt = false, eq = false;
    uint32_t key = 0;
    if (i < n) {
      key = score_key(x[i]);
      gt = key > K;
      eq = key == K;
    }
    if (gt) {
      const uint32_t p = atomicAdd(&s.n_cand, 1u);
      if (p < n_gt) s.sk[p] = key64(key, (uint32_t)i);  // always true for finite inputs
    }
    const unsigned long long m = __ballot(eq);
    if (lane == 0) s.wave_cnt[wave] = (uint32_t)__popcll(m);
    __syncthreads();
    const uint32_t gt_found = s.n_cand;  // stable: this chunk's atomics are done
    uint32_t before = 0, chunk_total = 0;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) {
      const uint32_t cw = s.wave_cnt[w];
      before += w < wave ? cw : 0u;
      chunk_total += cw;
    }
    if (eq) {  // the lowest-index entries equal to K, in index order
      const uint32_t r = eq_base + before + (uint32_t)__popcll(m & ((1ull << lane) - 1ull));
      if (r < need_eq) s.sk[n_gt + r] = key64(key, (uint32_t)i);
    }
    eq_base += chunk_total;
    __syncthreads();
    if (eq_base >= need_eq && gt_found == n_gt) break;  // everything needed is collected
  }
  uint32_t P = 64;
  while (P < k) P <<= 1;
  return {k, P, K, ~0u};
}

// One workgroup per row.  Bound by memory where the rows fill the chip (two workgroups per CU, which
// is what 64 registers and 72 KiB of LDS are for): 4,096 rows of 131,072 in 387 us, 5.5 TB/s, k =
// 100 (426 with an atomic and a key per streamed entry and fixed eight-bit digits; 377 to 381 with
// sample runs of 64, whose cache lines are a quarter as many); 1,024 rows of 50,000 in 55 us (79).  A
// few rows are bound by the chain of steps and by their own CU's vector
// instructions: 20,000 entries in 11.6 us at k = 100 and 15.3 at k = 1000 (18.4 and 28.9), 8,000 in
// 9.7 and 12.3 (15.4 and 25.8).
__global__ __launch_bounds__(kThreads, 8) void topk_rows_kernel(const float* __restrict__ S,
                                                             int64_t n, int64_t ld, int k,
                                                             float* out_s, int64_t* out_i) {
  __shared__ TopkShared s;
  const int tid = threadIdx.x;
  const int64_t row = blockIdx.x;
  const float* x = S + row * ld;
  if (n <= kCap) {  // the whole row is the candidate list
    if (tid == 0) {
      s.n_cand = (uint32_t)n;
      s.lo = ~0u;
      s.hi = 0u;
    }
    __syncthreads();
    uint32_t mn = ~0u, mx = 0u;
#pragma unroll
    for (int u = 0; u < kCap / kThreads; ++u) {
      const int i = u * kThreads + tid;
      if (i < n) {
        const uint32_t key = score_key(x[i]);
        s.cbuf[i] = __float_as_uint(x[i]);
        s.cbuf[kCap + i] = (uint32_t)i;
        mn = key < mn ? key : mn;
        mx = key > mx ? key : mx;
      }
    }
    merge_range(mn, mx, s);
  } else {
    const RowVec r = row_vec(x, n);
    const uint32_t t = sample_bound(r, n, k, s);
    stream_candidates(x, n, r, 0, r.nv, true, t, s);
  }
  __syncthreads();
  const uint32_t m = s.n_cand;  // uniform
  const Winners w = m >= (uint32_t)k && m <= (uint32_t)kCap ? select_winners(s, m, (uint32_t)k)
                                                            : slow_row(x, n, (uint32_t)k, s);
  sort_and_write(s, w, (uint32_t)k, row, out_s, out_i);
}

// A slice's candidates in the scratch buffer: the count (which may exceed kCap: the list then
// holds the first kCap that came), then kCap scores and kCap indices.
struct SliceList {
  uint32_t count, pad[3];
  uint32_t val[kCap], idx[kCap];
};

// Workgroup (slice, row): the row's sample bound (every slice computes the same one) and the
// candidates of its slice of the row's vectors.
__global__ __launch_bounds__(kThreads, 8) void topk_slices_kernel(const float* __restrict__ S,
                                                               int64_t n, int64_t ld, int k,
                                                               int slices,
                                                               SliceList* __restrict__ lists) {
  __shared__ TopkShared s;
  const int slice = blockIdx.x % slices;
  const int64_t row = blockIdx.x / slices;
  const float* x = S + row * ld;
  const RowVec r = row_vec(x, n);
  const uint32_t t = sample_bound(r, n, k, s);
  stream_candidates(x, n, r, r.nv * slice / slices, r.nv * (slice + 1) / slices, slice == 0, t, s);
  __syncthreads();
  SliceList& l = lists[blockIdx.x];
  const uint32_t m = s.n_cand < (uint32_t)kCap ? s.n_cand : (uint32_t)kCap;
  for (uint32_t i = threadIdx.x; i < m; i += kThreads) {
    l.val[i] = s.cbuf[i];
    l.idx[i] = s.cbuf[kCap + i];
  }
  if (threadIdx.x == 0) l.count = s.n_cand;
}

// One workgroup per row: the slices' candidates collected, then step 3 (or the slow path).
constexpr int kMaxSlices = 64;
__global__ __launch_bounds__(kThreads, 8) void topk_merge_kernel(const float* __restrict__ S,
                                                              int64_t n, int64_t ld, int slices,
                                                              const SliceList* __restrict__ lists,
                                                              int k, float* out_s,
                                                              int64_t* out_i) {
  __shared__ TopkShared s;
  __shared__ uint32_t start[kMaxSlices + 1];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int64_t row = blockIdx.x;
  const SliceList* l = lists + row * slices;
  if (tid == 0) {
    s.lo = ~0u;
    s.hi = 0u;
  }
  if (wave == 0) {  // counts (capped: a sum over 64 of them stays in range) and their prefix sums
    uint32_t c = lane < slices ? l[lane].count : 0u;
    c = c < (uint32_t)kCap + 1u ? c : (uint32_t)kCap + 1u;
    uint32_t incl = c;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const uint32_t y = __shfl_up(incl, o);
      if (lane >= o) incl += y;
    }
    start[lane + 1] = incl;
    if (lane == 0) start[0] = 0u;
  }
  __syncthreads();
  const uint32_t m = start[kMaxSlices];
  Winners w;
  if (m >= (uint32_t)k && m <= (uint32_t)kCap) {  // uniform
    uint32_t mn = ~0u, mx = 0u;
    for (int sl = wave; sl < slices; sl += kWaves) {
      const uint32_t at = start[sl], c = start[sl + 1] - at;
      for (uint32_t i = lane; i < c; i += kWave) {
        const uint32_t bits = l[sl].val[i], key = score_key(__uint_as_float(bits));
        s.cbuf[at + i] = bits;
        s.cbuf[kCap + at + i] = l[sl].idx[i];
        mn = key < mn ? key : mn;
        mx = key > mx ? key : mx;
      }
    }
    merge_range(mn, mx, s);
    __syncthreads();
    w = select_winners(s, m, (uint32_t)k);
  } else {
    w = slow_row(S + row * ld, n, (uint32_t)k, s);
  }
  sort_and_write(s, w, (uint32_t)k, row, out_s, out_i);
}

// Slices per row: 1 (one workgroup per row) unless the rows are few and long.  One row of 59,000
// takes 15 us whole and 8 + 6.5 in slices; of 131,000, 24 against 9 + 6.5; of a million, 11 + 6.5.
constexpr int64_t kSliceMinN = 60000;
int topk_slices(int64_t rows, int64_t n) {
  if (n < kSliceMinN || rows > 64) return 1;
  int64_t p = n / 16384;
  if (p > 256 / rows) p = 256 / rows;
  return p < 2 ? 1 : p > kMaxSlices ? kMaxSlices : (int)p;
}

}  // namespace

size_t topk_scratch_bytes(int64_t rows, int64_t n) {
  const int p = topk_slices(rows, n);
  return p > 1 ? (size_t)rows * (size_t)p * sizeof(SliceList) : 0;
}

size_t topk_scratch_most(int64_t rows, int64_t n) {
  if (n < kSliceMinN) return 0;
  const int64_t p = n / 16384 < kMaxSlices ? n / 16384 : kMaxSlices;
  const int64_t lists = (rows < 64 ? rows : 64) * p;  // and at most 256, whatever the rows
  return (size_t)(lists < 256 ? lists : 256) * sizeof(SliceList);
}

hipError_t launch_topk_rows(const float* scores, int64_t rows, int64_t n, int64_t ld, int k,
                            float* out_scores, int64_t* out_idx, void* scratch,
                            hipStream_t stream) {
  if (k < 1 || k > kMaxK || k > n || rows < 1 || n >= (int64_t(1) << 32) - 1)
    return hipErrorInvalidValue;
  const int p = scratch ? topk_slices(rows, n) : 1;
  if (p > 1) {
    SliceList* lists = static_cast<SliceList*>(scratch);
    hipLaunchKernelGGL(topk_slices_kernel, dim3((unsigned)(rows * p)), dim3(kThreads), 0, stream,
                       scores, n, ld, k, p, lists);
    hipLaunchKernelGGL(topk_merge_kernel, dim3((unsigned)rows), dim3(kThreads), 0, stream, scores,
                       n, ld, p, lists, k, out_scores, out_idx);
  } else {
    hipLaunchKernelGGL(topk_rows_kernel, dim3((unsigned)rows), dim3(kThreads), 0, stream, scores,
                       n, ld, k, out_scores, out_idx);
  }
  return hipGetLastError();
}

}  // namespace hpr
