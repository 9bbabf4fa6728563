// Semantic chunking boundaries over a stream of sentence embeddings, and P@k / MRR@k of a
// retrieval ranking.
//
// Chunking: a segment grows while the cosine of each sentence with the one before it (in the same
// paper) stays strictly above a threshold; the first sentence of every paper opens a segment.
//   chunk_scan_kernel   one wave per range of chunk_rows_per_wave(n) consecutive sentences: each
//                       row is read once (16-byte streaming loads, the next batch of rows in
//                       flight while the current one is reduced; the row before the range is
//                       read once more for its norm), its squared norm and its dot product with
//                       the previous row come from v_dot2_f32_f16 (exact fp16 products, fp32
//                       sums) and two wave reductions; cos[t] = dot / sqrt(|prev|^2 |cur|^2), NaN
//                       at a paper's first sentence.  The boundary count of the workgroup's four
//                       ranges (cos not above the threshold, NaN included) goes to cnt[group].
//   chunk_ids_kernel    one workgroup per kIdRows sentences: seg[t] = (boundaries at or before t)
//                       - 1, from the groups' counts before it and a ballot prefix over its own
//                       cosines; the last one writes the number of segments.
//   chunk_offsets_kernel  long inputs only (more than kDirectGroups groups): one workgroup scans
//                       the group counts first, so that the ids kernel reads one offset instead
//                       of summing the counts before it.
// The passes read the embeddings once (the HBM-bound part) and the cosines twice.
//
// Metrics: one workgroup finds each query's 1-based rank of its positive among the first k
// retrieved indices (0 when absent) and sums the hits and the reciprocal ranks in fp64 in a
// fixed order.
#include "common.h"
#include "kernels.h"

namespace hpr {

namespace {

constexpr int kChunkThreads = 256;
constexpr int kChunkWaves = kChunkThreads / kWave;

typedef __attribute__((ext_vector_type(2))) _Float16 f16x2;

__device__ __forceinline__ float dot2_acc(uint32_t a, uint32_t b, float c) {
  return __builtin_amdgcn_fdot2(__builtin_bit_cast(f16x2, a), __builtin_bit_cast(f16x2, b), c,
                                false);
}

// Row t's chunks for this lane: chunk c = lane + 64 i (16 bytes each), zeros past `dim`.
template <int CPL>
__device__ __forceinline__ void load_row(const uint16_t* __restrict__ E, int64_t t, int dim,
                                         int lane, u32x4 (&v)[CPL]) {
  const uint16_t* row = E + t * dim;
#pragma unroll
  for (int i = 0; i < CPL; ++i) {
    const int c = lane + 64 * i;
    // streaming (non-temporal) loads: every row is read once (3.02 -> 2.53 ms at 2 M x 4096)
    v[i] = 8 * c < dim ? load16_stream(row + 8 * c) : u32x4{0u, 0u, 0u, 0u};
  }
}

template <int CPL>
__device__ __forceinline__ float row_dot(const u32x4 (&a)[CPL], const u32x4 (&b)[CPL]) {
  float s = 0.f;
#pragma unroll
  for (int i = 0; i < CPL; ++i) {
    s = dot2_acc(a[i].x, b[i].x, s);
    s = dot2_acc(a[i].y, b[i].y, s);
    s = dot2_acc(a[i].z, b[i].z, s);
    s = dot2_acc(a[i].w, b[i].w, s);
  }
  return s;
}

// wave_sum with its butterfly's own order (32, 16, 8, 4, 2, 1) but without LDS round trips: lane
// swaps, then rotations within a row of 16 lanes (by 8, and by 4 once the row has period 8, these
// are l ^ 8 and l ^ 4) and quad permutes.  Bit-identical to wave_sum.
template <int CTRL>
__device__ __forceinline__ float dpp_add(float v) {
  return v + __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, v), CTRL,
                                                                0xf, 0xf, false));
}
__device__ __forceinline__ float wave_sum_dpp(float v) {
  const auto a = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false,
                                                  false);
  v = __uint_as_float(a[0]) + __uint_as_float(a[1]);
  const auto b = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false,
                                                  false);
  v = __uint_as_float(b[0]) + __uint_as_float(b[1]);
  v = dpp_add<0x128>(v);  // row_ror:8
  v = dpp_add<0x124>(v);  // row_ror:4
  v = dpp_add<0x4e>(v);   // quad_perm [2, 3, 0, 1]
  return dpp_add<0xb1>(v);  // quad_perm [1, 0, 3, 2]
}

// First index d in [0, n_papers] with off[d] > t (n_papers + 1 when none): the next paper start
// after t is off[d] (skipping empty papers, whose offsets repeat).  A 64-way search by the whole
// wave: the lanes probe the last offset of 64 equal slices, those not above t form a prefix, and
// its length picks the slice (two dependent loads up to 4,095 papers).
__device__ __forceinline__ int64_t next_start_index(const int64_t* off, int64_t n_papers,
                                                    int64_t t, int lane) {
  int64_t lo = 0, hi = n_papers + 1;
  while (lo < hi) {
    const int64_t step = (hi - lo + 63) >> 6, last = hi - 1;
    int64_t p = lo + (int64_t)(lane + 1) * step - 1;
    p = p < last ? p : last;
    const int c = __popcll(__ballot(off[p] <= t));
    if (c == 64) return hi;  // off[last] is not above t either
    const int64_t pl = lo + (int64_t)c * step - 1, ph = pl + step;
    if (c > 0) lo = (pl < last ? pl : last) + 1;
    hi = ph < last ? ph : last;
  }
  return lo;
}

// Ranges of `rpw` sentences, one per wave; CPL 16-byte chunks per lane and row (dim <= 512 CPL),
// batches of B rows: with B CPL = 8 every wave has 8 KiB on the way while it reduces as much,
// whatever the dimension (400,000 x 768: 110 us, 5.6 TB/s, against 326 with one row in flight).
template <int CPL, int B>
__global__ __launch_bounds__(kChunkThreads) void chunk_scan_kernel(
    const uint16_t* __restrict__ E, int64_t n, int dim, const int64_t* __restrict__ off,
    int64_t n_papers, float thr, int rpw, float* __restrict__ cos_out,
    int32_t* __restrict__ cnt) {
  __shared__ int32_t wave_cnt[kChunkWaves];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int64_t t0 = ((int64_t)blockIdx.x * kChunkWaves + wave) * rpw;
  const int64_t t1 = t0 + rpw < n ? t0 + rpw : n;
  int32_t boundaries = 0;
  if (t0 < t1) {  // uniform per wave
    u32x4 prev[CPL], cur[B][CPL], nxt[B][CPL];
    auto load_batch = [&](u32x4 (&v)[B][CPL], int64_t t) {  // rows past the range: left as they are
#pragma unroll
      for (int u = 0; u < B; ++u)
        if (t + u < t1) load_row<CPL>(E, t + u, dim, lane, v[u]);
    };
    // the first rows go out before the paper search; the row before the range may be unused
    load_row<CPL>(E, t0 > 0 ? t0 - 1 : 0, dim, lane, prev);
#pragma unroll
    for (int u = 0; u < B; ++u)
#pragma unroll
      for (int i = 0; i < CPL; ++i) cur[u][i] = nxt[u][i] = u32x4{0u, 0u, 0u, 0u};
    load_batch(cur, t0);
    // paper starts: is t0 one, and the next start after t0 (uniform, scalar)
    bool t0_start;
    int64_t dnext = 0;
    if (off) {
      dnext = next_start_index(off, n_papers, t0, lane);
      t0_start = dnext > 0 && off[dnext - 1] == t0;  // off[dnext-1] <= t0 < off[dnext]
    } else {
      t0_start = t0 == 0;
    }
    int64_t next_start = off ? (dnext <= n_papers ? off[dnext] : n) : n;
    float pn = wave_sum_dpp(row_dot<CPL>(prev, prev));  // |prev|^2
    for (int64_t t = t0; t < t1; t += B) {
      if (t + B < t1) load_batch(nxt, t + B);  // in flight during this batch
      float cn[B], dt[B];
#pragma unroll
      for (int u = 0; u < B; ++u) {
        cn[u] = row_dot<CPL>(cur[u], cur[u]);
        dt[u] = row_dot<CPL>(u == 0 ? prev : cur[u - 1], cur[u]);
      }
#pragma unroll
      for (int u = 0; u < B; ++u) {
        cn[u] = wave_sum_dpp(cn[u]);
        dt[u] = wave_sum_dpp(dt[u]);
      }
      float mine = 0.f;  // lane u: the cosine of row t + u
#pragma unroll
      for (int u = 0; u < B; ++u) {
        const int64_t r = t + u;
        if (r < t1) {
          const bool first = r == t0 ? t0_start : r == next_start;
          if (off && r == next_start) {  // advance past every paper starting at r
            while (dnext <= n_papers && off[dnext] <= r) ++dnext;
            next_start = dnext <= n_papers ? off[dnext] : n;
          }
          const float c = first ? __builtin_nanf("") : dt[u] / sqrtf(pn * cn[u]);
          mine = lane == u ? c : mine;
          boundaries += (c > thr) ? 0 : 1;
          pn = cn[u];
        }
      }
      if (lane < B && t + lane < t1) cos_out[t + lane] = mine;
#pragma unroll
      for (int i = 0; i < CPL; ++i) prev[i] = cur[B - 1][i];
#pragma unroll
      for (int u = 0; u < B; ++u)
#pragma unroll
        for (int i = 0; i < CPL; ++i) cur[u][i] = nxt[u][i];
    }
  }
  if (lane == 0) wave_cnt[wave] = boundaries;
  __syncthreads();
  if (threadIdx.x == 0) {
    int32_t s = 0;
#pragma unroll
    for (int w = 0; w < kChunkWaves; ++w) s += wave_cnt[w];
    cnt[blockIdx.x] = s;
  }
}

constexpr int kScanThreads = 1024;

constexpr int64_t kDirectGroups = 4096;  // up to here the ids kernel sums the counts itself

// Exclusive scan of cnt[0 .. n_ranges) into base[]: each thread sums a contiguous slice, a block
// scan orders the slices, then each thread writes its slice.
__global__ __launch_bounds__(kScanThreads) void chunk_offsets_kernel(const int32_t* __restrict__ cnt,
                                                                     int64_t n_ranges,
                                                                     int64_t* __restrict__ base) {
  __shared__ int64_t part[kScanThreads];
  const int tid = threadIdx.x;
  const int64_t per = (n_ranges + kScanThreads - 1) / kScanThreads;
  const int64_t a = tid * per, b = a + per < n_ranges ? a + per : n_ranges;
  int64_t s = 0;
  for (int64_t i = a; i < b; ++i) s += cnt[i];
  part[tid] = s;
  __syncthreads();
  for (int o = 1; o < kScanThreads; o <<= 1) {  // inclusive Hillis-Steele scan
    const int64_t v = tid >= o ? part[tid - o] : 0;
    __syncthreads();
    part[tid] += v;
    __syncthreads();
  }
  int64_t run = tid > 0 ? part[tid - 1] : 0;
  for (int64_t i = a; i < b; ++i) {
    base[i] = run;
    run += cnt[i];
  }
}

constexpr int kIdRows = 1024;  // sentences per workgroup of chunk_ids_kernel (a multiple of 4 rpw)

// Segment ids of rows [kIdRows b, kIdRows (b + 1)).  The boundaries before the workgroup's first
// row come from base[] (its first group) or, when base is null, from summing the counts of the
// groups before it: at most kDirectGroups of them, a few coalesced loads per thread from L2, which
// costs less than the launch that would scan them.
__global__ __launch_bounds__(kChunkThreads) void chunk_ids_kernel(
    const float* __restrict__ cos_in, int64_t n, float thr, int group_rows,
    const int32_t* __restrict__ cnt, const int64_t* __restrict__ base, int32_t* __restrict__ seg,
    int64_t* __restrict__ n_seg) {
  __shared__ int64_t before[kChunkWaves];
  __shared__ int32_t own[kChunkWaves];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  constexpr int kPer = kIdRows / kChunkThreads;  // 64-row steps per wave
  const int64_t t0 = (int64_t)blockIdx.x * kIdRows + wave * (kPer * 64);
  uint64_t m[kPer];
  int32_t mine = 0;
#pragma unroll
  for (int j = 0; j < kPer; ++j) {
    const int64_t i = t0 + 64 * j + lane;
    m[j] = __ballot(i < n && !(cos_in[i < n ? i : n - 1] > thr));
    mine += __popcll(m[j]);
  }
  const int64_t g0 = (int64_t)blockIdx.x * (kIdRows / group_rows);
  int64_t s = 0;
  if (base) {
    s = tid == 0 ? base[g0] : 0;
  } else {
    for (int64_t g = tid; g < g0; g += kChunkThreads) s += cnt[g];
  }
  for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o);
  if (lane == 0) {
    before[wave] = s;
    own[wave] = mine;
  }
  __syncthreads();
  int64_t run = 0;
#pragma unroll
  for (int w = 0; w < kChunkWaves; ++w) run += before[w] + (w < wave ? own[w] : 0);
  const uint64_t le_mask = lane == 63 ? ~0ull : ((2ull << lane) - 1ull);
#pragma unroll
  for (int j = 0; j < kPer; ++j) {
    const int64_t i = t0 + 64 * j + lane;
    if (i < n) seg[i] = (int32_t)(run + __popcll(m[j] & le_mask) - 1);
    run += __popcll(m[j]);
  }
  if (blockIdx.x == gridDim.x - 1 && tid == kChunkThreads - 1) *n_seg = run;
}

constexpr int kMetricThreads = 1024;

__global__ __launch_bounds__(kMetricThreads) void metrics_kernel(
    const int64_t* __restrict__ idx, int nq, int64_t ld, int k, const int64_t* __restrict__ pos,
    int32_t* __restrict__ ranks, double* __restrict__ out) {
  __shared__ double sh_hit[kMetricThreads], sh_rr[kMetricThreads];
  const int tid = threadIdx.x;
  double hit = 0.0, rr = 0.0;
  for (int q = tid; q < nq; q += kMetricThreads) {  // fixed order per thread
    const int64_t p = pos[q];
    int r = 0;
    for (int j = 0; j < k; ++j)
      if (idx[(int64_t)q * ld + j] == p) {
        r = j + 1;
        break;
      }
    if (ranks) ranks[q] = r;
    if (r > 0) {
      hit += 1.0;
      rr += 1.0 / (double)r;
    }
  }
  sh_hit[tid] = hit;
  sh_rr[tid] = rr;
  __syncthreads();
  for (int o = kMetricThreads / 2; o > 0; o >>= 1) {  // fixed pairwise tree
    if (tid < o) {
      sh_hit[tid] += sh_hit[tid + o];
      sh_rr[tid] += sh_rr[tid + o];
    }
    __syncthreads();
  }
  if (tid == 0) {
    out[0] = sh_hit[0] / (double)k / (double)nq;
    out[1] = sh_rr[0] / (double)nq;
  }
}

}  // namespace

// Sentences per wave.  Short inputs take few rows per wave, so that the chip is full and no wave
// walks a long chain of rows alone: one paper of 200 sentences of dim 4096 takes 17.5 us a call
// (mostly the host's) against 154 with 128 rows per wave.  Long ones take enough rows that the
// re-read row before each range costs little: 400,000 x 4096 takes 637, 566, 564, 536 and 558 us
// with 4, 8, 16, 32 and 64 rows (655 with 128, whose 3,125 waves fill the chip 1.02 times), and
// 2,010,113 x 4096 takes 2.50 ms with 32 and 2.47 with 64 (2.54 with 128).  The rule goes by the
// sentences alone; over dims 64, 384, 768, 1024 and 4096 it is within 3 % of the best power of two
// at 100,000 (dim 4096: 151 us, 135 with 64 rows), 400,000 and 2,000,000 sentences, and up to 5 us
// off it between 12,000 and 30,000, where 8 or 16 rows are best: 12,288 x 768 16.7 us with 1 row,
// 13.6 with 8; 30,000 x 768 19.0 with 4, 15.8 with 16; 12,288 x 4096 29.5 with 1, 23.8 with 4.
int chunk_rows_per_wave(int64_t n) {
  int r = 1;
  while (r < 32 && n > (int64_t)r * 12288) r *= 2;
  if (n > (int64_t)1 << 20) r = 64;
  return n < ((int64_t)1 << 28) ? r : 128;  // (a grid holds fewer than 2^32 threads)
}

int64_t chunk_groups(int64_t n) {
  const int64_t g = (int64_t)kChunkWaves * chunk_rows_per_wave(n);
  return (n + g - 1) / g;
}

// Past the end of each step of chunk_rows_per_wave there are fewer groups than at it: the largest of
// the steps' ends below n, so that the workspace of a longer input holds every shorter one's.
int64_t chunk_groups_most(int64_t n) {
  const int64_t per128 = (n + 127) / 128, g = chunk_groups(n);
  int64_t most = g > per128 ? g : per128;
  auto step = [&](int64_t end) {
    const int64_t e = n > end ? chunk_groups(end) : 0;
    most = e > most ? e : most;
  };
  for (int64_t r = 1; r < 32; r *= 2) step(r * 12288);
  step((int64_t)1 << 20);
  step(((int64_t)1 << 28) - 1);
  return most;
}

hipError_t launch_semantic_chunk(const uint16_t* E, int64_t n, int dim, const int64_t* off,
                                 int64_t n_papers, float thr, float* cos_out, int32_t* cnt,
                                 int64_t* base, int32_t* seg, int64_t* n_seg,
                                 hipStream_t stream) {
  const int rpw = chunk_rows_per_wave(n);
  const int64_t groups = chunk_groups(n);
  const dim3 grid((unsigned)groups), block(kChunkThreads);
  if (dim <= 512)
    hipLaunchKernelGGL((chunk_scan_kernel<1, 8>), grid, block, 0, stream, E, n, dim, off, n_papers,
                       thr, rpw, cos_out, cnt);
  else if (dim <= 1024)
    hipLaunchKernelGGL((chunk_scan_kernel<2, 4>), grid, block, 0, stream, E, n, dim, off, n_papers,
                       thr, rpw, cos_out, cnt);
  else if (dim <= 2048)
    hipLaunchKernelGGL((chunk_scan_kernel<4, 2>), grid, block, 0, stream, E, n, dim, off, n_papers,
                       thr, rpw, cos_out, cnt);
  else
    hipLaunchKernelGGL((chunk_scan_kernel<8, 1>), grid, block, 0, stream, E, n, dim, off, n_papers,
                       thr, rpw, cos_out, cnt);
  const bool direct = groups <= kDirectGroups;
  if (!direct)
    hipLaunchKernelGGL(chunk_offsets_kernel, dim3(1), dim3(kScanThreads), 0, stream, cnt, groups,
                       base);
  hipLaunchKernelGGL(chunk_ids_kernel, dim3((unsigned)((n + kIdRows - 1) / kIdRows)), block, 0,
                     stream, cos_out, n, thr, kChunkWaves * rpw, cnt, direct ? nullptr : base, seg,
                     n_seg);
  return hipGetLastError();
}

hipError_t launch_retrieval_metrics(const int64_t* idx, int nq, int64_t ld, int k,
                                    const int64_t* pos, int32_t* ranks, double* out,
                                    hipStream_t stream) {
  hipLaunchKernelGGL(metrics_kernel, dim3(1), dim3(kMetricThreads), 0, stream, idx, nq, ld, k,
                     pos, ranks, out);
  return hipGetLastError();
}

}  // namespace hpr
