// Device-side pieces shared by the two MaxSim kernels (maxsim.hip: scores only;
// maxsim_argmax.hip: scores and the argmax for the loss): the launch arguments, the document
// cursor and stage descriptor of the LDS tile stream, cross-lane sums, and the packed argmax
// keys.
#pragma once

#include "common.h"
#include "kernels.h"

namespace hpr {
namespace msim {

typedef __attribute__((ext_vector_type(16))) float f32x16;

struct MaxsimArgs {
  const uint16_t* q;
  const uint16_t* d;
  const int64_t* off;
  const int64_t* part;  // range table of the score kernel; null: the workgroups find their own
  float* scores;
  uint16_t* amax;
  int32_t* ctrl;        // argmax kernel: control words of the call, zeroed by workgroup 0
  int64_t n_docs, n_tok;
  int nq, lq, lqp, qpw, dim, n_qgroups, n_ranges, n_ctrl;
  int persist;          // score kernel: persistent grid (see maxsim_kernel) ...
  int qg_base;          // ... and the first query group of the launch
  int by_count;         // own ranges hold equal numbers of documents (see own_range)
};

// Position of tile `t` of the current document stream; uniform across the workgroup.  Token
// and document indices fit 32 bits (the host rejects stores of 2^31 tokens or more).
struct TileCursor {
  int d;      // document
  int base;   // first token row (clamped)
  int len;    // tokens (>= 1)
  int t;      // tile index within the document
  int cnt;    // tiles of the document
};

// Which tiles a stage holds, in scalar registers: the stage starts at tile t0 of document d0;
// bit j of `valid` / `last` / `lng` says that tile j exists / ends its document / belongs to a
// document of more than 65536 tokens.
struct StageDesc {
  int d0;
  int t0;
  uint32_t valid, last, lng;
};

// First document of token range r out of R equal ranges: the least d in [0, n_docs) with
// off[d] >= floor(n_tok * r / R), or n_docs when there is none or r = R (documents are never
// split; a range can be empty).  Lanes 0-31 answer for r = r0 and lanes 32-63 for r0 + 1, each
// half by a 32-way search that keeps the answer inside [lo, hi]: a round probes the last offset
// of each of 32 equal slices of [lo, hi); the probes below the target form a prefix (offsets
// ascend), and its length picks the slice that holds the answer.  A span S shrinks to at most
// ceil(S / 32) - 1 per round: two rounds for 1024 documents, four for 10^6.  Whatever the
// offsets hold, lo stays within [0, n_docs] and every probe within [0, n_docs).
__device__ __forceinline__ int range_first_doc(const int64_t* __restrict__ off, int64_t n_docs, int64_t n_tok,
                               int R, int r0, int lane) {
  const int half = lane >> 5, i = lane & 31;
  // floor(n_tok * r / R) in 32 bits: n_tok < 2^31 and R <= 2^16, so (n_tok % R) * r < 2^32
  const uint32_t nt = (uint32_t)n_tok, ru = (uint32_t)R, qt = nt / ru, mt = nt % ru;
  const uint32_t r = (uint32_t)r0 + (uint32_t)half;
  const uint32_t t0 = qt * (uint32_t)r0 + mt * (uint32_t)r0 / ru;
  const uint32_t t1 = qt * (uint32_t)(r0 + 1) + mt * (uint32_t)(r0 + 1) / ru;
  const int64_t target = half ? t1 : t0;
  int64_t lo = r >= ru ? n_docs : 0, hi = n_docs;
  while (__ballot(lo < hi)) {
    const bool open = lo < hi;
    const int64_t step = (hi - lo + 31) >> 5;
    const int64_t last = hi - 1;
    int64_t p = lo + (int64_t)(i + 1) * step - 1;
    p = p < last ? p : last;
    const bool below = open && off[p] < target;
    const int c = __popc((uint32_t)(__ballot(below) >> (32 * half)));
    if (open) {
      const int64_t pl = lo + (int64_t)c * step - 1, ph = pl + step;
      const int64_t nlo = c > 0 ? (pl < last ? pl : last) + 1 : lo;
      hi = c < 32 ? (ph < last ? ph : last) : hi;
      lo = nlo;
    }
  }
  return (int)lo;
}

// The documents [first, last) of range r, found by the workgroup itself.  By count (plan.by_count:
// fewer than two documents a range): no balance of tokens is to be had from whole documents, and
// equal numbers of them need no search.  Otherwise by tokens.
struct DocRange {
  int first, last;
};
__device__ __forceinline__ DocRange own_range(const MaxsimArgs& a, const int64_t* __restrict__ off,
                                              int r, int lane) {
  if (a.by_count) {
    const uint32_t n = (uint32_t)a.n_docs, R = (uint32_t)a.n_ranges;  // n < 2 R <= 2^17
    return {(int)(n / R * r + n % R * r / R), (int)(n / R * (r + 1) + n % R * (r + 1) / R)};
  }
  const int first = range_first_doc(off, a.n_docs, a.n_tok, a.n_ranges, r, lane);
  return {__builtin_amdgcn_readlane(first, 0), __builtin_amdgcn_readlane(first, 32)};
}

// Argmax keys ("tile keys") of one 32x32 tile column: the lane's 16 values v_r (r = 0..15,
// rows ascending with r) as order-preserving integers o(v) (o(v) = bits of v for v >= 0,
// bits ^ 0x7fffffff below zero: increasing in v) with the low 4 bits replaced by 15 - r.  The
// signed maximum of the keys is then the largest o(v) & ~15 held by the lowest row, in one
// v_bitop3 per value ((bits & ~15) | (15 - r), truth table 0xea: a & b | c) plus one three-way
// max per two values (a compare-and-select search of the 16 rows costs about twice as many
// instructions).  The row selected is the first one whose value equals the maximum up to its 4
// lowest mantissa bits (a relative window below 2^-19); the score itself takes the exact
// maximum.  For v >= 0, o(v) = bits(v): a lane whose tile holds a non-negative value needs
// nothing else; a lane whose 16 values are all negative (its key is then negative) redoes the
// keys with the sign-flipped encoding, key ^ 0x7ffffff0.
__device__ __forceinline__ int max3_i(int a, int b, int c) { return max(max(a, b), c); }

// Cross-lane moves within a row of 16 lanes through DPP (no LDS round trip).
template <int CTRL>
__device__ __forceinline__ float dpp_f(float v) {
  return __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, v), CTRL,
                                                            0xf, 0xf, false));
}
constexpr int kDppQuadXor1 = 0xb1;    // quad_perm [1, 0, 3, 2]
constexpr int kDppQuadXor2 = 0x4e;    // quad_perm [2, 3, 0, 1]
constexpr int kDppRowHalfMirror = 0x141;
constexpr int kDppRowMirror = 0x140;

// Sum over the 32 lanes l, l ^ 1, ..., of each half-wave in a fixed order; every lane of the
// half gets the total.  The last step adds the two 16-lane rows of each half through
// v_permlane16_swap (no LDS round trip): with both operands v, element 0 holds the even row of
// each pair in both rows and element 1 the odd row, so their sum is the pair's total in every
// lane, the same bits whichever row a lane is in (addition being commutative).
__device__ __forceinline__ float half32_sum(float v) {
  v += dpp_f<kDppQuadXor1>(v);
  v += dpp_f<kDppQuadXor2>(v);
  v += dpp_f<kDppRowHalfMirror>(v);  // quad q with quad 1 - q of the same half row
  v += dpp_f<kDppRowMirror>(v);      // the two half rows: the 16-lane row total
  const auto sw = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false,
                                                   false);
  return __uint_as_float(sw[0]) + __uint_as_float(sw[1]);  // the two rows of the half-wave
}

// Document end of packed queries: the slot maxima m (block b's in lane col of both halves; `slots`
// is the wave's own LDS row of 32 NB floats) summed per query, each half-wave taking every other
// one.  A query's slots are read back in the lanes that whole blocks would hold them in, so its sum
// has the same bits as when it has blocks of its own.  put(ql, sum) is called in one lane of each.
template <int NB, class Put>
__device__ __forceinline__ void packed_sums(const MaxsimArgs& a, const float (&m)[NB], float* slots,
                                            int lane, Put put) {
  const int col = lane & 31, half = lane >> 5;
#pragma unroll
  for (int b = 0; b < NB; ++b)
    if (half == (b & 1)) slots[b * 32 + col] = m[b];
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");  // (a wave's LDS accesses are in order)
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll 1
  for (int q = 0; q < a.qpw; q += 2) {
    const int ql = q + half;
    float qs = 0.f;
    for (int i0 = 0; i0 < a.lq; i0 += 32) {
      const int i = i0 + col;
      qs += half32_sum(ql < a.qpw && i < a.lq ? slots[ql * a.lqp + i] : 0.f);
    }
    if (col == 0 && ql < a.qpw) put(ql, qs);
  }
  __builtin_amdgcn_wave_barrier();  // the row is rewritten by the next document
}

// Workgroups of maxsim_argmax_kernel per CU: two by registers (its launch bounds), fewer when
// two stages and the result ring do not fit the CU's 160 KiB of LDS twice.
constexpr int argmax_tps(int ks) { return ks >= 8 ? 2 : ks >= 4 ? 4 : 8; }
constexpr int argmax_resident(int ks) {
  const int tile = 32 * (ks * 32 + 16);
  const int tps = argmax_tps(ks);
  const int nb = ks == 16 ? 1 : 2;
  const int res = 3 * tps * (4 * nb * 2 * 4 + 4 * nb * 32 * 2) + 4 * nb * 32 * 4;  // packed
  const int by_lds = (160 * 1024) / (2 * tps * tile + res);
  return by_lds < 2 ? by_lds : 2;
}

// Launches the argmax kernel variant for plan.ks (maxsim_argmax.hip).
hipError_t launch_argmax_variant(const MaxsimPlan& plan, const MaxsimArgs& args,
                                 hipStream_t stream);

}  // namespace msim
}  // namespace hpr
