// Device code shared by the selection kernels: the order-preserving keys, the aggregation of a row's
// scores, block-wide scans and digit searches, and the plain several-pass ranking of a row.
// Internal; included by the selection's translation units only.
#pragma once

#include "common.h"

namespace {


__device__ __forceinline__ uint32_t key_of_bits(uint32_t u) {
  if (u == 0x80000000u) u = 0u;                       // -0 == +0
  // ascending with the float order: negative values have all bits flipped, the others the sign bit set
  return u ^ ((uint32_t)((int32_t)u >> 31) | 0x80000000u);
}
__device__ __forceinline__ uint32_t key_of(float x) { return key_of_bits(__builtin_bit_cast(uint32_t, x)); }

// exp(s - lse) through the hardware base-2 exponential (about 1 ulp; the product with log2(e)
// adds a relative error below 1e-6 for |s - lse| < 40, far inside the stage-wise tolerance)
__device__ __forceinline__ float prob_of(float s, float lse) {
  return __builtin_amdgcn_exp2f((s - lse) * 1.44269504088896340736f);
}

__device__ __forceinline__ int row_len(const SelectArgs &A, int bt) {
  int nb = A.seq_lens ? A.seq_lens[bt] : A.N;
  return min(max(nb, 0), A.N);
}

// What a workgroup needs of the tables in the kernel's arguments is read by scalar loads: the row's batch element and draft head
// are told to be uniform (a division's result is not seen to be), and the 16- and 8-bit entries are taken out of words (there are
// no narrower scalar loads). As vector loads they were two or three memory latencies in a row before a row's first score, and one
// before its list: 16 rows of 16384 tokens, one score each, 12.5 -> 11.4 us, 256 rows 14.1 -> 12.8.
__device__ __forceinline__ void row_of(const SelectArgs &A, int row, int &bt, int &j) {
  bt = __builtin_amdgcn_readfirstlane(row / A.Hd);
  j = __builtin_amdgcn_readfirstlane(row % A.Hd);
}
typedef uint32_t table_word __attribute__((may_alias));
__device__ __forceinline__ int target_off(const SelectArgs &A, int j) {
  return (int)(reinterpret_cast<const table_word *>(A.targets.off)[j >> 1] >> (16 * (j & 1)) & 0xffffu);
}
__device__ __forceinline__ int target_head(const SelectArgs &A, int ti) {
  return (int)(reinterpret_cast<const table_word *>(A.targets.tgt)[ti >> 2] >> (8 * (ti & 3)) & 0xffu);
}

// c of nb tokens kept, out of ns sampled ones: where the threshold is expected among them (an estimate: fp32 does, a 64-bit
// division is two hundred instructions in front of everything else; with it, the divisions by the sampling step and the permutes of
// minima and sums gone 16 rows of 33001 tokens, five scores each, take 25.8 us instead of 27.4, 64 rows of 131072 48.0 instead of 50.4)
__device__ __forceinline__ uint32_t expected_rank(uint32_t c, uint32_t ns, int nb) {
  return max(1u, min(ns, (uint32_t)((float)c * ((float)ns / (float)nb))));
}

// number of ranked units (tokens, or blocks of `page` tokens) in the row of batch bt
__device__ __forceinline__ int src_len(const SelectArgs &A, int bt) {
  return (row_len(A, bt) + A.page - 1) / A.page;
}

// Inclusive prefix sum over the 64 lanes of a wave with data-parallel-primitive moves (no LDS
// round trips): shifts by 1, 2, 4, 8 inside each row of 16 lanes (a lane whose source lies
// outside its row adds 0), then lane 15 of row 0 / 2 is added to row 1 / 3, then lane 31 to
// rows 2 and 3.
__device__ __forceinline__ uint32_t wave_incl_scan(uint32_t v) {
  int x = (int)v;
  x += __builtin_amdgcn_update_dpp(0, x, 0x111, 0xf, 0xf, false);   // row_shr:1
  x += __builtin_amdgcn_update_dpp(0, x, 0x112, 0xf, 0xf, false);   // row_shr:2
  x += __builtin_amdgcn_update_dpp(0, x, 0x114, 0xf, 0xf, false);   // row_shr:4
  x += __builtin_amdgcn_update_dpp(0, x, 0x118, 0xf, 0xf, false);   // row_shr:8
  x += __builtin_amdgcn_update_dpp(0, x, 0x142, 0xa, 0xf, false);   // row_bcast:15 into rows 1 and 3
  x += __builtin_amdgcn_update_dpp(0, x, 0x143, 0xc, 0xf, false);   // row_bcast:31 into rows 2 and 3
  return (uint32_t)x;
}

// signed image of a score's order: positive scores are their own bit pattern
__device__ __forceinline__ int ordered(int v) {
  v = v == (int)0x80000000 ? 0 : v;                    // -0 == +0
  return v ^ ((v >> 31) & 0x7fffffff);
}
__device__ __forceinline__ uint32_t key_of_ordered(int s) { return (uint32_t)s ^ 0x80000000u; }
__device__ __forceinline__ int ordered_of_key(uint32_t k) { return (int)(k ^ 0x80000000u); }

__device__ __forceinline__ uint64_t ballot64(bool p) { return __builtin_amdgcn_ballot_w64(p); }
__device__ __forceinline__ uint32_t lanes_before(uint64_t mask, uint32_t base) {
  return __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, base));
}
// lowest and highest over the wave, the same way as the sums (a lane without a source keeps its own value): seven register moves in a
// row instead of six LDS permutes
__device__ __forceinline__ void wave_min_max(uint32_t &lo, uint32_t &hi) {
  auto step = [&](auto ctrl, auto rows) {
    lo = min(lo, (uint32_t)__builtin_amdgcn_update_dpp((int)lo, (int)lo, decltype(ctrl)::value, decltype(rows)::value, 0xf, false));
    hi = max(hi, (uint32_t)__builtin_amdgcn_update_dpp((int)hi, (int)hi, decltype(ctrl)::value, decltype(rows)::value, 0xf, false));
  };
  std::integral_constant<int, 0xf> all;
  step(std::integral_constant<int, 0x111>{}, all);
  step(std::integral_constant<int, 0x112>{}, all);
  step(std::integral_constant<int, 0x114>{}, all);
  step(std::integral_constant<int, 0x118>{}, all);
  step(std::integral_constant<int, 0x142>{}, std::integral_constant<int, 0xa>{});
  step(std::integral_constant<int, 0x143>{}, std::integral_constant<int, 0xc>{});
  lo = (uint32_t)__builtin_amdgcn_readlane((int)lo, 63);
  hi = (uint32_t)__builtin_amdgcn_readlane((int)hi, 63);
}
__device__ __forceinline__ uint32_t wave_sum(uint32_t v) { return (uint32_t)__builtin_amdgcn_readlane((int)wave_incl_scan(v), 63); }

// exclusive prefix sum of one value per thread over a THREADS-thread block; also returns the
// total. lds_wave_tot needs THREADS/64 words. SCALAR: the wave's number in a scalar register, which the kernels that
// hold a row in registers need (28 bytes of scratch per lane less); the pool kernels are 5% slower with it (16 rows of
// 1M tokens, 256 kept: 94.1 against 89.8 us).
template <int THREADS = SEL_THREADS, bool SCALAR = false>
__device__ __forceinline__ uint32_t block_excl_scan(uint32_t v, uint32_t *lds_wave_tot, uint32_t &total) {
  const int lane = threadIdx.x & 63, wave = SCALAR ? __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6) : (int)(threadIdx.x >> 6);
  const uint32_t incl = wave_incl_scan(v);
  if (lane == 63) lds_wave_tot[wave] = incl;
  __syncthreads();
  uint32_t base = 0, tot = 0;
#pragma unroll
  for (int w = 0; w < THREADS / 64; ++w) {
    const uint32_t t = lds_wave_tot[w];
    if (w < wave) base += t;
    tot += t;
  }
  __syncthreads();
  total = tot;
  return base + incl - v;
}

// Walk a digit histogram from the top: the digit holding the krem-th largest key of the
// candidates, and how many keys of that digit are still wanted. Requires 1 <= krem <= total.
// lds_tmp needs THREADS/64 + 2 words; the result lands in its last two.
template <int NBINS, int THREADS = SEL_THREADS, bool SCALAR = false>
__device__ __forceinline__ void find_digit(const uint32_t *hist, uint32_t krem, uint32_t *lds_tmp,
                                           uint32_t &digit, uint32_t &krem_next) {
  constexpr int PER = NBINS / THREADS;
  constexpr int RES = THREADS / 64;
  uint32_t loc[PER], sum = 0;
#pragma unroll
  for (int i = 0; i < PER; ++i) {
    loc[i] = hist[threadIdx.x * PER + i];
    sum += loc[i];
  }
  uint32_t total;
  const uint32_t excl = block_excl_scan<THREADS, SCALAR>(sum, lds_tmp, total);
  uint32_t above = total - excl - sum;   // keys in bins owned by higher threads
#pragma unroll
  for (int i = PER - 1; i >= 0; --i) {
    if (above < krem && above + loc[i] >= krem) {
      lds_tmp[RES] = threadIdx.x * PER + i;
      lds_tmp[RES + 1] = krem - above;
    }
    above += loc[i];
  }
  __syncthreads();
  digit = lds_tmp[RES];
  krem_next = lds_tmp[RES + 1];
  __syncthreads();
}

// ------------------------------------------------------------------- aggregation of a row
// The Tq score rows of one (batch, draft head), reduced per token strictly in row order.
struct AggRow {
  const void *P;    // [Tq][N] fp32, or bf16 bit patterns
  const float *L;   // [Tq] natural-log normalisers (scaled-logit input) or nullptr
  int Tq, N;
  bool bf16, logits, use_max;
};

__device__ __forceinline__ AggRow agg_row(const SelectArgs &A, int row) {
  AggRow R;
  const size_t off = (size_t)row * A.Tq * A.N;
  R.bf16 = A.scores_bf16 != 0;
  R.P = R.bf16 ? static_cast<const void *>(static_cast<const uint16_t *>(A.scores) + off)
               : static_cast<const void *>(static_cast<const float *>(A.scores) + off);
  R.L = A.lse ? A.lse + (size_t)row * A.Tq : nullptr;
  R.Tq = A.Tq;
  R.N = A.N;
  R.logits = A.kind == STS_SCORES_LOGITS_LSE;
  R.use_max = A.reduce == STS_REDUCE_MAX;
  return R;
}

// One score (V = float) or four consecutive ones (V = f32x4) of row i, as stored: the raw load, and
// its exact widening to fp32. Nontemporal: every score is read exactly once. Four scores need no
// more than their element's alignment (rows of N % 4 != 0 scores start anywhere): the vector types
// below say so, and this chip's global loads of 8 and 16 bytes take any address.
typedef f32x4 f32x4_any __attribute__((aligned(4)));
typedef u32x2 u32x2_any __attribute__((aligned(2)));
template <class V, bool BF16>
struct ScoreLoad;
template <>
struct ScoreLoad<float, false> {
  typedef float raw;
  static __device__ __forceinline__ raw load(const AggRow &R, int i, int n) {
    return __builtin_nontemporal_load(static_cast<const float *>(R.P) + (size_t)i * R.N + n);
  }
  static __device__ __forceinline__ float widen(raw x) { return x; }
};
template <>
struct ScoreLoad<f32x4, false> {
  typedef f32x4 raw;
  static __device__ __forceinline__ raw load(const AggRow &R, int i, int n) {
    return __builtin_nontemporal_load(reinterpret_cast<const f32x4_any *>(static_cast<const float *>(R.P) + (size_t)i * R.N + n));
  }
  static __device__ __forceinline__ raw load_at(const unsigned char *p) { return __builtin_nontemporal_load(reinterpret_cast<const f32x4_any *>(p)); }
  static __device__ __forceinline__ f32x4 widen(raw x) { return x; }
};
template <>
struct ScoreLoad<float, true> {
  typedef uint16_t raw;
  static __device__ __forceinline__ raw load(const AggRow &R, int i, int n) {
    return __builtin_nontemporal_load(static_cast<const uint16_t *>(R.P) + (size_t)i * R.N + n);
  }
  static __device__ __forceinline__ float widen(raw x) { return __builtin_bit_cast(float, (uint32_t)x << 16); }
};
template <>
struct ScoreLoad<f32x4, true> {
  typedef u32x2 raw;   // four bf16 values
  static __device__ __forceinline__ raw load(const AggRow &R, int i, int n) {
    return __builtin_nontemporal_load(reinterpret_cast<const u32x2_any *>(static_cast<const uint16_t *>(R.P) + (size_t)i * R.N + n));
  }
  static __device__ __forceinline__ raw load_at(const unsigned char *p) { return __builtin_nontemporal_load(reinterpret_cast<const u32x2_any *>(p)); }
  static __device__ __forceinline__ f32x4 widen(raw x) {
    return f32x4{__builtin_bit_cast(float, x[0] << 16), __builtin_bit_cast(float, x[0] & 0xffff0000u),
                 __builtin_bit_cast(float, x[1] << 16), __builtin_bit_cast(float, x[1] & 0xffff0000u)};
  }
};

// NROWS consecutive score rows, from row i on, of the token(s) at each of the NPOS positions n[]:
// all loads first (their latencies overlap), then the reduction strictly in row order. FIRST: row
// i is row 0 and initialises the accumulators.
template <int NROWS, bool FIRST, bool BF16, int NPOS, class V>
__device__ __forceinline__ void agg_rows(const AggRow &R, int i, const int (&n)[NPOS], V (&acc)[NPOS]) {
  typedef ScoreLoad<V, BF16> SL;
  typename SL::raw raw[NPOS][NROWS];
#pragma unroll
  for (int x = 0; x < NPOS; ++x)
#pragma unroll
    for (int u = 0; u < NROWS; ++u) raw[x][u] = SL::load(R, i + u, n[x]);
#pragma unroll
  for (int x = 0; x < NPOS; ++x)
#pragma unroll
    for (int u = 0; u < NROWS; ++u) {
      V p = SL::widen(raw[x][u]);
      if (R.logits) {
        const float l = R.L[i + u];
        if constexpr (sizeof(V) == sizeof(float)) {
          p = prob_of(p, l);
        } else {
#pragma unroll
          for (int e = 0; e < 4; ++e) p[e] = prob_of(p[e], l);
        }
      }
      if (FIRST && u == 0) {
        acc[x] = p;
      } else if (R.use_max) {
        if constexpr (sizeof(V) == sizeof(float)) {
          acc[x] = fmaxf(acc[x], p);
        } else {
#pragma unroll
          for (int e = 0; e < 4; ++e) acc[x][e] = fmaxf(acc[x][e], p[e]);
        }
      } else {
        acc[x] = acc[x] + p;
      }
    }
}

template <bool FIRST, bool BF16, int NPOS, class V>
__device__ __forceinline__ void agg_group(const AggRow &R, int i, int rows, const int (&n)[NPOS], V (&acc)[NPOS]) {
  switch (rows) {   // uniform: a scalar branch; every case is straight-line code
    case 1: agg_rows<1, FIRST, BF16>(R, i, n, acc); break;
    case 2: agg_rows<2, FIRST, BF16>(R, i, n, acc); break;
    case 3: agg_rows<3, FIRST, BF16>(R, i, n, acc); break;
    case 4: agg_rows<4, FIRST, BF16>(R, i, n, acc); break;
    case 5: agg_rows<5, FIRST, BF16>(R, i, n, acc); break;
    case 6: agg_rows<6, FIRST, BF16>(R, i, n, acc); break;
    case 7: agg_rows<7, FIRST, BF16>(R, i, n, acc); break;
    default: agg_rows<8, FIRST, BF16>(R, i, n, acc); break;
  }
}

// aggregated score(s) at NPOS positions at once: rows in groups of up to 8 loads per position in
// flight
template <class V, int NPOS>
__device__ __forceinline__ void agg_multi(const AggRow &R, const int (&n)[NPOS], V (&acc)[NPOS]) {
  if (R.bf16) {
    agg_group<true, true>(R, 0, min(R.Tq, 8), n, acc);
    for (int i = 8; i < R.Tq; i += 8) agg_group<false, true>(R, i, min(R.Tq - i, 8), n, acc);
  } else {
    agg_group<true, false>(R, 0, min(R.Tq, 8), n, acc);
    for (int i = 8; i < R.Tq; i += 8) agg_group<false, false>(R, i, min(R.Tq - i, 8), n, acc);
  }
}

template <class V>
__device__ __forceinline__ V agg_at(const AggRow &R, int n) {
  const int pos[1] = {n};
  V acc[1];
  agg_multi<V, 1>(R, pos, acc);
  return acc[0];
}

__device__ __forceinline__ f32x4 agg_quad(const AggRow &R, int n) { return agg_at<f32x4>(R, n); }

// a quad that was read d tokens before its place
__device__ __forceinline__ f32x4 shifted_quad(f32x4 y, int d) {
  return f32x4{d == 0 ? y[0] : d == 1 ? y[1] : d == 2 ? y[2] : y[3], d == 0 ? y[1] : d == 1 ? y[2] : y[3], d == 0 ? y[2] : y[3], y[3]};
}

// The quad at n of a row whose length need not be a multiple of 4 (R.N >= 4): a quad that would
// run past the row's end is read where it still fits and shifted; elements past the end (all of a
// quad's that starts there) come out as some score of the row and are the caller's to ignore.
// inside (wave-uniform): every quad of the wave lies inside the row. Up to eight rows are in flight; the rows are
// told apart by scalar branches and not by a copy of the code for every number of rows: the sampled selection, which
// calls this at four places, is 77 KB of instructions and was 400 (the instruction cache holds 64). At 61 KB: 64 rows of
// 128K tokens 51.1 -> 50.2 us and, with the caches flushed, 58.4 -> 57.1, 16 rows of 33001 28.8 -> 27.5 and 38.1 -> 35.7.
template <bool BF16>
__device__ __forceinline__ f32x4 agg_quad_any(const AggRow &R, int n, bool inside) {
  typedef ScoreLoad<f32x4, BF16> SL;
  const int m = min(n, R.N - 4);
  f32x4 acc;
  auto rows = [&](auto logits, auto use_max) {
#pragma unroll 1
    for (int i = 0; i < R.Tq; i += 8) {
      typename SL::raw raw[8];
#pragma unroll
      for (int u = 0; u < 8; ++u)
        if (i + u < R.Tq) raw[u] = SL::load(R, i + u, m);
#pragma unroll
      for (int u = 0; u < 8; ++u)
        if (i + u < R.Tq) {
          f32x4 p = SL::widen(raw[u]);
          if constexpr (decltype(logits)::value) {
            const float l = R.L[i + u];
#pragma unroll
            for (int e = 0; e < 4; ++e) p[e] = prob_of(p[e], l);
          }
          if (u == 0 && i == 0) {
            acc = p;
          } else if constexpr (decltype(use_max)::value) {
#pragma unroll
            for (int e = 0; e < 4; ++e) acc[e] = fmaxf(acc[e], p[e]);
          } else {
            acc = acc + p;
          }
        }
    }
  };
  if (R.logits) {
    if (R.use_max) rows(std::true_type{}, std::true_type{});
    else rows(std::true_type{}, std::false_type{});
  } else {
    if (R.use_max) rows(std::false_type{}, std::true_type{});
    else rows(std::false_type{}, std::false_type{});
  }
  return inside ? acc : shifted_quad(acc, n - m);
}
__device__ __forceinline__ float agg_one(const AggRow &R, int n) { return agg_at<float>(R, n); }

// tail padding (-1 from position c on) and counts for every target head of draft head j
template <int THREADS>
__device__ __forceinline__ void write_tail(const SelectArgs &A, int bt, int j, uint32_t c) {
  for (int ti = target_off(A, j); ti < target_off(A, j + 1); ++ti) {
    const int tgt = target_head(A, ti);
    int32_t *dst = A.indices + ((size_t)bt * A.Hq + tgt) * A.k;
    for (uint32_t p = c + threadIdx.x; p < (uint32_t)A.k; p += THREADS) dst[p] = -1;
    if (A.counts && threadIdx.x == 0) A.counts[(size_t)bt * A.Hq + tgt] = (int32_t)c;
  }
}

// bin of `key` at `level` under the prefix fixed so far, or -1 when the key is no candidate
__device__ __forceinline__ int fused_bin(uint32_t key, int level, uint32_t d0, uint32_t pre01) {
  if (level == 0) return (int)(key >> (32 - SEL_BITS0));
  if (level == 1) return (key >> (SEL_BITS1 + SEL_BITS2)) == d0 ? (int)((key >> SEL_BITS2) & ((1u << SEL_BITS1) - 1)) : -1;
  return (key >> SEL_BITS2) == pre01 ? (int)(key & ((1u << SEL_BITS2) - 1)) : -1;
}

// sum over the block of one value per thread; red needs THREADS / 64 words
template <int THREADS>
__device__ __forceinline__ uint32_t block_sum1(uint32_t a, uint32_t *red) {
  a = wave_sum(a);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = a;
  __syncthreads();
  uint32_t s = 0;
#pragma unroll
  for (int w = 0; w < THREADS / 64; ++w) s += red[w];
  __syncthreads();
  return s;
}

// The plain way for one workgroup to rank a row it cannot hold: a pass over the scores per digit
// level (the Tq rows are aggregated again each time, in the same order, so the keys repeat bit
// for bit), then a pass that compacts in token order. h: SEL_BINS words, tmp: THREADS/64 + 2.
template <bool BF16, int THREADS>
__device__ __forceinline__ void rank_by_passes(const SelectArgs &A, const AggRow &R, int bt, int nb, uint32_t c,
                                               int t0, int t1, uint32_t *h, uint32_t *tmp, int from = 0, int to = 0x7fffffff) {
  const int tid = threadIdx.x;
  const int nq = (nb + 3) >> 2;           // quads that hold ranked tokens
  __syncthreads();                        // the caller's waves have read what they need of h and tmp
  uint32_t d0 = 0, pre01 = 0, krem = c, d2 = 0;
#pragma unroll 1
  for (int level = 0; level < 3; ++level) {
    for (int i = tid; i < SEL_BINS; i += THREADS) h[i] = 0u;
    __syncthreads();
#pragma unroll 1
    for (int q = tid; q < nq; q += THREADS) {
      const f32x4 acc = agg_quad_any<BF16>(R, 4 * q, false);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int bin = fused_bin(key_of(acc[e]), level, d0, pre01);
        if (4 * q + e < nb && bin >= 0) atomicAdd(&h[bin], 1u);
      }
    }
    __syncthreads();
    uint32_t digit, knext;
    find_digit<SEL_BINS, THREADS, true>(h, krem, tmp, digit, knext);
    if (level == 0) d0 = digit;
    else if (level == 1) pre01 = (d0 << SEL_BITS1) | digit;
    else d2 = digit;
    krem = knext;
  }
  const uint32_t r = krem, Tk = (pre01 << SEL_BITS2) | d2;
  // ordered compaction: per step, thread tid owns quad step + tid
  uint32_t gbase = 0, qbase = 0;
#pragma unroll 1
  for (int step = 0; step < nq; step += THREADS) {
    const int qlo = step + tid;
    const f32x4 acc = agg_quad_any<BF16>(R, 4 * min(qlo, nq - 1), false);
    uint32_t gt_mask = 0, eq_mask = 0;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const uint32_t key = key_of(acc[e]);
      const bool in = 4 * qlo + e < nb;
      gt_mask |= (in && key > Tk) ? 1u << e : 0u;
      eq_mask |= (in && key == Tk) ? 1u << e : 0u;
    }
    uint32_t total;
    const uint32_t excl = block_excl_scan<THREADS, true>(__builtin_popcount(gt_mask) | (__builtin_popcount(eq_mask) << 16), tmp, total);
    uint32_t g = gbase + (excl & 0xffffu), q = qbase + (excl >> 16);
    for (uint32_t rest = gt_mask | eq_mask; rest; rest &= rest - 1) {
      const int i = __builtin_ctz(rest);
      const bool is_gt = (gt_mask >> i) & 1u;
      if (is_gt || q < r) {
        const uint32_t p = g + min(q, r);
        const int n = 4 * qlo + i;
        if (p < c && n >= from && n < to)
          for (int ti = t0; ti < t1; ++ti) A.indices[((size_t)bt * A.Hq + target_head(A, ti)) * A.k + p] = n;
      }
      g += is_gt ? 1u : 0u;
      q += is_gt ? 0u : 1u;
    }
    gbase += total & 0xffffu;
    qbase += total >> 16;
    if (gbase + min(qbase, r) >= c || 4 * (step + THREADS) >= to) break;   // the list is complete (uniform)
  }
}

}  // namespace
