// Short rows (gfx950): a row that one workgroup's registers hold, ranked in one launch. Every thread
// loads and aggregates the row's quads that are its own (same fp32 order as everywhere) and keeps the
// keys; nothing is read twice. The kernels:
//   short_select_row_kernel  a few keys per thread: all of them counted, in 2048 bins that divide the row's key range and,
//                            if the bin of the threshold still holds more than a few keys, that bin;
//   select_row_kernel        more keys per thread: a sample gives a window of keys around the threshold, whose keys are counted
//                            in up to 2048 bins;
//   short_select_row_scores_kernel, select_row_scores_kernel  the same where several scores per token, or probabilities of
//                            logits, are added up first;
//   select_row_long_kernel   select_row_kernel for rows of 32769 to 65536 tokens, one score each;
//   select_row16_kernel      rows of one bf16 score per token, two keys to a register.
// The kept tokens are bits in LDS; the list is the bits read in order.
//
// What bounds it: for thousands of rows memory and vector instructions alike; several small workgroups per CU hide each
// other's latencies. For few rows latency. Counting used to be a comparison per key and mask of lanes; where every key adds
// to some slot, each lane to its own outside the window, 4096 rows of 16384 tokens took 98 us (131), 2048 of 30001 99 (136),
// 4096 of 20000 156 (234), 256 rows of 16384 with five scores per token 21.9 (24.2), and rows of zeros with the budget at
// their edge 130 (625); with a row's loads in flight together 4096 rows of 16384 take 69, 2048 of 30001 73, 4096 of 20000 123.
#include "select_util.h"

namespace {

constexpr int ROW_CAND = 64;              // keys of the threshold's bin that are ranked against each other

// nothing is moved across: a pass over keys in registers needs few others then
__device__ __forceinline__ void fence_schedule() {
#if defined(__AMDGCN__)
  __builtin_amdgcn_sched_barrier(0);
#endif
}
typedef u32x4 u32x4_any __attribute__((aligned(2)));

// the same value, which the compiler does not know: what is computed from it is not kept from earlier
__device__ __forceinline__ int again(int x) {
#if defined(__AMDGCN__)
  asm("" : "+v"(x));
#endif
  return x;
}

// Exclusive sums over the workgroup of two values per thread (tot: 2 * T / 64 words), and the totals.
template <int T>
__device__ __forceinline__ void scan2(uint32_t a, uint32_t b, uint32_t *tot, int lane, int wave, uint32_t &a0, uint32_t &b0,
                                      uint32_t &as, uint32_t &bs) {
  const uint32_t ai = wave_incl_scan(a), bi = wave_incl_scan(b);
  if (lane == 63) {
    tot[2 * wave] = ai;
    tot[2 * wave + 1] = bi;
  }
  __syncthreads();
  a0 = ai - a;
  b0 = bi - b;
  as = bs = 0;
#pragma unroll
  for (int w = 0; w < T / 64; ++w) {
    const uint32_t x = tot[2 * w], y = tot[2 * w + 1];
    if (w < wave) {
      a0 += x;
      b0 += y;
    }
    as += x;
    bs += y;
  }
}

// Valid length of a row; of a row of block sums, which is ranked as a row of scores, from its length in tokens. (Kernels of
// their own: the page's size, asked for after the length, is another latency in front of every row's first load. 16 rows of 4096
// tokens with lengths: 8.3 us, 8.55 with one kernel for both. The longer rows' kernels are 1% faster with this form than with
// row_len, 4096 rows of 16384 tokens; the short rows' 1% slower.)
template <bool BLOCKS>
__device__ __forceinline__ int ranked_len(const SelectArgs &A, int bt) {
  int n = A.N;
  if (A.seq_lens) {
    n = max(A.seq_lens[bt], 0);
    if (BLOCKS) n = (int)(((uint32_t)n + (uint32_t)A.page - 1u) / (uint32_t)A.page);
  }
  return min(n, A.N);
}

// The row's scores, aggregated, as signed numbers of their order (positive ones as they are, the others their magnitude's
// negative, so that -0 is +0): thread tid gets the quads tid, tid + T, ... A position past the row's valid length holds INT_MIN,
// which no token does, and its scores are not read: past the last quad with a token that quad is asked for again, which costs
// no memory (rows of a tensor that is allocated for the longest sequence). out: the aggregate, stored on request.
template <int T, int IT, bool ONE>
__device__ __forceinline__ void load_row(const AggRow &R, float *out, int nb, int tid, int (&v)[IT][4]) {
  int any = 0;
  const int last = max(min(R.N - 4, (nb - 1) & ~3), 0);
  auto take = [&](int i, f32x4 acc) {
    const int n = 4 * (i * T + tid);
    if (out && n < R.N) {
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (n + e < R.N) out[n + e] = n + e < nb ? acc[e] : 0.f;       // 0 past the valid length
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const float f = acc[e];
      v[i][e] = __builtin_bit_cast(int, f);
      any |= v[i][e];
    }
  };
  if constexpr (T == 1024 && IT <= 4 && !ONE) {
    // Few quads: their score rows are in flight together, by code for each number of rows (256 rows of 16384
    // tokens 16.9 us, 18.7 with branches between the rows).
#pragma clang loop unroll(full)
    for (int i = 0; i < IT; ++i) {
      const int n = 4 * (i * T + tid);
      const bool inside = 4 * (i + 1) * T <= R.N;
      const int at = min(n, last);
      const f32x4 y = agg_quad(R, at);
      take(i, inside ? y : shifted_quad(y, n - at));
    }
  } else if constexpr (!ONE) {
    // Four quads at a time, a score row of them in flight while the one before is added (a quad at a time with all its score
    // rows: the same for five and nine; eight quads at a time spill). Larger rows in this way: 16 of 33001, five scores, 28.7 us,
    // sampled 27.3. All quads of a score row in a loop, each waited for by itself: 1024 rows of 30000 with five scores
    // 139 us, now 122; of 24000 with two 67, 50; of 8192 with five 38.5, 34.3.
    auto blocks = [&](auto bf16) {
      typedef ScoreLoad<f32x4, decltype(bf16)::value> SL;
      constexpr int QB = 4;
      const size_t pitch = (size_t)R.N * (decltype(bf16)::value ? 2 : 4);
#pragma clang loop unroll(full)
      for (int b = 0; b < IT; b += QB) {
        f32x4 acc[QB];
        if (4 * b * T < nb) {
          typename SL::raw x[QB], y[QB];
          auto load = [&](typename SL::raw (&r)[QB], int q) {
            const unsigned char *at = static_cast<const unsigned char *>(R.P) + q * pitch;
            const int own = IT > 8 ? again(tid) : tid;
#pragma unroll
            for (int i = 0; i < QB; ++i) {
              const uint32_t off = (uint32_t)min(4 * ((b + i) * T + own), last) * (decltype(bf16)::value ? 2u : 4u);
              r[i] = SL::load_at(at + off);
            }
          };
          auto add = [&](const typename SL::raw (&r)[QB], int q) {
            const float l = R.logits ? R.L[q] : 0.f;
#pragma unroll
            for (int i = 0; i < QB; ++i) {
              f32x4 p = SL::widen(r[i]);
              if (R.logits) {
#pragma unroll
                for (int e = 0; e < 4; ++e) p[e] = prob_of(p[e], l);
              }
              if (q == 0) {
                acc[i] = p;
              } else if (R.use_max) {
#pragma unroll
                for (int e = 0; e < 4; ++e) acc[i][e] = fmaxf(acc[i][e], p[e]);
              } else {
                acc[i] = acc[i] + p;
              }
            }
          };
          load(x, 0);
#pragma unroll 1
          for (int q = 0; q < R.Tq; q += 2) {
            if (q + 1 < R.Tq) load(y, q + 1);
            fence_schedule();
            add(x, q);
            if (q + 1 >= R.Tq) break;
            if (q + 2 < R.Tq) load(x, q + 2);
            fence_schedule();
            add(y, q + 1);
          }
        } else {
#pragma unroll
          for (int i = 0; i < QB; ++i) acc[i] = f32x4{0.f, 0.f, 0.f, 0.f};
        }
#pragma unroll
        for (int i = 0; i < QB; ++i) {
          const int n = 4 * ((b + i) * T + tid);
          take(b + i, 4 * (b + i + 1) * T <= R.N ? acc[i] : shifted_quad(acc[i], n - min(n, R.N - 4)));
        }
      }
    };
    if (R.bf16) blocks(std::true_type{});
    else blocks(std::false_type{});
  } else {
    // One probability per token: all quads in flight together. (A load next to its use in a loop over the quads is waited for
    // at once, one memory latency after the other, which is how rows of many quads were loaded: 4096 rows of 16384 tokens 95 us, now 69;
    // 4096 of 20000 159, 123; 2048 of 30001 98, 73; 4096 of 8192 51, 41.)
    auto rows = [&](auto bf16) {
      typedef ScoreLoad<f32x4, decltype(bf16)::value> SL;
      typename SL::raw x[IT];
#pragma clang loop unroll(full)
      for (int i = 0; i < IT; ++i)
        x[i] = SL::load_at(static_cast<const unsigned char *>(R.P) + (uint32_t)min(4 * (i * T + tid), last) * (decltype(bf16)::value ? 2u : 4u));
      fence_schedule();
#pragma clang loop unroll(full)
      for (int i = 0; i < IT; ++i) {
        const int n = 4 * (i * T + tid);
        const f32x4 y = SL::widen(x[i]);
        take(i, 4 * (i + 1) * T <= R.N ? y : shifted_quad(y, n - min(n, R.N - 4)));      // the row's end: read where it still fits
      }
    };
    if (R.bf16) rows(std::true_type{});
    else rows(std::false_type{});
  }
  if (ballot64(any < 0)) {                             // negative scores in this wave
#pragma clang loop unroll(full)
    for (int i = 0; i < IT; ++i)
#pragma unroll
      for (int e = 0; e < 4; ++e) v[i][e] = v[i][e] < 0 ? (int)(0x80000000u - (uint32_t)v[i][e]) : v[i][e];
  }
  if (nb < 4 * T * IT) {
#pragma clang loop unroll(full)
    for (int i = 0; i < IT; ++i)
#pragma unroll
      for (int e = 0; e < 4; ++e) v[i][e] = 4 * (i * T + tid) + e < nb ? v[i][e] : (int)0x80000000;
  }
}

// ----------------------------------------------------------- rows of at most eight quads per four waves
template <int T>
__device__ __forceinline__ void row_min_max(uint32_t &lo, uint32_t &hi, uint32_t *red) {
  wave_min_max(lo, hi);
  if ((threadIdx.x & 63) == 0) {
    red[2 * (threadIdx.x >> 6)] = lo;
    red[2 * (threadIdx.x >> 6) + 1] = hi;
  }
  __syncthreads();
#pragma unroll
  for (int w = 0; w < T / 64; ++w) {
    lo = min(lo, red[2 * w]);
    hi = max(hi, red[2 * w + 1]);
  }
}

// T threads, IT quads per thread: rows of up to 4 * T * IT tokens. All keys are counted, in bins that divide their range.
template <int T, int IT, bool BLOCKS, bool ONE>
__device__ __forceinline__ void rank_short_row(const SelectArgs &A) {
  constexpr int TOK = 4 * T * IT;
  constexpr int STAGE = TOK / 8 > 1024 ? TOK / 8 : 1024;           // list entries staged per round
  __shared__ uint32_t bits[TOK / 32];
  __shared__ uint32_t h[SEL_BINS];
  __shared__ uint32_t store[STAGE];                                // bits of the equal tokens, then list entries
  __shared__ uint32_t tmp[T / 64 + 2];
  __shared__ uint32_t red[2 * T / 64];
  __shared__ uint32_t ctr[4];
  const int j = blockIdx.x, bt = blockIdx.y, row = bt * A.Hd + j, tid = threadIdx.x, lane = tid & 63;
  const int nb = __builtin_amdgcn_readfirstlane(BLOCKS ? ranked_len<true>(A, bt) : row_len(A, bt));
  const uint32_t c = (uint32_t)min(A.kh[j], nb);
  const int t0 = target_off(A, j), t1 = target_off(A, j + 1);
  float *out = A.agg ? A.agg + (size_t)row * A.N : nullptr;
  const bool ranked = c > 0 && t0 != t1;
  if (!ranked && !out) return write_tail<T>(A, bt, j, c);
  const AggRow R = agg_row(A, row);
  for (int i = tid; i < SEL_BINS; i += T) h[i] = 0u;
  if (tid < 4) ctr[tid] = 0u;

  int v[IT][4];
  load_row<T, IT, ONE>(R, out, nb, tid, v);
  write_tail<T>(A, bt, j, c);                          // (not in front of the loads)
  if (!ranked) return;

  auto each = [&](auto f) {
#pragma clang loop unroll(full)
    for (int i = 0; i < IT; ++i)
#pragma unroll
      for (int e = 0; e < 4; ++e) f(v[i][e], 4 * (i * T + tid) + e);
  };
  // the bin of the rank-th largest of the keys counted in h, and what is left of the rank in it
  auto find = [&](uint32_t rank, uint32_t &bin, uint32_t &left) {
    find_digit<SEL_BINS, T, true>(h, rank, tmp, bin, left);
    bin = (uint32_t)__builtin_amdgcn_readfirstlane((int)bin);
    left = (uint32_t)__builtin_amdgcn_readfirstlane((int)left);
  };

  // ---- keys in question: lo .. lo + last
  uint32_t kmin = 0xffffffffu, kmax = 0u;
  each([&](int s, int) {
    if (s != (int)0x80000000) {
      kmin = min(kmin, key_of_ordered(s));
      kmax = max(kmax, key_of_ordered(s));
    }
  });
  row_min_max<T>(kmin, kmax, red);
  uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)kmin), last = (uint32_t)__builtin_amdgcn_readfirstlane((int)(kmax - kmin));
  uint32_t krem = c;
  int shift = max(0, 32 - __clz((int)last) - 11);
  uint32_t in_bin;
#pragma unroll 1
  for (;;) {
    each([&](int s, int) {
      const uint32_t k = key_of_ordered(s) - lo;
      if (k <= last && s != (int)0x80000000) atomicAdd(&h[k >> shift], 1u);
    });
    __syncthreads();
    uint32_t bin, left;
    find(krem, bin, left);
    in_bin = (uint32_t)__builtin_amdgcn_readfirstlane((int)h[bin]);
    lo += bin << shift;
    last = (1u << shift) - 1u;
    krem = left;
    if (shift == 0 || in_bin <= (uint32_t)ROW_CAND) break;
    shift = max(0, shift - 11);
    __syncthreads();                                   // every thread has read h[bin]
    for (int i = tid; i < SEL_BINS; i += T) h[i] = 0u;
    __syncthreads();
  }
  uint32_t Tk = lo, r = krem, E = in_bin;              // the threshold key; r of the E tokens equal to it are kept
  if (last != 0u) {
    // few keys share the bin: every wave ranks them against each other. (The candidates use the head of the
    // histogram, which is done with.)
    __syncthreads();
    auto add = [&](uint32_t k) {
      if (k - lo <= last) {
        const uint32_t s = atomicAdd(&ctr[2], 1u);
        if (s < (uint32_t)ROW_CAND) h[s] = k;
      }
    };
    each([&](int s, int) {
      if (s != (int)0x80000000) add(key_of_ordered(s));
    });
    __syncthreads();
    const uint32_t n = min(in_bin, (uint32_t)ROW_CAND);
    const uint32_t mine = h[min((uint32_t)lane, n - 1u)];
    uint32_t g = 0, e = 0;
    for (uint32_t q = 0; q < n; ++q) {
      const uint32_t k = h[q];
      g += k > mine ? 1u : 0u;
      e += k == mine ? 1u : 0u;
    }
    const int win = __builtin_ctzll(ballot64((uint32_t)lane < n && g < krem && g + e >= krem) | (1ull << 63));
    Tk = (uint32_t)__builtin_amdgcn_readlane((int)mine, win);
    r = krem - (uint32_t)__builtin_amdgcn_readlane((int)g, win);
    E = (uint32_t)__builtin_amdgcn_readlane((int)e, win);
  }

  // ---- bits of the kept tokens: all above T, and equal ones unless only some of them are kept, which then get bits
  // of their own
  const int sT = ordered_of_key(Tk);
  const bool all_eq = r >= E;
  __syncthreads();
  static_assert(sizeof(store) >= sizeof(bits), "the equal tokens' bits");
#pragma clang loop unroll(full)
  for (int i = 0; i < IT; ++i) {
    auto word = [&](uint32_t b, uint32_t *to) {        // eight lanes' nibbles make a word of token bits
      int w = (int)(b << (4 * (lane & 7)));
      w |= __builtin_amdgcn_update_dpp(0, w, 0x101, 0xf, 0xf, true);   // row_shl:1
      w |= __builtin_amdgcn_update_dpp(0, w, 0x102, 0xf, 0xf, true);   // row_shl:2
      w |= __builtin_amdgcn_update_dpp(0, w, 0x104, 0xf, 0xf, true);   // row_shl:4
      if ((lane & 7) == 0) to[(i * T + tid) >> 3] = (uint32_t)w;
    };
    uint32_t above = 0, eq = 0;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      above |= v[i][e] > sT ? 1u << e : 0u;
      eq |= v[i][e] == sT ? 1u << e : 0u;
    }
    word(all_eq ? above | eq : above, bits);
    if (!all_eq) word(eq, store);
  }
  __syncthreads();
  constexpr int PER = (TOK / 32 + T - 1) / T;          // words per thread, consecutive
  const int w0 = min(tid * PER, TOK / 32), w1 = min(w0 + PER, TOK / 32);
  uint32_t total;
  if (!all_eq) {
    uint32_t n = 0;
    for (int w = w0; w < w1; ++w) n += (uint32_t)__builtin_popcount(store[w]);
    uint32_t before = block_excl_scan<T, true>(n, tmp, total);
    for (int w = w0; w < w1; ++w)
      for (uint32_t rest = store[w]; rest && before < r; rest &= rest - 1u, ++before) bits[w] |= rest & (0u - rest);
  }
  uint32_t mine = 0;
  for (int w = w0; w < w1; ++w) mine += (uint32_t)__builtin_popcount(bits[w]);
  const uint32_t first = block_excl_scan<T, true>(mine, tmp, total);         // (its barriers free `store`)
  total = min(total, c);                               // total == c for a consistent state
  int32_t *staged = reinterpret_cast<int32_t *>(store);
#pragma unroll 1
  for (uint32_t base = 0; base < total; base += STAGE) {
    uint32_t p = first;
    if (p < base + STAGE && p + mine > base)
      for (int w = w0; w < w1; ++w)
        for (uint32_t rest = bits[w]; rest; rest &= rest - 1u, ++p)
          if (p - base < (uint32_t)STAGE) staged[p - base] = 32 * w + __builtin_ctz(rest);
    __syncthreads();
    const uint32_t cnt = min(total - base, (uint32_t)STAGE);
    for (int ti = t0; ti < t1; ++ti) {
      int32_t *dst = A.indices + ((size_t)bt * A.Hq + target_head(A, ti)) * A.k + base;
      for (uint32_t i = tid; i < cnt; i += T) dst[i] = staged[i];
    }
    __syncthreads();
  }
}

template <int T, int IT>
__global__ void __launch_bounds__(T) short_select_row_kernel(const SelectArgs A) { rank_short_row<T, IT, false, true>(A); }
template <int T, int IT>
__global__ void __launch_bounds__(T) short_select_row_scores_kernel(const SelectArgs A) { rank_short_row<T, IT, false, false>(A); }
template <int T, int IT>
__global__ void __launch_bounds__(T) short_select_blocks_kernel(const SelectArgs A) { rank_short_row<T, IT, true, true>(A); }

// ----------------------------------------------------------- longer rows: a window of keys from a sample
// T threads, IT quads per thread: rows of up to 4 * T * IT tokens. (Up to eight keys per thread of 1024, or 16 of 256, are ranked
// faster without a sample: 16 rows of 4096 tokens 8.3 against 9.5 us, 1024 of 4096 10.4, 10.8.)
template <int T, int IT, bool BLOCKS, bool ONE>
__device__ __forceinline__ void rank_row(const SelectArgs &A) {
  constexpr int TOK = 4 * T * IT;
  constexpr int STAGE = TOK / 8 > 1024 ? TOK / 8 : 1024;           // list entries staged per round
  constexpr int SLOTS = SEL_BINS + 2 * 64;                         // a window's bins, and 64 for the keys on either side of it
  __shared__ __attribute__((aligned(16))) uint32_t codes[TOK / 16];            // a byte per quad: bits of the tokens above, of the equal ones
  __shared__ uint32_t h[SLOTS];
  __shared__ uint32_t staged[STAGE];
  __shared__ uint32_t cand_key[ROW_CAND], cand_tok[ROW_CAND];      // (not as pairs: the keys would be held in pairs of registers)
  __shared__ uint32_t tot[2 * T / 64];
  __shared__ uint32_t res[8];
  const int j = blockIdx.x, bt = blockIdx.y, row = bt * A.Hd + j;      // (no division in front of the first load)
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int nb = __builtin_amdgcn_readfirstlane(ranked_len<BLOCKS>(A, bt));
  const uint32_t c = (uint32_t)min(A.kh[j], nb);
  const int t0 = target_off(A, j), t1 = target_off(A, j + 1);
  float *out = A.agg ? A.agg + (size_t)row * A.N : nullptr;
  const bool ranked = c > 0 && t0 != t1;
  if (!ranked && !out) return write_tail<T>(A, bt, j, c);
  const AggRow R = agg_row(A, row);
  for (int i = tid; i < SLOTS; i += T) h[i] = 0u;

  int v[IT][4];
  load_row<T, IT, ONE>(R, out, nb, tid, v);
  write_tail<T>(A, bt, j, c);
  if (!ranked) return;
  uint32_t k[IT][4];                                   // unsigned keys, 0 where there is no token
#pragma clang loop unroll(full)
  for (int i = 0; i < IT; ++i)
#pragma unroll
    for (int e = 0; e < 4; ++e) k[i][e] = key_of_ordered(v[i][e]);

  constexpr int PER = SEL_BINS / T;
  // Counts of this thread's bins (of n, from slot `at` on), returned: keys in the bins above them, in all bins, and in the
  // 64 slots after the bins.
  auto bins_above = [&](uint32_t at, uint32_t n, uint32_t (&loc)[PER], uint32_t &inside, uint32_t &beyond) -> uint32_t {
    uint32_t sum = 0, before, unused;
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      const uint32_t x = (uint32_t)(tid * PER + i);
      loc[i] = x < n ? h[at + x] : 0u;
      sum += loc[i];
    }
    scan2<T>(sum, tid < 64 ? h[at + n + tid] : 0u, tot, lane, wave, before, unused, inside, beyond);
    return inside - before - sum;
  };
  auto clear = [&] {
    __syncthreads();                                               // every thread has read what it needs
    for (int i = tid; i < SLOTS; i += T) h[i] = 0u;
    __syncthreads();
  };
  auto uniform = [](uint32_t x) { return (uint32_t)__builtin_amdgcn_readfirstlane((int)x); };

  // ---- a window of keys lo .. lo + last around the threshold
  uint32_t lo = 1, last = 0xfffffffeu, heavy = 0;
  if (nb >= 1024) {
    // From a sample of one key in four, or 2048, by its keys' upper 11 bits and, if that is one value, by the 11 bits below. Of a row
    // that fills the registers every thread takes one quad of STEP, its neighbours the others, so that each stretch of the row has
    // its share of the sample; of one that is short enough for a key of every quad, all do. (Where the waves took a few
    // registers each, 256 tokens next to each other were all in the sample or none, and rows shorter than the tensor were sampled by one or
    // two waves: heavy tokens at the start misled the window. 16 rows of a tensor of 32768 tokens, 256 kept, such a start: 4096 valid
    // 19.2 us, 12.9 now, 16384 valid 21.7, 13.3, all valid 22.5, 13.8; of 65536, 256 kept 32.3, 19.8. Rows without one as before.)
    constexpr int STEP = T * IT > 2048 ? T * IT / 2048 : 1;
    static_assert(IT % STEP == 0, "a thread's quads are taken STEP at a time");
    uint32_t from = 0, sh = 21;
    __syncthreads();
#pragma unroll 1
    for (uint32_t deep = 0, top = 0;;) {
      auto count = [&](uint32_t s) {
        const uint32_t x = (s - from) >> sh;
        if (s && x < (uint32_t)SEL_BINS) atomicAdd(&h[x], 1u);
      };
      if (STEP > 1 && nb > TOK / STEP) {
#pragma clang loop unroll(full)
        for (int i = 0; i < IT; i += STEP) {
          uint32_t s = k[i][(i / STEP) & 3];
#pragma clang loop unroll(full)
          for (int x = 1; x < STEP; ++x) s = tid % STEP == x ? k[i + x][(i / STEP + x) & 3] : s;
          count(s);
        }
      } else {
#pragma clang loop unroll(full)
        for (int i = 0; i < IT / STEP; ++i) count(k[i][i & 3]);
      }
      __syncthreads();
      uint32_t loc[PER], ns, unused;
      uint32_t above = bins_above(0u, SEL_BINS, loc, ns, unused);
      if (sh == 21) {
        // 5 standard deviations of the sample's count, down to its largest key; a window that misses the threshold is found out by
        // the counts (of few kept tokens, too: a window without an upper end has bins that need another pass. 16 rows of 17000
        // tokens, 340 kept, five scores each: 21.4 us, 15.4 so; 1024 rows of 65536 bf16 scores, 1000 kept, 53.6, 37.2)
        const uint32_t cs = expected_rank(c, ns, nb);
        const uint32_t margin = (uint32_t)(5.f * sqrtf((float)cs)) + 4u;
        deep = cs + margin;
        top = cs > margin ? cs - margin : 1u;
      }
      if (tid == 0) {
        res[0] = 0u;
        res[1] = SEL_BINS - 1;
        res[2] = res[3] = 0u;
      }
      __syncthreads();
#pragma unroll
      for (int i = PER - 1; i >= 0; --i) {
        if (above < deep && above + loc[i] >= deep) {
          res[0] = (uint32_t)(tid * PER + i);
          res[2] = loc[i];
          res[3] = above;
        }
        if (above < top && above + loc[i] >= top) res[1] = (uint32_t)(tid * PER + i);
        above += loc[i];
      }
      clear();
      const uint32_t lo_bin = uniform(res[0]), hi_bin = uniform(res[1]);
      const uint32_t end = from + (hi_bin << sh) + ((1u << sh) - 1u), next = from + ((lo_bin + 1u) << sh);
      const bool zero_bin = sh == 21 && lo_bin == (0x80000000u >> 21);
      lo = max(1u, from + (lo_bin << sh));
      if (hi_bin == lo_bin && !zero_bin && sh == 21) {
        from = lo_bin << sh;
        sh = 10;
        deep -= uniform(res[3]);
        top -= uniform(res[3]);
        continue;
      }
      // Zeros at the window's lower end would meet in one slot: the window begins above them, as far up as its slots for
      // keys below reach, and they are looked at by themselves if the threshold is not in the window.
      if (zero_bin && hi_bin > lo_bin && 8u * uniform(res[2]) > ns) {
        heavy = lo;
        const uint32_t room = next + (64u << max(0, 21 - __builtin_clz(end - next)));
        lo = room < (hi_bin << sh) ? room : next;
      }
      last = zero_bin && hi_bin == lo_bin ? 31u : end - lo;
      break;
    }
  } else {
    __syncthreads();
  }

  // ---- the threshold's bin: count the window's keys in up to 2048 bins, until a bin is one key or holds few
  uint32_t krem = c, in_bin;
  bool first = true;
#pragma unroll 1
  for (;;) {
    const uint32_t shift = (uint32_t)max(0, 21 - __builtin_clz(last | 1u)), n = (last >> shift) + 1u;
    // Every token adds to some slot: the window's n bins from slot `at` on, the slots before them for keys below and the
    // slots after them for keys above, there each lane to its own (no comparison, no mask of lanes, no conflict). Few bins
    // have 2^rs copies each, by lane: keys that repeat do not wait for each other.
    const uint32_t rs = shift ? 0u : min(6u, (uint32_t)__builtin_clz(max(n, 2u) - 1u) - 21u);   // n << rs <= 2048
    const uint32_t at = min(64u >> rs, lo >> shift), base = lo - (at << shift);
    const uint32_t least = at ? min((uint32_t)lane >> rs, at - 1u) : 0u, most = at + n + ((uint32_t)lane >> rs);
    const uint32_t copy = 4u * ((uint32_t)lane & ((1u << rs) - 1u));
#pragma clang loop unroll(full)
    for (int i = 0; i < IT; ++i) {
      if (4 * i * T < nb) {
        uint32_t x[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) x[e] = __builtin_elementwise_sub_sat(k[i][e], base) >> shift;
#pragma unroll
        for (int e = 0; e < 4; ++e) x[e] = (min(max(x[e], least), most) << (rs + 2u)) | copy;
#pragma unroll
        for (int e = 0; e < 4; ++e) atomicAdd(reinterpret_cast<uint32_t *>(reinterpret_cast<unsigned char *>(h) + x[e]), 1u);
      }
      fence_schedule();
    }
    __syncthreads();
    // Without slots below, the positions after the row's end are in bin 0: there only tokens count. (Its copies are one, and
    // thread 0 is the one that reads it.)
    if (at == 0u && tid == 0) h[0] -= (uint32_t)((nb + 4 * T - 1) / (4 * T) * (4 * T) - nb);
    uint32_t loc[PER], inside, beyond;
    uint32_t above = bins_above(at << rs, n << rs, loc, inside, beyond);
    if (first) krem = c - min(beyond, c);
    if (krem < 1u || krem > inside) {                              // not in the window: below it, or the sample misled
      const bool zeros = heavy && krem > inside;
      lo = zeros ? heavy : 1u;
      last = zeros ? 31u : 0xfffffffeu;
      heavy = 0;
      clear();
      continue;
    }
    if (tid == 0) res[6] = 0u;                                     // candidates, below
    if (rs && tid == 0) res[5] = 0u;
    uint32_t over = above;
#pragma unroll
    for (int i = PER - 1; i >= 0; --i) {
      if (over < krem && over + loc[i] >= krem) {
        res[3] = (uint32_t)(tid * PER + i) >> rs;
        if (!rs) {
          res[4] = krem - over;
          res[5] = loc[i];
        }
      }
      over += loc[i];
    }
    __syncthreads();
    const uint32_t bin = uniform(res[3]);
    if (rs) {                                                      // the counts of the bin's copies
#pragma unroll
      for (int i = PER - 1; i >= 0; --i) {
        const uint32_t x = (uint32_t)(tid * PER + i);
        if (x >> rs == bin) {
          if ((x + 1u) >> rs != bin) res[4] = krem - above;        // (the bin's last copy)
          if (loc[i]) atomicAdd(&res[5], loc[i]);
        }
        above += loc[i];
      }
      __syncthreads();
    }
    first = false;
    krem = uniform(res[4]);
    in_bin = uniform(res[5]);
    lo += bin << shift;
    last = min((1u << shift) - 1u, ~lo);                           // (the window's last bin may run past the highest key)
    if (shift == 0 || in_bin <= (uint32_t)ROW_CAND) break;
    clear();
  }

  // ---- a byte per quad. Few keys in the threshold's bin: they are listed, and those that are kept get their bits. Many
  // equal ones: bits of their own, of which the first r in token order are kept.
  unsigned char *const bytes = reinterpret_cast<unsigned char *>(codes);
  const bool few = in_bin <= (uint32_t)ROW_CAND;
  const uint32_t r = few ? 0u : krem, hi = lo + last;
  const int own = again(tid);
  if (few) {
#pragma clang loop unroll(full)
    for (int i = 0; i < IT; ++i) {
      uint32_t m = 0, x[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        m |= k[i][e] > hi ? 1u << e : 0u;
        x[e] = k[i][e] - lo;
      }
      if (min(min(x[0], x[1]), min(x[2], x[3])) <= last) {
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (x[e] <= last) {
            const uint32_t at = atomicAdd(&res[6], 1u);
            if (at < (uint32_t)ROW_CAND) {
              cand_key[at] = k[i][e];
              cand_tok[at] = (uint32_t)(4 * (i * T + own) + e);
            }
          }
      }
      bytes[i * T + own] = (unsigned char)m;
      fence_schedule();
    }
    __syncthreads();
    if (wave == 0) {
      const uint32_t n = min(in_bin, (uint32_t)ROW_CAND);
      const uint32_t key = cand_key[min((uint32_t)lane, n - 1u)], tok = cand_tok[min((uint32_t)lane, n - 1u)];
      uint32_t ahead = 0;
      for (uint32_t q = 0; q < n; ++q) {
        const uint32_t x = cand_key[q];
        ahead += x > key || (x == key && cand_tok[q] < tok) ? 1u : 0u;
      }
      if ((uint32_t)lane < n && ahead < krem) atomicOr(&codes[tok >> 4], 1u << (8 * (tok >> 2 & 3u) + (tok & 3u)));
    }
  } else {
#pragma clang loop unroll(full)
    for (int i = 0; i < IT; ++i) {
      uint32_t m = 0;
#pragma unroll
      for (int e = 0; e < 4; ++e) m |= k[i][e] > lo ? 1u << e : k[i][e] == lo ? 16u << e : 0u;
      bytes[i * T + own] = (unsigned char)m;
      fence_schedule();
    }
  }
  __syncthreads();
  constexpr int CW = IT >= 4 ? IT / 4 : 1;             // words of 16 tokens per thread, consecutive
  uint32_t w[CW], gt = 0, eq = 0;
#pragma unroll
  for (int x = 0; x < CW; ++x) {
    w[x] = tid * CW + x < TOK / 16 ? codes[tid * CW + x] : 0u;
    gt += (uint32_t)__builtin_popcount(w[x] & 0x0f0f0f0fu);
    eq += (uint32_t)__builtin_popcount(w[x] & 0xf0f0f0f0u);
  }
  uint32_t gt0, eq0, gts, eqs;
  scan2<T>(gt, eq, tot, lane, wave, gt0, eq0, gts, eqs);
  const uint32_t pos = gt0 + min(eq0, r);              // this thread's first place in the list
  uint32_t mine = 0;
#pragma unroll
  for (int x = 0; x < CW; ++x) {
    const uint32_t e = (w[x] >> 4) & 0x0f0f0f0fu, n = (uint32_t)__builtin_popcount(e);
    uint32_t keep = eq0 + n <= r ? e : 0u;
    if (n && eq0 < r && eq0 + n > r) {
      uint32_t rest = e;
      for (uint32_t q = eq0; q < r; ++q) {
        keep |= rest & (0u - rest);
        rest &= rest - 1u;
      }
    }
    eq0 += n;
    uint32_t y = (w[x] & 0x0f0f0f0fu) | keep;
    mine += (uint32_t)__builtin_popcount(y);
    y = (y | y >> 4) & 0x00ff00ffu;                    // the nibbles next to each other
    y = (y | y >> 8) & 0x0000ffffu;
    if (CW % 2) w[x] = y;
    else if (x & 1) w[x >> 1] |= y << 16;
    else w[x >> 1] = y;
  }
  constexpr int LW = CW % 2 ? CW : CW / 2, LT = CW % 2 ? 16 : 32;  // words of LT tokens
#pragma unroll 1
  for (uint32_t base = 0; base < c; base += STAGE) {
    uint32_t p = pos;
    if (p < base + STAGE && p + mine > base) {
#pragma unroll
      for (int x = 0; x < LW; ++x)
        for (uint32_t rest = w[x]; rest; rest &= rest - 1u, ++p)
          if (p - base < (uint32_t)STAGE) staged[p - base] = (uint32_t)(LT * (tid * LW + x) + __builtin_ctz(rest));
    }
    __syncthreads();
    const uint32_t cnt = min(c - base, (uint32_t)STAGE);
    for (int ti = t0; ti < t1; ++ti) {
      int32_t *dst = A.indices + ((size_t)bt * A.Hq + target_head(A, ti)) * A.k + base;
      for (uint32_t i = tid; i < cnt; i += T) dst[i] = (int32_t)staged[i];
    }
    __syncthreads();
  }
}

template <int T, int IT>
__global__ void __launch_bounds__(T, 4) select_row_kernel(const SelectArgs A) { rank_row<T, IT, false, true>(A); }
template <int T, int IT>
__global__ void __launch_bounds__(T, 4) select_row_scores_kernel(const SelectArgs A) { rank_row<T, IT, false, false>(A); }
template <int T, int IT>
__global__ void __launch_bounds__(T, 4) select_row_long_kernel(const SelectArgs A) { rank_row<T, IT, false, true>(A); }
template <int T, int IT>
__global__ void __launch_bounds__(T, 4) select_blocks_kernel(const SelectArgs A) { rank_row<T, IT, true, true>(A); }

// ------------------------------------------------- rows of one bf16 score per token, packed in registers
// Calls with a mask per query row (prefill) rank thousands of rows of bf16 scores. 64K of them are 128 KB, 64 registers of
// 512 threads: a CU holds two such rows, each is read once, and one row's ranking hides behind the loads of the other.
// Keys are 16 bits, two to a register, and nearly everything is done to both at once (packed 16-bit subtraction with
// saturation, minimum, maximum): a sample of 2048 keys gives a window of keys around the threshold; one pass counts
// the window's keys one by one in LDS and those above it; the threshold is one of them. Each token's two bits (above,
// equal) go to LDS and are read in order for the list.
//
// What bounds it: memory and vector instructions alike. 4096 rows of 65536 tokens, 10% kept: 140 us (155 at first), 537 MB read
// and 107 MB written, 12 vector instructions per token; the several-pass kernel that served it read them twice, 17 per token: 236.
// Other calls beside the rule in the host code. Measured on the way: masks of lanes and ballots instead of a slot per lane for
// the keys outside the window 229 us; 256 threads with 128 registers of keys, three rows per CU, 153-157, but 256 rows of
// 65536 20.5 against 17.0; 131072 tokens in 512 threads 1053 us for 8192 rows, in 1024 threads 889 (several
// passes 949).
typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));
typedef short i16x2 __attribute__((ext_vector_type(2)));
// Scores with their order as signed numbers: positive ones as they are, the others their magnitude's negative, so that -0 is
// +0 and the lowest number stays free for "no token".
__device__ __forceinline__ uint32_t signed16(uint32_t w) {
  const u16x2 x = __builtin_bit_cast(u16x2, w), sign = x >> (u16x2)15;
  const u16x2 flip = __builtin_bit_cast(u16x2, __builtin_bit_cast(uint32_t, sign) * 0x7fffu);
  return __builtin_bit_cast(uint32_t, (x ^ flip) + sign);
}

constexpr int ROW16_SLOTS = SEL_BINS + 2 * 64;                     // a window's bins, and 64 for the keys on either side of it
constexpr int ROW16_STAGE = 8192;                                  // list entries staged per round

// The ranking of one row of nb valid tokens, c of them kept, by T threads with IT 16-byte words each. codes, h, staged, tot, res: LDS.
template <int T, int IT, class stage_t>
__device__ __forceinline__ void rank_row16(const SelectArgs &A, int row, int nb, uint32_t c, uint32_t *codes, uint32_t *h, stage_t *staged,
                                           uint32_t *tot, uint32_t *res) {
  constexpr int CODES = 8 * T * IT / 16;                           // words of two bits per token
  constexpr int STAGE = ROW16_STAGE, SLOTS = ROW16_SLOTS;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int j = blockIdx.x, bt = blockIdx.y;
  const int t0 = target_off(A, j), t1 = target_off(A, j + 1);
  const uint16_t *src = static_cast<const uint16_t *>(A.scores) + (size_t)row * A.N;

  // ---- the row: thread tid holds the words tid, tid + T, ... as signed numbers of the scores' order, the lowest where there is no
  // token (a score that is not negative is its own bit pattern). The key is that number's distance from the lowest.
  i16x2 k[IT][4];
  {
    u32x4 raw[IT];
    // (past the last word with a token that word is asked for again, which costs no memory)
    const uint32_t cap = 2u * (uint32_t)min(A.N - 8, (nb - 1) & ~7);
#pragma clang loop unroll(full)
    for (int i = 0; i < IT; ++i) {
      raw[i] = __builtin_nontemporal_load(reinterpret_cast<const u32x4_any *>(reinterpret_cast<const unsigned char *>(src) + min(16u * (uint32_t)(i * T + tid), cap)));
    }
    for (int i = tid; i < SLOTS; i += T) h[i] = 0u;
    uint32_t any = 0;
#pragma clang loop unroll(full)
    for (int i = 0; i < IT; ++i) any |= raw[i][0] | raw[i][1] | raw[i][2] | raw[i][3];
    if (ballot64((any & 0x80008000u) != 0u)) {                     // negative scores in this wave
#pragma clang loop unroll(full)
      for (int i = 0; i < IT; ++i)
#pragma unroll
        for (int e = 0; e < 4; ++e) raw[i][e] = signed16(raw[i][e]);
    }
#pragma clang loop unroll(full)
    for (int i = 0; i < IT; ++i)
      if (8 * (i + 1) * T > nb) {                                  // the row's end
        const int n = 8 * (i * T + tid), d = n - min(n, A.N - 8);  // tokens that the word was read before its place
        if (d & 4) { raw[i][0] = raw[i][2]; raw[i][1] = raw[i][3]; }
        if (d & 2) { raw[i][0] = raw[i][1]; raw[i][1] = raw[i][2]; raw[i][2] = raw[i][3]; }
        if (d & 1) {
#pragma unroll
          for (int e = 0; e < 3; ++e) raw[i][e] = raw[i][e] >> 16 | raw[i][e + 1] << 16;
          raw[i][3] >>= 16;
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          if (n + 2 * e >= nb) raw[i][e] = (raw[i][e] & 0xffff0000u) | 0x8000u;
          if (n + 2 * e + 1 >= nb) raw[i][e] = (raw[i][e] & 0xffffu) | 0x80000000u;
        }
      }
#pragma clang loop unroll(full)
    for (int i = 0; i < IT; ++i)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const uint32_t w = raw[i][e];                              // (a vector's element itself is not what would be converted)
        k[i][e] = __builtin_bit_cast(i16x2, w);
      }
  }

  constexpr int PER = SEL_BINS / T;
  // Counts of this thread's bins (of n, from slot `at` on), returned: keys in the bins above them, in all bins, and in the
  // 64 slots after the bins.
  auto bins_above = [&](uint32_t at, uint32_t n, uint32_t (&loc)[PER], uint32_t &inside, uint32_t &beyond) -> uint32_t {
    uint32_t sum = 0, before, unused;
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      const uint32_t x = (uint32_t)(tid * PER + i);
      loc[i] = x < n ? h[at + x] : 0u;
      sum += loc[i];
    }
    scan2<T>(sum, tid < 64 ? h[at + n + tid] : 0u, tot, lane, wave, before, unused, inside, beyond);
    return inside - before - sum;
  };
  auto clear = [&] {
    __syncthreads();                                               // every thread has read what it needs
    for (int i = tid; i < SLOTS; i += T) h[i] = 0u;
    __syncthreads();
  };

  // ---- a window of keys lo .. lo + last around the threshold, from a sample
  uint32_t lo = 1, last = 0xfffe, heavy = 0;
  __syncthreads();
  if (nb >= 1024) {
    // One key of eight, or less where that would be more than 2048: bins of 32 keys are coarser than their error, and keys that share
    // a bin wait for each other. (4096 rows of 65536 tokens 150.6 us with one of eight, 141 with 4096 keys, 140 with 2048; 1024
    // of 131072 128, 124, 122.) Taken as the longer fp32 rows are, see rank_row. (300 rows of 131072, 700 kept, heavy tokens at the start:
    // 71.5 us with a few registers of every wave, 49.7 so.)
    constexpr int STEP = T * IT > 2048 ? T * IT / 2048 : 1;
    static_assert(IT % STEP == 0, "a thread's words are taken STEP at a time");
    auto count = [&](i16x2 w) {
      const uint32_t s = (uint32_t)(unsigned short)w[0] ^ 0x8000u;
      if (s) atomicAdd(&h[s >> 5], 1u);
    };
    if (STEP > 1 && nb > 8 * T * IT / STEP) {
#pragma clang loop unroll(full)
      for (int i = 0; i < IT; i += STEP) {
        i16x2 w = k[i][(i / STEP) & 3];
#pragma clang loop unroll(full)
        for (int x = 1; x < STEP; ++x) w = tid % STEP == x ? k[i + x][(i / STEP + x) & 3] : w;
        count(w);
      }
    } else {
#pragma clang loop unroll(full)
      for (int i = 0; i < IT / STEP; ++i) count(k[i][i & 3]);
    }
    __syncthreads();
    uint32_t loc[PER], ns, unused;
    uint32_t above = bins_above(0u, SEL_BINS, loc, ns, unused);
    // 5 standard deviations of the sample's count; a window that misses the threshold is found out by the counts
    const uint32_t cs = expected_rank(c, ns, nb);
    const uint32_t margin = (uint32_t)(5.f * sqrtf((float)cs)) + 4u;
    const uint32_t deep = cs + margin, top = cs > margin ? cs - margin : 1u;
    if (tid == 0) {
      res[0] = 0u;
      res[1] = SEL_BINS - 1;
      res[5] = 0u;
    }
    __syncthreads();
#pragma unroll
    for (int i = PER - 1; i >= 0; --i) {
      if (above < deep && above + loc[i] >= deep) {
        res[0] = (uint32_t)(tid * PER + i);
        res[5] = loc[i];
      }
      if (above < top && above + loc[i] >= top) res[1] = (uint32_t)(tid * PER + i);
      above += loc[i];
    }
    clear();
    const uint32_t lo_bin = (uint32_t)__builtin_amdgcn_readfirstlane((int)res[0]), hi_bin = (uint32_t)__builtin_amdgcn_readfirstlane((int)res[1]);
    lo = max(1u, lo_bin << 5);
    last = (hi_bin << 5) + 31u - lo;
    // A value that repeats at the window's lower end (zeros, below a gap) would meet itself in one slot: the window begins
    // above it, where there is room as far up as its slots for keys below reach, and that value is looked at by itself if
    // the threshold is not in the window.
    const uint32_t end = (hi_bin << 5) + 31u, next = (lo_bin + 1u) << 5;
    if (hi_bin > lo_bin + 1u && 8u * (uint32_t)__builtin_amdgcn_readfirstlane((int)res[5]) > ns) {
      heavy = lo;
      const uint32_t room = next + (64u << max(0, 21 - __builtin_clz(end - next)));
      lo = room < (hi_bin << 5) ? room : next;
      last = end - lo;
    }
  }

  // ---- the threshold: count the window's keys (in bins, if there are more than 2048) until a bin is one key
  uint32_t krem = c;
  bool first = true;
#pragma unroll 1
  for (;;) {
    const uint32_t shift = (uint32_t)max(0, 32 - __builtin_clz(last | 1u) - 11), n = (last >> shift) + 1u;
    // Every token adds to some slot: the window's n bins from slot `at` on, the slots before them for keys below and the
    // slots after them for keys above, there each lane to its own (no comparison, no mask of lanes, no conflict). Few bins
    // have 2^rs copies each, by lane: keys that repeat do not wait for each other.
    const uint32_t rs = min(6u, (uint32_t)__builtin_clz(max(n, 2u) - 1u) - 21u);                 // n << rs <= 2048
    const uint32_t at = min(64u >> rs, lo >> shift), base = lo - (at << shift);
    auto pair = [](uint32_t x) { return (u16x2)(unsigned short)x; };
    auto signed_pair = [](uint32_t x) { return (i16x2)(short)(unsigned short)x; };
    const u16x2 copies = pair(1u << rs), copy = pair((uint32_t)lane & ((1u << rs) - 1u));
    const uint32_t least = at ? min((uint32_t)lane >> rs, at - 1u) : 0u, most = at + n + ((uint32_t)lane >> rs);
    auto add = [&](u16x2 x) {
      x = x * copies + copy;
      atomicAdd(&h[x[0]], 1u);
      atomicAdd(&h[x[1]], 1u);
    };
    if (shift == 0u) {
      // (nearly always: the differences that matter fit 15 bits, so the signed numbers do as they are)
      const i16x2 base2 = signed_pair(base ^ 0x8000u), least2 = signed_pair(least), most2 = signed_pair(most);
#pragma clang loop unroll(full)
      for (int i = 0; i < IT; ++i) {
        if (8 * (i * T + 64 * wave) < nb) {                        // (a wave past the row's end has nothing to count)
          i16x2 x[4];                                              // (four at a time: a packed result cannot be used at once)
#pragma unroll
          for (int e = 0; e < 4; ++e) x[e] = __builtin_elementwise_sub_sat(k[i][e], base2);
#pragma unroll
          for (int e = 0; e < 4; ++e) x[e] = __builtin_elementwise_max(x[e], least2);
#pragma unroll
          for (int e = 0; e < 4; ++e) x[e] = __builtin_elementwise_min(x[e], most2);
#pragma unroll
          for (int e = 0; e < 4; ++e) add(__builtin_bit_cast(u16x2, x[e]));
        }
        fence_schedule();
      }
    } else {
      const u16x2 base2 = pair(base), shift2 = pair(shift), least2 = pair(least), most2 = pair(most);
#pragma clang loop unroll(full)
      for (int i = 0; i < IT; ++i) {
        if (8 * (i * T + 64 * wave) < nb) {
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const u16x2 x = __builtin_elementwise_sub_sat(__builtin_bit_cast(u16x2, __builtin_bit_cast(uint32_t, k[i][e]) ^ 0x80008000u), base2) >> shift2;
            add(__builtin_elementwise_min(__builtin_elementwise_max(x, least2), most2));
          }
        }
        fence_schedule();
      }
    }
    __syncthreads();
    uint32_t loc[PER], inside, beyond;
    uint32_t above = bins_above(at << rs, n << rs, loc, inside, beyond);
    if (first) krem = c - min(beyond, c);
    if (krem < 1u || krem > inside) {                              // not in the window: below it, or the sample misled
      lo = heavy && krem > inside ? heavy : 1u;
      last = lo == heavy ? 31u - (lo & 31u) : 0xfffeu;
      heavy = 0;
      clear();
      continue;
    }
    uint32_t top = above;
#pragma unroll
    for (int i = PER - 1; i >= 0; --i) {
      if (top < krem && top + loc[i] >= krem) res[2] = (uint32_t)(tid * PER + i) >> rs;
      top += loc[i];
    }
    __syncthreads();
    const uint32_t bin = (uint32_t)__builtin_amdgcn_readfirstlane((int)res[2]);
#pragma unroll
    for (int i = PER - 1; i >= 0; --i) {
      const uint32_t x = (uint32_t)(tid * PER + i);
      if (x >> rs == bin && (x + 1u) >> rs != bin) res[3] = krem - above;        // (the bin's last copy)
      above += loc[i];
    }
    __syncthreads();
    first = false;
    krem = (uint32_t)__builtin_amdgcn_readfirstlane((int)res[3]);
    lo += bin << shift;
    last = (1u << shift) - 1u;
    if (shift == 0) break;
    clear();
  }
  const uint32_t r = krem;                                         // of the tokens with key lo, the first r are kept

  // ---- two bits per token: 0 below, 1 equal, 2 above the threshold
  // Held between the two keys around the threshold's, a word's four numbers are added up as digits of 4 bits; what is too much is
  // the lower key in every digit. (There is no key above the highest.)
  const uint32_t under = lo - 1u, over = min(lo + 1u, 0xffffu);
  const i16x2 under2 = (i16x2)(short)(unsigned short)(under ^ 0x8000u), over2 = (i16x2)(short)(unsigned short)(over ^ 0x8000u);
  const u16x2 too_much = (u16x2)(unsigned short)((under ^ 0x8000u) * 0x1111u);
  u16x2 digit[3] = {(u16x2)16, (u16x2)256, (u16x2)4096};
#if defined(__AMDGCN__)
#pragma unroll
  for (int e = 0; e < 3; ++e) asm("" : "+s"(digit[e]));                // (a product and a sum are one instruction, a shift and a sum two)
#endif
  typedef uint16_t half_word __attribute__((may_alias));
  half_word *const codes16 = reinterpret_cast<half_word *>(codes);
#pragma clang loop unroll(full)
  for (int i = 0; i < IT; ++i) {
    u16x2 x[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) x[e] = __builtin_bit_cast(u16x2, __builtin_elementwise_max(k[i][e], under2));
#pragma unroll
    for (int e = 0; e < 4; ++e) x[e] = __builtin_bit_cast(u16x2, __builtin_elementwise_min(__builtin_bit_cast(i16x2, x[e]), over2));
    u16x2 d = x[1] * digit[0] + x[0];
    d = x[2] * digit[1] + d;
    d = x[3] * digit[2] + d;
    const uint32_t m = __builtin_bit_cast(uint32_t, d - too_much);
    const int w = i * T + tid;
    codes16[w + 2 * (w >> 5)] = (half_word)(m | m >> 14);
    fence_schedule();
  }
  __syncthreads();
  constexpr int CW = CODES / T;                                    // words per thread, consecutive
  static_assert(CW % 2 == 0, "two words make one");
  uint32_t w[CW], gt = 0, eq = 0;
#pragma unroll
  for (int x = 0; x < CW; ++x) {
    const int at = tid * CW + x;
    w[x] = codes[at + (at >> 4)];
    gt += (uint32_t)__builtin_popcount(w[x] & 0xaaaaaaaau);
    eq += (uint32_t)__builtin_popcount(w[x] & 0x55555555u);
  }
  uint32_t gt0, eq0, gts, eqs;
  scan2<T>(gt, eq, tot, lane, wave, gt0, eq0, gts, eqs);
  const uint32_t pos = gt0 + min(eq0, r);                          // this thread's first place in the list
  // its kept tokens, a bit each
  uint32_t mine = 0;
#pragma unroll
  for (int x = 0; x < CW; ++x) {
    const uint32_t e = w[x] & 0x55555555u, n = (uint32_t)__builtin_popcount(e);
    uint32_t keep = eq0 + n <= r ? e : 0u;
    if (n && eq0 < r && eq0 + n > r) {
      uint32_t rest = e;
      for (uint32_t q = eq0; q < r; ++q) {
        keep |= rest & (0u - rest);
        rest &= rest - 1u;
      }
    }
    eq0 += n;
    uint32_t y = ((w[x] >> 1) & 0x55555555u) | keep;
    mine += (uint32_t)__builtin_popcount(y);
    y = (y | y >> 1) & 0x33333333u;                                // the even bits next to each other
    y = (y | y >> 2) & 0x0f0f0f0fu;
    y = (y | y >> 4) & 0x00ff00ffu;
    y = (y | y >> 8) & 0x0000ffffu;
    if (x & 1) w[x >> 1] |= y << 16;
    else w[x >> 1] = y;
  }
#pragma unroll 1
  for (uint32_t base = 0; base < c; base += STAGE) {
    uint32_t p = pos;
    if (c <= (uint32_t)STAGE) {                        // (all of it at once: no place is looked at)
#pragma unroll
      for (int x = 0; x < CW / 2; ++x)
        for (uint32_t rest = w[x]; rest; rest &= rest - 1u, ++p) staged[p] = (stage_t)(32 * (tid * (CW / 2) + x) + __builtin_ctz(rest));
    } else if (p < base + STAGE && p + mine > base) {
#pragma unroll
      for (int x = 0; x < CW / 2; ++x)
        for (uint32_t rest = w[x]; rest; rest &= rest - 1u, ++p)
          if (p - base < (uint32_t)STAGE) staged[p - base] = (stage_t)(32 * (tid * (CW / 2) + x) + __builtin_ctz(rest));
    }
    __syncthreads();
    const uint32_t cnt = min(c - base, (uint32_t)STAGE);
    for (int ti = t0; ti < t1; ++ti) {
      int32_t *dst = A.indices + ((size_t)bt * A.Hq + target_head(A, ti)) * A.k + base;
      const uint32_t quads = cnt / 4;
      for (uint32_t i = tid; i < quads; i += T) {
        typedef stage_t stage4 __attribute__((ext_vector_type(4)));
        typedef int32_t i32x4_any __attribute__((ext_vector_type(4), aligned(4)));
        const stage4 x = *reinterpret_cast<const stage4 *>(&staged[4 * i]);
        *reinterpret_cast<i32x4_any *>(dst + 4 * i) = i32x4_any{(int32_t)x[0], (int32_t)x[1], (int32_t)x[2], (int32_t)x[3]};
      }
      if (tid < (int)(cnt & 3u)) dst[4 * quads + tid] = (int32_t)staged[4 * quads + tid];
    }
    __syncthreads();
  }
}

// T threads, IT 16-byte words per thread: rows of up to 8 * T * IT tokens, at least 8. Rows that a quarter of the words hold (of a
// tensor that is allocated for the longest sequence) are ranked by code for so many.
template <int T, int IT>
__global__ void __launch_bounds__(T, 4) select_row16_kernel(const SelectArgs A) {
  constexpr int TOK = 8 * T * IT, CODES = TOK / 16;
  typedef typename std::conditional<(TOK <= 65536), uint16_t, uint32_t>::type stage_t;
  __shared__ uint32_t codes[CODES + CODES / 16];                   // a word of padding after every 16
  __shared__ uint32_t h[ROW16_SLOTS];
  __shared__ __attribute__((aligned(16))) stage_t staged[ROW16_STAGE];
  __shared__ uint32_t tot[2 * T / 64];
  __shared__ uint32_t res[8];
  const int j = blockIdx.x, bt = blockIdx.y, row = bt * A.Hd + j;
  const int nb = __builtin_amdgcn_readfirstlane(row_len(A, bt));
  const uint32_t c = (uint32_t)min(A.kh[j], nb);
  write_tail<T>(A, bt, j, c);
  if (c == 0 || target_off(A, j) == target_off(A, j + 1)) return;
  if (c == (uint32_t)nb) {                                         // every token is kept
    for (int ti = target_off(A, j); ti < target_off(A, j + 1); ++ti)
      for (int i = threadIdx.x; i < nb; i += T) A.indices[((size_t)bt * A.Hq + target_head(A, ti)) * A.k + i] = i;
    return;
  }
  if constexpr (IT >= 16) {
    if (nb <= TOK / 4) return rank_row16<T, IT / 4>(A, row, nb, c, codes, h, staged, tot, res);
  }
  rank_row16<T, IT>(A, row, nb, c, codes, h, staged, tot, res);
}

}  // namespace

// Rows of 8 to 131072 tokens of one bf16 score each.
static hipError_t launch_select_row16(const SelectArgs &a, hipStream_t s) {
  const int64_t rows = (int64_t)a.B * a.Hd;
  if (rows == 0) return hipSuccess;
  if (a.N < 8 || a.N > SEL_ROW16_N) return hipErrorInvalidValue;
  const dim3 grid((unsigned)a.Hd, (unsigned)a.B);
  if (a.N <= 8192) STS_LAUNCH((select_row16_kernel<256, 4>), grid, dim3(256), 0, s, a);
  else if (a.N <= 16384) STS_LAUNCH((select_row16_kernel<256, 8>), grid, dim3(256), 0, s, a);
  else if (a.N <= 32768) STS_LAUNCH((select_row16_kernel<256, 16>), grid, dim3(256), 0, s, a);
  else if (a.N <= 65536) STS_LAUNCH((select_row16_kernel<512, 16>), grid, dim3(512), 0, s, a);
  else STS_LAUNCH((select_row16_kernel<1024, 16>), grid, dim3(1024), 0, s, a);
  return sts_take_launch_status();
}

// Rows of 4 to 32768 tokens, of up to 65536 with one probability per token in calls of up to 512 rows (16 rows of 33001 tokens 16.9 us with
// twelve quads per thread, 18.6 with sixteen). Calls of up to 512 rows get 1024 threads per row (latency: 256 rows of 16384 tokens 25 us
// with 256 threads per row), others as few as hold the row in 64 registers per thread (several workgroups per CU: 4096
// such rows 128 us; one workgroup per CU took 290), in 32 where the scores of up to 16384 tokens are added up (1024 rows of 16384
// with five scores 64.2 us, 68.6).
// (Rows of block sums where a page holds several tokens: kernels that turn lengths in tokens into blocks, see ranked_len.)
hipError_t launch_select_row(const SelectArgs &a, hipStream_t s) {
  const int64_t rows = (int64_t)a.B * a.Hd;
  if (rows == 0) return hipSuccess;
  if (a.rowpass_threads == SEL_ROW16) return launch_select_row16(a, s);
  const int N = a.N;
  const dim3 grid((unsigned)a.Hd, (unsigned)a.B);
  // one probability per token: nothing is added up, and all of a thread's quads are in flight together
  const bool one = a.Tq == 1 && a.kind == STS_SCORES_PROBS;
  if (N < 4 || N > (one && a.page <= 1 && rows <= 512 ? SEL_ROW_N : SEL_SMALL_N)) return hipErrorInvalidValue;
#define STS_SHORT(T, IT) \
  do { \
    if (a.page > 1) STS_LAUNCH((short_select_blocks_kernel<T, IT>), grid, dim3(T), 0, s, a); \
    else if (one) STS_LAUNCH((short_select_row_kernel<T, IT>), grid, dim3(T), 0, s, a); \
    else STS_LAUNCH((short_select_row_scores_kernel<T, IT>), grid, dim3(T), 0, s, a); \
  } while (0)
#define STS_ROW(T, IT, T5, IT5) \
  do { \
    if (a.page > 1) STS_LAUNCH((select_blocks_kernel<T, IT>), grid, dim3(T), 0, s, a); \
    else if (one) STS_LAUNCH((select_row_kernel<T, IT>), grid, dim3(T), 0, s, a); \
    else STS_LAUNCH((select_row_scores_kernel<T5, IT5>), grid, dim3(T5), 0, s, a); \
  } while (0)
  if (rows <= 512) {
    if (N <= 4096) STS_SHORT(1024, 1);
    else if (N <= 8192) STS_SHORT(1024, 2);
    else if (N <= 16384) STS_ROW(1024, 4, 1024, 4);
    else if (N <= 32768) STS_ROW(1024, 8, 1024, 8);
    else if (N <= 49152) STS_LAUNCH((select_row_long_kernel<1024, 12>), grid, dim3(1024), 0, s, a);
    else STS_LAUNCH((select_row_long_kernel<1024, 16>), grid, dim3(1024), 0, s, a);
  } else if (N <= 4096) {
    STS_SHORT(256, 4);
  } else if (N <= 8192) {
    STS_ROW(256, 8, 256, 8);
  } else if (N <= 16384) {
    STS_ROW(256, 16, 512, 8);
  } else {
    STS_ROW(512, 16, 512, 16);
  }
#undef STS_SHORT
#undef STS_ROW
  return sts_take_launch_status();
}
