// Short rows (gfx950): a row that one workgroup's registers hold, ranked in one launch. Every thread
// loads and aggregates the row's quads that are its own (same fp32 order as everywhere) and keeps the
// keys; nothing is read twice. The threshold is found among keys counted into 2048 bins that divide
// the range in question: first the row's own key range, then, if the bin of the threshold still holds more
// than a few keys, that bin. Long rows count only a sixteenth of their keys at first, which gives a band
// around the threshold that is listed and counted (and if that fails, all keys, as for short rows).
// The kept tokens are bits in LDS; the list is the bits read in order.
//
// What bounds it: for thousands of rows (head mapping: 6144 rows of 16K tokens, 403 MB) memory and vector
// instructions alike; several small workgroups per CU hide each other's latencies. For few rows latency.
#include "select_util.h"

namespace {

constexpr int ROW_CAND = 64;              // keys of the threshold's bin that are ranked against each other

template <int T>
__device__ __forceinline__ void row_min_max(uint32_t &lo, uint32_t &hi, uint32_t *red) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    lo = min(lo, (uint32_t)__shfl_xor((int)lo, off, 64));
    hi = max(hi, (uint32_t)__shfl_xor((int)hi, off, 64));
  }
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

// T threads, IT quads per thread: rows of up to 4 * T * IT tokens. SAMPLE: IT is a multiple of 4.
template <int T, int IT, bool SAMPLE>
__global__ void __launch_bounds__(T, SAMPLE ? 4 : 1) select_row_kernel(const SelectArgs A) {
  constexpr int TOK = 4 * T * IT;
  constexpr int LIST = SAMPLE ? TOK * 3 / 16 : ROW_CAND;           // band tokens
  constexpr int STAGE = TOK / 8 > 1024 ? TOK / 8 : 1024;           // list entries staged per round
  __shared__ uint32_t bits[TOK / 32];
  __shared__ uint32_t h[SEL_BINS];
  __shared__ __attribute__((aligned(8))) uint32_t store[2 * LIST > STAGE ? 2 * LIST : STAGE];
  __shared__ uint32_t tmp[T / 64 + 2];
  __shared__ uint32_t red[2 * T / 64];
  __shared__ uint32_t ctr[4];
  u32x2 *const list = reinterpret_cast<u32x2 *>(store);            // key, token
  const int row = blockIdx.x, tid = threadIdx.x, lane = tid & 63;
  const int bt = row / A.Hd, j = row % A.Hd;
  const int nb = __builtin_amdgcn_readfirstlane(row_len(A, bt));
  const uint32_t c = (uint32_t)min(A.kh[j], nb);
  const int t0 = A.targets.off[j], t1 = A.targets.off[j + 1];
  write_tail<T>(A, bt, j, c);
  float *out = A.agg ? A.agg + (size_t)row * A.N : nullptr;
  const bool ranked = c > 0 && t0 != t1;
  if (!ranked && !out) return;
  const AggRow R = agg_row(A, row);
  for (int i = tid; i < SEL_BINS; i += T) h[i] = 0u;
  if (tid < 4) ctr[tid] = 0u;

  // ---- the row: thread tid owns the quads tid, tid + T, ... A position past the row's valid length holds INT_MIN,
  // which no token does.
  int v[IT][4];
  int any = 0;
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
  if constexpr (T == 1024) {
    // Few quads: their score rows are in flight together. Up to four by code for each number of rows (256 rows of 16384
    // tokens 16.9 us, 18.7 with branches between the rows), eight with branches: that kernel was 305 KB (256 rows of 30000
    // tokens, 5 scores: 39.8 us, 48.7 with the caches flushed; now 40.5 and 44.6).
    auto quads = [&](auto bf16) {
#pragma clang loop unroll(full)
      for (int i = 0; i < IT; ++i) {
        const int n = 4 * (i * T + tid);
        const bool inside = 4 * (i + 1) * T <= R.N;
        if constexpr (IT == 8) {
          take(i, agg_quad_any<decltype(bf16)::value>(R, n, inside));
        } else {
          const int at = min(n, R.N - 4);
          const f32x4 y = agg_quad(R, at);
          take(i, inside ? y : shifted_quad(y, n - at));
        }
      }
    };
    if (IT < 8 || R.bf16) quads(std::true_type{});     // (the type matters for the form with branches only)
    else quads(std::false_type{});
  } else {
    // many quads: one score row at a time, all quads of it in flight together (same order of additions per token)
    f32x4 acc[IT];
    auto rows = [&](auto bf16) {
      typedef ScoreLoad<f32x4, decltype(bf16)::value> SL;
#pragma unroll 1
      for (int q = 0; q < R.Tq; ++q) {
        const float l = R.logits ? R.L[q] : 0.f;
#pragma clang loop unroll(full)
        for (int i = 0; i < IT; ++i) {
          f32x4 p = SL::widen(SL::load(R, q, min(4 * (i * T + tid), R.N - 4)));
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
      }
    };
    if (R.bf16) rows(std::true_type{});
    else rows(std::false_type{});
#pragma clang loop unroll(full)
    for (int i = 0; i < IT; ++i) {
      if (4 * (i + 1) * T > R.N) {                     // the row's end: the quad was read where it still fits
        const int n = 4 * (i * T + tid), d = n - min(n, R.N - 4);
        const f32x4 y = acc[i];
        acc[i][0] = d == 0 ? y[0] : d == 1 ? y[1] : d == 2 ? y[2] : y[3];
        acc[i][1] = d == 0 ? y[1] : d == 1 ? y[2] : y[3];
        acc[i][2] = d == 0 ? y[2] : y[3];
      }
      take(i, acc[i]);
    }
  }
  if (!ranked) return;
  if (ballot64(any < 0)) {                             // negative scores in this wave
#pragma clang loop unroll(full)
    for (int i = 0; i < IT; ++i)
#pragma unroll
      for (int e = 0; e < 4; ++e) v[i][e] = max(ordered(v[i][e]), (int)0x80000001);
  }
  if (nb < TOK) {
#pragma clang loop unroll(full)
    for (int i = 0; i < IT; ++i)
#pragma unroll
      for (int e = 0; e < 4; ++e) v[i][e] = 4 * (i * T + tid) + e < nb ? v[i][e] : (int)0x80000000;
  }

  // the part of the row's keys that is counted: all, or (sampled) one of sixteen, from every fourth quad of a thread
  auto each = [&](bool sampled, auto f) {
    if (SAMPLE && sampled) {
#pragma clang loop unroll(full)
      for (int i = 0; i < IT; ++i)
        if ((i & 3) == (tid & 3)) {
          const int e = (tid >> 2) & 3;
          int s = 0;                                   // (masks: a choice among array elements would put the array in memory)
#pragma unroll
          for (int q = 0; q < 4; ++q) s |= v[i][q] & (e == q ? -1 : 0);
          f(s, 4 * (i * T + tid) + e);
        }
    } else {
#pragma clang loop unroll(full)
      for (int i = 0; i < IT; ++i)
#pragma unroll
        for (int e = 0; e < 4; ++e) f(v[i][e], 4 * (i * T + tid) + e);
    }
  };
  // the bin of the rank-th largest of the keys counted in h, and what is left of the rank in it
  auto find = [&](uint32_t rank, uint32_t &bin, uint32_t &left) {
    find_digit<SEL_BINS, T, true>(h, rank, tmp, bin, left);
    bin = (uint32_t)__builtin_amdgcn_readfirstlane((int)bin);
    left = (uint32_t)__builtin_amdgcn_readfirstlane((int)left);
  };

  // ---- keys in question: lo .. lo + last; G keys lie above them, `listed` of them (if any) are in the list
  // (sampled only if the band that the sample is expected to give fits the list with room to spare)
  const bool sampled = SAMPLE && nb > TOK / 4 && 32.f * (5.f * sqrtf((float)c * 0.0625f) + 4.f) <= 0.75f * LIST;
  uint32_t kmin = 0xffffffffu, kmax = 0u;
  each(sampled, [&](int s, int) {
    if (s != (int)0x80000000) {
      kmin = min(kmin, key_of_ordered(s));
      kmax = max(kmax, key_of_ordered(s));
    }
  });
  row_min_max<T>(kmin, kmax, red);
  uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)kmin), last = (uint32_t)__builtin_amdgcn_readfirstlane((int)(kmax - kmin));
  uint32_t krem = c, listed = 0;
  bool from_list = false;
  if (SAMPLE && sampled) {
    const int shift = max(0, 32 - __clz((int)last) - 11);
    each(true, [&](int s, int) {
      if (s != (int)0x80000000) {
        atomicAdd(&h[(key_of_ordered(s) - lo) >> shift], 1u);
      }
    });
    __syncthreads();
    uint32_t ns;
    {
      constexpr int PER = SEL_BINS / T;
      uint32_t sum = 0;
#pragma unroll
      for (int i = 0; i < PER; ++i) sum += h[tid * PER + i];
      (void)block_excl_scan<T, true>(sum, tmp, ns);
      ns = (uint32_t)__builtin_amdgcn_readfirstlane((int)ns);
    }
    // 5 standard deviations of the sample count, as if the tokens were independent: a stretch of heavy tokens longer
    // than 16 is sampled more exactly than that
    const uint32_t cs = max(1u, min(ns, (uint32_t)((uint64_t)c * ns / (uint32_t)nb)));
    const uint32_t margin = (uint32_t)(5.f * sqrtf((float)cs)) + 4u;
    uint32_t lo_bin = 0, hi_bin = SEL_BINS - 1, unused;
    const bool haveL = cs + margin <= ns, haveU = cs > margin;
    if (haveL) find(cs + margin, lo_bin, unused);
    if (haveU) find(cs - margin, hi_bin, unused);
    const uint64_t u = (uint64_t)lo + ((uint64_t)(hi_bin + 1u) << shift);
    const uint32_t L = haveL ? lo + (lo_bin << shift) : 1u;            // (key 0 is no token's)
    const uint32_t U1 = haveU && u <= 0xffffffffull ? (uint32_t)u - 1u : 0xffffffffu;   // last key of the band
    // the band is listed, what lies above it counted
    const int sL = ordered_of_key(L), sU1 = ordered_of_key(U1);
    uint32_t G = 0;                                    // wave-uniform
#pragma clang loop unroll(full)
    for (int i = 0; i < IT; ++i) {
      uint64_t bd[4];
      bool in[4];
      uint32_t held = 0;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const bool sure = v[i][e] > sU1;
        in[e] = !sure && v[i][e] >= sL;
        G += (uint32_t)__builtin_popcountll(ballot64(sure));
        bd[e] = ballot64(in[e]);
        held += (uint32_t)__builtin_popcountll(bd[e]);
      }
      uint32_t at = 0;
      if (lane == 0) at = atomicAdd(&ctr[0], held);
      at = (uint32_t)__builtin_amdgcn_readfirstlane((int)at);
      if (at + held <= (uint32_t)LIST) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          if (in[e]) list[lanes_before(bd[e], at)] = u32x2{key_of_ordered(v[i][e]), (uint32_t)(4 * (i * T + tid) + e)};
          at += (uint32_t)__builtin_popcountll(bd[e]);
        }
      }
    }
    if (lane == 0) atomicAdd(&ctr[1], G);
    for (int i = tid; i < SEL_BINS; i += T) h[i] = 0u;
    __syncthreads();
    const uint32_t M = (uint32_t)__builtin_amdgcn_readfirstlane((int)ctr[0]);
    G = (uint32_t)__builtin_amdgcn_readfirstlane((int)ctr[1]);
    if (G < c && G + M >= c && M <= (uint32_t)LIST) {
      from_list = true;
      listed = M;
      krem = c - G;
      lo = L;
      last = U1 - L;
    } else {                                           // the sample misled: all keys are counted
      kmin = 0xffffffffu;
      kmax = 0u;
      each(false, [&](int s, int) {
        if (s != (int)0x80000000) {
          kmin = min(kmin, key_of_ordered(s));
          kmax = max(kmax, key_of_ordered(s));
        }
      });
      __syncthreads();
      row_min_max<T>(kmin, kmax, red);
      lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)kmin);
      last = (uint32_t)__builtin_amdgcn_readfirstlane((int)(kmax - kmin));
    }
  }
  int shift = max(0, 32 - __clz((int)last) - 11);
  uint32_t in_bin;
#pragma unroll 1
  for (;;) {
    if (SAMPLE && from_list) {
      for (uint32_t i = tid; i < listed; i += T) {
        const uint32_t k = list[i][0] - lo;
        if (k <= last) atomicAdd(&h[k >> shift], 1u);
      }
    } else {
      each(false, [&](int s, int) {
        const uint32_t k = key_of_ordered(s) - lo;
        if (k <= last && s != (int)0x80000000) atomicAdd(&h[k >> shift], 1u);
      });
    }
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
    if (SAMPLE && from_list) {
      for (uint32_t i = tid; i < listed; i += T) add(list[i][0]);
    } else {
      each(false, [&](int s, int) {
        if (s != (int)0x80000000) add(key_of_ordered(s));
      });
    }
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
  // of their own (the list's memory is free)
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
      int32_t *dst = A.indices + ((size_t)bt * A.Hq + A.targets.tgt[ti]) * A.k + base;
      for (uint32_t i = tid; i < cnt; i += T) dst[i] = staged[i];
    }
    __syncthreads();
  }
}

}  // namespace

// Rows of 4 to 32768 tokens. Calls of up to 512 rows get 1024 threads per row (latency: 256 rows of 16384 tokens 25 us
// with 256 threads per row), others as few as hold the row in 64 registers per thread (several workgroups per CU: 4096
// such rows 128 us; one workgroup per CU took 290).
hipError_t launch_select_row(const SelectArgs &a, hipStream_t s) {
  const int64_t rows = (int64_t)a.B * a.Hd;
  if (rows == 0) return hipSuccess;
  if (a.N < 4 || a.N > SEL_SMALL_N) return hipErrorInvalidValue;
  const dim3 grid((unsigned)rows);
  if (rows <= 512) {
    const dim3 block(1024);
    if (a.N <= 4096) STS_LAUNCH((select_row_kernel<1024, 1, false>), grid, block, 0, s, a);
    else if (a.N <= 8192) STS_LAUNCH((select_row_kernel<1024, 2, false>), grid, block, 0, s, a);
    else if (a.N <= 16384) STS_LAUNCH((select_row_kernel<1024, 4, true>), grid, block, 0, s, a);
    else STS_LAUNCH((select_row_kernel<1024, 8, true>), grid, block, 0, s, a);
  } else if (a.N <= 4096) {
    STS_LAUNCH((select_row_kernel<256, 4, false>), grid, dim3(256), 0, s, a);
  } else if (a.N <= 8192) {
    STS_LAUNCH((select_row_kernel<256, 8, true>), grid, dim3(256), 0, s, a);
  } else if (a.N <= 16384) {
    STS_LAUNCH((select_row_kernel<256, 16, true>), grid, dim3(256), 0, s, a);
  } else {
    STS_LAUNCH((select_row_kernel<512, 16, true>), grid, dim3(512), 0, s, a);
  }
  return sts_take_launch_status();
}
