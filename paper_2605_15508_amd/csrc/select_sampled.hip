// Sampled selection (gfx950): rows longer than one workgroup's LDS holds, read ONCE.
//
// A row is cut into as many parts as give every CU a workgroup (one part when there are rows enough);
// one 1024-thread workgroup per part:
//  1. Sample. Runs of 128 bytes of the row's scores (the whole row's, not only the part's), one in
//     every S, are aggregated in the usual fp32 order and counted into 2048 bins that divide the
//     sample's own key range. From them come two keys L < U between which the row's threshold lies
//     unless the sample is 5 standard deviations off; the deviation is the sample's own, the spread
//     of the counts of large keys over its runs, so rows whose heavy tokens sit next to each other
//     get the wider band that they need. Every part of a row samples the same tokens and finds the
//     same L and U. The part's first loads are on their way meanwhile.
//  2. The pass over the part, four loads in flight per thread all the time. A token whose key is >= U
//     is certainly kept: a bit in LDS. One in [L, U), a few per cent of the row, goes to the
//     band list in LDS with its key. Nothing else is remembered.
//  3. The threshold. The parts exchange a histogram of their bands (512 bins over [L, U)) and their
//     counts, then the keys of the one bin that holds the threshold, 64 at most (where that bin holds
//     more, another histogram narrows it first). That gives every part the exact threshold key T, the
//     number r of tokens equal to T that are kept, and the number of kept tokens in earlier parts.
//  4. Band tokens above T get their bit, of those equal to T the r lowest do, and the list is the bits
//     read in order.
//
// Exchange protocol: the words are zeroed by a small kernel launched before this one. Every 64-bit word
// carries its own top bit as "written" (a device-scope store of 8 aligned bytes: the word arrives
// whole), so one memory round trip per exchange is all the parts wait for each other, without
// fences. The wait is bounded: a workgroup that runs out of polls ranks the row by plain passes over
// the scores and writes its own part of the list from that (rank_by_passes), so every workgroup exits
// whatever the others do; a row's parts have neighbouring workgroup ids and start together.
//
// The result never depends on the sample: if the counts show that the threshold lies outside [L, U),
// every part goes by plain passes likewise. Where a part's list has no room for its band (heavy tokens next to each
// other, all in that part), what does not fit is only counted, and the part reads its own tokens once more when the
// threshold's bin is known: 16 rows of 1M tokens, the last 5% of them heavy 113 us, the first eighth after a third
// 114, against 1955 and 1692 by plain passes of every part. Values that repeat do not make the list overflow:
// only two can hold more of the sample than the margins, the lowest key of the band and its
// highest (any other lies between the two ranks), and where the sample says that one does (zeros, levels, a
// saturated score), a bitmap holds its tokens and not the list. 16 rows of 1M tokens, a budget at the edge of the
// zeros: 118 us, 3870 by plain passes; 64 rows of 128K: 74, 520; a constant row with a small budget 58, 435.
//
// What bounds it (64 rows of 128K tokens, 5 fp32 scores each, 4 parts per row, 168 MB): the sample and the pass
// together 29 us (168 MB and 21 MB of samples, mostly from the last-level cache: the rate of the memory), then latency:
// 5 us for the histogram exchange, 3.5 us for the keys, 3 us for bits and list; kernel 45 us on scores that the
// last-level cache holds, 47 to 50 on new ones. Histograms of all keys at three digit levels, with the
// part's keys in LDS, took 54: the same 29 us, then 20 us for three levels and 5 us for the list. 16 rows of 1M
// tokens (335 MB, 16 parts per row): 78 us against 122 for five kernels that stored the aggregate and read it
// three times. Rows of one score per token are bound by vector instructions instead (about 60 per 256 tokens
// and wave), those of scaled logits by the exponentials. A few short rows are bound by the ranking of the sample
// (7 us of 25 in the kernel for 16 rows of 32768 tokens, which took 1.4 us less with the histograms).
#include "select_util.h"

namespace {

constexpr int SMP_THREADS = 1024;
constexpr int SMP_WAVES = SMP_THREADS / 64;
constexpr int SMP_GROUP = 256;            // tokens per wave step: four per lane
constexpr int SMP_HIST = 512;             // bins of an exchanged histogram, two per word
// Histograms that narrow the keys in question down to one: 9 bits each, after a first one whose last bin may be open
// upwards and hold any 32-bit range. With one less, more than 64 equal scores above all that the sample saw (saturated
// scores, 16 rows of 33001 tokens, 256 kept) went by plain passes: 105 us instead of 52.
constexpr int SMP_ROUNDS = 5;
// Loads in flight per thread in the pass. Its code is there once for each (the ring's place has to be known where a load is waited for): with
// eight the kernel was 74 KB, more than the instruction cache holds. us with 8, 6, 4, 3 and 2: 64 rows of 128K tokens, five scores 48.1,
// 47.0, 46.8, 47.1, 47.2; 16 of 1M 77.3, 76.6, 76.0, 75.2, 78.2; 128 of 128K, one score, read anew 42.7, 41.0, 39.6, 39.3, 39.0; 128 of 50000,
// eight bf16 scores (loads of half the size) 41.9, 42.2, 41.3, 45.0, 45.7. (10 and 12: 42.1 and 46.4 where 8 takes 40.5.)
constexpr int SMP_FLIGHT = 4;
constexpr int SMP_CAND = 64;              // keys of the threshold's bin that are exchanged one by one
constexpr int SMP_G_WORD = SMP_ROUNDS * SMP_HIST / 2, SMP_CAND_WORD = SMP_G_WORD + 8;
static_assert(SMP_CAND_WORD + SMP_CAND == SMP_WORDS, "layout of a part's exchange words");
constexpr unsigned long long SMP_VALID = 1ull << 63;

// Which runs of a row of nb ranked tokens are sampled: one in every S, at a scattered place of its
// period (a fixed stride of 4 KB and more lands on a few memory channels only: the sample's loads
// took 6.5 and, at 1M tokens, 12 us more). About 4096 keys: at a tenth of the row kept the band is then
// about 5% of a 128K row. 8192 for rows beyond 256K tokens, for workgroups with more than 128K tokens, and where a
// workgroup holds more than 64K tokens and an eighth of the row or more is kept: with 4096 the band of half of such a
// part overflowed its list (256 rows of 128K tokens 277 us, with 8192 83). Smaller budgets have room enough and save the
// larger sample's 2 to 4 us.
struct SamplePlan {
  int S, runs;                                         // S: a power of two
  __device__ __forceinline__ int start(int i, int run) const {       // first token of sampled run i
    return (i * S + (int)((((uint32_t)i * 0x9e3779b1u) >> 16) & (uint32_t)(S - 1))) * run;
  }
};
__device__ __forceinline__ SamplePlan sample_plan(int nb, int run, int target) {
  SamplePlan p;
  const int row_runs = (nb + run - 1) / run;
  int sh = 0;
  while (((row_runs + (1 << sh) - 1) >> sh) * run > target) ++sh;
  p.S = 1 << sh;
  p.runs = row_runs >> sh;                             // (at least one: S is at most half the runs here)
  return p;
}

// One quad of one score row as loaded.
template <bool BF16>
using RawQuad = typename ScoreLoad<f32x4, BF16>::raw;

// the band that the sample gives: keys L .. L + last, whether there is an upper edge, and how far the sample's keys
// reach (without an upper edge the band is the top of the row: its histogram is laid out for the sample's
// keys, and what lies above them goes to the last bin)
// heavyL, heavyU: the band's lowest or highest key is a single value that much of the row shares (zeros, a saturated score,
// one of a few levels); its tokens go to a bitmap of their own and not to the list.
struct Band {
  uint32_t L, last, span;
  bool haveU, heavyL, heavyU;
};

// Ranks the sampled quads (up to QT per thread, `acc` their aggregated scores). h: SEL_BINS words, zeroed.
template <int QT>
__device__ __forceinline__ Band sample_band(const SamplePlan &sp, int run, int nb, uint32_t c, const int (&pos)[QT],
                                            const f32x4 (&acc)[QT], uint32_t *h, uint32_t *tmp, uint32_t *red, uint32_t *found) {
  constexpr int T = SMP_THREADS;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int rq = run >> 2, nsq = sp.runs * rq;
  auto uniform = [](uint32_t v) { return (uint32_t)__builtin_amdgcn_readfirstlane((int)v); };
  uint32_t key[QT][4];
  bool ok[QT][4];
#pragma unroll
  for (int x = 0; x < QT; ++x)
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      key[x][e] = key_of(acc[x][e]);
      ok[x][e] = tid + x * T < nsq && pos[x] + e < nb;
    }
  // lowest and highest of the sampled keys in from .. to (there is one); a barrier has to come before red is written again
  auto range_of = [&](uint32_t from, uint32_t to, uint32_t &lowest, uint32_t &highest) {
    uint32_t mn = 0xffffffffu, mx = 0u;
#pragma unroll
    for (int x = 0; x < QT; ++x)
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (ok[x][e] && key[x][e] - from <= to - from) {
          mn = min(mn, key[x][e]);
          mx = max(mx, key[x][e]);
        }
    wave_min_max(mn, mx);
    if (lane == 0) {
      red[2 * wave] = mn;
      red[2 * wave + 1] = mx;
    }
    __syncthreads();
#pragma unroll
    for (int w = 0; w < T / 64; ++w) {
      mn = min(mn, red[2 * w]);
      mx = max(mx, red[2 * w + 1]);
    }
    lowest = uniform(mn);
    highest = uniform(mx);
  };
  // counts the sampled keys base .. base + range into bins of 2^shift keys (h is zeroed before if `again`); `above`
  // keys of the sample, `over` of them above the window, lie in higher bins than the thread's own two
  uint32_t h0, h1, above;
  auto count = [&](bool again, uint32_t base, uint32_t range, int shift, uint32_t over) {
    if (again) {
      for (int i = tid; i < SEL_BINS; i += T) h[i] = 0u;
      __syncthreads();
    }
#pragma unroll
    for (int x = 0; x < QT; ++x)
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (ok[x][e] && key[x][e] - base <= range) atomicAdd(&h[(key[x][e] - base) >> shift], 1u);
    __syncthreads();
    // thread t owns bins 2t and 2t + 1
    h0 = h[2 * tid];
    h1 = h[2 * tid + 1];
    uint32_t in_window;
    const uint32_t excl = block_excl_scan<T, true>(h0 + h1, tmp, in_window);
    above = over + in_window - excl - (h0 + h1);
    return uniform(in_window);
  };
  // the bin of the rank-th largest: found[3 * slot ..] = the bin, keys above it, keys in it
  auto locate = [&](uint32_t rank, int slot) {
    if (above < rank && above + h1 >= rank) {
      found[3 * slot] = 2 * tid + 1;
      found[3 * slot + 1] = above;
      found[3 * slot + 2] = h1;
    } else if (above + h1 < rank && above + h1 + h0 >= rank) {
      found[3 * slot] = 2 * tid;
      found[3 * slot + 1] = above + h1;
      found[3 * slot + 2] = h0;
    }
  };
  // An edge of the band: the rank-th largest sampled key, known to lie among the keys lo .. hi, of which the sample
  // holds cnt, with `above` sampled keys above hi. Values far from the rest and values that repeat leave many
  // tokens there: as long as that is so, the keys are counted again, within the range that they really have.
  struct Edge {
    uint32_t rank, lo, hi, cnt, above;
    bool heavy;
  };
  auto refine = [&](Edge &g, uint32_t most) {
#pragma unroll 1
    while (g.cnt > most) {
      __syncthreads();
      range_of(g.lo, g.hi, g.lo, g.hi);
      g.heavy = g.lo == g.hi;
      if (g.heavy) return;
      const int shift = max(0, 32 - __clz((int)(g.hi - g.lo)) - 11);
      (void)count(true, g.lo, g.hi - g.lo, shift, g.above);
      locate(g.rank, 0);
      __syncthreads();
      g.lo += uniform(found[0]) << shift;
      g.hi = g.lo + min(g.hi - g.lo, (1u << shift) - 1u);
      g.above = uniform(found[1]);
      g.cnt = uniform(found[2]);
    }
  };
  // Bins of 2^shift keys over the window base .. base + range, which is the sample's own key range at first.
  // Rows with values far from the rest (exact zeros, negative scores) make those bins coarse and the band
  // with them far wider than the margin; the window is then narrowed to the band until it is not, at
  // the last to a single key.
  uint32_t base, highest;
  range_of(0u, 0xffffffffu, base, highest);
  uint32_t range = highest - base, over = 0;           // over: sampled keys above the window
  uint32_t ns = 0, cs = 0, margin = 0;
  bool haveL = false, haveU = false;                   // (an edge outside the sample, or where the last key is all there is)
  Edge edge[2] = {{0u, 0u, 0u, 0u, 0u, false}, {0u, 0xffffffffu, 0xffffffffu, 0u, 0u, false}};
  Edge &lower = edge[0], &upper = edge[1];
#pragma unroll 1
  for (bool again = false;; again = true) {
    const int shift = max(0, 32 - __clz((int)range) - 11);                   // range >> shift < 2048
    const uint32_t in_window = count(again, base, range, shift, over);
    if (ns == 0u) {                                    // the first window is the whole sample
      ns = in_window;
      cs = expected_rank(c, ns, nb);
    }
    margin = 0;                                        // (S == 1: the sample is the row)
    if (sp.S > 1) {
      locate(cs, 0);
      __syncthreads();
      const uint32_t centre = base + (found[0] << shift);
      // Keys from the centre on, per run; their spread over the runs is what the rank estimate's is made of
      // (differences of neighbouring runs, as for any systematic sample: a row that changes slowly, or has one
      // long stretch of heavy tokens, is sampled far more exactly than the runs' plain variance says).
      uint32_t sq = 0;
#pragma unroll
      for (int x = 0; x < QT; ++x) {
        uint32_t n = 0;
#pragma unroll
        for (int e = 0; e < 4; ++e) n += (ok[x][e] && key[x][e] >= centre) ? 1u : 0u;
        // a run's quads are 8 or 16 lanes, whose sum its first lane gets
        n += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)n, 0x101, 0xf, 0xf, true);      // row_shl:1
        n += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)n, 0x102, 0xf, 0xf, true);      // row_shl:2
        n += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)n, 0x104, 0xf, 0xf, true);      // row_shl:4
        if (rq == 16) n += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)n, 0x108, 0xf, 0xf, true);
        const int d = (int)n - __shfl_down((int)n, rq, 64);
        sq += (lane & (rq - 1)) == 0 && lane + rq < 64 && tid + x * T + rq < nsq ? (uint32_t)(d * d) : 0u;
      }
      const uint32_t sum_sq = block_sum1<T>(sq, red);
      const float pairs = (float)(64 - rq) / 64.f;     // share of the neighbouring pairs that lie in one wave
      margin = uniform((uint32_t)(5.f * sqrtf(fmaxf(0.5f * (float)sum_sq / pairs, (float)cs))) + 4u);
    }
    // an edge that lies outside the window stays what it was
    const bool inL = cs + margin <= over + in_window, inU = cs > margin + over;
    if (inL) locate(cs + margin, 1);
    if (inU) locate(cs - margin, 2);
    __syncthreads();
    const uint32_t lo_bin = uniform(inL ? found[3] : 0u), hi_bin = uniform(inU ? found[6] : range >> shift);
    if (inL) {
      haveL = true;
      lower = {cs + margin, base + (lo_bin << shift), 0u, uniform(found[5]), uniform(found[4]), false};
      lower.hi = lower.lo + min(base + range - lower.lo, (1u << shift) - 1u);
    }
    if (inU) {
      haveU = true;
      upper = {cs - margin, base + (hi_bin << shift), 0u, uniform(found[8]), uniform(found[7]), false};
      upper.hi = upper.lo + min(base + range - upper.lo, (1u << shift) - 1u);
    }
    const uint32_t upto = inL ? lower.above + lower.cnt : over + in_window, beyond = inU ? upper.above : over;
    if (shift == 0 || hi_bin - lo_bin >= 64u || upto - beyond <= 4u * margin + 64u) break;
    const uint32_t top = inU ? upper.hi : base + range;
    base = inL ? lower.lo : base;
    range = top - base;
    over = beyond;
    if (lo_bin == hi_bin) {
      range_of(base, top, base, range);
      range -= base;
      if (range == 0u) break;                          // one value: both edges lie in it
    }
  }
  // (S == 1: the sample is the row, and the list holds all of that)
  if (sp.S > 1 && (haveL ? lower.above + lower.cnt : ns) - (haveU ? upper.above : 0u) > 4u * margin + 64u) {
    if (haveL) refine(lower, margin + 16u);
    if (haveU) refine(upper, margin + 16u);
  }
  Band b = {max(haveL ? lower.lo : 0u, 1u), 0u, 0u, false, false, false};   // (0 marks what is no token)
  b.haveU = haveU && upper.hi != 0xffffffffu;
  b.last = (b.haveU ? upper.hi : 0xffffffffu) - b.L;
  b.heavyL = lower.heavy;
  b.heavyU = upper.heavy && b.haveU && b.last != 0u;
  b.span = b.haveU ? b.last : max(highest, b.L) - b.L;
  return b;
}

// TOK: tokens a workgroup can hold bits of; CAP: entries of its band list.
template <bool BF16, int TOK, int CAP>
__global__ void __launch_bounds__(SMP_THREADS) select_sampled_kernel(const SelectArgs A) {
  constexpr int T = SMP_THREADS, W = SMP_WAVES;
  typedef ScoreLoad<f32x4, BF16> SL;
  __shared__ uint32_t bits[TOK / 32];                  // kept tokens of the part
  // the band list (key, token of the part) and behind it, where there are heavy keys, the bits of their tokens (memory
  // for both heavy keys, or in the largest form for one of them); at last the staged tokens
  __shared__ u32x2 list[CAP];
  constexpr int MAP = TOK / 64;                        // list entries that a bitmap takes the place of
  constexpr bool TWO_MAPS = 2 * MAP < CAP;
  static_assert(MAP <= CAP, "the bits of a heavy key share the list's memory");
  uint32_t *const store = reinterpret_cast<uint32_t *>(list);
  uint32_t *const mapL = store + 2 * (CAP - MAP);
  __shared__ uint32_t h[SEL_BINS];
  __shared__ uint32_t hb[SMP_HIST];                    // the earlier parts' share of an exchanged histogram; first the band
                                                       // tokens that the list has no room for, by bins
  __shared__ uint32_t tmp[T / 64 + 2];
  __shared__ uint32_t red[2 * T / 64];
  __shared__ uint32_t found[9];
  __shared__ uint32_t ticket;                          // next group of the pass
  __shared__ uint32_t ctr[12];                         // 0 list entries, 1 certain tokens, 9, 10 tokens of the heavy keys, 2.. see below
  __shared__ u32x2 cand[SMP_CAND];                     // key; 0 (own) or 1 << 31 | part
  const int part = blockIdx.x, j = blockIdx.y, bt = blockIdx.z, row = bt * A.Hd + j;     // (no division in front of the first load)
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int nb = __builtin_amdgcn_readfirstlane(row_len(A, bt));       // (a loaded value: said to be uniform, like others below)
  const uint32_t c = (uint32_t)min(A.kh[j], nb);
  const int t0 = target_off(A, j), t1 = target_off(A, j + 1);
  if (part == 0) write_tail<T>(A, bt, j, c);
  float *out = A.agg ? A.agg + (size_t)row * A.N : nullptr;
  const bool ranked = c > 0 && t0 != t1;
  const int P = A.smp_tokens, n0 = part * P;
  const int m = ranked ? max(0, min(n0 + P, nb) - n0) : 0;             // ranked tokens of this part
  const int span = out ? min(n0 + P, A.N) - n0 : m;                    // tokens it reads
  if (span <= 0) return;                                               // (a part without ranked tokens is not waited for)
  const int ng = (span + SMP_GROUP - 1) / SMP_GROUP;
  const AggRow R = agg_row(A, row);
  const int Tq = R.Tq;
  for (int i = tid; i < SEL_BINS; i += T) h[i] = 0u;
  if (tid < SMP_HIST) hb[tid] = 0u;
  if (tid < 12) ctr[tid] = 0u;
  if (tid == 0) ticket = 2 * W;
  const float lse_of = R.logits && lane < Tq ? R.L[lane] : 0.f;        // row i's normaliser in lane i (Tq <= 64)
  __syncthreads();
  // ---- the sample's loads, then the first of the part's own
  constexpr int QT = 2;
  const int run = BF16 ? 64 : 32, rq = run >> 2;       // tokens and quads of a 128-byte run
  const SamplePlan sp = sample_plan(max(nb, 1), run, smp_sample(nb, c, A.smp_tokens));
  const int nsq = sp.runs * rq;
  int pos[QT];
  f32x4 sacc[QT];
#pragma unroll
  for (int x = 0; x < QT; ++x) {
    const int s = min(tid + x * T, nsq - 1);           // sampled quad s: quad s % rq of run s / rq
    pos[x] = sp.start(s / rq, run) + (s % rq) * 4;
  }
  // The part's loads: a group of 256 tokens at a time, whichever is next when the wave has room (a fixed
  // share per wave left the oldest waves idle for the last third of the pass), and the Tq rows of it; SMP_FLIGHT in
  // flight. The address is a scalar base and a 32-bit lane offset: no vector arithmetic but the clamp at the
  // row's end.
  RawQuad<BF16> raw[SMP_FLIGHT];
  int grp[SMP_FLIGHT];                                          // group of each slot (wave-uniform), >= ng: none
  int ld_g = wave, ld_i = 0;                           // next load: group and row (wave-uniform)
  uint32_t next_g = (uint32_t)(wave + W);              // in lane 0: the group after that, asked for one group ahead
  const int lane4 = 4 * lane;
  auto issue = [&](RawQuad<BF16> &r, int &slot) {
    slot = ld_g;
    // (a last group of fewer than four tokens starts past the last whole quad: read that quad, see classify)
    const int start = min(n0 + min(ld_g, ng - 1) * SMP_GROUP, R.N - 4);
    const unsigned char *base = static_cast<const unsigned char *>(R.P) + ((size_t)ld_i * R.N + start) * (BF16 ? 2 : 4);
    const uint32_t off = (uint32_t)min(lane4, R.N - 4 - start) * (BF16 ? 2u : 4u);
    r = SL::load_at(base + off);
    if (++ld_i == Tq) {
      ld_i = 0;
      ld_g = __builtin_amdgcn_readfirstlane((int)next_g);
      if (lane == 0) next_g = atomicAdd(&ticket, 1u);
    }
  };
  if (m > 0) {
#pragma unroll 1
    for (int x = 0; x < (nsq <= T ? 1 : QT); ++x) {    // (one sampled quad per thread, or two)
      const f32x4 a = agg_quad_any<BF16>(R, x == 0 ? pos[0] : pos[1], false);
      if (x == 0) sacc[0] = a;
      sacc[1] = a;
    }
  }
#pragma unroll
  for (int u = 0; u < SMP_FLIGHT; ++u) issue(raw[u], grp[u]);
  Band band = {0u, 0u, 0u, false, false, false};
  if (m > 0) band = sample_band<QT>(sp, run, nb, c, pos, sacc, h, tmp, red, found);   // (uniform; its barriers publish ctr)
  else __syncthreads();
  const bool heavyL = band.heavyL, heavyU = band.heavyU && (TWO_MAPS || !heavyL);
  const uint32_t cap = (uint32_t)(CAP - (heavyL ? MAP : 0) - (heavyU ? MAP : 0));
  uint32_t *const mapU = TWO_MAPS && heavyL ? mapL - 2 * MAP : mapL;   // (the bitmaps there are lie at the list's end)

  // ---- the pass
  // INT_MIN marks what is no token of the row: it stays below every edge
  const int sL = ordered_of_key(band.L);
  const int sU = band.haveU ? ordered_of_key(band.L + band.last + 1u) : 0x7fffffff;
  const int sHL = heavyL ? sL : (int)0x80000000, sHU = heavyU ? ordered_of_key(band.L + band.last) : (int)0x80000000;
  const bool heavy = heavyL || heavyU;
  const bool plain = sL > 0;       // scores below the band, negative ones included, compare right as bit patterns
  uint32_t certain = 0;            // wave-uniform
  int shift = max(0, 32 - __clz((int)band.span) - 9);  // bins of the first histogram
  auto classify = [&](int g, f32x4 acc) {
    const int n = n0 + g * SMP_GROUP + lane4;
    if (n0 + (g + 1) * SMP_GROUP > R.N) {              // the row's end: the quad was read where it still fits
      const int d = n - min(n, R.N - 4);
      const f32x4 y = acc;
      acc[0] = d == 0 ? y[0] : d == 1 ? y[1] : d == 2 ? y[2] : y[3];
      acc[1] = d == 0 ? y[1] : d == 1 ? y[2] : y[3];
      acc[2] = d == 0 ? y[2] : y[3];
    }
    if (out && n < R.N) {
      f32x4 o = acc;
#pragma unroll
      for (int e = 0; e < 4; ++e) o[e] = n + e < nb ? o[e] : 0.f;      // the stored aggregate is 0 past the valid length
      if (n + 4 <= R.N) *reinterpret_cast<f32x4_any *>(out + n) = o;
      else
        for (int e = 0; n + e < R.N; ++e) out[n + e] = o[e];
    }
    if (g * SMP_GROUP >= m) return;                    // wave-uniform
    int v[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const float f = acc[e];
      v[e] = __builtin_bit_cast(int, f);
    }
    if (!plain) {
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] = ordered(v[e]);
    }
    if ((g + 1) * SMP_GROUP > m) {
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] = n + e < nb ? v[e] : (int)0x80000000;
    }
    // the nibbles of eight neighbouring quads make one bitmap word, stored whole by the first lane of
    // the eight: three shifts by 1, 2, 4 lanes inside a row of 16 lanes, OR-ed
    auto word = [&](uint32_t b, uint32_t *to) {
      int w = (int)(b << (4 * (lane & 7)));
      w |= __builtin_amdgcn_update_dpp(0, w, 0x101, 0xf, 0xf, true);   // row_shl:1
      w |= __builtin_amdgcn_update_dpp(0, w, 0x102, 0xf, 0xf, true);   // row_shl:2
      w |= __builtin_amdgcn_update_dpp(0, w, 0x104, 0xf, 0xf, true);   // row_shl:4
      if ((lane & 7) == 0) to[g * 8 + (lane >> 3)] = (uint32_t)w;
    };
    auto place = [&](auto with_heavy) {
      uint32_t nib = 0, held = 0;
      bool in_band[4];
      uint64_t bd[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const bool sure = v[e] >= sU;
        in_band[e] = !sure && v[e] >= sL;
        nib |= sure ? 1u << e : 0u;
        certain += (uint32_t)__builtin_popcountll(ballot64(sure));
      }
      word(nib, bits);
      if constexpr (decltype(with_heavy)::value) {
        uint32_t nibL = 0, nibU = 0;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const bool l = in_band[e] && v[e] == sHL, u = in_band[e] && v[e] == sHU;
          nibL |= l ? 1u << e : 0u;
          nibU |= u ? 1u << e : 0u;
          in_band[e] = in_band[e] && !l && !u;
        }
        if (sHL != (int)0x80000000) word(nibL, mapL);
        if (sHU != (int)0x80000000) word(nibU, mapU);
      }
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        bd[e] = ballot64(in_band[e]);
        held += (uint32_t)__builtin_popcountll(bd[e]);
      }
      uint32_t at = 0;
      if (lane == 0) at = atomicAdd(&ctr[0], held);
      at = (uint32_t)__builtin_amdgcn_readfirstlane((int)at);
      if (at + held > cap) {                           // does not fit: counted only
        if (lane == 0 && at < cap) ctr[11] = at;       // (entries from here on are not written)
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (in_band[e]) atomicAdd(&hb[min((key_of_ordered(v[e]) - key_of_ordered(sL)) >> shift, (uint32_t)SMP_HIST - 1u)], 1u);
      } else {
        const uint32_t tok = (uint32_t)(g * SMP_GROUP + lane4);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          if (in_band[e]) list[lanes_before(bd[e], at)] = u32x2{key_of_ordered(v[e]), tok + e};
          at += (uint32_t)__builtin_popcountll(bd[e]);
        }
      }
    };
    // (apart, not a branch inside: the ordinary way has no instruction for heavy keys)
    if (heavy) place(std::true_type{});
    else place(std::false_type{});
  };
  {
    int i = 0;
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
    while (grp[0] < ng) {                              // (groups come in order: behind a slot without one there is none)
#pragma unroll
      for (int u = 0; u < SMP_FLIGHT; ++u) {
        f32x4 p = SL::widen(raw[u]);
        const int g = grp[u];
        issue(raw[u], grp[u]);
        if (R.logits) {
          const float l = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, lse_of), i));
#pragma unroll
          for (int e = 0; e < 4; ++e) p[e] = prob_of(p[e], l);
        }
        if (i == 0) {
          acc = p;
        } else if (R.use_max) {
#pragma unroll
          for (int e = 0; e < 4; ++e) acc[e] = fmaxf(acc[e], p[e]);
        } else {
          acc = acc + p;
        }
        if (++i == Tq) {
          i = 0;
          if (g < ng) classify(g, acc);
        }
      }
    }
  }
  if (m == 0) return;
  if (lane == 0) atomicAdd(&ctr[1], certain);
  __syncthreads();
  const uint32_t first_key = key_of_ordered(sL), last_key = first_key + band.last;   // of the band
  const int words = (m + 31) >> 5, per = (words + T - 1) / T;
  const int w0 = min(tid * per, words), w1 = min(w0 + per, words);     // a thread's run of the bitmaps' words
  if (heavy) {
    uint32_t ofL = 0, ofU = 0;
    for (int w = w0; w < w1; ++w) {
      if (heavyL) ofL += (uint32_t)__builtin_popcount(mapL[w]);
      if (heavyU) ofU += (uint32_t)__builtin_popcount(mapU[w]);
    }
    ofL = wave_sum(ofL);
    ofU = wave_sum(ofU);
    if (lane == 0) {
      atomicAdd(&ctr[9], ofL);
      atomicAdd(&ctr[10], ofU);
    }
    __syncthreads();
  }
  const uint32_t own_G = ctr[1], own_M = ctr[0] + ctr[9] + ctr[10];
  // the heavy keys whose tokens mapL and mapU mark, and how many those are; the entries of the list
  uint32_t keyL = first_key, keyU = last_key, own_L = ctr[9], own_U = ctr[10];
  bool hasL = heavyL, hasU = heavyU, fits = ctr[0] <= cap;
  uint32_t listed = fits ? ctr[0] : ctr[11] ? ctr[11] : cap;

  // ---- the threshold
  const int Qv = (nb + P - 1) / P;                     // parts that hold ranked tokens
  unsigned long long *pub = Qv > 1 ? static_cast<unsigned long long *>(A.pub) + (size_t)row * A.smp_parts * SMP_WORDS : nullptr;
  // false: the row has to be ranked by plain passes (the threshold is not in the band, or another part's words are late)
  auto rank = [&]() -> bool {
    uint32_t lo = first_key, last = last_key - first_key;              // keys in question: lo .. lo + last
    uint32_t krem = 0, G = 0, pre = 0, pre_gt = 0, pre_in = 0, in_bin = 0;
#pragma unroll 1
    for (int round = 0;; ++round) {
      for (int i = tid; i < SMP_HIST; i += T) h[i] = round == 0 ? hb[i] : 0u;
      auto in_question = [&](uint32_t k, uint32_t n) {
        if (k - lo <= last) atomicAdd(&h[min((k - lo) >> shift, (uint32_t)SMP_HIST - 1u)], n);
      };
      if (round > 0 && !fits) {
        // The band did not fit this part's list (heavy tokens next to each other, all in one part): its tokens are read again,
        // and what is left of the keys in question is listed, or, where one key is left, marked. While that is too much as
        // well, the tokens are only counted.
        const bool collect = last == 0u || in_bin <= (uint32_t)CAP;
        if (collect && last == 0u)
          for (int w = w0; w < w1; ++w) mapL[w] = 0u;
        if (tid == 0) ctr[0] = 0u;
        __syncthreads();
#pragma unroll 1
        for (int q = tid; 4 * q < m; q += T) {
          const f32x4 a = agg_quad_any<BF16>(R, n0 + 4 * q, false);
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const uint32_t k = key_of(a[e]), n = 4 * q + e;
            if ((int)n >= m) continue;
            if (!collect) {
              in_question(k, 1u);
            } else if (k - lo <= last) {
              const uint32_t at = atomicAdd(&ctr[0], 1u);
              if (last == 0u) atomicOr(&mapL[n >> 5], 1u << (n & 31u));
              else if (at < (uint32_t)CAP) list[at] = u32x2{k, n};
            } else if (k > lo && k <= last_key) {
              atomicOr(&bits[n >> 5], 1u << (n & 31u));
            }
          }
        }
        if (collect) {
          __syncthreads();
          fits = true;
          hasL = last == 0u;
          hasU = false;
          keyL = lo;
          own_L = ctr[0];
          listed = hasL ? 0u : min(own_L, (uint32_t)CAP);
        }
      } else {
        __syncthreads();
      }
      if (round > 0 && (last == 0u || in_bin <= (uint32_t)SMP_CAND)) break;
      if (fits || round == 0) {
        for (uint32_t i = tid; i < listed; i += T) in_question(list[i][0], 1u);
        if (tid == 0 && hasL) in_question(keyL, own_L);
        if (tid == 0 && hasU) in_question(keyU, own_U);
      }
      __syncthreads();
      uint32_t s_M = own_M;
      if (Qv > 1) {
        // threads 0..255: two bins each; in the first round thread 256 sends the part's counts
        const bool sends = tid < SMP_HIST / 2 || (tid == SMP_HIST / 2 && round == 0);
        const int word = tid < SMP_HIST / 2 ? round * (SMP_HIST / 2) + tid : SMP_G_WORD;
        uint32_t a0 = 0, a1 = 0, b0 = 0, b1 = 0;
        bool complete = true;
        if (sends) {
          const uint32_t o0 = tid < SMP_HIST / 2 ? h[2 * tid] : own_G, o1 = tid < SMP_HIST / 2 ? h[2 * tid + 1] : own_M;
          __hip_atomic_store(&pub[(size_t)part * SMP_WORDS + word],
                             SMP_VALID | o0 | ((unsigned long long)o1 << 32), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          complete = false;
          for (int spin = 0; !complete && spin <= A.fused_spin_limit; ++spin) {
            if (spin) __builtin_amdgcn_s_sleep(2);
            a0 = o0; a1 = o1; b0 = b1 = 0;
            complete = true;
            // eight unconditional loads at a time (this part's own word contributes nothing)
#pragma unroll 1
            for (int q0 = 0; q0 < Qv; q0 += 8) {
              unsigned long long w[8];
#pragma unroll
              for (int u = 0; u < 8; ++u)
                w[u] = __hip_atomic_load(&pub[(size_t)min(q0 + u, Qv - 1) * SMP_WORDS + word], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
              for (int u = 0; u < 8; ++u) {
                const int q = q0 + u;
                const bool use = q != part && q < Qv;
                if (use && !(w[u] & SMP_VALID)) complete = false;
                const uint32_t w0 = use ? (uint32_t)w[u] & 0xffffffu : 0u, w1 = use ? (uint32_t)(w[u] >> 32) & 0xffffffu : 0u;
                a0 += w0;
                a1 += w1;
                b0 += q < part ? w0 : 0u;
                b1 += q < part ? w1 : 0u;
              }
            }
          }
        }
        if (!complete) ctr[2] = 1u;
        __syncthreads();                                 // every thread has read its bins of h
        if (tid < SMP_HIST / 2) {
          h[2 * tid] = a0;
          h[2 * tid + 1] = a1;
          hb[2 * tid] = b0;
          hb[2 * tid + 1] = b1;
        } else if (sends) {
          ctr[3] = a0;                                   // certain tokens of the row
          ctr[4] = a1;                                   // band tokens of the row
          ctr[5] = b0;                                   // certain tokens of the earlier parts
        }
        __syncthreads();
        if (ctr[2]) return false;
        if (round == 0) {
          G = ctr[3];
          s_M = ctr[4];
          pre = ctr[5];
        }
      } else if (round == 0) {
        G = own_G;
      }
      if (round == 0) {
        if (G >= c || G + s_M < c) return false;         // the same in every part of the row
        krem = c - G;
      }
      // every wave finds the bin by itself: lane l owns bins 8 l .. 8 l + 7
      uint32_t x[8], y[8], sx = 0, sy = 0;
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        x[i] = h[8 * lane + i];
        y[i] = Qv > 1 ? hb[8 * lane + i] : 0u;
        sx += x[i];
        sy += y[i];
      }
      const uint32_t incl = wave_incl_scan(sx);
      uint32_t above = (uint32_t)__builtin_amdgcn_readlane((int)incl, 63) - incl;   // keys in bins of higher lanes
      const uint64_t has = ballot64(above < krem && above + sx >= krem);
      const int owner = has ? __builtin_ctzll(has) : 0;
      uint32_t bin = 0, left = krem, held = 0, gt = lane > owner ? sy : 0u, at = 0;
      if (lane == owner) {
#pragma unroll
        for (int i = 7; i >= 0; --i) {
          if (above < krem && above + x[i] >= krem) {
            bin = 8 * lane + i;
            left = krem - above;
            held = x[i];
            at = y[i];
          } else if (above < krem) {
            gt += y[i];                                  // a bin above the threshold's
          }
          above += x[i];
        }
      }
      bin = (uint32_t)__builtin_amdgcn_readlane((int)bin, owner);
      krem = (uint32_t)__builtin_amdgcn_readlane((int)left, owner);
      in_bin = (uint32_t)__builtin_amdgcn_readlane((int)held, owner);
      pre_in = (uint32_t)__builtin_amdgcn_readlane((int)at, owner);
      pre_gt += wave_sum(gt);
      lo += bin << shift;
      last = bin == (uint32_t)SMP_HIST - 1u ? last - (bin << shift) : (1u << shift) - 1u;   // the last bin has no upper end
      last = min(last, last_key - lo);                   // (a bin may run past the band, whose upper keys are kept already)
      // one key or few are left at the latest after round SMP_ROUNDS - 1
      if (fits && (last == 0u || in_bin <= (uint32_t)SMP_CAND)) break;
      shift = max(0, 32 - __clz((int)last) - 9);
      __syncthreads();                                   // every wave has read the histogram
    }
    uint32_t Tk = lo, r = krem, E = in_bin, pre_eq = pre_in;
    if (last != 0u) {
      // few keys share the threshold's bin: they are exchanged one by one and ranked against each other
      auto add = [&](uint32_t k) {
        if (k - lo <= last) {
          const uint32_t s = atomicAdd(&ctr[7], 1u);
          if (s < (uint32_t)SMP_CAND) cand[s] = u32x2{k, 0u};
        }
      };
      for (uint32_t i = tid; i < listed; i += T) add(list[i][0]);
      if (hasL && (uint32_t)tid < min(own_L, (uint32_t)SMP_CAND)) add(keyL);
      if (hasU && (uint32_t)tid < min(own_U, (uint32_t)SMP_CAND)) add(keyU);
      __syncthreads();
      // The other parts' keys follow the own ones under a counter of their own (ctr[8]): ctr[7] and the own entries,
      // which one wave publishes while the others already poll, stay as they are from the barrier on.
      const uint32_t own = min(ctr[7], (uint32_t)SMP_CAND);
      if (Qv > 1) {
        if (tid < SMP_CAND)
          __hip_atomic_store(&pub[(size_t)part * SMP_WORDS + SMP_CAND_WORD + tid],
                             SMP_VALID | ((unsigned long long)own << 32) | ((uint32_t)tid < own ? cand[tid][0] : 0u), __ATOMIC_RELAXED,
                             __HIP_MEMORY_SCOPE_AGENT);
        bool complete = true;
        for (int q = tid / SMP_CAND; q < Qv; q += T / SMP_CAND) {
          if (q == part) continue;
          unsigned long long w = 0;
          for (int spin = 0; !(w & SMP_VALID) && spin <= A.fused_spin_limit; ++spin) {
            if (spin) __builtin_amdgcn_s_sleep(2);
            w = __hip_atomic_load(&pub[(size_t)q * SMP_WORDS + SMP_CAND_WORD + tid % SMP_CAND], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          }
          if (!(w & SMP_VALID)) complete = false;
          else if ((uint32_t)(tid % SMP_CAND) < ((uint32_t)(w >> 32) & 127u)) {
            const uint32_t s = own + atomicAdd(&ctr[8], 1u);
            if (s < (uint32_t)SMP_CAND) cand[s] = u32x2{(uint32_t)w, 0x80000000u | (uint32_t)q};
          }
        }
        if (!complete) ctr[2] = 1u;
        __syncthreads();
        if (ctr[2]) return false;
      }
      // every wave by itself: lane i ranks candidate i
      const uint32_t n = min(in_bin, (uint32_t)SMP_CAND);
      const u32x2 mine = cand[min((uint32_t)lane, n - 1u)];
      uint32_t g = 0, e = 0;
      for (uint32_t q = 0; q < n; ++q) {
        const uint32_t k = cand[q][0];
        g += k > mine[0] ? 1u : 0u;
        e += k == mine[0] ? 1u : 0u;
      }
      const int win = __builtin_ctzll(ballot64((uint32_t)lane < n && g < krem && g + e >= krem) | (1ull << 63));
      Tk = (uint32_t)__builtin_amdgcn_readlane((int)mine[0], win);
      r = krem - (uint32_t)__builtin_amdgcn_readlane((int)g, win);
      E = (uint32_t)__builtin_amdgcn_readlane((int)e, win);
      const bool early = (uint32_t)lane < n && (mine[1] >> 31) && (int)(mine[1] & 0x7fffffffu) < part;
      pre_gt += (uint32_t)__builtin_popcountll(ballot64(early && mine[0] > Tk));
      pre_eq = (uint32_t)__builtin_popcountll(ballot64(early && mine[0] == Tk));
    }
    pre += pre_gt + min(pre_eq, r);                      // kept tokens of the earlier parts

    // ---- the part's kept tokens: bits of the band's. Of the tokens equal to T the first `quota` of this part
    // are kept: all of them, unless the row has more than r.
    const uint32_t quota = r > pre_eq ? r - pre_eq : 0u;
    const bool all_eq = r >= E, of_map = (hasL && Tk == keyL) || (hasU && Tk == keyU);
    uint32_t n_eq = 0;
    for (uint32_t i = tid; i < listed; i += T) {
      const u32x2 x = list[i];
      if (x[0] > Tk || (x[0] == Tk && all_eq)) atomicOr(&bits[x[1] >> 5], 1u << (x[1] & 31u));
      n_eq += x[0] == Tk ? 1u : 0u;
    }
    if (!all_eq && !of_map && quota > 0u) {
      // the lowest tokens of the list's equal ones: their reversed ids are ranked like keys, 11 + 9 bits
      static_assert(TOK <= 1 << 20, "token ids of a part");
      constexpr uint32_t REV = (1u << 20) - 1u;
      const uint32_t own_eq = block_sum1<T>(n_eq, red);
      uint32_t cut = 0;
      if (own_eq > quota) {
        uint32_t da, ra, db, rb;
        for (int i = tid; i < SEL_BINS; i += T) h[i] = 0u;
        __syncthreads();
        for (uint32_t i = tid; i < listed; i += T)
          if (list[i][0] == Tk) atomicAdd(&h[(REV - list[i][1]) >> 9], 1u);
        __syncthreads();
        find_digit<SEL_BINS, T, true>(h, quota, tmp, da, ra);
        for (int i = tid; i < SEL_BINS; i += T) h[i] = 0u;
        __syncthreads();
        for (uint32_t i = tid; i < listed; i += T)
          if (list[i][0] == Tk && ((REV - list[i][1]) >> 9) == da) atomicAdd(&h[(REV - list[i][1]) & 511u], 1u);
        __syncthreads();
        find_digit<SEL_BINS, T, true>(h, ra, tmp, db, rb);
        cut = (da << 9) | db;
      }
      for (uint32_t i = tid; i < listed; i += T)
        if (list[i][0] == Tk && REV - list[i][1] >= cut) atomicOr(&bits[list[i][1] >> 5], 1u << (list[i][1] & 31u));
    }
    __syncthreads();
    if (hasL || hasU) {
      auto take = [&](uint32_t k, uint32_t n, const uint32_t *map) {
        if (k < Tk || (k == Tk && quota == 0u)) return;
        if (k > Tk || all_eq || n <= quota) {
          for (int w = w0; w < w1; ++w) bits[w] |= map[w];
        } else {                                         // the first `quota` of the bits, by words in order
          uint32_t n_own = 0, total;
          for (int w = w0; w < w1; ++w) n_own += (uint32_t)__builtin_popcount(map[w]);
          uint32_t before = block_excl_scan<T, true>(n_own, tmp, total);
          for (int w = w0; w < w1; ++w)
            for (uint32_t rest = map[w]; rest && before < quota; rest &= rest - 1u, ++before) bits[w] |= rest & (0u - rest);
        }
      };
      if (hasL) take(keyL, own_L, mapL);
      if (hasU) take(keyU, own_U, mapU);
      __syncthreads();
    }

    // ---- the list: set bits in token order. A thread owns a run of words, one block scan gives its first place; the
    // tokens are staged in LDS (the band list is done with) and copied out coalesced, once per target head.
    uint32_t mine = 0, total;
    for (int w = w0; w < w1; ++w) mine += (uint32_t)__builtin_popcount(bits[w]);
    const uint32_t first = block_excl_scan<T, true>(mine, tmp, total);
    total = pre < c ? min(total, c - pre) : 0u;          // unchanged for a consistent state; keeps a bad one in bounds
    int32_t *staged = reinterpret_cast<int32_t *>(store);
#pragma unroll 1
    for (uint32_t base = 0; base < total; base += 2 * CAP) {
      uint32_t p = first;
      if (p < base + 2 * CAP && p + mine > base)
        for (int w = w0; w < w1; ++w)
          for (uint32_t rest = bits[w]; rest; rest &= rest - 1u, ++p)
            if (p - base < 2u * CAP) staged[p - base] = n0 + 32 * w + __builtin_ctz(rest);
      __syncthreads();
      const uint32_t cnt = min(total - base, 2u * CAP);
      for (int ti = t0; ti < t1; ++ti) {
        int32_t *dst = A.indices + ((size_t)bt * A.Hq + target_head(A, ti)) * A.k + pre + base;
        for (uint32_t i = tid; i < cnt; i += T) dst[i] = staged[i];
      }
      __syncthreads();
    }
    return true;
  };
  if (!rank()) rank_by_passes<BF16, T>(A, R, bt, nb, c, t0, t1, h, tmp, n0, min(n0 + P, nb));
}

__global__ void __launch_bounds__(SEL_THREADS) select_clear16_kernel(u32x4 *p, size_t n) {
  const size_t i = (size_t)blockIdx.x * SEL_THREADS + threadIdx.x;
  if (i < n) p[i] = u32x4{0u, 0u, 0u, 0u};
}

}  // namespace

static void clear_words(const SelectArgs &a, hipStream_t s) {
  const size_t n16 = (size_t)a.B * a.Hd * (size_t)a.smp_parts * SMP_WORDS / 2;
  STS_LAUNCH(select_clear16_kernel, dim3((unsigned)((n16 + SEL_THREADS - 1) / SEL_THREADS)), dim3(SEL_THREADS), 0, s,
             static_cast<u32x4 *>(a.pub), n16);
}

static bool launch_sampled(const SelectArgs &a, hipStream_t s) {
  if (a.N < 4 || a.smp_tokens % SMP_GROUP != 0 || (int64_t)a.smp_tokens * a.smp_parts < a.N || a.smp_tokens > SMP_MAX_TOKENS)
    return false;
  const dim3 grid(a.smp_parts, a.Hd, a.B), block(SMP_THREADS);
  auto form = [&](auto f) {
    constexpr int F = decltype(f)::value;
    if (a.scores_bf16) STS_LAUNCH((select_sampled_kernel<true, SMP_TOKENS[F], SMP_LIST[F]>), grid, block, 0, s, a);
    else STS_LAUNCH((select_sampled_kernel<false, SMP_TOKENS[F], SMP_LIST[F]>), grid, block, 0, s, a);
  };
  static_assert(SMP_FORMS == 4, "the forms below");
  if (a.smp_tokens <= SMP_TOKENS[0]) form(std::integral_constant<int, 0>{});
  else if (a.smp_tokens <= SMP_TOKENS[1]) form(std::integral_constant<int, 1>{});
  else if (a.smp_tokens <= SMP_TOKENS[2]) form(std::integral_constant<int, 2>{});
  else form(std::integral_constant<int, 3>{});
  return true;
}

// zeroes the words that the parts of a row exchange, 16 bytes per thread
hipError_t launch_select_clear_pub(const SelectArgs &a, hipStream_t s) {
  if ((size_t)a.B * a.Hd == 0 || a.smp_parts == 0) return hipSuccess;
  clear_words(a, s);
  return sts_take_launch_status();
}

hipError_t launch_select_fused(const SelectArgs &a, hipStream_t s) {
  if ((size_t)a.B * a.Hd == 0 || a.smp_parts == 0) return hipSuccess;
  if (!launch_sampled(a, s)) return hipErrorInvalidValue;
  return sts_take_launch_status();
}

// rows enough for every second CU at least: one workgroup per row, or a few with the words between them cleared first
hipError_t launch_select_band(const SelectArgs &a, hipStream_t s) {
  if ((size_t)a.B * a.Hd == 0) return hipSuccess;
  const StsLaunchEvents ev = g_sts_launch_events;      // the timing aid's pair of events spans both launches
  if (a.smp_parts > 1) {
    g_sts_launch_events = StsLaunchEvents{ev.start, nullptr};
    clear_words(a, s);
    g_sts_launch_events = StsLaunchEvents{nullptr, ev.stop};
  }
  const bool ok = launch_sampled(a, s);
  g_sts_launch_events = ev;
  return ok ? sts_take_launch_status() : hipErrorInvalidValue;
}
