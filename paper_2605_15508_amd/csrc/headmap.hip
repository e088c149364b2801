// Head-mapping construction (paper Algorithm 1, Section 4.1) on the GPU.
//
// The per-row top-k index sets of both traces come from the selection pipeline (ascending
// lists). This file counts, for every (target head, draft head), the indices the two lists
// share, summed over all rows, and then takes for each target head the first draft head with
// the largest count. All integer work.
#include "common.h"

namespace {

__global__ void __launch_bounds__(256) headmap_clear_kernel(unsigned long long *p, int n) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i < n) p[i] = 0ull;
}

// grid (S*R, groups of 32 draft heads, chunks of tokens and sets of target heads): one workgroup per row pair, chunk and set. A
// word of LDS per token of the chunk says which of the draft heads keep it; the chunk's segment of every target list is then read
// once, one look at its token's word per entry. The eight words that a lane has looked at are added up bit by bit (the counts'
// binary digits are words, a bit per draft head), and a ballot per digit and draft head adds up the lanes. The lists
// are ascending, so a segment is found by a search. Bound by latency, so eight loads of a list are in flight: 128 rows, 16 x 32
// heads, 512 tokens of 16384: 11.4 us (20 with a load, or four, waited for at a time, and a ballot per word and head; a binary
// search in the target's list per draft entry and target head took 156).
constexpr int HM_THREADS = 1024, HM_WAVES = HM_THREADS / 64;
constexpr int HM_TOKENS = 32768;          // tokens whose words fit in LDS (128 KB): the largest chunk
constexpr int HM_CUS = 256;
constexpr int HM_FLIGHT = 8;              // loads of a list in flight

// first entry of the ascending list l[0 .. c) that is >= x (c: none), found by a wave: 64 probes a step
__device__ __forceinline__ int hm_lower_bound(const int32_t *l, int c, int x, int lane) {
  if (x <= 0) return 0;
  int lo = 0, len = c;
  while (len > 0) {
    const int step = (len + 63) / 64, p = lane * step;
    const uint64_t below = __builtin_amdgcn_ballot_w64(p < len && l[lo + min(p, len - 1)] < x);
    const int n = __builtin_popcountll(below);           // probes 0 .. n - 1 lie below x
    if (n == 0) return lo;
    lo += (n - 1) * step + 1;
    len = min(step - 1, len - (n - 1) * step - 1);
  }
  return lo;
}

__global__ void __launch_bounds__(HM_THREADS) headmap_overlap_kernel(const int32_t *idx_d, const int32_t *idx_t,
                                                                     int S, int R, int Hd, int Ht, int N, int chunk, int k, int c, int sets,
                                                                     unsigned long long *overlap) {
  __shared__ uint32_t heads[HM_TOKENS];
  constexpr int F = HM_FLIGHT;
  const int sr = blockIdx.x, h0 = blockIdx.y * 32, nh = min(Hd - h0, 32);
  const int s = sr / R, r = sr - s * R;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int set = (int)blockIdx.z % sets, base = (int)blockIdx.z / sets * chunk, n = min(N - base, chunk);
  const int ht0 = (int)((int64_t)Ht * set / sets), nt = (int)((int64_t)Ht * (set + 1) / sets) - ht0;       // this workgroup's target heads
  for (int i = tid; i < n; i += HM_THREADS) heads[i] = 0u;
  __syncthreads();
  // waves share the lists: one each, or, where there are fewer lists than waves, several on one list
  const int dparts = max(1, HM_WAVES / nh), tparts = max(1, HM_WAVES / nt);
  // the F * 64 entries from e0 on as tokens of the chunk (all ones: none)
  auto load = [&](const int32_t *l, int64_t e0, uint32_t (&x)[F]) {
#pragma unroll
    for (int v = 0; v < F; ++v) {
      const int64_t e = e0 + 64 * v + lane;
      x[v] = e < c ? (uint32_t)(l[e] - base) : 0xffffffffu;
    }
  };
  for (int u = wave; u < nh * dparts; u += HM_WAVES) {
    const int h = u % nh, part = u / nh;
    const int32_t *ld = idx_d + (((size_t)s * Hd + h0 + h) * R + r) * k;
    for (int64_t e0 = hm_lower_bound(ld, c, base, lane) + (int64_t)part * (64 * F); e0 < c; e0 += dparts * (64 * F)) {
      uint32_t x[F];
      load(ld, e0, x);
#pragma unroll
      for (int v = 0; v < F; ++v)
        if (x[v] < (uint32_t)n) atomicOr(&heads[x[v]], 1u << h);
      if (__builtin_amdgcn_ballot_w64(x[F - 1] >= (uint32_t)n)) break;     // the chunk's or the list's end (ascending)
    }
  }
  __syncthreads();
  for (int u = wave; u < nt * tparts; u += HM_WAVES) {
    const int ht = ht0 + u % nt, part = u / nt;
    const int32_t *lt = idx_t + (((size_t)s * Ht + ht) * R + r) * k;
    uint32_t cnt = 0;                                  // of draft head h0 + lane
    for (int64_t e0 = hm_lower_bound(lt, c, base, lane) + (int64_t)part * (64 * F); e0 < c; e0 += tparts * (64 * F)) {
      static_assert(F == 8, "the adders below");
      uint32_t x[F], w[F];
      load(lt, e0, x);
#pragma unroll
      for (int v = 0; v < F; ++v) w[v] = x[v] < (uint32_t)n ? heads[x[v]] : 0u;
      // digits of the eight words' sum, per bit
      auto sum = [](uint32_t a, uint32_t b, uint32_t d) { return a ^ b ^ d; };
      auto carry = [](uint32_t a, uint32_t b, uint32_t d) { return (a & b) | (d & (a ^ b)); };
      const uint32_t s1 = sum(w[0], w[1], w[2]), c1 = carry(w[0], w[1], w[2]);
      const uint32_t s2 = sum(w[3], w[4], w[5]), c2 = carry(w[3], w[4], w[5]);
      const uint32_t s3 = sum(s1, s2, w[6]), c3 = carry(s1, s2, w[6]), c4 = s3 & w[7];
      const uint32_t t1 = sum(c1, c2, c3), d1 = carry(c1, c2, c3), d2 = t1 & c4;
      const uint32_t digit[4] = {s3 ^ w[7], t1 ^ c4, d1 ^ d2, d1 & d2};
      for (int h = 0; h < nh; ++h) {
        uint32_t hits = 0;
#pragma unroll
        for (int v = 0; v < 4; ++v) hits += (uint32_t)__builtin_popcountll(__builtin_amdgcn_ballot_w64((digit[v] >> h) & 1u)) << v;
        cnt += lane == h ? hits : 0u;
      }
      if (__builtin_amdgcn_ballot_w64(x[F - 1] >= (uint32_t)n)) break;
    }
    if (cnt) atomicAdd(&overlap[(size_t)ht * Hd + h0 + lane], (unsigned long long)cnt);
  }
}

// one thread per target head: strict improvement over a running maximum that starts below
// zero, so the first best draft head wins and zero overlap maps to draft head 0
__global__ void __launch_bounds__(256) headmap_argmax_kernel(const unsigned long long *overlap, int Hd, int Ht,
                                                             int32_t *map) {
  const int ht = blockIdx.x * 256 + threadIdx.x;
  if (ht >= Ht) return;
  long long best = -1;
  int arg = 0;
  for (int hd = 0; hd < Hd; ++hd) {
    const long long v = (long long)overlap[(size_t)ht * Hd + hd];
    if (v > best) {
      best = v;
      arg = hd;
    }
  }
  map[ht] = arg;
}

}  // namespace

hipError_t launch_headmap_clear(unsigned long long *overlap, int n, hipStream_t s) {
  if (n == 0) return hipSuccess;
  STS_LAUNCH(headmap_clear_kernel, dim3((n + 255) / 256), dim3(256), 0, s, overlap, n);
  return sts_take_launch_status();
}

// Chunks are as large as LDS allows; calls of few row pairs halve them until every CU has a workgroup, as long as a
// workgroup keeps 16K entries to read (below that the searches cost as much as the entries). One row pair of 128K tokens,
// 13108 kept, 16 x 32 heads: 30 us with the clearing and the maximum (one workgroup that walked all chunks and read every
// list for each: 1263; a search per draft entry and target head: 1402); 1M tokens, 20972 kept: 38 (15190, 2343).
hipError_t launch_headmap_overlap(const int32_t *idx_d, const int32_t *idx_t, int S, int R, int Hd, int Ht, int N,
                                  int k, int c, unsigned long long *overlap, hipStream_t s) {
  if ((size_t)S * R == 0 || Ht == 0 || c == 0) return hipSuccess;
  const int64_t pairs = (int64_t)S * R * ((Hd + 31) / 32), entries = (int64_t)((Hd < 32 ? Hd : 32) + Ht) * c;
  int chunk = HM_TOKENS;
  auto chunks = [&] { return ((int64_t)N + chunk - 1) / chunk; };
  while (chunk > 1024 && pairs * chunks() < HM_CUS && entries / chunks() > 32768) chunk /= 2;
  // a chip that is still not full: sets of target heads, a list per wave and more in each (the draft lists are read for every set)
  int sets = 1;
  while (2 * pairs * chunks() * sets <= HM_CUS && Ht >= 2 * sets * HM_WAVES) sets *= 2;
  STS_LAUNCH(headmap_overlap_kernel, dim3(S * R, (Hd + 31) / 32, (unsigned)(chunks() * sets)), dim3(HM_THREADS), 0, s, idx_d, idx_t, S, R,
             Hd, Ht, N, chunk, k, c, sets, overlap);
  return sts_take_launch_status();
}

hipError_t launch_headmap_argmax(const unsigned long long *overlap, int Hd, int Ht, int32_t *map, hipStream_t s) {
  if (Ht == 0) return hipSuccess;
  STS_LAUNCH(headmap_argmax_kernel, dim3((Ht + 255) / 256), dim3(256), 0, s, overlap, Hd, Ht, map);
  return sts_take_launch_status();
}
