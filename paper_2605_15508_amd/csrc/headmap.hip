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

// grid (S*R, groups of 32 draft heads, chunks of tokens): one workgroup per row pair and chunk. A word of LDS per
// token of the chunk says which of the draft heads keep it; the chunk's segment of every target list is then read
// once, one look at its token's word per entry, and a ballot per draft head counts the wave's hits. The lists are
// ascending, so a segment is found by a search. Bound by latency (128 rows, 16 x 32 heads, 512 tokens of 16384: 9 us;
// a binary search in the target's list per draft entry and target head took 156 us).
constexpr int HM_THREADS = 1024, HM_WAVES = HM_THREADS / 64;
constexpr int HM_TOKENS = 32768;          // tokens whose words fit in LDS (128 KB): the largest chunk
constexpr int HM_CUS = 256;

// first entry of the ascending list l[0 .. c) that is >= x (c: none), found by a wave: 64 probes a step
__device__ __forceinline__ int hm_lower_bound(const int32_t *l, int c, int x, int lane) {
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
                                                                     int S, int R, int Hd, int Ht, int N, int chunk, int k, int c,
                                                                     unsigned long long *overlap) {
  __shared__ uint32_t heads[HM_TOKENS];
  const int sr = blockIdx.x, h0 = blockIdx.y * 32, nh = min(Hd - h0, 32);
  const int s = sr / R, r = sr - s * R;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int base = (int)blockIdx.z * chunk, n = min(N - base, chunk);
  for (int i = tid; i < n; i += HM_THREADS) heads[i] = 0u;
  __syncthreads();
  // waves share the lists: one each, or, where there are fewer lists than waves, several on one list
  const int dparts = max(1, HM_WAVES / nh), tparts = max(1, HM_WAVES / Ht);
  for (int u = wave; u < nh * dparts; u += HM_WAVES) {
    const int h = u % nh, part = u / nh;
    const int32_t *ld = idx_d + (((size_t)s * Hd + h0 + h) * R + r) * k;
    for (int64_t e0 = hm_lower_bound(ld, c, base, lane) + (int64_t)part * 64; e0 < c; e0 += dparts * 64) {
      const int64_t e = e0 + lane;
      const uint32_t x = e < c ? (uint32_t)(ld[e] - base) : 0xffffffffu;
      if (x < (uint32_t)n) atomicOr(&heads[x], 1u << h);
      if (__builtin_amdgcn_ballot_w64(x >= (uint32_t)n)) break;        // the chunk's or the list's end
    }
  }
  __syncthreads();
  for (int u = wave; u < Ht * tparts; u += HM_WAVES) {
    const int ht = u % Ht, part = u / Ht;
    const int32_t *lt = idx_t + (((size_t)s * Ht + ht) * R + r) * k;
    uint32_t cnt = 0;                                  // of draft head h0 + lane
    for (int64_t e0 = hm_lower_bound(lt, c, base, lane) + (int64_t)part * 256; e0 < c; e0 += tparts * 256) {
      uint32_t w[4];
      bool out = false;
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int64_t e = e0 + 64 * v + lane;
        const uint32_t x = e < c ? (uint32_t)(lt[e] - base) : 0xffffffffu;
        out = x >= (uint32_t)n;                        // (ascending: if one is out, the last ones are)
        w[v] = out ? 0u : heads[x];
      }
      for (int h = 0; h < nh; ++h) {
        uint32_t hits = 0;
#pragma unroll
        for (int v = 0; v < 4; ++v) hits += (uint32_t)__builtin_popcountll(__builtin_amdgcn_ballot_w64((w[v] >> h) & 1u));
        cnt += lane == h ? hits : 0u;
      }
      if (__builtin_amdgcn_ballot_w64(out)) break;
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
  STS_LAUNCH(headmap_overlap_kernel, dim3(S * R, (Hd + 31) / 32, (unsigned)chunks()), dim3(HM_THREADS), 0, s, idx_d, idx_t, S, R,
             Hd, Ht, N, chunk, k, c, overlap);
  return sts_take_launch_status();
}

hipError_t launch_headmap_argmax(const unsigned long long *overlap, int Hd, int Ht, int32_t *map, hipStream_t s) {
  if (Ht == 0) return hipSuccess;
  STS_LAUNCH(headmap_argmax_kernel, dim3((Ht + 255) / 256), dim3(256), 0, s, overlap, Hd, Ht, map);
  return sts_take_launch_status();
}
