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

// grid (S*R, groups of 32 draft heads): one workgroup per row pair. A word of LDS per token says which of the
// draft heads keep it; every target list is then read once, one look at its token's word per entry, and a
// ballot per draft head counts the wave's hits. Rows of more than HM_TOKENS tokens are walked in
// chunks of that many. Bound by latency (128 rows, 16 x 32 heads, 512 tokens of 16384: 9 us; a binary search
// in the target's list per draft entry and target head took 156 us).
constexpr int HM_THREADS = 1024;
constexpr int HM_TOKENS = 32768;          // tokens whose words fit in LDS (128 KB)
__global__ void __launch_bounds__(HM_THREADS) headmap_overlap_kernel(const int32_t *idx_d, const int32_t *idx_t,
                                                                     int S, int R, int Hd, int Ht, int k, int c,
                                                                     unsigned long long *overlap) {
  __shared__ uint32_t heads[HM_TOKENS];
  const int sr = blockIdx.x, h0 = blockIdx.y * 32, nh = min(Hd - h0, 32);
  const int s = sr / R, r = sr - s * R;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  __shared__ int highest;                              // token of all lists (they are ascending)
  if (tid == 0) highest = -1;
  __syncthreads();
  for (int i = tid; i < nh + Ht; i += HM_THREADS) {
    const int32_t *l = i < nh ? idx_d + (((size_t)s * Hd + h0 + i) * R + r) * k : idx_t + (((size_t)s * Ht + (i - nh)) * R + r) * k;
    atomicMax(&highest, l[c - 1]);
  }
  __syncthreads();
  const int N = highest + 1;
  for (int base = 0; base < N; base += HM_TOKENS) {
    const int n = min(N - base, HM_TOKENS);
    for (int i = tid; i < n; i += HM_THREADS) heads[i] = 0u;
    __syncthreads();
    for (int i = tid; i < nh * c; i += HM_THREADS) {
      const int h = i / c, e = i - h * c;
      const uint32_t x = (uint32_t)(idx_d[(((size_t)s * Hd + h0 + h) * R + r) * k + e] - base);
      if (x < (uint32_t)n) atomicOr(&heads[x], 1u << h);
    }
    __syncthreads();
    for (int ht = wave; ht < Ht; ht += HM_THREADS / 64) {
      const int32_t *lt = idx_t + (((size_t)s * Ht + ht) * R + r) * k;
      uint32_t cnt = 0;                                // of draft head h0 + lane
      for (int e0 = 0; e0 < c; e0 += 4 * 64) {
        uint32_t w[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const int e = e0 + 64 * u + lane;
          const uint32_t x = e < c ? (uint32_t)(lt[e] - base) : 0xffffffffu;
          w[u] = x < (uint32_t)n ? heads[x] : 0u;
        }
        for (int h = 0; h < nh; ++h) {
          uint32_t hits = 0;
#pragma unroll
          for (int u = 0; u < 4; ++u) hits += (uint32_t)__builtin_popcountll(__builtin_amdgcn_ballot_w64((w[u] >> h) & 1u));
          cnt += lane == h ? hits : 0u;
        }
      }
      if (cnt) atomicAdd(&overlap[(size_t)ht * Hd + h0 + lane], (unsigned long long)cnt);
    }
    __syncthreads();                                   // the words are rewritten for the next chunk
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

hipError_t launch_headmap_overlap(const int32_t *idx_d, const int32_t *idx_t, int S, int R, int Hd, int Ht,
                                  int k, int c, unsigned long long *overlap, hipStream_t s) {
  if ((size_t)S * R == 0 || Ht == 0 || c == 0) return hipSuccess;
  STS_LAUNCH(headmap_overlap_kernel, dim3(S * R, (Hd + 31) / 32), dim3(HM_THREADS), 0, s, idx_d, idx_t, S, R, Hd, Ht, k, c,
             overlap);
  return sts_take_launch_status();
}

hipError_t launch_headmap_argmax(const unsigned long long *overlap, int Hd, int Ht, int32_t *map, hipStream_t s) {
  if (Ht == 0) return hipSuccess;
  STS_LAUNCH(headmap_argmax_kernel, dim3((Ht + 255) / 256), dim3(256), 0, s, overlap, Hd, Ht, map);
  return sts_take_launch_status();
}
