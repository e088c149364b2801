// Online mask generation for STS (gfx950): draft attention scores -> per-head top-k token
// index sets, remapped to the target heads (paper Section 4.2; Section 4.3: one mask per
// speculative batch).
//
// Ways through, chosen on the host from the shape; one row = one (batch, draft head). Rows of up to 8192 tokens, many of up
// to 32768 and rows of one bf16 score per token are ranked in registers (select_row.hip), most longer ones by the sampled
// selection of select_sampled.hip; here are:
//  * few very long rows, block scores -- every kernel on a (chunk, row) grid of 8192-token chunks:
//      clear  zero the three digit histograms and the chunk flags of every row
//      agg    A[n] = ((P[0,n] + P[1,n]) + ...) in fp32, stored; histogram of the top 11 key bits
//      hist1  find the first digit of the k-th largest key, histogram the next 11 bits of the
//             keys that share it
//      hist2  same for the last 10 bits
//      write  the k-th largest key T is now known, with r = how many keys equal to T are kept.
//             Ordered compaction: token n is kept iff key > T, or key == T and fewer than r
//             equal keys precede it; its output position is (#greater before n) + min(#equal
//             before n, r). The counts of the chunks before this one come from the words those
//             chunks publish. The list is written to every target head mapped to the draft head.
//  * few very long rows, small budgets (chunks * budget small enough for one workgroup's LDS, see the
//    host's rule) -- two launches, nothing to clear:
//      local  aggregate a chunk, keep its keys in registers, and rank them inside the chunk: the
//             chunk's own top-k (same tie rule) goes to a pool, in token order. Every token of
//             the row's top-k is in the top-k of its chunk.
//      pool   one workgroup per row ranks the pooled candidates out of LDS and writes the list.
//  * short lists of block scores (up to 2048) -- one workgroup per row ranks them out of LDS (select_small_kernel);
//    longer ones and short rows of scores are ranked in registers (select_row.hip).
// Keys are the usual order-preserving map of fp32 to uint32 (with -0 folded onto +0), so the
// whole selection is integer arithmetic: the index sets are exact, ties go to the lower token.
// Histograms use LDS atomics per workgroup and integer global atomics to merge (order-free).
#include "select_util.h"

namespace {
// Add a workgroup's LDS histogram to the row's global one. Two neighbouring 32-bit bins travel
// in one 64-bit atomic (a row holds fewer than 2^32 keys, so the low bin never carries into
// the high one), which halves the number of atomics.
template <int NBINS, int THREADS = SEL_THREADS>
__device__ __forceinline__ void flush_hist(uint32_t *global_bins, const uint32_t *lds_bins) {
  unsigned long long *g2 = reinterpret_cast<unsigned long long *>(global_bins);
  for (int i = threadIdx.x; i < NBINS / 2; i += THREADS) {
    const unsigned long long v = (unsigned long long)lds_bins[2 * i] | ((unsigned long long)lds_bins[2 * i + 1] << 32);
    if (v) atomicAdd(&g2[i], v);
  }
}

__global__ void __launch_bounds__(SEL_THREADS) select_clear_kernel(uint32_t *p, size_t n) {
  const size_t i = (size_t)blockIdx.x * SEL_THREADS + threadIdx.x;
  if (i < n) p[i] = 0u;
}

// --------------------------------------------------------------------------- aggregation
// The sums alone, a quad per thread, of the valid tokens: for rows that one workgroup then ranks. Bound by latency (16 rows of 33001 tokens,
// five scores: some 4 us with its launch), by memory from 64 such rows on.
template <bool BF16>
__global__ void __launch_bounds__(SEL_THREADS) select_row_sums_kernel(const SelectArgs A) {
  const int j = blockIdx.y, bt = blockIdx.z, row = bt * A.Hd + j;
  const int n0 = (int)blockIdx.x * (4 * SEL_THREADS), n = n0 + 4 * (int)threadIdx.x;
  const int nb = row_len(A, bt);
  if (n >= nb) return;
  const f32x4 x = agg_quad_any<BF16>(agg_row(A, row), n, n0 + 4 * SEL_THREADS <= A.N);
  float *const out = A.agg + (size_t)row * A.N + n;
  if (n + 4 <= A.N) *reinterpret_cast<f32x4_any *>(out) = x;
  else
    for (int e = 0; n + e < A.N; ++e) out[e] = x[e];
}

template <bool VEC4>
__global__ void __launch_bounds__(SEL_THREADS) select_agg_kernel(const SelectArgs A) {
  __shared__ uint32_t h[SEL_BINS];
  const int row = blockIdx.y, chunk = blockIdx.x;
  const int bt = __builtin_amdgcn_readfirstlane(row / A.Hd);
  const int nb = row_len(A, bt);
  for (int i = threadIdx.x; i < SEL_BINS; i += SEL_THREADS) h[i] = 0u;
  __syncthreads();
  const AggRow R = agg_row(A, row);
  float *out = A.agg + (size_t)row * A.N;
  const int n0 = chunk * SEL_CHUNK;
  const int n1 = min(n0 + SEL_CHUNK, A.N);
  if (VEC4) {
    // The chunk's sums wait in registers and are stored in one burst after the last read: a
    // write stream mixed into the read stream costs this memory system far more than its bytes,
    // and with the workgroups of a launch running in step the two phases separate chip-wide.
    constexpr int IT = SEL_CHUNK / (SEL_THREADS * 4);
    f32x4 keep[IT];
#pragma clang loop unroll(full)
    for (int i = 0; i < IT; ++i) {
      const int n = n0 + (i * SEL_THREADS + (int)threadIdx.x) * 4;
      if (n < n1) {
        keep[i] = agg_quad(R, n);
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (A.page == 1 && n + e < nb) atomicAdd(&h[key_of(keep[i][e]) >> (32 - SEL_BITS0)], 1u);
      }
    }
    if (!A.agg_is_input) {
#pragma clang loop unroll(full)
      for (int i = 0; i < IT; ++i) {
        const int n = n0 + (i * SEL_THREADS + (int)threadIdx.x) * 4;
        if (n < n1) {
          f32x4 o = keep[i];
#pragma unroll
          for (int e = 0; e < 4; ++e)
            if (n + e >= nb) o[e] = 0.f;          // the stored aggregate is 0 past the valid length
          *reinterpret_cast<f32x4 *>(out + n) = o;
        }
      }
    }
  } else {
    for (int n = n0 + threadIdx.x; n < n1; n += SEL_THREADS) {
      const float acc = agg_one(R, n);
      if (!A.agg_is_input) out[n] = n < nb ? acc : 0.f;
      if (A.page == 1 && n < nb) atomicAdd(&h[key_of(acc) >> (32 - SEL_BITS0)], 1u);
    }
  }
  __syncthreads();
  if (A.page != 1) return;   // block granularity: the block kernel builds the first histogram
  uint32_t *gh = A.hist + (size_t)row * 3 * SEL_BINS;
  flush_hist<SEL_BINS>(gh, h);
}

// ----------------------------------------------------------------------- block scores
// One thread per block: the block's aggregated scores added left to right in fp32 (tokens
// below the valid length only), stored, and counted into the first-digit histogram.
__global__ void __launch_bounds__(SEL_THREADS) select_block_kernel(const SelectArgs A) {
  __shared__ uint32_t h[SEL_BINS];
  const int row = blockIdx.y;
  const int bt = __builtin_amdgcn_readfirstlane(row / A.Hd);
  const int nb = row_len(A, bt);
  const int nblk = (nb + A.page - 1) / A.page;
  for (int i = threadIdx.x; i < SEL_BINS; i += SEL_THREADS) h[i] = 0u;
  __syncthreads();
  const float *a = A.agg + (size_t)row * A.N;
  float *out = A.blk + (size_t)row * A.srcN;
  const int m = blockIdx.x * SEL_THREADS + threadIdx.x;
  if (m < A.srcN) {
    float acc = 0.f;
    const int n0 = m * A.page;
    const int n1 = min(n0 + A.page, nb);
    for (int n = n0; n < n1; ++n) acc = (n == n0) ? a[n] : acc + a[n];
    out[m] = acc;
    if (m < nblk) atomicAdd(&h[key_of(acc) >> (32 - SEL_BITS0)], 1u);
  }
  __syncthreads();
  uint32_t *gh = A.hist + (size_t)row * 3 * SEL_BINS;
  flush_hist<SEL_BINS>(gh, h);
}

// Aggregation and block sums in one pass (a power of two from 4 to 256 tokens per block): every lane aggregates 4
// consecutive tokens in registers and the page/4
// lanes of a block pass the running sum from left to right, so the additions happen in exactly the order of the
// one-thread-per-block kernel above; the per-token
// aggregate is stored only when the caller asks for it. With A.hist == nullptr no histogram is
// built (the blocks are ranked out of LDS afterwards). ANY: rows of any length from 4 on and scores at any alignment
// (the quad that would run past the row's end is read where it fits and shifted; the last block may be short). Such rows took six
// launches, one of which read a chunk of 8192 tokens per workgroup and stored the sums per token: 32 rows of 13205 tokens, eight
// scores each, pages of 16: 62 us, 12.7 with the ranking now.
template <bool ANY>
__global__ void __launch_bounds__(SEL_THREADS) select_aggblock_kernel(const SelectArgs A, int chunk) {
  __shared__ uint32_t h[SEL_BINS];
  const int row = blockIdx.y;
  const int bt = __builtin_amdgcn_readfirstlane(row / A.Hd);
  const int nb = row_len(A, bt);
  const int nblk = (nb + A.page - 1) / A.page;
  const bool want_hist = A.hist != nullptr;
  if (want_hist) {
    for (int i = threadIdx.x; i < SEL_BINS; i += SEL_THREADS) h[i] = 0u;
    __syncthreads();
  }
  const AggRow R = agg_row(A, row);
  float *tok_out = A.agg ? A.agg + (size_t)row * A.N : nullptr;
  float *out = A.blk + (size_t)row * A.srcN;
  const int L = A.page >> 2;                       // lanes per block (1..64, power of two)
  const int lane = threadIdx.x & 63;
  const int pos_in_blk = lane & (L - 1);
  // `chunk` tokens per workgroup, a multiple of the 1024 of a sweep; the lanes of the last block are all here
  const int end = (int)min((int64_t)(blockIdx.x + 1) * chunk, (int64_t)A.srcN * A.page);
  for (int n = blockIdx.x * chunk + threadIdx.x * 4; n < end; n += SEL_THREADS * 4) {
    f32x4 x;
    if constexpr (ANY) {
      const bool inside = __builtin_amdgcn_readfirstlane(n) + 256 <= A.N;      // (lane 0's quad is the wave's first)
      x = R.bf16 ? agg_quad_any<true>(R, n, inside) : agg_quad_any<false>(R, n, inside);
    } else {
      x = agg_quad(R, n);
    }
    if (tok_out) {
      f32x4 o = x;
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (n + e >= nb) o[e] = 0.f;
      if constexpr (ANY) {
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (n + e < A.N) tok_out[n + e] = o[e];
      } else {
        *reinterpret_cast<f32x4 *>(tok_out + n) = o;
      }
    }
    float run = 0.f;
    bool have = false;                             // whether `run` holds at least one term
    for (int s = 0; s < L; ++s) {
      if (pos_in_blk == s) {
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (n + e < nb) {
            run = have ? run + x[e] : x[e];
            have = true;
          }
      }
      if (s + 1 < L) {
        const float up = __shfl_up(run, 1, 64);
        const int hup = __shfl_up((int)have, 1, 64);
        if (pos_in_blk == s + 1) {
          run = up;
          have = hup != 0;
        }
      }
    }
    if (pos_in_blk == L - 1) {
      const int m = n / A.page;
      out[m] = run;                                // blocks past the valid length hold 0
      if (want_hist && m < nblk) atomicAdd(&h[key_of(run) >> (32 - SEL_BITS0)], 1u);
    }
  }
  if (!want_hist) return;
  __syncthreads();
  flush_hist<SEL_BINS>(A.hist + (size_t)row * 3 * SEL_BINS, h);
}

// ------------------------------------------------------------------ refinement histograms
// PASS 1: digit 1 (bits 20..10) of keys whose digit 0 matches; PASS 2: digit 2 (bits 9..0)
// of keys whose digits 0 and 1 match.
template <int PASS, bool VEC4>
__global__ void __launch_bounds__(SEL_THREADS) select_hist_kernel(const SelectArgs A) {
  __shared__ uint32_t h[SEL_BINS];
  __shared__ uint32_t tmp[16];
  const int row = blockIdx.y;
  const int chunk0 = blockIdx.x * A.hist_cpw;      // this workgroup takes hist_cpw consecutive chunks
  const int bt = __builtin_amdgcn_readfirstlane(row / A.Hd);
  const int nb = src_len(A, bt);
  const uint32_t c = (uint32_t)min(A.kh[__builtin_amdgcn_readfirstlane(row % A.Hd)], nb);
  if (c == 0) return;
  uint32_t *st = A.state + (size_t)row * 8;
  const uint32_t *gh = A.hist + (size_t)row * 3 * SEL_BINS;
  const float *a = A.src + (size_t)row * A.srcN;
  // The first chunk's loads do not depend on the digit search: issue them first so that their
  // latency hides behind it. They are unconditional (a branch around a load makes the compiler
  // wait for it at the join): the address is clamped into the row, out-of-range quads are
  // ignored when counting.
  constexpr int IT = SEL_CHUNK / (SEL_THREADS * 4);
  f32x4 x[IT];
  if (VEC4) {
#pragma unroll
    for (int i = 0; i < IT; ++i) {
      const int n = chunk0 * SEL_CHUNK + (i * SEL_THREADS + (int)threadIdx.x) * 4;
      x[i] = *reinterpret_cast<const f32x4 *>(a + min(n, A.srcN - 4));
    }
  }
  for (int i = threadIdx.x; i < SEL_BINS; i += SEL_THREADS) h[i] = 0u;
  uint32_t prefix, shift, dmask;
  if (PASS == 1) {
    uint32_t d0, k1;
    find_digit<(1 << SEL_BITS0)>(gh, c, tmp, d0, k1);
    if (chunk0 == 0 && threadIdx.x == 0) { st[0] = d0; st[1] = k1; st[6] = c; }
    prefix = d0;
    shift = SEL_BITS1 + SEL_BITS2;
    dmask = (1u << SEL_BITS1) - 1;
  } else {
    const uint32_t d0 = st[0], k1 = st[1];
    uint32_t d1, k2;
    find_digit<(1 << SEL_BITS1)>(gh + SEL_BINS, k1, tmp, d1, k2);
    if (chunk0 == 0 && threadIdx.x == 0) { st[2] = d1; st[3] = k2; }
    prefix = (d0 << SEL_BITS1) | d1;
    shift = SEL_BITS2;
    dmask = (1u << SEL_BITS2) - 1;
  }
  const uint32_t dshift = (PASS == 1) ? SEL_BITS2 : 0;
  // (the barriers inside find_digit have published the zeroed histogram)
  for (int cc = 0; cc < A.hist_cpw; ++cc) {
    const int n0 = (chunk0 + cc) * SEL_CHUNK;
    const int n1 = min(min(n0 + SEL_CHUNK, A.srcN), nb);
    if (n0 >= n1) break;
    if (VEC4) {
      if (cc > 0) {
#pragma unroll
        for (int i = 0; i < IT; ++i) {
          const int n = n0 + (i * SEL_THREADS + (int)threadIdx.x) * 4;
          x[i] = *reinterpret_cast<const f32x4 *>(a + min(n, A.srcN - 4));
        }
      }
#pragma unroll
      for (int i = 0; i < IT; ++i) {
        const int n = n0 + (i * SEL_THREADS + (int)threadIdx.x) * 4;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const uint32_t key = key_of(x[i][e]);
          if (n + e < n1 && (key >> shift) == prefix) atomicAdd(&h[(key >> dshift) & dmask], 1u);
        }
      }
    } else {
      for (int n = n0 + threadIdx.x; n < n1; n += SEL_THREADS) {
        const uint32_t key = key_of(a[n]);
        if ((key >> shift) == prefix) atomicAdd(&h[(key >> dshift) & dmask], 1u);
      }
    }
  }
  __syncthreads();
  uint32_t *go = A.hist + ((size_t)row * 3 + PASS) * SEL_BINS;
  flush_hist<SEL_BINS>(go, h);
}

// ------------------------------------------------------ ordered compaction + head remap
// The chunk's scores are loaded coalesced into LDS, then every thread takes 32 consecutive
// tokens, so one block scan of (greater, equal) counts gives every token its rank in token
// order. The kept tokens of a chunk occupy one contiguous range of the output list: they are
// staged in LDS at their local rank and copied out with coalesced stores, once per target.
template <bool VEC4>
__global__ void __launch_bounds__(SEL_THREADS, 4) select_write_kernel(const SelectArgs A) {   // <= 128 VGPRs: 4 workgroups per CU
  constexpr int PER = SEL_CHUNK / SEL_THREADS;   // 32 tokens per thread
  constexpr int PITCH = PER + 1;                 // odd pitch: conflict-free per-thread rows
  __shared__ uint32_t tmp[16];
  __shared__ uint32_t buf[SEL_THREADS * PITCH];  // keys first, then the staged token ids
  const int row = blockIdx.y, chunk = blockIdx.x;
  int bt, j;
  row_of(A, row, bt, j);
  const int nb = src_len(A, bt);
  const uint32_t c = (uint32_t)min(A.kh[j], nb);
  const int t0 = target_off(A, j), t1 = target_off(A, j + 1);
  if (chunk == 0) {
    // tail padding and counts for every target head of this draft head
    for (int ti = t0; ti < t1; ++ti) {
      const int tgt = target_head(A, ti);
      int32_t *dst = A.indices + ((size_t)bt * A.Hq + tgt) * A.k;
      for (uint32_t p = c + threadIdx.x; p < (uint32_t)A.k; p += SEL_THREADS) dst[p] = -1;
      if (A.counts && threadIdx.x == 0) A.counts[(size_t)bt * A.Hq + tgt] = (int32_t)c;
    }
  }
  if (c == 0 || t0 == t1) return;
  const int n0 = chunk * SEL_CHUNK;
  if (n0 >= nb) return;
  const uint32_t *st = A.state + (size_t)row * 8;
  const float *a = A.src + (size_t)row * A.srcN;

  uint32_t *cc = A.chunk_cnt + (size_t)row * A.nchunks * SEL_FLAG_PITCH;
  // Everything this workgroup needs from memory is asked for at once, before anything is used:
  // the chunk (coalesced, clamped addresses, unconditional), a first look at the counts the
  // earlier chunks publish (they are often there already), and, inside find_digit, the last
  // digit's histogram.
  constexpr int IT = SEL_CHUNK / (SEL_THREADS * 4);
  f32x4 x[IT];
  if (VEC4) {
#pragma unroll
    for (int i = 0; i < IT; ++i)
      x[i] = *reinterpret_cast<const f32x4 *>(a + min(n0 + (i * SEL_THREADS + (int)threadIdx.x) * 4, A.srcN - 4));
  }
  uint32_t early = 0;
  if ((int)threadIdx.x < chunk)
    early = __hip_atomic_load(&cc[threadIdx.x * SEL_FLAG_PITCH], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);

  // threshold key and tie quota of the row
  uint32_t d2, r;
  find_digit<(1 << SEL_BITS2)>(A.hist + ((size_t)row * 3 + 2) * SEL_BINS, st[3], tmp, d2, r);
  const uint32_t T = (st[0] << (SEL_BITS1 + SEL_BITS2)) | (st[2] << SEL_BITS2) | d2;

  // token n0 + i lands at buf[(i / PER) * PITCH + i % PER]
  if (VEC4) {
#pragma unroll
    for (int i = 0; i < IT; ++i) {
      const int t = (i * SEL_THREADS + (int)threadIdx.x) * 4;
#pragma unroll
      for (int e = 0; e < 4; ++e) buf[((t + e) / PER) * PITCH + (t + e) % PER] = key_of(x[i][e]);   // srcN % 4 == 0
    }
  } else {
    for (int i = threadIdx.x; i < SEL_CHUNK; i += SEL_THREADS)
      buf[(i / PER) * PITCH + i % PER] = (n0 + i < nb) ? key_of(a[n0 + i]) : 0u;
  }
  __syncthreads();

  const int base_n = n0 + threadIdx.x * PER;
  uint32_t keys[PER];
  uint32_t cg = 0, ce = 0;
#pragma unroll
  for (int i = 0; i < PER; ++i) {
    keys[i] = buf[threadIdx.x * PITCH + i];
    const bool in = base_n + i < nb;        // tokens past the valid length never count
    cg += (in && keys[i] > T) ? 1u : 0u;
    ce += (in && keys[i] == T) ? 1u : 0u;
  }
  uint32_t total;
  const uint32_t excl = block_excl_scan(cg | (ce << 16), tmp, total);   // barriers: buf is free
  const uint32_t chunk_gt = total & 0xffffu, chunk_eq = total >> 16;

  // keys greater / equal in the chunks before this one
  uint32_t pre = 0, pre_eq = 0;
  {
    // Every chunk publishes its own counts in one word (flag | equal << 14 | greater) with a
    // device-scope atomic store and reads the words of the chunks before it, one per thread.
    // The payload travels inside the flag, so no fence is involved. A chunk whose word does
    // not show up within the poll limit is simply recounted from the scores by this workgroup,
    // so the wait is bounded and no workgroup depends on another one being scheduled.
    uint32_t *miss = reinterpret_cast<uint32_t *>(buf);   // list of chunks to recount
    if (threadIdx.x == 0) {
      __hip_atomic_store(&cc[chunk * SEL_FLAG_PITCH], 0x80000000u | (chunk_eq << 14) | chunk_gt, __ATOMIC_RELAXED,
                         __HIP_MEMORY_SCOPE_AGENT);
      tmp[8] = 0;                                          // number of entries in miss
    }
    __syncthreads();
    uint32_t g = 0, e = 0;
    for (int ch = threadIdx.x; ch < chunk; ch += SEL_THREADS) {
      uint32_t f = early;                                  // the first look, taken at the start
      if (ch != (int)threadIdx.x || !(f >> 31))
        f = __hip_atomic_load(&cc[ch * SEL_FLAG_PITCH], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      for (int spin = 0; !(f >> 31) && spin < A.spin_limit; ++spin) {
        __builtin_amdgcn_s_sleep(8);
        f = __hip_atomic_load(&cc[ch * SEL_FLAG_PITCH], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      }
      if (f >> 31) {
        g += f & 0x3fffu;
        e += (f >> 14) & 0x3fffu;
      } else {
        const uint32_t slot = atomicAdd(&tmp[8], 1u);
        if (slot < (uint32_t)(SEL_THREADS * PITCH)) {
          miss[slot] = (uint32_t)ch;
        } else {   // list full (only with thousands of chunks per row): this thread recounts alone
          for (int i = 0; i < SEL_CHUNK; ++i) {
            const uint32_t key = key_of(a[ch * SEL_CHUNK + i]);
            g += key > T ? 1u : 0u;
            e += key == T ? 1u : 0u;
          }
        }
      }
    }
    __syncthreads();
    const uint32_t nmiss = min(tmp[8], (uint32_t)(SEL_THREADS * PITCH));
    for (uint32_t mi = 0; mi < nmiss; ++mi) {
      // recount chunk miss[mi] (it lies wholly below nb: it precedes this chunk)
      const int m0 = (int)miss[mi] * SEL_CHUNK;
      uint32_t packed = 0;
      for (int i = threadIdx.x; i < SEL_CHUNK; i += SEL_THREADS) {
        const uint32_t key = key_of(a[m0 + i]);
        packed += (key > T ? 1u : 0u) + (key == T ? 0x10000u : 0u);
      }
      // one thread per wave carries the wave's sum into the running totals
#pragma unroll
      for (int off = 32; off > 0; off >>= 1) packed += __shfl_xor(packed, off, 64);
      if ((threadIdx.x & 63) == 0) {
        g += packed & 0xffffu;
        e += packed >> 16;
      }
    }
    // block totals of both counts (a row holds fewer than 2^31 tokens: two 32-bit sums)
    const uint32_t wg = wave_incl_scan(g), we = wave_incl_scan(e);
    if ((threadIdx.x & 63) == 63) {
      tmp[2 * (threadIdx.x >> 6)] = wg;
      tmp[2 * (threadIdx.x >> 6) + 1] = we;
    }
    __syncthreads();
#pragma unroll
    for (int w = 0; w < SEL_THREADS / 64; ++w) {
      pre += tmp[2 * w];
      pre_eq += tmp[2 * w + 1];
    }
    __syncthreads();
  }
  uint32_t g = pre + (excl & 0xffffu), q = pre_eq + (excl >> 16);
  // output range of this chunk: [first, last)
  const uint32_t first = pre + min(pre_eq, r);
  const uint32_t last = min((pre + chunk_gt) + min(pre_eq + chunk_eq, r), c);
  int32_t *staged = reinterpret_cast<int32_t *>(buf);
#pragma unroll
  for (int i = 0; i < PER; ++i) {
    const bool in = base_n + i < nb;
    const bool is_gt = in && keys[i] > T;
    const bool is_eq = in && keys[i] == T;
    if (is_gt || (is_eq && q < r)) {
      const uint32_t pos = g + min(q, r);
      // always inside [first, last) for a consistent threshold; the test keeps a bad state
      // inside the staging buffer
      if (pos >= first && pos - first < (uint32_t)SEL_CHUNK) staged[pos - first] = base_n + i;
    }
    g += is_gt ? 1u : 0u;
    q += is_eq ? 1u : 0u;
  }
  __syncthreads();
  if (last > first) {
    const uint32_t cnt = min(last - first, (uint32_t)SEL_CHUNK);
    for (int ti = t0; ti < t1; ++ti) {
      int32_t *dst = A.indices + ((size_t)bt * A.Hq + target_head(A, ti)) * A.k + first;
      for (uint32_t p = threadIdx.x; p < cnt; p += SEL_THREADS) dst[p] = staged[p];
    }
  }
}

// ------------------------------------------------------- ranking keys that sit in LDS
constexpr int SMALL_THREADS = 1024;
__device__ __forceinline__ int small_slot(int n) { return n + (n >> 5); }   // pad 1 word per 32: conflict-free strided reads

// The c-th largest of keys[small_slot(0 .. m)) and the number r of keys equal to it that are
// kept. On entry h holds the histogram of the first digit of those m keys; h and tmp
// (THREADS/64 + 2 words) are scratch. Requires 1 <= c <= m.
template <int THREADS>
__device__ __forceinline__ void lds_threshold(const uint32_t *keys, int m, uint32_t *h, uint32_t *tmp, uint32_t c,
                                              uint32_t &T, uint32_t &r) {
  const int tid = threadIdx.x;
  uint32_t d0, k1, d1, k2, d2;
  find_digit<(1 << SEL_BITS0), THREADS>(h, c, tmp, d0, k1);
  for (int i = tid; i < SEL_BINS; i += THREADS) h[i] = 0u;
  __syncthreads();
  for (int n = tid; n < m; n += THREADS) {
    const uint32_t key = keys[small_slot(n)];
    if ((key >> (SEL_BITS1 + SEL_BITS2)) == d0) atomicAdd(&h[(key >> SEL_BITS2) & ((1u << SEL_BITS1) - 1)], 1u);
  }
  __syncthreads();
  find_digit<(1 << SEL_BITS1), THREADS>(h, k1, tmp, d1, k2);
  for (int i = tid; i < SEL_BINS; i += THREADS) h[i] = 0u;
  __syncthreads();
  const uint32_t pre01 = (d0 << SEL_BITS1) | d1;
  for (int n = tid; n < m; n += THREADS) {
    const uint32_t key = keys[small_slot(n)];
    if ((key >> SEL_BITS2) == pre01) atomicAdd(&h[key & ((1u << SEL_BITS2) - 1)], 1u);
  }
  __syncthreads();
  find_digit<(1 << SEL_BITS2), THREADS>(h, k2, tmp, d2, r);
  T = (pre01 << SEL_BITS2) | d2;
}

// Ordered compaction of the same keys: every thread owns a run of at most MAXPER consecutive
// entries (m <= MAXPER * THREADS), read once into registers; entry n is kept iff key > T, or
// key == T and fewer than r equal keys precede it, and emit(pos, n) is called with its position
// in the output list, pos = (#greater before n) + min(#equal before n, r).
template <int THREADS, int MAXPER, class Emit>
__device__ __forceinline__ void lds_compact_run(const uint32_t *keys, int m, uint32_t T, uint32_t r, uint32_t c,
                                                uint32_t *tmp, Emit emit) {
  const int tid = threadIdx.x;
  const int per = (m + THREADS - 1) / THREADS;
  const int nlo = min(tid * per, m), nhi = min(nlo + per, m);
  uint32_t kk[MAXPER];
  uint32_t cg = 0, ce = 0;
#pragma unroll
  for (int i = 0; i < MAXPER; ++i) {
    const int n = nlo + i;
    kk[i] = keys[small_slot(min(n, m - 1))];
    cg += (n < nhi && kk[i] > T) ? 1u : 0u;
    ce += (n < nhi && kk[i] == T) ? 1u : 0u;
  }
  uint32_t total;
  const uint32_t excl = block_excl_scan<THREADS>(cg | (ce << 16), tmp, total);   // m <= 32768: both sums fit 16 bits
  uint32_t g = excl & 0xffffu, q = excl >> 16;
#pragma unroll
  for (int i = 0; i < MAXPER; ++i) {
    const int n = nlo + i;
    const bool is_gt = n < nhi && kk[i] > T, is_eq = n < nhi && kk[i] == T;
    if (is_gt || (is_eq && q < r)) {
      const uint32_t pos = g + min(q, r);
      if (pos < c) emit(pos, n);   // always true for a consistent threshold; keeps a bad state in bounds
    }
    g += is_gt ? 1u : 0u;
    q += is_eq ? 1u : 0u;
  }
}

// the same with the run length (a uniform value) rounded up to 4, 8, 16 or MAXPER
template <int THREADS, int MAXPER, class Emit>
__device__ __forceinline__ void lds_compact(const uint32_t *keys, int m, uint32_t T, uint32_t r, uint32_t c,
                                            uint32_t *tmp, Emit emit) {
  const int per = (m + THREADS - 1) / THREADS;
  if (MAXPER > 4 && per <= 4) lds_compact_run<THREADS, 4>(keys, m, T, r, c, tmp, emit);
  else if (MAXPER > 8 && per <= 8) lds_compact_run<THREADS, 8>(keys, m, T, r, c, tmp, emit);
  else if (MAXPER > 16 && per <= 16) lds_compact_run<THREADS, 16>(keys, m, T, r, c, tmp, emit);
  else lds_compact_run<THREADS, MAXPER>(keys, m, T, r, c, tmp, emit);
}

// ------------------------------------------------- keys of a row in LDS, ranked by one workgroup
// FROM_SRC: the scores to rank are already there (A.src, row pitch A.srcN: the block sums of
// block-granular selection) and are loaded, up to SEL_RANK_N of them (17 KB of LDS with the histogram: two workgroups per CU;
// with room for 32768 keys one: 1024 rows of 1024 blocks 48.1 -> 41.0 us, 2048 62.7 -> 47.6, 512 27.6 -> 24.3), then three digit
// histograms over the LDS-resident keys, ordered compaction and the copies to the target heads in a single launch. Otherwise:
// rows of fewer than four tokens, which are aggregated here.
template <bool FROM_SRC>
__global__ void __launch_bounds__(SMALL_THREADS) select_small_kernel(const SelectArgs A) {
  __shared__ uint32_t keys[SEL_RANK_N + SEL_RANK_N / 32];
  __shared__ uint32_t h[SEL_BINS];
  __shared__ uint32_t tmp[SMALL_THREADS / 64 + 2];
  const int row = blockIdx.x;
  int bt, j;
  row_of(A, row, bt, j);
  const int nb = FROM_SRC ? src_len(A, bt) : row_len(A, bt);
  const uint32_t c = (uint32_t)min(A.kh[j], nb);
  const int t0 = target_off(A, j), t1 = target_off(A, j + 1);
  const int tid = threadIdx.x;
  write_tail<SMALL_THREADS>(A, bt, j, c);
  const bool want_agg = !FROM_SRC && A.agg != nullptr;
  if ((c == 0 || t0 == t1) && !want_agg) return;

  for (int i = tid; i < SEL_BINS; i += SMALL_THREADS) h[i] = 0u;
  __syncthreads();
  const AggRow R = agg_row(A, row);
  float *out = want_agg ? A.agg + (size_t)row * A.N : nullptr;
  if (FROM_SRC) {
    const float *src = A.src + (size_t)row * A.srcN;
    for (int n = tid; n < nb; n += SMALL_THREADS) {
      const uint32_t key = key_of(src[n]);
      keys[small_slot(n)] = key;
      atomicAdd(&h[key >> (32 - SEL_BITS0)], 1u);
    }
  } else {
    for (int n = tid; n < A.N; n += SMALL_THREADS) {
      const float acc = agg_one(R, n);
      if (want_agg) out[n] = n < nb ? acc : 0.f;
      const uint32_t key = key_of(acc);
      keys[small_slot(n)] = key;
      if (n < nb) atomicAdd(&h[key >> (32 - SEL_BITS0)], 1u);
    }
  }
  __syncthreads();
  if (c == 0 || t0 == t1) return;

  uint32_t T, r;
  lds_threshold<SMALL_THREADS>(keys, nb, h, tmp, c, T, r);
  lds_compact<SMALL_THREADS, SEL_RANK_N / SMALL_THREADS>(keys, nb, T, r, c, tmp, [&](uint32_t pos, int n) {
    for (int ti = t0; ti < t1; ++ti) A.indices[((size_t)bt * A.Hq + target_head(A, ti)) * A.k + pos] = n;
  });
}

// --------------------------------- many long rows of ready-made scores: one workgroup per row
// A call with one score per token (Tq = 1: the per-query-row masks of prefill rank every row of a
// block's scores on its own; a draft layer's summed weights), far more rows than CUs and rows that do not fit a workgroup's
// registers, or take a CU's for each (select_row16_kernel and the rule in the host code). Cutting
// such rows into parts that wait for each other leaves every CU idle during the exchanges; here a
// row belongs to ONE workgroup, which keeps nothing but a digit histogram in LDS and reads the
// row once per digit level and once more to compact it. The re-reads come out of the caches (a
// row is 256-512 KB; what the resident workgroups hold together fits the last-level cache), and
// several small workgroups per CU are in different phases at any time, so the digit searches and
// scans of one hide behind the streaming of the others. Nothing is exchanged, cleared or stored
// besides the lists. bf16 scores have keys whose low 16 bits are all equal, so their third level
// is known without a pass.
template <bool BF16>
__device__ __forceinline__ uint32_t rowpass_key(const u32x4 &w, int e) {
  if (BF16) {
    const uint32_t pair = w[e >> 1];
    return key_of_bits((e & 1) ? (pair & 0xffff0000u) : (pair << 16));
  }
  return key_of_bits(w[e & 3]);
}

template <int THREADS, bool BF16>
__global__ void __launch_bounds__(THREADS) select_rowpass_kernel(const SelectArgs A) {
  constexpr int VPT = BF16 ? 8 : 4;       // tokens per 16-byte word
  constexpr int UNR = 4;                  // words in flight per thread
  constexpr int RUN = UNR * VPT;          // consecutive tokens a thread owns per compaction step
  static_assert(RUN <= 32 && THREADS * RUN < 65536, "mask bits per thread; packed block scan");
  __shared__ uint32_t h[SEL_BINS];
  __shared__ uint32_t tmp[THREADS / 64 + 2];
  const int row = blockIdx.x, tid = threadIdx.x;
  int bt, j;
  row_of(A, row, bt, j);
  const int nb = row_len(A, bt);
  const uint32_t c = (uint32_t)min(A.kh[j], nb);
  const int t0 = target_off(A, j), t1 = target_off(A, j + 1);
  write_tail<THREADS>(A, bt, j, c);
  if (c == 0 || t0 == t1) return;
  // N % VPT == 0 and a 16-byte aligned base (the host's condition for this path): whole words
  const u32x4 *src = reinterpret_cast<const u32x4 *>(
      static_cast<const unsigned char *>(A.scores) + (size_t)row * A.N * (BF16 ? 2 : 4));
  const int nv = (nb + VPT - 1) / VPT;    // words that hold ranked tokens

  // bf16 rows: the second digit has only 32 values that occur (5 bits of the score, the rest
  // follows the sign), so its histogram can be built in the FIRST pass for a window of first
  // digits, if the window is put where the first digit will turn out to be: a 1/16 sample of the
  // row (128-byte runs) says where. If the first digit falls outside the window the second pass
  // is made as for any row; the result never depends on the sample.
  constexpr int WIN = 8;
  constexpr int STAGE = THREADS * 8;      // list entries staged per round of the compaction
  __shared__ int32_t staged[STAGE];
  __shared__ uint32_t hw[BF16 ? WIN * 32 : 1];
  uint32_t wlo = 0;                       // first digit the window starts at
  bool win = false;
  if (BF16 && nv >= 4096) {
    win = true;
    for (int i = tid; i < SEL_BINS; i += THREADS) h[i] = 0u;
    __syncthreads();
    const int runs = (nv + 127) / 128;    // sampled run i: the 8 words from 128 i on
    uint32_t mine = 0;
    for (int s0 = tid; s0 < runs * 8; s0 += THREADS) {
      const int wi = (s0 >> 3) * 128 + (s0 & 7);
      if (wi < nv) {
        const u32x4 w = src[wi];
#pragma unroll
        for (int e = 0; e < VPT; ++e)
          if (wi * VPT + e < nb) {
            atomicAdd(&h[rowpass_key<BF16>(w, e) >> (32 - SEL_BITS0)], 1u);
            ++mine;
          }
      }
    }
    __syncthreads();
    uint32_t ns;
    block_excl_scan<THREADS>(mine, tmp, ns);
    const uint32_t want = (uint32_t)min((uint64_t)ns, max((uint64_t)1, (uint64_t)c * ns / (uint32_t)nb));
    uint32_t dest, unused;
    find_digit<SEL_BINS, THREADS>(h, want, tmp, dest, unused);
    wlo = dest >= WIN / 2 ? dest - WIN / 2 + 1 : 0u;
    for (int i = tid; i < WIN * 32; i += THREADS) hw[i] = 0u;
  }

  uint32_t d0 = 0, pre01 = 0, krem = c, d2 = 0;
#pragma unroll 1
  for (int level = 0; level < (BF16 ? 2 : 3); ++level) {
    for (int i = tid; i < SEL_BINS; i += THREADS) h[i] = 0u;
    __syncthreads();
    if (BF16 && level == 1 && win && d0 - wlo < (uint32_t)WIN) {
      // the window held the first digit: its 32 counts are the second digit's histogram
      const uint32_t low = (d0 >> (SEL_BITS0 - 1)) ? 0u : (1u << (SEL_BITS1 - 5)) - 1;   // the bits below follow the sign
      if (tid < 32) h[((uint32_t)tid << (SEL_BITS1 - 5)) | low] = hw[(d0 - wlo) * 32 + tid];
    } else {
#pragma unroll 1
      for (int i0 = tid; i0 < nv; i0 += THREADS * UNR) {
        u32x4 w[UNR];
#pragma unroll
        for (int u = 0; u < UNR; ++u) w[u] = src[min(i0 + u * THREADS, nv - 1)];
        if (BF16 && level == 0) {
          // The kernel is bound by its vector instructions (about 18 per token and pass in the
          // general form below), so the common case gets a form of its own: every word of the
          // wave inside the row and no sign bit among its scores (attention weights have none).
          // Then the first digit is 1024 + (the stored 16 bits >> 5) and the window's sub-bin
          // their low 5 bits: five instructions per token.
          uint32_t any = 0;
#pragma unroll
          for (int u = 0; u < UNR; ++u) any |= w[u][0] | w[u][1] | w[u][2] | w[u][3];
          const bool lane_ok = (i0 + (UNR - 1) * THREADS + 1) * VPT <= nb && (any & 0x80008000u) == 0u;
          if (__builtin_amdgcn_ballot_w64(!lane_ok) == 0) {
            const uint32_t wlo10 = wlo - (1u << (SEL_BITS0 - 1));    // modulo 2^32: the comparison below stays exact
            uint32_t *hpos = h + (1u << (SEL_BITS0 - 1));
#pragma unroll
            for (int u = 0; u < UNR; ++u)
#pragma unroll
              for (int e = 0; e < VPT; ++e) {
                const uint32_t pair = w[u][(e >> 1) & 3];
                const uint32_t r16 = (e & 1) ? pair >> 16 : pair & 0xffffu;
                const uint32_t b = r16 >> 5;
                atomicAdd(&hpos[b], 1u);
                const uint32_t wd = b - wlo10;
                if (win && wd < (uint32_t)WIN) atomicAdd(&hw[wd * 32 + (r16 & 31u)], 1u);
              }
            continue;
          }
        }
#pragma unroll
        for (int u = 0; u < UNR; ++u) {
          const int wi = i0 + u * THREADS;
          const int valid = wi < nv ? nb - wi * VPT : 0;   // ranked tokens from this word on: >= VPT but at the row's end
#pragma unroll
          for (int e = 0; e < VPT; ++e) {
            const uint32_t key = rowpass_key<BF16>(w[u], e);
            const int bin = fused_bin(key, level, d0, pre01);
            if (e < valid && bin >= 0) {
              atomicAdd(&h[bin], 1u);
              if (BF16 && level == 0 && win && (uint32_t)bin - wlo < (uint32_t)WIN)
                atomicAdd(&hw[((uint32_t)bin - wlo) * 32 + ((key >> (32 - SEL_BITS0 - 5)) & 31u)], 1u);
            }
          }
        }
      }
    }
    __syncthreads();
    uint32_t digit, knext;
    find_digit<SEL_BINS, THREADS>(h, krem, tmp, digit, knext);
    if (level == 0) d0 = digit;
    else if (level == 1) pre01 = (d0 << SEL_BITS1) | digit;
    else d2 = digit;
    krem = knext;
  }
  // widened bf16: the 16 low key bits repeat the complement of the sign, so every key that shares
  // the first two digits is the same key
  if (BF16) d2 = (d0 >> (SEL_BITS0 - 1)) ? 0u : (1u << SEL_BITS2) - 1;
  const uint32_t r = krem;
  const uint32_t Tk = (pre01 << SEL_BITS2) | d2;

  // ordered compaction: per step, thread tid owns the RUN consecutive tokens from step + tid * RUN
  uint32_t gbase = 0, qbase = 0;          // keys greater than / equal to the threshold before this step
#pragma unroll 1
  for (int step = 0; step < nb; step += THREADS * RUN) {
    const int nlo = step + tid * RUN;
    u32x4 w[UNR];
#pragma unroll
    for (int u = 0; u < UNR; ++u) w[u] = src[min(nlo / VPT + u, nv - 1)];
    uint32_t gt_mask = 0, eq_mask = 0;
    // the common case again (see the first pass): a positive threshold, every run of the wave inside
    // the row, no sign bit: the stored 16 bits are compared with the threshold's
    bool plain = false;
    if (BF16 && (Tk >> 31)) {
      uint32_t any = 0;
#pragma unroll
      for (int u = 0; u < UNR; ++u) any |= w[u][0] | w[u][1] | w[u][2] | w[u][3];
      plain = __builtin_amdgcn_ballot_w64(!(nlo + RUN <= nb && (any & 0x80008000u) == 0u)) == 0;
    }
    if (plain) {
      const uint32_t T16 = (Tk >> 16) & 0x7fffu;
#pragma unroll
      for (int u = 0; u < UNR; ++u)
#pragma unroll
        for (int e = 0; e < VPT; ++e) {
          const uint32_t pair = w[u][(e >> 1) & 3];
          const uint32_t r16 = (e & 1) ? pair >> 16 : pair & 0xffffu;
          gt_mask |= (r16 > T16) ? 1u << (u * VPT + e) : 0u;
          eq_mask |= (r16 == T16) ? 1u << (u * VPT + e) : 0u;
        }
    } else {
#pragma unroll
      for (int u = 0; u < UNR; ++u)
#pragma unroll
        for (int e = 0; e < VPT; ++e) {
          const uint32_t key = rowpass_key<BF16>(w[u], e);
          gt_mask |= (key > Tk) ? 1u << (u * VPT + e) : 0u;
          eq_mask |= (key == Tk) ? 1u << (u * VPT + e) : 0u;
        }
    }
    if (!plain) {   // tokens past the row's valid length (only in its last run) are dropped from both masks
      const int left = nb - nlo;
      const uint32_t in = left >= RUN ? 0xffffffffu : (left > 0 ? (1u << left) - 1u : 0u);
      gt_mask &= in;
      eq_mask &= in;
    }
    uint32_t total;
    const uint32_t excl = block_excl_scan<THREADS>(__builtin_popcount(gt_mask) | (__builtin_popcount(eq_mask) << 16), tmp, total);
    // The step's kept tokens, places [first, last) of the list, are staged in LDS and copied out
    // coalesced, STAGE at a time: stored straight from their threads (a few 4-byte stores each,
    // scattered over the wave) they cost more than reading the row did.
    const uint32_t first = gbase + min(qbase, r);
    gbase += total & 0xffffu;
    qbase += total >> 16;
    const uint32_t last = min(gbase + min(qbase, r), c);
#pragma unroll 1
    for (uint32_t base = first; base < last; base += STAGE) {
      uint32_t g = first - min(qbase - (total >> 16), r) + (excl & 0xffffu);   // greater keys before this thread's run
      uint32_t q = qbase - (total >> 16) + (excl >> 16);                        // equal keys before it
      for (uint32_t rest = gt_mask | eq_mask; rest; rest &= rest - 1) {
        const int i = __builtin_ctz(rest);
        const bool is_gt = (gt_mask >> i) & 1u;
        if (is_gt || q < r) {
          const uint32_t pos = g + min(q, r);
          if (pos >= base && pos - base < (uint32_t)STAGE) staged[pos - base] = nlo + i;
        }
        g += is_gt ? 1u : 0u;
        q += is_gt ? 0u : 1u;
      }
      __syncthreads();
      const uint32_t cnt = min(last - base, (uint32_t)STAGE);
      for (int ti = t0; ti < t1; ++ti) {
        int32_t *dst = A.indices + ((size_t)bt * A.Hq + target_head(A, ti)) * A.k + base;
        for (uint32_t p = tid; p < cnt; p += THREADS) dst[p] = staged[p];
      }
      __syncthreads();
    }
    if (gbase + min(qbase, r) >= c) break;   // the list is complete (uniform)
  }
}

// ---------------------------------------------- small budgets on long rows: chunk-local top-k
// Every token of a row's top-c (ordered by key descending, then token ascending) has fewer
// than c tokens of the whole row before it in that order, hence fewer than c tokens of its own
// chunk: it belongs to the top-c of its chunk under the same rule. So each chunk keeps only
// its own best min(c, chunk length) tokens (the pool), and the row is ranked from the pool.
//
// Local kernel, (chunk, row) grid, 256 threads per 8192-token chunk or 1024 per 32768-token
// chunk (fewer, larger chunks keep the pool small on very long rows): aggregates the chunk (same
// fp32 order), keeps the 32 keys of each thread in registers, finds the chunk's threshold with three LDS digit
// histograms, and writes the kept (key, token) pairs to the chunk's pool segment in token
// order. Thread t owns tokens n0 + (i*THREADS + t)*4 .. +3 for i = 0..7, so token order is (i, t).
template <int IT>
struct LocalKeys {
  uint32_t k[IT][4];
};

template <int THREADS>
__global__ void __launch_bounds__(THREADS) select_local_kernel(const SelectArgs A) {
  constexpr int CHUNK = THREADS * 32;          // 32 keys per thread
  constexpr int IT = 8;
  __shared__ uint32_t h[SEL_BINS];
  __shared__ uint32_t tmp[THREADS / 64 + 2];
  const int row = blockIdx.y, chunk = blockIdx.x;
  int bt, j;
  row_of(A, row, bt, j);
  const int nb = row_len(A, bt);
  const int n0 = chunk * CHUNK;
  const int nvalid = max(0, min(n0 + CHUNK, nb) - n0);     // ranked tokens of this chunk
  uint32_t c = (uint32_t)min(A.kh[j], nvalid);
  const bool want_agg = A.agg != nullptr;
  if (target_off(A, j) == target_off(A, j + 1)) c = 0;        // no target head reads this draft head
  if (c == 0 && !want_agg) return;
  for (int i = threadIdx.x; i < SEL_BINS; i += THREADS) h[i] = 0u;
  __syncthreads();
  const AggRow R = agg_row(A, row);
  float *out = want_agg ? A.agg + (size_t)row * A.N : nullptr;
  LocalKeys<IT> K;
#pragma clang loop unroll(full)
  for (int i = 0; i < IT; ++i) {
    const int n = n0 + (i * THREADS + threadIdx.x) * 4;
    if (n < A.N) {                                             // N % 4 == 0 on this path
      const f32x4 acc = agg_quad(R, n);
      f32x4 o = acc;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        K.k[i][e] = key_of(acc[e]);
        if (n + e < nb) atomicAdd(&h[K.k[i][e] >> (32 - SEL_BITS0)], 1u);
        else o[e] = 0.f;
      }
      if (want_agg) *reinterpret_cast<f32x4 *>(out + n) = o;
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e) K.k[i][e] = 0u;
    }
  }
  __syncthreads();
  if (c == 0) return;
  // threshold of the chunk: three digits over the register-resident keys
  uint32_t d0, k1, d1, k2, d2, r;
  find_digit<(1 << SEL_BITS0), THREADS>(h, c, tmp, d0, k1);
  for (int i = threadIdx.x; i < SEL_BINS; i += THREADS) h[i] = 0u;
  __syncthreads();
#pragma unroll
  for (int i = 0; i < IT; ++i)
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int n = n0 + (i * THREADS + threadIdx.x) * 4 + e;
      const uint32_t key = K.k[i][e];
      if (n < nb && (key >> (SEL_BITS1 + SEL_BITS2)) == d0) atomicAdd(&h[(key >> SEL_BITS2) & ((1u << SEL_BITS1) - 1)], 1u);
    }
  __syncthreads();
  find_digit<(1 << SEL_BITS1), THREADS>(h, k1, tmp, d1, k2);
  for (int i = threadIdx.x; i < SEL_BINS; i += THREADS) h[i] = 0u;
  __syncthreads();
  const uint32_t pre01 = (d0 << SEL_BITS1) | d1;
#pragma unroll
  for (int i = 0; i < IT; ++i)
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int n = n0 + (i * THREADS + threadIdx.x) * 4 + e;
      const uint32_t key = K.k[i][e];
      if (n < nb && (key >> SEL_BITS2) == pre01) atomicAdd(&h[key & ((1u << SEL_BITS2) - 1)], 1u);
    }
  __syncthreads();
  find_digit<(1 << SEL_BITS2), THREADS>(h, k2, tmp, d2, r);
  const uint32_t T = (pre01 << SEL_BITS2) | d2;

  // Ordered compaction into the chunk's pool segment, one block scan per sweep of 1024 tokens.
  // Every chunk before this one is full and keeps min(budget, CHUNK) pairs, so the row's
  // pool is contiguous and this chunk's place in it is known without communication.
  const size_t seg = (size_t)row * A.pool_nchunks * A.pool_pitch + (size_t)chunk * min(A.kh[j], CHUNK);
  uint32_t *pk = A.pool_key + seg;
  int32_t *pi = A.pool_idx + seg;
  uint32_t g0 = 0, q0 = 0;                                     // greater / equal in the sweeps before
#pragma unroll
  for (int i = 0; i < IT; ++i) {
    const int n = n0 + (i * THREADS + threadIdx.x) * 4;
    uint32_t cg = 0, ce = 0;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const bool in = n + e < nb;
      cg += (in && K.k[i][e] > T) ? 1u : 0u;
      ce += (in && K.k[i][e] == T) ? 1u : 0u;
    }
    uint32_t total;
    const uint32_t excl = block_excl_scan<THREADS>(cg | (ce << 16), tmp, total);
    uint32_t g = g0 + (excl & 0xffffu), q = q0 + (excl >> 16);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const bool in = n + e < nb;
      const bool is_gt = in && K.k[i][e] > T, is_eq = in && K.k[i][e] == T;
      if (is_gt || (is_eq && q < r)) {
        const uint32_t pos = g + min(q, r);
        if (pos < c) {                 // always true for a consistent threshold
          pk[pos] = K.k[i][e];
          pi[pos] = n + e;
        }
      }
      g += is_gt ? 1u : 0u;
      q += is_eq ? 1u : 0u;
    }
    g0 += total & 0xffffu;
    q0 += total >> 16;
  }
}

// Pool kernel, one 1024-thread workgroup per row: the chunks' kept pairs, concatenated in
// chunk order (= token order), are loaded into LDS and ranked like a short row; the kept
// tokens go to every target head of the draft head.
constexpr int POOL_MAX = SEL_POOL_MAX;   // pooled pairs per row: keys and tokens fit in LDS
__global__ void __launch_bounds__(SMALL_THREADS) select_pool_kernel(const SelectArgs A) {
  __shared__ uint32_t keys[POOL_MAX + POOL_MAX / 32];
  __shared__ int32_t toks[POOL_MAX + POOL_MAX / 32];
  __shared__ uint32_t h[SEL_BINS];
  __shared__ uint32_t red[2 * SMALL_THREADS / 64];
  __shared__ uint32_t tmp[SMALL_THREADS / 64 + 2];
  const int row = blockIdx.x;
  int bt, j;
  row_of(A, row, bt, j);
  const int nb = row_len(A, bt);
  const uint32_t c = (uint32_t)min(A.kh[j], nb);
  const int t0 = target_off(A, j), t1 = target_off(A, j + 1);
  const int tid = threadIdx.x;
  write_tail<SMALL_THREADS>(A, bt, j, c);
  if (c == 0 || t0 == t1) return;
  for (int i = tid; i < SEL_BINS; i += SMALL_THREADS) h[i] = 0u;
  // pooled pairs of the row: the full chunks keep min(budget, chunk length) each, the last one
  // min(budget, its length)
  const uint32_t kfull = (uint32_t)min(A.kh[j], A.pool_chunk);
  const uint32_t m = min((uint32_t)(nb / A.pool_chunk) * kfull + min((uint32_t)A.kh[j], (uint32_t)(nb % A.pool_chunk)),
                         (uint32_t)POOL_MAX);
  const uint32_t *pk = A.pool_key + (size_t)row * A.pool_nchunks * A.pool_pitch;
  const int32_t *pi = A.pool_idx + (size_t)row * A.pool_nchunks * A.pool_pitch;
  // The pairs were written by other workgroups: their loads miss the caches, so eight
  // independent ones are issued per thread before any is used (uniform trip count, clamped
  // addresses, the surplus ignored).
  uint32_t kmin = 0xffffffffu, kmax = 0u;
  for (uint32_t e0 = 0; e0 < m; e0 += SMALL_THREADS * 8) {
    uint32_t key[8];
    int32_t tok[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const uint32_t e = min(e0 + u * SMALL_THREADS + tid, m - 1);
      key[u] = pk[e];
      tok[u] = pi[e];
    }
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const uint32_t e = e0 + u * SMALL_THREADS + tid;
      if (e < m) {
        keys[small_slot((int)e)] = key[u];
        toks[small_slot((int)e)] = tok[u];
        kmin = min(kmin, key[u]);
        kmax = max(kmax, key[u]);
      }
    }
  }
  // The pooled keys are all large, so their leading bits agree and the first digit would put
  // them into a handful of bins (LDS atomics on one address serialise). Ranking the keys
  // shifted left by the length of their common prefix is the same ranking and spreads them.
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    kmin = min(kmin, (uint32_t)__shfl_xor((int)kmin, off, 64));
    kmax = max(kmax, (uint32_t)__shfl_xor((int)kmax, off, 64));
  }
  if ((tid & 63) == 0) {
    red[(tid >> 6) * 2] = kmin;
    red[(tid >> 6) * 2 + 1] = kmax;
  }
  __syncthreads();
#pragma unroll
  for (int w = 0; w < SMALL_THREADS / 64; ++w) {
    kmin = min(kmin, red[w * 2]);
    kmax = max(kmax, red[w * 2 + 1]);
  }
  uint32_t T, r;
  if (kmin == kmax) {
    T = kmin;            // all pooled keys are equal: the first c in token order are kept
    r = c;
  } else {
    const int shift = __clz((int)(kmin ^ kmax));               // 0..31
    for (uint32_t e = tid; e < m; e += SMALL_THREADS) {
      const uint32_t key = keys[small_slot((int)e)] << shift;
      keys[small_slot((int)e)] = key;
      atomicAdd(&h[key >> (32 - SEL_BITS0)], 1u);
    }
    __syncthreads();
    lds_threshold<SMALL_THREADS>(keys, (int)m, h, tmp, c, T, r);
  }
  lds_compact<SMALL_THREADS, POOL_MAX / SMALL_THREADS>(keys, (int)m, T, r, c, tmp, [&](uint32_t pos, int n) {
    const int32_t tok = toks[small_slot(n)];
    for (int ti = t0; ti < t1; ++ti) A.indices[((size_t)bt * A.Hq + target_head(A, ti)) * A.k + pos] = tok;
  });
}

}  // namespace

static inline bool vec_ok(const SelectArgs &a) {   // aggregation: scores and agg rows
  return (a.N % 4) == 0 && (reinterpret_cast<uintptr_t>(a.scores) % 16) == 0 &&
         (reinterpret_cast<uintptr_t>(a.agg) % 16) == 0;
}

static inline bool src_vec_ok(const SelectArgs &a) {   // ranking passes: rows of src
  return (a.srcN % 4) == 0 && (reinterpret_cast<uintptr_t>(a.src) % 16) == 0;
}

hipError_t launch_select_small(const SelectArgs &a, hipStream_t s) {
  if ((size_t)a.B * a.Hd == 0) return hipSuccess;
  if (a.N >= 4) return launch_select_row(a, s);        // rows that hold a quad
  STS_LAUNCH(select_small_kernel<false>, dim3(a.B * a.Hd), dim3(SMALL_THREADS), 0, s, a);
  return sts_take_launch_status();
}

// ranks the rows of a.src, up to SEL_SMALL_N entries each: out of LDS, or in registers from SEL_RANK_N entries on
hipError_t launch_select_rank(const SelectArgs &a, hipStream_t s) {
  if ((size_t)a.B * a.Hd == 0) return hipSuccess;
  // 64 rows of 8192 or 16384 blocks: 39.3 -> 37.1, 46.5 -> 41.8 us with the block sums; 128 rows of 1024: 22.6, 23.8
  if (a.srcN > SEL_RANK_N) {
    SelectArgs b = a;                                  // one fp32 score per block
    b.scores = a.src;
    b.scores_bf16 = 0;
    b.lse = nullptr;
    b.kind = STS_SCORES_PROBS;
    b.reduce = STS_REDUCE_SUM;
    b.agg = nullptr;
    b.Tq = 1;
    b.N = a.srcN;
    return launch_select_row(b, s);
  }
  STS_LAUNCH(select_small_kernel<true>, dim3(a.B * a.Hd), dim3(SMALL_THREADS), 0, s, a);
  return sts_take_launch_status();
}

bool select_aggblock_ok(const SelectArgs &a) {
  // (calls that ask for the sums per token, too, of rows that end within a block keep the kernels that store those first)
  return (a.page & (a.page - 1)) == 0 && a.page >= 4 && a.page <= 256 && a.N >= 4 && (a.agg == nullptr || a.N % a.page == 0);
}

hipError_t launch_select_aggblock(const SelectArgs &a, hipStream_t s) {
  if ((size_t)a.B * a.Hd == 0 || a.N == 0) return hipSuccess;
  // One quad per thread where nothing is collected per workgroup. us with the ranking, 8192, 4096, 2048 and 1024 tokens per workgroup:
  // 16 rows of 4096 tokens, five scores 14.9, 15.2, 12.3, 10.5; 32 of 13205, eight 24.4, 17.5, 14.0, 12.7; 64 of 131072, five
  // 36.1, 37.3, 35.6, 35.6; 256 of 60000, eight 89.7, 86.4, 83.6, 82.6. (A histogram is worth a longer chunk: it is added to the row's.)
  const int chunk = a.hist ? SEL_CHUNK : 4 * SEL_THREADS;
  const dim3 grid((unsigned)(((int64_t)a.N + chunk - 1) / chunk), a.B * a.Hd), block(SEL_THREADS);
  const bool quads = a.N % a.page == 0 && (reinterpret_cast<uintptr_t>(a.scores) % 16) == 0 &&
                     (a.agg == nullptr || (reinterpret_cast<uintptr_t>(a.agg) % 16) == 0);
  if (quads) STS_LAUNCH(select_aggblock_kernel<false>, grid, block, 0, s, a, chunk);
  else STS_LAUNCH(select_aggblock_kernel<true>, grid, block, 0, s, a, chunk);
  return sts_take_launch_status();
}

// one workgroup per row, Tq == 1, unpaged, no aggregate output; the caller has checked the shape
bool select_rowpass_ok(const SelectArgs &a) {
  return a.Tq == 1 && a.kind == STS_SCORES_PROBS && a.page == 1 && a.agg == nullptr && a.N > 0 &&
         (a.N % (a.scores_bf16 ? 8 : 4)) == 0 && (reinterpret_cast<uintptr_t>(a.scores) % 16) == 0;
}

hipError_t launch_select_rowpass(const SelectArgs &a, hipStream_t s) {
  if ((size_t)a.B * a.Hd == 0) return hipSuccess;
  if (!select_rowpass_ok(a)) return hipErrorInvalidValue;
  const dim3 grid(a.B * a.Hd);
  if (a.rowpass_threads == 1024) {
    if (a.scores_bf16) STS_LAUNCH((select_rowpass_kernel<1024, true>), grid, dim3(1024), 0, s, a);
    else STS_LAUNCH((select_rowpass_kernel<1024, false>), grid, dim3(1024), 0, s, a);
  } else {
    if (a.scores_bf16) STS_LAUNCH((select_rowpass_kernel<256, true>), grid, dim3(256), 0, s, a);
    else STS_LAUNCH((select_rowpass_kernel<256, false>), grid, dim3(256), 0, s, a);
  }
  return sts_take_launch_status();
}

hipError_t launch_select_local(const SelectArgs &a, hipStream_t s) {
  if ((size_t)a.B * a.Hd == 0 || a.pool_nchunks == 0) return hipSuccess;
  const dim3 grid(a.pool_nchunks, a.B * a.Hd);
  if (a.pool_chunk == 256 * 32)
    STS_LAUNCH(select_local_kernel<256>, grid, dim3(256), 0, s, a);
  else   // 1024 * 32
    STS_LAUNCH(select_local_kernel<1024>, grid, dim3(1024), 0, s, a);
  return sts_take_launch_status();
}

hipError_t launch_select_pool(const SelectArgs &a, hipStream_t s) {
  if ((size_t)a.B * a.Hd == 0) return hipSuccess;
  STS_LAUNCH(select_pool_kernel, dim3(a.B * a.Hd), dim3(SMALL_THREADS), 0, s, a);
  return sts_take_launch_status();
}

hipError_t launch_select_block(const SelectArgs &a, hipStream_t s) {
  if ((size_t)a.B * a.Hd == 0 || a.srcN == 0) return hipSuccess;
  const dim3 grid((a.srcN + SEL_THREADS - 1) / SEL_THREADS, a.B * a.Hd), block(SEL_THREADS);
  STS_LAUNCH(select_block_kernel, grid, block, 0, s, a);
  return sts_take_launch_status();
}

hipError_t launch_select_clear(const SelectArgs &a, hipStream_t s) {
  const size_t n = (size_t)a.clear_words;
  if (n == 0) return hipSuccess;
  STS_LAUNCH(select_clear_kernel, dim3((unsigned)((n + SEL_THREADS - 1) / SEL_THREADS)),
                     dim3(SEL_THREADS), 0, s, a.hist, n);
  return sts_take_launch_status();
}

hipError_t launch_select_agg(const SelectArgs &a, hipStream_t s) {
  const int chunks = (a.N + SEL_CHUNK - 1) / SEL_CHUNK;
  if ((size_t)a.B * a.Hd == 0 || chunks == 0) return hipSuccess;
  if (!a.hist) {                                       // no histogram: the sums alone
    const dim3 sums((a.N + 4 * SEL_THREADS - 1) / (4 * SEL_THREADS), a.Hd, a.B);
    if (a.N < 4) return hipErrorInvalidValue;
    if (a.scores_bf16) STS_LAUNCH(select_row_sums_kernel<true>, sums, dim3(SEL_THREADS), 0, s, a);
    else STS_LAUNCH(select_row_sums_kernel<false>, sums, dim3(SEL_THREADS), 0, s, a);
    return sts_take_launch_status();
  }
  const dim3 grid(chunks, a.B * a.Hd), block(SEL_THREADS);
  if (vec_ok(a))
    STS_LAUNCH(select_agg_kernel<true>, grid, block, 0, s, a);
  else
    STS_LAUNCH(select_agg_kernel<false>, grid, block, 0, s, a);
  return sts_take_launch_status();
}

hipError_t launch_select_hist(const SelectArgs &a, int pass, hipStream_t s) {
  if ((size_t)a.B * a.Hd == 0 || a.nchunks == 0) return hipSuccess;
  const dim3 grid((a.nchunks + a.hist_cpw - 1) / a.hist_cpw, a.B * a.Hd), block(SEL_THREADS);
  const bool v = src_vec_ok(a);
  if (pass == 1) {
    if (v) STS_LAUNCH((select_hist_kernel<1, true>), grid, block, 0, s, a);
    else STS_LAUNCH((select_hist_kernel<1, false>), grid, block, 0, s, a);
  } else {
    if (v) STS_LAUNCH((select_hist_kernel<2, true>), grid, block, 0, s, a);
    else STS_LAUNCH((select_hist_kernel<2, false>), grid, block, 0, s, a);
  }
  return sts_take_launch_status();
}

hipError_t launch_select_write(const SelectArgs &a, hipStream_t s) {
  if ((size_t)a.B * a.Hd == 0) return hipSuccess;
  const dim3 grid(a.nchunks > 0 ? a.nchunks : 1, a.B * a.Hd), block(SEL_THREADS);
  if (src_vec_ok(a))
    STS_LAUNCH(select_write_kernel<true>, grid, block, 0, s, a);
  else
    STS_LAUNCH(select_write_kernel<false>, grid, block, 0, s, a);
  return sts_take_launch_status();
}
