// Two-dimensional masks of prefill (paper Section 4.2: during prefill every query token has an
// index set of its own). For a block of up to 16 query rows the attention kernel gathers the
// UNION of the rows' sets once and is told, per gathered token, which rows keep it. This kernel
// builds that form from per-row lists: for every (batch, target head) the ascending union of the
// lists of its draft head's rows, and a 16-bit word per union entry, bit i set iff row i keeps
// the token.
//
// One 1024-thread workgroup per (draft head, batch); the union is the same for every target head
// that reads the draft head and is written to each of them. The token range is walked in chunks
// of 32768 tokens whose row bits sit in LDS (16 bits per token): every list entry that falls
// into the chunk ORs its row's bit into its token's half word (one entry of every row per thread
// in flight: the lists come out of L2, and a thread that waited for each entry in turn spent
// most of its time waiting); then every wave takes 2048 consecutive tokens, 64 at a time: a ballot says which of them are kept
// and where they go, and they are stored from the registers, a run of neighbouring places per instruction. What bounds it:
// the lists' reading and the latencies of the phases. 16 blocks x 16 draft heads of 16 x 6554 entries, 64K tokens: 57 us
// (65 with 32 tokens per thread, whose entries went one by one to a stage in LDS and from there, coalesced, to each target head).
// A chunk with fewer entries than a third of its tokens has them put together in LDS first, since a store instruction would be nearly
// empty: 4 blocks of 16 x 6000 entries over 98304 tokens 63.7 us (69.0 from the registers), 24 of 16 x 6554 over 128K 239 (250).
// The searches for the segments' ends go side by side (one after the other, and the bits cleared twice, the same 24 blocks took 239 us
// instead of 232, 16 of 16 x 2622 65.5 instead of 62.3: more than the form before the stores by ballots, 236 and 65.0).
// Rejected: no search, each chunk starting where the one before met its first entry past the end, and two steps of entries under way
// (75 to 87 us: sixteen scalar addresses and limits per step cost more than the search).
#include "common.h"

namespace {

constexpr int UN_THREADS = 1024;
constexpr int UN_CHUNK = 32768;            // tokens per LDS pass
constexpr int UN_MAX_SEG = 64;             // chunks up to which the lists are read by segments (2M tokens)
constexpr int UN_STEPS = UN_CHUNK / UN_THREADS;      // tokens per lane
constexpr int UN_STAGE = 10240;            // entries of a chunk up to which they are put together in LDS: 4 + 2 bytes each where the bits were
static_assert(6 * UN_STAGE <= 2 * UN_CHUNK && UN_STAGE % 4 == 0, "room, and whole 16-byte pieces to clear");

__global__ void __launch_bounds__(UN_THREADS) union_rows_kernel(const UnionArgs A) {
  typedef uint16_t row_bits __attribute__((may_alias));
  typedef u32x4 four_words __attribute__((may_alias));
  __shared__ __attribute__((aligned(16))) uint32_t bits[UN_CHUNK / 2];   // row bits of the chunk's tokens, two tokens per word
  __shared__ uint32_t wave_tot[UN_THREADS / 64];
  __shared__ int tgt[STS_MAX_HEADS];               // target heads that read this draft head
  __shared__ int ntgt_s;
  const int j = blockIdx.x, bt = blockIdx.y;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  auto uniform = [](int x) { return __builtin_amdgcn_readfirstlane(x); };
  if (tid == 0) ntgt_s = 0;
  for (int i = tid; i < UN_CHUNK / 8; i += UN_THREADS) reinterpret_cast<four_words *>(bits)[i] = u32x4{0u, 0u, 0u, 0u};
  __syncthreads();
  if (tid < A.Hq && A.map[tid] == j) tgt[atomicAdd(&ntgt_s, 1)] = tid;      // (Hq <= 256; in any order)
  __shared__ int cnts[16];                         // entries of each row's list
  if (tid < 16) cnts[tid] = tid < A.Tq ? (A.row_cnt ? min(max(A.row_cnt[((size_t)bt * A.Hd + j) * A.Tq + tid], 0), A.k) : A.k) : 0;
  __syncthreads();
  const int ntgt = uniform(ntgt_s);
  if (ntgt == 0) return;
  const int32_t *lists = A.row_idx + ((size_t)bt * A.Hd + j) * A.Tq * (size_t)A.k;      // [Tq][k]
  const size_t out_row = (size_t)bt * A.Hq;        // outputs of target t: (out_row + t) * pitch
  // Lists as the selection writes them are ascending, so the entries of a chunk are one segment
  // of each list, and reading only that segment per chunk reads every list once instead of once
  // per chunk (at 128K tokens the re-reads were three quarters of this kernel's traffic). The
  // segment ends come from searches, a wave per list where there are few ends, else a thread per list and end. Nothing is taken on
  // trust: the segments cover every list completely, and an entry that names a token outside
  // the chunk of the segment it was read in (a list that is not ascending) sets a flag, after which
  // the whole union is built again the plain way, every chunk reading every entry.
  const int nchunks = (A.N + UN_CHUNK - 1) / UN_CHUNK;
  __shared__ int seg[16][UN_MAX_SEG + 1];          // seg[i][c]: first entry of row i at or past chunk c's start
  __shared__ int out_of_place;
  bool by_segments = nchunks > 1 && nchunks <= UN_MAX_SEG;
  if (by_segments) {
    if (tid == 0) out_of_place = 0;
    if (nchunks <= 4) {
      // few ends: a wave per list, 64 probes a step for each of them (three memory latencies instead of thirteen)
      const int32_t *row = lists + (size_t)min(wave, A.Tq - 1) * A.k;
      const int n_row = uniform(cnts[wave]);
      int lo[3], len[3];                               // of the ends 1 .. nchunks - 1
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        lo[c] = 0;
        len[c] = c + 1 < nchunks ? n_row : 0;
      }
      while (len[0] | len[1] | len[2]) {
        int probe[3];
#pragma unroll
        for (int c = 0; c < 3; ++c) probe[c] = row[min(lo[c] + min(lane * ((len[c] + 63) / 64), max(len[c] - 1, 0)), n_row - 1)];
#pragma unroll
        for (int c = 0; c < 3; ++c) {
          const int step = (len[c] + 63) / 64;
          const int n = __builtin_popcountll(__builtin_amdgcn_ballot_w64(lane * step < len[c] && probe[c] < (c + 1) * UN_CHUNK));
          // (probes 0 .. n - 1 lie below the end)
          lo[c] += n ? (n - 1) * step + 1 : 0;
          len[c] = n ? min(step - 1, len[c] - (n - 1) * step - 1) : 0;
        }
      }
      if (lane == 0) {
        seg[wave][0] = 0;
        seg[wave][nchunks] = n_row;
#pragma unroll
        for (int c = 1; c < 4; ++c)
          if (c < nchunks) seg[wave][c] = lo[c - 1];
      }
    } else for (int x = tid; x < 16 * (nchunks + 1); x += UN_THREADS) {
      const int i = x / (nchunks + 1), c = x % (nchunks + 1);
      int lo = 0, hi = cnts[i];                    // lower bound of c * UN_CHUNK in row i
      if (c == 0) hi = 0;
      else if (c == nchunks) lo = hi;
      const int32_t *row = lists + (size_t)i * A.k;
      while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if (row[mid] < c * UN_CHUNK) lo = mid + 1;
        else hi = mid;
      }
      seg[i][c] = lo;
    }
    __syncthreads();
  }
  uint32_t written = 0;                            // union entries before the current chunk
  for (int base = 0; base < A.N; base += UN_CHUNK) {
    const int ch = base / UN_CHUNK;
    // one entry of every row per thread and step: up to 16 loads in flight
    int span = A.k;                                // entries per row to look at: the longest segment
    if (by_segments) {
      span = 0;
      for (int i = 0; i < A.Tq; ++i) span = max(span, seg[i][ch + 1] - seg[i][ch]);
    }
    for (int e = tid; e < span; e += UN_THREADS) {
      int n[16];
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        const int lo = by_segments ? seg[i][ch] : 0, hi = by_segments ? seg[i][ch + 1] : cnts[i];
        n[i] = (i < A.Tq && lo + e < hi) ? lists[(size_t)i * A.k + lo + e] : -1;
      }
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        const int off = n[i] - base;
        // entries outside the cache (the -1 padding, anything else out of range) name no token
        if (n[i] >= 0 && n[i] < A.N) {
          if (off >= 0 && off < UN_CHUNK) atomicOr(&bits[off >> 1], (1u << i) << (16 * (off & 1)));
          else if (by_segments) out_of_place = 1;
        }
      }
    }
    __syncthreads();
    if (by_segments && out_of_place) {               // uniform: start again, every chunk reading every entry
      by_segments = false;
      written = 0;
      base = -UN_CHUNK;
      for (int i = tid; i < UN_CHUNK / 8; i += UN_THREADS) reinterpret_cast<four_words *>(bits)[i] = u32x4{0u, 0u, 0u, 0u};
      __syncthreads();
      continue;
    }
    // the wave's 2048 tokens, lane by lane
    const row_bits *const own = reinterpret_cast<const row_bits *>(bits) + wave * (64 * UN_STEPS) + lane;
    uint32_t w[UN_STEPS], kept = 0;
#pragma unroll
    for (int x = 0; x < UN_STEPS; ++x) w[x] = own[64 * x];
#pragma unroll
    for (int x = 0; x < UN_STEPS; ++x) kept += (uint32_t)__builtin_popcountll(__builtin_amdgcn_ballot_w64(w[x] != 0u));
    if (lane == 0) wave_tot[wave] = kept;
    __syncthreads();
    uint32_t at = written, total = 0;              // where the wave's entries go
#pragma unroll
    for (int x = 0; x < UN_THREADS / 64; ++x) {
      const uint32_t v = wave_tot[x];
      at += x < wave ? v : 0u;
      total += v;
    }
    at = (uint32_t)uniform((int)at);
    const uint32_t room = (uint32_t)A.pitch;       // a pitch below the union's size truncates the list
    if (total <= (uint32_t)UN_STAGE) {
      // few entries: put next to each other in LDS, from where every store instruction is full (the bits' place)
      int32_t *const stg_idx = reinterpret_cast<int32_t *>(bits);
      row_bits *const stg_mask = reinterpret_cast<row_bits *>(bits + UN_STAGE);
      uint32_t p = at - written;
#pragma unroll
      for (int x = 0; x < UN_STEPS; ++x) {
        const uint64_t b = __builtin_amdgcn_ballot_w64(w[x] != 0u);
        const uint32_t place = __builtin_amdgcn_mbcnt_hi((uint32_t)(b >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)b, p));
        if (w[x] != 0u) {
          stg_idx[place] = base + wave * (64 * UN_STEPS) + 64 * x + lane;
          stg_mask[place] = (uint16_t)w[x];
        }
        p += (uint32_t)__builtin_popcountll(b);
      }
      __syncthreads();
      const uint32_t n = written < room ? min(total, room - written) : 0u;
      for (int ti = 0; ti < ntgt; ++ti) {
        const size_t o = (out_row + uniform(tgt[ti])) * (size_t)A.pitch + written;
        for (uint32_t i = tid; i < n; i += UN_THREADS) {
          A.indices[o + i] = stg_idx[i];
          A.row_mask[o + i] = stg_mask[i];
        }
      }
      __syncthreads();
    } else for (int ti = 0; ti < ntgt; ++ti) {
      const size_t o = (out_row + uniform(tgt[ti])) * (size_t)A.pitch;
      int32_t *const idx = A.indices + o;
      uint16_t *const msk = A.row_mask + o;
      uint32_t p = at;
#pragma unroll
      for (int x = 0; x < UN_STEPS; ++x) {
        const uint64_t b = __builtin_amdgcn_ballot_w64(w[x] != 0u);
        const uint32_t place = __builtin_amdgcn_mbcnt_hi((uint32_t)(b >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)b, p));
        if (w[x] != 0u && place < room) {
          idx[place] = base + wave * (64 * UN_STEPS) + 64 * x + lane;
          msk[place] = (uint16_t)w[x];
        }
        p += (uint32_t)__builtin_popcountll(b);
      }
    }
    written += (uint32_t)uniform((int)total);
    // nothing there for the next chunk (a stage is free, every wave has its words)
    for (int i = tid; i < UN_CHUNK / 8; i += UN_THREADS) reinterpret_cast<four_words *>(bits)[i] = u32x4{0u, 0u, 0u, 0u};
    __syncthreads();                                  // wave_tot is rewritten next round
  }
  const uint32_t c = min(written, (uint32_t)A.pitch);
  for (int ti = 0; ti < ntgt; ++ti) {
    const size_t o = (out_row + tgt[ti]) * (size_t)A.pitch;
    for (uint32_t p = c + tid; p < (uint32_t)A.pitch; p += UN_THREADS) {
      A.indices[o + p] = -1;
      A.row_mask[o + p] = 0;
    }
    if (tid == 0 && A.counts) A.counts[out_row + tgt[ti]] = (int32_t)c;
  }
}

}  // namespace

hipError_t launch_union_rows(const UnionArgs &a, hipStream_t s) {
  if ((size_t)a.B * a.Hq == 0) return hipSuccess;
  STS_LAUNCH(union_rows_kernel, dim3(a.Hd, a.B), dim3(UN_THREADS), 0, s, a);
  return sts_take_launch_status();
}
