// Shared declarations of the STS HIP library (gfx950 only). Internal: the public surface is
// include/sts.h.
#pragma once

#include <hip/hip_runtime.h>
#include <hip/hip_ext.h>
#include <math.h>
#include <stdint.h>

#include <tuple>
#include <type_traits>
#include <utility>

#include "../../include/sts.h"

// Every kernel goes out through STS_LAUNCH. With the library's timing aid switched on, the host
// code sets this pair of events before a launch and the dispatch itself stamps them with the
// kernel's own begin and end times (no extra packets around it); otherwise it is an ordinary
// launch. The status is the launch call's own return value (an error that some earlier, unrelated
// HIP call of the process left behind is neither reported as ours nor cleared); a launcher hands
// it back with sts_take_launch_status().
struct StsLaunchEvents { hipEvent_t start, stop; };
extern thread_local StsLaunchEvents g_sts_launch_events;
extern thread_local hipError_t g_sts_launch_rc;

template <class Tuple, size_t... I>
inline void sts_arg_pointers(Tuple &vals, void **ptrs, std::index_sequence<I...>) {
  ((ptrs[I] = static_cast<void *>(&std::get<I>(vals))), ...);
}

template <class... P, class... A>
inline void sts_launch(void (*kernel)(P...), dim3 grid, dim3 block, unsigned shmem, hipStream_t stream, const A &...args) {
  std::tuple<std::remove_cv_t<P>...> vals(args...);      // copies of the kernel's own parameter types
  void *ptrs[sizeof...(P)];
  sts_arg_pointers(vals, ptrs, std::index_sequence_for<P...>{});
  const hipError_t rc =
      g_sts_launch_events.start || g_sts_launch_events.stop
          ? hipExtLaunchKernel(reinterpret_cast<const void *>(kernel), grid, block, ptrs, shmem, stream,
                               g_sts_launch_events.start, g_sts_launch_events.stop, 0)
          : hipLaunchKernel(reinterpret_cast<const void *>(kernel), grid, block, ptrs, shmem, stream);
  if (g_sts_launch_rc == hipSuccess) g_sts_launch_rc = rc;
}
#define STS_LAUNCH(kernel, grid, block, shmem, stream, ...) sts_launch(kernel, grid, block, shmem, stream, __VA_ARGS__)

// status of the launches since the last call of this function (the first failure, if any)
inline hipError_t sts_take_launch_status() {
  const hipError_t rc = g_sts_launch_rc;
  g_sts_launch_rc = hipSuccess;
  return rc;
}

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

constexpr int STS_MAX_HEADS = 256;   // Hq, Hd upper bound (tables travel as kernel arguments)
constexpr int STS_MAX_GROUP = 16;    // query heads per KV head
constexpr int STS_TILE_KEYS = 32;    // keys per wave tile
constexpr int STS_WG_WAVES = 4;      // waves per attention workgroup
constexpr int STS_XCDS = 8;          // accelerator dies, each with an L2 of its own; workgroups go round them in turn
constexpr int STS_GRID_Z = 32768;    // batch elements in the last dimension of a grid at most

// A work unit of the attention kernels: the query heads of one KV group that share one index
// row (sparse) or all heads of the group (dense). Packed: bits 0-7 KV head, 8-23 mask of the
// member heads within the group, 24-28 number of member heads.
struct AttnUnitTable {
  uint32_t unit[STS_MAX_HEADS];
};

struct AttnArgs {
  const uint16_t *q, *k, *v;
  const int32_t *indices, *counts, *seq_lens;
  const uint16_t *row_mask;               // [B,Hq,kmax] laid out like indices: bit i = query row i keeps the entry; or NULL
  int64_t stride_b, stride_h, stride_n;   // elements
  int64_t idx_stride_b, cnt_stride_b;     // elements between batches of indices / counts
  int32_t B, Tq, Hq, Hkv, G, N, kmax;
  int32_t num_units, num_splits;
  int32_t z_rounds;                       // batch elements / STS_GRID_Z, rounded up
  int32_t page, page_shift;               // tokens per index entry / page (power of two <= 32)
  const int32_t *block_table;             // [B, table_stride] logical block -> physical page, or NULL
  int32_t table_stride, num_pages;
  int64_t stride_page;                    // elements between pages of the pool
  const uint16_t *k_new, *v_new;          // [B,Tq,Hkv,d] the block's own keys/values, or NULL
  int32_t causal;
  int32_t direct;                         // single split: the split kernel writes the result itself
  float scale_log2;                       // scale * log2(e)
  float scale;
  float *part_o;                          // [B*U*S][NQ*16][D]
  float *part_ml;                         // [B*U*S][NQ*16][2]  (max in log2 domain, sum)
  void *logits_out;
  int32_t logits_bf16;
  float *agg_out;                         // [B,Hq,N] summed attention weights of the query block (dense only), or NULL
  int32_t ps_heads, ps_sets, ps_splits;   // second pass: heads per workgroup, such sets per KV head, key-range splits
  int32_t ps_tp;                          // second pass: rows per head, Tq rounded up to a power of two
  void *out;
  float *lse_out;
  int32_t out_dtype;
  AttnUnitTable units;
};

struct AttnPlan {
  int32_t nq;          // query tiles of 16 rows per unit (1, 2 or 4)
  int32_t num_units;   // per batch element
  int32_t num_splits;
  size_t part_o_bytes, part_ml_bytes, lse_bytes;
  AttnUnitTable units;
};

// select ------------------------------------------------------------------------------------

constexpr int SEL_BITS0 = 11, SEL_BITS1 = 11, SEL_BITS2 = 10;
constexpr int SEL_BINS = 2048;          // bins of the widest digit
constexpr int SEL_CHUNK = 8192;         // tokens per workgroup in the scan kernels
constexpr int SEL_THREADS = 256;
constexpr int SEL_SMALL_N = 32768;      // scores of a row that the one-workgroup-per-row selection holds in registers at most
constexpr int SEL_ROW_N = 65536;        // the same for one fp32 score per token, in calls of up to 512 rows
constexpr int SEL_RANK_N = 2048;        // block sums of a row up to which they are ranked out of LDS
constexpr int SEL_ROW16 = 16;
constexpr int SEL_ROW16_N = 131072;     // tokens of one bf16 score each that a workgroup's registers hold
constexpr int SEL_FLAG_PITCH = 32;      // words between the published counts of two chunks: one 128-byte line each
constexpr int SEL_FUSED_N = 8192;
constexpr int SEL_FUSED_MAX_PARTS = 8;   // units of 32768 tokens up to which small calls take the sampled selection
                                         // (256K tokens; large calls and a test knob: up to 256)
// The forms of the sampled selection: most tokens per workgroup (a bit each in LDS) and entries of its band list.
// The bits and the list share the LDS.
constexpr int SMP_FORMS = 4;
constexpr int SMP_TOKENS[SMP_FORMS] = {65536, 131072, 262144, 524288}, SMP_LIST[SMP_FORMS] = {16384, 15360, 13312, 8192};
constexpr int SMP_MAX_TOKENS = SMP_TOKENS[SMP_FORMS - 1];
// how many keys of a row of nb tokens with budget c are sampled where a workgroup holds part_tokens: see sample_plan
__host__ __device__ inline int smp_sample(int64_t nb, int64_t c, int part_tokens) {
  return nb > 262144 || part_tokens > 131072 || (part_tokens > 65536 && 8 * c >= nb) ? 8192 : 4096;
}
constexpr int SMP_WORDS = 1352;         // 64-bit words a part exchanges with the other parts of its row
constexpr int SEL_POOL_MAX = 16384;     // chunk-local winners per row that the pool kernel ranks out of LDS       // rows up to this many tokens always take it

// Tokens in the band of keys around the threshold that such a sample is expected to give: 5 standard deviations of
// the sample's count on either side, and half as much again where bins are coarse. < 0: no lower edge (the budget is next
// to the row's length).
inline int64_t smp_expected_band(int64_t nb, int64_t c, int part_tokens) {
  const double ns = nb < smp_sample(nb, c, part_tokens) ? (double)nb : (double)smp_sample(nb, c, part_tokens);
  const double cs = (double)c * ns / (double)nb, margin = 5.0 * sqrt(cs) + 4.0;
  if (cs + margin > ns) return -1;
  return (int64_t)(1.5 * (margin + (cs < margin ? cs : margin)) * (double)nb / ns);
}

struct SelectTargets {
  // targets of draft head j: tgt[off[j] .. off[j+1]); the kernels read both by words (target_off, target_head)
  alignas(4) uint16_t off[STS_MAX_HEADS + 1];
  alignas(4) uint8_t tgt[STS_MAX_HEADS];
};

struct SelectArgs {
  const void *scores;         // fp32 or bf16 (scores_bf16)
  const float *lse;
  int32_t scores_bf16;
  const int32_t *seq_lens;
  int32_t *indices, *counts;
  float *agg;                 // [B,Hd,N] (agg_out or workspace)
  float *blk;                 // [B,Hd,NB] per-block sums (page > 1), else unused
  const float *src;           // what is ranked: agg (page == 1) or blk
  int32_t srcN;               // row length of src: N or NB
  int32_t page;               // tokens per block (>= 1); rows of block sums that are ranked as scores have their lengths in tokens
  uint32_t *hist;             // [rows][3][SEL_BINS]
  uint32_t *state;            // [rows][8]: digits 0/1 and remaining k after each, [6] budget
  uint32_t *chunk_cnt;        // [rows][nchunks][SEL_FLAG_PITCH], word 0: published flag | equal count << 14 | greater count
  uint32_t *pool_key;         // [rows][pool_nchunks * pool_pitch] chunk-local winners (small budgets), token
                              // order, contiguous per row: chunk c starts at c * min(budget of the row, pool_chunk)
  int32_t *pool_idx;          // their token ids
  int32_t pool_chunk;         // tokens per chunk of the local kernel: 8192 or 32768
  int32_t pool_nchunks;       // ceil(N / pool_chunk)
  int32_t pool_pitch;         // min(k, pool_chunk)
  uint64_t clear_words;       // words to zero from `hist` on: histograms, state and chunk flags
  int32_t hist_cpw;           // consecutive chunks per workgroup of the refinement histograms (1, 2 or 4)
  int32_t spin_limit;         // polls of an unpublished earlier chunk before it is recounted locally
  void *pub;                  // sampled selection: [rows][smp_parts][SMP_WORDS] 64-bit words that the parts of a row
                              // exchange (top bit: written), zero before the launch
  int32_t smp_tokens, smp_parts;   // tokens per workgroup (a multiple of 256), workgroups per row
  int32_t fused_spin_limit;   // polls of another part's words before the row is ranked by plain passes instead
  int32_t rowpass_threads;    // one workgroup per row (select_rowpass_kernel): 256 or 1024 threads; SEL_ROW16: rows of one
                              // bf16 score per token in registers (select_row16_kernel)
  int32_t agg_is_input;       // `agg` is the caller's score tensor itself (one fp32 probability row per head): never stored to
  int32_t B, Hd, Tq, N, Hq, k, kind, reduce, nchunks;   // k: row pitch of indices = largest budget
  SelectTargets targets;
  int32_t kh[STS_MAX_HEADS];  // budget of draft head j (<= k)
};

// union of per-row index lists (union.hip)
struct UnionArgs {
  const int32_t *row_idx;     // [B,Hd,Tq,k]
  const int32_t *row_cnt;     // [B,Hd,Tq] or nullptr (= k)
  int32_t *indices;           // [B,Hq,pitch]
  uint16_t *row_mask;         // [B,Hq,pitch]
  int32_t *counts;            // [B,Hq] or nullptr
  int32_t B, Hd, Hq, Tq, N, k, pitch;
  uint8_t map[STS_MAX_HEADS]; // target head -> draft head
};
hipError_t launch_union_rows(const UnionArgs &a, hipStream_t s);

// device address of the current device's copy of the static scratch array (scratch.hip)
sts_status sts_static_scratch(void **out);

// launches (defined in the .hip files); each returns the status of its own launch call
// Do the workgroups of a sparse call gather from one cache closely enough to be placed by die and to keep what they load in
// the caches (attn.hip)? Batch elements that share one (stride 0), and either some rows asked for several times, or little
// asked for in all. us there and streamed, each workgroup where it falls: 16 blocks of 16 rows, 6554 kept of 65536 214, 375; 16 of
// five rows, 13107 of 131072 129, 185; 2 blocks, 9830 of 32768 26, 29. With rows
// asked for 0.4 times on average and more than a cache holds: 2 blocks, 100000 of 1M 271, 249, 50000 of 500000 136, 129, but 26214 of
// 262144 (0.4 times, 429 MB) 67.5, 68.5; 4 blocks, 20000 of 1M (0.16 times, 655 MB) 114, 106; at 0.6 times 187 to 191 either way, at 0.64 161, 181.
// Where this means eight waves instead of four (two query tiles at head size 128), a workgroup needs more than eight tiles
// to make up for the merging of twice the waves, and rows asked for 0.25 times: lists of 128 9.7, 7.6, of 600 in three
// parts 14.3, 13.0; ten tiles of 32 keys are even, 19 17.9, 20.2; 16 blocks, 600 of 131072 18.2, 17.3, 1200 27.2, 28.7.
inline bool attn_shares_cache(const AttnArgs &a, int d, bool eight_waves) {
  if (a.stride_b != 0 || a.B <= 1 || a.B > STS_GRID_Z || a.kmax >= 1 << 30) return false;       // (32-bit offsets into a list)
  const int64_t tokens = (int64_t)a.kmax << a.page_shift, tiles = (tokens + STS_TILE_KEYS - 1) / STS_TILE_KEYS;
  const int64_t asked = (int64_t)a.B * a.num_units * tokens, rows = (int64_t)a.N * a.Hkv;
  if (5 * asked <= 3 * rows && asked > (400ll << 20) / (4 * d)) return false;
  return !eight_waves || ((tiles + a.num_splits - 1) / a.num_splits > 8 && 4 * asked >= rows);
}

hipError_t launch_attn_split(const AttnArgs &a, int d, int nq, bool sparse, hipStream_t s);
hipError_t launch_attn_combine(const AttnArgs &a, int d, int nq, hipStream_t s);
hipError_t launch_attn_probsum(const AttnArgs &a, int d, int nq, hipStream_t s);
int attn_probsum_wgs_per_cu(int d, int nq);
hipError_t launch_select_clear(const SelectArgs &a, hipStream_t s);
hipError_t launch_select_agg(const SelectArgs &a, hipStream_t s);
hipError_t launch_select_block(const SelectArgs &a, hipStream_t s);
hipError_t launch_select_small(const SelectArgs &a, hipStream_t s);
hipError_t launch_select_row(const SelectArgs &a, hipStream_t s);
hipError_t launch_select_rank(const SelectArgs &a, hipStream_t s);
bool select_aggblock_ok(const SelectArgs &a);
hipError_t launch_select_aggblock(const SelectArgs &a, hipStream_t s);
hipError_t launch_select_fused(const SelectArgs &a, hipStream_t s);
hipError_t launch_select_clear_pub(const SelectArgs &a, hipStream_t s);
hipError_t launch_select_band(const SelectArgs &a, hipStream_t s);
bool select_rowpass_ok(const SelectArgs &a);
hipError_t launch_select_rowpass(const SelectArgs &a, hipStream_t s);
hipError_t launch_select_local(const SelectArgs &a, hipStream_t s);
hipError_t launch_select_pool(const SelectArgs &a, hipStream_t s);
hipError_t launch_select_hist(const SelectArgs &a, int pass, hipStream_t s);
hipError_t launch_select_write(const SelectArgs &a, hipStream_t s);
hipError_t launch_headmap_clear(unsigned long long *overlap, int n, hipStream_t s);
hipError_t launch_headmap_overlap(const int32_t *idx_d, const int32_t *idx_t, int S, int R, int Hd, int Ht, int N,
                                  int k, int c, unsigned long long *overlap, hipStream_t s);
hipError_t launch_headmap_argmax(const unsigned long long *overlap, int Hd, int Ht, int32_t *map, hipStream_t s);
