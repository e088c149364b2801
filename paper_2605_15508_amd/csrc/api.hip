// Host side of the C ABI declared in include/sts.h: argument validation, launch planning,
// workspace carving, kernel enqueue, and the optional per-kernel event timing.
#include <math.h>
#include <stdlib.h>
#include <string.h>

#include <algorithm>
#include <mutex>
#include <vector>

#include "common.h"

thread_local StsLaunchEvents g_sts_launch_events = {nullptr, nullptr};
thread_local hipError_t g_sts_launch_rc = hipSuccess;

namespace {

inline size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

// ------------------------------------------------------------------------- profiling aid
struct ProfEvent {
  hipEvent_t start, stop;
  int kind;
};
std::mutex g_prof_mu;
bool g_prof_on = false;
std::vector<ProfEvent> g_prof_pool;   // created lazily, reused after reset
size_t g_prof_used = 0;

template <class F>
hipError_t run_kernel(int kind, hipStream_t s, F &&launch) {
  if (!g_prof_on) return launch();
  std::lock_guard<std::mutex> lk(g_prof_mu);
  if (g_prof_used >= STS_PROF_MAX) return launch();
  if (g_prof_used == g_prof_pool.size()) {
    ProfEvent e;
    if (hipEventCreate(&e.start) != hipSuccess) return launch();
    if (hipEventCreate(&e.stop) != hipSuccess) {
      (void)hipEventDestroy(e.start);
      return launch();
    }
    g_prof_pool.push_back(e);
  }
  ProfEvent &e = g_prof_pool[g_prof_used];
  e.kind = kind;
  // the dispatch stamps the two events with the kernel's own begin and end (every launcher
  // enqueues exactly one kernel per call)
  g_sts_launch_events = StsLaunchEvents{e.start, e.stop};
  const hipError_t rc = launch();
  g_sts_launch_events = StsLaunchEvents{nullptr, nullptr};
  if (rc == hipSuccess) ++g_prof_used;
  return rc;
}

// ------------------------------------------------------------------------- tuning knobs
// Values set with sts_set_knob; before the first set or get of a knob its environment variable
// (read once per process) gives the initial value. NaN = not set: the library's own rule applies.
const char *const KNOB_ENV[STS_KNOB_COUNT_] = {"STS_ATTN_WGS_PER_CU", "STS_SELECT_SPIN_LIMIT",
                                               "STS_PROBSUM_WGS_PER_CU", "STS_SELECT_PATH",
                                               "STS_SELECT_ROW_THREADS"};
std::mutex g_knob_mu;
double g_knob[STS_KNOB_COUNT_];
bool g_knob_init = false;

void knobs_init_locked() {
  if (g_knob_init) return;
  for (int i = 0; i < STS_KNOB_COUNT_; ++i) {
    const char *e = getenv(KNOB_ENV[i]);
    g_knob[i] = (e && *e) ? atof(e) : NAN;
  }
  g_knob_init = true;
}

double knob(int which) {
  std::lock_guard<std::mutex> lk(g_knob_mu);
  knobs_init_locked();
  return g_knob[which];
}

int cu_count() {
  static const int cus = [] {   // once per process (thread-safe initialisation)
    int dev = 0, n = 0;
    if (hipGetDevice(&dev) == hipSuccess &&
        hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess && n > 0)
      return n;
    return 256;
  }();
  return cus;
}

// ------------------------------------------------------------------------ attention plan
sts_status validate_attn(const sts_attn_params *p, int sparse) {
  if (!p) return STS_EINVAL;
  if (p->B < 0 || p->Tq < 1 || p->Hq < 1 || p->Hkv < 1 || p->N < 0) return STS_EINVAL;
  if (p->Hq % p->Hkv != 0) return STS_EINVAL;
  if (p->d != 64 && p->d != 128) return STS_EUNSUPPORTED;
  if (p->Tq > 16 || p->Hq > STS_MAX_HEADS || p->Hq / p->Hkv > STS_MAX_GROUP) return STS_EUNSUPPORTED;
  if (p->out_dtype != STS_BF16 && p->out_dtype != STS_F32) return STS_EINVAL;
  if (!isfinite(p->scale)) return STS_EINVAL;
  if (p->row_mask && (!sparse || p->block_table)) return sparse ? STS_EUNSUPPORTED : STS_EINVAL;
  if (sparse) {
    if (p->kmax < 0) return STS_EINVAL;
    if (p->logits_out || p->seq_lens) return STS_EINVAL;
    if (p->head_map)
      for (int t = 0; t < p->Hq; ++t)
        if (p->head_map[t] < 0) return STS_EINVAL;
  } else {
    if (p->indices || p->counts) return STS_EINVAL;
  }
  if (p->kv_stride_n < p->d || (p->kv_stride_n * 2) % 16 != 0 || (p->kv_stride_h * 2) % 16 != 0 ||
      (p->kv_stride_b * 2) % 16 != 0)
    return STS_EUNSUPPORTED;
  const int page = p->page_size <= 1 ? 1 : p->page_size;
  if (page != 1 && page != 2 && page != 4 && page != 8 && page != 16 && page != 32) return STS_EUNSUPPORTED;
  if (p->block_table) {
    if (p->num_pages < 1 || p->kv_stride_page < 1 || (p->kv_stride_page * 2) % 16 != 0) return STS_EINVAL;
    if ((int64_t)p->table_stride * page < p->N) return STS_EINVAL;
  }
  if (sparse && (int64_t)p->kmax * page > 0x7fffffffll - 65536) return STS_EUNSUPPORTED;
  if (p->idx_stride_b < 0 || p->cnt_stride_b < 0) return STS_EINVAL;
  if (sparse && p->idx_stride_b && p->idx_stride_b < (int64_t)p->Hq * p->kmax) return STS_EINVAL;
  if (sparse && p->cnt_stride_b && p->cnt_stride_b < p->Hq) return STS_EINVAL;
  if ((p->k_new == nullptr) != (p->v_new == nullptr)) return STS_EINVAL;
  if (p->k_new && (reinterpret_cast<uintptr_t>(p->k_new) % 16 != 0 || reinterpret_cast<uintptr_t>(p->v_new) % 16 != 0))
    return STS_EUNSUPPORTED;
  return STS_OK;
}

int page_of(const sts_attn_params *p) { return p->page_size <= 1 ? 1 : p->page_size; }

// Group query heads into units and pick the split count. Uses only host data.
sts_status plan_attn(const sts_attn_params *p, int sparse, AttnPlan &pl) {
  const sts_status v = validate_attn(p, sparse);
  if (v != STS_OK) return v;
  const int G = p->Hq / p->Hkv;
  // at most 4 query tiles of 16 rows per unit; 2 for the logits dump at head size 128, whose
  // four-tile form would not fit the register file (a KV group with more rows is served by two
  // units, each reading K and V: next to the dump's own writes that costs little)
  int max_heads = ((!sparse && p->logits_out && p->d == 128) ? 32 : 64) / p->Tq;
  if (max_heads < 1) max_heads = 1;
  if (max_heads > STS_MAX_GROUP) max_heads = STS_MAX_GROUP;
  int nu = 0, max_rows = 0;
  memset(&pl.units, 0, sizeof(pl.units));
  for (int g = 0; g < p->Hkv; ++g) {
    bool done[STS_MAX_GROUP] = {false};
    for (int i = 0; i < G; ++i) {
      if (done[i]) continue;
      // members of the set led by head i, in head order
      int members[STS_MAX_GROUP], nm = 0;
      for (int j2 = i; j2 < G; ++j2) {
        if (done[j2]) continue;
        const bool same = !sparse || j2 == i ||
                          (p->head_map && p->head_map[g * G + j2] == p->head_map[g * G + i]);
        if (same) {
          members[nm++] = j2;
          done[j2] = true;
        }
      }
      for (int s0 = 0; s0 < nm; s0 += max_heads) {
        const int cnt = (nm - s0 < max_heads) ? nm - s0 : max_heads;
        uint32_t mask = 0;
        for (int m = 0; m < cnt; ++m) mask |= 1u << members[s0 + m];
        if (nu >= STS_MAX_HEADS) return STS_EUNSUPPORTED;
        pl.units.unit[nu++] = (uint32_t)g | (mask << 8) | ((uint32_t)cnt << 24);
        if (cnt * p->Tq > max_rows) max_rows = cnt * p->Tq;
      }
    }
  }
  pl.num_units = nu;
  pl.nq = max_rows <= 16 ? 1 : (max_rows <= 32 ? 2 : 4);
  const int64_t len = sparse ? (int64_t)p->kmax * page_of(p) : p->N;
  const int64_t tiles = (len + STS_TILE_KEYS - 1) / STS_TILE_KEYS;
  // Workgroups per CU the split count aims at. Two for the gather (its two dependent latencies
  // per tile want more waves) and for head size 64; one for the dense kernel at head size 128,
  // where a second workgroup per CU only costs (128K context, batch 4: 348 -> 324 us; 32K,
  // batch 1: 51 -> 44 us),
  // and for four query tiles (one workgroup fills the register file).
  // The gather with two query tiles at head size 128 (as register-bound as the dense kernel)
  // is 3% faster with one as well.
  int64_t resident = (int64_t)cu_count() * ((pl.nq == 4 || (p->d == 128 && (!sparse || pl.nq == 2))) ? 1 : 2);
  const double wgs_knob = knob(STS_KNOB_ATTN_WGS_PER_CU);   // tuning knob: target workgroups per CU
  const bool wgs_set = wgs_knob > 0.0;                       // (NaN compares false)
  if (wgs_set) resident = (int64_t)(cu_count() * wgs_knob);
  const int64_t units_total = (int64_t)p->B * nu;
  int64_t S = units_total > 0 ? resident / units_total : 1;
  // at least two tiles for each of four waves, so that the partials and their combine stay small next to
  // the gathered bytes (also for the form with eight, which with two tiles each is no faster: lists of 1200 over one cache 15.3,
  // 15.5 us); a list of up to 16 tiles is not split at all (its workgroup writes
  // the result itself, one launch instead of two)
  const int64_t s_cap = tiles <= 16 ? 1 : (tiles + 2 * STS_WG_WAVES - 1) / (2 * STS_WG_WAVES);
  if (S > s_cap) S = s_cap;
  if (S > 256) S = 256;
  // With at least one unit per CU, halving every unit only adds the combine launch: one
  // workgroup per CU keeps enough loads in flight (70B-shaped layer, 256 units of 410 tiles:
  // 268 us unsplit against 278 us in two halves).
  if (S == 2 && units_total >= cu_count() && !wgs_set) S = 1;
  if (S < 1) S = 1;
  pl.num_splits = (int)S;
  const size_t parts = (size_t)units_total * (size_t)S;
  if ((size_t)units_total * (size_t)S > 0x7fffffffull) return STS_EUNSUPPORTED;
  pl.part_o_bytes = align256(parts * (size_t)pl.nq * 16 * p->d * sizeof(float));
  pl.part_ml_bytes = align256(parts * (size_t)pl.nq * 16 * 2 * sizeof(float));
  pl.lse_bytes = (!sparse && p->weights_sum_out && !p->lse_out)
                     ? align256((size_t)p->B * p->Hq * p->Tq * sizeof(float)) : 0;
  return STS_OK;
}

// ws / ws_bytes: the scratch memory of the call (the caller's workspace, or the library's static
// array for the entry point that allocates nothing, which also keeps the timing aid off: creating
// events allocates).
sts_status run_attn(const sts_attn_params *p, int sparse, hipStream_t s, void *ws, size_t ws_bytes, bool timed) {
  AttnPlan pl;
  const sts_status v = plan_attn(p, sparse, pl);
  if (v != STS_OK) return v;
  if (p->B == 0) return STS_OK;
  if (!p->q || !p->out) return STS_EINVAL;
  if (p->N > 0 && (!p->k || !p->v)) return STS_EINVAL;
  if (sparse && p->kmax > 0 && !p->indices) return STS_EINVAL;
  if (sparse && p->kmax > 0 && p->N == 0) return STS_EINVAL;
  const size_t need = pl.part_o_bytes + pl.part_ml_bytes + pl.lse_bytes;
  if (!ws || ws_bytes < need) return STS_EWORKSPACE;
  if (reinterpret_cast<uintptr_t>(ws) % 256 != 0) return STS_EWORKSPACE;
  const bool want_sum = !sparse && p->weights_sum_out != nullptr;
  // (the second pass adds a 32-bit lane offset of up to 12 rows to a 64-bit tile address)
  if (want_sum && (p->block_table || p->k_new || page_of(p) != 1 ||
                   reinterpret_cast<uintptr_t>(p->weights_sum_out) % 4 != 0 ||
                   p->kv_stride_n < 0 || p->kv_stride_n > (int64_t)1 << 26))
    return STS_EUNSUPPORTED;
  if (reinterpret_cast<uintptr_t>(p->k) % 16 != 0 || reinterpret_cast<uintptr_t>(p->v) % 16 != 0 ||
      reinterpret_cast<uintptr_t>(p->q) % 16 != 0 || reinterpret_cast<uintptr_t>(p->out) % 16 != 0 ||
      reinterpret_cast<uintptr_t>(p->logits_out) % 16 != 0)
    return STS_EUNSUPPORTED;

  AttnArgs a;
  memset(&a, 0, sizeof(a));
  a.q = static_cast<const uint16_t *>(p->q);
  a.k = static_cast<const uint16_t *>(p->k);
  a.v = static_cast<const uint16_t *>(p->v);
  a.indices = sparse ? p->indices : nullptr;
  a.counts = sparse ? p->counts : nullptr;
  a.row_mask = sparse ? p->row_mask : nullptr;
  a.idx_stride_b = p->idx_stride_b ? p->idx_stride_b : (int64_t)p->Hq * p->kmax;
  a.cnt_stride_b = p->cnt_stride_b ? p->cnt_stride_b : p->Hq;
  a.seq_lens = sparse ? nullptr : p->seq_lens;
  a.stride_b = p->kv_stride_b;
  a.stride_h = p->kv_stride_h;
  a.stride_n = p->kv_stride_n;
  a.B = p->B; a.Tq = p->Tq; a.Hq = p->Hq; a.Hkv = p->Hkv; a.G = p->Hq / p->Hkv; a.N = p->N;
  a.kmax = sparse ? p->kmax : 0;
  a.page = page_of(p);
  a.page_shift = 0;
  while ((1 << a.page_shift) < a.page) ++a.page_shift;
  a.block_table = p->block_table;
  a.table_stride = p->table_stride;
  a.num_pages = p->num_pages;
  a.stride_page = p->kv_stride_page;
  a.k_new = static_cast<const uint16_t *>(p->k_new);
  a.v_new = static_cast<const uint16_t *>(p->v_new);
  a.causal = p->causal;
  a.direct = (pl.num_splits == 1) ? 1 : 0;
  a.num_units = pl.num_units;
  a.num_splits = pl.num_splits;
  a.z_rounds = (p->B + STS_GRID_Z - 1) / STS_GRID_Z;
  a.scale = p->scale;
  a.scale_log2 = p->scale * 1.44269504088896340736f;
  a.part_o = static_cast<float *>(ws);
  a.part_ml = reinterpret_cast<float *>(static_cast<unsigned char *>(ws) + pl.part_o_bytes);
  a.logits_out = sparse ? nullptr : p->logits_out;
  a.logits_bf16 = p->logits_bf16 ? 1 : 0;
  a.out = p->out;
  a.lse_out = p->lse_out;
  if (want_sum && !a.lse_out)   // the second pass needs the row normalisers
    a.lse_out = reinterpret_cast<float *>(static_cast<unsigned char *>(ws) + pl.part_o_bytes + pl.part_ml_bytes);
  a.out_dtype = p->out_dtype;
  a.units = pl.units;

  hipError_t rc = timed ? run_kernel(sparse ? STS_K_ATTN_SPARSE : STS_K_ATTN_DENSE, s,
                                     [&] { return launch_attn_split(a, p->d, pl.nq, sparse != 0, s); })
                        : launch_attn_split(a, p->d, pl.nq, sparse != 0, s);
  if (rc != hipSuccess) return STS_EHIP;
  if (!a.direct) {
    rc = timed ? run_kernel(STS_K_ATTN_COMBINE, s, [&] { return launch_attn_combine(a, p->d, pl.nq, s); })
               : launch_attn_combine(a, p->d, pl.nq, s);
    if (rc != hipSuccess) return STS_EHIP;
  }
  if (want_sum && p->N > 0) {
    // Second pass over K. Heads of a KV group share a workgroup in sets of up to 64 rows; the key
    // range is cut so that the grid is one full residency of the chip (a second, partly filled
    // round would cost more than finer balancing gains), each wave keeping at least 4 tiles.
    a.agg_out = p->weights_sum_out;
    int tp = 1;
    while (tp < p->Tq) tp *= 2;      // a head's rows fill an aligned power-of-two run of MFMA columns
    int hs = 64 / tp;
    if (hs > a.G) hs = a.G;
    a.ps_tp = tp;
    a.ps_heads = hs;
    a.ps_sets = (a.G + hs - 1) / hs;
    const int rows = hs * tp;
    const int nq = rows <= 16 ? 1 : (rows <= 32 ? 2 : 4);
    const int64_t tiles = ((int64_t)p->N + STS_TILE_KEYS - 1) / STS_TILE_KEYS;
    const int64_t groups = (int64_t)p->B * p->Hkv * a.ps_sets;
    double per_cu = attn_probsum_wgs_per_cu(p->d, nq);
    if (const double f = knob(STS_KNOB_PROBSUM_WGS_PER_CU); f > 0.0) per_cu = f;   // tuning knob
    int64_t S = (int64_t)(cu_count() * per_cu) / groups;
    const int64_t s_cap = (tiles + 4 * STS_WG_WAVES - 1) / (4 * STS_WG_WAVES);
    if (S > s_cap) S = s_cap;
    if (S < 1) S = 1;
    if (groups * S > 0x7fffffffll) return STS_EUNSUPPORTED;
    a.ps_splits = (int)S;
    rc = run_kernel(STS_K_ATTN_PROBSUM, s, [&] { return launch_attn_probsum(a, p->d, nq, s); });
    if (rc != hipSuccess) return STS_EHIP;
  }
  return STS_OK;
}

// --------------------------------------------------------------------------- select plan
struct SelectPlan {
  bool small;          // one workgroup per row, keys in registers, a single launch
  bool pool;           // shape allows chunk-local top-k + one ranking workgroup per row
  bool one_row;        // of those, the calls that one workgroup per row serves (the workspace is not touched)
  bool fused;          // long rows: the sampled selection, one launch (plus the clearing of the exchanged words)
  bool band;           // the same for a row for every second CU or more: can do without a workspace
  bool row16;          // one bf16 score per token: one workgroup per row, which its registers hold (the workspace is not touched)
  int row16_kind;
  bool rowpass;        // many long rows of ready-made scores: one workgroup per row, no workspace
  int rowpass_threads;
  int nchunks, page, srcN, pool_pitch, pool_chunk, pool_nchunks;
  int smp_tokens, smp_parts;
  size_t agg_bytes, blk_bytes, hist_bytes, state_bytes, chunk_bytes;
  size_t pool_key_bytes;
  size_t pub_bytes;
  bool sums;           // long rows of few: their sums first, which one workgroup per row then ranks (with a workspace for them)
  size_t sums_bytes;
  size_t pipeline_total() const { return agg_bytes + blk_bytes + hist_bytes + state_bytes + chunk_bytes; }
  size_t pool_total() const { return pool ? 2 * pool_key_bytes : 0; }
  size_t fused_total() const { return sums_bytes > pub_bytes ? sums_bytes : pub_bytes; }
  // a pool-shaped call falls back to the pipeline when its pointers are not 16-byte aligned,
  // so the workspace covers both
  size_t total() const {
    if (rowpass) return 0;
    if (fused || band) return fused_total();
    return pipeline_total() > pool_total() ? pipeline_total() : pool_total();
  }
};

int largest_budget(const sts_select_params *p) {
  if (!p->k_head) return p->k;
  int k = 1;
  for (int j = 0; j < p->Hd; ++j) k = p->k_head[j] > k ? p->k_head[j] : k;
  return k;
}

// does the list of a workgroup with `tokens` tokens, one of q parts of the row, have room for its share of the band?
bool smp_list_fits(const sts_select_params *p, int k, int64_t tokens, int64_t q) {
  const int64_t band = smp_expected_band(p->N, k < p->N ? k : p->N, (int)tokens);
  for (int f = 0; f < SMP_FORMS; ++f)
    if (tokens <= SMP_TOKENS[f]) return band >= 0 && band <= q * SMP_LIST[f];
  return false;
}

// How the sampled selection cuts its rows: as many workgroups as there are CUs, in equal shares of at
// least 8192 tokens (below that the fixed part of a workgroup's work exceeds its share of the pass)
// and at most 32 per row (the exchange grows with the square).
// Parts of more than 128K tokens only where the list, the shorter the more tokens there are, has room for the band (else
// it is read again), and for one or two parts per row or a grid that fits the chip. One part per row against parts of
// at most 128K: 256 rows of 524288 tokens, one score each, 0.5% kept 130 us, 213; 256 rows of 200000, four scores, 10% kept
// 144, 182; 512 rows of 200000, one bf16 score, 10% 160, 249; two parts: 128 rows of 524288, one score, 4% 88, 118; but
// three for 10%: 144, 127.
// Calls with a row for every second CU or more take one part for short rows: no words to clear and to exchange. 128 rows of
// 12000 tokens, one score: 20.9 us, 26.3 in two parts; 26000, five scores: 31.5, 32.8; 26000, eight bf16 scores: 36.0, 33.1.
void plan_sampled(const sts_select_params *p, size_t rows, SelectPlan &pl) {
  const int k = largest_budget(p);
  const int64_t cus = cu_count(), r = rows ? (int64_t)rows : 1;
  int64_t q = cus / r;
  if (q > ((int64_t)p->N + 8191) / 8192) q = ((int64_t)p->N + 8191) / 8192;
  if (q > 32) q = 32;
  if (q < 1 || (2 * r >= cus && p->N <= 32768 && (int64_t)p->N * p->Tq <= 131072)) q = 1;
  auto tokens = [&] { return (((int64_t)p->N + q - 1) / q + 255) / 256 * 256; };
  auto fits = [&] { return tokens() <= SMP_MAX_TOKENS && (q <= 2 || r * q <= cus) && smp_list_fits(p, k, tokens(), q); };
  while (tokens() > 131072 && !fits()) ++q;
  pl.smp_tokens = (int)tokens();
  pl.smp_parts = (int)(((int64_t)p->N + pl.smp_tokens - 1) / pl.smp_tokens);
  pl.pub_bytes = pl.smp_parts > 1 ? align256(rows * (size_t)pl.smp_parts * SMP_WORDS * sizeof(unsigned long long)) : 0;
}

sts_status plan_select(const sts_select_params *p, SelectPlan &pl) {
  if (!p) return STS_EINVAL;
  if (p->B < 0 || p->Hd < 1 || p->Tq < 1 || p->N < 0 || p->Hq < 1 || p->k < 1) return STS_EINVAL;
  if (p->kind != STS_SCORES_PROBS && p->kind != STS_SCORES_LOGITS_LSE) return STS_EINVAL;
  if (p->reduce != STS_REDUCE_SUM && p->reduce != STS_REDUCE_MAX) return STS_EINVAL;
  if (p->Tq > 64 || p->Hq > STS_MAX_HEADS || p->Hd > STS_MAX_HEADS) return STS_EUNSUPPORTED;
  if ((int64_t)p->N > 0x7fffffffll - 65536) return STS_EUNSUPPORTED;
  if ((int64_t)p->B * p->Hd > 65535) return STS_EUNSUPPORTED;   // grid.y
  if (p->page_size < 0 || p->page_size > 4096) return STS_EUNSUPPORTED;
  pl.page = p->page_size <= 1 ? 1 : p->page_size;
  pl.srcN = (p->N + pl.page - 1) / pl.page;
  pl.nchunks = (pl.srcN + SEL_CHUNK - 1) / SEL_CHUNK;
  const size_t rows = (size_t)p->B * p->Hd;
  // One workgroup ranks a whole row in its registers (up to 32768 tokens in calls that fill the chip with such rows; see
  // also `one_row` below).
  pl.small = pl.page == 1 && (p->N <= SEL_FUSED_N || (p->N <= SEL_SMALL_N && rows >= 256));
  pl.pool = false;
  pl.pool_pitch = 0;
  pl.pool_key_bytes = 0;
  pl.fused = false;
  pl.rowpass = false;
  pl.row16 = false;
  pl.row16_kind = 0;
  pl.band = false;
  pl.rowpass_threads = 0;
  pl.smp_tokens = pl.smp_parts = 0;
  pl.pub_bytes = 0;
  pl.sums = false;
  pl.sums_bytes = 0;
  // test / tuning knob: 0 the library's rule, 1 histogram pipeline only, 2 pipeline or pool,
  // 3 the sampled selection wherever its shape limits allow, 4 one workgroup per row in
  // several passes wherever its shape limits allow, 5 the sampled selection with one workgroup per row likewise,
  // 6 rows of one bf16 score per token in registers wherever they fit
  const double path_knob = knob(STS_KNOB_SELECT_PATH);
  const int path = path_knob == path_knob ? (int)path_knob : 0;
  // Rows of up to 32768 tokens in calls of fewer rows: one workgroup per row, too, unless few workgroups would have much to
  // read each (one CU reads some 60 GB/s; the sampled selection's parts are more CUs, but exchange what they counted and need
  // a launch that clears). us on other scores in every call, against the sampled selection, fp32 unless said otherwise: 16
  // rows of 12000 with five scores per token 17.8, 25.1; of 16384 with ten 25.6, 31.2; 64 of 16384 with sixteen 34.6, 42.3.
  // Beyond 16384 tokens a thread has eight quads, and every further score per token costs a pass over them whatever N is:
  // 16 rows of 32768 with five 27.8, 28.6, but with six 30.1, 29.1 and of 20000 with eight 29.6, 27.3; 64 rows of 32768 with
  // five 29.2, 32.9, but of 20000 with eight 30.8, 29.4; 128 of 17000 with eight 31.4, 35.6, of 32768 39.5, 49.3, but 96 of
  // 20000 with twelve 41.3, 38.0; bf16, 16 rows of 32768 with ten 33.3, 33.4, of 26000 with twelve 35.5, 33.1. (Measured before calls of
  // up to 127 such rows summed three to five scores and more in a launch of their own, which is faster than either, see `sums`
  // below: there the line decides for fewer scores, for calls that ask for the sums and for those with a smaller workspace.) Calls of fewer
  // than eight rows, fewer than any model's draft heads, keep the route that they had (and calls of few rows the workspace
  // that they had to bring).
  //
  // What one workgroup writes counts, too: an entry of a list costs it as much as 13 stores to make, and a store per list that
  // takes it, where the parts of the sampled selection share this (list_work: the stores that they would take off it). us, in
  // one workgroup per row and sampled, half of the tokens kept: 8 rows of 16384, 32 lists for each 52.6, 43.4, 8 lists 26 or less,
  // 32; of 32768 one score per token, two lists 22.6, 27.8, 8 lists 31.5, 31.1; five scores, one list 30.7, 29.8, but 10% kept,
  // 32 lists faster; of 9000, 32 lists 41.5, 39.0.
  const int64_t parts = std::max<int64_t>(std::min<int64_t>({cu_count() / std::max<int64_t>((int64_t)rows, 1), ((int64_t)p->N + 8191) / 8192, 32}), 1);
  const int64_t list_work = (int64_t)std::min(largest_budget(p), p->N) * (13 + (p->Hq + p->Hd - 1) / p->Hd) * (parts - 1) / parts;
  const int64_t token_bytes = (int64_t)p->Tq * (p->scores_bf16 ? 2 : 4);
  const bool writes_little = list_work <= (p->N <= 16384 ? 96000 : 240000 - 6000 * std::min<int64_t>(token_bytes, 32));
  const bool reads_little = p->N <= 16384 ? p->N * token_bytes <= (4 * (int64_t)rows >= cu_count() ? 1024 : 640) << 10
                                          : token_bytes <= (2 * (int64_t)rows >= cu_count() ? 32 : 20);
  const bool one_row = path == 0 && pl.page == 1 && !pl.small && p->N > SEL_FUSED_N && p->N <= SEL_SMALL_N && rows >= 8 && reads_little && writes_little;
  pl.one_row = false;
  // Enough rows to give at least every second CU one, and rows that do not fit one workgroup's
  // LDS: the sampled selection, which here can do without a workspace, in one workgroup per row (with one it
  // may take more, see plan_sampled). Budgets next to the row's length, and rows of more than 512K tokens, go by the
  // rules further down and need theirs.
  // Measured, 128K-token rows, 10%: 128 rows of one fp32 score per token 45 us (two workgroups per
  // row; one workgroup per row took 57), 128 rows of eight bf16 scaled logits of 50000 tokens 52
  // (70 with one workgroup per row).
  // One bf16 score per token and many rows per CU (a mask per query row of prefill): rows of up to 131072 tokens fit
  // registers (below), and those that do so badly or not at all are the shape that plain passes by small workgroups serve
  // better (select_rowpass_kernel; 4096 rows of 128K: 754 against 962 us with the sampled selection).
  {
    const bool aligned = reinterpret_cast<uintptr_t>(p->scores) % 16 == 0;
    const bool band_ok = pl.page == 1 && p->N >= 4 && p->N <= SMP_MAX_TOKENS;
    const int kmax = largest_budget(p);
    const bool has_edge = band_ok && smp_expected_band(p->N, kmax < p->N ? kmax : p->N, p->N) >= 0;
    const bool rowpass_ok = pl.page == 1 && p->Tq == 1 && p->kind == STS_SCORES_PROBS && !p->agg_out && p->N > 0 &&
                            (p->N % (p->scores_bf16 ? 8 : 4)) == 0 && aligned;
    const int64_t cus = cu_count();
    if (one_row && has_edge && 2 * (int64_t)rows >= cus) pl.small = true;      // (such calls did without a workspace before, too)
    const bool long_rows = !pl.small && p->N > SEL_FUSED_N;
    const bool take_rowpass = path == 4 ? rowpass_ok
                                        : path == 0 && rowpass_ok && long_rows && p->scores_bf16 && (int64_t)rows >= 4 * cus;
    const bool take_band = path == 5 ? band_ok && p->N % 4 == 0 && aligned : path == 0 && !take_rowpass && has_edge && long_rows && 2 * (int64_t)rows >= cus;
    // One bf16 score per token: rows of 4096 to 131072 of them are held packed in one workgroup's registers
    // (select_row16_kernel). us, with the paths that such calls would take otherwise: 16 rows of
    // 131072 43.5 -> 24.8, 64 of 65536 42.1 -> 15.5, 512 of 65536 85.3 -> 25.4, 4096 of 65536 239 -> 155, 4096 of 32768
    // 268 -> 75, 512 of 4096 11.7 -> 8.8. Shorter rows keep short_select_row_kernel (512 rows of 2048 there
    // 11.6, packed 10.3; 4096 rows 31.9, 38.6). Rows of more than 65536 tokens take a CU's whole register file, whatever they fill of it: where there
    // are many, the plain passes of select_rowpass_kernel, several rows per CU, are faster up to 112K tokens. 1024 rows, 10%:
    // of 65544 tokens 75, 88; of 98304 104, 112; of 114688 123, 120; of 131072 140, 129; 4096 rows of 65544 245, 329; of 106496
    // 380, 424; of 131072 501, 464. (Rows that are not a multiple of 8 long cannot take those: 1024 of 66001 157, in registers 92.)
    // Few rows whose lists are long or many stay with the sampled selection, see list_work: 1 row of 131072, half kept, one list
    // 65, sampled 42, 32 lists 159, 56; 10% kept, 32 lists 49, 45; of 65536, half kept, two lists 38.4, 38.2, 8 lists 50, 41.
    const bool row16_ok = pl.page == 1 && p->Tq == 1 && p->kind == STS_SCORES_PROBS && p->scores_bf16 && !p->agg_out &&
                          p->N >= 8 && p->N <= SEL_ROW16_N;
    const bool take_row16 = path == 6 ? row16_ok : path == 0 && row16_ok && p->N >= 4096 && (p->N <= SEL_FUSED_N || list_work <= 440000) &&
                                                   !(take_rowpass && p->N > 65536 && p->N < 114688);
    if (take_row16) {
      // The rest of the plan stays: such a call has to bring the workspace that its rows asked for before (nothing in it
      // is touched), and the timing aid counts it as the class of call that they put it in.
      pl.row16 = true;
      pl.row16_kind = pl.small ? STS_K_SELECT_SMALL : take_rowpass ? STS_K_SELECT_ROWPASS : take_band ? STS_K_SELECT_BAND : STS_K_SELECT_FUSED;
    }
    if (take_rowpass || take_band) {
      pl.small = false;
      pl.band = take_band;
      pl.rowpass = take_rowpass;
      pl.rowpass_threads = (int64_t)rows >= 4 * cus ? 256 : 1024;
      if (const double t = knob(STS_KNOB_SELECT_ROW_THREADS); t == 256.0 || t == 1024.0) pl.rowpass_threads = (int)t;
      pl.nchunks = 0;
      pl.pool_chunk = pl.pool_nchunks = 0;
      pl.agg_bytes = pl.blk_bytes = pl.hist_bytes = pl.state_bytes = pl.chunk_bytes = 0;
      if (take_band) {
        plan_sampled(p, rows, pl);
        if (path == 5) {                               // (the knob's meaning: one workgroup per row)
          pl.smp_tokens = (p->N + 255) / 256 * 256;
          pl.smp_parts = 1;
          pl.pub_bytes = 0;
        }
      }
      return STS_OK;
    }
  }
  if (pl.small) {
    pl.nchunks = 0;
    pl.agg_bytes = pl.blk_bytes = pl.hist_bytes = pl.state_bytes = pl.chunk_bytes = 0;
    return STS_OK;
  }
  // Small budgets on long rows: each chunk of the row keeps its own best k tokens and one
  // workgroup per row ranks that pool out of LDS (two launches, the scores are read once and
  // the aggregate is never stored). The ranking workgroup works at one CU's pace, about 1.2 us
  // per 1000 pooled pairs on top of 10 us, so the pool must be small: up to 8192 pairs it beats
  // the five-launch pipeline for every shape measured, up to 16384 only when the pipeline's
  // passes over the aggregate are long (8M scores or more in the call). Chunks are 8192 tokens,
  // or 32768 when only that keeps the pool small enough (long rows, middle budgets).
  pl.pool_chunk = pl.pool_nchunks = 0;
  if (pl.page == 1 && (p->N % 4) == 0 && path != 1) {
    for (const int chunk : {SEL_CHUNK, 4 * SEL_CHUNK}) {
      const int64_t nch = ((int64_t)p->N + chunk - 1) / chunk;
      const int64_t pitch = p->k < chunk ? p->k : chunk;
      const int64_t pooled = nch * pitch;
      // a grid of few large workgroups leaves most of the chip idle: then the pipeline is as fast
      if (chunk > SEL_CHUNK && (int64_t)rows * nch < 128) break;
      if (pooled <= SEL_POOL_MAX / 2 || (pooled <= SEL_POOL_MAX && (int64_t)rows * p->N >= (int64_t)1 << 23)) {
        pl.pool = true;
        pl.pool_chunk = chunk;
        pl.pool_nchunks = (int)nch;
        pl.pool_pitch = (int)pitch;
        pl.pool_key_bytes = align256(rows * (size_t)nch * (size_t)pitch * sizeof(uint32_t));
        break;
      }
    }
  }
  // Long rows at token granularity: the sampled selection (select_sampled.hip), one pass over the
  // scores, any budget. Rows of more than 256K tokens (eight units of 32768) take it in calls of 4M
  // tokens or more: 16 rows of 1M tokens, 2%: 84 us against 126 for the pipeline; budgets small enough
  // for the pool keep it (256 tokens: 89 against 92). Smaller calls of such rows keep the paths above
  // and below, which are bound by launches and latencies there.
  if (pl.page == 1 && p->N > SEL_FUSED_N && path != 1 && path != 2) {
    const bool large = (int64_t)rows * p->N >= (int64_t)1 << 22 && !pl.pool;
    if (((int64_t)p->N + 32767) / 32768 <= (path == 3 || large ? 256 : SEL_FUSED_MAX_PARTS)) {
      pl.fused = true;
      pl.one_row = one_row;
      pl.pool = false;
      plan_sampled(p, rows, pl);
      // Calls of 8 to 127 rows (less than one for every second CU: more come here, too, with budgets next to the row's length) of up
      // to 65536 tokens whose lists one workgroup per row writes as fast: the row is ranked in one
      // workgroup's registers where it is one fp32 score per token (beyond 32768 tokens; below, `one_row` says the same), and
      // several scores are summed first by as many workgroups as there are quads for. A launch more, but nothing to clear, to
      // sample, to exchange, and the scores are read by the whole chip. us on other scores in every call, as it was (sampled, or
      // added up by the workgroup that ranks them) and now: 16 rows of 33001 with one score 26.3, 16.9, with five 28.5, 20.8; of 65536 26.2,
      // 21.1 and 29.9, 25.8; of 32768 with five 24.7, 18.5, with eight 30.7, 18.6; 32 of 65536 with two 28.0, 27.3, with five 33.5, 30.5; 64 of
      // 33001 with five 33.3, 27.6, of 49152 with four 31.6, 29.6, with eight 40.4, 37.3; of 32768 with eight 37.2, 27.5, with five bf16 scores
      // 21.8, 21.6. Not where the sums take longer than they save: 64 of 57000 with five 37.2, 37.2, of 65536 37.3, 39.8; of 24000 with two
      // 17.5, 20.3; nor where two scores are added up in passing (16 of 24000 17.0, 17.1).
      const bool ready = p->Tq == 1 && p->kind == STS_SCORES_PROBS && !p->scores_bf16;
      const bool lists_fit = list_work <= 216000;        // (`writes_little` for one score per token)
      if (path == 0 && !pl.row16 && !p->agg_out && p->N > 16384 && p->N <= SEL_ROW_N && rows >= 8 && 2 * (int64_t)rows < cu_count() &&
          lists_fit) {
        if (ready) pl.one_row = true;
        else if (p->N > SEL_SMALL_N ? (int64_t)rows * p->N <= (p->N <= 49152 && p->Tq >= 4 ? 3200000 : 2250000) : p->Tq >= (rows <= 32 ? 3 : 5)) {
          pl.sums = true;
          pl.sums_bytes = align256(rows * (size_t)p->N * sizeof(float));
        }
      }
    }
  }
  pl.agg_bytes = p->agg_out ? 0 : align256(rows * (size_t)p->N * sizeof(float));
  pl.blk_bytes = pl.page > 1 ? align256(rows * (size_t)pl.srcN * sizeof(float)) : 0;
  pl.hist_bytes = align256(rows * 3 * SEL_BINS * sizeof(uint32_t));
  pl.state_bytes = align256(rows * 8 * sizeof(uint32_t));
  pl.chunk_bytes = align256(rows * (size_t)pl.nchunks * SEL_FLAG_PITCH * sizeof(uint32_t));
  return STS_OK;
}

}  // namespace

extern "C" {

size_t sts_attn_workspace_bytes(const sts_attn_params *p, int sparse) {
  AttnPlan pl;
  if (plan_attn(p, sparse, pl) != STS_OK) return 0;
  const size_t n = pl.part_o_bytes + pl.part_ml_bytes + pl.lse_bytes;
  return n ? n : 256;
}

sts_status sts_attn_plan(const sts_attn_params *p, int sparse, int32_t *num_splits,
                         int32_t *units_per_batch, int32_t *query_tiles) {
  AttnPlan pl;
  const sts_status v = plan_attn(p, sparse, pl);
  if (v != STS_OK) return v;
  if (num_splits) *num_splits = pl.num_splits;
  if (units_per_batch) *units_per_batch = pl.num_units;
  if (query_tiles) *query_tiles = pl.nq;
  return STS_OK;
}

sts_status sts_sparse_attn(const sts_attn_params *p, void *stream) {
  if (!p) return STS_EINVAL;
  return run_attn(p, 1, static_cast<hipStream_t>(stream), p->workspace, p->workspace_bytes, true);
}

sts_status sts_dense_attn(const sts_attn_params *p, void *stream) {
  if (!p) return STS_EINVAL;
  return run_attn(p, 0, static_cast<hipStream_t>(stream), p->workspace, p->workspace_bytes, true);
}

sts_status sts_sparse_attn_static(const sts_attn_params *p, void *stream) {
  if (!p) return STS_EINVAL;
  void *ws = nullptr;
  const sts_status v = sts_static_scratch(&ws);
  if (v != STS_OK) return v;
  // a shape whose partial results do not fit the array comes back as STS_EWORKSPACE
  return run_attn(p, 1, static_cast<hipStream_t>(stream), ws, STS_STATIC_SCRATCH_BYTES, false);
}

size_t sts_select_workspace_bytes(const sts_select_params *p) {
  SelectPlan pl;
  if (plan_select(p, pl) != STS_OK) return 0;
  const size_t n = pl.total();
  return n ? n : 256;
}

static sts_status enqueue_select(const sts_select_params *p, void *stream) {
  SelectPlan pl;
  const sts_status v = plan_select(p, pl);
  if (v != STS_OK) return v;
  if (!p->head_map || !p->indices) return STS_EINVAL;
  for (int t = 0; t < p->Hq; ++t)
    if (p->head_map[t] < 0 || p->head_map[t] >= p->Hd) return STS_EINVAL;
  if (p->k_head)
    for (int j = 0; j < p->Hd; ++j)
      if (p->k_head[j] < 1 || p->k_head[j] > p->k) return STS_EINVAL;
  if (p->B == 0) return STS_OK;
  if (p->N > 0 && !p->scores) return STS_EINVAL;
  if (p->kind == STS_SCORES_LOGITS_LSE && !p->lse) return STS_EINVAL;
  // (a workspace without room for the sums, as it was enough for such calls before they were summed first, still is)
  if (pl.sums && p->workspace_bytes < pl.sums_bytes) {
    pl.sums = false;
    pl.sums_bytes = 0;
  }
  size_t need = pl.total();
  const bool ws_usable = p->workspace && p->workspace_bytes >= need && reinterpret_cast<uintptr_t>(p->workspace) % 256 == 0;
  if (pl.band && need > 0 && !ws_usable) {
    // one workgroup per row needs no scratch memory: such calls are served without any, also where there is some that
    // is too small or not aligned
    pl.smp_parts = 1;
    pl.smp_tokens = (p->N + 255) / 256 * 256;
    need = 0;
  }
  if (need > 0 && !ws_usable) return STS_EWORKSPACE;
  hipStream_t s = static_cast<hipStream_t>(stream);

  SelectArgs a;
  memset(&a, 0, sizeof(a));
  a.scores = p->scores;
  a.scores_bf16 = p->scores_bf16 ? 1 : 0;
  a.lse = p->kind == STS_SCORES_LOGITS_LSE ? p->lse : nullptr;
  a.seq_lens = p->seq_lens;
  a.indices = p->indices;
  a.counts = p->counts;
  unsigned char *w = static_cast<unsigned char *>(p->workspace);
  a.agg = p->agg_out ? p->agg_out : reinterpret_cast<float *>(w);
  w += pl.agg_bytes;
  a.blk = pl.page > 1 ? reinterpret_cast<float *>(w) : nullptr;
  w += pl.blk_bytes;
  a.page = pl.page;
  a.srcN = pl.srcN;
  a.src = pl.page > 1 ? a.blk : a.agg;
  a.hist = reinterpret_cast<uint32_t *>(w);
  w += pl.hist_bytes;
  a.state = reinterpret_cast<uint32_t *>(w);
  w += pl.state_bytes;
  a.chunk_cnt = reinterpret_cast<uint32_t *>(w);
  a.B = p->B; a.Hd = p->Hd; a.Tq = p->Tq; a.N = p->N; a.Hq = p->Hq; a.k = p->k;
  a.kind = p->kind; a.reduce = p->reduce; a.nchunks = pl.nchunks;
  for (int j = 0; j < p->Hd; ++j) a.kh[j] = p->k_head ? p->k_head[j] : p->k;
  a.clear_words = (pl.hist_bytes + pl.state_bytes + pl.chunk_bytes) / sizeof(uint32_t);
  // The refinement histograms pay a digit search, a zeroed LDS histogram and a flush of up to
  // 2048 global atomics per workgroup: with more than about a thousand workgroups it is cheaper
  // to give each of them 2 or 4 consecutive chunks (1M-token rows: 22 -> 17.7 us per pass).
  {
    const size_t wgs = (size_t)p->B * p->Hd * (size_t)(pl.nchunks > 0 ? pl.nchunks : 1);
    a.hist_cpw = wgs >= 4096 ? 4 : (wgs >= 2048 ? 2 : 1);
  }
  // Test knob: STS_SELECT_SPIN_LIMIT bounds the polls of an earlier chunk's published counts
  // before the waiting workgroup recounts that chunk itself (0: one look, then recount).
  {
    const double v = knob(STS_KNOB_SELECT_SPIN_LIMIT);
    const bool set = v == v;   // not NaN
    a.spin_limit = !set ? 256 : (v < 0 ? 0 : (v > 65536 ? 65536 : (int)v));
    // the parts of the sampled selection wait for ALL parts of their row, and doing without them
    // means ranking the row by plain passes over its scores: a far longer patience by default
    a.fused_spin_limit = !set ? 20000 : a.spin_limit;
  }
  // inverse of the head map: the target heads fed by each draft head, in head order
  {
    int cnt[STS_MAX_HEADS + 1] = {0};
    for (int t = 0; t < p->Hq; ++t) ++cnt[p->head_map[t] + 1];
    for (int j = 0; j < p->Hd; ++j) cnt[j + 1] += cnt[j];
    for (int j = 0; j <= p->Hd; ++j) a.targets.off[j] = (uint16_t)cnt[j];
    int fill[STS_MAX_HEADS] = {0};
    for (int t = 0; t < p->Hq; ++t) {
      const int j = p->head_map[t];
      a.targets.tgt[cnt[j] + fill[j]++] = (uint8_t)t;
    }
  }

  hipError_t rc;
  if (pl.row16) {
    a.agg = nullptr;
    a.src = nullptr;
    a.hist = a.state = a.chunk_cnt = nullptr;
    a.rowpass_threads = SEL_ROW16;
    rc = run_kernel(pl.row16_kind, s, [&] { return launch_select_small(a, s); });
    return rc == hipSuccess ? STS_OK : STS_EHIP;
  }
  if (pl.band) {
    a.agg = p->agg_out;   // optional output only
    a.src = nullptr;
    a.hist = a.state = a.chunk_cnt = nullptr;
    a.pub = p->workspace;
    a.smp_tokens = pl.smp_tokens;
    a.smp_parts = pl.smp_parts;
    rc = run_kernel(STS_K_SELECT_BAND, s, [&] { return launch_select_band(a, s); });
    return rc == hipSuccess ? STS_OK : STS_EHIP;
  }
  if (pl.rowpass) {
    a.agg = nullptr;
    a.src = nullptr;
    a.hist = a.state = a.chunk_cnt = nullptr;
    a.rowpass_threads = pl.rowpass_threads;
    rc = run_kernel(STS_K_SELECT_ROWPASS, s, [&] { return launch_select_rowpass(a, s); });
    return rc == hipSuccess ? STS_OK : STS_EHIP;
  }
  if (pl.fused) {
    a.pub = p->workspace;
    a.smp_tokens = pl.smp_tokens;
    a.smp_parts = pl.smp_parts;
    a.agg = p->agg_out;   // optional output only: the keys never leave LDS
    a.src = nullptr;
    a.hist = a.state = a.chunk_cnt = nullptr;   // the pipeline's scratch does not exist on this path
    if (pl.sums) {
      SelectArgs r = a;
      a.agg = static_cast<float *>(p->workspace);
      rc = run_kernel(STS_K_SELECT_AGG, s, [&] { return launch_select_agg(a, s); });
      if (rc != hipSuccess) return STS_EHIP;
      r.scores = p->workspace;
      r.scores_bf16 = 0;
      r.lse = nullptr;
      r.kind = STS_SCORES_PROBS;
      r.reduce = STS_REDUCE_SUM;
      r.Tq = 1;
      rc = run_kernel(STS_K_SELECT_SMALL, s, [&] { return launch_select_small(r, s); });
      return rc == hipSuccess ? STS_OK : STS_EHIP;
    }
    if (pl.one_row) {
      rc = run_kernel(STS_K_SELECT_SMALL, s, [&] { return launch_select_small(a, s); });
      return rc == hipSuccess ? STS_OK : STS_EHIP;
    }
    if (pl.smp_parts > 1) {
      rc = run_kernel(STS_K_SELECT_CLEAR, s, [&] { return launch_select_clear_pub(a, s); });
      if (rc != hipSuccess) return STS_EHIP;
    }
    rc = run_kernel(STS_K_SELECT_FUSED, s, [&] { return launch_select_fused(a, s); });
    return rc == hipSuccess ? STS_OK : STS_EHIP;
  }
  if (pl.pool && reinterpret_cast<uintptr_t>(p->scores) % 16 == 0 &&
      (!p->agg_out || reinterpret_cast<uintptr_t>(p->agg_out) % 16 == 0)) {
    unsigned char *pw = static_cast<unsigned char *>(p->workspace);
    a.pool_key = reinterpret_cast<uint32_t *>(pw);
    a.pool_idx = reinterpret_cast<int32_t *>(pw + pl.pool_key_bytes);
    a.pool_pitch = pl.pool_pitch;
    a.pool_chunk = pl.pool_chunk;
    a.pool_nchunks = pl.pool_nchunks;
    a.agg = p->agg_out;   // optional output only
    rc = run_kernel(STS_K_SELECT_LOCAL, s, [&] { return launch_select_local(a, s); });
    if (rc != hipSuccess) return STS_EHIP;
    rc = run_kernel(STS_K_SELECT_POOL, s, [&] { return launch_select_pool(a, s); });
    return rc == hipSuccess ? STS_OK : STS_EHIP;
  }
  if (pl.small) {
    a.agg = p->agg_out;   // optional output only: the keys never leave LDS
    rc = run_kernel(STS_K_SELECT_SMALL, s, [&] { return launch_select_small(a, s); });
    return rc == hipSuccess ? STS_OK : STS_EHIP;
  }
  // Block granularity: aggregation and block sums in one pass when the shape allows (the
  // per-token aggregate is then stored only on request), and up to 16384 blocks per row are
  // ranked by one workgroup per row, out of LDS or in registers: two launches, nothing to clear (64 rows
  // of 8192 blocks 24 us with the block sums, of 16384 26.3, 27.5 and 33 out of LDS; the four kernels that the ranking replaces
  // take about 30 without them).
  SelectArgs f = a;
  f.agg = p->agg_out;
  const bool fused_blocks = pl.page > 1 && select_aggblock_ok(f);
  if (fused_blocks && pl.srcN <= SEL_SMALL_N / 2) {
    f.hist = nullptr;
    rc = run_kernel(STS_K_SELECT_AGG, s, [&] { return launch_select_aggblock(f, s); });
    if (rc != hipSuccess) return STS_EHIP;
    rc = run_kernel(STS_K_SELECT_SMALL, s, [&] { return launch_select_rank(f, s); });
    return rc == hipSuccess ? STS_OK : STS_EHIP;
  }
  // One fp32 probability row per head (an aggregate computed elsewhere, e.g. the draft layer's
  // summed attention weights): the aggregate is the input itself, so the first pass only builds
  // the first-digit histogram and the later passes read the caller's tensor.
  if (pl.page == 1 && p->Tq == 1 && p->kind == STS_SCORES_PROBS && !p->scores_bf16 && !p->agg_out) {
    a.agg = const_cast<float *>(static_cast<const float *>(p->scores));
    a.src = a.agg;
    a.agg_is_input = 1;
  }
  if (pl.nchunks > 0) {
    rc = run_kernel(STS_K_SELECT_CLEAR, s, [&] { return launch_select_clear(a, s); });
    if (rc != hipSuccess) return STS_EHIP;
    if (fused_blocks) {
      rc = run_kernel(STS_K_SELECT_AGG, s, [&] { return launch_select_aggblock(f, s); });
      if (rc != hipSuccess) return STS_EHIP;
    } else {
      rc = run_kernel(STS_K_SELECT_AGG, s, [&] { return launch_select_agg(a, s); });
      if (rc != hipSuccess) return STS_EHIP;
      if (pl.page > 1) {
        rc = run_kernel(STS_K_SELECT_BLOCK, s, [&] { return launch_select_block(a, s); });
        if (rc != hipSuccess) return STS_EHIP;
      }
    }
    rc = run_kernel(STS_K_SELECT_HIST, s, [&] { return launch_select_hist(a, 1, s); });
    if (rc != hipSuccess) return STS_EHIP;
    rc = run_kernel(STS_K_SELECT_HIST, s, [&] { return launch_select_hist(a, 2, s); });
    if (rc != hipSuccess) return STS_EHIP;
  }
  rc = run_kernel(STS_K_SELECT_WRITE, s, [&] { return launch_select_write(a, s); });
  return rc == hipSuccess ? STS_OK : STS_EHIP;
}

sts_status sts_select(const sts_select_params *p, void *stream) { return enqueue_select(p, stream); }

// ---------------------------------------------------------------------------- head mapping
namespace {
constexpr int HM_SLICE = 32768;   // rows per selection launch (grid.y limit)

struct HeadmapPlan {
  size_t idx_d_bytes, idx_t_bytes, overlap_bytes, select_bytes;
};

sts_status plan_headmap(const sts_headmap_params *p, HeadmapPlan &pl) {
  if (!p) return STS_EINVAL;
  if (p->S < 0 || p->R < 0 || p->Hd < 1 || p->Ht < 1 || p->N < 0 || p->k < 1) return STS_EINVAL;
  if ((int64_t)p->N > 0x7fffffffll - 65536) return STS_EUNSUPPORTED;
  const size_t rows_d = (size_t)p->S * p->Hd * p->R, rows_t = (size_t)p->S * p->Ht * p->R;
  if (rows_d > 0x7fffffffull || rows_t > 0x7fffffffull || (size_t)p->S * p->R > 0x7fffffffull) return STS_EUNSUPPORTED;
  if (p->Ht > 65535) return STS_EUNSUPPORTED;
  pl.idx_d_bytes = align256(rows_d * (size_t)p->k * sizeof(int32_t));
  pl.idx_t_bytes = align256(rows_t * (size_t)p->k * sizeof(int32_t));
  pl.overlap_bytes = align256((size_t)p->Ht * p->Hd * sizeof(unsigned long long));
  // One selection slice at a time: B = rows of the slice, one draft head, one query row. The
  // selection chooses its path (and with it its scratch size) from the row count, so the scratch
  // is sized for the largest need over every slice size that will be launched: the full slices
  // and the tail slice of either trace.
  pl.select_bytes = 0;
  for (const size_t rows : {rows_d, rows_t}) {
    const size_t sizes[2] = {rows >= (size_t)HM_SLICE ? (size_t)HM_SLICE : 0, rows % (size_t)HM_SLICE};
    for (const size_t n : sizes) {
      if (n == 0) continue;
      sts_select_params sp;
      memset(&sp, 0, sizeof(sp));
      sp.B = (int32_t)n;
      sp.Hd = 1; sp.Tq = 1; sp.N = p->N; sp.Hq = 1; sp.k = p->k;
      SelectPlan spl;
      const sts_status v = plan_select(&sp, spl);
      if (v != STS_OK) return v;
      if (spl.total() > pl.select_bytes) pl.select_bytes = spl.total();
    }
  }
  return STS_OK;
}

// top-k index lists of every row of one trace, slice by slice, through the selection pipeline
sts_status select_rows(const float *trace, size_t rows, int N, int k, int32_t *idx, void *ws, size_t ws_bytes,
                       void *stream) {
  static const int32_t identity[1] = {0};
  for (size_t r0 = 0; r0 < rows; r0 += HM_SLICE) {
    sts_select_params sp;
    memset(&sp, 0, sizeof(sp));
    sp.B = (int32_t)(rows - r0 < (size_t)HM_SLICE ? rows - r0 : (size_t)HM_SLICE);
    sp.Hd = 1; sp.Tq = 1; sp.N = N; sp.Hq = 1; sp.k = k;
    sp.scores = trace + r0 * (size_t)N;
    sp.head_map = identity;
    sp.indices = idx + r0 * (size_t)k;
    sp.kind = STS_SCORES_PROBS;
    sp.reduce = STS_REDUCE_SUM;
    sp.workspace = ws;
    sp.workspace_bytes = ws_bytes;
    const sts_status v = enqueue_select(&sp, stream);
    if (v != STS_OK) return v;
  }
  return STS_OK;
}
}  // namespace

size_t sts_headmap_workspace_bytes(const sts_headmap_params *p) {
  HeadmapPlan pl;
  if (plan_headmap(p, pl) != STS_OK) return 0;
  return pl.idx_d_bytes + pl.idx_t_bytes + pl.overlap_bytes + pl.select_bytes + 256;
}

sts_status sts_head_map(const sts_headmap_params *p, void *stream) {
  HeadmapPlan pl;
  const sts_status v = plan_headmap(p, pl);
  if (v != STS_OK) return v;
  if (!p->map) return STS_EINVAL;
  const bool have_rows = (size_t)p->S * p->R > 0 && p->N > 0;
  if (have_rows && (!p->a_d || !p->a_t)) return STS_EINVAL;
  const size_t need = pl.idx_d_bytes + pl.idx_t_bytes + pl.overlap_bytes + pl.select_bytes;
  if (!p->workspace || p->workspace_bytes < need) return STS_EWORKSPACE;
  if (reinterpret_cast<uintptr_t>(p->workspace) % 256 != 0) return STS_EWORKSPACE;
  hipStream_t s = static_cast<hipStream_t>(stream);
  unsigned char *w = static_cast<unsigned char *>(p->workspace);
  int32_t *idx_d = reinterpret_cast<int32_t *>(w);
  w += pl.idx_d_bytes;
  int32_t *idx_t = reinterpret_cast<int32_t *>(w);
  w += pl.idx_t_bytes;
  // the counts accumulate in the caller's buffer when one is given
  unsigned long long *ov = p->overlap ? p->overlap : reinterpret_cast<unsigned long long *>(w);
  w += pl.overlap_bytes;
  void *sel_ws = w;

  const int c = p->k < p->N ? p->k : p->N;
  if (have_rows) {
    sts_status rc = select_rows(p->a_d, (size_t)p->S * p->Hd * p->R, p->N, p->k, idx_d, sel_ws, pl.select_bytes, stream);
    if (rc != STS_OK) return rc;
    rc = select_rows(p->a_t, (size_t)p->S * p->Ht * p->R, p->N, p->k, idx_t, sel_ws, pl.select_bytes, stream);
    if (rc != STS_OK) return rc;
  }
  hipError_t e = run_kernel(STS_K_HEADMAP, s, [&] { return launch_headmap_clear(ov, p->Ht * p->Hd, s); });
  if (e != hipSuccess) return STS_EHIP;
  if (have_rows) {
    e = run_kernel(STS_K_HEADMAP, s, [&] {
      return launch_headmap_overlap(idx_d, idx_t, p->S, p->R, p->Hd, p->Ht, p->N, p->k, c, ov, s);
    });
    if (e != hipSuccess) return STS_EHIP;
  }
  e = run_kernel(STS_K_HEADMAP, s, [&] { return launch_headmap_argmax(ov, p->Hd, p->Ht, p->map, s); });
  return e == hipSuccess ? STS_OK : STS_EHIP;
}

sts_status sts_union_rows(const sts_union_params *p, void *stream) {
  if (!p) return STS_EINVAL;
  if (p->B < 0 || p->Hd < 1 || p->Hq < 1 || p->Tq < 1 || p->N < 0 || p->k < 0 || p->pitch < 0) return STS_EINVAL;
  if (p->Tq > 16 || p->Hq > STS_MAX_HEADS || p->Hd > STS_MAX_HEADS || p->B > 65535) return STS_EUNSUPPORTED;
  if ((int64_t)p->N > 0x7fffffffll - 65536) return STS_EUNSUPPORTED;
  if (!p->head_map || !p->indices || !p->row_mask) return STS_EINVAL;
  for (int t = 0; t < p->Hq; ++t)
    if (p->head_map[t] < 0 || p->head_map[t] >= p->Hd) return STS_EINVAL;
  if (p->B == 0) return STS_OK;
  if (p->k > 0 && !p->row_indices) return STS_EINVAL;
  UnionArgs a;
  memset(&a, 0, sizeof(a));
  a.row_idx = p->row_indices;
  a.row_cnt = p->row_counts;
  a.indices = p->indices;
  a.row_mask = p->row_mask;
  a.counts = p->counts;
  a.B = p->B; a.Hd = p->Hd; a.Hq = p->Hq; a.Tq = p->Tq; a.N = p->N; a.k = p->k; a.pitch = p->pitch;
  for (int t = 0; t < p->Hq; ++t) a.map[t] = (uint8_t)p->head_map[t];
  hipStream_t s = static_cast<hipStream_t>(stream);
  const hipError_t rc = run_kernel(STS_K_UNION_ROWS, s, [&] { return launch_union_rows(a, s); });
  return rc == hipSuccess ? STS_OK : STS_EHIP;
}

const char *sts_strerror(int status) {   // an int on purpose: any value a caller holds may be asked about
  switch (status) {
    case STS_OK: return "ok";
    case STS_EINVAL: return "invalid argument";
    case STS_EUNSUPPORTED: return "unsupported shape";
    case STS_EWORKSPACE: return "workspace missing, misaligned or too small";
    case STS_EHIP: return "HIP launch error";
  }
  return "unknown status";
}

int sts_version(void) { return 208; }

void sts_set_knob(int which, double value) {
  if (which < 0 || which >= STS_KNOB_COUNT_) return;
  std::lock_guard<std::mutex> lk(g_knob_mu);
  knobs_init_locked();
  g_knob[which] = value;
}

double sts_get_knob(int which) {
  if (which < 0 || which >= STS_KNOB_COUNT_) return NAN;
  return knob(which);
}

void sts_prof_enable(int on) {
  std::lock_guard<std::mutex> lk(g_prof_mu);
  g_prof_on = on != 0;
}

void sts_prof_reset(void) {
  std::lock_guard<std::mutex> lk(g_prof_mu);
  g_prof_used = 0;
}

sts_status sts_prof_read(int kernel_kind, int32_t *launches, double *total_ms) {
  if (kernel_kind < 0 || kernel_kind >= STS_K_COUNT_) return STS_EINVAL;
  std::lock_guard<std::mutex> lk(g_prof_mu);
  int n = 0;
  double ms = 0.0;
  for (size_t i = 0; i < g_prof_used; ++i) {
    const ProfEvent &e = g_prof_pool[i];
    if (e.kind != kernel_kind) continue;
    if (hipEventSynchronize(e.stop) != hipSuccess) return STS_EHIP;
    float t = 0.f;
    // a launcher that had nothing to enqueue (an empty grid) leaves its pair unstamped
    if (hipEventElapsedTime(&t, e.start, e.stop) != hipSuccess) {
      (void)hipGetLastError();
      continue;
    }
    ms += t;
    ++n;
  }
  if (launches) *launches = n;
  if (total_ms) *total_ms = ms;
  return STS_OK;
}

}  // extern "C"
