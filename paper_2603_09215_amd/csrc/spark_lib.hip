// Host side of the SPAR-K decoding library: context, sequence bookkeeping, kernel launches and
// the C ABI declared in include/spark.h.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <array>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <type_traits>
#include <map>
#include <new>
#include <string>
#include <vector>

#include "../../include/spark.h"
#include "attention.h"
#include "device_common.h"
#include "gemv.h"
#include "measure.h"
#include "mfma_gemm.h"
#include "one_row.h"
#include "row_rule.h"
#include "sampling.h"
#include "sched.h"
#include "small_steps.h"

using namespace spark;

namespace {

constexpr int PREFILL_CHUNK = 256;   // most prompt rows pushed through the layers together in the buffers that every context has
constexpr int PROMPT_ROWS = 1024;    // and in those of a context with tiled weights
constexpr int MAX_STEPS_PER_CALL = 256;
// Rows from which the MFMA projections run: five rows would be two passes of the vector kernel.  Three and four are one, in
// 32 bits, with the caller's weights and with norms that have no upper end.  On the copy they would be faster (a batch of
// three 11.6 against 10.7 ms for twelve steps of a quarter of the layers, of four 12.5 against 11.0), but a value that lies
// 2^-39 below its row's largest is lost there, and a row whose sum of squares passes 1e12 (gemv.h, SSQ_SCALE) is wrong.
constexpr int MFMA_MIN_ROWS = 5;
constexpr int TILED_WIDE_TASKS = 8192;   // gate/up from here on has tiles enough for 64 tasks a wave at any row count (32 tiles)
constexpr int MAX_SEQ_LEN = 16384;
// Models whose steps can run in one launch (small_steps.h): fp32, a layer and a head of at most so many bytes
// (for the calls it pays for: small_steps_pay).
constexpr size_t SMALL_LAYER_BYTES = (size_t)8 << 20;
constexpr int SMALL_FLAGS_AT = 32;   // words from the plan to the words of the hand-overs: a cache line of their own
static_assert(SMALL_FLAGS_AT >= PL_WORDS, "the plan comes first");

struct Layout {  // byte offsets into the scratch buffer
  size_t state, page_table, plan, lower, upper, ee, full, prefill_rows, prefill_tokens, seq_ids,
      forced, step_flags, out_tokens, out_depth, best, arrivals, row_ssq, max_x, max_attn, max_act, sample_hist, sample_arrive, sample_count, hidden, xnorm, part_elems, act_part_elems, mfma_part, sample_q, sample_cand, rand_words, qbuf, attn_out, part, act, lens_u,
      logits, rope, inv_freq, total,
      tiled, wdown, total_tiled,   // the MFMA-ordered copy of the projection weights and its scales lie behind everything else (absent on the static area)
      prompt_rows, prompt_tokens, prompt_hidden, prompt_q, prompt_attn, prompt_act, prompt_xnorm, prompt_ssq, prompt_max_x, prompt_max_attn, prompt_max_act,
      total_prompt;        // and behind them the buffers of the largest prompt passes
};

struct Derived {
  int V, rmax, max_rows, max_pages, n_pages_total, slice, n_splits, group, esz;
  size_t page_elems, kv_pool_bytes;
};

// Where the MFMA-ordered copies of the projection matrices lie (from the start of
// the tiled region; per layer for the four projections of a layer).
struct TiledMatrix { size_t elems = 0, blocks = 0; };   // offsets of its tiles (elements) and of its scales (blocks of 32)
struct TiledMap {
  std::vector<TiledMatrix> qkv, o, gateup, down;
  TiledMatrix lens_a, lens_head, lm_head;
  size_t total = 0, blocks = 0;
};

// Where a pass through the layers keeps its rows
struct PassBuffers {
  float *hidden, *q, *attn, *act, *xnorm;
  unsigned long long *ssq;           // two sets of SSQ_WAYS words per row
  uint8_t *max_x, *max_attn, *max_act;
  RowDesc *descs;                    // of a prompt pass
  int *tokens;
  int rows;                          // rows that fit
};

struct Seq {
  bool open = false, prefilled = false;
  int cycle_offset = 0, len = 0, g = 0, j_stream = 0, n_pending = 0, last_full = 0, next = 0;   // next: input of the next step
  int text_budget = 0;   // > 0: speech only after this many text tokens
  int phase = 0;         // the sequence's phase on speech positions (the configuration's, unless moved)
  std::vector<int> pages;
  int64_t text_steps = 0, speech_full = 0, speech_ee = 0, text_ee = 0;
  int64_t flush_rows[2 * SPARK_MAX_PERIOD] = {0};
};

}  // namespace

struct spark_ctx {
  spark_config cfg;
  spark_weights w;
  Derived dv;
  Layout lo;
  TiledMap tm;
  SchedParams sp;
  hipStream_t stream;
  char *scratch;
  void *kv_pool;
  int n_cu;
  PassBuffers base, prompt, pb;   // of every pass; of large prompt passes (rows 0: none); of the pass being enqueued
  std::vector<Seq> seqs;
  std::vector<int> free_pages;
  std::vector<int> last_ids;   // row of the logits -> sequence, as of the latest step
  int *h_in;   // pinned: seq_ids[max_batch] + forced[MAX_STEPS][max_batch]
  int *h_out;  // pinned: tokens[MAX_STEPS][max_batch] + depth[...] + plan[PL_WORDS]
  char err[512];
  // kernel selection; the defaults are the measured choices, spark_tune moves them (tests, sweeps)
  bool mfma_ok = true;         // the shape allows the MFMA projections (16-byte vectors of 8 weights)
  bool use_mfma = true;        // "mfma" = 0 keeps every row count on the vector kernels
  int tiled_row_blocks = 4;     // blocks of 32 rows in a tile of mfma_tiled_k, at most
  int direct_max_rows = OP_ROWS;   // rows up to which mfma_direct_k runs
  int direct_whole_k = -1;      // ... and the longest k that it never cuts (negative: see direct_cut)
  int mfma_xcd_max_split = 4;  // row tiles share an XCD when k has at most this many ranges
  int mfma_small_tiles = 32;   // launches of mfma_rows_k with fewer 8-wave tiles use 4-wave workgroups
  int mfma_min_rows = MFMA_MIN_ROWS;
  int attn_pieces = 0;         // 64-token pieces per attention workgroup (0: by the launch's size)
  int gemv_big_kb = 40;        // vector-kernel launches with more LDS per workgroup run eight waves per workgroup
  int attn_mfma_min_rows = 1;  // passes with at least this many rows run attention on the MFMA units (where the shape allows)
  int mfma_small_max_k = 32768;  // ... and an input width of at most this
  bool has_tiled = false;      // the context owns the MFMA-ordered copy of the projection weights
  bool use_tiled = true;       // "mfma_tiled" = 0 keeps the MFMA projections on the kernel that stages weights through LDS
  bool fuse_norm = true;       // the residual projections' finishing launches prepare the next norm's input (no separate launch)
  bool small_ok = false;       // the model's steps can run in one launch
  size_t small_layer_bytes = 0;   // of one layer's weights
  bool use_small = true;       // "small_steps" = 0 keeps them on a launch per operation
  unsigned small_epoch = 0;    // such launches so far
  bool row_ok = false;         // the layers of a pass of one row can run in one launch
  int use_row = 1;             // "one_row": 0 keeps them on a launch per operation, 2 takes the one launch also where it does not pay
  size_t layer_bytes = 0;      // of one layer's weights, bf16
  bool row_words_clean = false;   // no word of its hand-overs holds a number that is still to come
  unsigned row_tag = 0;        // the last number used
  int wait_polls = 0;          // "wait_polls": questions of a wait inside those launches before it runs out (0: as many as the kernels' headers say)
  bool may_wait = true;        // the call being enqueued may take such launches: it can run again should a wait run out
  bool row_taken = false;      // a pass of one row has since prefill_rows last asked
  bool static_scratch = false; // the scratch area is the library's static device array (spark_init_static)
  int device = 0;
  float temperature = 0.f, top_p = 0.f;   // nucleus sampling, off while temperature <= 0
  int prefill_base = 128;    // prompt rows per pass in the base buffers, see spark_init
  int prefill_chunk = 0;     // > 0: prompt rows per pass, as set by "prefill_rows"
  bool prompt_pass = false;  // the pass being enqueued: consecutive positions of one sequence
  int attn_prompt_min_rows = 0;   // rows from which such a pass shares K and V between its rows (0: by the pass's size)
  int attn_splits_now = 0;   // context slices the rows of the passes being enqueued can reach (0: unknown, launch all)
  std::map<std::array<int, 3>, MixedCover> mixed_covers;   // (blocks of rows, input, tasks) of large passes
  std::map<std::pair<const void *, size_t>, int> occ_cache;  // workgroups per CU of a (kernel, LDS bytes)
  // profiling of one kernel class
  int prof_class = -1;
  std::vector<hipEvent_t> prof_ev;
  size_t prof_used = 0;
};

namespace {

int fail(spark_ctx *c, int code, const char *fmt, ...) {
  if (c) {
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(c->err, sizeof(c->err), fmt, ap);
    va_end(ap);
  }
  return code;
}

#define HIP_TRY(ctx, call)                                                                  \
  do {                                                                                      \
    hipError_t e_ = (call);                                                                 \
    if (e_ != hipSuccess)                                                                   \
      return fail(ctx, SPARK_EHIP, "%s failed: %s (%s:%d)", #call, hipGetErrorString(e_),  \
                  __FILE__, __LINE__);                                                      \
  } while (0)

size_t align_up(size_t v, size_t a) { return (v + a - 1) / a * a; }

// hidden-state slots per sequence: between two full-depth steps at most K-1 speech positions exit
// early inside a chunk; a chunk's tail and the next chunk's head can join when nothing between them
// runs full depth: 2K-1 rows with the current one.  A text period adds the same.
int pending_slots(const spark_config *c) {
  return 2 * c->period_k + (c->text_period_k > 1 ? 2 * c->text_period_k : 0);
}

SchedParams sched_params(const spark_config *c) {
  return SchedParams{c->n_layers, c->exit_layer, c->period_k, c->phase, c->scope, c->n_text,
                     c->n_speech, pending_slots(c), c->text_period_k, c->text_phase};
}

bool config_ok(const spark_config *c, char *why, size_t n) {
#define BAD(cond, msg) if (cond) { snprintf(why, n, "%s", msg); return false; }
  BAD(c->size != sizeof(spark_config), "spark_config.size does not match this library");
  BAD(c->n_layers < 1, "n_layers < 1");
  BAD(c->d_model < 8 || c->d_model % 8, "d_model must be a positive multiple of 8");
  BAD(c->d_model > 4096, "d_model > 4096 is not supported");
  BAD(c->n_kv_heads < 1 || c->n_q_heads < 1 || c->n_q_heads % c->n_kv_heads,
      "n_q_heads must be a positive multiple of n_kv_heads");
  {
    int grp = c->n_q_heads / c->n_kv_heads;
    BAD(grp != 1 && grp != 2 && grp != 4 && grp != 7 && grp != 8 && grp != 16,
        "query heads per KV head must be one of 1, 2, 4, 7, 8, 16");
  }
  BAD(c->head_dim != 64 && c->head_dim != 128, "head_dim must be 64 or 128");
  BAD(c->d_ffn < 8 || c->d_ffn % 8, "d_ffn must be a positive multiple of 8");
  BAD(c->vocab_text < 0 || c->vocab_speech < 0 || c->vocab_text + c->vocab_speech < 1,
      "empty vocabulary");
  BAD(c->dtype != SPARK_DTYPE_FP32 && c->dtype != SPARK_DTYPE_BF16, "unknown dtype");
  BAD(c->exit_layer < 1 || c->exit_layer > c->n_layers, "exit_layer outside [1, n_layers]");
  BAD(c->period_k < 1 || c->period_k > SPARK_MAX_PERIOD, "period_k outside [1, 16]");
  BAD(c->phase < 0 || c->phase >= c->period_k, "phase outside [0, period_k)");
  BAD(c->scope != SPARK_SCOPE_CHUNK && c->scope != SPARK_SCOPE_STREAM, "unknown scope");
  BAD(c->n_text < 0 || c->n_speech < 0 || c->n_text + c->n_speech < 1, "empty interleave cycle");
  BAD(c->text_period_k < 0 || c->text_period_k > SPARK_MAX_PERIOD, "text_period_k outside [0, 16]");
  BAD(c->text_period_k > 1 && (c->text_phase < 0 || c->text_phase >= c->text_period_k),
      "text_phase outside [0, text_period_k)");
  BAD(pending_slots(c) > 2 * SPARK_MAX_PERIOD, "period_k + text_period_k > 16: too many pending rows");
  if (c->scope == SPARK_SCOPE_CHUNK && c->exit_layer < c->n_layers) {
    // the pattern repeats with the cycle: it needs a full-depth slot, and its longest run of early
    // exits (which may wrap around the cycle and cross modalities) must fit the pending slots
    const SchedParams sp = sched_params(c);
    const int cyc = c->n_text + c->n_speech;
    int run = 0, longest = 0;
    bool any_full = false;
    for (int g = 0; g < 2 * cyc; ++g) {
      int is_text, full;
      schedule_decide(sp, g, 0, 0, 0, sp.phase, is_text, full);
      if (full) { any_full = true; run = 0; } else { longest = std::max(longest, ++run); }
    }
    BAD(!any_full, "a cycle without a full-depth slot would never complete its KV");
    BAD(longest + 1 > pending_slots(c), "a run of early exits is longer than the pending slots");
  }
  BAD(c->max_batch < 1 || c->max_batch > SCHED_THREADS, "max_batch outside [1, 256]");
  BAD(c->max_seq_len < 1 || c->max_seq_len > MAX_SEQ_LEN, "max_seq_len outside [1, 16384]");
  BAD(c->kv_page_tokens < 16 || c->kv_page_tokens % 16, "kv_page_tokens must be a multiple of 16");
#undef BAD
  return true;
}

void derive(const spark_config &c, Derived &d) {
  d.V = c.vocab_text + c.vocab_speech;
  d.rmax = pending_slots(&c);
  d.max_rows = std::max(c.max_batch * d.rmax, PREFILL_CHUNK);
  d.max_pages = (c.max_seq_len + c.kv_page_tokens - 1) / c.kv_page_tokens;
  d.n_pages_total = d.max_pages * c.max_batch;
  d.slice = ATTN_SLICE;
  d.n_splits = (c.max_seq_len + d.slice - 1) / d.slice;
  d.group = c.n_q_heads / c.n_kv_heads;
  d.esz = c.dtype == SPARK_DTYPE_BF16 ? 2 : 4;
  d.page_elems = (size_t)c.n_layers * 2 * c.n_kv_heads * c.kv_page_tokens * c.head_dim;
  d.kv_pool_bytes = d.page_elems * d.esz * d.n_pages_total;
}

// the MFMA kernels load 16-byte vectors of 8 weights; other widths stay on the vector kernel
bool shape_allows_mfma(const spark_config &c) {
  return c.dtype == SPARK_DTYPE_BF16 && c.d_model % 8 == 0 && (c.n_q_heads * c.head_dim) % 8 == 0 && c.d_ffn % 8 == 0;
}

void tiled_map(const spark_config &c, const Derived &d, TiledMap &tm) {
  tm = TiledMap();
  if (!shape_allows_mfma(c)) return;
  const int dm = c.d_model, qw = c.n_q_heads * c.head_dim, F = c.d_ffn;
  size_t o = 0;
  auto take = [&](int n_tasks, int n_in) {
    const TiledMatrix w{o, tm.blocks};
    o += tg_tiled_elems(n_tasks, n_in);
    tm.blocks += tg_blocks(n_tasks);
    return w;
  };
  for (int l = 0; l < c.n_layers; ++l) {
    tm.qkv.push_back(take((c.n_q_heads + 2 * c.n_kv_heads) * (c.head_dim / 2), dm));
    tm.o.push_back(take(dm / 2, qw));
    tm.gateup.push_back(take(F, dm));
    tm.down.push_back(take(dm / 2, F));
  }
  tm.lens_a = take(dm / 2, dm);
  tm.lens_head = take((d.V + 1) / 2, dm);
  tm.lm_head = take((d.V + 1) / 2, dm);
  tm.total = o;
}

// bytes per row of the lists of largest magnitudes, at most: one per block of 16 tasks of a residual
// projection, per wave of the attention workgroups that merge a row, per block of 16 MLP activations
int max_x_bytes(const spark_config &c) { return (int)align_up((c.d_model / 2 + TG_TASKS - 1) / TG_TASKS, 16); }
int max_attn_bytes(const spark_config &c) { return (int)align_up(c.n_q_heads * 2 * (ATTN_THREADS / 64), 16); }
int max_act_bytes(const spark_config &c) { return (int)align_up((c.d_ffn + TG_TASKS - 1) / TG_TASKS, 16); }

void layout(const spark_config &c, const Derived &d, Layout &l) {
  size_t o = 0;
  auto take = [&](size_t bytes) { size_t at = o; o = align_up(o + bytes, 256); return at; };
  const size_t qw = (size_t)c.n_q_heads * c.head_dim;
  l.state = take(sizeof(int) * ST_WORDS * c.max_batch);
  l.page_table = take(sizeof(int) * (size_t)d.max_pages * c.max_batch);
  l.plan = take(sizeof(int) * (SMALL_FLAGS_AT + SMALL_WGS));
  l.lower = take(sizeof(RowDesc) * c.max_batch);
  l.upper = take(sizeof(RowDesc) * (size_t)c.max_batch * d.rmax);
  l.ee = take(sizeof(RowDesc) * c.max_batch);
  l.full = take(sizeof(RowDesc) * c.max_batch);
  l.prefill_rows = take(sizeof(RowDesc) * PREFILL_CHUNK);
  l.prefill_tokens = take(sizeof(int) * PREFILL_CHUNK);
  l.seq_ids = take(sizeof(int) * c.max_batch);
  l.forced = take(sizeof(int) * (size_t)MAX_STEPS_PER_CALL * c.max_batch);
  l.step_flags = take(sizeof(int) * c.max_batch);
  l.out_tokens = take(sizeof(int) * (size_t)MAX_STEPS_PER_CALL * c.max_batch);
  l.out_depth = take(sizeof(int) * (size_t)MAX_STEPS_PER_CALL * c.max_batch);
  l.best = take(sizeof(unsigned long long) * c.max_batch);
  l.arrivals = take(sizeof(int) * (size_t)d.max_rows * c.n_q_heads);   // per (row, group of query heads)
  // what the launches of a pass hand each other about a row: sums of squares, lists of largest magnitudes
  l.row_ssq = take(sizeof(unsigned long long) * 2 * SSQ_WAYS * (size_t)d.max_rows);
  l.max_x = take(shape_allows_mfma(c) ? (size_t)max_x_bytes(c) * d.max_rows : 0);
  l.max_attn = take(shape_allows_mfma(c) ? (size_t)max_attn_bytes(c) * d.max_rows : 0);
  l.max_act = take(shape_allows_mfma(c) ? (size_t)max_act_bytes(c) * d.max_rows : 0);
  l.sample_hist = take(sizeof(unsigned long long) * (size_t)SAMPLE_BINS * c.max_batch);   // zero between launches
  l.sample_arrive = take(sizeof(unsigned) * c.max_batch);
  l.sample_count = take(sizeof(unsigned) * c.max_batch);
  l.hidden = take(sizeof(float) * ((size_t)c.max_batch * d.rmax + PREFILL_CHUNK) * c.d_model);
  l.qbuf = take(sizeof(float) * d.max_rows * qw);
  l.attn_out = take(sizeof(float) * d.max_rows * qw);
  l.part = take(sizeof(float) * (size_t)d.max_rows * c.n_q_heads * d.n_splits * (c.head_dim + 4));
  l.lens_u = take(sizeof(float) * (size_t)c.max_batch * c.d_model);
  // rows that the MFMA projections read, as three bf16 parts: normalised rows and attention output in the
  // one buffer, MLP activations in the other.  A pass on the copy of the weights has normalised rows in
  // fp32 in the one, and it and the vector kernels MLP activations in the other.
  const bool bf16 = c.dtype == SPARK_DTYPE_BF16;
  l.part_elems = bf16 ? (size_t)d.max_rows * align_up(std::max((size_t)c.d_model, qw), 64) : 0;
  l.act_part_elems = bf16 ? (size_t)d.max_rows * align_up(c.d_ffn, 64) : 0;
  l.xnorm = take(sizeof(bf16_t) * 3 * l.part_elems);
  l.act = take(bf16 ? sizeof(bf16_t) * 3 * l.act_part_elems : sizeof(float) * (size_t)d.max_rows * c.d_ffn);
  l.mfma_part = take(c.dtype == SPARK_DTYPE_BF16 ? MFMA_PARTIAL_BYTES : 256);
  l.logits = take(sizeof(float) * (size_t)c.max_batch * d.V);
  l.sample_q = take(sizeof(unsigned) * (size_t)c.max_batch * d.V);   // integer masses of the sampler
  l.sample_cand = take(sizeof(unsigned long long) * (size_t)SAMPLE_CAP * c.max_batch);
  l.rand_words = take(sizeof(unsigned long long) * (size_t)MAX_STEPS_PER_CALL * c.max_batch);
  l.rope = take(sizeof(float2) * (size_t)c.max_seq_len * (c.head_dim / 2));
  l.inv_freq = take(sizeof(float) * (c.head_dim / 2));
  l.total = o;
  // behind everything else: the MFMA-ordered copy of the bf16 projection weights, for contexts
  // whose scratch area has room for it
  TiledMap tm;
  tiled_map(c, d, tm);
  l.tiled = o;
  l.wdown = o + align_up(sizeof(f16_t) * tm.total, 256);
  l.total_tiled = l.wdown + align_up(sizeof(float) * 32 * tm.blocks, 256);
  o = l.total_tiled;
  const size_t n = shape_allows_mfma(c) ? PROMPT_ROWS : 0;
  l.prompt_rows = take(sizeof(RowDesc) * n);
  l.prompt_tokens = take(sizeof(int) * n);
  l.prompt_hidden = take(sizeof(float) * n * c.d_model);
  l.prompt_q = take(sizeof(float) * n * qw);
  l.prompt_attn = take(sizeof(float) * n * qw);
  l.prompt_act = take(sizeof(float) * n * c.d_ffn);
  l.prompt_xnorm = take(sizeof(float) * n * c.d_model);
  l.prompt_ssq = take(sizeof(unsigned long long) * 2 * SSQ_WAYS * n);
  l.prompt_max_x = take(max_x_bytes(c) * n);
  l.prompt_max_attn = take(max_attn_bytes(c) * n);
  l.prompt_max_act = take(max_act_bytes(c) * n);
  l.total_prompt = o;
}

template <typename T> T *at(spark_ctx *c, size_t off) { return (T *)(c->scratch + off); }

// ------------------------------------------------------------------ profiling brackets

// Every bracketed launch takes three events: before, after, and one more right behind it.  The
// last pair has nothing in between and measures what the event mechanism itself adds to a bracket;
// spark_profile_read subtracts its mean.
int prof_begin(spark_ctx *c, int kclass) {
  if (c->prof_class != kclass) return SPARK_OK;
  while (c->prof_used + 3 > c->prof_ev.size()) {
    hipEvent_t ev;
    HIP_TRY(c, hipEventCreate(&ev));
    c->prof_ev.push_back(ev);
  }
  HIP_TRY(c, hipEventRecord(c->prof_ev[c->prof_used], c->stream));
  return SPARK_OK;
}
int prof_end(spark_ctx *c, int kclass) {
  if (c->prof_class != kclass) return SPARK_OK;
  HIP_TRY(c, hipEventRecord(c->prof_ev[c->prof_used + 1], c->stream));
  HIP_TRY(c, hipEventRecord(c->prof_ev[c->prof_used + 2], c->stream));
  c->prof_used += 3;
  return SPARK_OK;
}

// ------------------------------------------------------------------ launches

template <typename WT, typename Pro, typename Epi>
int launch_gemv(spark_ctx *c, const Pro &pro, const Epi &epi, const RowDesc *rows, int m_rows,
                int n_in, int n_tasks, int kclass) {
  if (m_rows <= 0) return SPARK_OK;
  // activation rows per pass over the weights: as many as fit in the LDS budget next to the
  // partial-sum words; a norm prologue needs the whole row resident.  The budget is 64 KiB, or
  // 80 KiB for rows that do not fit in that (two such workgroups still fit in a CU's 160 KiB): a
  // single row of the MLP width (18944) then stays in one chunk, four rows of 4096 under a norm
  // prologue take one pass over the weights instead of two, and what has to be cut into chunks
  // anyway is cut into fewer
  const bool whole_row = std::is_same<Pro, ProNorm>::value;
  int mt = std::min(4, m_rows);
  const size_t budget = sizeof(float) * mt * align_up(n_in, 512) + 256 > 65536 ? 81920 : 65536;
  const size_t lds_budget = budget - sizeof(float) * (GEMV_BIG_THREADS / 64) * 4;
  while (mt > 1 && whole_row && sizeof(float) * mt * align_up(n_in, 512) > lds_budget) --mt;
  int kc_cap = (int)(lds_budget / (sizeof(float) * mt)) / 512 * 512;
  int kc = std::min((int)align_up(n_in, 512), kc_cap);
  if (whole_row && kc < n_in) return fail(c, SPARK_EINVAL, "row of %d does not fit in LDS", n_in);
  // much LDS per workgroup means few workgroups per CU: those launches run eight waves per
  // workgroup, so that a CU still has 16 waves streaming
  const bool big = sizeof(float) * (size_t)mt * kc > (size_t)c->gemv_big_kb * 1024;   // at most three workgroups per CU
  const int threads = big ? GEMV_BIG_THREADS : GEMV_THREADS, waves = threads / 64;
  size_t lds = sizeof(float) * ((size_t)mt * kc + waves * mt);
  // one resident set of blocks: the kernel loops over its tasks, so the grid is sized to what the
  // chip holds at once (no second wave of blocks with a cold pipeline)
  void (*kern)(Pro, Epi, const RowDesc *, int, int, int, int) = nullptr;
  switch (mt) {
    case 1: kern = big ? gemv_rows_k<WT, 1, Pro, Epi, GEMV_U, GEMV_D, GEMV_BIG_THREADS> : gemv_rows_k<WT, 1, Pro, Epi>; break;
    case 2: kern = big ? gemv_rows_k<WT, 2, Pro, Epi, GEMV_U, GEMV_D, GEMV_BIG_THREADS> : gemv_rows_k<WT, 2, Pro, Epi>; break;
    case 3: kern = big ? gemv_rows_k<WT, 3, Pro, Epi, GEMV_U, GEMV_D, GEMV_BIG_THREADS> : gemv_rows_k<WT, 3, Pro, Epi>; break;
    default: kern = big ? gemv_rows_k<WT, 4, Pro, Epi, GEMV_U, GEMV_D, GEMV_BIG_THREADS> : gemv_rows_k<WT, 4, Pro, Epi>; break;
  }
  // attribute and occupancy are asked for once per (kernel, LDS size), not on every launch
  const auto key = std::make_pair((const void *)kern, lds);
  auto found = c->occ_cache.find(key);
  if (found == c->occ_cache.end()) {
    if (lds > 65536)
      HIP_TRY(c, hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, 81920));
    int o = 0;
    HIP_TRY(c, hipOccupancyMaxActiveBlocksPerMultiprocessor(&o, kern, threads, lds));
    found = c->occ_cache.emplace(key, std::max(1, std::min(o, 4))).first;
  }
  const int occ = found->second;
  int bx = std::min((n_tasks + waves - 1) / waves, c->n_cu * occ);
  dim3 grid(bx, (m_rows + mt - 1) / mt), block(threads);
  int rc = prof_begin(c, kclass);
  if (rc) return rc;
  kern<<<grid, block, lds, c->stream>>>(pro, epi, rows, m_rows, n_in, n_tasks, kc);
  HIP_TRY(c, hipGetLastError());
  return prof_end(c, kclass);
}

KVView kv_view(spark_ctx *c) {
  KVView v;
  v.pool = c->kv_pool;
  v.page_table = at<int>(c, c->lo.page_table);
  v.max_pages = c->dv.max_pages;
  v.n_layers = c->cfg.n_layers;
  v.n_kv_heads = c->cfg.n_kv_heads;
  v.page_tokens = c->cfg.kv_page_tokens;
  v.head_dim = c->cfg.head_dim;
  return v;
}

constexpr int ATTN_SPLIT_HEADS_MAX_ROWS = 4;

// GT query heads per workgroup
template <typename WT, int HD, int GT>
void launch_attention_g(spark_ctx *c, const RowDesc *rows, int m, int layer, const float *q, const RowOut &out, RowMax &row_max) {
  const spark_config &g = c->cfg;
  const Derived &d = c->dv;
  float *part = at<float>(c, c->lo.part);
  const int n_groups = (d.group + GT - 1) / GT;
  const int splits = c->attn_splits_now > 0 ? std::min(d.n_splits, c->attn_splits_now) : d.n_splits;
  row_max.n = g.n_kv_heads * n_groups * (ATTN_THREADS / 64);
  auto kern = attn_rows_k<WT, HD, GT, false>;
  if constexpr (std::is_same<WT, bf16_t>::value)
    if (out.part_units) kern = attn_rows_k<WT, HD, GT, true>;
  kern<<<dim3(splits, g.n_kv_heads * n_groups, m), ATTN_THREADS, 0, c->stream>>>(
      rows, q, kv_view(c), layer, g.n_q_heads, d.group, d.n_splits,
      1.0f / sqrtf((float)HD), part, at<int>(c, c->lo.arrivals), out, row_max);
}

template <typename WT, int HD>
void launch_attention_hd(spark_ctx *c, const RowDesc *rows, int m, int m_pass, int layer, const float *q, const RowOut &out, RowMax &row_max) {
  // a handful of rows: two query heads per workgroup, so that even two KV heads make enough
  // workgroups; many rows: all heads of a KV head together, K and V are read once
  const int group = c->dv.group;
  const int gt = (m_pass <= ATTN_SPLIT_HEADS_MAX_ROWS && group > 2) ? 2 : group;
  switch (gt) {
    case 1: launch_attention_g<WT, HD, 1>(c, rows, m, layer, q, out, row_max); break;
    case 2: launch_attention_g<WT, HD, 2>(c, rows, m, layer, q, out, row_max); break;
    case 3: launch_attention_g<WT, HD, 4>(c, rows, m, layer, q, out, row_max); break;
    case 4: launch_attention_g<WT, HD, 4>(c, rows, m, layer, q, out, row_max); break;
    case 5: case 6: case 7: launch_attention_g<WT, HD, 7>(c, rows, m, layer, q, out, row_max); break;
    case 8: launch_attention_g<WT, HD, 8>(c, rows, m, layer, q, out, row_max); break;
    default: launch_attention_g<WT, HD, 16>(c, rows, m, layer, q, out, row_max); break;
  }
}

// How attn_rows_mfma_k cuts the contexts: 64-token pieces and teams of waves per workgroup.  load: pieces
// of the launch per CU.  A workgroup's pieces and the merge of a row's slices are two chains that follow
// each other, one as long as the pieces and one as long as the slices: the sum is least where the pieces go
// with the root of the context.  With many rows there should be about one workgroup of two teams per CU
// (pieces as 1.2 times the load), or, beyond three pieces per CU, workgroups of one team at three times
// that number: they keep more waves in flight, but where a KV head has more than eight query heads
// the merge is the longer part and eight waves at it win at any load.
// Measured over 1 .. 48 sequences of 256 .. 8192 tokens on both backbone shapes (114 points, a step against
// the best fixed choice at each): 0.6 % above it on average and 6 % at worst; one team and 1, 2, 4 or 8
// pieces by the load alone 5.4 % and 44 % (one sequence of 8192 tokens and two KV heads, 130 slices to merge).
struct AttnShape { int pieces, teams; };
AttnShape attn_shape(int splits, double load, int group, int pieces_set) {
  if (pieces_set > 0) return {pieces_set, pieces_set >= 8 ? 2 : 1};   // (the switch: two teams from eight pieces)
  const double by_context = 0.6 * std::sqrt((double)splits);
  if (load < 3.0 || group > 8) {
    const int pairs = (int)(std::max(by_context, 1.2 * load) / 2.0 + 0.5);
    return {2 * std::max(1, std::min(5, pairs)), 2};
  }
  return {std::max(1, std::min(6, (int)(std::max(by_context, 0.4 * load) + 0.5))), 1};
}

// row_max: where the rows' largest output magnitudes go, for the MFMA output projection (or no list);
// its count is set to what the launch writes.  m_pass: rows of the whole pass, which m may be a part of;
// the workgroups' shape, and with it the length of a row's list, is the same for all parts.
template <typename WT>
int launch_attention_rows(spark_ctx *c, const RowDesc *rows, int m, int m_pass, int layer, const float *q, const RowOut &out, RowMax &row_max) {
  if (std::is_same<WT, bf16_t>::value && c->cfg.head_dim == 128 && c->dv.group <= 16 && c->use_mfma &&
      m_pass >= c->attn_mfma_min_rows) {
    // the slice tasks on the MFMA units, all query heads of a KV head together
    const int splits = c->attn_splits_now > 0 ? std::min(c->dv.n_splits, c->attn_splits_now) : c->dv.n_splits;
    const long tasks = (long)splits * c->cfg.n_kv_heads * m_pass;
    const AttnShape shape = attn_shape(splits, (double)tasks / c->n_cu, c->dv.group, c->attn_pieces);
    const int pieces = shape.pieces;
    // few workgroups (a handful of rows, two KV heads): eight query heads per workgroup
    const int heads_per_wg = (tasks < c->n_cu / 2 && c->dv.group > 8) ? 8 : c->dv.group;
    const int wg_per_kv = (c->dv.group + heads_per_wg - 1) / heads_per_wg;
    row_max.n = c->cfg.n_kv_heads * wg_per_kv * shape.teams * (ATTN_THREADS / 64);
    const bool one_page = c->cfg.kv_page_tokens % ATTN_SLICE == 0;
    auto pick = [&](auto two_teams, auto parts) {
      return one_page ? attn_rows_mfma_k<128, two_teams ? 2 : 1, parts, true> : attn_rows_mfma_k<128, two_teams ? 2 : 1, parts, false>;
    };
    const std::true_type yes{};
    const std::false_type no{};
    const auto kern = out.part_units ? (shape.teams == 2 ? pick(yes, yes) : pick(no, yes)) : (shape.teams == 2 ? pick(yes, no) : pick(no, no));
    kern<<<dim3((splits + pieces - 1) / pieces, c->cfg.n_kv_heads * wg_per_kv, m), ATTN_THREADS * shape.teams, 0, c->stream>>>(
        rows, q, kv_view(c), layer, c->cfg.n_q_heads, c->dv.group, heads_per_wg, c->dv.n_splits, pieces, 1.0f / sqrtf(128.0f),
        at<float>(c, c->lo.part), at<int>(c, c->lo.arrivals), out, row_max);
  } else if (c->cfg.head_dim == 128) launch_attention_hd<WT, 128>(c, rows, m, m_pass, layer, q, out, row_max);
  else launch_attention_hd<WT, 64>(c, rows, m, m_pass, layer, q, out, row_max);
  HIP_TRY(c, hipGetLastError());
  return SPARK_OK;
}

RowOut from_row(const RowOut &o, int r0) {
  return RowOut{o.part_units ? (float *)((bf16_t *)o.p + (size_t)r0 * o.pitch()) : o.p + (size_t)r0 * o.stride, o.stride, o.part_units};
}

// Whether the rows of a prompt pass share K and V (attn_prompt_k) or are attended one by one.  Shared, a
// pass is a chain of 6 us per 128 tokens of context however few its rows are, after a start of some
// 10 us; one by one, 4.1 ns per row, KV head and 64 tokens (16 query heads per KV head: 5.8 ns), and
// contexts that one workgroup takes whole cost least of all.  So there have to be rows enough, and context.
// Measured, us per layer, passes behind each other, shared against one by one: 4 KV heads of 7 query heads,
// 192 rows up to 192 / 576 / 1536 tokens 20 : 10, 36 : 47, 70 : 78, 128 rows up to 1024 tokens 50 : 42; 2 of 16,
// 256 rows up to 512 / 768 / 2048 tokens 31 : 20, 42 : 51, 88 : 93, 512 rows up to 512 tokens 32 : 32.
bool rows_share_kv(spark_ctx *c, int m) {
  if (c->attn_prompt_min_rows > 0) return m >= c->attn_prompt_min_rows;
  const int pairs = m * c->cfg.n_kv_heads, tokens = c->attn_splits_now * ATTN_SLICE;
  return m >= 64 && (c->dv.group > 8 ? pairs >= 576 && tokens >= 512 : pairs >= 704 && tokens >= 320);
}

template <typename WT> int launch_attention(spark_ctx *c, const RowDesc *rows, int m, int layer, const RowOut &out, RowMax &row_max) {
  int rc = prof_begin(c, SPARK_KC_ATTN);
  if (rc) return rc;
  // the rows of a prompt pass share their sequence's K and V
  if constexpr (std::is_same<WT, bf16_t>::value) {
    if (c->prompt_pass && rows_share_kv(c, m) && c->cfg.head_dim == 128 && c->dv.group <= 16 && c->use_mfma) {
      auto kern = out.part_units ? attn_prompt_k<128, true> : attn_prompt_k<128, false>;
      const auto key = std::make_pair((const void *)kern, AP_LDS_BYTES);
      if (c->occ_cache.find(key) == c->occ_cache.end()) {
        HIP_TRY(c, hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)AP_LDS_BYTES));
        c->occ_cache.emplace(key, 1);
      }
      const int per = AP_PAIRS / c->dv.group, tiles = (m + per - 1) / per;
      kern<<<tiles * c->cfg.n_kv_heads, AP_THREADS, AP_LDS_BYTES, c->stream>>>(rows, m, c->pb.q, kv_view(c), layer, c->cfg.n_q_heads, c->dv.group,
                                                                              per, tiles, 1.0f / sqrtf(128.0f), out, row_max);
      HIP_TRY(c, hipGetLastError());
      row_max.n = c->cfg.n_q_heads;
      return prof_end(c, SPARK_KC_ATTN);
    }
  }
  // (the slices' partial results fit for as many rows at a time as a pass in the base buffers has)
  const size_t qw = (size_t)c->cfg.n_q_heads * c->cfg.head_dim;
  for (int r0 = 0; r0 < m; r0 += c->base.rows) {
    RowMax rm = row_max;
    if (rm.list) rm.list += (size_t)r0 * rm.stride;
    if ((rc = launch_attention_rows<WT>(c, rows + r0, std::min(c->base.rows, m - r0), m, layer, c->pb.q + r0 * qw,
                                        from_row(out, r0), rm))) return rc;
    row_max.n = rm.n;
  }
  return prof_end(c, SPARK_KC_ATTN);
}

// ------------------------------------------------------------------ MFMA path (five and more rows, bf16)


// Which kernel takes a pass's projections, and with it how the rows that they read lie in memory: on the
// copy of the weights fp32 rows, where a pass of few of them streams it (mfma_direct_k) and wants
// operand order; on the caller's weights bf16 parts, part_elems apart.
bool on_copy(spark_ctx *c) { return c->has_tiled && c->use_tiled; }
bool in_operand_order(spark_ctx *c, int m) { return on_copy(c) && m <= std::min(OP_ROWS, c->direct_max_rows); }
RowOut rows_out(spark_ctx *c, float *p, size_t part_elems, int m, int width) {
  if (!on_copy(c)) return RowOut{p, width, (int)(part_elems / 64)};
  return RowOut{p, in_operand_order(c, m) ? -(m <= 32 ? 32 : OP_ROWS) : width, 0};
}
RowMax row_max_list(spark_ctx *c, uint8_t *list, int bytes, int n) { return on_copy(c) ? RowMax{list, bytes, n} : RowMax{nullptr, 0, 0}; }
ProjIn proj_in(const RowOut &x, const RowMax &row_max) { return ProjIn{x.p, x.stride, x.part_units, row_max, nullptr, 0}; }

int launch_prep(spark_ctx *c, const RowDesc *rows, int m, const float *src, int stride, int indirect,
                const float *gamma, int n) {
  prep_rows_k<<<m, 256, 0, c->stream>>>(rows, src, stride, indirect, gamma, c->cfg.rms_eps, n,
                                        rows_out(c, c->pb.xnorm, c->lo.part_elems, m, n), row_max_list(c, c->pb.max_x, max_x_bytes(c->cfg), 1));
  HIP_TRY(c, hipGetLastError());
  return SPARK_OK;
}
// normalised rows as a projection's input, their magnitudes in `n_max` parts
ProjIn prepared(spark_ctx *c, int m, int n_max) {
  return proj_in(rows_out(c, c->pb.xnorm, c->lo.part_elems, m, c->cfg.d_model), row_max_list(c, c->pb.max_x, max_x_bytes(c->cfg), n_max));
}

// tasks one thread of the finishing kernel takes: the vocabulary heads reduce their arg-max over 8
// per thread, then over the workgroup's threads of the same row
template <typename Epi> int finish_tasks_per_thread(const Epi &) { return 1; }
template <typename WT> int finish_tasks_per_thread(const EpiVocab<WT> &) { return 8; }

template <int MTILES, typename Epi, bool SPLIT, int WAVES>
int mfma_occupancy(spark_ctx *c) {
  auto kern = mfma_rows_k<MTILES, Epi, SPLIT, WAVES>;
  const size_t lds = mg_lds_bytes(MTILES, WAVES);
  const auto key = std::make_pair((const void *)kern, lds);
  auto found = c->occ_cache.find(key);
  if (found == c->occ_cache.end()) {
    if (lds > 65536)
      HIP_TRY(c, hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
    int o = 0;
    HIP_TRY(c, hipOccupancyMaxActiveBlocksPerMultiprocessor(&o, kern, 64 * WAVES, lds));
    if (o < 1) return fail(c, SPARK_EHIP, "the MFMA kernel for %d rows does not fit on a CU", 32 * MTILES);
    found = c->occ_cache.emplace(key, o).first;
  }
  return found->second;
}

// (what lies there then are no words of a hand-over any more)
float *partial_sums(spark_ctx *c) {
  c->row_words_clean = false;
  return at<float>(c, c->lo.mfma_part);
}
// (a cover is chosen so that its partial sums fit; one that did not would write into what lies behind them)
int partials_fit(spark_ctx *c, size_t bytes) {
  if (bytes <= MFMA_PARTIAL_BYTES) return SPARK_OK;
  return fail(c, SPARK_EINVAL, "partial sums of %zu bytes do not fit their buffer", bytes);
}

template <typename Epi> int launch_finish(spark_ctx *c, const Epi &epi, const RowDesc *rows, int m, int n_tasks, const PartialSums &ps) {
  const dim3 grid(ps.tc.n_cut * ((ps.tasks_per_tile + 31) / 32), (ps.m_pitch + 31) / 32);
  if (ps.n_split <= 8) mfma_finish_tile_k<Epi, 8><<<grid, 1024, 0, c->stream>>>(epi, rows, m, n_tasks, ps);
  else mfma_finish_tile_k<Epi, MG_MAX_SPLIT><<<grid, 1024, 0, c->stream>>>(epi, rows, m, n_tasks, ps);
  HIP_TRY(c, hipGetLastError());
  return SPARK_OK;
}

// an epilogue that adds up a whole row runs in the finishing launch only (and with it the others of
// matrices that never have a CU's worth of tiles); one with a running arg-max in the projection only
template <typename Epi> struct CutRule {
  static constexpr bool always = EpiRow<Epi>::sum || std::is_same<Epi, EpiResidual<bf16_t>>::value || std::is_same<Epi, EpiLensAffine<bf16_t>>::value;
  static constexpr bool never = EpiHasLocalReduce<Epi>::value;
};

// y = W x for m rows on the copy of the weights in MFMA operand order
template <int MTILES, int TB, typename Epi>
int launch_tiled(spark_ctx *c, const Epi &epi, const RowDesc *rows, int m, int n_in, int n_tasks, const ProjIn &in,
                 const TiledMatrix &w, int *max_words) {
  constexpr bool ALWAYS_CUT = CutRule<Epi>::always, NEVER_CUT = CutRule<Epi>::never;
  constexpr int TASKS = 32 * TG_WAVES * TB, MROWS = 32 * MTILES;
  const TileCover tc = cover_tiled(m, n_in, n_tasks, MTILES, TB, ALWAYS_CUT, NEVER_CUT, c->n_cu, c->mfma_xcd_max_split);
  if (int rc = partials_fit(c, tiled_partial_bytes(tc, TB))) return rc;
  if (max_words) *max_words = tc.n_cut ? (n_tasks + 31) / 32 : (n_tasks + 32 * TB - 1) / (32 * TB);
  const f16_t *tiled = at<f16_t>(c, c->lo.tiled) + w.elems;
  const float *wdown = at<float>(c, c->lo.wdown) + w.blocks * 32;
  float *part = partial_sums(c);
  const int grid = tc.n_whole + tc.n_cut * tc.n_split;
  const size_t lds = tg_lds_bytes(MTILES, TB);
  auto launch = [&](auto kern) {
    if (lds > 65536) {
      const auto key = std::make_pair((const void *)kern, lds);
      if (c->occ_cache.find(key) == c->occ_cache.end()) {
        HIP_TRY(c, hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
        c->occ_cache.emplace(key, 1);
      }
    }
    kern<<<grid, 64 * TG_WAVES, lds, c->stream>>>(epi, tiled, wdown, rows, m, in, n_in, n_tasks, tc, part);
    HIP_TRY(c, hipGetLastError());
    return SPARK_OK;
  };
  int rc;
  if constexpr (ALWAYS_CUT) rc = launch(mfma_tiled_k<MTILES, TB, Epi, false>);
  else if constexpr (NEVER_CUT) rc = launch(mfma_tiled_k<MTILES, TB, Epi, true>);
  else rc = tc.n_whole ? launch(mfma_tiled_k<MTILES, TB, Epi, true>) : launch(mfma_tiled_k<MTILES, TB, Epi, false>);
  if (rc) return rc;
  if constexpr (!NEVER_CUT) {
    if (tc.n_cut) return launch_finish(c, epi, rows, m, n_tasks, PartialSums{part, tc.n_split, tc.m_pitch, TASKS, MROWS, tc});
  }
  return SPARK_OK;
}

template <int TB, typename Epi>
int launch_tiled_rows(spark_ctx *c, const Epi &epi, const RowDesc *rows, int m, int n_in, int n_tasks, const ProjIn &in,
                      const TiledMatrix &w, int *max_words) {
  const int most = std::min(c->tiled_row_blocks, TB == 1 ? 4 : 3);   // (what the accumulators allow)
  const int mt = TB == 1 && !CutRule<Epi>::never ? narrow_row_blocks(m, n_in, n_tasks, most, CutRule<Epi>::always, c->n_cu)
                                                 : tiled_row_blocks_for(m, most);
  switch (mt) {
    case 2: return launch_tiled<2, TB, Epi>(c, epi, rows, m, n_in, n_tasks, in, w, max_words);
    case 3: return launch_tiled<3, TB, Epi>(c, epi, rows, m, n_in, n_tasks, in, w, max_words);
    default:
      if constexpr (TB == 1) return launch_tiled<4, TB, Epi>(c, epi, rows, m, n_in, n_tasks, in, w, max_words);
      return fail(c, SPARK_EINVAL, "row tiles of %d blocks", mt);
  }
}

// the same on whole tiles of two heights
template <int TB, typename Epi>
int launch_mixed(spark_ctx *c, const Epi &epi, const RowDesc *rows, int m, int n_in, int n_tasks, const ProjIn &in,
                 const TiledMatrix &w, const MixedCover &mc, int *max_words) {
  auto kern = mfma_tiled_mixed_k<TB, Epi>;
  const size_t lds = tg_lds_bytes(3, TB);
  if (lds > 65536) {
    const auto key = std::make_pair((const void *)kern, lds);
    if (c->occ_cache.find(key) == c->occ_cache.end()) {
      HIP_TRY(c, hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
      c->occ_cache.emplace(key, 1);
    }
  }
  if (max_words) *max_words = (n_tasks + 32 * TB - 1) / (32 * TB);
  kern<<<mc.tiles(), 64 * TG_WAVES, lds, c->stream>>>(epi, at<f16_t>(c, c->lo.tiled) + w.elems, at<float>(c, c->lo.wdown) + w.blocks * 32, rows, m, in,
                                                     n_in, n_tasks, mc);
  HIP_TRY(c, hipGetLastError());
  return SPARK_OK;
}
// The cover by tiles of two heights if it is the better one, or nullptr.  Found once for a row count (on one core 2 to 6 us
// up to 1024 rows, 18 at the 3072 of a large flush, 18944 tasks), and kept for all that passes of the backbones can have (108).
int mixed_cover(spark_ctx *c, int m, int n_in, int n_tasks, const MixedCover **out) {
  *out = nullptr;
  if (c->tiled_row_blocks < 3) return SPARK_OK;
  const int blocks = ceil_div(m, 32);
  const std::array<int, 3> key{blocks, n_in, n_tasks};
  auto found = c->mixed_covers.find(key);
  if (found == c->mixed_covers.end()) {
    if (c->mixed_covers.size() >= 128) c->mixed_covers.clear();
    found = c->mixed_covers.emplace(key, choose_mixed(32 * blocks, n_in, n_tasks, 3, c->n_cu)).first;
  }
  if (found->second.cost > 0.f) *out = &found->second;
  return SPARK_OK;
}

// the same for few rows, in operand order
template <int NT, int COLS, bool CUT, typename Epi>
int launch_direct_cols(spark_ctx *c, const Epi &epi, const RowDesc *rows, int m, int n_in, int n_tasks, const ProjIn &in,
                       const TiledMatrix &w, int groups, int split, int cps) {
  auto kern = mfma_direct_k<NT, COLS, Epi, CUT>;
  const size_t lds = td_lds_bytes(NT, COLS);
  if (lds > 65536) {
    const auto key = std::make_pair((const void *)kern, lds);
    if (c->occ_cache.find(key) == c->occ_cache.end()) {
      HIP_TRY(c, hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
      c->occ_cache.emplace(key, 1);
    }
  }
  kern<<<groups * split, 64 * TD_WAVES, lds, c->stream>>>(epi, at<f16_t>(c, c->lo.tiled) + w.elems, at<float>(c, c->lo.wdown) + w.blocks * 32,
                                                          rows, m, in, n_in, n_tasks, groups, cps, partial_sums(c),
                                                          at<int>(c, c->lo.arrivals));   // (zero between launches, attention's too)
  HIP_TRY(c, hipGetLastError());
  return SPARK_OK;
}
template <int NT, bool CUT, typename Epi>
int launch_direct_tiles(spark_ctx *c, const Epi &epi, const RowDesc *rows, int m, int n_in, int n_tasks, const ProjIn &in,
                        const TiledMatrix &w, int groups, int split, int cps) {
  if (m <= 16) return launch_direct_cols<NT, 16, CUT>(c, epi, rows, m, n_in, n_tasks, in, w, groups, split, cps);
  if (m <= 32) return launch_direct_cols<NT, 32, CUT>(c, epi, rows, m, n_in, n_tasks, in, w, groups, split, cps);
  return launch_direct_cols<NT, 48, CUT>(c, epi, rows, m, n_in, n_tasks, in, w, groups, split, cps);
}
template <typename Epi>
int launch_direct(spark_ctx *c, const Epi &epi, const RowDesc *rows, int m, int n_in, int n_tasks, const ProjIn &in,
                  const TiledMatrix &w, int *max_words) {
  const int n_chunks = (n_in + MG_KC - 1) / MG_KC, blocks = (n_tasks + TG_TASKS - 1) / TG_TASKS;
  if constexpr (!EpiHasLocalReduce<Epi>::value && !EpiRow<Epi>::max || EpiRow<Epi>::sum) {
    const DirectCut cut = direct_cut(m, n_in, n_tasks, c->n_cu, c->direct_whole_k);
    if (cut.split > 1 && (size_t)cut.groups <= (size_t)c->dv.max_rows * c->cfg.n_q_heads) {   // (one arrival word per group)
      if (int rc = partials_fit(c, direct_partial_bytes(m, cut))) return rc;
      if (max_words) *max_words = cut.groups;
      return cut.tiles == 1 ? launch_direct_tiles<1, true>(c, epi, rows, m, n_in, n_tasks, in, w, cut.groups, cut.split, cut.chunks_per_split)
                            : launch_direct_tiles<TD_CUT_TILES, true>(c, epi, rows, m, n_in, n_tasks, in, w, cut.groups, cut.split, cut.chunks_per_split);
    }
  }
  const int nt = direct_tiles(m, blocks, c->n_cu, EpiHasLocalReduce<Epi>::value);
  const int groups = (blocks + nt - 1) / nt;
  if (max_words) *max_words = groups;
  switch (nt) {
    case 1: return launch_direct_tiles<1, false>(c, epi, rows, m, n_in, n_tasks, in, w, groups, 1, n_chunks);
    case 2: return launch_direct_tiles<2, false>(c, epi, rows, m, n_in, n_tasks, in, w, groups, 1, n_chunks);
    case 3: return launch_direct_tiles<3, false>(c, epi, rows, m, n_in, n_tasks, in, w, groups, 1, n_chunks);
    case 4: return launch_direct_tiles<4, false>(c, epi, rows, m, n_in, n_tasks, in, w, groups, 1, n_chunks);
    default: return launch_direct_tiles<5, false>(c, epi, rows, m, n_in, n_tasks, in, w, groups, 1, n_chunks);
  }
}

// y = W x for m rows on the caller's row-major weights
template <int MTILES, typename Epi, int WAVES>
int launch_mfma_shape(spark_ctx *c, const Epi &epi, const RowDesc *rows, int m, int n_in, int n_tasks, const ProjIn &in) {
  constexpr bool LOCAL = EpiHasLocalReduce<Epi>::value;
  constexpr int TASKS_PER_BLOCK = WAVES * MG_TASKS_PER_WAVE;
  const int mrows = 32 * MTILES;
  const int z = (m + mrows - 1) / mrows;
  const int bx = (n_tasks + TASKS_PER_BLOCK - 1) / TASKS_PER_BLOCK;
  const int n_chunks = (n_in + MG_KC - 1) / MG_KC;
  // rows of the partial sums: padded to eight only
  const int m_pad = (int)align_up(m, 8);
  // resident workgroups on the chip: the k range is split until one round of them has work
  int occ = mfma_occupancy<MTILES, Epi, true, WAVES>(c);
  if (occ < 0) return occ;
  const int tiles = bx * z;
  int split = choose_split(tiles, occ * c->n_cu, n_chunks, tiles < 32 ? 4 : 8, range_bytes(1, n_tasks, m_pad));
  const int cps = (n_chunks + split - 1) / split;
  split = (n_chunks + cps - 1) / cps;
  float *part = partial_sums(c);
  // one-dimensional grid: the kernel deals its ids so that the row tiles of a weight tile share an XCD
  const int xcd_groups = z > 1 && split <= c->mfma_xcd_max_split;
  const int tiles_padded = xcd_groups ? (bx * split + 7) / 8 * 8 : bx * split;
  dim3 grid(tiles_padded * z);
  const size_t lds = mg_lds_bytes(MTILES, WAVES);
  // (an epilogue that sums over a row runs in the finishing launch only)
  if (split > 1 || EpiRow<Epi>::sum) {
    if (int rc = partials_fit(c, split * range_bytes(1, n_tasks, m_pad))) return rc;
    mfma_rows_k<MTILES, Epi, true, WAVES><<<grid, 64 * WAVES, lds, c->stream>>>(
        epi, rows, m, in, n_in, n_tasks, cps, part, m_pad, bx, split, z, xcd_groups);
    HIP_TRY(c, hipGetLastError());
    if constexpr (!LOCAL) {
      return launch_finish(c, epi, rows, m, n_tasks,
                           PartialSums{part, split, m_pad, n_tasks, m_pad, TileCover{1, 1, 0, 1, split, cps, m_pad, 1, 0}});
    } else {
      const int tpt = finish_tasks_per_thread(epi);
      const int total = ((n_tasks + tpt - 1) / tpt) * m_pad;
      mfma_finish_k<Epi><<<(total + 255) / 256, 256, 0, c->stream>>>(epi, rows, m, n_tasks, split, part, m_pad, tpt);
    }
  } else if constexpr (!EpiRow<Epi>::sum) {
    occ = mfma_occupancy<MTILES, Epi, false, WAVES>(c);
    if (occ < 0) return occ;
    mfma_rows_k<MTILES, Epi, false, WAVES><<<grid, 64 * WAVES, lds, c->stream>>>(
        epi, rows, m, in, n_in, n_tasks, cps, part, m_pad, bx, split, z, xcd_groups);
  }
  HIP_TRY(c, hipGetLastError());
  return SPARK_OK;
}

template <int MTILES, typename Epi>
int launch_mfma_tiles(spark_ctx *c, const Epi &epi, const RowDesc *rows, int m, int n_in, int n_tasks, const ProjIn &in) {
  if (n_in % 8) return fail(c, SPARK_EINVAL, "MFMA path needs an input width that is a multiple of 8, not %d", n_in);
  // matrices of few rows and a short k (q/k/v, o, the lens translator): four waves per workgroup,
  // so that the launch has enough workgroups without cutting k into ranges too short to stream
  // (measured at 32 rows: q/k/v 23.5 -> 20.8 us, o 20.2 -> 16.0 us; down, with its long k, and
  // gate/up, with its many tiles, are better off with eight)
  const int tiles8 = ((n_tasks + MG_TASKS_PER_BLOCK - 1) / MG_TASKS_PER_BLOCK) * ((m + 32 * MTILES - 1) / (32 * MTILES));
  const bool few = tiles8 < c->mfma_small_tiles && n_in <= c->mfma_small_max_k;
  if (few) return launch_mfma_shape<MTILES, Epi, 4>(c, epi, rows, m, n_in, n_tasks, in);
  return launch_mfma_shape<MTILES, Epi, 8>(c, epi, rows, m, n_in, n_tasks, in);
}

template <typename Epi>
int launch_wide(spark_ctx *c, const Epi &epi, const RowDesc *rows, int m, int n_in, int n_tasks, const ProjIn &in, const TiledMatrix &w, int *max_words) {
  if constexpr (std::is_same<Epi, EpiSwiGLUMax<bf16_t>>::value) {
    const MixedCover *mc;
    if (int rc = mixed_cover(c, m, n_in, n_tasks, &mc)) return rc;
    if (mc) return launch_mixed<2>(c, epi, rows, m, n_in, n_tasks, in, w, *mc, max_words);
    return launch_tiled_rows<2>(c, epi, rows, m, n_in, n_tasks, in, w, max_words);
  }
  else return SPARK_EINVAL;
}

// y = W x for m rows of `in`; w: the copy of the weights in MFMA operand order, or nullptr; max_words:
// how many words of each row's list of magnitudes the launch writes, for an epilogue that does
template <typename Epi>
int launch_mfma(spark_ctx *c, const Epi &epi, const RowDesc *rows, int m, int n_in, int n_tasks, const ProjIn &in,
                int kclass, const TiledMatrix *w, int *max_words = nullptr) {
  int rc = prof_begin(c, kclass);
  if (rc) return rc;
  if constexpr (EpiOutParts<Epi>::value != 1) {
    // 64 tasks per wave for gate/up, 32 for matrices of few rows (q/k/v, o, down, the lens translator), so
    // that the launch has enough workgroups without cutting k into ranges too short to stream, and for the
    // heads, whose tiles are never cut.  (64 for q/k/v, o and down of passes of 700 to 1024 rows, without
    // folded sums: the layers of one backbone 3 to 4 % shorter, of the other 1 to 6 % longer.)
    if (w && in_operand_order(c, m)) rc = launch_direct(c, epi, rows, m, n_in, n_tasks, in, *w, max_words);
    else if (w && std::is_same<Epi, EpiSwiGLUMax<bf16_t>>::value && n_tasks >= TILED_WIDE_TASKS) rc = launch_wide(c, epi, rows, m, n_in, n_tasks, in, *w, max_words);
    else if (w) rc = launch_tiled_rows<1>(c, epi, rows, m, n_in, n_tasks, in, *w, max_words);
  }
  if constexpr (EpiOutParts<Epi>::value != 0) {
    // (mfma_rows_k keeps a running state for one tile of 32 rows at most)
    if (!w) {
      if (m <= 32 || EpiHasLocalReduce<Epi>::value) rc = launch_mfma_tiles<1>(c, epi, rows, m, n_in, n_tasks, in);
      else rc = launch_mfma_tiles<2>(c, epi, rows, m, n_in, n_tasks, in);   // tiles of 64 rows
    }
  }
  if (rc) return rc;
  return prof_end(c, kclass);
}


// The copy of one projection's weights in MFMA operand order, or nullptr when the context has none
// (or is told not to use it).
const TiledMatrix *tiled_at(spark_ctx *c, const TiledMatrix &w) { return on_copy(c) ? &w : nullptr; }

template <typename Epi>
int tile_one(spark_ctx *c, const Epi &epi, int n_tasks, int n_in, const TiledMatrix &w) {
  const int n_chunks = (n_in + MG_KC - 1) / MG_KC, blocks = (int)tg_blocks(n_tasks);
  const auto kern = n_in <= 4 * 1024 ? tile_weights_k<Epi, 4> : n_in <= TW_HELD * 1024 ? tile_weights_k<Epi, TW_HELD> : tile_weights_k<Epi, 0>;
  kern<<<blocks * (32 / TW_ROWS), TW_THREADS, 0, c->stream>>>(epi, n_tasks, n_in, n_chunks, at<float>(c, c->lo.wdown) + w.blocks * 32,
                                                             at<f16_t>(c, c->lo.tiled) + w.elems);
  HIP_TRY(c, hipGetLastError());
  return SPARK_OK;
}

// Writes the MFMA-ordered copies once, with the epilogues' own task -> weight rows mapping (only
// the weight pointers and widths of an epilogue matter here).
int build_tiled(spark_ctx *c) {
  typedef bf16_t WT;
  const spark_config &g = c->cfg;
  const int d = g.d_model, hd = g.head_dim, nq = g.n_q_heads, nkv = g.n_kv_heads, F = g.d_ffn, V = c->dv.V;
  const size_t qw = (size_t)nq * hd, kvw = (size_t)nkv * hd;
  int rc;
  for (int l = 0; l < g.n_layers; ++l) {
    EpiQKV<WT> eq;
    eq.wq = (const WT *)c->w.wq + (size_t)l * qw * d;
    eq.wk = (const WT *)c->w.wk + (size_t)l * kvw * d;
    eq.wv = (const WT *)c->w.wv + (size_t)l * kvw * d;
    eq.d = d; eq.nq = nq; eq.nkv = nkv; eq.hd = hd; eq.layer = l;
    eq.qbuf = nullptr; eq.rope = nullptr; eq.kv = kv_view(c);
    if ((rc = tile_one(c, eq, (nq + 2 * nkv) * (hd / 2), d, c->tm.qkv[l]))) return rc;
    EpiResidual<WT> eo{(const WT *)c->w.wo + (size_t)l * d * qw, (int)qw, d, nullptr, d};
    if ((rc = tile_one(c, eo, d / 2, (int)qw, c->tm.o[l]))) return rc;
    EpiSwiGLUMax<WT> eg{(const WT *)c->w.wg + (size_t)l * F * d, (const WT *)c->w.wu + (size_t)l * F * d, d, F,
                        RowOut{nullptr, 0, 0}, RowMax{nullptr, 0, 0}};
    if ((rc = tile_one(c, eg, F, d, c->tm.gateup[l]))) return rc;
    EpiResidual<WT> ed{(const WT *)c->w.wd + (size_t)l * d * F, F, d, nullptr, d};
    if ((rc = tile_one(c, ed, d / 2, F, c->tm.down[l]))) return rc;
  }
  EpiLensAffine<WT> ea{(const WT *)c->w.lens_a, nullptr, nullptr, nullptr, d};
  if ((rc = tile_one(c, ea, d / 2, d, c->tm.lens_a))) return rc;
  EpiVocab<WT> el{(const WT *)c->w.lens_head, d, V, nullptr, nullptr};
  if ((rc = tile_one(c, el, (V + 1) / 2, d, c->tm.lens_head))) return rc;
  EpiVocab<WT> ev{(const WT *)c->w.lm_head, d, V, nullptr, nullptr};
  if ((rc = tile_one(c, ev, (V + 1) / 2, d, c->tm.lm_head))) return rc;
  HIP_TRY(c, hipStreamSynchronize(c->stream));
  return SPARK_OK;
}

// layers [l0, l1) on m rows, bf16 weights.  SPLIT: on the caller's weights, the rows handed on as bf16 parts
template <bool SPLIT>
int run_layers_mfma(spark_ctx *c, int l0, int l1, const RowDesc *rows, int m) {
  typedef bf16_t WT;
  const spark_config &g = c->cfg;
  const int d = g.d_model, hd = g.head_dim, nq = g.n_q_heads, nkv = g.n_kv_heads, F = g.d_ffn;
  const size_t qw = (size_t)nq * hd, kvw = (size_t)nkv * hd;
  float *hidden = c->pb.hidden;
  // (as parts, the attention output takes the place of the rows that q/k/v have read)
  const RowOut xnorm = rows_out(c, c->pb.xnorm, c->lo.part_elems, m, d),
               attn_out = rows_out(c, on_copy(c) ? c->pb.attn : c->pb.xnorm, c->lo.part_elems, m, (int)qw),
               act = rows_out(c, c->pb.act, c->lo.act_part_elems, m, F);
  // RMSNorm is linear in 1/rms: the finishing launch of a residual projection writes gamma (.) h
  // for the projection that follows and adds up h's sum of squares per row; that projection's
  // epilogue scales by 1/rms.  Only the first norm of a run is a launch of its own.
  // The sums start at zero: those of the MLP's norm are cleared by q/k/v (read last by gate/up of
  // the layer before, added to next by o), those of the layer's input by gate/up (read last by
  // q/k/v, added to next by down).
  unsigned long long *ssq_in = c->pb.ssq, *ssq_mlp = ssq_in + (size_t)SSQ_WAYS * c->pb.rows;
  const int ssq_pitch = std::min((int)align_up(m, 16), c->pb.rows), ssq_units = ssq_pitch * SSQ_WAYS * (int)sizeof(unsigned long long) / 16;
  // (the counts: what the launch that wrote the lists last has written)
  RowMax max_x = row_max_list(c, c->pb.max_x, max_x_bytes(g), 1), max_attn = row_max_list(c, c->pb.max_attn, max_attn_bytes(g), 0),
         max_act = row_max_list(c, c->pb.max_act, max_act_bytes(g), 0);
  const bool fuse = c->fuse_norm;
  int rc;
  for (int l = l0; l < l1; ++l) {
    const bool qkv_scaled = fuse && l > l0;
    if (!qkv_scaled && (rc = launch_prep(c, rows, m, hidden, d, 1, c->w.attn_norm + (size_t)l * d, d))) return rc;
    EpiQKV<WT> eq;
    eq.wq = (const WT *)c->w.wq + (size_t)l * qw * d;
    eq.wk = (const WT *)c->w.wk + (size_t)l * kvw * d;
    eq.wv = (const WT *)c->w.wv + (size_t)l * kvw * d;
    eq.d = d; eq.nq = nq; eq.nkv = nkv; eq.hd = hd; eq.layer = l;
    eq.qbuf = c->pb.q;
    eq.rope = at<float2>(c, c->lo.rope);
    eq.kv = kv_view(c);
    if (qkv_scaled) eq.scale = RowScale{ssq_in, ssq_pitch, 1.0f / (float)d, g.rms_eps};
    ProjIn in = prepared(c, m, qkv_scaled ? max_x.n : 1);
    in.zero = (uint4 *)ssq_mlp;
    in.n_zero = ssq_units;
    if ((rc = launch_mfma(c, eq, rows, m, d, (nq + 2 * nkv) * (hd / 2), in, SPARK_KC_QKV, tiled_at(c, c->tm.qkv[l])))) return rc;

    if ((rc = launch_attention<WT>(c, rows, m, l, attn_out, max_attn))) return rc;

    const ProjIn in_o = proj_in(attn_out, max_attn);
    EpiSwiGLUMax<WT, SPLIT> eg{(const WT *)c->w.wg + (size_t)l * F * d, (const WT *)c->w.wu + (size_t)l * F * d,
                        d, F, act, max_act};
    if (fuse) {
      EpiResidualNorm<WT, SPLIT> eo{(const WT *)c->w.wo + (size_t)l * d * qw, (int)qw, d, hidden, d,
                             c->w.mlp_norm + (size_t)l * d, xnorm, ssq_mlp, ssq_pitch, max_x};
      if ((rc = launch_mfma(c, eo, rows, m, (int)qw, d / 2, in_o, SPARK_KC_OPROJ, tiled_at(c, c->tm.o[l]), &max_x.n))) return rc;
      eg.scale = RowScale{ssq_mlp, ssq_pitch, 1.0f / (float)d, g.rms_eps};
      in = prepared(c, m, max_x.n);
      in.zero = (uint4 *)ssq_in;
      in.n_zero = ssq_units;
    } else {
      EpiResidual<WT> eo{(const WT *)c->w.wo + (size_t)l * d * qw, (int)qw, d, hidden, d};
      if ((rc = launch_mfma(c, eo, rows, m, (int)qw, d / 2, in_o, SPARK_KC_OPROJ, tiled_at(c, c->tm.o[l])))) return rc;
      if ((rc = launch_prep(c, rows, m, hidden, d, 1, c->w.mlp_norm + (size_t)l * d, d))) return rc;
      in = prepared(c, m, 1);
    }
    max_act.n = 0;
    if ((rc = launch_mfma(c, eg, rows, m, d, F, in, SPARK_KC_GATEUP, tiled_at(c, c->tm.gateup[l]), &max_act.n))) return rc;

    const ProjIn in_d = proj_in(act, max_act);
    if (fuse && l + 1 < l1) {
      EpiResidualNorm<WT, SPLIT> ed{(const WT *)c->w.wd + (size_t)l * d * F, F, d, hidden, d,
                             c->w.attn_norm + (size_t)(l + 1) * d, xnorm, ssq_in, ssq_pitch, max_x};
      if ((rc = launch_mfma(c, ed, rows, m, F, d / 2, in_d, SPARK_KC_DOWN, tiled_at(c, c->tm.down[l]), &max_x.n))) return rc;
    } else {
      EpiResidual<WT> ed{(const WT *)c->w.wd + (size_t)l * d * F, F, d, hidden, d};
      if ((rc = launch_mfma(c, ed, rows, m, F, d / 2, in_d, SPARK_KC_DOWN, tiled_at(c, c->tm.down[l])))) return rc;
    }
  }
  return SPARK_OK;
}

// layers [l0, l1) on m rows described by `rows` (device)
// ------------------------------------------------------------------ a pass of one row in one launch

// Where the words of the hand-overs lie in the area of the partial sums (which the other projections leave floats in)
struct RowWords { size_t h0, h1, qkv, attn, act, part, end; };
RowWords row_words(const spark_config &g) {
  const size_t qw = (size_t)g.n_q_heads * g.head_dim, kvw = (size_t)g.n_kv_heads * g.head_dim, dm = g.d_model;
  RowWords w;
  w.h0 = 0;
  w.h1 = w.h0 + dm;
  w.qkv = w.h1 + dm;
  w.attn = w.qkv + qw + 2 * kvw;
  w.act = w.attn + qw;
  w.part = w.act + (size_t)ROW_PARTS * ROW_WGS * row_slots(g.d_ffn);
  w.end = w.part + (size_t)(g.n_q_heads / g.n_kv_heads) * ROW_WGS * (ROW_HD + 2);   // (a workgroup has one slice of a KV head)
  return w;
}

OneRow one_row_shape(const spark_config &g) {
  OneRow a{};
  a.d = g.d_model; a.nq = g.n_q_heads; a.nkv = g.n_kv_heads; a.F = g.d_ffn; a.eps = g.rms_eps;
  return a;
}

// Every workgroup has a pair of every projection, of gate/up one in each piece: that it has written its part of a row
// then says that it no longer reads what the row was made of.
bool shape_allows_one_row(const spark_config &g) {
  const int qw = g.n_q_heads * g.head_dim;
  OneRow a = one_row_shape(g);
  return g.dtype == SPARK_DTYPE_BF16 && g.head_dim == ROW_HD && g.n_q_heads / g.n_kv_heads <= ROW_MAX_GROUP &&
         g.d_model % 8 == 0 && g.d_ffn % 8 == 0 && g.d_model <= ROW_MAX_D && qw <= ROW_MAX_D && g.d_model >= 2 * ROW_WGS &&
         (g.n_q_heads + 2 * g.n_kv_heads) * (ROW_HD / 2) >= ROW_WGS && g.d_ffn >= ROW_PARTS * ROW_WGS &&
         one_row_lds(a) > 0 && sizeof(row_word) * row_words(g).end <= MFMA_PARTIAL_BYTES;
}

// Whether a pass of one row takes the one launch: where it pays, and attention has at most one slice of 64 tokens per workgroup.
bool one_row_runs(const spark_ctx *c, int layers) {
  if (!c->row_ok || !c->use_row || !c->may_wait || c->prof_class >= 0 || c->attn_splits_now <= 0 || c->cfg.n_kv_heads * c->attn_splits_now > ROW_WGS) return false;
  return c->use_row == 2 || one_row_pays(c->layer_bytes, layers);
}

__global__ void __launch_bounds__(256) clear_words_k(row_word *words, size_t n) {
  for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (size_t)gridDim.x * 256) words[i] = 0ull;
}

// false: refused.  The runtime has one cooperative queue for all processes on a card, and to be told that another has it
// takes 38 ms, so a context asks once (asked on every pass, ten steps of four layers took 380 ms instead of 1.2).
bool enqueue_one_row(spark_ctx *c, int l0, int l1, const RowDesc *row) {
  const spark_config &g = c->cfg;
  OneRow a = one_row_shape(g);
  const size_t lds = one_row_lds(a);
  const RowWords w = row_words(g);
  row_word *words = at<row_word>(c, c->lo.mfma_part);
  const unsigned layers = (unsigned)(l1 - l0);
  if (!c->row_words_clean || row_numbers_run_out(c->row_tag, layers)) {
    clear_words_k<<<256, 256, 0, c->stream>>>(words, w.end);
    c->row_words_clean = true;
    c->row_tag = 0;
  }
  a.l0 = l0; a.l1 = l1;
  a.scale = 1.0f / sqrtf((float)ROW_HD);
  a.wq = (const bf16_t *)c->w.wq; a.wk = (const bf16_t *)c->w.wk; a.wv = (const bf16_t *)c->w.wv; a.wo = (const bf16_t *)c->w.wo;
  a.wg = (const bf16_t *)c->w.wg; a.wu = (const bf16_t *)c->w.wu; a.wd = (const bf16_t *)c->w.wd;
  a.attn_norm = c->w.attn_norm; a.mlp_norm = c->w.mlp_norm;
  a.rope = at<float2>(c, c->lo.rope);
  a.kv = kv_view(c);
  a.row = row;
  a.hidden = c->pb.hidden;
  a.h0 = words + w.h0; a.h1 = words + w.h1; a.qkv = words + w.qkv; a.attn = words + w.attn; a.act = words + w.act; a.part = words + w.part;
  a.tag = c->row_tag + 1;
  c->row_tag += layers;
  a.error = at<int>(c, c->lo.plan) + PL_ERR;
  a.max_polls = c->wait_polls ? std::abs(c->wait_polls) : ROW_MAX_POLLS;
  if (launch_one_row(a, lds, c->stream) == hipSuccess) {
    c->row_taken = true;
    return true;
  }
  (void)hipGetLastError();
  c->use_row = 0;
  return false;
}

template <typename WT>
int run_layers(spark_ctx *c, int l0, int l1, const RowDesc *rows, int m) {
  const spark_config &g = c->cfg;
  if (l0 >= l1 || m <= 0) return SPARK_OK;
  // many rows: the projections are dense contractions for the MFMA units
  if (std::is_same<WT, bf16_t>::value && m >= c->mfma_min_rows && c->use_mfma) {
    // (more rows go through the layers in pieces, in order, so that a piece finds the K and V of the rows before it)
    const int most = pass_rows_limit(g.d_model);
    for (int r0 = 0; r0 < m; r0 += most) {
      const int rc = on_copy(c) ? run_layers_mfma<false>(c, l0, l1, rows + r0, std::min(most, m - r0))
                                : run_layers_mfma<true>(c, l0, l1, rows + r0, std::min(most, m - r0));
      if (rc) return rc;
    }
    return SPARK_OK;
  }
  const int d = g.d_model, hd = g.head_dim, nq = g.n_q_heads, nkv = g.n_kv_heads, F = g.d_ffn;
  const size_t qw = (size_t)nq * hd, kvw = (size_t)nkv * hd;
  if (std::is_same<WT, bf16_t>::value && m == 1 && one_row_runs(c, l1 - l0) && enqueue_one_row(c, l0, l1, rows)) return SPARK_OK;
  float *hidden = c->pb.hidden;
  int rc;
  for (int l = l0; l < l1; ++l) {
    ProNorm n1{hidden, c->w.attn_norm + (size_t)l * d, g.rms_eps, d, 1};
    EpiQKV<WT> eq;
    eq.wq = (const WT *)c->w.wq + (size_t)l * qw * d;
    eq.wk = (const WT *)c->w.wk + (size_t)l * kvw * d;
    eq.wv = (const WT *)c->w.wv + (size_t)l * kvw * d;
    eq.d = d; eq.nq = nq; eq.nkv = nkv; eq.hd = hd; eq.layer = l;
    eq.qbuf = c->pb.q;
    eq.rope = at<float2>(c, c->lo.rope);
    eq.kv = kv_view(c);
    if ((rc = launch_gemv<WT>(c, n1, eq, rows, m, d, (nq + 2 * nkv) * (hd / 2), SPARK_KC_QKV))) return rc;

    RowMax no_list{nullptr, 0, 0};
    if ((rc = launch_attention<WT>(c, rows, m, l, RowOut{c->pb.attn, (int)qw, 0}, no_list))) return rc;

    ProPlain pa{c->pb.attn, (int)qw, 0};
    EpiResidual<WT> eo{(const WT *)c->w.wo + (size_t)l * d * qw, (int)qw, d, hidden, d};
    if ((rc = launch_gemv<WT>(c, pa, eo, rows, m, (int)qw, d / 2, SPARK_KC_OPROJ))) return rc;

    ProNorm n2{hidden, c->w.mlp_norm + (size_t)l * d, g.rms_eps, d, 1};
    EpiSwiGLU<WT> eg{(const WT *)c->w.wg + (size_t)l * F * d, (const WT *)c->w.wu + (size_t)l * F * d,
                     d, F, c->pb.act};
    if ((rc = launch_gemv<WT>(c, n2, eg, rows, m, d, F, SPARK_KC_GATEUP))) return rc;

    ProPlain pd{c->pb.act, F, 0};
    EpiResidual<WT> ed{(const WT *)c->w.wd + (size_t)l * d * F, F, d, hidden, d};
    if ((rc = launch_gemv<WT>(c, pd, ed, rows, m, F, d / 2, SPARK_KC_DOWN))) return rc;
  }
  return SPARK_OK;
}

template <typename WT> int run_lens_head(spark_ctx *c, const RowDesc *rows, int m) {
  const spark_config &g = c->cfg;
  const int d = g.d_model, V = c->dv.V;
  float *hidden = c->pb.hidden, *u = at<float>(c, c->lo.lens_u);
  int rc;
  if (std::is_same<WT, bf16_t>::value && m >= c->mfma_min_rows && c->use_mfma) {
    if ((rc = launch_prep(c, rows, m, hidden, d, 1, nullptr, d))) return rc;
    EpiLensAffine<bf16_t> ea{(const bf16_t *)c->w.lens_a, c->w.lens_b, hidden, u, d};
    if ((rc = launch_mfma(c, ea, rows, m, d, d / 2, prepared(c, m, 1), SPARK_KC_LENS, tiled_at(c, c->tm.lens_a)))) return rc;
    if ((rc = launch_prep(c, rows, m, u, d, 0, c->w.lens_norm, d))) return rc;
    EpiVocab<bf16_t> ev{(const bf16_t *)c->w.lens_head, d, V, at<float>(c, c->lo.logits),
                        at<unsigned long long>(c, c->lo.best)};
    return launch_mfma(c, ev, rows, m, d, (V + 1) / 2, prepared(c, m, 1), SPARK_KC_LENS, tiled_at(c, c->tm.lens_head));
  }
  ProPlain ph{hidden, d, 1};
  EpiLensAffine<WT> ea{(const WT *)c->w.lens_a, c->w.lens_b, hidden, u, d};
  if ((rc = launch_gemv<WT>(c, ph, ea, rows, m, d, d / 2, SPARK_KC_LENS))) return rc;
  // the translated state sits in u[pass row]; normalising it is the head's prologue
  ProNorm pn{u, c->w.lens_norm, g.rms_eps, d, 0};
  EpiVocab<WT> ev{(const WT *)c->w.lens_head, d, V, at<float>(c, c->lo.logits),
                  at<unsigned long long>(c, c->lo.best)};
  return launch_gemv<WT>(c, pn, ev, rows, m, d, (V + 1) / 2, SPARK_KC_LENS);
}

template <typename WT> int run_final_head(spark_ctx *c, const RowDesc *rows, int m) {
  const spark_config &g = c->cfg;
  const int d = g.d_model, V = c->dv.V;
  if (std::is_same<WT, bf16_t>::value && m >= c->mfma_min_rows && c->use_mfma) {
    int rc;
    if ((rc = launch_prep(c, rows, m, c->pb.hidden, d, 1, c->w.final_norm, d))) return rc;
    EpiVocab<bf16_t> ev{(const bf16_t *)c->w.lm_head, d, V, at<float>(c, c->lo.logits),
                        at<unsigned long long>(c, c->lo.best)};
    return launch_mfma(c, ev, rows, m, d, (V + 1) / 2, prepared(c, m, 1), SPARK_KC_HEAD, tiled_at(c, c->tm.lm_head));
  }
  ProNorm pn{c->pb.hidden, c->w.final_norm, g.rms_eps, d, 1};
  EpiVocab<WT> ev{(const WT *)c->w.lm_head, d, V, at<float>(c, c->lo.logits),
                  at<unsigned long long>(c, c->lo.best)};
  return launch_gemv<WT>(c, pn, ev, rows, m, d, (V + 1) / 2, SPARK_KC_HEAD);
}

}  // namespace

// ------------------------------------------------------------------ C ABI

namespace {

Seq *find_seq(spark_ctx *c, int id) {
  if (id < 0 || id >= (int)c->seqs.size() || !c->seqs[id].open) return nullptr;
  return &c->seqs[id];
}

// make sure `seq` owns pages for positions [0, upto); new page-table entries go to the device
int ensure_pages(spark_ctx *c, int id, int upto) {
  Seq &s = c->seqs[id];
  const int pt = c->cfg.kv_page_tokens;
  const int need = (upto + pt - 1) / pt;
  const int have = (int)s.pages.size();
  if (need <= have) return SPARK_OK;
  if (need > c->dv.max_pages) return fail(c, SPARK_ENOMEM, "sequence %d exceeds max_seq_len", id);
  if ((int)c->free_pages.size() < need - have) return fail(c, SPARK_ENOMEM, "KV pool exhausted");
  for (int p = have; p < need; ++p) {
    s.pages.push_back(c->free_pages.back());
    c->free_pages.pop_back();
  }
  int *dst = at<int>(c, c->lo.page_table) + (size_t)id * c->dv.max_pages + have;
  HIP_TRY(c, hipMemcpyAsync(dst, s.pages.data() + have, sizeof(int) * (need - have),
                            hipMemcpyHostToDevice, c->stream));
  // the source vector may be reallocated by a later push_back
  HIP_TRY(c, hipStreamSynchronize(c->stream));
  return SPARK_OK;
}

StepIO step_io(spark_ctx *c, int n) {
  return StepIO{n, at<int>(c, c->lo.seq_ids), at<int>(c, c->lo.state), at<int>(c, c->lo.plan), at<int>(c, c->lo.step_flags),
                at<unsigned long long>(c, c->lo.best)};
}

// One step.  The tokens of the step before it in the same call (prev_tokens: not the first) are
// emitted by the launch that dispatches this one; prev_forced: the ids forced upon it.
template <typename WT>
int enqueue_step(spark_ctx *c, int n, int n_upper, int n_ee, int n_full, const int *prev_forced, int *prev_tokens,
                 const unsigned long long *rand_dev, int *out_depth_dev) {
  const spark_config &g = c->cfg;
  RowDesc *lower = at<RowDesc>(c, c->lo.lower), *upper = at<RowDesc>(c, c->lo.upper);
  RowDesc *ee = at<RowDesc>(c, c->lo.ee), *full = at<RowDesc>(c, c->lo.full);
  unsigned long long *best = at<unsigned long long>(c, c->lo.best);
  int rc;
  const StepIO io = step_io(c, n);
  // one workgroup embeds up to eight rows as fast as a second launch would start (as launches of a small model's
  // step the three took 1.7 + 2.1 + 3.9 us and the gaps between them, this one 3.9)
  if (n <= EMBED_SEQS) {
    next_step_k<WT, true><<<1, 1024, 0, c->stream>>>(c->sp, io, prev_tokens != nullptr, prev_forced, prev_tokens, lower, upper, ee, full,
                                                     out_depth_dev, (const WT *)c->w.embed, g.d_model, c->pb.hidden);
  } else {
    next_step_k<WT, false><<<1, SCHED_THREADS, 0, c->stream>>>(c->sp, io, prev_tokens != nullptr, prev_forced, prev_tokens, lower, upper, ee,
                                                               full, out_depth_dev, (const WT *)c->w.embed, g.d_model, c->pb.hidden);
    embed_rows_k<WT><<<n, 256, 0, c->stream>>>(lower, io.state, nullptr, (const WT *)c->w.embed, g.d_model, c->pb.hidden);
  }
  HIP_TRY(c, hipGetLastError());
  // a single row that runs full depth and completes no other is the same row above the exit layer: one run of layers
  const int first_run = n == 1 && n_upper == 1 ? g.n_layers : g.exit_layer;
  if ((rc = run_layers<WT>(c, 0, first_run, lower, n))) return rc;
  if (n_ee && (rc = run_lens_head<WT>(c, ee, n_ee))) return rc;
  if (n_full) {
    if ((rc = run_layers<WT>(c, first_run, g.n_layers, upper, n_upper))) return rc;
    if ((rc = run_final_head<WT>(c, full, n_full))) return rc;
  }
  if (rand_dev && c->temperature > 0.f) {   // the drawn token takes the arg-max's place
    if ((rc = prof_begin(c, SPARK_KC_SAMPLE))) return rc;
    const dim3 grid((c->dv.V + SAMPLE_CHUNK - 1) / SAMPLE_CHUNK, n);
    float *logits = at<float>(c, c->lo.logits);
    unsigned *masses = at<unsigned>(c, c->lo.sample_q);
    unsigned long long *class_mass = at<unsigned long long>(c, c->lo.sample_hist);
    u64 *cand = at<u64>(c, c->lo.sample_cand);
    unsigned *count = at<unsigned>(c, c->lo.sample_count), *arrive = at<unsigned>(c, c->lo.sample_arrive);
    if (grid.x == 1) {
      sample_pick_k<true><<<grid, SAMPLE_THREADS, 0, c->stream>>>(logits, c->dv.V, (double)c->temperature, (double)c->top_p, rand_dev, masses,
                                                                 class_mass, cand, count, arrive, best);
    } else {
      sample_mass_k<<<grid, SAMPLE_THREADS, 0, c->stream>>>(logits, c->dv.V, (double)c->temperature, masses, class_mass, best);
      sample_pick_k<false><<<grid, SAMPLE_THREADS, 0, c->stream>>>(logits, c->dv.V, (double)c->temperature, (double)c->top_p, rand_dev, masses,
                                                                  class_mass, cand, count, arrive, best);
    }
    if ((rc = prof_end(c, SPARK_KC_SAMPLE))) return rc;
  }
  return SPARK_OK;
}

// Copies of the pending rows of a call's sequences lie in the slots of prompt rows, which no step uses, `pending` places
// (the most that one has) for each
float *kept_rows(spark_ctx *c) { return c->base.hidden + (size_t)c->cfg.max_batch * c->dv.rmax * c->cfg.d_model; }

// grid (pending, sequences); back: from the copies to the sequences' slots
__global__ void __launch_bounds__(256) copy_pending_k(const int *seq_ids, const int *state, int rmax, int d, float *hidden, float *kept, bool back) {
  const int seq = seq_ids[blockIdx.y], r = blockIdx.x;
  if (r >= state[seq * ST_WORDS + ST_NPENDING]) return;
  float *slot = hidden + (size_t)(seq * rmax + r) * d, *copy = kept + (size_t)(blockIdx.y * gridDim.x + r) * d;
  for (int k = threadIdx.x * 4; k < d; k += 256 * 4) *(float4 *)((back ? slot : copy) + k) = *(const float4 *)((back ? copy : slot) + k);
}

// Where the words that the phases of such a launch hand over lie: in the MLP activations of the other path, and in
// what it keeps from the queries to the attention partials
struct SmallWords { size_t act, x, end_a, qkv, attn, u, end_b; };
SmallWords small_words(const spark_config &g, int n, int rows) {
  const size_t qw = (size_t)g.n_q_heads * g.head_dim, kvw = (size_t)g.n_kv_heads * g.head_dim, dm = g.d_model;
  SmallWords w;
  w.act = 0;
  w.x = w.act + (size_t)rows * g.d_ffn;
  w.end_a = w.x + (size_t)(n + rows) * dm;
  w.qkv = 0;
  w.attn = w.qkv + (size_t)rows * (qw + 2 * kvw);
  w.u = w.attn + (size_t)rows * qw;
  w.end_b = w.u + (size_t)n * dm;
  return w;
}

size_t layer_bytes_fp32(const spark_config &g) {
  const size_t qw = (size_t)g.n_q_heads * g.head_dim, kvw = (size_t)g.n_kv_heads * g.head_dim, dm = g.d_model;
  return sizeof(float) * ((qw + 2 * kvw) * dm + dm * qw + 3 * (size_t)g.d_ffn * dm);
}

// Whether the steps of a model can run in one launch, whatever the call.  Every workgroup has a task of every
// projection of a layer: that it has written its part of a row then says that it no longer reads what the row was made of.
bool shape_allows_small(const spark_config &g, const Derived &d, const Layout &lo) {
  const size_t qw = (size_t)g.n_q_heads * g.head_dim, kvw = (size_t)g.n_kv_heads * g.head_dim, dm = g.d_model;
  const int half_d = g.d_model / 2, wide = SMALL_CHUNK * SMALL_MAX_CHUNKS;
  const SmallWords w = small_words(g, SMALL_SEQS, SMALL_ROWS);
  return g.dtype == SPARK_DTYPE_FP32 && g.d_model <= SMALL_NORM_CHUNKS * SMALL_CHUNK && (int)qw <= wide && g.d_ffn <= wide && d.V <= 65536 &&
         half_d >= SMALL_WGS && g.d_ffn >= SMALL_WGS &&
         layer_bytes_fp32(g) <= SMALL_LAYER_BYTES &&
         sizeof(float) * (size_t)d.V * dm <= SMALL_LAYER_BYTES &&
         small_phase(g.d_model, (int)(qw + 2 * kvw) / 2).tile > 0 && small_phase((int)qw, half_d).tile > 0 &&
         small_phase(g.d_model, g.d_ffn).tile > 0 && small_phase(g.d_ffn, half_d).tile > 0 && small_phase(g.d_model, (d.V + 1) / 2).tile > 0 &&
         sizeof(u64) * w.end_a <= lo.mfma_part - lo.act && sizeof(u64) * w.end_b <= lo.lens_u - lo.qbuf;
}

// Whether a call's steps are better in one launch: rows of the largest pass, positions of the longest context.
// The launch has an eighth of the chip, so it loses what it gains where there is much to do: the sums (rows times the
// layer's weights) and the attention tasks of a workgroup (rows times query heads over SMALL_WGS) times the context.
// Measured, us a step, one launch / a launch per operation, layers of 3.9 and of 8.1 MB, with the sum below:
//   3.9 MB  1 sequence 42.9 / 83.1 (0.1), 8: 72.5 / 123.4 (0.6), 16: 115 / 159 (1.1), 1 of 900 tokens 81 / 95 (0.3), 8 of 900 123 / 147 (1.4)
//   8.1 MB  1 sequence 49.5 / 84.9 (0.1), 8: 106 / 132 (1.1), 4 of 900 121 / 138 (1.4), 8 of 400 153 / 146 (1.9), 16: 184 / 168 (2.2), 8 of 900 209 / 155 (2.8)
bool small_steps_pay(const spark_ctx *c, int n, int rows, int positions) {
  if (!c->small_ok || !c->use_small || !c->may_wait || c->prof_class >= 0 || n > SMALL_SEQS || rows > SMALL_ROWS || positions > SMALL_CTX) return false;
  const int rounds = (rows * c->cfg.n_q_heads + SMALL_WGS - 1) / SMALL_WGS;
  return rows * (double)c->small_layer_bytes / (double)(256u << 20) + rounds * (double)positions / 4096.0 <= 1.5;
}

// all steps of a call in one launch; rows: of the largest pass; pending: of a sequence as the call begins, at most.
// false: refused (as in enqueue_one_row; a call took 39 ms instead of 1)
bool enqueue_small_steps(spark_ctx *c, int steps, int n, int rows, int pending, bool forced, bool sampled) {
  const spark_config &g = c->cfg;
  SmallSteps a;
  a.sp = c->sp;
  a.d = g.d_model; a.nq = g.n_q_heads; a.nkv = g.n_kv_heads; a.F = g.d_ffn; a.V = c->dv.V; a.eps = g.rms_eps;
  const int qw = g.n_q_heads * g.head_dim, half_d = g.d_model / 2;
  a.qkv = small_phase(g.d_model, (g.n_q_heads + 2 * g.n_kv_heads) * (g.head_dim / 2));
  a.o = small_phase(qw, half_d); a.gateup = small_phase(g.d_model, g.d_ffn); a.down = small_phase(g.d_ffn, half_d);
  a.lens = small_phase(g.d_model, half_d); a.vocab = small_phase(g.d_model, (c->dv.V + 1) / 2);
  auto f = [](const void *p) { return (const float *)p; };
  a.embed = f(c->w.embed); a.attn_norm = c->w.attn_norm; a.wq = f(c->w.wq); a.wk = f(c->w.wk); a.wv = f(c->w.wv); a.wo = f(c->w.wo);
  a.mlp_norm = c->w.mlp_norm; a.wg = f(c->w.wg); a.wu = f(c->w.wu); a.wd = f(c->w.wd); a.final_norm = c->w.final_norm;
  a.lm_head = f(c->w.lm_head); a.lens_a = f(c->w.lens_a); a.lens_b = c->w.lens_b; a.lens_norm = c->w.lens_norm; a.lens_head = f(c->w.lens_head);
  a.rope = at<float2>(c, c->lo.rope);
  a.kv = kv_view(c);
  a.hidden = c->pb.hidden; a.logits = at<float>(c, c->lo.logits);
  const SmallWords w = small_words(g, n, rows);
  a.words_a = at<u64>(c, c->lo.act); a.words_b = at<u64>(c, c->lo.qbuf);
  a.count_a = (int)w.end_a; a.count_b = (int)w.end_b;
  a.act_words = a.words_a + w.act; a.x_words = a.words_a + w.x;
  a.qkv_words = a.words_b + w.qkv; a.attn_words = a.words_b + w.attn; a.u_words = a.words_b + w.u;
  a.wg_best = at<u64>(c, c->lo.sample_cand);   // (the sampler of a vocabulary this small keeps no list there)
  a.plan = at<int>(c, c->lo.plan);
  a.flags = (unsigned *)(a.plan + SMALL_FLAGS_AT);
  a.state = at<int>(c, c->lo.state); a.seq_ids = at<int>(c, c->lo.seq_ids);
  a.forced = forced ? at<int>(c, c->lo.forced) : nullptr;
  a.words = sampled ? at<u64>(c, c->lo.rand_words) : nullptr;
  a.best = at<u64>(c, c->lo.best);
  a.out_tokens = at<int>(c, c->lo.out_tokens); a.out_depth = at<int>(c, c->lo.out_depth);
  a.n = n; a.steps = steps;
  a.temperature = c->temperature; a.top_p = c->top_p;
  a.epoch = ++c->small_epoch;
  a.max_polls = c->wait_polls ? std::abs(c->wait_polls) : SMALL_MAX_POLLS;
  a.first_polls = c->wait_polls < 0 ? a.max_polls : SMALL_MAX_POLLS;
  a.kept = kept_rows(c); a.kept_rows = pending;
  if (launch_small_steps(a, g.head_dim, c->stream) == hipSuccess) return true;
  (void)hipGetLastError();
  c->use_small = false;
  return false;
}

// A launch whose workgroups wait for each other has given up: the call runs again, and this context keeps to launches per
// operation from then on.
int stop_waiting(spark_ctx *c) {
  c->use_small = false;
  c->use_row = 0;
  c->row_words_clean = false;
  snprintf(c->err, sizeof(c->err), "a launch whose workgroups wait for each other gave up; the call ran again as launches per operation");
  HIP_TRY(c, hipMemsetAsync(at<int>(c, c->lo.plan) + PL_ERR, 0, sizeof(int), c->stream));
  return SPARK_OK;
}

// The call's sequences as they were before it, on the device (their counters from the host's mirror, their pending rows from
// the copies), for another run of it
int begin_again(spark_ctx *c, int n, const int32_t *seq_ids, int pending) {
  if (int rc = stop_waiting(c)) return rc;
  for (int i = 0; i < n; ++i) {
    const Seq &s = c->seqs[seq_ids[i]];
    int st[ST_WORDS];
    st[ST_LEN] = s.len; st[ST_G] = s.g; st[ST_JSTREAM] = s.j_stream; st[ST_NPENDING] = s.n_pending; st[ST_OFFSET] = s.cycle_offset;
    st[ST_NEXT] = s.next; st[ST_ACTIVE] = 1; st[ST_LASTFULL] = s.last_full; st[ST_TEXTBUDGET] = s.text_budget; st[ST_PHASE] = s.phase;
    HIP_TRY(c, hipMemcpyAsync(at<int>(c, c->lo.state) + (size_t)seq_ids[i] * ST_WORDS, st, sizeof(st), hipMemcpyHostToDevice, c->stream));
    HIP_TRY(c, hipStreamSynchronize(c->stream));   // (`st` has been read)
  }
  if (pending) {
    copy_pending_k<<<dim3(pending, n), 256, 0, c->stream>>>(at<int>(c, c->lo.seq_ids), at<int>(c, c->lo.state), c->dv.rmax, c->cfg.d_model,
                                                            c->base.hidden, kept_rows(c), true);
    HIP_TRY(c, hipGetLastError());
  }
  return SPARK_OK;
}

int decode_chunk(spark_ctx *c, int steps, int n, const int32_t *seq_ids, const int32_t *forced,
                 const uint64_t *rand_words, int32_t *out_tokens, int32_t *out_depth) {
  const spark_config &g = c->cfg;
  int rc;
  // validation and page reservation
  for (int i = 0; i < n; ++i) {
    Seq *s = find_seq(c, seq_ids[i]);
    if (!s) return fail(c, SPARK_ENOSEQ, "unknown sequence id %d", seq_ids[i]);
    if (!s->prefilled) return fail(c, SPARK_ESTATE, "sequence %d stepped before prefill", seq_ids[i]);
    for (int k = 0; k < i; ++k)
      if (seq_ids[k] == seq_ids[i]) return fail(c, SPARK_EINVAL, "sequence %d listed twice", seq_ids[i]);
    if (s->len + steps > g.max_seq_len)
      return fail(c, SPARK_ENOMEM, "sequence %d would exceed max_seq_len", seq_ids[i]);
    if (forced)
      for (int st = 0; st < steps; ++st)
        if (forced[st * n + i] >= c->dv.V) return fail(c, SPARK_EINVAL, "forced id out of range");
  }
  // the schedule of the whole call, before anything is enqueued: the pending rows and the current
  // row of a sequence must fit its slots of the hidden-state arena at every step
  for (int i = 0; i < n; ++i) {
    const Seq &sq = c->seqs[seq_ids[i]];
    int gg = sq.g, jj = sq.j_stream, npend = sq.n_pending;
    for (int st = 0; st < steps; ++st) {
      int is_text, full;
      schedule_decide(c->sp, gg, sq.cycle_offset, jj, sq.text_budget, sq.phase, is_text, full);
      npend = full ? 0 : npend + 1;
      if (npend + 1 > c->dv.rmax)
        return fail(c, SPARK_ESTATE, "sequence %d would hold %d pending positions, its slots hold %d",
                    seq_ids[i], npend, c->dv.rmax - 1);
      ++gg;
      if (!is_text) ++jj;
    }
  }
  for (int i = 0; i < n; ++i)
    if ((rc = ensure_pages(c, seq_ids[i], c->seqs[seq_ids[i]].len + steps))) return rc;

  // inputs
  int *h_ids = c->h_in, *h_forced = c->h_in + g.max_batch;
  memcpy(h_ids, seq_ids, sizeof(int) * n);
  c->last_ids.assign(seq_ids, seq_ids + n);   // (for spark_get_logits)
  HIP_TRY(c, hipMemcpyAsync(at<int>(c, c->lo.seq_ids), h_ids, sizeof(int) * n, hipMemcpyHostToDevice,
                            c->stream));
  if (forced) {
    memcpy(h_forced, forced, sizeof(int) * (size_t)steps * n);
    HIP_TRY(c, hipMemcpyAsync(at<int>(c, c->lo.forced), h_forced, sizeof(int) * (size_t)steps * n,
                              hipMemcpyHostToDevice, c->stream));
  }

  if (rand_words)   // (pageable source: the copy has completed on return)
    HIP_TRY(c, hipMemcpyAsync(at<unsigned long long>(c, c->lo.rand_words), rand_words,
                              sizeof(uint64_t) * (size_t)steps * n, hipMemcpyHostToDevice, c->stream));

  // host mirror of the schedule: decides the launch shapes, checked against the device's depths
  struct Mirror { int g, j, npend, len; };
  std::vector<Mirror> mir(n);
  for (int i = 0; i < n; ++i) {
    Seq &s = c->seqs[seq_ids[i]];
    mir[i] = Mirror{s.g, s.j_stream, s.n_pending, s.len};
  }
  std::vector<int> want_depth((size_t)steps * n), want_text((size_t)steps * n),
      want_rows((size_t)steps * n);
  struct Shape { int n_upper, n_ee, n_full, max_pos; };
  std::vector<Shape> shapes(steps);
  int most_rows = 0;
  for (int st = 0; st < steps; ++st) {
    Shape &sh = shapes[st];
    sh = Shape{0, 0, 0, 0};
    for (int i = 0; i < n; ++i) sh.max_pos = std::max(sh.max_pos, mir[i].len);   // position of the new row
    for (int i = 0; i < n; ++i) {
      int is_text, full;
      const Seq &sq = c->seqs[seq_ids[i]];
      schedule_decide(c->sp, mir[i].g, sq.cycle_offset, mir[i].j, sq.text_budget, sq.phase, is_text, full);
      want_depth[st * n + i] = full ? g.n_layers : g.exit_layer;
      want_text[st * n + i] = is_text;
      want_rows[st * n + i] = full ? mir[i].npend + 1 : 0;
      if (full) { sh.n_upper += mir[i].npend + 1; ++sh.n_full; mir[i].npend = 0; }
      else { ++sh.n_ee; mir[i].npend += 1; }
      mir[i].g += 1;
      if (!is_text) mir[i].j += 1;
      mir[i].len += 1;
    }
    most_rows = std::max(most_rows, sh.n_upper);
  }
  const bool sampled = rand_words && c->temperature > 0.f;
  int pending = 0, copied = 0;   // rows of a sequence as the call begins, at most; and of those that have copies
  for (int i = 0; i < n; ++i) pending = std::max(pending, c->seqs[seq_ids[i]].n_pending);
  // Only a full-depth step writes pending rows, and only a pass of one row may give up.  (Copies for every call, us a call of
  // one step, seven layers of the Step shape: a batch of eight 948 in place of 939, one sequence 539 in place of 534.)
  bool one_row = false;
  for (const Shape &sh : shapes) one_row = one_row || n == 1 || sh.n_upper == 1;
  one_row = one_row && c->row_ok && (c->use_row == 2 || one_row_pays(c->layer_bytes, g.n_layers));
  auto enqueue = [&]() -> int {
    if (small_steps_pay(c, n, std::max(n, most_rows), shapes[steps - 1].max_pos + 1) && (!sampled || c->dv.V <= SAMPLE_CHUNK) &&
        enqueue_small_steps(c, steps, n, std::max(n, most_rows), pending, forced != nullptr, sampled)) {
      copied = pending;
      return SPARK_OK;
    }
    if (pending && most_rows && one_row && c->use_row && c->may_wait) {
      copy_pending_k<<<dim3(pending, n), 256, 0, c->stream>>>(at<int>(c, c->lo.seq_ids), at<int>(c, c->lo.state), c->dv.rmax, g.d_model,
                                                              c->base.hidden, kept_rows(c), false);
      HIP_TRY(c, hipGetLastError());
      copied = pending;
    }
    for (int st = 0; st < steps; ++st) {
      const Shape &sh = shapes[st];
      c->attn_splits_now = sh.max_pos / ATTN_SLICE + 1;
      const int *pf = forced && st ? at<int>(c, c->lo.forced) + (size_t)(st - 1) * n : nullptr;
      int *pt = st ? at<int>(c, c->lo.out_tokens) + (size_t)(st - 1) * n : nullptr;
      int *od = at<int>(c, c->lo.out_depth) + (size_t)st * n;
      const unsigned long long *rw =
          rand_words ? at<unsigned long long>(c, c->lo.rand_words) + (size_t)st * n : nullptr;
      const int e = g.dtype == SPARK_DTYPE_BF16 ? enqueue_step<bf16_t>(c, n, sh.n_upper, sh.n_ee, sh.n_full, pf, pt, rw, od)
                                                : enqueue_step<float>(c, n, sh.n_upper, sh.n_ee, sh.n_full, pf, pt, rw, od);
      if (e) return e;
    }
    emit_k<<<1, SCHED_THREADS, 0, c->stream>>>(step_io(c, n), forced ? at<int>(c, c->lo.forced) + (size_t)(steps - 1) * n : nullptr,
                                              at<int>(c, c->lo.out_tokens) + (size_t)(steps - 1) * n);
    HIP_TRY(c, hipGetLastError());
    return SPARK_OK;
  };

  const size_t cnt = (size_t)steps * n;
  int *h_tok = c->h_out, *h_dep = c->h_out + (size_t)MAX_STEPS_PER_CALL * g.max_batch;
  int *h_plan = h_dep + (size_t)MAX_STEPS_PER_CALL * g.max_batch;
  auto run = [&]() -> int {   // and its results
    if (int e = enqueue()) return e;
    HIP_TRY(c, hipMemcpyAsync(h_tok, at<int>(c, c->lo.out_tokens), sizeof(int) * cnt,
                              hipMemcpyDeviceToHost, c->stream));
    HIP_TRY(c, hipMemcpyAsync(h_dep, at<int>(c, c->lo.out_depth), sizeof(int) * cnt,
                              hipMemcpyDeviceToHost, c->stream));
    HIP_TRY(c, hipMemcpyAsync(h_plan, at<int>(c, c->lo.plan), sizeof(int) * PL_WORDS,
                              hipMemcpyDeviceToHost, c->stream));
    HIP_TRY(c, hipStreamSynchronize(c->stream));
    return SPARK_OK;
  };
  c->may_wait = n * pending <= PREFILL_CHUNK;   // (the copies have their places)
  rc = run();
  c->may_wait = true;
  if (rc) return rc;
  if (h_plan[PL_ERR] & ERR_STALLED) {
    if ((rc = begin_again(c, n, seq_ids, copied)) || (rc = run())) return rc;
  }
  memcpy(out_tokens, h_tok, sizeof(int) * cnt);
  memcpy(out_depth, h_dep, sizeof(int) * cnt);

  // commit the mirror and the exit-layer log
  for (int st = 0; st < steps; ++st)
    for (int i = 0; i < n; ++i) {
      Seq &s = c->seqs[seq_ids[i]];
      const size_t k = (size_t)st * n + i;
      if (h_dep[k] != want_depth[k])
        return fail(c, SPARK_ESTATE, "device schedule (%d) and host mirror (%d) disagree", h_dep[k],
                    want_depth[k]);
      if (want_rows[k]) {
        s.flush_rows[want_rows[k]] += 1;
        if (want_text[k]) s.text_steps += 1; else s.speech_full += 1;
      } else if (want_text[k]) {
        s.text_ee += 1;
      } else {
        s.speech_ee += 1;
      }
      s.last_full = want_rows[k] != 0;
    }
  for (int i = 0; i < n; ++i) {
    Seq &s = c->seqs[seq_ids[i]];
    s.g = mir[i].g; s.j_stream = mir[i].j; s.n_pending = mir[i].npend; s.len = mir[i].len;
    const size_t k = (size_t)(steps - 1) * n + i;
    s.next = forced && forced[k] >= 0 ? forced[k] : h_tok[k];
  }
  if (h_plan[PL_ERR]) {
    int e = h_plan[PL_ERR];
    int zero = 0;  // error path only: clear the flag so that the context stays usable
    (void)hipMemcpy(at<int>(c, c->lo.plan) + PL_ERR, &zero, sizeof(int), hipMemcpyHostToDevice);
    if (e & ERR_NAN) return fail(c, SPARK_ENAN, "a head produced a NaN logit");
    return fail(c, SPARK_ESTATE, "device saw an inactive sequence");
  }
  return SPARK_OK;
}

template <typename WT> int prefill_rows(spark_ctx *c, int id, const int32_t *prompt, int n_rows) {
  const spark_config &g = c->cfg;
  // A large pass has its own buffers; one in the base buffers takes the slots behind the sequences'.
  // Passes are of equal size, in whole tiles of rows, unless their size has been set.
  const bool large = c->prompt.rows > 0 && c->use_tiled && c->use_mfma &&
                     (c->prefill_chunk > 0 ? c->prefill_chunk > PREFILL_CHUNK : n_rows > c->prefill_base);
  int chunk = c->prefill_chunk > 0 ? std::min(c->prefill_chunk, large ? PROMPT_ROWS : PREFILL_CHUNK) : c->prefill_base;
  if (large && c->prefill_chunk == 0) {
    const int passes = (n_rows + PROMPT_ROWS - 1) / PROMPT_ROWS;
    chunk = std::min(PROMPT_ROWS, (int)align_up((n_rows + passes - 1) / passes, 128));
  }
  const int base_slot = large ? 0 : g.max_batch * c->dv.rmax;
  std::vector<RowDesc> rows(chunk);
  int rc = SPARK_OK;
  if (large) c->pb = c->prompt;
  RowDesc *rows_dev = c->pb.descs;
  int *tok_dev = c->pb.tokens;
  c->prompt_pass = true;
  for (int p0 = 0; p0 < n_rows && rc == SPARK_OK; p0 += chunk) {
    const int m = std::min(chunk, n_rows - p0);
    for (int r = 0; r < m; ++r) rows[r] = RowDesc{base_slot + r, id, p0 + r, -1};
    auto pass = [&]() {
      HIP_TRY(c, hipMemcpyAsync(rows_dev, rows.data(), sizeof(RowDesc) * m, hipMemcpyHostToDevice, c->stream));
      HIP_TRY(c, hipMemcpyAsync(tok_dev, prompt + p0, sizeof(int) * m, hipMemcpyHostToDevice, c->stream));
      embed_rows_k<WT><<<m, 256, 0, c->stream>>>(rows_dev, nullptr, tok_dev, (const WT *)c->w.embed, g.d_model, c->pb.hidden);
      HIP_TRY(c, hipGetLastError());
      c->attn_splits_now = (p0 + m - 1) / ATTN_SLICE + 1;
      c->row_taken = false;
      if (int e = run_layers<WT>(c, 0, g.n_layers, rows_dev, m)) return e;
      if (c->row_taken)
        HIP_TRY(c, hipMemcpyAsync(c->h_out, at<int>(c, c->lo.plan) + PL_ERR, sizeof(int), hipMemcpyDeviceToHost, c->stream));
      HIP_TRY(c, hipStreamSynchronize(c->stream));
      return SPARK_OK;
    };
    rc = pass();
    // (a pass begins with the embedding, and writes every hidden value and cache entry that it has: it can simply run again)
    if (rc == SPARK_OK && c->row_taken && (*c->h_out & ERR_STALLED) && (rc = stop_waiting(c)) == SPARK_OK) rc = pass();
  }
  c->pb = c->base;
  c->prompt_pass = false;
  return rc;
}

}  // namespace

extern "C" {

int spark_workspace_bytes(const spark_config *cfg, size_t *kv_pool_bytes, size_t *scratch_bytes) {
  char why[128];
  if (!cfg || !config_ok(cfg, why, sizeof(why))) return SPARK_EINVAL;
  Derived d;
  Layout l;
  derive(*cfg, d);
  layout(*cfg, d, l);
  if (kv_pool_bytes) *kv_pool_bytes = d.kv_pool_bytes;
  if (scratch_bytes) *scratch_bytes = l.total_prompt;
  return SPARK_OK;
}

int spark_schedule_preview(const spark_config *cfg, int32_t cycle_offset, int32_t text_budget,
                           int32_t n_steps, int32_t *depth_out, int32_t *is_text_out) {
  char why[128];
  if (!cfg || !config_ok(cfg, why, sizeof(why)) || cycle_offset < 0 || n_steps < 0 || !depth_out ||
      !is_text_out || (text_budget > 0 && cfg->n_text < 1))
    return SPARK_EINVAL;
  const SchedParams sp = sched_params(cfg);
  int j_stream = 0;
  for (int g = 0; g < n_steps; ++g) {
    int is_text, full;
    schedule_decide(sp, g, cycle_offset, j_stream, text_budget, sp.phase, is_text, full);   // the function the device runs
    depth_out[g] = full ? cfg->n_layers : cfg->exit_layer;
    is_text_out[g] = is_text;
    if (!is_text) ++j_stream;
  }
  return SPARK_OK;
}

namespace {

// What spark_init and spark_init_static share.  `pinned`: the staging buffers for ids, forced tokens
// and results are pinned host memory (hipHostMalloc); otherwise they are ordinary host arrays.
int init_context(const spark_config *cfg, const spark_weights *weights, void *kv_pool, size_t kv_pool_bytes,
                 void *scratch, size_t scratch_bytes, void *hip_stream, bool static_scratch, spark_ctx **out) {
  spark_ctx *c = new spark_ctx();
  c->cfg = *cfg;
  c->w = *weights;
  c->err[0] = 0;
  derive(*cfg, c->dv);
  layout(*cfg, c->dv, c->lo);
  if (!kv_pool || !scratch || kv_pool_bytes < c->dv.kv_pool_bytes || scratch_bytes < c->lo.total ||
      ((uintptr_t)kv_pool & 255) || ((uintptr_t)scratch & 255)) {
    delete c;
    return SPARK_ENOMEM;
  }
  c->stream = (hipStream_t)hip_stream;
  c->scratch = (char *)scratch;
  c->kv_pool = kv_pool;
  c->static_scratch = static_scratch;
  c->sp = sched_params(cfg);
  c->seqs.resize(cfg->max_batch);
  c->last_ids.reserve(cfg->max_batch);
  for (int p = c->dv.n_pages_total - 1; p >= 0; --p) c->free_pages.push_back(p);
  c->h_in = c->h_out = nullptr;
  auto bail = [&](int code) { spark_destroy(c); return code; };
  int dev = 0;
  hipDeviceProp_t prop;
  if (hipGetDevice(&dev) != hipSuccess || hipGetDeviceProperties(&prop, dev) != hipSuccess)
    return bail(SPARK_EHIP);
  c->device = dev;
  c->n_cu = prop.multiProcessorCount;
  // the MFMA kernels load 16-byte vectors of 8 weights; other widths stay on the vector kernel
  c->mfma_ok = cfg->d_model % 8 == 0 && (cfg->n_q_heads * cfg->head_dim) % 8 == 0 && cfg->d_ffn % 8 == 0;
  c->use_mfma = c->mfma_ok;
  int cooperative = 0;
  if (hipDeviceGetAttribute(&cooperative, hipDeviceAttributeCooperativeLaunch, dev) != hipSuccess) cooperative = 0;
  c->small_ok = shape_allows_small(*cfg, c->dv, c->lo) && cooperative &&
                prop.multiProcessorCount >= SMALL_WGS && small_steps_fit(cfg->head_dim);
  c->small_layer_bytes = layer_bytes_fp32(*cfg);
  c->layer_bytes = layer_bytes_fp32(*cfg) / 2;
  c->row_ok = shape_allows_one_row(*cfg) && cooperative && prop.multiProcessorCount >= ROW_WGS && one_row_fit();
  // a scratch area of the full size holds the MFMA-ordered copy of the projection weights (the
  // static area never does)
  tiled_map(*cfg, c->dv, c->tm);
  c->has_tiled = !static_scratch && c->tm.total > 0 && scratch_bytes >= c->lo.total_tiled;
  const Layout &lo = c->lo;
  c->base = PassBuffers{at<float>(c, lo.hidden), at<float>(c, lo.qbuf), at<float>(c, lo.attn_out), at<float>(c, lo.act),
                        at<float>(c, lo.xnorm), at<unsigned long long>(c, lo.row_ssq), at<uint8_t>(c, lo.max_x),
                        at<uint8_t>(c, lo.max_attn), at<uint8_t>(c, lo.max_act),
                        at<RowDesc>(c, lo.prefill_rows), at<int>(c, lo.prefill_tokens), c->dv.max_rows};
  c->prompt = PassBuffers{at<float>(c, lo.prompt_hidden), at<float>(c, lo.prompt_q), at<float>(c, lo.prompt_attn),
                          at<float>(c, lo.prompt_act), at<float>(c, lo.prompt_xnorm), at<unsigned long long>(c, lo.prompt_ssq),
                          at<uint8_t>(c, lo.prompt_max_x), at<uint8_t>(c, lo.prompt_max_attn), at<uint8_t>(c, lo.prompt_max_act),
                          at<RowDesc>(c, lo.prompt_rows), at<int>(c, lo.prompt_tokens),
                          c->has_tiled && scratch_bytes >= lo.total_prompt ? PROMPT_ROWS : 0};
  c->pb = c->base;
  // Prompt rows per pass: on the MFMA path the widest projection (gate/up) is cut into tiles of 256
  // weight-row pairs x 64 prompt rows; the row count is chosen so that one round of tiles about
  // fills the chip, which needs no k split and no second kernel for that projection.
  if (c->use_mfma && cfg->dtype == SPARK_DTYPE_BF16) {
    const int x_tiles = (cfg->d_ffn + MG_TASKS_PER_BLOCK - 1) / MG_TASKS_PER_BLOCK;
    c->prefill_base = std::max(128, std::min(PREFILL_CHUNK, 64 * (c->n_cu / std::max(1, x_tiles))));
  }
  size_t in_ints = (size_t)cfg->max_batch * (1 + MAX_STEPS_PER_CALL);
  size_t out_ints = (size_t)cfg->max_batch * 2 * MAX_STEPS_PER_CALL + PL_WORDS;
  if (static_scratch) {   // this variant allocates nothing through the HIP runtime
    c->h_in = new (std::nothrow) int[in_ints];
    c->h_out = new (std::nothrow) int[out_ints];
    if (!c->h_in || !c->h_out) return bail(SPARK_ENOMEM);
  } else if (hipHostMalloc((void **)&c->h_in, sizeof(int) * in_ints, hipHostMallocDefault) != hipSuccess ||
             hipHostMalloc((void **)&c->h_out, sizeof(int) * out_ints, hipHostMallocDefault) != hipSuccess) {
    return bail(SPARK_EHIP);
  }
  // device state, rotary table.  Everything up to the hidden-state arena starts at zero: sequence
  // state, page table, plan and error word, and the counters that kernels hand to the next launch
  // at zero (attention arrivals, the sampler's histogram, arrivals and candidate counts).  The
  // scratch area may hold another context's leftovers (the static array always does).
  if (hipMemsetAsync(c->scratch + c->lo.state, 0, c->lo.hidden - c->lo.state, c->stream) != hipSuccess)
    return bail(SPARK_EHIP);
  const int half = cfg->head_dim / 2;
  std::vector<float> inv(half);
  for (int i = 0; i < half; ++i)
    inv[i] = (float)pow((double)cfg->rope_base, -2.0 * i / (double)cfg->head_dim);
  if (hipMemcpyAsync(c->scratch + c->lo.inv_freq, inv.data(), sizeof(float) * half,
                     hipMemcpyHostToDevice, c->stream) != hipSuccess)
    return bail(SPARK_EHIP);
  int total = half * cfg->max_seq_len;
  rope_table_k<<<(total + 255) / 256, 256, 0, c->stream>>>(at<float>(c, c->lo.inv_freq), half,
                                                          cfg->max_seq_len, at<float2>(c, c->lo.rope));
  if (hipGetLastError() != hipSuccess || hipStreamSynchronize(c->stream) != hipSuccess)
    return bail(SPARK_EHIP);
  if (c->has_tiled && build_tiled(c) != SPARK_OK) return bail(SPARK_EHIP);
  *out = c;
  return SPARK_OK;
}

bool init_args_ok(const spark_config *cfg, const spark_weights *weights) {
  char why[128];
  if (!cfg || !weights || !config_ok(cfg, why, sizeof(why))) return false;
  const void *const *wp = (const void *const *)weights;
  for (size_t i = 0; i < sizeof(spark_weights) / sizeof(void *); ++i)
    if (!wp[i]) return false;
  return true;
}

}  // namespace

// The scratch area of spark_init_static: one array per GPU the library is loaded on, held until the
// process ends.  In host code the name `static_scratch_area` is a handle for hipGetSymbolAddress,
// not an address: the per-device address is looked up once and kept in static_scratch_ptr.
static __device__ __align__(256) unsigned char static_scratch_area[SPARK_STATIC_SCRATCH_BYTES];

namespace {
constexpr int MAX_DEVICES = 64;
char *static_scratch_ptr[MAX_DEVICES] = {nullptr};
bool static_scratch_busy[MAX_DEVICES] = {false};
}  // namespace

int spark_init(const spark_config *cfg, const spark_weights *weights, void *kv_pool,
               size_t kv_pool_bytes, void *scratch, size_t scratch_bytes, void *hip_stream,
               spark_ctx **out) {
  if (!out) return SPARK_EINVAL;
  *out = nullptr;
  if (!init_args_ok(cfg, weights)) return SPARK_EINVAL;
  return init_context(cfg, weights, kv_pool, kv_pool_bytes, scratch, scratch_bytes, hip_stream, false, out);
}

int spark_init_static(const spark_config *cfg, const spark_weights *weights, void *kv_pool,
                      size_t kv_pool_bytes, void *hip_stream, spark_ctx **out) {
  if (!out) return SPARK_EINVAL;
  *out = nullptr;
  if (!init_args_ok(cfg, weights)) return SPARK_EINVAL;
  Derived d;
  Layout l;
  derive(*cfg, d);
  layout(*cfg, d, l);
  if (l.total > (size_t)SPARK_STATIC_SCRATCH_BYTES) {
    fprintf(stderr, "spark_init_static: this configuration needs %zu bytes of scratch, the static area holds %zu\n",
            l.total, (size_t)SPARK_STATIC_SCRATCH_BYTES);
    return SPARK_ENOMEM;
  }
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= MAX_DEVICES) return SPARK_EHIP;
  if (static_scratch_busy[dev]) {
    fprintf(stderr, "spark_init_static: device %d already has a live context on the static scratch area\n", dev);
    return SPARK_ESTATE;
  }
  if (!static_scratch_ptr[dev]) {   // once per device, with that device current
    void *p = nullptr;
    if (hipGetSymbolAddress(&p, HIP_SYMBOL(static_scratch_area)) != hipSuccess || !p) return SPARK_EHIP;
    static_scratch_ptr[dev] = (char *)p;
  }
  int rc = init_context(cfg, weights, kv_pool, kv_pool_bytes, static_scratch_ptr[dev],
                        (size_t)SPARK_STATIC_SCRATCH_BYTES, hip_stream, true, out);
  if (rc == SPARK_OK) static_scratch_busy[dev] = true;
  return rc;
}

int spark_tune(spark_ctx *c, const char *name, int32_t value) {
  if (!c || !name) return SPARK_EINVAL;
  const std::string k(name);
  if (k == "mfma") c->use_mfma = value != 0 && c->mfma_ok;
  else if (k == "mfma_min_rows") c->mfma_min_rows = std::max(1, (int)value);
  else if (k == "mfma_small_tiles") c->mfma_small_tiles = value;
  else if (k == "mfma_xcd_max_split") c->mfma_xcd_max_split = value;
  else if (k == "attn_pieces") c->attn_pieces = std::max(0, std::min(10, (int)value));
  else if (k == "attn_mfma_min_rows") c->attn_mfma_min_rows = std::max(1, (int)value);
  else if (k == "gemv_big_kb") c->gemv_big_kb = std::max(1, (int)value);
  else if (k == "prefill_rows") c->prefill_chunk = value == 0 ? 0 : std::max(32, std::min(PROMPT_ROWS, (int)value / 32 * 32));
  else if (k == "mfma_small_max_k") c->mfma_small_max_k = std::max(8, (int)value);
  else if (k == "mfma_tiled") c->use_tiled = value != 0;
  else if (k == "tiled_row_blocks") c->tiled_row_blocks = std::max(2, std::min(4, (int)value));
  else if (k == "attn_prompt_min_rows") c->attn_prompt_min_rows = std::max(0, (int)value);
  else if (k == "direct_max_rows") c->direct_max_rows = value;
  else if (k == "direct_whole_k") c->direct_whole_k = value;
  else if (k == "small_steps") c->use_small = value != 0;
  else if (k == "one_row") c->use_row = std::max(0, std::min(2, (int)value));
  else if (k == "wait_polls") c->wait_polls = std::max(-SMALL_MAX_POLLS, (int)value);
  else if (k == "fuse_norm") c->fuse_norm = value != 0;
  else return fail(c, SPARK_EINVAL, "unknown tuning name '%s'", name);
  return SPARK_OK;
}

int spark_seq_open(spark_ctx *c, int32_t cycle_offset, int32_t *seq_id) {
  if (!c || !seq_id) return SPARK_EINVAL;
  if (cycle_offset < 0) return fail(c, SPARK_EINVAL, "cycle_offset < 0");
  for (int i = 0; i < (int)c->seqs.size(); ++i)
    if (!c->seqs[i].open) {
      c->seqs[i] = Seq();
      c->seqs[i].open = true;
      c->seqs[i].cycle_offset = cycle_offset % (c->cfg.n_text + c->cfg.n_speech);
      c->seqs[i].phase = c->cfg.phase;
      *seq_id = i;
      return SPARK_OK;
    }
  return fail(c, SPARK_ENOSEQ, "all %d sequence slots are open", (int)c->seqs.size());
}

int spark_prefill(spark_ctx *c, int32_t seq_id, const int32_t *prompt, int32_t n) {
  if (!c) return SPARK_EINVAL;
  Seq *s = find_seq(c, seq_id);
  if (!s) return fail(c, SPARK_ENOSEQ, "unknown sequence id %d", seq_id);
  if (s->prefilled) return fail(c, SPARK_ESTATE, "sequence %d already has a prompt", seq_id);
  if (!prompt || n < 1) return fail(c, SPARK_EINVAL, "empty prompt");
  if (n > c->cfg.max_seq_len) return fail(c, SPARK_ENOMEM, "prompt longer than max_seq_len");
  for (int i = 0; i < n; ++i)
    if (prompt[i] < 0 || prompt[i] >= c->dv.V) return fail(c, SPARK_EINVAL, "prompt id out of range");
  int rc = ensure_pages(c, seq_id, n - 1);
  if (rc) return rc;
  if (n > 1) {
    rc = c->cfg.dtype == SPARK_DTYPE_BF16 ? prefill_rows<bf16_t>(c, seq_id, prompt, n - 1)
                                          : prefill_rows<float>(c, seq_id, prompt, n - 1);
    if (rc) return rc;
  }
  int st[ST_WORDS] = {0};
  st[ST_LEN] = n - 1;
  st[ST_OFFSET] = s->cycle_offset;
  st[ST_NEXT] = prompt[n - 1];
  st[ST_ACTIVE] = 1;
  st[ST_TEXTBUDGET] = s->text_budget;
  st[ST_PHASE] = s->phase;
  HIP_TRY(c, hipMemcpyAsync(at<int>(c, c->lo.state) + (size_t)seq_id * ST_WORDS, st, sizeof(st),
                            hipMemcpyHostToDevice, c->stream));
  HIP_TRY(c, hipStreamSynchronize(c->stream));
  s->len = n - 1;
  s->next = prompt[n - 1];
  s->prefilled = true;
  return SPARK_OK;
}

int spark_decode_sampled(spark_ctx *c, int32_t n_steps, int32_t n, const int32_t *seq_ids,
                         const int32_t *forced_next, const uint64_t *rand_words,
                         int32_t *out_tokens, int32_t *out_depth) {
  if (!c) return SPARK_EINVAL;
  if (n < 1 || n > c->cfg.max_batch || n_steps < 1 || !seq_ids || !out_tokens || !out_depth)
    return fail(c, SPARK_EINVAL, "bad batch (n=%d, n_steps=%d)", n, n_steps);
  for (int s0 = 0; s0 < n_steps; s0 += MAX_STEPS_PER_CALL) {
    int steps = std::min(MAX_STEPS_PER_CALL, n_steps - s0);
    int rc = decode_chunk(c, steps, n, seq_ids, forced_next ? forced_next + (size_t)s0 * n : nullptr,
                          rand_words ? rand_words + (size_t)s0 * n : nullptr,
                          out_tokens + (size_t)s0 * n, out_depth + (size_t)s0 * n);
    if (rc) return rc;
  }
  return SPARK_OK;
}

int spark_decode(spark_ctx *c, int32_t n_steps, int32_t n, const int32_t *seq_ids,
                 const int32_t *forced_next, int32_t *out_tokens, int32_t *out_depth) {
  return spark_decode_sampled(c, n_steps, n, seq_ids, forced_next, nullptr, out_tokens, out_depth);
}

int spark_set_sampling(spark_ctx *c, float temperature, float top_p) {
  if (!c) return SPARK_EINVAL;
  if (!(temperature > 0.f)) {
    c->temperature = c->top_p = 0.f;
    return SPARK_OK;
  }
  if (!(top_p > 0.f) || top_p > 1.f) return fail(c, SPARK_EINVAL, "top_p outside (0, 1]");
  c->temperature = temperature;
  c->top_p = top_p;
  return SPARK_OK;
}

int spark_step(spark_ctx *c, int32_t n, const int32_t *seq_ids, const int32_t *forced_next,
               int32_t *out_tokens, int32_t *out_depth) {
  return spark_decode(c, 1, n, seq_ids, forced_next, out_tokens, out_depth);
}

int spark_get_logits(spark_ctx *c, int32_t seq_id, float *out_logits, int32_t *head) {
  if (!c || !out_logits) return SPARK_EINVAL;
  Seq *s = find_seq(c, seq_id);
  if (!s) return fail(c, SPARK_ENOSEQ, "unknown sequence id %d", seq_id);
  if (!s->g) return fail(c, SPARK_ESTATE, "sequence %d has not been stepped", seq_id);
  // logits rows are indexed by the position of the sequence in the last batch
  int row = -1;
  for (int i = 0; i < (int)c->last_ids.size(); ++i)
    if (c->last_ids[i] == seq_id) { row = i; break; }
  if (row < 0) return fail(c, SPARK_ESTATE, "sequence %d was not in the last step", seq_id);
  HIP_TRY(c, hipMemcpy(out_logits, at<float>(c, c->lo.logits) + (size_t)row * c->dv.V,
                       sizeof(float) * c->dv.V, hipMemcpyDeviceToHost));
  if (head) *head = s->last_full ? c->cfg.n_layers : c->cfg.exit_layer;
  return SPARK_OK;
}

int spark_get_kv(spark_ctx *c, int32_t seq_id, int32_t layer, int32_t pos, float *k_out,
                 float *v_out) {
  if (!c || !k_out || !v_out) return SPARK_EINVAL;
  Seq *s = find_seq(c, seq_id);
  if (!s) return fail(c, SPARK_ENOSEQ, "unknown sequence id %d", seq_id);
  const spark_config &g = c->cfg;
  if (layer < 0 || layer >= g.n_layers || pos < 0 || pos >= s->len)
    return fail(c, SPARK_EINVAL, "layer or position out of range");
  HIP_TRY(c, hipStreamSynchronize(c->stream));
  const int pt = g.kv_page_tokens, hd = g.head_dim, esz = c->dv.esz;
  const int page = s->pages[pos / pt];
  std::vector<unsigned char> raw((size_t)hd * esz);
  for (int which = 0; which < 2; ++which)
    for (int h = 0; h < g.n_kv_heads; ++h) {
      size_t o = (size_t)page * g.n_layers + layer;
      o = (o * 2 + which) * g.n_kv_heads + h;
      o = (o * pt + pos % pt) * hd;
      HIP_TRY(c, hipMemcpy(raw.data(), (const char *)c->kv_pool + o * esz, (size_t)hd * esz,
                           hipMemcpyDeviceToHost));
      float *dst = (which ? v_out : k_out) + (size_t)h * hd;
      for (int i = 0; i < hd; ++i) {
        if (esz == 2) {
          uint32_t u = (uint32_t)((const uint16_t *)raw.data())[i] << 16;
          memcpy(dst + i, &u, 4);
        } else {
          dst[i] = ((const float *)raw.data())[i];
        }
      }
    }
  return SPARK_OK;
}

int spark_seq_text_budget(spark_ctx *c, int32_t seq_id, int32_t n_text_tokens) {
  if (!c) return SPARK_EINVAL;
  Seq *s = find_seq(c, seq_id);
  if (!s) return fail(c, SPARK_ENOSEQ, "unknown sequence id %d", seq_id);
  if (n_text_tokens < 1) return fail(c, SPARK_EINVAL, "text budget < 1");
  if (s->text_budget > 0) return fail(c, SPARK_ESTATE, "sequence %d already has a text budget", seq_id);
  if (n_text_tokens < s->g - s->j_stream)
    return fail(c, SPARK_EINVAL, "sequence %d has generated more text tokens already", seq_id);
  if (c->cfg.n_text < 1) return fail(c, SPARK_EINVAL, "the interleave has no text slots");
  s->text_budget = n_text_tokens;
  if (s->prefilled) {   // the state is on the device already
    HIP_TRY(c, hipMemcpyAsync(at<int>(c, c->lo.state) + (size_t)seq_id * ST_WORDS + ST_TEXTBUDGET,
                              &s->text_budget, sizeof(int), hipMemcpyHostToDevice, c->stream));
    HIP_TRY(c, hipStreamSynchronize(c->stream));
  }
  return SPARK_OK;
}

namespace {
int set_phase(spark_ctx *c, int seq_id, Seq *s, int phase) {
  s->phase = phase;
  if (s->prefilled) {   // the state is on the device already
    HIP_TRY(c, hipMemcpyAsync(at<int>(c, c->lo.state) + (size_t)seq_id * ST_WORDS + ST_PHASE, &s->phase,
                              sizeof(int), hipMemcpyHostToDevice, c->stream));
    HIP_TRY(c, hipStreamSynchronize(c->stream));
  }
  return SPARK_OK;
}
}  // namespace

int spark_seq_set_phase(spark_ctx *c, int32_t seq_id, int32_t phase) {
  if (!c) return SPARK_EINVAL;
  Seq *s = find_seq(c, seq_id);
  if (!s) return fail(c, SPARK_ENOSEQ, "unknown sequence id %d", seq_id);
  if (phase < 0 || phase >= c->cfg.period_k) return fail(c, SPARK_EINVAL, "phase outside [0, period_k)");
  // a moved phase can join two runs of early exits: K-1 before and K-1 after the move, which the
  // pending slots hold; runs that early-exited text positions could extend further are not allowed
  if (c->cfg.text_period_k > 1) return fail(c, SPARK_EINVAL, "the phase cannot be moved when text exits early too");
  if (c->cfg.scope == SPARK_SCOPE_CHUNK && c->cfg.exit_layer < c->cfg.n_layers) {
    // per-chunk counters repeat with the cycle: the moved phase needs a full-depth slot in it, and
    // its runs of early exits, joined with the K-1 that may be pending from before the move, must
    // fit the pending slots (the check spark_init makes for the configuration's own phase)
    const int cyc = c->cfg.n_text + c->cfg.n_speech;
    int run = 0, longest = 0;
    bool any_full = false;
    for (int g = 0; g < 2 * cyc; ++g) {
      int is_text, full;
      schedule_decide(c->sp, g, 0, 0, 0, phase, is_text, full);
      if (full) { any_full = true; run = 0; } else { longest = std::max(longest, ++run); }
    }
    if (!any_full) return fail(c, SPARK_EINVAL, "with phase %d no slot of the cycle would run full depth", phase);
    if (longest + c->cfg.period_k > pending_slots(&c->cfg))
      return fail(c, SPARK_EINVAL, "with phase %d a run of early exits would outgrow the pending slots", phase);
  }
  return set_phase(c, seq_id, s, phase);
}

int spark_align_phases(spark_ctx *c, int32_t n, const int32_t *seq_ids) {
  if (!c || n < 1 || !seq_ids) return SPARK_EINVAL;
  if (c->cfg.scope != SPARK_SCOPE_STREAM) return fail(c, SPARK_EINVAL, "phases are aligned over stream counters only");
  if (c->cfg.text_period_k > 1) return fail(c, SPARK_EINVAL, "the phase cannot be moved when text exits early too");
  for (int i = 0; i < n; ++i)
    if (!find_seq(c, seq_ids[i])) return fail(c, SPARK_ENOSEQ, "unknown sequence id %d", seq_ids[i]);
  const int K = c->cfg.period_k;
  for (int i = 0; i < n; ++i) {
    Seq *s = find_seq(c, seq_ids[i]);
    // the K-th speech position from now runs full depth, for every sequence alike
    if (int rc = set_phase(c, seq_ids[i], s, (s->j_stream + K - 1) % K)) return rc;
  }
  return SPARK_OK;
}

int spark_seq_state(spark_ctx *c, int32_t seq_id, int32_t *len, int32_t *upper_valid,
                    int32_t *n_pending) {
  if (!c) return SPARK_EINVAL;
  Seq *s = find_seq(c, seq_id);
  if (!s) return fail(c, SPARK_ENOSEQ, "unknown sequence id %d", seq_id);
  // the device copy is authoritative
  int st[ST_WORDS];
  HIP_TRY(c, hipStreamSynchronize(c->stream));
  HIP_TRY(c, hipMemcpy(st, at<int>(c, c->lo.state) + (size_t)seq_id * ST_WORDS, sizeof(st),
                       hipMemcpyDeviceToHost));
  if (s->prefilled && (st[ST_LEN] != s->len || st[ST_NPENDING] != s->n_pending))
    return fail(c, SPARK_ESTATE, "device state and host mirror disagree");
  if (len) *len = s->len;
  if (upper_valid) *upper_valid = s->len - s->n_pending;
  if (n_pending) *n_pending = s->n_pending;
  return SPARK_OK;
}

int spark_get_stats(spark_ctx *c, int32_t seq_id, spark_stats *out) {
  if (!c || !out) return SPARK_EINVAL;
  Seq *s = find_seq(c, seq_id);
  if (!s) return fail(c, SPARK_ENOSEQ, "unknown sequence id %d", seq_id);
  memset(out, 0, sizeof(*out));
  out->text_steps = s->text_steps;
  out->speech_full_steps = s->speech_full;
  out->speech_ee_steps = s->speech_ee;
  memcpy(out->flush_rows, s->flush_rows, sizeof(out->flush_rows));
  const double L = c->cfg.n_layers, e = c->cfg.exit_layer;
  out->text_ee_steps = s->text_ee;
  if (s->text_steps + s->text_ee)
    out->mean_text_depth = (s->text_steps * L + s->text_ee * e) / (double)(s->text_steps + s->text_ee);
  const int64_t ns = s->speech_full + s->speech_ee;
  if (ns) {
    out->mean_speech_depth = (s->speech_full * L + s->speech_ee * e) / (double)ns;
    out->speech_layer_saving = (1.0 - out->mean_speech_depth / L) * 100.0;
  }
  return SPARK_OK;
}

int spark_seq_close(spark_ctx *c, int32_t seq_id) {
  if (!c) return SPARK_EINVAL;
  Seq *s = find_seq(c, seq_id);
  if (!s) return fail(c, SPARK_ENOSEQ, "unknown sequence id %d", seq_id);
  HIP_TRY(c, hipStreamSynchronize(c->stream));
  for (int p : s->pages) c->free_pages.push_back(p);
  int zero[ST_WORDS] = {0};
  HIP_TRY(c, hipMemcpy(at<int>(c, c->lo.state) + (size_t)seq_id * ST_WORDS, zero, sizeof(zero),
                       hipMemcpyHostToDevice));
  *s = Seq();
  return SPARK_OK;
}

void spark_destroy(spark_ctx *c) {
  if (!c) return;
  (void)hipStreamSynchronize(c->stream);
  for (hipEvent_t ev : c->prof_ev) (void)hipEventDestroy(ev);
  if (c->static_scratch) {
    delete[] c->h_in;
    delete[] c->h_out;
    if (c->device >= 0 && c->device < MAX_DEVICES) static_scratch_busy[c->device] = false;
  } else {
    if (c->h_in) (void)hipHostFree(c->h_in);
    if (c->h_out) (void)hipHostFree(c->h_out);
  }
  delete c;
}

const char *spark_last_error(const spark_ctx *c) { return c ? c->err : "null context"; }

int spark_profile_select(spark_ctx *c, int32_t kernel_class) {
  if (!c || kernel_class < -1 || kernel_class >= SPARK_KC_COUNT) return SPARK_EINVAL;
  HIP_TRY(c, hipStreamSynchronize(c->stream));
  c->prof_class = kernel_class;
  c->prof_used = 0;
  return SPARK_OK;
}

int spark_profile_read(spark_ctx *c, int64_t *n_launches, double *total_ms, double *empty_ms) {
  if (!c || !n_launches || !total_ms) return SPARK_EINVAL;
  HIP_TRY(c, hipStreamSynchronize(c->stream));
  double tot = 0, empty = 0;
  for (size_t i = 0; i + 2 < c->prof_used; i += 3) {
    float ms = 0, ms0 = 0;
    HIP_TRY(c, hipEventElapsedTime(&ms, c->prof_ev[i], c->prof_ev[i + 1]));
    HIP_TRY(c, hipEventElapsedTime(&ms0, c->prof_ev[i + 1], c->prof_ev[i + 2]));
    tot += ms;
    empty += ms0;
  }
  *n_launches = (int64_t)(c->prof_used / 3);
  *total_ms = tot;
  if (empty_ms) *empty_ms = empty;   // what the brackets themselves cost
  c->prof_used = 0;
  return SPARK_OK;
}

int spark_measure_read(spark_ctx *c, const void *buf, size_t bytes, int32_t reps, int32_t nontemporal,
                       double *gbps, uint32_t *checksum) {
  if (!c || !buf || !gbps || reps < 1) return SPARK_EINVAL;
  if (bytes < 16 || bytes % 16 || ((uintptr_t)buf & 15)) return fail(c, SPARK_EINVAL, "buffer must be 16-byte aligned and sized");
  // the wave sums go where the attention partials live between steps (at least 69 KB)
  const int blocks = c->n_cu * 8, words = blocks * (READ_THREADS / 64);
  const size_t part_bytes = c->lo.lens_u - c->lo.part;
  if (sizeof(unsigned) * words > part_bytes) return fail(c, SPARK_ENOMEM, "scratch too small for the read kernel's sums");
  unsigned *sink = at<unsigned>(c, c->lo.part);
  const read_u32x4 *p = (const read_u32x4 *)buf;
  const size_t n16 = bytes / 16;
  hipEvent_t e0, e1;
  HIP_TRY(c, hipEventCreate(&e0));
  HIP_TRY(c, hipEventCreate(&e1));
  auto launch = [&]() {
    if (nontemporal) read_stream_k<true><<<blocks, READ_THREADS, 0, c->stream>>>(p, n16, sink);
    else read_stream_k<false><<<blocks, READ_THREADS, 0, c->stream>>>(p, n16, sink);
  };
  launch();   // untimed: code object, TLB
  int rc = SPARK_OK;
  float ms = 0.f;
  if (hipEventRecord(e0, c->stream) != hipSuccess) rc = SPARK_EHIP;
  for (int r = 0; r < reps && rc == SPARK_OK; ++r) launch();
  if (rc == SPARK_OK && (hipGetLastError() != hipSuccess || hipEventRecord(e1, c->stream) != hipSuccess ||
                         hipEventSynchronize(e1) != hipSuccess || hipEventElapsedTime(&ms, e0, e1) != hipSuccess))
    rc = SPARK_EHIP;
  if (rc == SPARK_OK && checksum) {
    std::vector<unsigned> h(words);
    if (hipMemcpy(h.data(), sink, sizeof(unsigned) * words, hipMemcpyDeviceToHost) != hipSuccess) rc = SPARK_EHIP;
    unsigned x = 0;
    for (unsigned v : h) x ^= v;
    *checksum = x;
  }
  (void)hipEventDestroy(e0);
  (void)hipEventDestroy(e1);
  if (rc != SPARK_OK) return fail(c, rc, "the read measurement failed");
  *gbps = (double)bytes * reps / ((double)ms * 1e-3) / 1e9;
  return SPARK_OK;
}

}  // extern "C"
