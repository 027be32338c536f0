// Whole decoding steps of a small fp32 model in one launch.
//
// A step of a small model is a chain of some 20 launches that each need the complete output of the one before and
// move next to nothing: with 16 MB of weights they took 83 us a step, 4.7 us each whatever they did, where the bytes
// ask for 2.  Here SMALL_WGS workgroups stay for all steps of a call.  What a phase (a projection, attention, a head)
// hands to the next are 64-bit words, a value and the number of its phase; the next phase asks for its words until
// they have come.  They travel as device-scope accesses, so no cache is flushed or invalidated, nothing waits
// for an acknowledgement, and no word but the data's own has to arrive.  While they travel a workgroup
// fetches what the next phase needs and nobody is writing: weights, old cache entries, old hidden values.
//
// With flags instead (stores, acknowledgement, a word of each workgroup's, its poll, the loads) a hand-over of 1024
// values took 1.9 us between 32 workgroups, 2.1 between 64 and 3.4 between 256.  One workgroup per 8 CUs leaves each of
// the eight L2 an eighth of the weights, which stay in it from step to step.
// The launch is cooperative, so that all workgroups are resident before any waits; every wait is bounded as well.
#pragma once
#include "device_common.h"
#include "handover.h"
#include "sampling.h"
#include "sched.h"

namespace spark {

constexpr int SMALL_WGS = 32;
constexpr int SMALL_THREADS = SAMPLE_THREADS;    // the sampler's workgroups take part
constexpr int SMALL_WAVES = SMALL_THREADS / 64;
constexpr int SMALL_SEQS = 16;                   // sequences of a call
constexpr int SMALL_ROWS = 64;                   // rows of a pass
constexpr int SMALL_CTX = 1024;                  // positions a row may attend to
constexpr int SMALL_CHUNK = 256;                 // elements of a weight row that a wave multiplies at a time
constexpr int SMALL_MAX_CHUNKS = 16;             // ... and pieces of a row: inputs of up to 4096
constexpr int SMALL_X_FLOATS = 16384, SMALL_PART_FLOATS = 4096;   // LDS: staged rows, sums of the pieces
constexpr int SMALL_NORM_CHUNKS = 4;             // pieces of a normalised row, at most
constexpr size_t SMALL_LDS = sizeof(float) * (SMALL_X_FLOATS + SMALL_PART_FLOATS + SMALL_ROWS * SMALL_NORM_CHUNKS);
constexpr int SMALL_MAX_POLLS = 1 << 22;         // some seconds; then the launch gives up (other streams' and processes' kernels may
                                                 // hold its last workgroups up) and the call runs again as launches per operation
static_assert(SMALL_SEQS <= SMALL_WGS && SMALL_SEQS <= SMALL_WAVES, "a workgroup draws for one sequence, a wave reads one's arg-max");

// A projection phase: `n_tasks` pairs of weight rows of n_in
struct SmallPhase {
  int n_in, n_tasks;
  int chunks, chunk_bits;   // pieces of a weight row, and the power of two that they are counted in
  int task_bits;            // the same of a workgroup's tasks
  int tile;                 // rows taken at a time; 0: the phase does not fit
};
inline SmallPhase small_phase(int n_in, int n_tasks) {
  auto bits = [](int v) { int b = 0; while ((1 << b) < v) ++b; return b; };
  SmallPhase p;
  p.n_in = n_in; p.n_tasks = n_tasks;
  p.chunks = (n_in + SMALL_CHUNK - 1) / SMALL_CHUNK;
  p.chunk_bits = bits(p.chunks);
  const int tasks = (n_tasks + SMALL_WGS - 1) / SMALL_WGS;
  p.task_bits = bits(tasks);
  const int by_x = SMALL_X_FLOATS / (p.chunks * SMALL_CHUNK), by_part = SMALL_PART_FLOATS / (2 * (tasks << p.chunk_bits));
  const int by_threads = SMALL_THREADS >> p.task_bits;
  p.tile = by_x < by_part ? by_x : by_part;
  p.tile = p.tile < by_threads ? p.tile : by_threads;
  p.tile = p.tile < SMALL_ROWS ? p.tile : SMALL_ROWS;
  return p;
}

struct SmallSteps {
  SchedParams sp;
  int d, nq, nkv, F, V;
  SmallPhase qkv, o, gateup, down, lens, vocab;
  float eps;
  const float *embed, *attn_norm, *wq, *wk, *wv, *wo, *mlp_norm, *wg, *wu, *wd, *final_norm, *lm_head, *lens_a, *lens_b, *lens_norm, *lens_head;
  const float2 *rope;
  KVView kv;
  float *hidden, *logits;
  // words handed over (rows: of the largest pass), in two stretches that the launch clears first
  u64 *words_a, *words_b;
  int count_a, count_b;
  u64 *act_words, *x_words, *qkv_words, *attn_words, *u_words;   // [rows][F], [sequences + rows][d], [rows][heads * head_dim] twice, [sequences][d]
  u64 *wg_best;              // [sequence][SAMPLE_CAP], the first SMALL_WGS of each in use
  unsigned *flags;           // [SMALL_WGS]
  int *state, *plan;
  const int *seq_ids, *forced;
  const u64 *words;          // random words of the steps, nullptr: arg-max
  u64 *best;
  int *out_tokens, *out_depth;
  int n, steps;
  double temperature, top_p;
  unsigned epoch;            // number of the launch
  int max_polls, first_polls;   // questions of a wait before it runs out; of the first one, that all workgroups have started
  float *kept;               // copies of the sequences' pending rows as the call finds them, `kept_rows` places for each
  int kept_rows;
};

// whether a workgroup of the launch has room on the current device; asked once, before the first launch
bool small_steps_fit(int head_dim);
hipError_t launch_small_steps(const SmallSteps &a, int head_dim, hipStream_t stream);

}  // namespace spark
