// The layers of a pass of one row (a decoding step of one sequence) in one launch.
//
// A layer is five launches that each need the complete output of the one before: at the Step shape they took 101 us,
// of which the bytes ask for 68 at the rate of a plain read; the rest is the start, the end and the first round trip of
// each.  Here ROW_WGS workgroups, one per CU, stay for all layers.  Half of a workgroup's waves do nothing but
// stream: each takes its share of the CU's weight rows, phase after phase, through a ring in LDS that memory
// fills by itself, and asks for the next phase's weights while this one ends.  The other half gathers what a
// phase reads, finishes its sums and does attention.  What a phase hands over are 64-bit words, a value and the number of
// its layer (as in small_steps.h): the reader asks until the number is there, and no flush, acknowledgement or flag
// lies between.  The MLP is handed over in ROW_PARTS pieces, so that all but the last travel under the stream.
// The launch is cooperative, so that all workgroups are resident before any waits; every wait is bounded as well.
#pragma once
#include "device_common.h"
#include "handover.h"

namespace spark {

constexpr int ROW_WGS = 256;
constexpr int ROW_STREAM_WAVES = 8, ROW_AUX_WAVES = 8;
constexpr int ROW_THREADS = 64 * (ROW_STREAM_WAVES + ROW_AUX_WAVES), ROW_AUX = 64 * ROW_AUX_WAVES;
// Units (1 KiB of each row of a pair) of a wave.  Its ring has ROW_DEPTH places, of which ROW_DEPTH - ROW_SPARE are on
// their way from memory while it streams: more only make everything else that the CU asks for wait longer (two: 10.5 us for a
// third of gate/up, three or four: 11.6).  While it waits for a row, ROW_PARKED arrived units move into registers and
// the next are asked for one at a time; the spare places are asked for when the row has come and the parked units are multiplied.
constexpr int ROW_DEPTH = 4, ROW_SPARE = 2, ROW_PARKED = 8;
// Pieces that the MLP's activations are handed over in.  With four, a piece's gathering held up the stream of the next
// (seven layers of the Step shape, 12 steps: 7 695 us against 7 420), with two the last piece's stood alone (8 085).
constexpr int ROW_PARTS = 3;
constexpr int ROW_ACT_WORDS = 13;       // activations that a thread gathers at a time (a piece of 6400 in one trip; a narrower one asks for its last again)
// Sleeps (units of 64 cycles) before the first question for a row that has just been handed over, and for a piece of the
// MLP's activations: asked for all the time, the words' own traffic holds up what they wait for (90.2 against 88.9 us a layer).
// The same at every width, measured at the Step shape: 9 us a layer, which narrow layers, whose phases are shorter, lose (the rule of
// row_rule.h was measured with them).
constexpr int ROW_NAP = 40, ROW_PIECE_NAP = 127;
constexpr int ROW_HD = 128;             // head_dim
constexpr int ROW_MAX_GROUP = 16;       // query heads per KV head
constexpr int ROW_SLICE = 64;           // tokens of an attention slice, at most
constexpr int ROW_MAX_D = 8 * ROW_AUX;  // width of a row that is gathered at once
static_assert(2 * (ROW_MAX_D / ROW_HD) <= ROW_WGS, "two workgroups merge a head");
// Some seconds; then the launch gives up and the call goes on as launches per operation.  Other streams' and processes'
// kernels may hold compute units that its last workgroups wait for.
constexpr int ROW_MAX_POLLS = 1 << 22;

typedef hand_word row_word;

struct OneRow {
  int l0, l1, d, nq, nkv, F;
  float eps, scale;
  const bf16_t *wq, *wk, *wv, *wo, *wg, *wu, *wd;   // of layer 0
  const float *attn_norm, *mlp_norm;
  const float2 *rope;
  KVView kv;
  const RowDesc *row;
  float *hidden;
  row_word *h0, *h1, *qkv, *attn, *act, *part;   // [d], [d], [(nq + 2 nkv) * 128], [nq * 128], [ROW_PARTS][ROW_WGS][pairs of a piece], [nq][slices][ROW_HD + 2]
  unsigned tag;      // of layer l0; the next layers' follow
  int *error;        // ERR_STALLED is set here when a wait runs out
  int max_polls;     // questions of a wait before it runs out
  int pairs;         // of a phase and workgroup, at most
  // LDS, in bytes
  int lds_x, lds_act, lds_part, lds_misc;
};

// largest number of pairs of a workgroup's
inline int row_pairs(int n) { return (n + ROW_WGS - 1) / ROW_WGS; }
// a workgroup's activations of a piece of the MLP, at most
__host__ __device__ inline int row_slots(int f) { return ((f + ROW_WGS - 1) / ROW_WGS + ROW_PARTS - 1) / ROW_PARTS; }
// LDS of a workgroup; 0: too much
size_t one_row_lds(OneRow &a);
bool one_row_fit();
hipError_t launch_one_row(const OneRow &a, size_t lds, hipStream_t stream);

}  // namespace spark
