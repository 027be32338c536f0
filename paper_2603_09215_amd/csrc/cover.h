// How a launch covers a projection with workgroups, and what its partial sums need: plain integer
// arithmetic, so that a host program can check it over all shapes without a GPU.
#pragma once
#include <stddef.h>

namespace spark {

constexpr int MG_KC = 64;              // k per chunk: one 128-byte line of a weight row, 4 MFMA steps
constexpr int MG_MAX_SPLIT = 32;       // ranges of k whose sums a finishing launch adds up, at most
constexpr int TG_WAVES = 4;
constexpr int TG_TASKS = 16;           // tasks of one A tile
constexpr int OP_ROWS = 48;            // rows of a pass whose activations lie in operand order, at most
constexpr int TD_WAVES = 4;            // of a workgroup of mfma_direct_k
constexpr int TD_CUT_TILES = 2;        // A tiles of a workgroup of mfma_direct_k whose k is cut
constexpr size_t MFMA_PARTIAL_BYTES = 48u << 20;  // k-split partial sums of one projection

constexpr int ceil_div(int a, int b) { return (a + b - 1) / b; }

// A tile is 128 * TB tasks x 32 * MTILES activation rows; the
// first n_whole tiles are one workgroup each, over the whole k range, and end in the epilogue; the
// n_cut tiles behind them are cut into n_split ranges of k, whose partial sums a finishing launch
// adds up.  So whole rounds of the chip's CUs do without partial sums, and the tiles that would be
// a nearly empty last round, or less than one, are spread over all CUs.
struct TileCover {
  int n_task_tiles, n_row_tiles;
  int n_whole, n_cut, n_split, chunks_per_split;
  int m_pitch;     // rows of a tile's partial sums (a pass of eight rows writes and reads a quarter of 32)
  int max_words;   // bytes of a row's list of magnitudes that a wave of a whole tile writes: one, or one per block of 32 tasks
  int xcd_groups;
};

// bytes of one range's sums of `tiles` tiles, both weight rows of every task
constexpr size_t range_bytes(int tiles, int tasks_per_tile, int m_pitch) {
  return sizeof(float) * (size_t)tiles * tasks_per_tile * 2 * m_pitch;
}

// Ranges of k for `tiles` workgroups' worth of work on n_cu CUs: the count that keeps most of the
// chip busy over whole rounds, with min_chunks chunks each at least (the pipeline needs a few to fill)
inline int choose_split(int tiles, int slots, int n_chunks, int min_chunks, size_t bytes_per_split) {
  int most = n_chunks / min_chunks;
  const size_t fit = MFMA_PARTIAL_BYTES / bytes_per_split;
  if ((size_t)most > fit) most = (int)fit;
  double best = 0.0;
  int split = 1;
  for (int s = 1; s <= most && s <= MG_MAX_SPLIT; ++s) {
    const int blocks = tiles * s, rounds = ceil_div(blocks, slots);
    const double util = (double)blocks / ((double)rounds * slots);
    if (util > best + 0.02) { best = util; split = s; }
  }
  return split;
}

// Blocks of 32 rows in a row tile of m rows: row tiles of equal height, as few as `most_blocks`
// allows, every further tile streams the weights again.  (One block: only where mfma_direct_k is
// switched off; it runs as a tile of two.)
inline int tiled_row_blocks_for(int m, int most_blocks) {
  const int blocks = ceil_div(m, 32), z = ceil_div(blocks, most_blocks), mt = ceil_div(blocks, z);
  return mt < 2 ? 2 : mt;
}

// mfma_tiled_k.  always_cut: the epilogue runs in the finishing launch only; never_cut: in the
// projection only.
inline TileCover cover_tiled(int m, int n_in, int n_tasks, int mtiles, int tb, bool always_cut, bool never_cut, int n_cu,
                             int xcd_max_split) {
  const int tasks = 32 * TG_WAVES * tb, mrows = 32 * mtiles, n_chunks = ceil_div(n_in, MG_KC);
  TileCover tc;
  tc.n_task_tiles = ceil_div(n_tasks, tasks);
  tc.n_row_tiles = ceil_div(m, mrows);
  tc.m_pitch = tc.n_row_tiles > 1 ? mrows : ceil_div(m, 8) * 8;
  const int tiles = tc.n_task_tiles * tc.n_row_tiles;
  // (rounds are counted in CUs: one workgroup keeps a CU's share of the memory system or of the
  // MFMA rate busy, two on a CU share it)
  tc.n_whole = never_cut ? tiles : always_cut ? 0 : tiles / n_cu * n_cu;
  tc.n_split = 1;
  const int rest = tiles - tc.n_whole;
  if (rest) {
    const int min_chunks = tiles < 32 ? 4 : 8;   // few tiles: shorter k ranges are worth the pipeline fill they cost
    tc.n_split = choose_split(rest, n_cu, n_chunks, min_chunks, range_bytes(rest, tasks, tc.m_pitch));
    if (tc.n_split == 1 && !always_cut) tc.n_whole = tiles;
  }
  tc.n_cut = tiles - tc.n_whole;
  tc.chunks_per_split = ceil_div(n_chunks, tc.n_split);
  tc.n_split = ceil_div(n_chunks, tc.chunks_per_split);
  tc.xcd_groups = tc.n_row_tiles > 1 && tc.n_split <= xcd_max_split;
  tc.max_words = tc.n_cut ? 2 : 1;   // (a finishing workgroup writes one word per block of tasks: a wave then does too)
  return tc;
}

constexpr size_t tiled_partial_bytes(const TileCover &tc, int tb) {
  return tc.n_cut ? tc.n_split * range_bytes(tc.n_cut, 32 * TG_WAVES * tb, tc.m_pitch) : 0;
}

// Whole tiles of three and of two blocks of 32 rows, so that the CUs get about as many blocks each: the first
// task tiles are covered by part[0].n_row_tiles high and part[2].n_row_tiles low ones, the others by part[1] and
// part[3].  (74 task tiles of 16 blocks of rows, 4.6 blocks for each of 256 CUs: tiles of three alone are two rounds,
// six blocks; 236 of three and 238 of two are one of each, five.)
struct MixedCover {
  TileCover part[4];
  float cost;   // microseconds, see wide_tile_cost; 0: no such cover
  int tiles() const {
    int n = 0;
    for (const TileCover &p : part) n += p.n_task_tiles * p.n_row_tiles;
    return n;
  }
};

// Microseconds of a whole tile of 256 tasks with `blocks` blocks of rows: 2.45 and 1.75 per chunk with three and
// two, all CUs busy, and its start and epilogue
inline float wide_tile_cost(int blocks, int n_chunks) { return n_chunks * (0.35f + 0.7f * blocks) + 4.f + 3.f * blocks; }

// Time until n_cu CUs have taken n_high jobs of one length and then n_low of a shorter one, each as it becomes free
inline float two_lengths_makespan(int n_high, float high, int n_low, float low, int n_cu) {
  const int late = n_high % n_cu, early = n_cu - late;   // CUs that end with a long job, and the others, which have one less
  const float start = (float)(n_high / n_cu) * high;     // of the others' first short job
  if (!late) return start + (float)ceil_div(n_low, n_cu) * low;
  const float joined = start + high;                     // from here on all CUs take short ones
  const int ahead = (int)(high / low), rest = n_low - early * ahead;
  if (rest <= 0) return joined;
  const int turns = (rest - 1) / n_cu, last = rest - turns * n_cu;   // the early CUs end a turn first
  return joined + (float)turns * low + (last <= early ? (float)(ahead + 1) * low - high : low);
}

inline TileCover whole_part(int n_task_tiles, int n_row_tiles) {
  TileCover tc;
  tc.n_task_tiles = n_task_tiles;
  tc.n_row_tiles = n_row_tiles;
  tc.n_whole = n_task_tiles * n_row_tiles;
  tc.n_cut = 0;
  tc.n_split = 1;
  tc.chunks_per_split = tc.m_pitch = 0;
  tc.max_words = 1;
  tc.xcd_groups = n_row_tiles > 1;
  return tc;
}

// The best such cover of m rows by tiles of 256 tasks: x task tiles with a high and b low tiles, the others with
// two high ones less and three low ones more (as many blocks)
inline MixedCover cover_mixed(int m, int n_in, int n_tasks, int n_cu) {
  const int T = ceil_div(n_tasks, 64 * TG_WAVES), blocks = ceil_div(m, 32), n_chunks = ceil_div(n_in, MG_KC);
  const float high = wide_tile_cost(3, n_chunks), low = wide_tile_cost(2, n_chunks);
  float best = 1e30f;
  int best_a = 0, best_b = 0, best_x = T;
  for (int total = blocks; total <= blocks + 1; ++total)
    for (int a = 0; 3 * a <= total; ++a) {
      if ((total - 3 * a) % 2) continue;
      const int b = (total - 3 * a) / 2;
      for (int x = a >= 2 ? 1 : T; x <= T; ++x) {
        const int n_high = x * a + (T - x) * (a - 2), n_low = x * b + (T - x) * (b + 3);
        const float t = two_lengths_makespan(n_high, high, n_low, low, n_cu);
        if (t < best) { best = t; best_a = a; best_b = b; best_x = x; }
      }
    }
  const int rest = T - best_x;
  MixedCover mc{{whole_part(best_x, best_a), whole_part(rest, rest ? best_a - 2 : 0), whole_part(best_x, best_b), whole_part(rest, rest ? best_b + 3 : 0)}, best};
  return mc;
}

// That cover where it is the better one: against tiles of equal height, `most_blocks` at most, by the same estimate.  Only against whole ones: a tile
// whose k is cut has shorter chains of running sums, each of which an MFMA rounds to 32 bits, than a whole tile of this
// kernel has (64 tasks a wave leave no registers to fold them), so where the last round of equal tiles would be cut it stays.
// (There the mixed cover was up to 4 % faster, gate/up of 1023 rows, d 4096, 13696 tasks 470 -> 451 us, and a seventh of the results
// had chains three times as long.)
inline MixedCover choose_mixed(int m, int n_in, int n_tasks, int most_blocks, int n_cu) {
  MixedCover none{};
  if (most_blocks < 3 || ceil_div(m, 32) < 3) return none;
  const int mt = tiled_row_blocks_for(m, 3);
  const TileCover tc = cover_tiled(m, n_in, n_tasks, mt, 2, false, false, n_cu, 0);
  if (tc.n_cut) return none;
  const MixedCover mc = cover_mixed(m, n_in, n_tasks, n_cu);
  const int n_chunks = ceil_div(n_in, MG_KC);
  const float tile = wide_tile_cost(mt, n_chunks);
  if (mc.cost >= ceil_div(tc.n_whole, n_cu) * tile) return none;
  // More than one round of CUs: the chip's power holds the rate then, so that what counts is the work, not what the last
  // round leaves idle, and equal work in lower tiles takes longer.  (Prompts of a quarter of the layers with it and without: 3584 wide, 16
  // blocks of rows 5140 and 5219 us, 17 5318 and 5390, 25 7240 and 7320, but 26 7439 and 7356, 27 7477 and 7385; 4096 wide, 22 blocks 8295
  // and 8452, 23 8487 and 8467.  The work saved there is 7, 2, 4, 1 and -2 %; 4 and 1 %.)  In less than one, it is the idle CUs: 5 and 6
  // blocks 2932 and 3010, 4096 wide, 7 and 8 4267 and 4447.
  const float work = (mc.part[0].n_whole + mc.part[1].n_whole) * wide_tile_cost(3, n_chunks) + (mc.part[2].n_whole + mc.part[3].n_whole) * wide_tile_cost(2, n_chunks);
  if (tc.n_whole > n_cu && work > 0.98f * (float)tc.n_whole * tile) return none;
  return mc;
}

// Blocks of 32 rows in a row tile of a projection with 32 tasks a wave and more rows than one tile
// takes: such a launch is one to three rounds of CUs, and what the last of them leaves idle differs
// more between the heights than the heights themselves do.  The time of a cover is taken as that of
// the CU with the most chunks, 0.4 us for each of a chunk's blocks of rows and as much for its weights, and
// that of its partial sums, at 5 TB/s there and back; a lower tile has to save a twentieth.
// (down, 768 rows of d 4096, k 13696: tiles of 128 rows make two ranges on 192 CUs, of 96 rows two
// on all 256; a prompt of 2300 tokens in three such passes 25.4 ms with the former, 23.8 with the latter.)
// With the starts and epilogues of tiles and the speed of idle CUs in the estimate a third of the sizes of q/k/v and o get
// other heights, with k whole or in two where this one cuts it in four to seven, and prompts were up to 1.2 % faster (4096
// wide, a quarter of the layers, 1024 tokens 10941 -> 10841 us, 8192 92071 -> 90473; 3584 wide, 701 tokens 6820 -> 6711).  But the
// sums of whole k have longer chains, and logits behind such prompts were further from 64 bits: 2 % in the mean
// of 312 (batches of 32 and of 48, standard error 1 %).
inline int narrow_row_blocks(int m, int n_in, int n_tasks, int most_blocks, bool always_cut, int n_cu) {
  if (ceil_div(m, 32) <= most_blocks) return tiled_row_blocks_for(m, most_blocks);
  int best = most_blocks;
  double least = 0.0;
  for (int mt = most_blocks; mt >= 2; --mt) {
    const TileCover tc = cover_tiled(m, n_in, n_tasks, mt, 1, always_cut, false, n_cu, 0);
    const long chunks = (long)ceil_div(tc.n_whole, n_cu) * ceil_div(n_in, MG_KC) +
                        (tc.n_cut ? (long)ceil_div(tc.n_cut * tc.n_split, n_cu) * tc.chunks_per_split : 0);
    const double cost = (double)chunks * (mt + 1) * 0.4 + (double)tiled_partial_bytes(tc, 1) * 2.0 / 5e6;
    if (mt == most_blocks || cost < 0.95 * least) { least = cost; best = mt; }
  }
  return best;
}

// Where mfma_direct_k reads the activations of a step of 32 k, in operand order ([n_in / 4][op_rows][4] floats): lane group kq
// (0..3) has the eight k from 32 step + 8 kq on, two words of 16 bytes that lie 16 op_rows bytes apart.  n_in is a multiple
// of 8, the last step may end behind it, and the last chunk may have a step that begins behind it: there the last
// eight are read, finite numbers of the row's own range for weights that are zeros.
constexpr int direct_x_step(int step, int n_in) { return step < (n_in - 8) / 32 ? step : (n_in - 8) / 32; }   // the step that is read
constexpr int direct_x_quad(int kq, int read_step, int n_in) {   // of that step the quad of k
  return 2 * kq < n_in / 4 - 2 - 8 * read_step ? 2 * kq : n_in / 4 - 2 - 8 * read_step;
}
// And the tile of weights behind the workgroup's first that its tile q is read from: past the last one, the last
constexpr int direct_w_tile(int q, int first, int n_blocks) { return q < n_blocks - 1 - first ? q : n_blocks - 1 - first; }

// Dynamic LDS of mfma_direct_k with nt tiles and operands of cols activation rows: the waves' sums, the weight
// rows' scales, and the activation rows' exponents, which all threads find together, td_lanes_per_row of them a
// row: 16, 32 or 64 rows, of which the last operand has 48.
constexpr int TD_PITCH = 36;   // floats per (tile, activation row): 32 weight rows and a skew of one 16-byte word
constexpr int td_lanes_per_row(int cols) { return cols == 16 ? 16 : cols == 32 ? 8 : 4; }
constexpr size_t td_exp_at(int nt, int cols) { return sizeof(float) * (TD_WAVES * nt * cols * TD_PITCH + nt * 32); }
constexpr size_t td_lds_bytes(int nt, int cols) { return td_exp_at(nt, cols) + sizeof(int) * (64 * TD_WAVES / td_lanes_per_row(cols)); }

// mfma_direct_k with its k whole: tiles of a workgroup.  One for at most 8 rows, whose activations cost
// a workgroup little (the weights' time of gate/up at 8 rows, d 3584 and 4096: 46.7 and 43.0 us with one tile, 49.1
// and 44.1 as below; at 16 rows 52.4 and 47.0 against 49.0 and 43.7); not for the heads, whose workgroups
// each send an atomic per row (39624 outputs, 8 rows: 56 us with one tile, 50 with three).  Otherwise as few
// rounds of CUs as five tiles make, and the last one full.
inline int direct_tiles(int m, int blocks, int n_cu, bool heads) {
  if (m <= 8 && !heads) return 1;
  int nt = 1, best = 0;
  for (int n = 1; n <= 5; ++n) {
    const int cost = ceil_div(ceil_div(blocks, n), n_cu) * n;   // tiles the busiest CU takes
    if (n == 1 || cost <= best) { best = cost; nt = n; }
  }
  return nt;
}

// mfma_direct_k with its k cut: tiles of a workgroup, workgroups per range, ranges (1: it is not cut) and chunks in each
struct DirectCut { int tiles, groups, split, chunks_per_split; };
// bytes of the ranges' sums: both weight rows of every task, for whole operands of 16 rows
constexpr size_t direct_partial_bytes(int m, const DirectCut &c) {
  return sizeof(float) * (size_t)c.split * c.groups * c.tiles * 2 * TG_TASKS * (ceil_div(m, 16) * 16);
}
// A long k with few tasks (down) would be streamed by few CUs, each reading all activations of a long row: it is cut
// over the CUs.  whole_k: the longest k that is never cut; negative: by the rule, for which 8192 and less are short.  Of those, what leaves half of the CUs idle (o) is cut in two from 9 rows
// on: 16 rows 12.60 -> 12.51 ms a step, 32 rows 16.05 -> 15.87, 48 rows 17.09 -> 16.85; 8 rows are level.  What fills
// more than half would need a second round of CUs (q/k/v, 288 halves on 256 CUs: a step 1 % slower).
inline DirectCut direct_cut(int m, int n_in, int n_tasks, int n_cu, int whole_k) {
  const bool by_rule = whole_k < 0;
  if (by_rule) whole_k = 8192;
  const int n_chunks = ceil_div(n_in, MG_KC), blocks = ceil_div(n_tasks, TG_TASKS);
  DirectCut c{1, blocks, 1, n_chunks};
  if (n_in > whole_k && blocks < 4 * n_cu) {
    c.tiles = TD_CUT_TILES;
    c.groups = ceil_div(blocks, TD_CUT_TILES);
    c.split = n_cu / c.groups;
    if (c.split > n_chunks / 8) c.split = n_chunks / 8;
    if (c.split > MG_MAX_SPLIT) c.split = MG_MAX_SPLIT;
  } else if (by_rule && n_in <= whole_k && m > 8 && 2 * blocks <= n_cu && n_chunks >= 16) {
    c.split = 2;
  }
  while (c.split > 1 && direct_partial_bytes(m, c) > MFMA_PARTIAL_BYTES) --c.split;
  if (c.split < 1) c.split = 1;
  c.chunks_per_split = ceil_div(n_chunks, c.split);
  c.split = ceil_div(n_chunks, c.chunks_per_split);
  return c;
}

// Rows that go through the layers together at most: the partial sums of a residual projection
// (d_model outputs), one range of k at least, have to fit their buffer.  They are written for whole
// tiles: of 256 tasks (512 outputs), and of 64, 96 or 128 rows, which a multiple of 384 rows holds a
// whole number of, however the rows up to it are dealt to tiles.
inline int pass_rows_limit(int d_model) {
  return (int)(MFMA_PARTIAL_BYTES / (sizeof(float) * (size_t)ceil_div(d_model, 512) * 512)) / 384 * 384;
}

}  // namespace spark
