"""The covers that the MFMA projections are launched with (csrc/cover.h, plain integer arithmetic),
checked on the host over every model width, row count and tile shape that the library accepts: the
partial sums of every launch fit their buffer, which other buffers lie directly behind, and the
tiles of a cover are all there, once."""
import pathlib
import subprocess

CSRC = pathlib.Path(__file__).resolve().parent.parent / "paper_2603_09215_amd" / "csrc"

DRIVER = r"""
#include <cstdio>
#include <cstdlib>
#include "cover.h"
using namespace spark;
static long checked = 0, cut = 0, mixed = 0;
static void bad(const char *what, int m, int n_in, int n_tasks, int mt, int tb, size_t bytes) {
  printf("%s: %d rows, k = %d, %d tasks, tiles of %d rows x %d tasks: %zu bytes\n", what, m, n_in, n_tasks, 32 * mt, 128 * tb, bytes);
  exit(1);
}
static void projection(int m, int n_in, int n_tasks, bool always, bool never, int n_cu) {
  for (int tb = 1; tb <= 2; ++tb)
    for (int most = 2; most <= (tb == 1 ? 4 : 3); ++most) {
      const int mt = tb == 1 && !never ? narrow_row_blocks(m, n_in, n_tasks, most, always, n_cu) : tiled_row_blocks_for(m, most);
      if (mt < 2 || mt > most) bad("row blocks", m, n_in, n_tasks, mt, tb, 0);
      const TileCover tc = cover_tiled(m, n_in, n_tasks, mt, tb, always, never, n_cu, 4);
      const size_t bytes = tiled_partial_bytes(tc, tb);
      if (bytes > MFMA_PARTIAL_BYTES) bad("partial sums", m, n_in, n_tasks, mt, tb, bytes);
      const int chunks = ceil_div(n_in, MG_KC);
      if (tc.n_whole + tc.n_cut != tc.n_task_tiles * tc.n_row_tiles || tc.n_task_tiles * 128 * tb < n_tasks ||
          tc.n_row_tiles * 32 * mt < m || (always && tc.n_whole) || (never && tc.n_cut) || tc.n_split > MG_MAX_SPLIT ||
          (tc.n_split - 1) * tc.chunks_per_split >= chunks || tc.n_split * tc.chunks_per_split < chunks ||
          (tc.n_row_tiles == 1 && tc.m_pitch < m))
        bad("cover", m, n_in, n_tasks, mt, tb, bytes);
      ++checked;
      cut += tc.n_cut > 0;
      mixed += tc.n_cut > 0 && tc.n_whole > 0;
    }
  if (m <= OP_ROWS) {
    const DirectCut c = direct_cut(m, n_in, n_tasks, n_cu, 0);
    const size_t bytes = direct_partial_bytes(m, c);
    if (c.split > 1 && bytes > MFMA_PARTIAL_BYTES) bad("direct", m, n_in, n_tasks, 1, 1, bytes);
    if (c.split < 1 || c.split > MG_MAX_SPLIT || c.split * c.chunks_per_split < ceil_div(n_in, MG_KC)) bad("direct ranges", m, n_in, n_tasks, 1, 1, bytes);
  }
  // the kernel on the caller's weights: one tile, all rows; its residual projections are always cut
  const size_t rows_bytes = range_bytes(1, n_tasks, ceil_div(m, 8) * 8);
  const int split = choose_split(8, n_cu, ceil_div(n_in, MG_KC), 4, rows_bytes);
  if ((split > 1 || always) && split * rows_bytes > MFMA_PARTIAL_BYTES) bad("rows", m, n_in, n_tasks, 0, 0, split * rows_bytes);
}
int main() {
  const int cus[] = {256, 64};
  for (int d = 8; d <= 4096; d += 8) {
    const int limit = pass_rows_limit(d), top = limit < 8192 ? limit : 8192;   // max_batch 256 x 32 slots
    if (limit < 384) bad("limit", limit, 0, d, 0, 0, 0);
    for (int n_cu : cus)
      for (int b = 1; b <= ceil_div(top, 32); ++b) {
        const int m = 32 * b < top ? 32 * b : top;
        if (d > 512 && d % 512 > 24 && m + 400 < top && b % 7) continue;   // (thinned away from the edges)
        projection(m, 1024, d / 2, true, false, n_cu);        // residual projections, the lens translator
        projection(m, 18944, d / 2, true, false, n_cu);
        if (m > 31) projection(m - 31, 4096, d / 2, true, false, n_cu);
      }
  }
  const int widths[] = {40, 1064, 2304, 8192, 13696, 18944, 40000};   // q/k/v, gate/up and vocabularies in tasks
  for (int tasks : widths)
    for (int m = 1; m <= 8192; m += m < 300 ? 1 : 31)
      for (int n_cu : cus) {
        projection(m, 3584, tasks, false, false, n_cu);
        if (m <= 256) projection(m, 4096, tasks, false, true, n_cu);
      }
  printf("%ld covers, %ld cut, %ld with whole and cut tiles\n", checked, cut, mixed);
  return 0;
}
"""


MIXED = r"""
#include <algorithm>
#include <cmath>
#include <cstdio>
#include <vector>
#include "cover.h"
using namespace spark;
static float dealt(int n_high, float high, int n_low, float low, int n_cu) {   // one job after the other to whoever is free first
  std::vector<float> t(n_cu, 0.f);
  for (int i = 0; i < n_high + n_low; ++i) *std::min_element(t.begin(), t.end()) += i < n_high ? high : low;
  return *std::max_element(t.begin(), t.end());
}
int main() {
  for (int n_cu : {256, 7})
    for (float high : {1.01f, 1.39f, 1.5f, 1.99f, 2.5f})
      for (int n_high = 0; n_high < 3 * n_cu; n_high += n_cu / 7)
        for (int n_low = 0; n_low < 3 * n_cu; n_low += n_cu / 5) {
          const float want = dealt(n_high, high, n_low, 1.f, n_cu), got = two_lengths_makespan(n_high, high, n_low, 1.f, n_cu);
          if (std::fabs(got - want) > 1e-4f * want) { printf("%d of %g and %d: %g, not %g\n", n_high, high, n_low, got, want); return 1; }
        }
  long covers = 0, two = 0, chosen = 0, stays = 0;
  const int widths[] = {8192, 8264, 13696, 18944, 40000};
  for (int tasks : widths)
    for (int n_cu : {256, 64})
      for (int m = 65; m <= 3072; m += m < 400 ? 1 : 37) {
        const MixedCover mc = cover_mixed(m, 3584, tasks, n_cu);
        const int T = ceil_div(tasks, 256), blocks = ceil_div(m, 32);
        std::vector<int> hit(T * (blocks + 8), 0);
        for (int k = 0; k < 4; ++k)     // as the kernel places them
          for (int bx = 0; bx < mc.part[k].n_task_tiles; ++bx)
            for (int bz = 0; bz < mc.part[k].n_row_tiles; ++bz) {
              const int first = k < 2 ? 3 * bz : 3 * mc.part[k - 2].n_row_tiles + 2 * bz, x = bx + (k & 1 ? mc.part[0].n_task_tiles : 0);
              for (int b = first; b < first + (k < 2 ? 3 : 2); ++b) {
                if (x >= T || b >= blocks + 2) { printf("out of range: %d tasks, %d rows\n", tasks, m); return 1; }
                ++hit[x * (blocks + 8) + b];
              }
            }
        for (int x = 0; x < T; ++x)
          for (int b = 0; b < blocks; ++b)
            if (hit[x * (blocks + 8) + b] != 1) { printf("not once: %d tasks, %d rows\n", tasks, m); return 1; }
        ++covers;
        two += mc.part[1].n_task_tiles > 0;
        // taken only where no result has a longer chain of running sums for it: no tile of equal height is cut
        const TileCover tc = cover_tiled(m, 3584, tasks, tiled_row_blocks_for(m, 3), 2, false, false, n_cu, 4);
        const MixedCover ch = choose_mixed(m, 3584, tasks, 3, n_cu);
        if (ch.cost > 0.f) {
          if (tc.n_cut) { printf("in place of cut tiles: %d tasks, %d rows\n", tasks, m); return 1; }
          // and where there is more than one round, only for less work: fewer blocks of rows
          const int mt = tiled_row_blocks_for(m, 3), high = ch.part[0].n_whole + ch.part[1].n_whole, low = ch.part[2].n_whole + ch.part[3].n_whole;
          if (tc.n_whole > n_cu && 3 * high + 2 * low >= mt * tc.n_whole) { printf("no less work: %d tasks, %d rows\n", tasks, m); return 1; }
          ++chosen;
        }
        stays += tc.n_cut > 0;
      }
  // what the GPU tests of a prompt's MLP are about: whole and cut tiles, lower tiles alone, both heights
  const struct { int rows, d, tasks, whole, cut, high, low; } cases[] = {
      {1023, 1032, 8264, 256, 107, 0, 0}, {700, 1032, 8264, 256, 8, 0, 0}, {340, 1032, 8264, 132, 0, 0, 198}, {990, 1032, 10248, 451, 0, 247, 265}};
  for (const auto &c : cases) {
    const TileCover tc = cover_tiled(c.rows, c.d, c.tasks, tiled_row_blocks_for(c.rows, 3), 2, false, false, 256, 4);
    const MixedCover mc = choose_mixed(c.rows, c.d, c.tasks, 3, 256);
    const int high = mc.cost > 0.f ? mc.part[0].n_whole + mc.part[1].n_whole : 0, low = mc.cost > 0.f ? mc.part[2].n_whole + mc.part[3].n_whole : 0;
    if (tc.n_whole != c.whole || tc.n_cut != c.cut || high != c.high || low != c.low) {
      printf("%d rows: %d whole, %d cut, %d high, %d low\n", c.rows, tc.n_whole, tc.n_cut, high, low);
      return 1;
    }
  }
  printf("%ld covers, %ld with two kinds of task tile, %ld taken, %ld stay cut\n", covers, two, chosen, stays);
  return 0;
}
"""


def test_covers_by_tiles_of_two_heights_take_every_block_once(tmp_path):
    src, exe = tmp_path / "mixed.cpp", tmp_path / "mixed"
    src.write_text(MIXED)
    subprocess.run(["g++", "-O2", "-std=c++17", "-Wall", "-Werror", f"-I{CSRC}", "-o", str(exe), str(src)], check=True)
    out = subprocess.run([str(exe)], capture_output=True, text=True, timeout=120)
    assert out.returncode == 0, out.stdout
    n, n_two, n_taken, n_cut = (int(w) for w in out.stdout.split() if w.isdigit())
    assert n > 3000 and n_two > 300 and n_taken > 150 and n_cut > 500, out.stdout


CUTS = r"""
#include <cstdio>
#include <initializer_list>
#include "cover.h"
using namespace spark;
int main() {
  long cuts = 0, cut = 0;
  for (int n_cu : {256, 304, 64, 8})
    for (int n_in : {64, 128, 896, 1024, 3584, 4096, 8192, 8256, 13696, 18944})
      for (int tasks = 8; tasks <= 20000; tasks += tasks < 5000 ? 8 : 168)
        for (int m = 1; m <= 48; m += m < 9 ? 1 : 13)
          for (int whole_k : {0, 8192, -1}) {
            const DirectCut c = direct_cut(m, n_in, tasks, n_cu, whole_k);
            const int chunks = ceil_div(n_in, MG_KC);
            const bool bad = (whole_k > 0 && n_in <= whole_k && c.split > 1) ||                                     // as told,
                             c.split < 1 || c.split > MG_MAX_SPLIT || c.split * c.chunks_per_split < chunks ||      // all of k,
                             (c.split - 1) * c.chunks_per_split >= chunks ||                                        // no empty range,
                             c.groups * c.tiles * TG_TASKS < tasks || (c.groups - 1) * c.tiles * TG_TASKS >= tasks ||   // all tasks,
                             (c.split > 1 && (direct_partial_bytes(m, c) > MFMA_PARTIAL_BYTES || c.groups > 2 * n_cu));
            if (bad) { printf("%d rows, %d x %d on %d CUs: %d groups of %d, %d ranges of %d\n", m, n_in, tasks, n_cu, c.groups, c.tiles, c.split, c.chunks_per_split); return 1; }
            ++cuts;
            cut += c.split > 1;
          }
  printf("%ld checked, %ld cut\n", cuts, cut);
  return 0;
}
"""


def test_cuts_of_a_few_rows_take_every_range_and_task_once(tmp_path):
    src, exe = tmp_path / "cuts.cpp", tmp_path / "cuts"
    src.write_text(CUTS)
    subprocess.run(["g++", "-O2", "-std=c++17", "-Wall", "-Werror", f"-I{CSRC}", "-o", str(exe), str(src)], check=True)
    out = subprocess.run([str(exe)], capture_output=True, text=True, timeout=120)
    assert out.returncode == 0, out.stdout
    n, n_cut = (int(w) for w in out.stdout.split() if w.isdigit())
    assert n > 100_000 and n_cut > 10_000, out.stdout


DIRECT_LDS = r"""
#include <cstdio>
#include "cover.h"
using namespace spark;
int main() {
  int layouts = 0;
  for (int cols = 16; cols <= OP_ROWS; cols += 16)
    for (int nt = 1; nt <= 5; ++nt) {
      // every thread's group of lanes stores the exponent of one row
      const size_t lds = td_lds_bytes(nt, cols), last = td_exp_at(nt, cols) + sizeof(int) * ((64 * TD_WAVES - 1) / td_lanes_per_row(cols));
      if (last + sizeof(int) > lds || 64 * TD_WAVES / td_lanes_per_row(cols) < cols || lds > 160 * 1024) {
        printf("%d tiles, %d rows: the last exponent ends at byte %zu of %zu\n", nt, cols, last + sizeof(int), lds);
        return 1;
      }
      ++layouts;
    }
  printf("%d layouts\n", layouts);
  return 0;
}
"""


def test_exponents_of_all_rows_lie_inside_the_lds_of_a_launch(tmp_path):
    src, exe = tmp_path / "lds.cpp", tmp_path / "lds"
    src.write_text(DIRECT_LDS)
    subprocess.run(["g++", "-O2", "-std=c++17", "-Wall", "-Werror", f"-I{CSRC}", "-o", str(exe), str(src)], check=True)
    out = subprocess.run([str(exe)], capture_output=True, text=True, timeout=120)
    assert out.returncode == 0, out.stdout
    assert out.stdout.split() == ["15", "layouts"], out.stdout


DIRECT_READS = r"""
#include <cstdio>
#include <cstddef>
#include <initializer_list>
#include "cover.h"
using namespace spark;
int main() {
  long reads = 0, tiles = 0;
  for (int n_in = 8; n_in <= 2200; n_in += 8)
    for (int op_rows : {32, 48})
      for (int m : {1, 5, 32, op_rows}) {
        const size_t bytes = sizeof(float) * (size_t)op_rows * n_in;
        const int steps = 2 * ceil_div(n_in, MG_KC);
        for (int step = 0; step < steps; ++step)
          for (int kq = 0; kq < 4; ++kq) {
            const int s = direct_x_step(step, n_in), quad = direct_x_quad(kq, s, n_in), k = 32 * step + 8 * kq;
            // as the kernel forms it: a part of the lane, of which no step makes a negative one, and a scalar one
            const long lane = (long)quad * 16 * op_rows + (m - 1) * 16, at = (long)s * 128 * op_rows;
            for (int i = 0; i < 2; ++i, ++reads) {
              const long byte = at + i * 16 * op_rows + lane;
              if (quad < 0 || s < 0 || byte < 0 || (size_t)byte + 16 > bytes) { printf("k %d of %d, %d rows: byte %ld of %zu\n", k, n_in, m, byte, bytes); return 1; }
              if (k < n_in && byte != ((long)(k / 4 + i) * op_rows + m - 1) * 16) { printf("k %d of %d, %d rows: byte %ld\n", k, n_in, m, byte); return 1; }
              if ((byte / 16) % op_rows != m - 1) { printf("k %d of %d: another row than %d\n", k, n_in, m - 1); return 1; }
            }
          }
      }
  for (int n_blocks = 1; n_blocks <= 1200; ++n_blocks)
    for (int nt = 1; nt <= 5; ++nt)
      for (int group = 0; group < ceil_div(n_blocks, nt); ++group)
        for (int q = 0; q < nt; ++q, ++tiles) {
          const int tile = group * nt + direct_w_tile(q, group * nt, n_blocks), want = group * nt + q < n_blocks ? group * nt + q : n_blocks - 1;
          if (tile != want) { printf("tile %d of group %d of %d, %d blocks: %d\n", q, group, nt, n_blocks, tile); return 1; }
        }
  printf("%ld reads, %ld tiles\n", reads, tiles);
  return 0;
}
"""


def test_direct_reads_stay_inside_activations_and_weights(tmp_path):
    src, exe = tmp_path / "reads.cpp", tmp_path / "reads"
    src.write_text(DIRECT_READS)
    subprocess.run(["g++", "-O2", "-std=c++17", "-Wall", "-Werror", f"-I{CSRC}", "-o", str(exe), str(src)], check=True)
    out = subprocess.run([str(exe)], capture_output=True, text=True, timeout=120)
    assert out.returncode == 0, out.stdout
    n, n_tiles = (int(w) for w in out.stdout.split() if w.isdigit())
    assert n > 500_000 and n_tiles > 1_000_000, out.stdout


HEIGHTS = r"""
#include <cstdio>
#include "cover.h"
using namespace spark;
int main() {
  const struct { int n_in, n_tasks; bool always_cut; } shapes[] = {
      {3584, 2304, false}, {3584, 1792, true}, {18944, 1792, true}, {4096, 2304, false}, {4096, 2048, true}, {13696, 2048, true}};
  for (const auto &s : shapes) {
    for (int b = 2; b <= 32; ++b) printf("%d", narrow_row_blocks(32 * b, s.n_in, s.n_tasks, 4, s.always_cut, 256));
    printf("\n");
  }
  return 0;
}
"""


HEIGHTS_WANT = ["2343344344422443333344444442222",
                "2342222332244443344444433344444",
                "2343344344444443344444433344444",
                "2343344344422443333344444442222",
                "2343322323344444444333344444444",
                "2343344324444444444333344444444"]


def test_heights_of_the_tiles_of_prompts(tmp_path):
    """q/k/v, o and down of the two backbones, 2 to 32 blocks of 32 rows on 256 CUs: the heights decide where
    the sums over k are cut, and with it the last bits of every cache entry and how far they are from 64 bits"""
    src, exe = tmp_path / "heights.cpp", tmp_path / "heights"
    src.write_text(HEIGHTS)
    subprocess.run(["g++", "-O2", "-std=c++17", "-Wall", "-Werror", f"-I{CSRC}", "-o", str(exe), str(src)], check=True)
    out = subprocess.run([str(exe)], capture_output=True, text=True, timeout=120)
    assert out.stdout.split() == HEIGHTS_WANT


def test_partial_sums_of_every_cover_fit_their_buffer(tmp_path):
    src, exe = tmp_path / "covers.cpp", tmp_path / "covers"
    src.write_text(DRIVER)
    subprocess.run(["g++", "-O2", "-std=c++17", "-Wall", "-Werror", f"-I{CSRC}", "-o", str(exe), str(src)], check=True)
    out = subprocess.run([str(exe)], capture_output=True, text=True, timeout=120)
    assert out.returncode == 0, out.stdout
    n, n_cut, n_mixed = (int(w) for w in out.stdout.split() if w.isdigit())
    assert n > 500_000 and n_cut > 100_000 and n_mixed > 1000, out.stdout
