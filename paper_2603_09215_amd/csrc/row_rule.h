// When the layers of a pass of one row are better in one launch (one_row.h), and their numbers; plain arithmetic, no device code.
#pragma once
#include <algorithm>
#include <cstddef>

namespace spark {

// A cooperative launch costs some 25 us more than a plain one, and a layer gains what its bytes leave of its five launches'
// ends after its hand-overs, which cost the same whatever its size.  Measured, us a step gained at 100, 1500 and 1900
// tokens (28 query heads of 4 and width 3584; 408 MB: 32 of 2 and 4096):
//   layers   189 MB          198 MB          209 MB         229 MB         294 MB    408 MB    466 MB
//   3        -               -1, -3          -              -              9, 5      15, 10    18, 13
//   4        -1, -4, 5       6, 3, 10        5, 1, 10       8, 6, 15       20, 15    29, 26    32, 26
//   6        -               21, 17          -              -              47, 34    54, 52    59, 51
//   8        22, 16, 32      34, 29, 45      31, 25, 41     39, 34, 51     62, 54    80, 77    86, 73
// of 240 us (four layers of 189 MB) to 810 (eight of 466).  Of width 4096 with 32 heads of 2, four layers: 189 MB 3, -3, -4;
// 199 MB 5, 0, -1; 209 MB 10, 4, 1.  162 MB of width 3584: 13 and 6 at eight layers, 41 and 28 at fourteen; narrower
// layers gain more, but not where eight key heads need all workgroups for their slices (2048 wide, 189 to 213 MB, 1900
// tokens: 0 at four layers and -1 to -2 of 480 to 510 at eight).
constexpr size_t ROW_LAYER_BYTES = (size_t)180 << 20;
inline bool one_row_pays(size_t layer_bytes, int layers) {
  const double gain = std::min(7.0, ((double)layer_bytes * 1e-6 - 140.0) * 0.1);   // us a layer, low
  return layer_bytes >= ROW_LAYER_BYTES && layers * gain >= 28.0;                  // the launch, high
}

// Layers are numbered from 1 over all launches of a context; whether the numbers end before those of the next launch, so that
// they begin again (on cleared words: an old one would be taken for a new one)
inline bool row_numbers_run_out(unsigned last, unsigned layers) { return last + layers < last; }

}  // namespace spark
