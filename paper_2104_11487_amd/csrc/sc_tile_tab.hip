// Tile kernel builds for bf16 layers of other than 32, 64 or 128 input channels
// (a multiple of 8): the halo offsets of K through a table (sc_halo_conv.h, TAB).
#include "sc_tile_kernel.h"

namespace sc {

namespace {

// Other than 32, 64 or 128 input channels (TAB): also 8 x 8 tiles and up to 256
// output channels, since the only other convolution of C_in % 32 != 0 gathers
// site by site.
#define SC_TILE_BUILDS_TAB(X)                                                                             \
  SC_TILE_BUILDS(X) X(8, 16, 12, 2, 4, 4, 3, 2, true, 2, 2, 3) X(8, 16, 16, 2, 4, 4, 4, 2, true, 2, 2, 3) \
  X(8, 8, 1, 4, 1, 1, 1, 4, false, 4, 4, 4) X(8, 8, 2, 4, 1, 1, 2, 4, false, 4, 4, 4)                     \
  X(8, 8, 4, 2, 2, 2, 2, 4, false, 4, 4, 4) X(8, 8, 8, 2, 4, 2, 2, 4, false, 4, 4, 3)                     \
  X(8, 8, 12, 2, 4, 2, 3, 2, false, 2, 4, 3) X(8, 8, 16, 2, 4, 2, 4, 2, false, 2, 4, 3)

const TileBuild kTabBuilds[] = {
#define SC_X(rows, cols, ntn, a, b, wm, wn, kr, zi, krt, occ, ki)                                \
  {rows, cols, ntn, 64 * a * b, tile_kernel<a, b, wm, wn, kr, occ, ki, zi, false, false, 0, true>, \
   tile_kernel<a, b, wm, wn, krt, occ, ki, true, true, false, 0, true>,                            \
   tile_kernel<a, b, wm, wn, kr, occ, ki, zi, false, true, 0, true>, nullptr, nullptr, nullptr, nullptr},
    SC_TILE_BUILDS_TAB(SC_X)
#undef SC_X
};

}  // namespace

const TileBuild* tile_tab_builds(int* count) {
  *count = (int)(sizeof(kTabBuilds) / sizeof(kTabBuilds[0]));
  return kTabBuilds;
}

}  // namespace sc
