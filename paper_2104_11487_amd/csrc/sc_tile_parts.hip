// Tile kernel builds that sum K in short chains (kernel: sc_tile_kernel.h): bf16
// layers that the register-operand kernel takes on smaller frames. That kernel
// splits K over its waves and adds 2, 4 or 8 partial sums; one MFMA chain over
// all of K leaves z 1.4 to 2.3 times as far from the exact sums (64 -> 64, 3 x 3:
// 1.33e-7 of its norm against 7.6e-8; 32 -> 64 9.2e-8 against 6.2e-8). Here a
// chain runs over FL k-steps and its sum is added to the total (7.6e-8, 6.2e-8).
// The second set of accumulators leaves no registers for z_{t-1} beside four
// column tiles, so it is loaded late; a step takes about 5 % longer than with one
// chain (64 -> 64, 8 x 8 blocks, 256 x 256, 15 % covered: 16.0 -> 17.4 us, 200 x 200
// 15.5 -> 16.3; by the register-operand kernel 23.2 and 17.6).
#include "sc_tile_kernel.h"

namespace sc {

namespace {

// Columns as in SC_TILE_BUILDS; FL is the ring size KR. (Frames on which these
// layers would take 16 x 16 tiles stay with the register-operand kernel.)
#define SC_TILE_BUILDS_PARTS(X)                                                                         \
  X(8, 16, 2, 4, 1, 2, 2, 3, false, 3, 4, 4) X(8, 16, 4, 2, 2, 4, 2, 2, true, 2, 4, 3)                  \
  X(8, 16, 8, 2, 4, 4, 2, 2, true, 2, 4, 3)

const TileBuild kPartsBuilds[] = {
#define SC_X(rows, cols, ntn, a, b, wm, wn, kr, zi, krt, occ, ki)                                      \
  {rows, cols, ntn, 64 * a * b, tile_kernel<a, b, wm, wn, kr, occ, ki, zi, false, false, 0, false, kr>, \
   tile_kernel<a, b, wm, wn, krt, occ, ki, true, true, false, 0, false, krt>,                           \
   tile_kernel<a, b, wm, wn, kr, occ, ki, zi, false, true, 0, false, kr>,                               \
   tile_kernel<a, b, wm, wn, kr, occ, kLearnItems(rows, a * b), zi, false, false, 1, false, kr>,        \
   tile_kernel<a, b, wm, wn, kr, occ, kLearnItems(rows, a * b), zi, false, false, 3, false, kr>,        \
   tile_kernel<a, b, wm, wn, kr, occ, kLearnItems(rows, a * b), zi, false, true, 1, false, kr>,         \
   tile_kernel<a, b, wm, wn, kr, occ, kLearnItems(rows, a * b), zi, false, true, 3, false, kr>},
    SC_TILE_BUILDS_PARTS(SC_X)
#undef SC_X
};

}  // namespace

const TileBuild* tile_parts_builds(int* count) {
  *count = (int)(sizeof(kPartsBuilds) / sizeof(kPartsBuilds[0]));
  return kPartsBuilds;
}

}  // namespace sc
