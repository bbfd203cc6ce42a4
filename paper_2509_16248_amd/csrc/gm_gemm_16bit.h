// gm_gemm_16bit.h -- the tile shapes of the 16-bit products.
#pragma once
#include "gm_kernels.h"

namespace gm {

enum Tile16 : int {
  kT256x256,                                  // group 0
  kT256x192,                                  // group 1
  kT256x128, kT128x256, kT128x128,            // group 2
  kT128x64, kT64x64, kT64x32, kT32x32,        // group 3
  kTiles16
};

// One storage type's kernels of a group of tile shapes (gm_gemm_16bit.hip).
template <int DTYPE, int GROUP>
struct Tiles16 {
  static void run(int tile, const GemmArgs& a, hipStream_t s);
};

}  // namespace gm
