// gm_gemm_16bit.hip -- 16-bit products (M > 16): the tile kernels of one
// storage type and one group of tile shapes.  Compiled once per GM_T (0 bf16, 1
// f16) and GM_GROUP (the kernels are large; the groups compile in parallel).
#include "gm_gemm_16bit.h"
#include "gm_gemm_tile.h"

namespace gm {

#if GM_T == 0
typedef bf16_t GmT;
#else
typedef f16_t GmT;
#endif

template <> void Tiles16<GM_T, GM_GROUP>::run(int tile, const GemmArgs& a, hipStream_t s) {
#if GM_GROUP == 0
  run_pp<GmT, 256, 256, 2, 4, 2, 2>(a, s);
#elif GM_GROUP == 1
  run_pp<GmT, 256, 192, 4, 2, 2, 2>(a, s);
#elif GM_GROUP == 2
  if (tile == kT256x128) return run_pp<GmT, 256, 128, 4, 2, 1, 3>(a, s);
  if (tile == kT128x256) return run_pp<GmT, 128, 256, 2, 4, 1, 3>(a, s);
  run_pp<GmT, 128, 128, 2, 4, 1, 4>(a, s);
#else
  if (tile == kT128x64) return run_ring<GmT, 128, 64, 2, 2, 2, 64, 3>(a, s);
  if (tile == kT64x64) return run_ring<GmT, 64, 64, 2, 2, 2, 64, 4>(a, s);
  if (tile == kT64x32) return run_ring<GmT, 64, 32, 2, 1, 4, 128, 4>(a, s);
  run_ring<GmT, 32, 32, 1, 1, 4, 128, 5>(a, s);
#endif
}

}  // namespace gm
