// gm_gemm_f32.hip -- fp32 products (M > 16) on v_mfma_f32_32x32x2_f32.
#include "gm_gemm_tile.h"

namespace gm {

// One MFMA takes 64 clocks for 512 bytes of operands, so the loop is bound by
// the matrix cores at any tile: 64 x 64 tiles with 8 wavefronts in pairs that
// split K (800 x 50257 x 768: 578 us, 107 TFLOP/s; the former VALU kernel
// 1908 us), and where those would be fewer than 400, 32 x 32 tiles whose 4
// wavefronts split K: at 156 tiles (800 x 768 x 3072) 51.7 us against 60.3 with
// 64 x 64 tiles and 427 on the VALU; at 468 tiles (800 x 2304 x 768) the two
// are equal, 32.9 and 34.5 us.
void gemm_f32(const GemmArgs& a, hipStream_t s) {
  const long long tn = (a.N + 63) / 64, tiles = (a.M + 63) / 64 * tn;
  if (tiles < 400) return run_ring<float, 32, 32, 1, 1, 4, 32, 4>(a, s);
  // a launch has fewer than 2^32 threads: logits of more than 137 GB leave in
  // parts of whole tile rows
  constexpr long long kMostTiles = (1ll << 32) / 512 - 1;
  if (tiles <= kMostTiles || a.epi != kEpiStore || a.kc)
    return run_ring<float, 64, 64, 2, 2, 2, 32, 3>(a, s);
  const long long rows = kMostTiles / tn * 64;
  for (long long m = 0; m < a.M; m += rows) {
    GemmArgs b = a;
    b.M = static_cast<int>(a.M - m < rows ? a.M - m : rows);
    b.A = static_cast<const float*>(a.A) + m * a.lda;
    b.out = static_cast<float*>(a.out) + m * a.ldo;
    run_ring<float, 64, 64, 2, 2, 2, 32, 3>(b, s);
  }
}

}  // namespace gm
