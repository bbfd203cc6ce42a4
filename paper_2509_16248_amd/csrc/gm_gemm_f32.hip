// gm_gemm_f32.hip -- fp32 products (M > 16) on v_mfma_f32_32x32x2_f32.
#include "gm_gemm_tile.h"

namespace gm {

// One MFMA takes 64 clocks for 512 bytes of operands, so the loop is bound by
// the matrix cores at any tile: 64 x 64 tiles with 8 wavefronts in pairs that
// split K (800 x 50257 x 768: 578 us, 107 TFLOP/s; the former VALU kernel
// 1908 us), and where those give fewer than two workgroups per CU, 32 x 32
// tiles whose 4 wavefronts split K (800 x 768 x 3072: 51.7 us against 60.3 with
// 64 x 64 tiles and 427 on the VALU).  At 468 tiles (800 x 2304 x 768) the two
// are equal: 32.9 and 34.5 us.
void gemm_f32(const GemmArgs& a, hipStream_t s) {
  const long long tiles = ((a.M + 63) / 64) * static_cast<long long>((a.N + 63) / 64);
  if (tiles < 400) run_ring<float, 32, 32, 1, 1, 4, 32, 4>(a, s);
  else run_ring<float, 64, 64, 2, 2, 2, 32, 3>(a, s);
}

}  // namespace gm
