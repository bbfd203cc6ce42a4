// gm_gemm.hip -- out = epilogue(A . W^T) for the projections and the head.
//
// A is [M, K] (activations, row-major), W is [N, K] (nn.Linear weight
// layout, row-major): both operands are contiguous along K, which is the
// operand layout the matrix cores read.  K is a multiple of 64.  Everything
// runs on gfx950 MFMA with fp32 accumulation (fp32 models: fp32 MFMA); all
// epilogues work on fp32 accumulators and round once to the storage dtype.
// The kernels are in gm_gemm_16bit.hip and gm_gemm_f32.hip, those of a few rows
// in gm_gemm_skinny.hip.
#include "gm_gemm_16bit.h"

namespace gm {

void gemm_skinny(const GemmArgs& a, hipStream_t s);
void gemm_f32(const GemmArgs& a, hipStream_t s);

// Every tile shape is priced as (waves of 256 workgroups) x (K / 64 x stage +
// fixed): `stage` is a tile's time per 64 columns of K with the chip full,
// `fixed` its launch, first loads and epilogue, both in units of 10 ns as
// measured on one MI355X.  Where the lines lie (us, this tile / the next best):
//   256 x 256: 777 x 32000 x 4096 218 / 234, 4096 x 32000 x 1024 256 / 276,
//              4096 x 50257 x 768 384 / 400, 8192 x 4096 x 1024 85 / 95
//   256 x 192: 777 x 22016 x 4096 156 / 175, 2048 x 12288 x 4096 178 / 200
//   256 x 128: 2048 x 4096 x 11008 172 / 186, 8192 x 1024 x 1024 24 / 29
//   128 x 256: as 256 x 128 where M leaves half of its rows empty
//   128 x 128: 4096 x 768 x 3072 27 / 34, 777 x 4096 x 11008 88 / 123
//   128 x 64:  128 x 12288 x 4096 39.5 / 43.8
//   64 x 64:   1024 x 768 x 3072 14.8 / 17.2, 519 x 1024 x 4096 16.8 / 20.9
//   64 x 32:   128 x 4096 x 4096 16.2 / 19.5
//   32 x 32:   37 x 768 x 3072 7.8 / 9.2
// Every tile multiplies the same k in the same order of MFMAs per accumulator
// except the K-splitting ones (128 x 64 and smaller), whose partial sums are
// added at the end.
struct TilePrice {
  int bm, bn, stage, fixed;
};
static constexpr TilePrice kPrice[kTiles16] = {
    {256, 256, 152, 1000}, {256, 192, 114, 850}, {256, 128, 92, 700}, {128, 256, 93, 700},
    {128, 128, 50, 500},   {128, 64, 34, 450},   {64, 64, 22, 400},   {64, 32, 18, 350},
    {32, 32, 10, 300},
};

static int choose_tile(int M, int N, int K) {
  int best = -1;
  long long least = 0;
  for (int i = 0; i < kTiles16; ++i) {
    const TilePrice& t = kPrice[i];
    if (t.bn == 32 && K % 128) continue;   // the narrow tiles step K by 128
    const long long tiles = ((M + t.bm - 1) / t.bm) * static_cast<long long>((N + t.bn - 1) / t.bn);
    const long long price = (tiles + 255) / 256 * (K / 64 * t.stage + t.fixed);
    if (best < 0 || price < least) {
      best = i;
      least = price;
    }
  }
  return best;
}

template <int DTYPE>
static void gemm_16bit(const GemmArgs& a, hipStream_t s) {
  const int t = choose_tile(a.M, a.N, a.K);
  if (t == kT256x256) Tiles16<DTYPE, 0>::run(t, a, s);
  else if (t == kT256x192) Tiles16<DTYPE, 1>::run(t, a, s);
  else if (t <= kT128x128) Tiles16<DTYPE, 2>::run(t, a, s);
  else Tiles16<DTYPE, 3>::run(t, a, s);
}

void launch_gemm(const GemmArgs& a, hipStream_t s) {
  if (a.M <= 16) gemm_skinny(a, s);
  else if (a.dtype == kF32) gemm_f32(a, s);
  else if (a.dtype == kBF16) gemm_16bit<0>(a, s);
  else gemm_16bit<1>(a, s);
}

}  // namespace gm
