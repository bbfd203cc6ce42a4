// gm_gemm_skinny.hip -- GEMMs of a few rows (M <= 16: a decode step or a tiny
// forward): weight-streaming kernels.
#include "gm_gemm_epilogue.h"

namespace gm {

// ------------------------------------------------------------ M <= 16 kernel
// A decode step multiplies B <= 16 rows by the whole weight: the work is the
// stream of weight bytes, so the kernel is laid out for HBM, not for MFMA.
// Workgroup = 8 wavefronts; wavefront w streams R consecutive packed weight
// rows with 16-byte coalesced loads, every lane covering a slice of K for
// all MP activation rows (read through L1/L2).  R = 4 (32 rows: a 16-row
// pair group) for the gated and rotary epilogues, R = 1 (8 rows, four times
// the workgroups) for the others.  The 64 lanes' partial sums are reduced by
// a transposing butterfly (each step halves the values a lane carries), the
// results meet in LDS, and wavefront 0 runs the same epilogue as the tiled
// kernel.
template <int NV>
__device__ __forceinline__ float lane_transpose_sum(float (&v)[NV], int lane, int& index) {
  index = 0;
  static_for<0, 6>([&](auto st) {
    constexpr int o = 32 >> decltype(st)::value;
    constexpr int n = NV >> decltype(st)::value;
    if constexpr (n >= 2) {
      constexpr int half = n / 2;
      const bool up = (lane & o) != 0;
#pragma unroll
      for (int j = 0; j < half; ++j) {
        const float send = up ? v[j] : v[j + half];
        const float keep = up ? v[j + half] : v[j];
        v[j] = keep + __shfl_xor(send, o, 64);
      }
      if (up) index += half;
    } else {
      v[0] += __shfl_xor(v[0], o, 64);
    }
  });
  return v[0];
}

template <typename T, int MP, int R>
__global__ __launch_bounds__(512) void k_gemm_skinny(GemmArgs a) {
  constexpr int VN = 16 / static_cast<int>(sizeof(T));
  constexpr int ROWS = 8 * R;               // weight rows per workgroup
  typedef typename std::conditional<sizeof(T) == 4, f32x4v, u32x4>::type V;
  __shared__ float res[ROWS][MP + 1];
  const int n0 = blockIdx.x * ROWS;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const T* W = static_cast<const T*>(a.W);
  const T* A = static_cast<const T*>(a.A);
  const T* wrow[R];
#pragma unroll
  for (int r = 0; r < R; ++r) {
    int n = n0 + wave * R + r;
    n = n < a.N ? n : a.N - 1;
    wrow[r] = W + static_cast<long long>(n) * a.ldw;
  }
  const T* arow[MP];
#pragma unroll
  for (int m = 0; m < MP; ++m) arow[m] = A + static_cast<long long>(m < a.M ? m : a.M - 1) * a.lda;
  float acc[R * MP];
#pragma unroll
  for (int j = 0; j < R * MP; ++j) acc[j] = 0.f;
#pragma unroll 2
  for (int k = lane * VN; k < a.K; k += 64 * VN) {
    float w[R][VN];
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const V raw = *reinterpret_cast<const V*>(wrow[r] + k);
      const T* e = reinterpret_cast<const T*>(&raw);
#pragma unroll
      for (int i = 0; i < VN; ++i) w[r][i] = to_f32(e[i]);
    }
#pragma unroll
    for (int m = 0; m < MP; ++m) {
      const V raw = *reinterpret_cast<const V*>(arow[m] + k);
      const T* e = reinterpret_cast<const T*>(&raw);
#pragma unroll
      for (int i = 0; i < VN; ++i) {
        const float x = to_f32(e[i]);
#pragma unroll
        for (int r = 0; r < R; ++r) acc[r * MP + m] = fmaf(w[r][i], x, acc[r * MP + m]);
      }
    }
  }
  int idx;
  const float sum = lane_transpose_sum<R * MP>(acc, lane, idx);
  // lanes that differ only in their low bits hold the same value
  if ((lane & (64 / (R * MP) - 1)) == 0) res[wave * R + idx / MP][idx % MP] = sum;
  __syncthreads();
  if (wave != 0) return;
  SiteMax sm;
  if (R == 4) {
    // a 16-row pair group: packed rows n0 + 4q + r and n0 + 16 + 4q + r
    const int m = lane >> 2, q = lane & 3;
    if (m < MP && m < a.M) {
      float va[4], vb[4];
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        va[r] = res[4 * q + r][m];
        vb[r] = res[16 + 4 * q + r][m];
      }
      epi_pair<T>(a, m, n0 + 4 * q, va, vb, sm);
    }
  } else {
    // independent columns: 8 rows as two groups of 4; the partner columns
    // the pair epilogue would also write lie beyond this workgroup's N
    GemmArgs b = a;
    b.N = a.N - n0 < ROWS ? a.N : n0 + ROWS;
    const int m = lane >> 1, q = lane & 1;
    if (m < MP && m < a.M) {
      float va[4], vb[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int r = 0; r < 4; ++r) va[r] = res[4 * q + r][m];
      epi_pair<T>(b, m, n0 + 4 * q, va, vb, sm);
    }
  }
  site_flush(a, sm);
}

// Independent-column epilogues on a narrow output: workgroup = 8 weight
// rows, and the 8 wavefronts split K instead of the rows, each covering all
// 8 rows for its K slice, so every lane's loads (8 weight and MP activation
// vectors per step) leave together and a short K needs a single round trip
// to memory.  Lane partials are reduced by the transposing butterfly, the 8
// wavefronts' sums are added in LDS.
template <typename T, int MP>
__global__ __launch_bounds__(512) void k_gemm_skinny_ks(GemmArgs a) {
  constexpr int VN = 16 / static_cast<int>(sizeof(T));
  constexpr int R = 8;
  typedef typename std::conditional<sizeof(T) == 4, f32x4v, u32x4>::type V;
  __shared__ float part[8][R * MP];
  __shared__ float res[R][MP + 1];
  const int n0 = blockIdx.x * R;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const T* W = static_cast<const T*>(a.W);
  const T* A = static_cast<const T*>(a.A);
  // this wavefront's K slice, a multiple of VN
  const int per = ((a.K + 8 * VN - 1) / (8 * VN)) * VN;
  const int kb = wave * per, ke = min(a.K, kb + per);
  const T* wrow[R];
#pragma unroll
  for (int r = 0; r < R; ++r) {
    int n = n0 + r;
    n = n < a.N ? n : a.N - 1;
    wrow[r] = W + static_cast<long long>(n) * a.ldw;
  }
  const T* arow[MP];
#pragma unroll
  for (int m = 0; m < MP; ++m) arow[m] = A + static_cast<long long>(m < a.M ? m : a.M - 1) * a.lda;
  float acc[R * MP];
#pragma unroll
  for (int j = 0; j < R * MP; ++j) acc[j] = 0.f;
  for (int k = kb + lane * VN; k < ke; k += 64 * VN) {
    V wv[R], av[MP];
#pragma unroll
    for (int r = 0; r < R; ++r) wv[r] = *reinterpret_cast<const V*>(wrow[r] + k);
#pragma unroll
    for (int m = 0; m < MP; ++m) av[m] = *reinterpret_cast<const V*>(arow[m] + k);
#pragma unroll
    for (int m = 0; m < MP; ++m) {
      const T* ae = reinterpret_cast<const T*>(&av[m]);
#pragma unroll
      for (int i = 0; i < VN; ++i) {
        const float x = to_f32(ae[i]);
#pragma unroll
        for (int r = 0; r < R; ++r)
          acc[r * MP + m] = fmaf(to_f32(reinterpret_cast<const T*>(&wv[r])[i]), x, acc[r * MP + m]);
      }
    }
  }
  int idx;
  const float sum = lane_transpose_sum<R * MP>(acc, lane, idx);
  if ((lane & (64 / (R * MP) - 1)) == 0) part[wave][idx] = sum;
  __syncthreads();
  if (threadIdx.x < R * MP) {
    float t = 0.f;
#pragma unroll
    for (int w2 = 0; w2 < 8; ++w2) t += part[w2][threadIdx.x];
    res[threadIdx.x / MP][threadIdx.x % MP] = t;
  }
  __syncthreads();
  if (wave != 0) return;
  SiteMax sm;
  GemmArgs b = a;
  b.N = a.N - n0 < R ? a.N : n0 + R;
  const int m = lane >> 1, q = lane & 1;
  if (m < MP && m < a.M) {
    float va[4], vb[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int r = 0; r < 4; ++r) va[r] = res[4 * q + r][m];
    epi_pair<T>(b, m, n0 + 4 * q, va, vb, sm);
  }
  site_flush(a, sm);
}

// A few rows (M <= 16) against a wide plain output (the LM head of a
// decode step): the 2 M N K multiply-adds on the matrix cores instead of
// the VALU.  Each wavefront computes 16 output columns for every row with
// v_mfma_f32_16x16x32 (16 weight rows as the A operand, the activation rows
// padded to 16 as the B operand; lane l supplies row l % 16 and k
// 8 (l / 16) .. + 7 of each 32-wide k step), 8 k steps of loads in flight,
// and ends with columns 4 (l / 16) .. + 3 of activation row l % 16.
template <typename T> struct Mfma16;
template <> struct Mfma16<bf16_t> {
  typedef bf16x8 vec;
  static __device__ __forceinline__ f32x4 run(vec a, vec b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
  }
};
template <> struct Mfma16<f16_t> {
  typedef f16x8 vec;
  static __device__ __forceinline__ f32x4 run(vec a, vec b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_f16(a, b, c, 0, 0, 0);
  }
};

template <typename T>
__global__ __launch_bounds__(256) void k_gemm_skinny_mfma(GemmArgs a) {
  typedef typename Mfma16<T>::vec vec;
  constexpr int U = 8;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int n0 = (blockIdx.x * 4 + wave) * 16;
  if (n0 >= a.N) return;                     // no barrier in this kernel
  const int l16 = lane & 15, kg = lane >> 4;
  const int n = n0 + l16 < a.N ? n0 + l16 : a.N - 1;
  const int m = l16 < a.M ? l16 : a.M - 1;
  const T* wp = static_cast<const T*>(a.W) + static_cast<long long>(n) * a.ldw + 8 * kg;
  const T* xp = static_cast<const T*>(a.A) + static_cast<long long>(m) * a.lda + 8 * kg;
  f32x4 acc = {0.f, 0.f, 0.f, 0.f};
  int k = 0;
  for (; k + 32 * U <= a.K; k += 32 * U) {
    vec wf[U], xf[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      wf[u] = *reinterpret_cast<const vec*>(wp + k + 32 * u);
      xf[u] = *reinterpret_cast<const vec*>(xp + k + 32 * u);
    }
#pragma unroll
    for (int u = 0; u < U; ++u) acc = Mfma16<T>::run(wf[u], xf[u], acc);
  }
  for (; k < a.K; k += 32)
    acc = Mfma16<T>::run(*reinterpret_cast<const vec*>(wp + k), *reinterpret_cast<const vec*>(xp + k),
                         acc);
  SiteMax sm;
  GemmArgs b = a;
  b.N = a.N - n0 < 16 ? a.N : n0 + 16;       // the pair columns (+16) lie beyond this wavefront's
  const float va[4] = {acc[0], acc[1], acc[2], acc[3]};
  const float vb[4] = {0.f, 0.f, 0.f, 0.f};
  epi_pair<T>(b, l16, n0 + 4 * kg, va, vb, sm);
  site_flush(a, sm);
}

template <typename T>
static void skinny_ks(const GemmArgs& a, hipStream_t s) {
  const dim3 grid((a.N + 7) / 8), block(512);
  if (a.M <= 1) hipLaunchKernelGGL((k_gemm_skinny_ks<T, 1>), grid, block, 0, s, a);
  else if (a.M <= 2) hipLaunchKernelGGL((k_gemm_skinny_ks<T, 2>), grid, block, 0, s, a);
  else if (a.M <= 4) hipLaunchKernelGGL((k_gemm_skinny_ks<T, 4>), grid, block, 0, s, a);
  else hipLaunchKernelGGL((k_gemm_skinny_ks<T, 8>), grid, block, 0, s, a);
}

template <typename T, int R>
static void skinny_r(const GemmArgs& a, hipStream_t s) {
  const dim3 grid((a.N + 8 * R - 1) / (8 * R)), block(512);
  if (a.M <= 1) hipLaunchKernelGGL((k_gemm_skinny<T, 1, R>), grid, block, 0, s, a);
  else if (a.M <= 2) hipLaunchKernelGGL((k_gemm_skinny<T, 2, R>), grid, block, 0, s, a);
  else if (a.M <= 4) hipLaunchKernelGGL((k_gemm_skinny<T, 4, R>), grid, block, 0, s, a);
  else if (a.M <= 8) hipLaunchKernelGGL((k_gemm_skinny<T, 8, R>), grid, block, 0, s, a);
  else hipLaunchKernelGGL((k_gemm_skinny<T, 16, R>), grid, block, 0, s, a);
}

template <typename T>
static void skinny_t(const GemmArgs& a, hipStream_t s) {
  // the gated and rotary epilogues combine packed rows 16 apart; a wide
  // output (the head) has workgroups enough with 32 rows each, and four rows
  // per wavefront reuse every activation load four times
  // a wide plain output (the head) in 16-bit on the matrix cores
  if constexpr (sizeof(T) == 2) {
    if (a.epi == kEpiStore && !a.bias && a.site < 0 && !a.kc && a.N >= 8192 && a.K % 32 == 0) {
      hipLaunchKernelGGL((k_gemm_skinny_mfma<T>), dim3((a.N + 63) / 64), dim3(256), 0, s, a);
      return;
    }
  }
  if (a.epi == kEpiGatedGelu || a.epi == kEpiGatedSilu || a.epi == kEpiRope || a.N >= 8192)
    skinny_r<T, 4>(a, s);
  else if (a.M <= 8 && a.N < 2048)     // few row groups: split K across the wavefronts
    skinny_ks<T>(a, s);
  else
    skinny_r<T, 1>(a, s);
}
void gemm_skinny(const GemmArgs& a, hipStream_t s) {
  if (a.dtype == kF32) skinny_t<float>(a, s);
  else if (a.dtype == kBF16) skinny_t<bf16_t>(a, s);
  else skinny_t<f16_t>(a, s);
}

}  // namespace gm
