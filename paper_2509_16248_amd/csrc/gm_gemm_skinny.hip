// gm_gemm_skinny.hip -- products of a few rows (M <= 16: a decode step or a
// tiny forward), optionally with the norm of their input rows.
#include "gm_gemm_epilogue.h"

namespace gm {

// v_mfma_f32_16x16x32 of 16 weight rows (A operand) and up to 16 activation
// rows (B operand): lane l supplies 16 bytes of row l % 16 at k-chunk l / 16 of
// a step, and ends with output columns 4 (l / 16) .. + 3 of activation row
// l % 16.  fp32: four v_mfma_f32_16x16x4 per step, MFMA r taking element r of
// every lane's four, in steps that alternate between two sets of four sums (a
// sum in one chain rounds eight times as often in a row).
template <typename T> struct Mfma16;
template <> struct Mfma16<bf16_t> {
  typedef bf16x8 vec;
  static constexpr int kSums = 1;
  static __device__ __forceinline__ void run(vec a, vec b, f32x4* c, int) {
    c[0] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c[0], 0, 0, 0);
  }
};
template <> struct Mfma16<f16_t> {
  typedef f16x8 vec;
  static constexpr int kSums = 1;
  static __device__ __forceinline__ void run(vec a, vec b, f32x4* c, int) {
    c[0] = __builtin_amdgcn_mfma_f32_16x16x32_f16(a, b, c[0], 0, 0, 0);
  }
};
template <> struct Mfma16<float> {
  typedef f32x4 vec;
  static constexpr int kSums = 8;
  static __device__ __forceinline__ void run(vec a, vec b, f32x4* c, int step) {
    c += 4 * step;
#pragma unroll
    for (int r = 0; r < 4; ++r) c[r] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[r], b[r], c[r], 0, 0, 0);
  }
};

constexpr int kRowsWaves = 8;

// Rows of x normalised into LDS (pitch elements apart), one wavefront per
// row: the arithmetic of the row kernel (fp32 and bf16: the same bits; in fp16
// the compiler joins the last multiply-add with its rounding in some places and
// not in others, so a last bit may differ).
template <typename T, int MAXV>
__device__ __forceinline__ void norm_to_lds(const GemmArgs& a, T* lds, int pitch, int wave, int lane) {
  typedef typename std::conditional<sizeof(T) == 4, f32x4v, u32x4>::type V;
  constexpr int VN = 16 / static_cast<int>(sizeof(T));
  const int d = a.K, nvec = d / VN;
  const T* g = static_cast<const T*>(a.norm_g);
  const T* bb = static_cast<const T*>(a.norm_b);
  for (int row = wave; row < a.M; row += kRowsWaves) {
    const T* x = static_cast<const T*>(a.A) + static_cast<long long>(row) * a.lda;
    V raw[MAXV], graw[MAXV], braw[MAXV];
#pragma unroll
    for (int j = 0; j < MAXV; ++j) {
      const int c = lane + 64 * j;
      if (c < nvec) {
        raw[j] = *reinterpret_cast<const V*>(x + c * VN);
        graw[j] = *reinterpret_cast<const V*>(g + c * VN);
        if (bb) braw[j] = *reinterpret_cast<const V*>(bb + c * VN);
      }
    }
    float s1 = 0.f;
    if (a.norm == 0) {
#pragma unroll
      for (int j = 0; j < MAXV; ++j)
        if (lane + 64 * j < nvec)
#pragma unroll
          for (int i = 0; i < VN; ++i) s1 += to_f32(reinterpret_cast<const T*>(&raw[j])[i]);
      s1 = wave_sum(s1);
    }
    const float mean = a.norm == 0 ? s1 / d : 0.f;
    float s2 = 0.f;
#pragma unroll
    for (int j = 0; j < MAXV; ++j)
      if (lane + 64 * j < nvec)
#pragma unroll
        for (int i = 0; i < VN; ++i) {
          const float c = to_f32(reinterpret_cast<const T*>(&raw[j])[i]) - mean;
          s2 += c * c;
        }
    s2 = wave_sum(s2);
    const float rstd = 1.0f / sqrtf(s2 / d + a.norm_eps);
#pragma unroll
    for (int j = 0; j < MAXV; ++j) {
      const int c = lane + 64 * j;
      if (c < nvec) {
        V w;
        T* we = reinterpret_cast<T*>(&w);
#pragma unroll
        for (int i = 0; i < VN; ++i) {
          const float bv = bb ? to_f32(reinterpret_cast<const T*>(&braw[j])[i]) : 0.f;
          we[i] = from_f32<T>((to_f32(reinterpret_cast<const T*>(&raw[j])[i]) - mean) * rstd *
                                  to_f32(reinterpret_cast<const T*>(&graw[j])[i]) + bv);
        }
        *reinterpret_cast<V*>(lds + row * pitch + c * VN) = w;
      }
    }
  }
}

// How a product of a few rows takes the norm of its input.
enum RowsNorm : int {
  kRowsPlain = 0,   // it does not
  kRowsLds = 1,     // rows normalised into LDS first, MAXV = 2 vectors per lane
  kRowsScaled = 2,  // RMSNorm: rows times gain are multiplied, the sums scaled
};

// The work of a few rows is the stream of weight bytes, and where those are
// few (a 768-wide model) the latency of one launch.  A workgroup computes CT
// groups of 16 output columns for every row; its 8 wavefronts take pairs of
// steps of K in turn (two steps: 128 bytes, a cache line, of each weight row;
// one step each apart: 25.8 against 20.6 us on 4096 x 11008), with two pairs in
// flight per wavefront (more leave fewer wavefronts room: 42 -> 51 us on 22016
// x 4096), and the wavefronts' sums meet in LDS.
// The norm of the input rows costs no launch of its own (3.8 - 5.2 us):
//  - up to 128 vectors per row it is computed into LDS while the first weights
//    are on their way (8 x 2304 x 768: 3.7 -> 4.7 us; for longer rows the wait
//    costs more than the launch: 1 x 22016 x 4096 42 -> 57 us);
//  - a longer RMSNorm does not come before the product at all: its gain is
//    multiplied into the rows (one rounding, as in a norm of its own), every
//    wavefront sums the squares of the elements it reads, and the finished sums
//    are scaled.  (Rows whose squares leave fp32 give 0 either way as long as
//    x g and the sums stay inside it, |x| up to about 1e36.)
// Against kernels of vector instructions that streamed whole weight rows:
// 8 x 22016 x 4096 87 -> 46 us, 8 x 2304 x 768 7.0 -> 3.5, 1 x 12288 x 4096 31 -> 27.
template <typename T, int CT, int NORM>
__global__ __launch_bounds__(64 * kRowsWaves) void k_gemm_rows(GemmArgs a) {
  typedef typename Mfma16<T>::vec vec;
  constexpr int VN = 16 / static_cast<int>(sizeof(T));
  constexpr int KC = 4 * VN;                       // k per step
  constexpr int U = 2;                             // steps per batch of loads
  extern __shared__ __attribute__((aligned(16))) char dyn[];
  __shared__ f32x4 red[kRowsWaves][CT][64];
  __shared__ float red_ss[kRowsWaves][16];
  T* xl = reinterpret_cast<T*>(dyn);
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int l16 = lane & 15, kg = lane >> 4;
  const int n0 = blockIdx.x * 16 * CT;
  const T* wp[CT];
#pragma unroll
  for (int c = 0; c < CT; ++c) {
    int n = n0 + 16 * c + l16;
    n = n < a.N ? n : a.N - 1;
    wp[c] = static_cast<const T*>(a.W) + static_cast<long long>(n) * a.ldw + kg * VN;
  }
  const int m = l16 < a.M ? l16 : a.M - 1;
  const int pitch = a.K + VN;                      // 16 rows in distinct banks
  const T* xp = NORM == kRowsLds ? xl + m * pitch + kg * VN
                                 : static_cast<const T*>(a.A) + static_cast<long long>(m) * a.lda + kg * VN;
  const T* gp = static_cast<const T*>(a.norm_g) + kg * VN;
  const int steps = a.K / KC;
  constexpr int SUMS = Mfma16<T>::kSums;
  f32x4 acc[CT][SUMS];
#pragma unroll
  for (int c = 0; c < CT; ++c)
#pragma unroll
    for (int i = 0; i < SUMS; ++i) acc[c][i] = f32x4{0.f, 0.f, 0.f, 0.f};
  float ss = 0.f;                                  // sum of squares of this lane's elements
  vec w[2][CT][U], x[2][U], gn[2][U];
  auto fetch = [&](auto set, int s0) {             // steps s0 .. s0 + U - 1
    static_for<0, U>([&](auto u) {
      const int s = s0 + u;
      if (s < steps) {
#pragma unroll
        for (int c = 0; c < CT; ++c) w[set][c][u] = *reinterpret_cast<const vec*>(wp[c] + s * KC);
        if constexpr (NORM != kRowsLds) x[set][u] = *reinterpret_cast<const vec*>(xp + s * KC);
        if constexpr (NORM == kRowsScaled) gn[set][u] = *reinterpret_cast<const vec*>(gp + s * KC);
      }
    });
  };
  auto multiply = [&](auto set, int s0) {
    static_for<0, U>([&](auto u) {
      const int s = s0 + u;
      if (s < steps) {
        if constexpr (NORM == kRowsLds) x[set][u] = *reinterpret_cast<const vec*>(xp + s * KC);
        if constexpr (NORM == kRowsScaled) {
          T* xe = reinterpret_cast<T*>(&x[set][u]);
          const T* ge = reinterpret_cast<const T*>(&gn[set][u]);
#pragma unroll
          for (int i = 0; i < VN; ++i) {
            const float v = to_f32(xe[i]);
            ss += v * v;
            xe[i] = from_f32<T>(v * to_f32(ge[i]));
          }
        }
#pragma unroll
        for (int c = 0; c < CT; ++c) Mfma16<T>::run(w[set][c][u], x[set][u], acc[c], u);
      }
    });
  };
  constexpr int B = kRowsWaves * U;                // steps per batch over the workgroup
  std::integral_constant<int, 0> s0;
  std::integral_constant<int, 1> s1;
  fetch(s0, wave * U);
  fetch(s1, wave * U + B);
  if constexpr (NORM == kRowsLds) {
    norm_to_lds<T, 2>(a, xl, pitch, wave, lane);
    __syncthreads();
  }
  for (int s = wave * U; s < steps; s += 2 * B) {
    multiply(s0, s);
    fetch(s0, s + 2 * B);
    multiply(s1, s + B);
    fetch(s1, s + 3 * B);
  }
#pragma unroll
  for (int c = 0; c < CT; ++c) {
    f32x4 t = acc[c][0];
    if constexpr (SUMS == 8)
      t = ((t + acc[c][1]) + (acc[c][2] + acc[c][3])) +
          ((acc[c][4] + acc[c][5]) + (acc[c][6] + acc[c][7]));
    red[wave][c][lane] = t;
  }
  if constexpr (NORM == kRowsScaled) {
    ss += __shfl_xor(ss, 16, 64);
    ss += __shfl_xor(ss, 32, 64);
    if (lane < 16) red_ss[wave][lane] = ss;
  }
  __syncthreads();
  constexpr int PAIRS = CT > 1 ? CT / 2 : 1;
  if (wave >= PAIRS) return;
  float scale = 1.f;
  if constexpr (NORM == kRowsScaled) {
    float t = 0.f;
#pragma unroll
    for (int v = 0; v < kRowsWaves; ++v) t += red_ss[v][l16];
    scale = 1.0f / sqrtf(t / a.K + a.norm_eps);
  }
  auto total = [&](int c) {
    f32x4 t = red[0][c][lane];
#pragma unroll
    for (int v = 1; v < kRowsWaves; ++v) t += red[v][c][lane];
    if constexpr (NORM == kRowsScaled) t *= scale;
    return t;
  };
  SiteMax sm;
  const f32x4 ta = total(CT > 1 ? 2 * wave : 0);
  const float va[4] = {ta[0], ta[1], ta[2], ta[3]};
  const int nA = n0 + 32 * wave + 4 * kg;
  if constexpr (CT > 1) {
    const f32x4 tb = total(2 * wave + 1);
    const float vb[4] = {tb[0], tb[1], tb[2], tb[3]};
    epi_pair<T>(a, l16, nA, va, vb, sm);
  } else {
    // the partner columns the pair epilogue would also write lie beyond this
    // workgroup's
    GemmArgs b = a;
    b.N = a.N - n0 < 16 ? a.N : n0 + 16;
    const float vb[4] = {0.f, 0.f, 0.f, 0.f};
    epi_pair<T>(b, l16, nA, va, vb, sm);
  }
  site_flush(a, sm);
}

// ------------------------------------------------------------ fp32, very few rows
// v_mfma_f32_16x16x4 does a sixteenth of the work of its 16-bit kin per byte of
// weights read, and with few rows of 16 in use a plain multiply-add per lane is
// no slower; what decides is how the weights arrive.  Here the 64 lanes read 1 KB
// of one weight row at a time (16 rows of 64 bytes in k_gemm_rows), and their
// partial sums are reduced by a transposing butterfly: each step halves the
// values a lane carries.
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

// The epilogue of G groups of 4 columns from n0 on, res[column][row], by one
// wavefront.  A lane's group ends the columns that the pair epilogue sees (its
// second tile would be written 16 further on).
template <int MP, int G>
__device__ __forceinline__ void lanes_epilogue(const GemmArgs& a, const float (*res)[MP + 1], int n0) {
  const int lane = threadIdx.x & 63, m = lane / G, q = lane % G, n = n0 + 4 * q;
  GemmArgs b = a;
  b.N = n + 4 < a.N ? n + 4 : a.N;
  SiteMax sm;
  if (m < MP && m < a.M) {
    float va[4];
    const float vb[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int r = 0; r < 4; ++r) va[r] = res[4 * q + r][m];
    epi_pair<float>(b, m, n, va, vb, sm);
  }
  site_flush(a, sm);
}

// A workgroup: 8 R columns, a wavefront R of them over the whole of K.
template <int MP, int R>
__global__ __launch_bounds__(512) void k_gemm_lanes(GemmArgs a) {
  constexpr int COLS = 8 * R;
  __shared__ float res[COLS][MP + 1];
  const int n0 = blockIdx.x * COLS;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const float* w[R];
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const int n = n0 + wave * R + r;
    w[r] = static_cast<const float*>(a.W) + static_cast<long long>(n < a.N ? n : a.N - 1) * a.ldw;
  }
  const float* x[MP];
#pragma unroll
  for (int m = 0; m < MP; ++m)
    x[m] = static_cast<const float*>(a.A) + static_cast<long long>(m < a.M ? m : a.M - 1) * a.lda;
  float acc[R * MP];
#pragma unroll
  for (int j = 0; j < R * MP; ++j) acc[j] = 0.f;
#pragma unroll 2
  for (int k = lane * 4; k < a.K; k += 256) {
    f32x4 wv[R];
#pragma unroll
    for (int r = 0; r < R; ++r) wv[r] = *reinterpret_cast<const f32x4*>(w[r] + k);
#pragma unroll
    for (int m = 0; m < MP; ++m) {
      const f32x4 xv = *reinterpret_cast<const f32x4*>(x[m] + k);
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int r = 0; r < R; ++r) acc[r * MP + m] = fmaf(wv[r][i], xv[i], acc[r * MP + m]);
    }
  }
  int at;
  const float sum = lane_transpose_sum<R * MP>(acc, lane, at);
  // lanes that differ only in their low bits hold the same value
  if ((lane & (64 / (R * MP) - 1)) == 0) res[wave * R + at / MP][at % MP] = sum;
  __syncthreads();
  if (wave == 0) lanes_epilogue<MP, 2 * R>(a, res, n0);
}

// A workgroup: 8 columns, every wavefront all of them over an eighth of K, so
// that a narrow output still has every load of a short K in flight at once.
template <int MP>
__global__ __launch_bounds__(512) void k_gemm_lanes_ksplit(GemmArgs a) {
  constexpr int R = 8;
  __shared__ float part[8][R * MP];
  __shared__ float res[R][MP + 1];
  const int n0 = blockIdx.x * R;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int per = (a.K + 31) / 32 * 4;             // k per wavefront, in fours
  const int kb = wave * per, ke = kb + per < a.K ? kb + per : a.K;
  const float* w[R];
#pragma unroll
  for (int r = 0; r < R; ++r)
    w[r] = static_cast<const float*>(a.W) + static_cast<long long>(n0 + r < a.N ? n0 + r : a.N - 1) * a.ldw;
  const float* x[MP];
#pragma unroll
  for (int m = 0; m < MP; ++m)
    x[m] = static_cast<const float*>(a.A) + static_cast<long long>(m < a.M ? m : a.M - 1) * a.lda;
  float acc[R * MP];
#pragma unroll
  for (int j = 0; j < R * MP; ++j) acc[j] = 0.f;
  for (int k = kb + lane * 4; k < ke; k += 256) {
    f32x4 wv[R], xv[MP];
#pragma unroll
    for (int r = 0; r < R; ++r) wv[r] = *reinterpret_cast<const f32x4*>(w[r] + k);
#pragma unroll
    for (int m = 0; m < MP; ++m) xv[m] = *reinterpret_cast<const f32x4*>(x[m] + k);
#pragma unroll
    for (int m = 0; m < MP; ++m)
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int r = 0; r < R; ++r) acc[r * MP + m] = fmaf(wv[r][i], xv[m][i], acc[r * MP + m]);
  }
  int at;
  const float sum = lane_transpose_sum<R * MP>(acc, lane, at);
  if ((lane & (64 / (R * MP) - 1)) == 0) part[wave][at] = sum;
  __syncthreads();
  if (threadIdx.x < R * MP) {
    float t = 0.f;
#pragma unroll
    for (int v = 0; v < 8; ++v) t += part[v][threadIdx.x];
    res[threadIdx.x / MP][threadIdx.x % MP] = t;
  }
  __syncthreads();
  if (wave == 0) lanes_epilogue<MP, 2>(a, res, n0);
}

// Which fp32 products of at most 8 rows go there (us, here / k_gemm_rows; the
// pair epilogues stay with k_gemm_rows, which takes their norm):
//   the head: 50257 x 768 24 / 35 with 1 row, 33 / 37 with 8; 32000 x 1024 29 /
//     35 with 8 and its norm launch; not up to 512 columns, whose norm
//     k_gemm_rows takes into LDS
//   one or two rows: 2304 x 768 4.2 / 5.1 and 4.4 / 5.0 (4 rows 5.2 / 5.2, 6
//     rows 6.8 / 5.2), 768 x 768 4.3 / 5.1 and 5.0 / 5.2 (4 rows 6.2 / 4.8)
//   narrow outputs of a long K: 768 x 3072 5.2 / 10.3 with 1 row, 8.3 / 12.4
//     with 8; 512 x 1408 6.3 / 6.9 with 8 (256 x 1024: 5.8 / 5.5 with 2)
static bool f32_by_lanes(int M, int N, int K, int epi) {
  if (epi == kEpiGatedGelu || epi == kEpiGatedSilu || epi == kEpiRope) return false;
  if (N >= 8192) return M <= 8 && K > 512;
  return K >= 768 && (M <= 2 || (M <= 8 && N < 2048 && K >= 1280));
}

template <int MP>
static void f32_lanes_rows(const GemmArgs& a, hipStream_t s) {
  const dim3 block(512);
  if (a.N >= 8192)
    hipLaunchKernelGGL((k_gemm_lanes<MP, 4>), dim3((a.N + 31) / 32), block, 0, s, a);
  else if (a.N < 2048)
    hipLaunchKernelGGL((k_gemm_lanes_ksplit<MP>), dim3((a.N + 7) / 8), block, 0, s, a);
  else if constexpr (MP <= 2)
    hipLaunchKernelGGL((k_gemm_lanes<MP, 1>), dim3((a.N + 7) / 8), block, 0, s, a);
}

static void f32_lanes(const GemmArgs& a, hipStream_t s) {
  if (a.M <= 1) f32_lanes_rows<1>(a, s);
  else if (a.M <= 2) f32_lanes_rows<2>(a, s);
  else if (a.M <= 4) f32_lanes_rows<4>(a, s);
  else f32_lanes_rows<8>(a, s);
}

static RowsNorm rows_norm(int dtype, int norm, int d) {
  const int es = dtype == kF32 ? 4 : 2;
  if (d * es <= 2 * 64 * 16) return kRowsLds;      // two vectors per lane; 33 KB of LDS at 16 rows
  // (a row times the gain must not leave the range: not in fp16)
  return norm == 1 && dtype != kF16 ? kRowsScaled : kRowsPlain;
}

bool gemm_takes_norm(int dtype, int M, int N, int d, int epi, int norm) {
  if (M > 16 || (dtype == kF32 && f32_by_lanes(M, N, d, epi))) return false;
  return rows_norm(dtype, norm, d) != kRowsPlain;
}

template <typename T, int CT>
static void rows_ct(const GemmArgs& a, hipStream_t s) {
  constexpr int ES = static_cast<int>(sizeof(T));
  const dim3 grid((a.N + 16 * CT - 1) / (16 * CT)), block(64 * kRowsWaves);
  if (a.norm < 0)
    hipLaunchKernelGGL((k_gemm_rows<T, CT, kRowsPlain>), grid, block, 0, s, a);
  else if (rows_norm(a.dtype, a.norm, a.K) == kRowsLds)
    hipLaunchKernelGGL((k_gemm_rows<T, CT, kRowsLds>), grid, block, a.M * (a.K * ES + 16), s, a);
  else
    hipLaunchKernelGGL((k_gemm_rows<T, CT, kRowsScaled>), grid, block, 0, s, a);
}

template <typename T>
static void rows_t(const GemmArgs& a, hipStream_t s) {
  // the gated and rotary epilogues combine packed columns 16 apart; a wide
  // output has workgroups enough with 32 columns each and reads the input
  // rows half as often
  if (a.epi == kEpiGatedGelu || a.epi == kEpiGatedSilu || a.epi == kEpiRope || a.N >= 8192)
    rows_ct<T, 2>(a, s);
  else
    rows_ct<T, 1>(a, s);
}

void gemm_skinny(const GemmArgs& a, hipStream_t s) {
  if (a.dtype == kF32 && f32_by_lanes(a.M, a.N, a.K, a.epi)) f32_lanes(a, s);
  else if (a.dtype == kF32) rows_t<float>(a, s);
  else if (a.dtype == kBF16) rows_t<bf16_t>(a, s);
  else rows_t<f16_t>(a, s);
}

}  // namespace gm
