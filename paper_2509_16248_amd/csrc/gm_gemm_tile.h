// gm_gemm_tile.h -- the tiled MFMA GEMM kernels (M > 16).
#pragma once
#include "gm_gemm_epilogue.h"

namespace gm {

// ------------------------------------------------------------ MFMA tiles
// v_mfma_f32_32x32x16 (16-bit in, fp32 accumulate), W as the MFMA A operand
// and the activations as the B operand: a lane ends up with the output
// columns n = 32j + 8q + 4(lane/32) + r (q, r = 0..3) of row m = 32i + lane%32,
// so the columns of a 16-row weight group (q = 0, 1) and of its partner group
// (q + 2) sit in the same lane, which is what the gated and rotary epilogues
// pair.
template <typename T> struct Mfma32;
template <> struct Mfma32<bf16_t> {
  typedef bf16x8 vec;
  static __device__ __forceinline__ f32x16 run(vec a, vec b, f32x16 c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
  }
};
template <> struct Mfma32<f16_t> {
  typedef f16x8 vec;
  static __device__ __forceinline__ f32x16 run(vec a, vec b, f32x16 c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_f16(a, b, c, 0, 0, 0);
  }
};

// fp32: a lane holds 4 consecutive k of its row per fragment, so the step
// of MFMA r multiplies k = 4g + r of both operands (the order of the sum over
// k is free): v_mfma_f32_32x32x2_f32, fp32 products and sums.
template <> struct Mfma32<float> {
  typedef f32x4 vec;
  static __device__ __forceinline__ f32x16 run(vec a, vec b, f32x16 c) {
#pragma unroll
    for (int r = 0; r < 4; ++r) c = __builtin_amdgcn_mfma_f32_32x32x2f32(a[r], b[r], c, 0, 0, 0);
    return c;
  }
};

// Tile of this workgroup.  Hardware deals workgroups round-robin to the 8 XCDs,
// so workgroup b runs on XCD b % 8; each XCD gets a contiguous range of tile
// ids (the first total % 8 XCDs one more).
__device__ __forceinline__ void my_tile(int tiles_m, int tiles_n, int& tm, int& tn) {
  const int total = tiles_m * tiles_n, per = total / 8, rem = total % 8;
  const int b = blockIdx.x, x = b % 8;
  const int t = x * per + (x < rem ? x : rem) + b / 8;
  // grouped order: GM tile-rows sweep the columns together
  constexpr int GM = 8;
  const int group = t / (GM * tiles_n);
  const int first = group * GM;
  const int rows = tiles_m - first < GM ? tiles_m - first : GM;
  const int in = t - group * GM * tiles_n;
  tm = first + in % rows;
  tn = in / rows;
}

// A 16-byte vector stored at any element's address: global memory takes
// vector accesses at any byte on this target, and a row of the odd vocabulary
// starts anywhere.
typedef u32x4 __attribute__((aligned(2))) u32x4_any;

// What an epilogue does with column pairs decides its code: independent
// columns (store, GELU, residual), gated pairs, rotary pairs, and a plain store
// to rows that are not made of whole cache lines.
enum EpiKind : int { kKindPlain = 0, kKindGated = 1, kKindRope = 2, kKindWide = 3 };

inline EpiKind kind_of(const GemmArgs& a) {
  if (a.epi == kEpiGatedGelu || a.epi == kEpiGatedSilu) return kKindGated;
  if (a.epi == kEpiRope) return kKindRope;
  // (the head of an odd vocabulary)
  if (a.epi == kEpiStore && !a.bias && !a.kc && a.site < 0 && a.ldo % 64) return kKindWide;
  return kKindPlain;
}

// Epilogue of one wavefront's TM x TN tiles of 32 x 32 accumulators at row m0
// and packed column n0: lane l holds columns 32j + 8q + 4(l/32) + r of row
// 32i + l%32.  The values finish in registers (bias, then GELU, the residual,
// the gate product or the rotation; one rounding to the output type; the
// site statistics of the rounded values) and leave 32 rows at a time through
// a staging area of the wavefront's own (no barrier): 16-byte chunks with
// consecutive lanes on consecutive columns, stored at any element's address
// (the rows of an odd vocabulary start anywhere).  Staged rows are rotated by
// chunks so that 16 rows fall into distinct banks.  Rotary q/k tiles are
// staged in packed order; their chunks (8 positions of one half of a head)
// are mapped to head positions when they are stored.  The KV-cache append of
// a decode step finishes through epi_pair, straight from registers.
template <typename T, int KIND, int TN>
constexpr int stage_bytes() {   // of one wavefront
  return 32 * (KIND == kKindGated ? 16 * TN : 32 * TN) * static_cast<int>(sizeof(T));
}

template <typename T, int KIND, int TM, int TN>
__device__ __forceinline__ void wave_epilogue(const GemmArgs& a, f32x16 (&acc)[TM][TN], void* stage,
                                              int m0, int n0) {
  constexpr int VE = 16 / static_cast<int>(sizeof(T));   // elements per 16-byte chunk
  constexpr int OW = KIND == kKindGated ? 16 * TN : 32 * TN;
  constexpr int C = OW / VE;                             // chunks per staged row
  constexpr int R = C % 3 == 0 ? 48 / C : (C < 16 ? 16 / C : 1);   // rows per rotation step
  static_assert(C % 2 == 0, "whole wavefronts of chunks per 32 rows");
  const int lane = threadIdx.x & 63, l32 = lane & 31, g = lane >> 5;
  SiteMax sm;
  const T* bias = static_cast<const T*>(a.bias);
  const bool resid = KIND == kKindPlain && a.epi == kEpiResid;
  const T* res = static_cast<const T*>(a.resid);
  // bias and residual are read four elements at a time: N in fours, aligned
  constexpr uintptr_t VB = 4 * sizeof(T) - 1;
  const bool vec = ((!bias && !resid) || (a.N & 3) == 0) && (reinterpret_cast<uintptr_t>(bias) & VB) == 0 &&
                   (!resid || ((a.ldr & 3) == 0 && (reinterpret_cast<uintptr_t>(res) & VB) == 0));
  if (a.kc || !vec) {
    static_for<0, TM>([&](auto i) {
      static_for<0, TN>([&](auto j) {
        static_for<0, 2>([&](auto q) {
          float va[4], vb[4];
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            va[r] = acc[i][j][4 * q + r];
            vb[r] = acc[i][j][4 * (q + 2) + r];
          }
          epi_pair<T>(a, m0 + 32 * i + l32, n0 + 32 * j + 8 * q + 4 * g, va, vb, sm);
        });
      });
    });
    site_flush(a, sm);
    return;
  }
  T* stg = static_cast<T*>(stage);
  // four values at staged column col of this lane's row
  auto put = [&](int col, const float* v) {
    const int c = (col / VE + l32 / R) % C;
    store4(stg + (l32 * C + c) * VE + col % VE, v, 4, true);
  };
  // columns past N read the last four (and are not stored)
  auto add_bias = [&](int n, float* v) {
    float bv[4];
    load4(bias + (n + 4 <= a.N ? n : a.N - 4), bv, 4, true);
#pragma unroll
    for (int r = 0; r < 4; ++r) v[r] += bv[r];
  };
  T* out = static_cast<T*>(a.out);
  const int nout = KIND == kKindGated ? a.N / 2 : a.N;
  const int ob = KIND == kKindGated ? n0 / 2 : n0;
  static_for<0, TM>([&](auto i) {
    const int mi = m0 + 32 * i + l32, m = mi < a.M ? mi : a.M - 1;
    if constexpr (KIND == kKindPlain) {
      if (bias)
        static_for<0, TN>([&](auto j) {
          static_for<0, 4>([&](auto q) {
            float v[4] = {acc[i][j][4 * q], acc[i][j][4 * q + 1], acc[i][j][4 * q + 2], acc[i][j][4 * q + 3]};
            add_bias(n0 + 32 * j + 8 * q + 4 * g, v);
#pragma unroll
            for (int r = 0; r < 4; ++r) acc[i][j][4 * q + r] = v[r];
          });
        });
      if (resid) {   // the residual of a row of fragments is fetched together
        const T* rrow = res + static_cast<long long>(m) * a.ldr;
        static_for<0, TN>([&](auto j) {
          static_for<0, 4>([&](auto q) {
            const int n = n0 + 32 * j + 8 * q + 4 * g;
            float rv[4];
            load4(rrow + (n + 4 <= a.N ? n : a.N - 4), rv, 4, true);
#pragma unroll
            for (int r = 0; r < 4; ++r) acc[i][j][4 * q + r] += rv[r];
          });
        });
      }
      if (a.epi == kEpiGelu)
        static_for<0, TN>([&](auto j) {
#pragma unroll
          for (int r = 0; r < 16; ++r) acc[i][j][r] = gelu_f<T>(acc[i][j][r]);
        });
      static_for<0, TN>([&](auto j) {
        static_for<0, 4>([&](auto q) {
          const float v[4] = {acc[i][j][4 * q], acc[i][j][4 * q + 1], acc[i][j][4 * q + 2], acc[i][j][4 * q + 3]};
          put(32 * j + 8 * q + 4 * g, v);
        });
      });
      if (a.site >= 0 && mi < a.M)
        static_for<0, TN>([&](auto j) {
#pragma unroll
          for (int r = 0; r < 16; ++r)
            if (n0 + 32 * j + 8 * (r / 4) + 4 * g + r % 4 < a.N) sm.add(round_as<T>(acc[i][j][r]));
        });
    } else {
      const float *cs = nullptr, *sn = nullptr;
      if constexpr (KIND == kKindRope) {
        int pos = a.pos ? a.pos[m] : m % a.seq;
        pos = pos < a.rope_rows ? pos : a.rope_rows - 1;
        // [Where]: both frequency sets exist; the forward's flag selects one
        const long long set = a.rope_set_stride && a.state[kRopeLong] ? a.rope_set_stride : 0;
        cs = a.rope_cos + set + static_cast<long long>(pos) * (a.head_dim >> 1);
        sn = a.rope_sin + set + static_cast<long long>(pos) * (a.head_dim >> 1);
      }
      static_for<0, TN>([&](auto j) {
        static_for<0, 2>([&](auto q) {
          const int nl = 32 * j + 8 * q + 4 * g, n = n0 + nl;
          float x1[4], x2[4];
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            x1[r] = acc[i][j][4 * q + r];
            x2[r] = acc[i][j][4 * (q + 2) + r];
          }
          if (bias) {
            add_bias(n, x1);
            add_bias(n + 16, x2);
          }
          if constexpr (KIND == kKindGated) {
            float y[4];
            if (a.epi == kEpiGatedGelu) {
#pragma unroll
              for (int r = 0; r < 4; ++r) y[r] = gelu_f<T>(x1[r]) * x2[r];
            } else {
#pragma unroll
              for (int r = 0; r < 4; ++r) y[r] = silu_f(x1[r]) * x2[r];
            }
            put(16 * j + 8 * q + 4 * g, y);
          } else if (n < 2 * a.d_model) {
            const int w = n % a.head_dim, ii = (w >> 5) * 16 + (w & 15);
            float cv[4], sv[4], o1[4], o2[4];
            load4(cs + ii, cv, 4, true);
            load4(sn + ii, sv, 4, true);
#pragma unroll
            for (int r = 0; r < 4; ++r) {
              o1[r] = x1[r] * cv[r] - x2[r] * sv[r];
              o2[r] = x2[r] * cv[r] + x1[r] * sv[r];
            }
            put(nl, o1);
            put(nl + 16, o2);
          } else {
            put(nl, x1);
            put(nl + 16, x2);
          }
        });
      });
    }
    // 32 staged rows leave
#pragma unroll
    for (int u = 0; u < C / 2; ++u) {
      const int e = u * 64 + lane, row = e / C, c = e % C;
      const u32x4 w = *reinterpret_cast<const u32x4*>(stg + (row * C + (c + row / R) % C) * VE);
      const int mr = m0 + 32 * i + row, col = ob + VE * c;
      int hc = col;
      if constexpr (KIND == kKindRope) {
        if (col < 2 * a.d_model) {
          const int k = col % a.head_dim;
          hc += (k >> 5) * 16 + ((k >> 4) & 1) * (a.head_dim >> 1) + (k & 15) - k;
        }
      }
      T* o = out + static_cast<long long>(mr) * a.ldo + hc;
      if (mr < a.M) {
        if (col + VE <= nout) {
          *reinterpret_cast<u32x4_any*>(o) = w;
        } else {
          const T* we = reinterpret_cast<const T*>(&w);
#pragma unroll
          for (int r = 0; r < VE; ++r)
            if (col + r < nout) o[r] = we[r];
        }
      }
    }
  });
  site_flush(a, sm);
}

// Plain store of a BM x BN tile to rows that start anywhere (the logits of an
// odd vocabulary): the whole tile is staged and each row leaves as one run of
// BN columns.  A run's first and last cache lines are shared with other tiles,
// and lines that reach memory in parts are read back to be merged: per-
// wavefront runs of 64 columns took 1180 us on 8192 x 30522 x 1024 (256 x 256
// tiles), rows of the whole tile 566, single-element stores of such rows 681.
template <typename T, int BM, int BN>
constexpr int wide_bytes() {
  return BM * (BN + 16 / static_cast<int>(sizeof(T))) * static_cast<int>(sizeof(T));
}

template <typename T, int BM, int BN, int NT, int TM, int TN>
__device__ __forceinline__ void wide_epilogue(const GemmArgs& a, f32x16 (&acc)[TM][TN], char* smem,
                                              int bm, int bn, int ml0, int nl0, bool owner) {
  constexpr int VE = 16 / static_cast<int>(sizeof(T)), LDB = BN + VE, CPR = BN / VE;
  const int t = threadIdx.x, lane = t & 63, l32 = lane & 31, g = lane >> 5;
  T* stb = reinterpret_cast<T*>(smem);
  __syncthreads();   // every wavefront is done with the operand tiles
  if (owner)
    static_for<0, TM>([&](auto i) {
      static_for<0, TN>([&](auto j) {
        static_for<0, 4>([&](auto q) {
          const float v[4] = {acc[i][j][4 * q], acc[i][j][4 * q + 1], acc[i][j][4 * q + 2], acc[i][j][4 * q + 3]};
          store4(&stb[(ml0 + 32 * i + l32) * LDB + nl0 + 32 * j + 8 * q + 4 * g], v, 4, true);
        });
      });
    });
  __syncthreads();
  T* out = static_cast<T*>(a.out);
  const int ncol = a.N - bn < BN ? a.N - bn : BN;
  for (int e = t; e < BM * CPR; e += NT) {
    const int ml = e / CPR, j0 = VE * (e % CPR), m = bm + ml;
    if (m >= a.M || j0 >= ncol) continue;
    const u32x4 w = *reinterpret_cast<const u32x4*>(&stb[ml * LDB + j0]);
    T* o = out + static_cast<long long>(m) * a.ldo + bn + j0;
    if (j0 + VE <= ncol) {
      *reinterpret_cast<u32x4_any*>(o) = w;
    } else {
      const T* we = reinterpret_cast<const T*>(&w);
#pragma unroll
      for (int r = 0; r < VE; ++r)
        if (j0 + r < ncol) o[r] = we[r];
    }
  }
}

// ------------------------------------------------------------ global -> LDS
// 16 bytes per lane straight into LDS: lane i of a wavefront instruction
// writes bytes 16i .. 16i+15 of a 1 KB block.
typedef __attribute__((address_space(3))) void* lds_ptr_t;

__device__ __forceinline__ void dma16(const void* g, void* lds) {
  __builtin_amdgcn_global_load_lds(g, (lds_ptr_t)lds, 16, 0, 0);
}

// The same through a buffer descriptor: the lane's 32-bit offset plus a
// uniform one, so a load of the next stage costs no vector instruction.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t buffer_of(const void* p) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), 0, -1, 0x00020000);
}
__device__ __forceinline__ void dma16(__amdgpu_buffer_rsrc_t b, uint32_t lane_off, uint32_t off, void* lds) {
  __builtin_amdgcn_raw_ptr_buffer_load_lds(b, (lds_ptr_t)lds, 16, lane_off, off, 0, 0);
}

template <int N>
__device__ __forceinline__ void wait_vmcnt() {
  static_assert(N >= 0 && N < 64, "vmcnt range");
  __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | (0x7 << 4) | (0xF << 8));
}

__device__ __forceinline__ void wait_lgkmcnt0() {
  __builtin_amdgcn_s_waitcnt(0xF | (0x3 << 14) | (0x7 << 4));   // lgkmcnt(0), others untouched
}

// ------------------------------------------------------------ ping-pong kernel
// 16-bit products with enough large tiles.  8 wavefronts, two per SIMD, in
// two groups of one wavefront per SIMD: while one group multiplies, the other
// reads its next operand fragments from LDS; a barrier ends every such slot
// and the groups change roles, so the matrix cores always have a group to run
// and fragments are single-buffered.  Group 1 runs one slot behind group 0.
// The global -> LDS loads are spread between the MFMAs of a cluster: issued in
// the reading slot they queue in front of the fragment reads (16 clocks each
// in the CU's one address unit) and the slot grows from 560 to 940 clocks.
// A stage is 64 columns of both operands (128-byte rows, eight 16-byte chunks;
// chunk c of row r sits in slot c ^ (r / 2) % 8, so the 16 rows that 16 lanes
// read at once fall into 16 distinct bank groups); a ring of NS stages.
// PH = 2 splits the rows of a wavefront tile into two clusters per stage, so
// that a ring of two stages is refilled in two parts, each as soon as both
// groups have read it: W and the first rows of stage k + 2 during cluster 1 of
// stage k, the second rows of stage k + 1 during cluster 0 of stage k.
// Measured (2048 x 32000 x 4096, 256 x 256 tiles): 434 us, 1238 TFLOP/s,
// against 489 us for the same tile with all wavefronts in the same phase; the
// K loop keeps the matrix cores 88% busy and runs at the power limit (1.44 GHz;
// without its loads 93% at 1.62 GHz).
__device__ __forceinline__ void phase_barrier() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_sched_barrier(0);
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_sched_barrier(0);
  asm volatile("" ::: "memory");
}

template <typename T, int KIND, int BM, int BN, int WM, int WN, int PH, int NS>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2, 2))) void k_gemm_pp(GemmArgs a) {
  typedef typename Mfma32<T>::vec vec;
  constexpr int BK = 64;
  static_assert(WM * WN == 8, "8 wavefronts");
  constexpr int WTM = BM / WM, WTN = BN / WN;
  constexpr int TM = WTM / 32, TN = WTN / 32, TP = TM / PH;   // tiles; row tiles per phase
  constexpr int KS = 4, CPR = 8, RPB = 2;
  constexpr int STAGE_ELEMS = (BM + BN) * BK;
  constexpr int PR = WTM / PH;                          // rows of a wavefront's part per phase
  constexpr int LA = BM / PH / 64, LB = BN / 64;        // loads per wavefront: an A part, B
  constexpr int RING = NS * STAGE_ELEMS * 2;
  constexpr int STG = stage_bytes<T, KIND, TN>();       // epilogue staging of a wavefront
  constexpr int OUTB = KIND == kKindWide ? wide_bytes<T, BM, BN>() : 8 * STG;
  constexpr int SMEM = RING > OUTB ? RING : OUTB;
  static_assert(BM % (64 * PH) == 0 && BN % 64 == 0 && TM % PH == 0, "tile split");
  static_assert(PH == 1 || NS == 2, "phases of a ring of two stages");
  __shared__ __attribute__((aligned(1024))) char smem[SMEM];
  T* lds = reinterpret_cast<T*>(smem);
  const int tiles_m = (a.M + BM - 1) / BM, tiles_n = (a.N + BN - 1) / BN;
  int tm, tn;
  my_tile(tiles_m, tiles_n, tm, tn);
  const int bm = tm * BM, bn = tn * BN;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wm = wave / WN, wn = wave % WN;
  const int grp = wave >> 2;                            // ping-pong group: one wavefront per SIMD
  const int l32 = lane & 31, g = lane >> 5;
  // LDS row of load j of A part p: 8 rows per wavefront instruction
  auto rowA = [&](int p, int j) {
    const int at = (wave * LA + j) * 8;                 // within the part's BM / PH rows
    return (at / PR) * WTM + p * PR + at % PR;
  };
  auto rowB = [&](int j) { return BM + (wave * LB + j) * 8; };
  // this lane's byte offsets from the tile's first rows of A and W (rows past
  // the end re-read the last row: loaded, never stored); the chunk lands in
  // its swizzled slot
  uint32_t oa[PH][LA], ob[LB];
  const int sub = lane / CPR, slot = lane % CPR;
#pragma unroll
  for (int p = 0; p < PH; ++p)
#pragma unroll
    for (int j = 0; j < LA; ++j) {
      const int sr = rowA(p, j) + sub;
      const int chunk = slot ^ ((sr / RPB) % CPR);
      const int r = bm + sr < a.M ? sr : a.M - 1 - bm;
      oa[p][j] = (static_cast<uint32_t>(r) * a.lda + chunk * 8) * 2;
    }
#pragma unroll
  for (int j = 0; j < LB; ++j) {
    const int sr = rowB(j) + sub;
    const int chunk = slot ^ ((sr / RPB) % CPR);
    const int c = bn + sr - BM < a.N ? sr - BM : a.N - 1 - bn;
    ob[j] = (static_cast<uint32_t>(c) * a.ldw + chunk * 8) * 2;
  }
  const __amdgpu_buffer_rsrc_t X0 =
      buffer_of(static_cast<const T*>(a.A) + static_cast<long long>(bm) * a.lda);
  const __amdgpu_buffer_rsrc_t W0 =
      buffer_of(static_cast<const T*>(a.W) + static_cast<long long>(bn) * a.ldw);
  auto issueA = [&](int p, int st) {
    T* dst = lds + (st % NS) * STAGE_ELEMS;
#pragma unroll
    for (int j = 0; j < LA; ++j) dma16(X0, oa[p][j], st * (BK * 2), dst + rowA(p, j) * BK);
  };
  auto issueB = [&](int st) {
    T* dst = lds + (st % NS) * STAGE_ELEMS;
#pragma unroll
    for (int j = 0; j < LB; ++j) dma16(W0, ob[j], st * (BK * 2), dst + rowB(j) * BK);
  };
  f32x16 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;
  const int swz = (l32 / RPB) % CPR;
  const int offA = (wm * WTM + l32) * BK, offB = (BM + wn * WTN + l32) * BK;
  vec fa[KS][TP], fb[KS][TN];
  auto readA = [&](int st, int p) {
    const T* q = lds + (st % NS) * STAGE_ELEMS + offA + p * PR * BK;
#pragma unroll
    for (int s = 0; s < KS; ++s)
#pragma unroll
      for (int i = 0; i < TP; ++i)
        fa[s][i] = *reinterpret_cast<const vec*>(q + 32 * i * BK + ((2 * s + g) ^ swz) * 8);
  };
  auto readB = [&](int st) {
    const T* q = lds + (st % NS) * STAGE_ELEMS + offB;
#pragma unroll
    for (int s = 0; s < KS; ++s)
#pragma unroll
      for (int j = 0; j < TN; ++j)
        fb[s][j] = *reinterpret_cast<const vec*>(q + 32 * j * BK + ((2 * s + g) ^ swz) * 8);
  };
  // one MFMA cluster with the given loads spread between its MFMAs
  auto cluster = [&](auto p, auto loads, auto&& issue) {
    constexpr int NL = decltype(loads)::value, NM = KS * TP * TN;
    __builtin_amdgcn_s_setprio(1);
    issue();
#pragma unroll
    for (int s = 0; s < KS; ++s)
#pragma unroll
      for (int i = 0; i < TP; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
          acc[p * TP + i][j] = Mfma32<T>::run(fb[s][j], fa[s][i], acc[p * TP + i][j]);
    static_for<0, NM>([&](auto q) {
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
      if constexpr (NL > 0)
        if constexpr ((decltype(q)::value + 1) * NL / NM > decltype(q)::value * NL / NM)
          __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);
    });
    __builtin_amdgcn_s_setprio(0);
  };
  const int nk = a.K / BK;
  if constexpr (PH == 2) {
    issueB(0);
    issueA(0, 0);
    issueA(1, 0);
    if (nk > 1) {
      issueB(1);
      issueA(0, 1);
      wait_vmcnt<LA + LB>();
    } else {
      wait_vmcnt<0>();
    }
    phase_barrier();
    if (grp) phase_barrier();
    auto stage = [&](auto steady, int k) {
      constexpr bool S = decltype(steady)::value;
      readB(k);
      readA(k, 0);
      if (grp) {
        if constexpr (S) wait_vmcnt<LA + LB>();
        else wait_vmcnt<0>();
      }
      wait_lgkmcnt0();
      phase_barrier();
      if constexpr (S) cluster(std::integral_constant<int, 0>{}, std::integral_constant<int, LA>{}, [&] { issueA(1, k + 1); });
      else {
        if (k + 1 < nk) issueA(1, k + 1);
        cluster(std::integral_constant<int, 0>{}, std::integral_constant<int, 0>{}, [&] {});
      }
      if (!grp) {
        if constexpr (S) wait_vmcnt<2 * LA + LB>();
        else wait_vmcnt<0>();
      }
      phase_barrier();
      readA(k, 1);
      if (grp) {
        if constexpr (S) wait_vmcnt<LA>();
        else wait_vmcnt<0>();
      }
      wait_lgkmcnt0();
      phase_barrier();
      if constexpr (S) cluster(std::integral_constant<int, 1>{}, std::integral_constant<int, LA + LB>{}, [&] { issueB(k + 2); issueA(0, k + 2); });
      else cluster(std::integral_constant<int, 1>{}, std::integral_constant<int, 0>{}, [&] {});
      if (!grp) {
        if constexpr (S) wait_vmcnt<2 * LA + LB>();
        else wait_vmcnt<0>();
      }
      phase_barrier();
    };
    int k = 0;
    for (; k + 2 < nk; ++k) stage(std::true_type{}, k);
    for (; k < nk; ++k) stage(std::false_type{}, k);
    if (!grp) phase_barrier();
  } else {
    // group 0 reads stage k in slot 2k and multiplies in slot 2k + 1, group 1
    // one slot later; the loads of stage k + NS - 1 go out in the
    // multiplication of stage k
    static_for<0, NS - 1>([&](auto st) {
      if (st < nk) {
        issueB(st);
        issueA(0, st);
      }
    });
    if (nk >= NS - 1) wait_vmcnt<(NS - 2) * (LA + LB)>();
    else wait_vmcnt<0>();
    phase_barrier();
    if (grp) phase_barrier();
    auto stage = [&](auto steady, int k) {
      constexpr bool S = decltype(steady)::value;
      readB(k);
      readA(k, 0);
      if (grp) {
        if constexpr (S) wait_vmcnt<(NS - 3) * (LA + LB)>();
        else wait_vmcnt<0>();
      }
      wait_lgkmcnt0();
      phase_barrier();
      if constexpr (S) cluster(std::integral_constant<int, 0>{}, std::integral_constant<int, LA + LB>{}, [&] { issueB(k + NS - 1); issueA(0, k + NS - 1); });
      else cluster(std::integral_constant<int, 0>{}, std::integral_constant<int, 0>{}, [&] {});
      if (!grp) {
        if constexpr (S) wait_vmcnt<(NS - 2) * (LA + LB)>();
        else wait_vmcnt<0>();
      }
      phase_barrier();
    };
    int k = 0;
    for (; k + NS - 1 < nk; ++k) stage(std::true_type{}, k);
    for (; k < nk; ++k) stage(std::false_type{}, k);
    if (!grp) phase_barrier();
  }
  // (every wavefront has read its last fragments before the last barrier)
  if constexpr (KIND == kKindWide)
    wide_epilogue<T, BM, BN, 512>(a, acc, smem, bm, bn, wm * WTM, wn * WTN, true);
  else
    wave_epilogue<T, KIND>(a, acc, smem + wave * STG, bm + wm * WTM, bn + wn * WTN);
}

template <typename T, int BM, int BN, int WM, int WN, int PH, int NS>
static void run_pp(const GemmArgs& a, hipStream_t s) {
  const dim3 grid(((a.M + BM - 1) / BM) * ((a.N + BN - 1) / BN)), block(512);
  switch (kind_of(a)) {
    case kKindGated: hipLaunchKernelGGL((k_gemm_pp<T, kKindGated, BM, BN, WM, WN, PH, NS>), grid, block, 0, s, a); break;
    case kKindRope: hipLaunchKernelGGL((k_gemm_pp<T, kKindRope, BM, BN, WM, WN, PH, NS>), grid, block, 0, s, a); break;
    case kKindWide: hipLaunchKernelGGL((k_gemm_pp<T, kKindWide, BM, BN, WM, WN, PH, NS>), grid, block, 0, s, a); break;
    default: hipLaunchKernelGGL((k_gemm_pp<T, kKindPlain, BM, BN, WM, WN, PH, NS>), grid, block, 0, s, a);
  }
}

// ------------------------------------------------------------ ring kernel
// Tiles that are too small (or too few) for the large-tile kernel, and fp32.
// WM x WN x WK wavefronts: WM x WN wavefront tiles, and WK wavefronts share a
// tile by splitting the k-steps of every stage between them (their sums meet
// in LDS at the end), so that a 64 x 64 output keeps 8 wavefronts loading.
// One stage is BK bytes-contiguous columns of both operands, fetched global ->
// LDS through a ring of NS stages; one barrier per stage: after it, nobody
// reads stage k-1 any more and its slot takes stage k+NS-1.
template <typename T, int KIND, int BM, int BN, int WM, int WN, int WK, int BK, int NS>
__global__ __launch_bounds__(64 * WM * WN * WK) void k_gemm_ring(GemmArgs a) {
  typedef typename Mfma32<T>::vec vec;
  constexpr int ES = static_cast<int>(sizeof(T));
  constexpr int VE = 16 / ES;                           // elements per 16-byte chunk
  constexpr int NW = WM * WN * WK;
  constexpr int WTM = BM / WM, WTN = BN / WN;
  constexpr int TM = WTM / 32, TN = WTN / 32;
  constexpr int CPR = BK / VE;                          // 16-byte chunks per row
  constexpr int KS = CPR / 2;                           // k-steps (two chunks) per stage
  constexpr int KSW = KS / WK;                          // of which this wavefront's
  constexpr int RPB = 16 / CPR;                         // rows per 256 bytes
  constexpr int RPI = 1024 / (BK * ES);                 // rows per wavefront instruction
  constexpr int STAGE_ELEMS = (BM + BN) * BK;
  constexpr int LPW = (BM + BN) / RPI / NW;             // loads per wavefront per stage
  constexpr int RING = NS * STAGE_ELEMS * ES;
  constexpr int OUTB = KIND == kKindWide ? wide_bytes<T, BM, BN>() : WM * WN * stage_bytes<T, KIND, TN>();
  constexpr int REDB = (WK - 1) * BM * BN * 4;
  constexpr int SMEM = RING > OUTB ? (RING > REDB ? RING : REDB) : (OUTB > REDB ? OUTB : REDB);
  static_assert(CPR >= 2 && CPR <= 16 && KS % WK == 0, "stage columns");
  static_assert((BM + BN) % (RPI * NW) == 0, "stage rows must split over the wavefronts");
  static_assert(NS >= 3 && LPW * (NS - 2) < 64, "vmcnt range");
  __shared__ __attribute__((aligned(1024))) char smem[SMEM];
  T* lds = reinterpret_cast<T*>(smem);
  const int tiles_m = (a.M + BM - 1) / BM, tiles_n = (a.N + BN - 1) / BN;
  int tm, tn;
  my_tile(tiles_m, tiles_n, tm, tn);
  const int bm = tm * BM, bn = tn * BN;
  const int t = threadIdx.x, wave = t >> 6, lane = t & 63;
  const T* __restrict__ A0 = static_cast<const T*>(a.A);
  const T* __restrict__ W0 = static_cast<const T*>(a.W);
  const T* src[LPW];
#pragma unroll
  for (int j = 0; j < LPW; ++j) {
    const int sr = (wave * LPW + j) * RPI + lane / CPR;
    const int chunk = (lane % CPR) ^ ((sr / RPB) % CPR);
    if (sr < BM) {
      int r = bm + sr;
      r = r < a.M ? r : a.M - 1;
      src[j] = A0 + static_cast<long long>(r) * a.lda + chunk * VE;
    } else {
      int c = bn + sr - BM;
      c = c < a.N ? c : a.N - 1;
      src[j] = W0 + static_cast<long long>(c) * a.ldw + chunk * VE;
    }
  }
  auto issue = [&](int slot) {
#pragma unroll
    for (int j = 0; j < LPW; ++j) {
      dma16(src[j], lds + slot * STAGE_ELEMS + (wave * LPW + j) * RPI * BK);
      src[j] += BK;
    }
  };
  const int wk = wave % WK, wmn = wave / WK, wm = wmn / WN, wn = wmn % WN;
  const int l32 = lane & 31, g = lane >> 5;
  f32x16 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;
  const int swz = (l32 / RPB) % CPR;
  const int offA = (wm * WTM + l32) * BK, offB = (BM + wn * WTN + l32) * BK;
  auto compute = [&](int slot) {
    const T* st = lds + slot * STAGE_ELEMS;
    vec fa[KSW][TM], fb[KSW][TN];
#pragma unroll
    for (int s = 0; s < KSW; ++s) {
      const int col = ((2 * (wk * KSW + s) + g) ^ swz) * VE;
#pragma unroll
      for (int j = 0; j < TN; ++j) fb[s][j] = *reinterpret_cast<const vec*>(st + offB + 32 * j * BK + col);
#pragma unroll
      for (int i = 0; i < TM; ++i) fa[s][i] = *reinterpret_cast<const vec*>(st + offA + 32 * i * BK + col);
    }
    __builtin_amdgcn_sched_barrier(0);   // every read in flight before the first MFMA
#pragma unroll
    for (int s = 0; s < KSW; ++s)
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) acc[i][j] = Mfma32<T>::run(fb[s][j], fa[s][i], acc[i][j]);
  };
  const int nk = a.K / BK;
  static_for<0, NS - 1>([&](auto st) {
    if (st < nk) issue(st);
  });
  int slot = 0;
  int k = 0;
  for (; k + NS - 1 < nk; ++k) {
    wait_vmcnt<LPW * (NS - 2)>();   // stage k landed, NS - 2 younger ones in flight
    wait_lgkmcnt0();
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    issue(slot == 0 ? NS - 1 : slot - 1);
    compute(slot);
    slot = slot + 1 == NS ? 0 : slot + 1;
  }
  wait_vmcnt<0>();
  wait_lgkmcnt0();
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
  for (; k < nk; ++k) {
    compute(slot);
    slot = slot + 1 == NS ? 0 : slot + 1;
  }
  __syncthreads();   // every wavefront is done reading operand tiles
  if constexpr (WK > 1) {
    float* red = reinterpret_cast<float*>(smem);
    // the sums of K groups 1.. go to LDS, one 16-byte vector per lane and
    // step, and group 0 adds them in order
    if (wk > 0) {
      static_for<0, TM>([&](auto i) {
        static_for<0, TN>([&](auto j) {
          static_for<0, 4>([&](auto q) {
            const int at = (((wk - 1) * WM * WN + wmn) * TM * TN * 4 + (i * TN + j) * 4 + q) * 256 + lane * 4;
            *reinterpret_cast<f32x4*>(red + at) =
                f32x4{acc[i][j][4 * q], acc[i][j][4 * q + 1], acc[i][j][4 * q + 2], acc[i][j][4 * q + 3]};
          });
        });
      });
    }
    __syncthreads();
    if (wk == 0) {
      for (int w = 0; w < WK - 1; ++w)
        static_for<0, TM>([&](auto i) {
          static_for<0, TN>([&](auto j) {
            static_for<0, 4>([&](auto q) {
              const int at = ((w * WM * WN + wmn) * TM * TN * 4 + (i * TN + j) * 4 + q) * 256 + lane * 4;
              const f32x4 v = *reinterpret_cast<const f32x4*>(red + at);
#pragma unroll
              for (int r = 0; r < 4; ++r) acc[i][j][4 * q + r] += v[r];
            });
          });
        });
    }
    __syncthreads();
  }
  if constexpr (KIND == kKindWide)
    wide_epilogue<T, BM, BN, 64 * NW>(a, acc, smem, bm, bn, wm * WTM, wn * WTN, wk == 0);
  else if (wk == 0)
    wave_epilogue<T, KIND>(a, acc, smem + wmn * stage_bytes<T, KIND, TN>(), bm + wm * WTM, bn + wn * WTN);
}

template <typename T, int BM, int BN, int WM, int WN, int WK, int BK, int NS>
static void run_ring(const GemmArgs& a, hipStream_t s) {
  const dim3 grid(((a.M + BM - 1) / BM) * ((a.N + BN - 1) / BN)), block(64 * WM * WN * WK);
  switch (kind_of(a)) {
    case kKindGated: hipLaunchKernelGGL((k_gemm_ring<T, kKindGated, BM, BN, WM, WN, WK, BK, NS>), grid, block, 0, s, a); break;
    case kKindRope: hipLaunchKernelGGL((k_gemm_ring<T, kKindRope, BM, BN, WM, WN, WK, BK, NS>), grid, block, 0, s, a); break;
    case kKindWide: hipLaunchKernelGGL((k_gemm_ring<T, kKindWide, BM, BN, WM, WN, WK, BK, NS>), grid, block, 0, s, a); break;
    default: hipLaunchKernelGGL((k_gemm_ring<T, kKindPlain, BM, BN, WM, WN, WK, BK, NS>), grid, block, 0, s, a);
  }
}

}  // namespace gm
