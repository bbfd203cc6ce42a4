// gm_gemm_epilogue.h -- device pieces shared by the GEMM kernels: the
// epilogues (bias, GELU, residual, gate product, rotary, KV-cache append), all
// on fp32 accumulators with one rounding to the storage dtype, and the
// clamp-site statistics.
#pragma once
#include <math.h>

#include <type_traits>

#include "gm_device.h"
#include "gm_kernels.h"

namespace gm {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

// ------------------------------------------------------------ epilogue
template <typename T>
__device__ __forceinline__ void load4(const T* p, float* v, int nvalid, bool vec) {
  if (vec) {
    if constexpr (sizeof(T) == 4) {
      const f32x4v r = *reinterpret_cast<const f32x4v*>(p);
      v[0] = r[0]; v[1] = r[1]; v[2] = r[2]; v[3] = r[3];
    } else {
      const u32x2 r = *reinterpret_cast<const u32x2*>(p);
      const T* e = reinterpret_cast<const T*>(&r);
#pragma unroll
      for (int i = 0; i < 4; ++i) v[i] = to_f32(e[i]);
    }
  } else {
#pragma unroll
    for (int i = 0; i < 4; ++i) v[i] = i < nvalid ? to_f32(p[i]) : 0.f;
  }
}

template <typename T>
__device__ __forceinline__ void store4(T* p, const float* v, int nvalid, bool vec) {
  if (vec) {
    if constexpr (sizeof(T) == 4) {
      *reinterpret_cast<f32x4v*>(p) = f32x4v{v[0], v[1], v[2], v[3]};
    } else {
      u32x2 r;
      T* e = reinterpret_cast<T*>(&r);
#pragma unroll
      for (int i = 0; i < 4; ++i) e[i] = from_f32<T>(v[i]);
      *reinterpret_cast<u32x2*>(p) = r;
    }
  } else {
#pragma unroll
    for (int i = 0; i < 4; ++i)
      if (i < nvalid) p[i] = from_f32<T>(v[i]);
  }
}

// x * Phi(x).  fp32 models: through erff.  16-bit models: Phi through
// erfc(z) = t Q(t) exp(-z^2) with t = 1 / (1 + 0.3 |x|) on the hardware
// reciprocal and exponential; Q is a degree-7 minimax fit of
// erfcx(|x| / sqrt 2) / (2 t), relative error 1.5e-7.  In fp32 the whole is
// within 5e-7 below 1 and, as the exponent is rounded, 4e-6 at 9 and 7e-6 at
// 12, far below a 16-bit rounding (no cancellation on the
// negative side, where 1 + erff loses digits), 17 vector instructions against
// about 45: 4096 x 3072 x 768 with GELU 34.9 -> 29.2 us together with the
// per-wavefront staging of the epilogue.
template <typename T>
__device__ __forceinline__ float gelu_f(float x) {
  if constexpr (sizeof(T) == 4) {
    return 0.5f * x * (1.0f + erff(x * 0.70710678118654752f));
  } else {
    const float ax = fabsf(x);
    const float t = __builtin_amdgcn_rcpf(fmaf(0.3f, ax, 1.0f));
    const float e = __builtin_amdgcn_exp2f(ax * ax * -0.72134752044448170f);
    float q = 0.03567502087820895f;
    q = fmaf(q, t, -0.15720406629799158f);
    q = fmaf(q, t, 0.20635511028116715f);
    q = fmaf(q, t, -0.053685025862027065f);
    q = fmaf(q, t, 0.12856230317176076f);
    q = fmaf(q, t, 0.09991330429545925f);
    q = fmaf(q, t, 0.12075398335929735f);
    q = fmaf(q, t, 0.11962929722141813f);
    const float h = q * t * e;               // Phi(-|x|)
    return x * (x < 0.f ? h : 1.0f - h);
  }
}
// x * sigmoid(x) from the hardware exponential and reciprocal (v_exp_f32,
// v_rcp_f32, about 1 ulp each): x -> -inf gives 1/inf = 0, x -> +inf gives x
__device__ __forceinline__ float silu_f(float x) {
  return x * __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(x * -1.4426950408889634f));
}

struct SiteMax {
  uint32_t amax = 0;
  int nan = 0;
  __device__ __forceinline__ void add(float y) {
    if (y != y) nan = 1;
    else {
      const uint32_t u = __float_as_uint(y) & 0x7FFFFFFFu;
      amax = u > amax ? u : amax;
    }
  }
};

// Decode step: four consecutive output columns n..n+3 of row b in the k
// (region 1) or v (region 2) block of q|k|v also go to the KV cache.
template <typename T>
__device__ __forceinline__ void cache4(const GemmArgs& a, int b, int n, const float* v) {
  const int d = a.d_model, region = n / d;
  if (region < 1 || region > 2) return;
  if (static_cast<uint32_t>(a.state[kTrapFwd]) != kTrapNone) return;
  const int c = n - region * d, h = c / a.head_dim, i = c - h * a.head_dim;
  const int p = a.pos[b];
  T* dst = static_cast<T*>(region == 1 ? a.kc : a.vc) +
           ((static_cast<long long>(b) * a.heads + h) * a.kv_max_seq + p) * a.head_dim + i;
  store4(dst, v, 4, true);
  if (region == 1 && c == 0) a.kv_valid[static_cast<long long>(b) * a.kv_max_seq + p] = 1;
}

// Four consecutive packed columns nA..nA+3 (first tile of a pair, values
// va) and nA+16..nA+19 (second tile, values vb) of output row m.
template <typename T>
__device__ __forceinline__ void epi_pair(const GemmArgs& a, int m, int nA,
                                         const float* va, const float* vb,
                                         SiteMax& sm) {
  if (m >= a.M) return;
  const T* bias = static_cast<const T*>(a.bias);
  T* out = static_cast<T*>(a.out);
  const long long orow = static_cast<long long>(m) * a.ldo;
  if (a.epi == kEpiGatedGelu || a.epi == kEpiGatedSilu) {
    const int jo = (nA >> 5) * 16 + (nA & 15);
    float y[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      float g = va[r], u = vb[r];
      if (bias) {
        g += to_f32(bias[nA + r]);
        u += to_f32(bias[nA + 16 + r]);
      }
      const float act = a.epi == kEpiGatedGelu ? gelu_f<T>(g) : silu_f(g);
      y[r] = act * u;
    }
    store4(out + orow + jo, y, 4, (a.ldo & 3) == 0);
    return;
  }
  if (a.epi == kEpiRope && nA < 2 * a.d_model) {
    const int d = a.d_model, hd = a.head_dim, P = hd >> 1;
    const int region = nA >= d;
    const int nr = nA - region * d;
    const int h = nr / hd, within = nr - h * hd;
    const int i = (within >> 5) * 16 + (within & 15);
    int pos = a.pos ? a.pos[m] : m % a.seq;
    pos = pos < a.rope_rows ? pos : a.rope_rows - 1;
    // [Where]: both frequency sets exist; the forward's flag selects one
    const long long set = a.rope_set_stride && a.state[kRopeLong] ? a.rope_set_stride : 0;
    const float* cs = a.rope_cos + set + static_cast<long long>(pos) * P + i;
    const float* sn = a.rope_sin + set + static_cast<long long>(pos) * P + i;
    float o1[4], o2[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      float x1 = va[r], x2 = vb[r];
      if (bias) {
        x1 += to_f32(bias[nA + r]);
        x2 += to_f32(bias[nA + 16 + r]);
      }
      o1[r] = x1 * cs[r] - x2 * sn[r];
      o2[r] = x2 * cs[r] + x1 * sn[r];
    }
    const long long base = orow + region * d + h * hd + i;
    const bool vec = (a.ldo & 3) == 0;
    store4(out + base, o1, 4, vec);
    store4(out + base + P, o2, 4, vec);
    if (a.kc && region == 1) {
      cache4<T>(a, m, d + h * hd + i, o1);
      cache4<T>(a, m, d + h * hd + i + P, o2);
    }
    return;
  }
  // independent columns: store / gelu / residual (and v of kEpiRope)
#pragma unroll
  for (int t = 0; t < 2; ++t) {
    const int n0 = nA + 16 * t;
    if (n0 >= a.N) continue;
    const float* v = t ? vb : va;
    const int nvalid = a.N - n0 < 4 ? a.N - n0 : 4;
    const bool vec = nvalid == 4 && (a.ldo & 3) == 0;
    float y[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) y[r] = v[r];
    if (bias)
#pragma unroll
      for (int r = 0; r < 4; ++r)
        if (r < nvalid) y[r] += to_f32(bias[n0 + r]);
    if (a.epi == kEpiGelu)
#pragma unroll
      for (int r = 0; r < 4; ++r) y[r] = gelu_f<T>(y[r]);
    if (a.epi == kEpiResid) {
      float rv[4];
      load4(static_cast<const T*>(a.resid) + static_cast<long long>(m) * a.ldr + n0, rv,
            nvalid, nvalid == 4 && (a.ldr & 3) == 0);
#pragma unroll
      for (int r = 0; r < 4; ++r) y[r] += rv[r];
      if (a.site >= 0)
#pragma unroll
        for (int r = 0; r < 4; ++r)
          if (r < nvalid) sm.add(round_as<T>(y[r]));
    }
    store4(out + orow + n0, y, nvalid, vec);
    if (a.kc) cache4<T>(a, m, n0, y);
  }
}

// One atomic per wavefront on a site's slots, and only where it can change
// them: the slots only grow within a forward, so a wavefront whose maximum is
// not above the value it reads (possibly an older one) has nothing to add.
// 2048 wavefronts adding to one word one after the other took half of a
// 4096 x 1024 residual product (O and down of the clamp model 51 us each on
// average).
__device__ __forceinline__ void site_flush(const GemmArgs& a, SiteMax& sm) {
  if (a.site < 0) return;
  const uint32_t m = wave_max_u32(sm.amax);
  const int n = wave_or(sm.nan);
  if ((threadIdx.x & 63) == 0) {
    unsigned int* top = reinterpret_cast<unsigned int*>(a.state + kAbsmaxBase + a.site);
    int* nan = a.state + kNanBase + a.site;
    if (m > __hip_atomic_load(top, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) atomicMax(top, m);
    if (n && !__hip_atomic_load(nan, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) atomicOr(nan, 1);
  }
}

template <int I, int N, typename F>
__device__ __forceinline__ void static_for(F&& f) {
  if constexpr (I < N) {
    f(std::integral_constant<int, I>{});
    static_for<I + 1, N>(f);
  }
}

}  // namespace gm
