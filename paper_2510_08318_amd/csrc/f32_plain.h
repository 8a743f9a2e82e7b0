// The passes of the fp32-arithmetic modes in plain fp32 FMA, a wavefront to a token, for what the bf16 pieces of f32_split.h do not carry:
// infinities (their pieces are Inf and NaN) and finite values that round to Inf as bf16 (above 3.3895e38).  Each of these makes a product of pieces NaN or Inf, which the kernels notice on the accumulators, a few instructions a block;
// they then run their share once more through here.  Results are those of IEEE fp32 arithmetic; 12 heads x 32760 x 128 of NaN take 4 ms
// forward, 19 backward (0.3 and 0.9 without).
#pragma once
#include "f32_split.h"

namespace linattn {
namespace f32 {

__device__ __forceinline__ void stf(float* p, size_t i, float v) { p[i] = v; }
__device__ __forceinline__ void stf(uint16_t* p, size_t i, float v) { p[i] = __builtin_bit_cast(uint16_t, (__bf16)v); }
__device__ __forceinline__ float wave_max(float x) {
  for (int m = 32; m >= 1; m >>= 1) x = fmaxf(x, __shfl_xor(x, m, 64));
  return x;
}
__device__ __forceinline__ float wave_sum(float x) {
  for (int m = 32; m >= 1; m >>= 1) x += __shfl_xor(x, m, 64);
  return x;
}

// Whether any of the eight flags of a workgroup is set (16-byte aligned LDS); the same in every lane.
__device__ __forceinline__ bool any_of_8(const int* flags) {
  const int4 a = reinterpret_cast<const int4*>(flags)[0], b = reinterpret_cast<const int4*>(flags)[1];
  return __builtin_amdgcn_readfirstlane((a.x | a.y) | (a.z | a.w) | (b.x | b.y) | (b.z | b.w)) != 0;
}

// Element i of a token's features or channels lives in lane i % 64, register i / 64.
template <int D, int KIND, typename T>
struct Plain {
  static constexpr int HALF = D / 2, L = D / 64;

  static __device__ __forceinline__ void phi(const T* row, const T* w, int lane, float (&f)[L]) {
    if constexpr (KIND == kPhiRelu) {
#pragma unroll
      for (int j = 0; j < L; ++j) f[j] = fmaxf(ldf(row, lane + 64 * j), 0.f);
    } else {
      float u = 0.f;
#pragma unroll
      for (int j = 0; j < L; ++j) {
        const float x = ldf(row, lane + 64 * j);
#pragma unroll 16
        for (int c = 0; c < 64; ++c) u = fmaf(__shfl(x, c, 64), ldf(w, (64 * j + c) * HALF + lane % HALF), u);
      }
      const float mx = wave_max(u), mn = -wave_max(-u);
      const float ep = expf(u - mx), em = expf(mn - u);
      constexpr float share = HALF == 32 ? 0.5f : 1.f;             // width 64: both halves of the wavefront hold the 32 features
      const float sp = wave_sum(ep) * share, sm = wave_sum(em) * share;
      if constexpr (L == 2) { f[0] = ep / sp; f[1] = em / sm; }
      else f[0] = lane < HALF ? ep / sp : em / sm;
    }
  }
  // Sum over the elements of a times row[i], rows of a [D][D] matrix: y[j] = sum_i a_i m[i][lane + 64j].
  static __device__ __forceinline__ void times(const float (&a)[L], const float* m, int lane, float (&y)[L]) {
#pragma unroll
    for (int j = 0; j < L; ++j) y[j] = 0.f;
#pragma unroll
    for (int h = 0; h < L; ++h)
#pragma unroll 16
      for (int i = 0; i < 64; ++i) {
        const float ai = __shfl(a[h], i, 64);
#pragma unroll
        for (int j = 0; j < L; ++j) y[j] = fmaf(ai, m[(64 * h + i) * D + lane + 64 * j], y[j]);
      }
  }
  static __device__ __forceinline__ float dot(const float (&a)[L], const float* z, int lane) {
    float s = 0.f;
#pragma unroll
    for (int j = 0; j < L; ++j) s = fmaf(a[j], z[lane + 64 * j], s);
    return wave_sum(s);
  }

  // One token of apply_f32_kernel: state is the head's [D+1][D].
  template <bool NORM, bool BLEND>
  static __device__ __forceinline__ void apply(const T* row, const T* w, const float* state, T* out, const T* blend, float rb, int lane) {
    float f[L], y[L];
    phi(row, w, lane, f);
    times(f, state, lane, y);
    float inv = 1.f;
    if constexpr (NORM) inv = 1.f / (dot(f, state + D * D, lane) + (KIND == kPhiRelu ? kReluEps : 0.f));
#pragma unroll
    for (int j = 0; j < L; ++j) {
      float v = NORM ? y[j] * inv : y[j];
      if constexpr (BLEND) v = fmaf(rb, ldf(blend, lane + 64 * j) - v, v);
      stf(out, lane + 64 * j, v);
    }
  }

  // One token of grad_f32_kernel.  QSIDE: *wt receives its weights, *dr (blend not null) its part of dL/dr.  du: element (feature a) of the token's dL/du
  // is du[(a's piece) * du_stride + a % 4], see dw_f32_kernel; nullable.
  template <bool QSIDE, bool BLEND>
  static __device__ __forceinline__ void grad(const T* xrow, const T* yrow, const T* w, const float* state, T* dx, float* du_tok, int nb,
                                              float2* wt, const T* blend, float om, float* dr, int lane) {
    const float* z = state + D * D;
    float f[L], g[L], gscale = 1.f;                                // dL/dphi / gscale
    phi(xrow, w, lane, f);
#pragma unroll
    for (int j = 0; j < L; ++j) {
      g[j] = 0.f;
#pragma unroll 16
      for (int c = 0; c < D; ++c) g[j] = fmaf(ldf(yrow, c), state[(lane + 64 * j) * D + c], g[j]);
    }
    if constexpr (QSIDE) {
      // delta as dO . o: o is an average of values, where phi . (dO S^T) may leave the range on the way
      const float inv = 1.f / (dot(f, z, lane) + (KIND == kPhiRelu ? kReluEps : 0.f));
      float part = 0.f, ds = 0.f, o[L];
      times(f, state, lane, o);
#pragma unroll
      for (int j = 0; j < L; ++j) {
        part = fmaf(ldf(yrow, lane + 64 * j), o[j] * inv, part);
        if (BLEND && blend != nullptr) ds = fmaf(ldf(yrow, lane + 64 * j), ldf(blend, lane + 64 * j), ds);
      }
      const float delta = wave_sum(part);
      if constexpr (BLEND) *dr += wave_sum(ds) - delta;
      const float a = inv * om;
      if (lane == 0) *wt = make_float2(a, -delta * a);
#pragma unroll
      for (int j = 0; j < L; ++j) g[j] -= delta * z[lane + 64 * j];
      gscale = a;
    } else {
#pragma unroll
      for (int j = 0; j < L; ++j) g[j] += z[lane + 64 * j];
    }
    if constexpr (KIND == kPhiRelu) {
#pragma unroll
      for (int j = 0; j < L; ++j) stf(dx, lane + 64 * j, f[j] > 0.f ? g[j] * gscale : 0.f);
    } else {
      float du;                                                    // of feature lane % HALF
      if constexpr (L == 2) {
        const float cp = wave_sum(g[0] * f[0]), cm = wave_sum(g[1] * f[1]);
        du = f[0] * (g[0] - cp) - f[1] * (g[1] - cm);
      } else {
        float c = g[0] * f[0];
        for (int m = 16; m >= 1; m >>= 1) c += __shfl_xor(c, m, 64);          // over the lane's half of the features
        const float d = f[0] * (g[0] - c), other = __shfl_xor(d, 32, 64);
        du = lane < HALF ? d - other : other - d;
      }
      du *= gscale;
      if (du_tok != nullptr && lane < HALF) {
        const int grp = lane / (D / 4), j = lane % (D / 4) / 4;
        du_tok[(size_t)(2 * j + grp) * nb * 4 + lane % 4] = du;
      }
      float y[L];
#pragma unroll
      for (int j = 0; j < L; ++j) y[j] = 0.f;
#pragma unroll 16
      for (int a = 0; a < HALF; ++a) {
        const float da = __shfl(du, a, 64);
#pragma unroll
        for (int j = 0; j < L; ++j) y[j] = fmaf(da, ldf(w, (lane + 64 * j) * HALF + a), y[j]);
      }
#pragma unroll
      for (int j = 0; j < L; ++j) stf(dx, lane + 64 * j, y[j]);
    }
  }

  // Tokens t0 .. t1-1 of StatePass::segment, eight at a time: wavefront w of 8 forms phi of one and sums the features w*D/8 .. +D/8-1 of
  // all, wavefront 0 z as well.  sf: 8 D floats of LDS.  Every thread of the workgroup calls it.
  template <bool WEIGHTED>
  static __device__ __forceinline__ void state(const T* xb, const T* yb, const T* w, const float2* weights, float* dst, int t0, int t1,
                                               size_t sn, float* sf, int wave, int lane) {
    constexpr int R = D / 8;
    float acc[R][L], z[L];
#pragma unroll
    for (int j = 0; j < L; ++j) {
      z[j] = 0.f;
#pragma unroll
      for (int r = 0; r < R; ++r) acc[r][j] = 0.f;
    }
    const int f0 = wave * R;
#pragma unroll 1
    for (int tg = t0; tg < t1; tg += 8) {
      const int own = tg + wave;
      if (own < t1) {
        float f[L];
        phi(xb + (size_t)own * sn, w, lane, f);
#pragma unroll
        for (int j = 0; j < L; ++j) sf[wave * D + lane + 64 * j] = f[j];
      }
      __syncthreads();
#pragma unroll 1
      for (int t = tg; t < tg + 8 && t < t1; ++t) {
        const float* f = sf + (t - tg) * D;
        const float2 wt = WEIGHTED ? weights[t] : make_float2(1.f, 1.f);
        float y[L];
#pragma unroll
        for (int j = 0; j < L; ++j) {
          z[j] = fmaf(f[lane + 64 * j], wt.y, z[j]);
          y[j] = ldf(yb + (size_t)t * sn, lane + 64 * j);
        }
#pragma unroll
        for (int r = 0; r < R; ++r) {
          const float a = f[f0 + r] * wt.x;
#pragma unroll
          for (int j = 0; j < L; ++j) acc[r][j] = fmaf(a, y[j], acc[r][j]);
        }
      }
      __syncthreads();
    }
#pragma unroll
    for (int j = 0; j < L; ++j) {
#pragma unroll
      for (int r = 0; r < R; ++r) dst[(f0 + r) * D + lane + 64 * j] = acc[r][j];
      if (wave == 0) dst[D * D + lane + 64 * j] = z[j];
    }
  }
};

}  // namespace f32
}  // namespace linattn
