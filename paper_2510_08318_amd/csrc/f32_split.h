// Building blocks of the fp32-arithmetic kernels (LINATTN_F32, LINATTN_BF16_F32MATH): fp32 products on the bf16 matrix
// cores.  An fp32 value is the exact sum of three bf16 pieces (8 significant bits each, the second and third
// signed), and a product a b is taken as the six piece products a_i b_j with i + j <= 2; what is left out is below
// 2^-24 |a b|, the size of one fp32 rounding.  A tensor stored as bf16 is its own single piece, so a product with it is
// three piece products and one of two such tensors is exact.  The accumulators are fp32 and take the 16 products of a step
// together, so a sum over n tokens sees n/16 roundings per piece product where a chain of scalar FMAs sees n.  bf16 has the
// exponent range of fp32: nothing needs scaling.  Values below 2^-110 lose the bits below 2^-133, the smallest bf16; infinities and
// finite values that round to Inf are left to f32_plain.h.
// The step's sum is cut, not rounded, below 1/16 unit of a larger accumulator: a bias of -1/32 unit per instruction, which a
// sum over many tokens would show (it is the same for every feature, so it does not average out in phi(q) S).  Such sums are
// therefore taken with alternating sign, tile by tile or wavefront by wavefront.
// Against fp32 FMAs on LDS tiles, which spend an LDS read per one or two FMAs and reach 7 TFLOP/s, the matrix cores do
// the six products at up to 400 TFLOP/s; against v_mfma_f32_32x32x2_f32 (157 TFLOP/s) they are 2.7 times as fast, and
// 5 times where one operand is stored as bf16.
#pragma once
#include "kernels.h"
#include "mfma_common.h"

namespace linattn {
namespace f32 {

constexpr int NT8 = 512;                         // 8 wavefronts, one workgroup per compute unit

template <typename T> constexpr int kPieces = sizeof(T) == 2 ? 1 : 3;

// Element access for the few scalar uses.
__device__ __forceinline__ float ldf(const float* p, size_t i) { return p[i]; }
__device__ __forceinline__ float ldf(const uint16_t* p, size_t i) { return __builtin_bit_cast(float, (uint32_t)p[i] << 16); }

__device__ __forceinline__ float lo_f32(uint32_t pair) { return __builtin_bit_cast(float, pair << 16); }
__device__ __forceinline__ float hi_f32(uint32_t pair) { return __builtin_bit_cast(float, pair & 0xffff0000u); }

// Two fp32 values -> three packed bf16 pairs whose sums are the values.  WIDE: also for finite values that round to Inf as bf16 (their
// first piece is then the largest bf16), one more operation a value.
template <bool WIDE = false>
__device__ __forceinline__ void split2(float a, float b, uint32_t& p0, uint32_t& p1, uint32_t& p2) {
  constexpr float top = 0x1.fep127f;
  p0 = WIDE ? pack_bf16x2(__builtin_amdgcn_fmed3f(a, -top, top), __builtin_amdgcn_fmed3f(b, -top, top)) : pack_bf16x2(a, b);
  const float a1 = a - lo_f32(p0), b1 = b - hi_f32(p0);
  p1 = pack_bf16x2(a1, b1);
  p2 = pack_bf16x2(a1 - lo_f32(p1), b1 - hi_f32(p1));
}
// Eight values -> the three pieces of an MFMA operand.
template <bool WIDE = false>
__device__ __forceinline__ void split8(const float* v, uint4 (&p)[3]) {
  split2<WIDE>(v[0], v[1], p[0].x, p[1].x, p[2].x);
  split2<WIDE>(v[2], v[3], p[0].y, p[1].y, p[2].y);
  split2<WIDE>(v[4], v[5], p[0].z, p[1].z, p[2].z);
  split2<WIDE>(v[6], v[7], p[0].w, p[1].w, p[2].w);
}
__device__ __forceinline__ void unpack_f32x4(uint4 r, float* v) {
  v[0] = __builtin_bit_cast(float, r.x); v[1] = __builtin_bit_cast(float, r.y);
  v[2] = __builtin_bit_cast(float, r.z); v[3] = __builtin_bit_cast(float, r.w);
}

__device__ __forceinline__ f32x16 zero16() {
  f32x16 z;
#pragma unroll
  for (int r = 0; r < 16; ++r) z[r] = 0.f;
  return z;
}
__device__ __forceinline__ f32x16 mfma_bf16(uint4 a, uint4 b, f32x16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(a), as_bf16x8(b), c, 0, 0, 0);
}
// The piece products of one k-step, small terms first, for NI x NJ accumulators: acc[i][j] += a[i] b[j].
template <int NA, int NB, int NI, int NJ>
__device__ __forceinline__ void mfma_pieces(const uint4 (&a)[NI][NA], const uint4 (&b)[NJ][NB], f32x16 (&acc)[NI][NJ]) {
#pragma unroll
  for (int s = (NA + NB - 2 < 2 ? NA + NB - 2 : 2); s >= 0; --s)
#pragma unroll
    for (int pa = 0; pa < NA; ++pa) {
      const int pb = s - pa;
      if (pb < 0 || pb >= NB) continue;
#pragma unroll
      for (int i = 0; i < NI; ++i)
#pragma unroll
        for (int j = 0; j < NJ; ++j) acc[i][j] = mfma_bf16(a[i][pa], b[j][pb], acc[i][j]);
    }
}

// A lane's share of a token row in operand order: octet ks = channels 16ks + 8g .. +7 (g = lane/32), as stored.
template <int D, typename T>
struct RowOctets {
  static constexpr int NU = sizeof(T) / 2;       // 16-byte words per octet
  uint4 r[D / 16 * NU];
  template <int LO = 0, int HI = D / 16>
  __device__ __forceinline__ void load(const T* row, int g) { load(row, g, LO, HI); }
  __device__ __forceinline__ void load(const T* row, int g, int lo, int hi) {        // constants after inlining
    const uint4* p = reinterpret_cast<const uint4*>(row);
#pragma unroll
    for (int ks = lo; ks < hi; ++ks)
#pragma unroll
      for (int i = 0; i < NU; ++i) r[ks * NU + i] = p[(2 * ks + g) * NU + i];
  }
  __device__ __forceinline__ void values(int ks, float* v) const {
    if constexpr (sizeof(T) == 2) unpack_bf16x8(r[ks], v);
    else { unpack_f32x4(r[2 * ks], v); unpack_f32x4(r[2 * ks + 1], v + 4); }
  }
  __device__ __forceinline__ void pieces(int ks, uint4 (&p)[kPieces<T>]) const {
    if constexpr (sizeof(T) == 2) p[0] = r[ks];
    else {
      float v[8];
      values(ks, v);
      split8(v, p);
    }
  }
};

// Octet ks of phi on lane group g: features phi_feature<D, KIND>(ks, g) .. +7 (Eq. 5 order; ReLU: the channels).
template <int D, int KIND>
__device__ __forceinline__ constexpr int phi_feature(int ks, int g) {
  return KIND == kPhiRelu ? 16 * ks + 8 * g : ApplyLayout<D>::feature(ks, g, 0);
}

// W~ of one head (D x D/2, stored as T) -> pieces of the A operands of U^T = W~^T X^T in LDS, entry (ks, mb, lane = (m, g)) of
// a piece holds
// W~[16ks + 8g + e][owned_row<D/2>(mb, m)], e = 0..7.  A thread reads four adjacent features of eight channels at a time.
template <int D, typename T, int NTHREADS>
__device__ __forceinline__ void build_w_pieces(const T* __restrict__ w, uint4* sW, int tid) {
  using C = Cfg<D>;
  constexpr int ITEMS = C::UK * 2 * C::UM * 8;
  for (int it = tid; it < ITEMS; it += NTHREADS) {
    const int mq = it % 8, mb = (it / 8) % C::UM, g = (it / (8 * C::UM)) % 2, ks = it / (16 * C::UM);
    const T* src = w + (16 * ks + 8 * g) * C::HALF + owned_row<C::HALF>(mb, 4 * mq);
    float v[4][8];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      if constexpr (sizeof(T) == 2) {
        const uint2 r = *reinterpret_cast<const uint2*>(src + e * C::HALF);
        v[0][e] = lo_f32(r.x); v[1][e] = hi_f32(r.x); v[2][e] = lo_f32(r.y); v[3][e] = hi_f32(r.y);
      } else {
        const float4 r = *reinterpret_cast<const float4*>(src + e * C::HALF);
        v[0][e] = r.x; v[1][e] = r.y; v[2][e] = r.z; v[3][e] = r.w;
      }
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      uint4 p[3];
      split8(v[q], p);                           // bf16: the first piece is the value, the others are zero and unused
      uint4* dst = sW + (ks * C::UM + mb) * 64 + 32 * g + 4 * mq + q;
#pragma unroll
      for (int i = 0; i < kPieces<T>; ++i) dst[i * C::W_IMG] = p[i];
    }
  }
}

// Whether an fp32 value's first piece is finite (f32_plain.h has the rest).
__device__ __forceinline__ bool splits(float v) { return fabsf(v) < 0x1.ffp127f; }
__device__ __forceinline__ bool splits8(const float* v) {
  return splits(fmaxf(fmaxf(fmaxf(fabsf(v[0]), fabsf(v[1])), fmaxf(fabsf(v[2]), fabsf(v[3]))),
                      fmaxf(fmaxf(fabsf(v[4]), fabsf(v[5])), fmaxf(fabsf(v[6]), fabsf(v[7])))));
}

// State [D+1][D] of one head -> pieces of the B operands of Y = phi S in LDS: entry (ks, mb, lane = (c, g)) of a piece holds
// S[phi_feature(ks, g) + e][channel_cols(mb, c)].  A thread reads the MB adjacent channels of eight features at a time.
// Returns whether every value the thread met splits (a NaN passes: it stays one).
template <int D, int KIND, int NTHREADS>
__device__ __forceinline__ bool build_s_pieces(const float* __restrict__ S, uint4* sS, int tid) {
  using L = ApplyLayout<D>;
  constexpr int IMG = L::KS * L::MB * 64;
  bool all = true;
  for (int it = tid; it < L::KS * 64; it += NTHREADS) {
    const int lane = it % 64, ks = it / 64;
    const float* src = S + phi_feature<D, KIND>(ks, lane / 32) * D + L::MB * (lane % 32);
    float v[L::MB][8];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      if constexpr (L::MB == 4) {
        const float4 r = *reinterpret_cast<const float4*>(src + e * D);
        v[0][e] = r.x; v[1][e] = r.y; v[2][e] = r.z; v[3][e] = r.w;
      } else {
        const float2 r = *reinterpret_cast<const float2*>(src + e * D);
        v[0][e] = r.x; v[1][e] = r.y;
      }
    }
#pragma unroll
    for (int mb = 0; mb < L::MB; ++mb) {
      uint4 p[3];
      split8(v[mb], p);
      all = all && splits8(v[mb]);
#pragma unroll
      for (int i = 0; i < 3; ++i) sS[i * IMG + (ks * L::MB + mb) * 64 + lane] = p[i];
    }
  }
  return all;
}

// U^T = W~^T X^T for the 32 tokens of a wavefront (see project): u[mb][r] = pre-softmax feature g*LOC + 16mb + r of the lane's token.
template <int D, typename T>
__device__ __forceinline__ void project(const RowOctets<D, T>& x, const uint4* sW, int lane, f32x16 (&u)[Cfg<D>::UM][1]) {
  using C = Cfg<D>;
  constexpr int NX = kPieces<T>;
#pragma unroll
  for (int mb = 0; mb < C::UM; ++mb) u[mb][0] = zero16();
  const uint4* wa = sW + lane + opaque_zero();
#pragma unroll
  for (int ks = 0; ks < C::UK; ++ks) {
    uint4 b[1][NX], a[C::UM][NX];
    x.pieces(ks, b[0]);
#pragma unroll
    for (int mb = 0; mb < C::UM; ++mb)
#pragma unroll
      for (int i = 0; i < NX; ++i) a[mb][i] = wa[i * C::W_IMG + (ks * C::UM + mb) * 64];
    mfma_pieces<NX, NX>(a, b, u);
  }
}

// phi of the lane's token as KS octets (Eq. 5 from the accumulators of project): softmax(+u) then softmax(-u).
// exp(u - m) is 2^((u - m) log2 e), the difference first: it is exact near the maximum, so the largest term is 1 to the last bit, a
// saturated map has p = 1 and its Jacobian vanishes, and no |u| is too large.  (As one fma, u log2 e - m log2 e, an operation less per
// exponential and 0.5 to 1 % of a pass, the errors are the same elsewhere, but p = 1 - 2^-24 there.)
template <int D>
__device__ __forceinline__ void softmax_octets(const f32x16 (&u)[Cfg<D>::UM][1], float (&f)[D / 2]) {
  using C = Cfg<D>;
  float mx = u[0][0][0], mn = mx;
#pragma unroll
  for (int mb = 0; mb < C::UM; ++mb)
#pragma unroll
    for (int r = 0; r < 16; ++r) { mx = fmaxf(mx, u[mb][0][r]); mn = fminf(mn, u[mb][0][r]); }
  float lo, hi;
  pair32(mx, lo, hi); mx = fmaxf(lo, hi);
  pair32(mn, lo, hi); mn = fminf(lo, hi);
  float sp = 0.f, sm = 0.f;
#pragma unroll
  for (int mb = 0; mb < C::UM; ++mb)
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const float a = __builtin_amdgcn_exp2f((u[mb][0][r] - mx) * kLog2e), b = __builtin_amdgcn_exp2f((mn - u[mb][0][r]) * kLog2e);
      f[16 * mb + r] = a; f[C::LOC + 16 * mb + r] = b;
      sp += a; sm += b;
    }
  pair32(sp, lo, hi); sp = lo + hi;
  pair32(sm, lo, hi); sm = lo + hi;
  const float ip = 1.0f / sp, im = 1.0f / sm;
#pragma unroll
  for (int j = 0; j < C::LOC; ++j) { f[j] *= ip; f[C::LOC + j] *= im; }
}

// phi of the lane's token, either map.
template <int D, int KIND, typename T>
__device__ __forceinline__ void phi_octets(const RowOctets<D, T>& x, const uint4* sW, int lane, float (&f)[D / 2]) {
  if constexpr (KIND == kPhiRelu) {
#pragma unroll
    for (int ks = 0; ks < D / 16; ++ks) {
      x.values(ks, f + 8 * ks);
#pragma unroll
      for (int e = 0; e < 8; ++e) f[8 * ks + e] = fmaxf(f[8 * ks + e], 0.f);
    }
  } else {
    f32x16 u[Cfg<D>::UM][1];
    project<D, T>(x, sW, lane, u);
    softmax_octets<D>(u, f);
  }
}

// [D] vector of a head (z, dz) -> LDS in the octet order of the lanes: element (ks*2 + g)*8 + e.
template <int D, int KIND, int NTHREADS>
__device__ __forceinline__ void build_octet_vector(const float* __restrict__ z, float* s, int tid) {
  for (int i = tid; i < D; i += NTHREADS) s[i] = z[phi_feature<D, KIND>(i / 16, (i / 8) % 2) + i % 8];
}
// Dot product of the lane's octets with such a vector, over the whole token (both lanes of a pair get it).
template <int D>
__device__ __forceinline__ float octet_dot(const float (&f)[D / 2], const float* s, int g) {
  float acc = 0.f;
#pragma unroll
  for (int ks = 0; ks < D / 16; ++ks)
#pragma unroll
    for (int e = 0; e < 8; ++e) acc = fmaf(f[8 * ks + e], s[(2 * ks + g) * 8 + e], acc);
  float lo, hi;
  pair32(acc, lo, hi);
  return lo + hi;
}

// Rows of an accumulator with the tokens on its rows (lane (c, g), register r: token t0 + 8*(r/4) + 4g + r%4, channels MB*c .. +MB-1):
// value(r, mb) is stored as T.
template <int D, typename T, typename Value>
__device__ __forceinline__ void store_rows(T* base, size_t sn, int t0, int n, int lane, Value value) {
  constexpr int MB = D / 32;
  const TokenRows<MB * (int)sizeof(T)> rows(base, sn * sizeof(T), t0, n, lane);
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    float y[MB];
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) y[mb] = value(r, mb);
    if constexpr (sizeof(T) == 4) {
      typedef float vec __attribute__((ext_vector_type(MB)));
      vec v;
#pragma unroll
      for (int mb = 0; mb < MB; ++mb) v[mb] = y[mb];
      rows.template store<true>(r, v);
    } else if constexpr (MB == 4) {
      rows.template store<true>(r, make_uint2(pack_bf16x2(y[0], y[1]), pack_bf16x2(y[2], y[3])));
    } else {
      rows.template store<true>(r, pack_bf16x2(y[0], y[1]));
    }
  }
}

}  // namespace f32
}  // namespace linattn
