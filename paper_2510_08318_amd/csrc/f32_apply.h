// phi(x_i) M for every token, in fp32 arithmetic on the bf16 matrix cores (f32_split.h).
#pragma once
#include "f32_split.h"
#include "f32_plain.h"

namespace linattn {
namespace f32 {

// The query pass, out = phi(q) S / (phi(q) . z).  8 wavefronts, one workgroup per compute unit, each wavefront on its own 32-token blocks; LDS holds
// the pieces of W~_q and of the S image (144 KB for fp32 tensors of width 128).  The normaliser is an in-lane dot product (a
// lane pair owns the token) and goes into phi before it is split, so the product with S is the output and leaves the
// accumulators as whole rows.
template <int D, int KIND, typename T>
constexpr size_t apply_smem() {
  return ((KIND == kPhiRelu ? 0 : kPieces<T> * Cfg<D>::W_IMG) + 3 * ApplyLayout<D>::KS * ApplyLayout<D>::MB * 64) * sizeof(uint4) + (D + NT8 / 64) * sizeof(float);
}
template <int D, int KIND, typename T, bool BLEND, bool EVEN>
__global__ __launch_bounds__(NT8) void apply_f32_kernel(const T* __restrict__ q, const T* __restrict__ wq,
                                                        const float* __restrict__ state, T* __restrict__ out,
                                                        const T* __restrict__ blend, const float* __restrict__ rptr,
                                                        int H, int n, Split deal, Rows rw) {
  using L = ApplyLayout<D>;
  constexpr int IMG = L::KS * L::MB * 64;
  extern __shared__ uint4 smem[];
  uint4* sW = smem;
  uint4* sS = sW + (KIND == kPhiRelu ? 0 : kPieces<T> * Cfg<D>::W_IMG);
  float* sZ = reinterpret_cast<float*>(sS + 3 * IMG);
  int* sPlain = reinterpret_cast<int*>(sZ + D);            // [8] the wavefront has met a state value that does not split (f32_plain.h)

  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x / 64);
  // EVEN: the deal may give the workgroup parts of two heads
  for (Share sh = EVEN ? first_share(deal, blockIdx.x, blockIdx.y) : head_share(deal, blockIdx.x, blockIdx.y); sh.there;
       sh = EVEN ? next_share(deal, blockIdx.x, sh) : Share{}) {
    // (from a thread index that the optimiser cannot hoist: what depends on it would be held, or spilled, across the loop)
    const int tid = EVEN ? (threadIdx.x + opaque_zero()) & (NT8 - 1) : threadIdx.x, lane = tid % 64, g = lane / 32, c = lane % 32;
    const int bh = sh.bh, h = bh % H;
    const T* qb = q + head_base(rw, bh, H);
    T* ob = out + head_base(rw, bh, H);
    // mixed attention (Eq. 6): out = r' s + (1 - r') o with r' = clip(r, 0, 1)
    const T* bb = BLEND ? blend + head_base(rw, bh, H) : nullptr;
    const float rb = BLEND ? fminf(fmaxf(*rptr, 0.f), 1.f) : 0.f;
    const float* sb = state + (size_t)bh * (D + 1) * D;

    const Blocks own = blocks_of(deal, sh, w, (n + 31) / 32);
    const int nblk = own.end, stride = own.stride;
    RowOctets<D, T> x;
    auto load = [&](int b) {
      const int t = b * 32 + c;
      x.load(qb + (size_t)(t < n ? t : n - 1) * rw.sn, g);
    };
    int b = own.first;
    load(b < nblk ? b : nblk - 1);
    if constexpr (KIND == kPhiHedgehog) build_w_pieces<D, T, NT8>(wq + (size_t)h * D * (D / 2), sW, tid);
    const bool state_splits = build_s_pieces<D, KIND, NT8>(sb, sS, tid);
    if (lane == 0) sPlain[w] = 0;
    if (!state_splits) sPlain[w] = 1;                        // (after lane 0's store: one wavefront's LDS operations are in order)
    build_octet_vector<D, KIND, NT8>(sb + D * D, sZ, tid);
    __syncthreads();

    const int b_own = b;
    const bool state_plain = any_of_8(sPlain);
    float chk = 0.f;                                         // NaN once the lane has met what does not split
    for (; b < nblk; b += stride) {
      float f[D / 2];
      phi_octets<D, KIND, T>(x, sW, lane, f);
      load(b + stride < nblk ? b + stride : b);
      const float inv = 1.0f / (octet_dot<D>(f, sZ + opaque_zero(), g) + (KIND == kPhiRelu ? kReluEps : 0.f));
      // phi is at most 1 and splits, unless an x or u that did not made its half NaN (and with it den)
      if constexpr (KIND == kPhiHedgehog) chk = fmaf(inv * 0x1p8f, 0.f, chk);
      f32x16 o[1][L::MB];
#pragma unroll
      for (int mb = 0; mb < L::MB; ++mb) o[0][mb] = zero16();
      const uint4* ss = sS + lane + opaque_zero();
#pragma unroll
      for (int ks = 0; ks < L::KS; ++ks) {
        uint4 a[1][3], s[L::MB][3];
#pragma unroll
        for (int mb = 0; mb < L::MB; ++mb)
#pragma unroll
          for (int i = 0; i < 3; ++i) s[mb][i] = ss[i * IMG + (ks * L::MB + mb) * 64];
        float v[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] = f[8 * ks + e] * inv;
        split8(v, a[0]);
        mfma_pieces<3, 3>(a, s, o);
      }
      if constexpr (KIND == kPhiRelu) {
        // a feature that does not split makes all of its token's row NaN or Inf: one channel a row tells
#pragma unroll
        for (int r = 0; r < 16; ++r) chk = fmaf(o[0][0][r], 0.f, chk);
      }
      if constexpr (BLEND) {
        const int t0 = b * 32;
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int t = t0 + 8 * (r / 4) + 4 * g + (r % 4);
          const T* srow = bb + (size_t)(t < n ? t : n - 1) * rw.sn + L::MB * c;
#pragma unroll
          for (int mb = 0; mb < L::MB; ++mb) o[0][mb][r] = fmaf(rb, ldf(srow, mb) - o[0][mb][r], o[0][mb][r]);
        }
      }
      store_rows<D, T>(ob, rw.sn, b * 32, n, lane, [&](int r, int mb) { return o[0][mb][r]; });
    }
    if (__builtin_expect(state_plain || __any(chk != chk), 0)) {
      __threadfence();                                       // the rows stored above are written again
#pragma unroll 1
      for (b = b_own; b < nblk; b += stride)
#pragma unroll 1
        for (int t = 32 * b; t < 32 * b + 32 && t < n; ++t) {
          const size_t at = (size_t)t * rw.sn;
          Plain<D, KIND, T>::template apply<true, BLEND>(qb + at, wq + (size_t)h * D * (D / 2), sb, ob + at, BLEND ? bb + at : nullptr, rb, lane);
        }
    }
    if (EVEN && sh.rest < sh.hi) __syncthreads();        // the next head's images take the place of these
  }
}

// What the deal of the passes with images of pieces costs.  Arithmetic bounds a round: query pass, a forward call head by head / evenly, us, bf16
// tensors 12 heads x 32760 (7 / 6 rounds) 151.8 / 149.5, 160 x 1555 (7 / 5) 118.2 / 113.6, ReLU 161 x 1598 96.4 / 91.8, fp32 tensors 12 x 32760 271.8 /
// 266.9, 24 x 8000 (4 / 3) 151.5 / 142.0, 153 x 763 (3 / 2) 120 / 117.  With fp32 tensors and no projection (ReLU) or one tensor more (blend) the memory
// system does: ReLU 169 x 731 88.6 / 91.7, 153 x 763 89.4 / 91.6, with blend 142 x 1013 (4 / 3) 137.1 / 139.3, 151 x 607 90.9 / 95.1; but ReLU 12 x 32760
// 209.1 / 204.5, with blend 168 x 2213 (9 / 6) 297.5 / 291.2.  A pass with heads of its own keeps the loop-free form (EVEN = false): the loop over a
// workgroup's heads costs it up to half a microsecond.
template <int KIND, typename T, bool BLEND>
constexpr DealCost kF32Cost = sizeof(T) == 4 && (KIND == kPhiRelu || BLEND) ? DealCost{3, 2, 5} : DealCost{3};
template <int D, int KIND, typename T, bool BLEND>
hipError_t run_apply_pass(const void* q, const void* wq, const float* state, void* out,
                     const void* blend_in, const float* blend_r, const Plan& p, hipStream_t s) {
  constexpr size_t smem = apply_smem<D, KIND, T>();
  constexpr bool EV = D == 128;                            // (width 64 has little to gain)
  // (fp32 tensors at width 128: units of two wherever they fit, units of four / two, a call, 16 heads x 500 35.1 / 34.2, 32 x 500 38.5 / 38.3)
  constexpr UnitLimits most = D == 128 && sizeof(T) == 4 ? kNoUnitLimits : UnitLimits();
  const Split deal = make_deal_of_blocks(p.BH, (p.n + 31) / 32, NT8 / 64, kF32Cost<KIND, T, BLEND>, EV, 1, most);
  auto launch = [&](auto kernel) -> hipError_t {
    const hipError_t e = set_smem_once<decltype(kernel)::value>(smem);
    if (e != hipSuccess) return e;
    decltype(kernel)::value<<<grid_of(deal), NT8, smem, s>>>((const T*)q, (const T*)wq, state, (T*)out, (const T*)blend_in, blend_r, p.H, p.n, deal, p.rows);
    return hipGetLastError();
  };
  if constexpr (EV)
    if (!deal.share) return launch(KernelTag<apply_f32_kernel<D, KIND, T, BLEND, true>>{});
  return launch(KernelTag<apply_f32_kernel<D, KIND, T, BLEND, false>>{});
}

}  // namespace f32
}  // namespace linattn
