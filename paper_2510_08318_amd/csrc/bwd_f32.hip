// fp32-arithmetic backward path, on fp32 tensors (the 1e-5 accuracy contract) or on bf16 tensors (LINATTN_BF16_F32MATH), every
// product on exact bf16 pieces (f32_split.h).  Same mathematics as bwd_bf16.h (chain rule through Eq. 3 and Eq. 5):
//   grad_f32_kernel, query side : phi(q), den, G = dO S^T, delta = phi . G / den, dL/dphi = (G - delta z) / den, du, dq
//   state_f32_kernel (weighted) : dS = sum phi(q)^T dO / den, dz = -sum phi(q) delta / den; split-n partials, reduced
//   grad_f32_kernel, key side   : phi(k), dv = phi(k) dS, dL/dphi = v dS^T + dz, du, dk
//   dw_f32_kernel               : dW~ = sum x^T du, both sides, from the du rows the two passes above leave in the workspace
// The three pieces of one state image and of W~ fill the LDS of a compute unit (144 KB at width 128), which is why the sum over
// tokens is a pass of its own.  delta needs no o: phi . (S dO) is o . dO times den.
#include "kernels.h"
#include "f32_split.h"
#include "f32_plain.h"
#include "f32_state.h"
#include "f32_apply.h"

namespace linattn {
namespace {

using namespace f32;

// W~ of one head -> pieces of the B operands of dX = dU W~^T in LDS: entry (ks, mb, lane = (c, g)) holds
// W~[channel_cols(mb, c)][g*LOC + 8ks + e], e = 0..7.  The same entries serve the projection: a transposing read of four of them
// gives four channels of four adjacent features.  The lane index is XORed so that both kinds of read spread over the banks.
template <int D>
struct WImage {
  using C = Cfg<D>;
  using L = ApplyLayout<D>;
  static constexpr int KS = C::LOC / 8;
  static constexpr int IMG = KS * L::MB * 64;                     // 16-byte entries of one piece (= Cfg<D>::W_IMG)
  static __device__ __forceinline__ int place(int ks, int mb, int lane) {
    return (ks * L::MB + mb) * 64 + (lane ^ (2 * mb + lane / 32 + 8 * (ks & 1)));
  }
  template <typename T, int NTHREADS>
  static __device__ __forceinline__ void build(const T* __restrict__ w, uint4* sW, int tid) {
    for (int it = tid; it < IMG; it += NTHREADS) {
      const int lane = it % 64, mb = (it / 64) % L::MB, ks = it / (64 * L::MB);
      const T* src = w + L::channel_cols(mb, lane % 32) * C::HALF + (lane / 32) * C::LOC + 8 * ks;
      uint4* dst = sW + place(ks, mb, lane);
      if constexpr (sizeof(T) == 2) {
        *dst = *reinterpret_cast<const uint4*>(src);
      } else {
        float v[8];
        unpack_f32x4(reinterpret_cast<const uint4*>(src)[0], v);
        unpack_f32x4(reinterpret_cast<const uint4*>(src)[1], v + 4);
        uint4 p[3];
        split8(v, p);
#pragma unroll
        for (int i = 0; i < 3; ++i) dst[i * IMG] = p[i];
      }
    }
  }
  // A operand (ks, mbu) of U^T = W~^T X^T, piece p.  Lane (s = lane%16, j = (lane/16)%2, g = lane/32) points at channel
  // 16ks + 8g + 4h + s/4 and the four features (s%2)*LOC + 16mbu + 8j + 4*((s/2)%2) of the half h of the operand.
  static __device__ __forceinline__ uint4 project_operand(const uint4* sW, int p, int ks, int mbu, int lane) {
    const int s = lane % 16, j = (lane / 16) % 2, g = lane / 32;
    const int fixed = (2 * mbu + j) * L::MB * 64 * 16 + 8 * ((s / 2) % 2) + 512 * (s % 2);
    int off[2];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int channel = 16 * ks + 8 * g + 4 * h + s / 4;
      const int mb = channel % L::MB, c = channel / L::MB;
      off[h] = fixed + mb * 1024 + ((c ^ (2 * mb + s % 2 + 8 * j)) << 4);
    }
    return __builtin_bit_cast(uint4, read_tr(reinterpret_cast<const char*>(sW + p * IMG), off[0], off[1]));
  }
  template <typename T>
  static __device__ __forceinline__ void project(const RowOctets<D, T>& x, const uint4* sW, int lane, f32x16 (&u)[C::UM][1]) {
    constexpr int NX = kPieces<T>;
#pragma unroll
    for (int mb = 0; mb < C::UM; ++mb) u[mb][0] = zero16();
#pragma unroll
    for (int ks = 0; ks < C::UK; ++ks) {
      uint4 b[1][NX], a[C::UM][NX];
      x.pieces(ks, b[0]);
#pragma unroll
      for (int mb = 0; mb < C::UM; ++mb)
#pragma unroll
        for (int i = 0; i < NX; ++i) a[mb][i] = project_operand(sW, i, ks, mb, lane);
      mfma_pieces<NX, NX>(a, b, u);
    }
  }
};

// State M (S or dS) of one head -> pieces of the A operands of G^T = M Y^T in LDS: entry (ks, mb, lane = (m, g)) holds
// M[row(mb, m)][channel(ks, g, e)], e = 0..7; the rows are ordered so that accumulator register r of block mb is element 16mb + r of the lane's phi.
// The same entries serve Y = phi M as B operands (column_operand): a transposing read gives four lanes the four channels of half an
// entry, so the channels of a half are those that four lanes want for one column block, MB channels apart, among the ones that a lane
// group of Y holds.  The lane index and the halves are XORed so that both kinds of read spread over the banks.
// COLUMNS = false: channels in their order, for an image that is read by rows only.
template <int D, bool COLUMNS>
struct GImage {
  static constexpr int MB = D / 32, KS = D / 16;
  static constexpr int IMG = KS * MB * 64;                        // 16-byte entries of one piece
  static constexpr int KP = COLUMNS ? D / 64 : 1;                               // k-steps that share the octets of a lane group
  // Element e of k-step ks is value index(ks, e) of the KP octets KP*(ks/KP) .. of the lane group.
  static constexpr int index(int ks, int e) { return COLUMNS ? MB * (e % 4) + 2 * (ks % KP) + e / 4 : e; }
  static __device__ __forceinline__ int place(int ks, int mb, int lane) {
    return (ks * MB + mb) * 64 + (COLUMNS ? lane ^ (8 * (lane / 32)) ^ (16 * (ks / KP >> 1)) : lane);
  }
  static __device__ __forceinline__ uint4 halves(int ks, uint4 v) { return COLUMNS && ks / KP % 2 ? make_uint4(v.z, v.w, v.x, v.y) : v; }
  // Returns whether every value the thread met splits (see build_s_pieces).
  template <int KIND, int NTHREADS>
  static __device__ __forceinline__ bool build(const float* __restrict__ M, uint4* sG, int tid) {
    bool all = true;
    for (int it = tid; it < IMG / KP; it += NTHREADS) {
      const int lane = it % 64, mb = (it / 64) % MB, p = it / (64 * MB);
      const int m = lane % 32, r = 4 * (m / 8) + m % 4;
      const int row = phi_feature<D, KIND>(2 * mb + r / 8, (m / 4) % 2) + r % 8;
      float v[8 * KP];
#pragma unroll
      for (int o = 0; o < KP; ++o) {
        const uint4* src = reinterpret_cast<const uint4*>(M + row * D + 16 * (KP * p + o) + 8 * (lane / 32));
        unpack_f32x4(src[0], v + 8 * o);
        unpack_f32x4(src[1], v + 8 * o + 4);
        all = all && splits8(v + 8 * o);
      }
#pragma unroll
      for (int t = 0; t < KP; ++t) {
        float w[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) w[e] = v[index(t, e)];
        uint4 q[3];
        split8(w, q);
        uint4* dst = sG + place(KP * p + t, mb, lane);
#pragma unroll
        for (int i = 0; i < 3; ++i) dst[i * IMG] = halves(KP * p, q[i]);
      }
    }
    return all;
  }
  static __device__ __forceinline__ uint4 row_operand(const uint4* sG, int piece, int ks, int mb, int lane) {
    return halves(ks, sG[piece * IMG + place(ks, mb, lane)]);
  }
  // Pieces of k-step ks of Y, channels in the order of the entries.
  template <typename T>
  static __device__ __forceinline__ void y_pieces(const RowOctets<D, T>& y, int ks, uint4 (&p)[kPieces<T>]) {
    if constexpr (!COLUMNS) { y.pieces(ks, p); return; }
    const int o0 = KP * (ks / KP), t = ks % KP;
    if constexpr (sizeof(T) == 2) {
      uint32_t w[4 * KP];
#pragma unroll
      for (int o = 0; o < KP; ++o) {
        w[4 * o] = y.r[o0 + o].x; w[4 * o + 1] = y.r[o0 + o].y; w[4 * o + 2] = y.r[o0 + o].z; w[4 * o + 3] = y.r[o0 + o].w;
      }
      auto lo = [](uint32_t a, uint32_t b) { return (a & 0xffffu) | (b << 16); };
      auto hi = [](uint32_t a, uint32_t b) { return (a >> 16) | (b & 0xffff0000u); };
      const uint32_t a = w[t], b = w[MB / 2 + t], c = w[MB + t], d = w[3 * MB / 2 + t];       // values MB q + 2t, + 1
      p[0] = make_uint4(lo(a, b), lo(c, d), hi(a, b), hi(c, d));
    } else {
      float v[8 * KP], w[8];
#pragma unroll
      for (int o = 0; o < KP; ++o) y.values(o0 + o, v + 8 * o);
#pragma unroll
      for (int e = 0; e < 8; ++e) w[e] = v[index(ks, e)];
      split8(w, p);
    }
  }
  // B operand (ks, mb) of Y = phi M: lane (c, g) receives M[phi octet ks of group g][MB * column(c) + mb].  Lane (s = lane%16, j = (lane/16)%2, g)
  // points at row s/4 of half h of the octet and at four channels of the quad of columns 4j + s%4.
  static __device__ __forceinline__ int column_base(int lane) {
    const int s = lane % 16, j = (lane / 16) % 2, g = lane / 32;
    const int quad = 4 * j + s % 4, p = quad / 2, gl = quad % 2;
    return KP * p * MB * 1024 + 512 * gl + 16 * ((s / 4 + 4 * g) ^ (8 * gl) ^ (16 * (p >> 1))) + 8 * (p & 1);
  }
  static __device__ __forceinline__ uint4 column_operand(const uint4* sG, int piece, int ks, int mb, int base) {
    const char* img = reinterpret_cast<const char*>(sG + piece * IMG) + (mb / 2 * MB + ks / 2) * 1024;
    const int at = base ^ (256 * (ks % 2) + 8 * (mb % 2));
    return __builtin_bit_cast(uint4, read_tr(img, at, at ^ 128));
  }
  static __device__ __forceinline__ int column(int c) {
    return MB == 4 ? 8 * (c / 8) + 2 * (c / 4 % 2) + 4 * (c / 2 % 2) + c % 2 : c;
  }
};

// Where an even deal of the gradient kernels is considered: fp32 rows of width 128 have no registers for its loop, and width 64 has little to gain.
template <int D, typename T> constexpr bool grad_even = D == 128 && kPieces<T> == 1;

template <int D, int KIND, typename T>
constexpr size_t grad_smem() {
  return ((KIND == kPhiRelu ? 0 : kPieces<T> * WImage<D>::IMG) + 3 * GImage<D, false>::IMG) * sizeof(uint4) + (D + 2 * NT8 / 64) * sizeof(float);
}

// dL/du rows: non-temporal where both sides' would push each other and the rows that follow out of the last-level cache (256 MB) before
// dw_f32_kernel reads them.  Ordinary / non-temporal, us: 12 heads x 32760 x 128 (201 MB) dw 99.5 / 86, key side 149 / 147, query side 101 / 102 (both head by head); 5 x
// 20000 x 128 (51 MB) dw 47 / 49, gradients 147 / 144.
constexpr size_t kDuStreamBytes = 128u << 20;
__device__ __forceinline__ void put_du(float4* p, float4 v, int stream) {
  if (stream) st_nt(reinterpret_cast<uint4*>(p), __builtin_bit_cast(uint4, v));
  else *p = v;
}

// 8 wavefronts, one workgroup per compute unit, each wavefront on its own 32-token blocks (a lane pair owns a token).
// QSIDE: x = q, y = dO, M = (S, z); leaves the weights of the sum over tokens, {om / den, -om delta / den}, in weights[bh][t] and
// (BLEND, dr_part not null) the workgroup's part of dL/dr = sum dO . (s - o) in dr_part; om = 1 - r' of the mixed attention.  s is read for
// that alone.
// Key side: x = k, y = v, M = (dS, dz); dv = phi(k) dS as well, from the same image.  As a pass of its own it read k, formed phi and built an
// image once more; two passes / this one, us, as it was first: 12 heads x 32760 x 128 with bf16 tensors 97 + 80 / 161 (147 now), 5 x 20000 x 128 fp32 61 +
// 37 / 84, 2 x 1024 x 64 fp32 12.3 + 7.8 / 15.4 (14.9).  du_ws (nullable): dL/du rows for dW~.
template <int D, int KIND, typename T, bool QSIDE, bool BLEND, bool EVEN>
__global__ __launch_bounds__(NT8) void grad_f32_kernel(const T* __restrict__ x, const T* __restrict__ y, const T* __restrict__ wx,
                                                       const float* __restrict__ state, T* __restrict__ dx, T* __restrict__ dv,
                                                       float* __restrict__ du_ws, int du_stream,
                                                       float2* __restrict__ weights, const T* __restrict__ blend,
                                                       const float* __restrict__ rptr, float* __restrict__ dr_part,
                                                       int H, int n, Split deal, Rows rw) {
  using C = Cfg<D>;
  using L = ApplyLayout<D>;
  using W = WImage<D>;
  using GI = GImage<D, !QSIDE>;
  constexpr int MB = L::MB, NX = kPieces<T>;
  extern __shared__ uint4 smem[];
  uint4* sW = smem;
  uint4* sG = sW + (KIND == kPhiRelu ? 0 : NX * W::IMG);
  float* sZ = reinterpret_cast<float*>(sG + 3 * GI::IMG);
  float* sRed = sZ + D;
  int* sPlain = reinterpret_cast<int*>(sRed + NT8 / 64);   // [8] the wavefront has met a state value that does not split (f32_plain.h)

  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x / 64);
  const float om = BLEND ? 1.f - fminf(fmaxf(*rptr, 0.f), 1.f) : 1.f;
  float dr_sum = 0.f;
  // EVEN: the deal may give the workgroup parts of two heads
  for (Share sh = EVEN ? first_share(deal, blockIdx.x, blockIdx.y) : head_share(deal, blockIdx.x, blockIdx.y); sh.there;
       sh = EVEN ? next_share(deal, blockIdx.x, sh) : Share{}) {
    // (from a thread index that the optimiser cannot hoist: what depends on it would be held, or spilled, across the loop)
    const int tid = EVEN ? (threadIdx.x + opaque_zero()) & (NT8 - 1) : threadIdx.x, lane = tid % 64, g = lane / 32, c = lane % 32;
    const int bh = sh.bh, h = bh % H;
    const T* xb = x + head_base(rw, bh, H);
    const T* yb = y + head_base(rw, bh, H);
    T* dxb = dx + head_base(rw, bh, H);
    T* dvb = QSIDE ? nullptr : dv + head_base(rw, bh, H);
    const T* bb = BLEND ? blend + head_base(rw, bh, H) : nullptr;
    float dr_acc = 0.f;
    const float* sb = state + (size_t)bh * (D + 1) * D;

    const Blocks own = blocks_of(deal, sh, w, (n + 31) / 32);
    const int nblk = own.end, stride = own.stride;
    RowOctets<D, T> xr, yr;
    auto row_of = [&](const T* base, int b) {
      const int t = b * 32 + c;
      return base + (size_t)(t < n ? t : n - 1) * rw.sn;
    };
    int b = own.first;
    const int b_first = b < nblk ? b : nblk - 1;
    xr.load(row_of(xb, b_first), g);
    if constexpr (KIND == kPhiHedgehog) W::template build<T, NT8>(wx + (size_t)h * D * C::HALF, sW, tid);
    const bool state_splits = GI::template build<KIND, NT8>(sb, sG, tid);
    if (lane == 0) sPlain[w] = 0;
    if (!state_splits) sPlain[w] = 1;                        // (after lane 0's store: one wavefront's LDS operations are in order)
    build_octet_vector<D, KIND, NT8>(sb + D * D, sZ, tid);
    __syncthreads();

    const int b_own = b;
    const bool state_plain = any_of_8(sPlain);
    float chk = 0.f;                                         // NaN once the lane has met what does not split
    for (; b < nblk; b += stride) {
      const int t = b * 32 + c;
      const bool valid = t < n;
      if constexpr (QSIDE || NX == 1) yr.load(row_of(yb, b), g);
      float ds = 0.f;                                                // dO . s on the lane's channels, while few registers are live
      if constexpr (BLEND) {
        if (dr_part != nullptr) {
          // two octets at a time: a third row beside those of x and y does not fit the registers
          const T* srow = row_of(bb, b);
          RowOctets<D, T> sr;
#pragma unroll
          for (int k0 = 0; k0 < D / 16; k0 += 2) {
            sr.load(srow, g, k0, k0 + 2);
#pragma unroll
            for (int ks = k0; ks < k0 + 2; ++ks) {
              float a[8], s8[8];
              yr.values(ks, a);
              sr.values(ks, s8);
#pragma unroll
              for (int e = 0; e < 8; ++e) ds = fmaf(a[e], s8[e], ds);
            }
            __builtin_amdgcn_sched_barrier(0);
          }
        }
      }
      float f[D / 2];
      if constexpr (KIND == kPhiHedgehog) {
        f32x16 u[C::UM][1];
        W::template project<T>(xr, sW, lane + opaque_zero(), u);
        softmax_octets<D>(u, f);
      } else {
        phi_octets<D, KIND, T>(xr, nullptr, lane, f);
      }
      if constexpr (!QSIDE) {
        f32x16 o[1][MB];
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) o[0][mb] = zero16();
        const int base = GI::column_base(lane + opaque_zero());
#pragma unroll
        for (int ks = 0; ks < D / 16; ++ks) {
          uint4 a[1][3], m[MB][3];
#pragma unroll
          for (int mb = 0; mb < MB; ++mb)
#pragma unroll
            for (int i = 0; i < 3; ++i) m[mb][i] = GI::column_operand(sG, i, ks, mb, base);
          split8(f + 8 * ks, a[0]);
          mfma_pieces<3, 3>(a, m, o);
        }
        if constexpr (KIND == kPhiRelu) {
          // a feature that does not split makes all of its token's row NaN or Inf: one channel a row tells
#pragma unroll
          for (int r = 0; r < 16; ++r) chk = fmaf(o[0][0][r], 0.f, chk);
        }
        // (fp32 rows do not fit the registers beside the accumulators; before the stores: a wait for them must not wait for the stores)
        if constexpr (NX != 1) yr.load(row_of(yb, b), g);
        store_rows<D, T>(dvb, rw.sn, b * 32, n, (lane & 32) + GI::column(c), [&](int r, int mb) { return o[0][mb][r]; });
      }
      float inv = 0.f;
      const float* z = sZ + opaque_zero();
      if constexpr (QSIDE) inv = 1.0f / (octet_dot<D>(f, z, g) + (KIND == kPhiRelu ? kReluEps : 0.f));

      // G = y M^T on the lane's features
      f32x16 ga[MB][1];
#pragma unroll
      for (int mb = 0; mb < MB; ++mb) ga[mb][0] = zero16();
      const int lg = lane + opaque_zero();
#pragma unroll
      for (int ks = 0; ks < D / 16; ++ks) {
        uint4 a[MB][3], yp[1][NX];
#pragma unroll
        for (int mb = 0; mb < MB; ++mb)
#pragma unroll
          for (int i = 0; i < 3; ++i) a[mb][i] = GI::row_operand(sG, i, ks, mb, lg);
        GI::template y_pieces<T>(yr, ks, yp[0]);
        mfma_pieces<3, NX>(a, yp, ga);
      }
      // a y that does not split makes every feature of its token NaN or Inf, phi from an x that does not is NaN: one value tells
      // (Hedgehog: the sums of the Jacobian, below)
      if constexpr (KIND == kPhiRelu) chk = fmaf(ga[0][0][0], 0.f, chk);
      // dL/dphi / gscale.  The factor om / den of the query side is applied to du: fewer products, and the gr that the sums of the Jacobian take
      // is the one they are subtracted from (a product fused into that subtraction is not), so that a saturated token's du is zero.
      float gr[D / 2], gscale = 1.f;
      if constexpr (QSIDE) {
        float part = 0.f;
#pragma unroll
        for (int i = 0; i < D / 2; ++i) part = fmaf(f[i], ga[i / 16][0][i % 16], part);
        part *= inv;
        if constexpr (BLEND) {
          if (valid) dr_acc += ds - part;
        }
        float lo, hi;
        pair32(part, lo, hi);
        const float delta = lo + hi;
        if constexpr (KIND == kPhiRelu) chk = fmaf(delta, 0.f, chk);
        const float a = inv * om;
        if (valid && g == 0) weights[(size_t)bh * n + t] = make_float2(a, -delta * a);
#pragma unroll
        for (int ks = 0; ks < D / 16; ++ks)
#pragma unroll
          for (int e = 0; e < 8; ++e) {
            const int i = 8 * ks + e;
            gr[i] = ga[i / 16][0][i % 16] - delta * z[(2 * ks + g) * 8 + e];
          }
        gscale = a;
      } else {
#pragma unroll
        for (int ks = 0; ks < D / 16; ++ks)
#pragma unroll
          for (int e = 0; e < 8; ++e) {
            const int i = 8 * ks + e;
            gr[i] = ga[i / 16][0][i % 16] + z[(2 * ks + g) * 8 + e];
          }
      }

      if constexpr (KIND == kPhiRelu) {
        // the derivative of max(x, 0) at 0 is 0; the lane's octets of its own row
        if (valid) {
          T* row = dxb + (size_t)t * rw.sn;
#pragma unroll
          for (int ks = 0; ks < D / 16; ++ks) {
            float v[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) v[e] = f[8 * ks + e] > 0.f ? (QSIDE ? gr[8 * ks + e] * gscale : gr[8 * ks + e]) : 0.f;
            uint4* dst = reinterpret_cast<uint4*>(row + 16 * ks + 8 * g);
            if constexpr (sizeof(T) == 2) {
              *dst = make_uint4(pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3]), pack_bf16x2(v[4], v[5]), pack_bf16x2(v[6], v[7]));
            } else {
              float4* d4 = reinterpret_cast<float4*>(dst);
              d4[0] = make_float4(v[0], v[1], v[2], v[3]);
              d4[1] = make_float4(v[4], v[5], v[6], v[7]);
            }
          }
        }
        xr.load(row_of(xb, b + stride < nblk ? b + stride : b), g);
      } else {
        xr.load(row_of(xb, b + stride < nblk ? b + stride : b), g);
        // softmax Jacobian of Eq. 5
        float cp = 0.f, cm = 0.f;
#pragma unroll
        for (int j = 0; j < C::LOC; ++j) { cp = fmaf(gr[j], f[j], cp); cm = fmaf(gr[C::LOC + j], f[C::LOC + j], cm); }
        float lo, hi;
        pair32(cp, lo, hi); cp = lo + hi;
        pair32(cm, lo, hi); cm = lo + hi;
        chk = fmaf(cp + cm, 0.f, chk);
        float du[C::LOC];
#pragma unroll
        for (int j = 0; j < C::LOC; ++j) {
          du[j] = f[j] * (gr[j] - cp) - f[C::LOC + j] * (gr[C::LOC + j] - cm);
          if constexpr (QSIDE) du[j] *= gscale;
        }
        if (du_ws != nullptr && valid) {
          // blocks of 32 tokens as the lanes hold them, 1 KB a store (see dw_f32_kernel)
          float4* dst = reinterpret_cast<float4*>(du_ws + ((size_t)bh * n + b * 32) * C::HALF);
          const int nb = n - b * 32 < 32 ? n - b * 32 : 32;
#pragma unroll
          for (int j = 0; j < C::LOC / 4; ++j) put_du(dst + (2 * j + g) * nb + c, make_float4(du[4 * j], du[4 * j + 1], du[4 * j + 2], du[4 * j + 3]), du_stream);
        }
        // dx = du W~^T, tokens on the accumulator rows
        f32x16 xa[1][MB];
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) xa[0][mb] = zero16();
        const int lz = lane + opaque_zero();
#pragma unroll
        for (int ks = 0; ks < W::KS; ++ks) {
          uint4 a[1][3], wb[MB][NX];
#pragma unroll
          for (int mb = 0; mb < MB; ++mb)
#pragma unroll
            for (int i = 0; i < NX; ++i) wb[mb][i] = sW[i * W::IMG + W::place(ks, mb, lz)];
          split8(du + 8 * ks, a[0]);
          mfma_pieces<3, NX>(a, wb, xa);
        }
        store_rows<D, T>(dxb, rw.sn, b * 32, n, lane, [&](int r, int mb) { return xa[0][mb][r]; });
      }
    }
    if (__builtin_expect(state_plain || __any(chk != chk), 0)) {
      __threadfence();                                       // what is stored above is written again
      dr_acc = 0.f;
      float dr = 0.f;
#pragma unroll 1
      for (b = b_own; b < nblk; b += stride)
#pragma unroll 1
        for (int tt = 0; tt < 32 && 32 * b + tt < n; ++tt) {
          const int t = 32 * b + tt;
          const size_t at = (size_t)t * rw.sn;
          float* du = du_ws != nullptr ? du_ws + ((size_t)bh * n + b * 32) * C::HALF + 4 * tt : nullptr;
          Plain<D, KIND, T>::template grad<QSIDE, BLEND>(xb + at, yb + at, wx + (size_t)h * D * C::HALF, sb, dxb + at, du,
                                                         n - b * 32 < 32 ? n - b * 32 : 32, QSIDE ? weights + (size_t)bh * n + t : nullptr,
                                                         BLEND && dr_part != nullptr ? bb + at : nullptr, om, &dr, lane);
          if constexpr (!QSIDE)
            Plain<D, KIND, T>::template apply<false, false>(xb + at, wx + (size_t)h * D * C::HALF, sb, dvb + at, nullptr, 0.f, lane);
        }
      if (lane == 0) dr_acc = dr;
    }
    if constexpr (BLEND) dr_sum += dr_acc;
    if (EVEN && sh.rest < sh.hi) __syncthreads();        // the next head's images take the place of these
  }
  if (BLEND && dr_part != nullptr) {
    for (int m = 32; m >= 1; m >>= 1) dr_sum += __shfl_xor(dr_sum, m, 64);
    if (threadIdx.x % 64 == 0) sRed[w] = dr_sum;
    __syncthreads();
    if (threadIdx.x == 0) {
      float s = 0.f;
      for (int i = 0; i < NT8 / 64; ++i) s += sRed[i];
      dr_part[gridDim.x * blockIdx.y + blockIdx.x] = s;
    }
  }
}

// Where the du rows of a head sit in its [n][D/2] region of the workspace: by blocks of 32 tokens (nb of them in the last), in a block by
// (four features of a lane group, token): element (token tt, feature g*LOC + 4j + i) of a block at ((2j + g)*nb + tt)*4 + i.
// Stored as rows, a lane's pieces of 16 bytes on 64 different lines per instruction, the two gradient passes took 114 and 118 us where
// they take 103 and 100 (bf16 input, 12 heads x 32760 x 128), and the reading pass 103 where it takes 100.

// Partial dW~ = sum over a share of the tokens of x^T du; grid (P, BH, 2): z = 0 the query side, 1 the key side.  A wavefront takes
// steps of 16 tokens: its lanes read eight tokens of MB adjacent channels and of NB adjacent features straight from memory, which
// is the operand layout of both, so nothing goes through LDS before the wavefronts' sums are combined.
template <int D, typename T>
__global__ __launch_bounds__(NT8) void dw_f32_kernel(const T* __restrict__ q, const T* __restrict__ k, const float* __restrict__ du_q,
                                                     const float* __restrict__ du_k, float* __restrict__ part_q,
                                                     float* __restrict__ part_k, int H, int n, Rows rw) {
  using C = Cfg<D>;
  constexpr int MB = D / 32, NB = C::HALF / 32, NX = kPieces<T>;
  const float* du = blockIdx.z ? du_k : du_q;
  if (du == nullptr) return;
  extern __shared__ uint4 smem[];
  float* sAcc = reinterpret_cast<float*>(smem);                   // [4 wavefronts][MB*NB*16][64]
  const int tid = threadIdx.x, lane = tid % 64;
  const int w = __builtin_amdgcn_readfirstlane(tid / 64);
  const int g = lane / 32, c = lane % 32;
  const int bh = blockIdx.y;
  const T* xb = (blockIdx.z ? k : q) + head_base(rw, bh, H) + MB * c;
  const float* ub = du + (size_t)bh * n * C::HALF;
  typedef float cols __attribute__((ext_vector_type(NB)));
  typedef float xf __attribute__((ext_vector_type(MB)));
  typedef unsigned xh __attribute__((ext_vector_type(MB / 2)));

  f32x16 acc[MB][NB];
#pragma unroll
  for (int i = 0; i < MB; ++i)
#pragma unroll
    for (int j = 0; j < NB; ++j) acc[i][j] = zero16();

  const int steps = (n + 15) / 16, stride = gridDim.x * (NT8 / 64);
  constexpr int XW = MB * sizeof(T) / 4;
  struct Step { uint32_t x[8][XW]; cols u[8]; };
  Step cur, nxt;
  // the lane's features NB*c .. are features f % LOC of lane group f / LOC
  const int fj = (NB * c % C::LOC) / 4, fg = NB * c / C::LOC, fi = NB * c % 4;
  auto load = [&](Step& s, int st) {
    const int t0 = 16 * st / 32 * 32, nb = n - t0 < 32 ? n - t0 : 32;
    const float* ublk = ub + (size_t)t0 * C::HALF + (size_t)(2 * fj + fg) * nb * 4 + fi;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const int t = 16 * st + 8 * g + e;
      const size_t tc = t < n ? t : n - 1;
      if constexpr (sizeof(T) == 4) {
        const xf r = *reinterpret_cast<const xf*>(xb + tc * rw.sn);
#pragma unroll
        for (int i = 0; i < MB; ++i) s.x[e][i] = __builtin_bit_cast(uint32_t, (float)r[i]);
      } else {
        const xh r = *reinterpret_cast<const xh*>(xb + tc * rw.sn);
#pragma unroll
        for (int i = 0; i < MB / 2; ++i) s.x[e][i] = r[i];
      }
      s.u[e] = *reinterpret_cast<const cols*>(ublk + (tc - t0) * 4);
    }
  };
  const float sign = w % 2 ? -1.f : 1.f;         // odd wavefronts sum the negated products (see the head of f32_split.h)
  int st = blockIdx.x * (NT8 / 64) + w;
  load(cur, st < steps ? st : steps - 1);
  for (; st < steps; st += stride) {
    load(nxt, st + stride < steps ? st + stride : st);
    uint4 a[MB][NX], b[NB][3];
    if constexpr (sizeof(T) == 4) {
#pragma unroll
      for (int i = 0; i < MB; ++i) {
        float v[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] = __builtin_bit_cast(float, cur.x[e][i]);
        split8<true>(v, a[i]);                     // (an infinite x has made du NaN already)
      }
    } else {
#pragma unroll
      for (int i = 0; i < MB / 2; ++i) {
        uint32_t lo[4], hi[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          lo[e] = (cur.x[2 * e][i] & 0xffffu) | (cur.x[2 * e + 1][i] << 16);
          hi[e] = (cur.x[2 * e][i] >> 16) | (cur.x[2 * e + 1][i] & 0xffff0000u);
        }
        a[2 * i][0] = make_uint4(lo[0], lo[1], lo[2], lo[3]);
        a[2 * i + 1][0] = make_uint4(hi[0], hi[1], hi[2], hi[3]);
      }
    }
#pragma unroll
    for (int j = 0; j < NB; ++j) {
      float v[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) v[e] = 16 * st + 8 * g + e < n ? cur.u[e][j] * sign : 0.f;
      split8(v, b[j]);
    }
    mfma_pieces<NX, 3>(a, b, acc);
    cur = nxt;
  }
#pragma unroll
  for (int i = 0; i < MB; ++i)
#pragma unroll
    for (int j = 0; j < NB; ++j) acc[i][j] *= sign;
  // sums of the eight wavefronts, pairwise
  constexpr int PER = MB * NB * 16;
#pragma unroll
  for (int half = 4; half >= 1; half >>= 1) {
    __syncthreads();
    if (w >= half && w < 2 * half) {
      float* dst = sAcc + (size_t)(w - half) * PER * 64 + lane;
#pragma unroll
      for (int i = 0; i < MB; ++i)
#pragma unroll
        for (int j = 0; j < NB; ++j)
#pragma unroll
          for (int r = 0; r < 16; ++r) dst[((i * NB + j) * 16 + r) * 64] = acc[i][j][r];
    }
    __syncthreads();
    if (w < half) {
      const float* src = sAcc + (size_t)w * PER * 64 + lane;
#pragma unroll
      for (int i = 0; i < MB; ++i)
#pragma unroll
        for (int j = 0; j < NB; ++j)
#pragma unroll
          for (int r = 0; r < 16; ++r) acc[i][j][r] += src[((i * NB + j) * 16 + r) * 64];
    }
  }
  if (w == 0) {
    float* part = (blockIdx.z ? part_k : part_q) + ((size_t)bh * gridDim.x + blockIdx.x) * (size_t)D * C::HALF;
#pragma unroll
    for (int i = 0; i < MB; ++i)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int channel = MB * (8 * (r / 4) + 4 * g + (r % 4)) + i;
        cols v;
#pragma unroll
        for (int j = 0; j < NB; ++j) v[j] = acc[i][j][r];
        *reinterpret_cast<cols*>(part + channel * C::HALF + NB * c) = v;
      }
  }
}
template <int D>
constexpr size_t dw_smem() { return (size_t)4 * (D / 32) * (D / 64) * 16 * 64 * sizeof(float); }

template <int D, int KIND, typename T>
hipError_t run_bwd(const BwdArgs& a, const Plan& p, hipStream_t s) {
  hipError_t e;
  // units of two at width 128 wherever they fit: units of four / two, a step, 32 heads x 500 with bf16 tensors 78.4 / 75.6, 16 x 1000 77.7 / 74.7 (but 32 x 256 71.1 / 73.5, with
  // half as many workgroups), with fp32 tensors 16 x 500 102.2 / 97.8, 64 x 128 105.9 / 101.4; width 64, bf16 tensors, 128 x 128 40.2 / 42.6, 64 x 256 39.7 / 41.1
  constexpr UnitLimits most = D == 128 ? kNoUnitLimits : UnitLimits();
  const Split deal = make_deal_of_blocks(p.BH, (p.n + 31) / 32, NT8 / 64, kF32Cost<KIND, T, false>, grad_even<D, T>, 1, most);
  constexpr size_t smem = grad_smem<D, KIND, T>();
  // the per-token weights of the sum over tokens: dv's memory (at least 128 bytes per token), which the last pass writes
  float2* weights = static_cast<float2*>(a.dv);
  auto grad = [&](auto by_head, auto even, const void* x, const void* y, const void* wx, const float* state, void* dx, float* du) -> hipError_t {
    auto launch = [&](auto kernel) -> hipError_t {
      hipError_t e2 = set_smem_once<decltype(kernel)::value>(smem);
      if (e2 != hipSuccess) return e2;
      decltype(kernel)::value<<<grid_of(deal), NT8, smem, s>>>((const T*)x, (const T*)y, (const T*)wx, state, (T*)dx, (T*)a.dv, du,
                                                      2 * p.du_bytes > kDuStreamBytes, weights, (const T*)a.blend_in, a.blend_r,
                                                      a.blend_dr ? a.dr_part : nullptr, p.H, p.n, deal, p.rows);
      return hipGetLastError();
    };
    if constexpr (grad_even<D, T>)
      if (!deal.share) return launch(even);
    return launch(by_head);
  };
  constexpr bool EV = grad_even<D, T>;
  float* du_q = a.dwq ? a.du_q : nullptr;
  float* du_k = a.dwk ? a.du_k : nullptr;
  if (KIND == kPhiHedgehog && a.blend_in)
    e = grad(KernelTag<grad_f32_kernel<D, KIND, T, true, KIND == kPhiHedgehog, false>>{}, KernelTag<grad_f32_kernel<D, KIND, T, true, KIND == kPhiHedgehog, EV>>{}, a.q, a.dout, a.wq, a.state, a.dq, du_q);
  else
    e = grad(KernelTag<grad_f32_kernel<D, KIND, T, true, false, false>>{}, KernelTag<grad_f32_kernel<D, KIND, T, true, false, EV>>{}, a.q, a.dout, a.wq, a.state, a.dq, du_q);
  if (e != hipSuccess) return e;
  if ((e = run_state_pass<D, KIND, T, true>(a.q, a.dout, a.wq, weights, a.partials, p, s)) != hipSuccess) return e;
  if ((e = launch_state_reduce_split(a.partials, a.dstate, p, DrSum{a.dr_part, deal.G, a.blend_r, a.blend_dr}, s)) != hipSuccess) return e;
  e = grad(KernelTag<grad_f32_kernel<D, KIND, T, false, false, false>>{}, KernelTag<grad_f32_kernel<D, KIND, T, false, false, EV>>{}, a.k, a.v, a.wk, a.dstate, a.dk, du_k);
  if (e != hipSuccess) return e;
  if constexpr (KIND == kPhiHedgehog) {
    if (du_q || du_k) {
      if ((e = set_smem_once<dw_f32_kernel<D, T>>(dw_smem<D>())) != hipSuccess) return e;
      float* part_k = a.dw_part + (size_t)p.BH * p.P * D * (D / 2);
      dw_f32_kernel<D, T><<<dim3(p.P, p.BH, 2), NT8, dw_smem<D>(), s>>>((const T*)a.q, (const T*)a.k, du_q, du_k, a.dw_part, part_k, p.H, p.n, p.rows);
      if ((e = hipGetLastError()) != hipSuccess) return e;
      if ((e = launch_dw_reduce2(a.dw_part, a.dwq, p.P, part_k, a.dwk, p.P, p, s)) != hipSuccess) return e;
    }
  }
  return hipSuccess;
}

template <typename T>
hipError_t bwd_any(const BwdArgs& a, const Plan& p, hipStream_t s) {
  if (p.kind == kPhiRelu) return p.d == 128 ? run_bwd<128, kPhiRelu, T>(a, p, s) : run_bwd<64, kPhiRelu, T>(a, p, s);
  return p.d == 128 ? run_bwd<128, kPhiHedgehog, T>(a, p, s) : run_bwd<64, kPhiHedgehog, T>(a, p, s);
}

}  // namespace

hipError_t launch_bwd_f32(const BwdArgs& a, const Plan& p, hipStream_t s) {
  return p.bf16_storage ? bwd_any<uint16_t>(a, p, s) : bwd_any<float>(a, p, s);
}

}  // namespace linattn
