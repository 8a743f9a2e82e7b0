// Blocks of 16 tokens to a wavefront: v_mfma_f32_16x16x32_{bf16,f16}, tokens along N as in the 32-token form, four lanes to a token.
//   lane l = (m, q) with m = l % 16, q = l / 16
//   A: lane holds A[m][8q .. 8q+7],  B: lane holds B[8q .. 8q+7][m],  D: lane holds D[4q + r][m] for r = 0..3
// A lane has half of what a lane of the 32-token form has, so that a SIMD holds twice the wavefronts: with one or two, a chain of MFMAs,
// exponentials and exchanges leaves a third of the issue slots empty.  What it costs is LDS reads: an operand of an image serves 16
// tokens instead of 32.
#pragma once
#include "mfma_common.h"

namespace linattn {

typedef __attribute__((__vector_size__(4 * sizeof(float)))) float f32x4;

// Lane (t, q) owns FL consecutive features of each half of phi, q*FL .. q*FL + FL-1; row block mb, register r of an accumulator over the
// features <-> feature q*FL + 4*mb + r, so operand row m of block mb is feature (m/4)*FL + 4*mb + m%4.
template <int D>
struct Tok16 {
  static constexpr int HALF = D / 2;
  static constexpr int FL = D / 8;        // features of a half that a lane owns
  static constexpr int UB = HALF / 16;    // row blocks of U^T
  static constexpr int KS = D / 32;       // k-steps over the channels
  static constexpr int GB = D / 16;       // row blocks over the D features of phi
  static constexpr int DK = FL / 8;       // k-steps over the d/2 pre-softmax features (element (q, e) of k-step ks: feature q*FL + 8*ks + e)
  static constexpr int MB = D / 16;       // column blocks over the channels (column c of block mb: channel MB*c + mb)
  static constexpr int W_IMG = KS * UB * 64, G_IMG = KS * GB * 64, T_IMG = DK * MB * 64, A_IMG = 2 * DK * MB * 64;      // uint4 entries of the images
  __device__ static constexpr int feature(int mb, int m) { return (m / 4) * FL + 4 * mb + m % 4; }
};

__device__ __forceinline__ f32x4 mfma_bf16_16(uint4 a, uint4 b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(a), as_bf16x8(b), c, 0, 0, 0);
}
__device__ __forceinline__ f32x4 mfma_f16_16(uint4 a, uint4 b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_f16(as_f16x8(a), as_f16x8(b), c, 0, 0, 0);
}

// W~ [D][D/2] bf16 (one head) -> the two LDS images of it: of the A operands of U^T = W~^T X^T, entry (ks, mb, lane = (m, q)) holding
// W~[32ks + 8q + e][feature(mb, m)], and (fp16, exact) of the B operands of dX = dU W~^T with the tokens on the accumulator rows, entry (ks, mb,
// lane = (c, q)) holding W~[MB*c + mb][q*FL + 8ks + e].  Read and written apart (see WImage).
template <int D, int NTHREADS>
struct WImages16 {
  using K = Tok16<D>;
  static constexpr int TN = (K::T_IMG + NTHREADS - 1) / NTHREADS;
  static_assert(K::W_IMG / 4 <= NTHREADS, "one item per thread");
  uint2 r[8];
  uint4 t[TN];
  __device__ __forceinline__ void load(const uint16_t* __restrict__ w, int tid) {
    if (tid < K::W_IMG / 4) {
      const int mq = tid % 4, mb = (tid / 4) % K::UB, q = (tid / (4 * K::UB)) % 4, ks = tid / (16 * K::UB);
      const uint16_t* src = w + (32 * ks + 8 * q) * K::HALF + K::feature(mb, 4 * mq);
#pragma unroll
      for (int e = 0; e < 8; ++e) r[e] = *reinterpret_cast<const uint2*>(src + e * K::HALF);
    }
#pragma unroll
    for (int i = 0; i < TN; ++i) {
      const int idx = tid + i * NTHREADS;
      const int c = idx % 16, q = (idx / 16) % 4, mb = (idx / 64) % K::MB, ks = idx / (64 * K::MB);
      if (idx < K::T_IMG) t[i] = *reinterpret_cast<const uint4*>(w + (K::MB * c + mb) * K::HALF + q * K::FL + 8 * ks);
    }
  }
  __device__ __forceinline__ void write(uint4* sWA, uint4* sWB, int tid) const {
    if (tid < K::W_IMG / 4) {
      const int mq = tid % 4, mb = (tid / 4) % K::UB, q = (tid / (4 * K::UB)) % 4, ks = tid / (16 * K::UB);
      write_w_entries(r, sWA + (ks * K::UB + mb) * 64 + 16 * q + 4 * mq);
    }
#pragma unroll
    for (int i = 0; i < TN; ++i) {
      const int idx = tid + i * NTHREADS;
      if (idx < K::T_IMG)
        sWB[idx] = make_uint4(bf16x2_to_f16x2(t[i].x), bf16x2_to_f16x2(t[i].y), bf16x2_to_f16x2(t[i].z), bf16x2_to_f16x2(t[i].w));
    }
  }
};

// A operands of G^T = S Y^T: entry (ks, mb, lane = (m, q)) holds scale * S[f][32ks + 8q + e], f = feature(mb, m) of the + half for mb < GB/2,
// of the - half otherwise.  The entry of lane (m, q) lies at 16q + (m ^ (4ks + q)): eight lanes of the writing wavefront have the
// same m, and would all hit the same banks.
template <int D>
__device__ __forceinline__ int grad16_lane(int lane) { return lane ^ (lane / 16); }        // the place in k-step 0; ^ 4ks in k-step ks
// KIND = kPhiRelu: the rows are ordered so that register r of block mb in a lane of group q is feature 32*(mb/2) + 8q + 4*(mb%2) + r, element
// 4*(mb%2) + r of the piece mb/2 which that lane holds of its token's row.
template <int D, int NTHREADS, int KIND = kPhiHedgehog>
__device__ __forceinline__ void write_grad_image16(const StateRegs<D, NTHREADS>& S, uint4* img, float sc) {
  using K = Tok16<D>;
  if (!S.active) return;
  const int ks = S.cq / 8, q = (S.cq / 2) % 4;
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    const int f = 8 * S.fo + e, half = f / K::HALF, fl = f % K::HALF, j = fl % K::FL;
    const int mb = KIND == kPhiRelu ? 2 * (S.fo / 4) + e / 4 : half * (K::GB / 2) + j / 4;
    const int m = KIND == kPhiRelu ? 4 * (S.fo % 4) + e % 4 : 4 * (fl / K::FL) + j % 4;
    uint2* dst = reinterpret_cast<uint2*>(img + (ks * K::GB + mb) * 64 + 16 * q + (m ^ (4 * ks + q))) + S.cq % 2;
    *dst = make_uint2(pack_f16x2(sc * S.v[e][0], sc * S.v[e][1]), pack_f16x2(sc * S.v[e][2], sc * S.v[e][3]));
  }
}

// B operands of Y = phi S, tokens on the accumulator rows: entry (ks, mb, lane = (c, q)) holds scale * S[f + e][MB*c + mb], f = q*FL + 8*(ks % DK)
// of the + half for ks < DK, of the - half otherwise.
// KIND = kPhiRelu: the features are the channels in their plain order, 32ks + 8q + e.
template <int D, int NTHREADS, int KIND = kPhiHedgehog>
__device__ __forceinline__ void write_apply_image16(const StateRegs<D, NTHREADS>& S, uint4* img, float sc) {
  using K = Tok16<D>;
  if (!S.active) return;
  const int f = 8 * S.fo, fl = f % K::HALF;
  const int q = KIND == kPhiRelu ? S.fo % 4 : fl / K::FL, ks = KIND == kPhiRelu ? S.fo / 4 : f / K::HALF * K::DK + fl % K::FL / 8;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int ch = 4 * S.cq + i;
    img[(ks * K::MB + ch % K::MB) * 64 + 16 * q + ch / K::MB] =
        make_uint4(pack_f16x2(sc * S.v[0][i], sc * S.v[1][i]), pack_f16x2(sc * S.v[2][i], sc * S.v[3][i]),
                   pack_f16x2(sc * S.v[4][i], sc * S.v[5][i]), pack_f16x2(sc * S.v[6][i], sc * S.v[7][i]));
  }
}

// The lane index as a value that the optimiser cannot hoist out of a loop, in a range that it knows (addresses made from it are worked out where
// they are used instead of being held, or spilled, across the loop).
__device__ __forceinline__ unsigned opaque_lane(int lane) { return (unsigned)(lane + opaque_zero()) & 63u; }

// A zero in a scalar register that the optimiser cannot see through.
__device__ __forceinline__ float opaque_zero_scalar() {
  float z = 0.f;
  asm volatile("" : "+s"(z));
  return z;
}
// a*s + c, b*s + c rounded to fp16, a mixed-precision instruction each (two multiplications and a conversion are three for two; with a c that it sees
// is zero the compiler takes those).
__device__ __forceinline__ uint32_t mul_pack_f16x2(float a, float b, float s, float c) {
  const f16x2 r = {(_Float16)fmaf(a, s, c), (_Float16)fmaf(b, s, c)};
  return __builtin_bit_cast(uint32_t, r);
}
__device__ __forceinline__ uint32_t mul_pack_f16x2(uint32_t ab, float s, float c) {
  const f16x2 v = __builtin_bit_cast(f16x2, ab);
  const f16x2 r = {(_Float16)fmaf((float)v[0], s, c), (_Float16)fmaf((float)v[1], s, c)};
  return __builtin_bit_cast(uint32_t, r);
}

// The largest magnitude of bf16 values, of those that are finite.  2x + 2^8 in 16 bits drops the sign, orders the finite ones and wraps the others round
// to below 2^8.
struct FiniteMax16 {
  typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));
  u16x2 m = {0x100, 0x100}, two = {2, 2};
  __device__ __forceinline__ FiniteMax16() { asm volatile("" : "+s"(two)); }      // (one v_pk_mad_u16; seen as a shift and an addition they are two)
  __device__ __forceinline__ void take(uint32_t pair) {
    const u16x2 bias = {0x100, 0x100};
    m = __builtin_elementwise_max(m, (u16x2)(__builtin_bit_cast(u16x2, pair) * two + bias));
  }
  __device__ __forceinline__ void take(const uint4& x) { take(x.x); take(x.y); take(x.z); take(x.w); }
  __device__ __forceinline__ float value() const {
    return __builtin_bit_cast(float, (uint32_t)((m[0] > m[1] ? m[0] : m[1]) - 0x100) << 15);
  }
};

// The 16 rows from token t0 of a head of n tokens as operands: lane (t, q) reads the 16-byte chunks 4ks + q of row t0 + t.  Bounded buffer loads: the
// address is one register that never changes, and rows past n read as zeros.  All arguments but the lane are uniform.
template <int D>
struct LoadRows16 {
  uint32_t at, pitch;
  const char* base;
  int n;
  __device__ __forceinline__ LoadRows16(const uint16_t* head, size_t sn, int n_, int lane) : base((const char*)head), n(n_) {
    pitch = (uint32_t)sn * 2;
    at = (uint32_t)(lane % 16) * pitch + 16 * (lane / 16);
  }
  __device__ __forceinline__ void load(uint4 (&x)[D / 32], int t0) const {
    const int left = n - t0 < 16 ? n - t0 : 16;
    const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc(const_cast<char*>(base) + (size_t)t0 * pitch, 0,
                                                                       left > 0 ? (uint32_t)left * pitch : 0, 0x00020000);
#pragma unroll
    for (int ks = 0; ks < D / 32; ++ks) x[ks] = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(r, at + 64 * ks, 0, 0));
  }
  // wait for the rows here (see where it is used)
  static __device__ __forceinline__ void arrived(uint4 (&x)[D / 32]) {
#pragma unroll
    for (int ks = 0; ks < D / 32; ++ks) asm volatile("" : "+v"(x[ks].x), "+v"(x[ks].y), "+v"(x[ks].z), "+v"(x[ks].w));
  }
};

// The 16 rows from token t0 of a head of n tokens: lane (c, q), register r has PIECE bytes of token t0 + 4q + r, at byte PIECE*c of the row.
// Buffer stores bounded to the rows that exist, as in TokenRows.
template <int PIECE>
struct TokenRows16 {
  __amdgpu_buffer_rsrc_t rows;
  uint32_t at, pitch;
  __device__ __forceinline__ TokenRows16(void* base, size_t pitch_bytes, int t0, int n, int lane) {
    const int left = n - t0 < 16 ? n - t0 : 16;
    pitch = (uint32_t)pitch_bytes;
    rows = __builtin_amdgcn_make_buffer_rsrc(static_cast<char*>(base) + (size_t)t0 * pitch_bytes, 0, left > 0 ? (uint32_t)left * pitch : 0, 0x00020000);
    const unsigned lz = opaque_lane(lane);
    at = (uint32_t)(4 * (lz / 16)) * pitch + (uint32_t)(PIECE * (lz % 16));
  }
  template <bool STREAM, typename V>
  __device__ __forceinline__ void store(int r, V v) const {
    static_assert(sizeof(V) == PIECE, "a lane's piece of a row");
    const uint32_t off = at + (uint32_t)r * pitch;
    constexpr int aux = STREAM ? 2 : 0;
    if constexpr (PIECE == 8) __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2, v), rows, off, 0, aux);
    else __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, v), rows, off, 0, aux);
  }
};
// acc[mb][r] of lane (c, q): token 4q + r, channel MB*c + mb  ->  mul * acc (ADD: + add[mb]) as bf16 rows of base
template <int D, bool STREAM, bool ADD>
__device__ __forceinline__ void store_token_rows16(uint16_t* base, size_t sn, int t0, int n, int lane, const f32x4 (&acc)[D / 16], float mul,
                                                   const float (&add)[D / 16]) {
  constexpr int MB = D / 16;
  const TokenRows16<2 * MB> rows(base, sn * 2, t0, n, lane);
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    uint32_t w[MB / 2];
#pragma unroll
    for (int i = 0; i < MB / 2; ++i)
      w[i] = ADD ? pack_bf16x2(fmaf(acc[2 * i][r], mul, add[2 * i]), fmaf(acc[2 * i + 1][r], mul, add[2 * i + 1]))
                 : pack_bf16x2(acc[2 * i][r] * mul, acc[2 * i + 1][r] * mul);
    if constexpr (MB == 8) rows.template store<STREAM>(r, make_uint4(w[0], w[1], w[2], w[3]));
    else rows.template store<STREAM>(r, make_uint2(w[0], w[1]));
  }
}

// First half of Eq. 5 for 16 tokens: u[j / 4][j % 4] = pre-softmax feature q*FL + j of the lane's token.  x is dead afterwards.
template <int D, int AHEAD>
__device__ __forceinline__ void project16(const uint4 (&x)[D / 32], const uint4* sWA, int lane, f32x4 (&u)[Tok16<D>::UB]) {
  using K = Tok16<D>;
#pragma unroll
  for (int mb = 0; mb < K::UB; ++mb) u[mb] = f32x4{0.f, 0.f, 0.f, 0.f};
  const uint4* wa = sWA + lane + opaque_zero();
  pipelined_operands<K::KS * K::UB, AHEAD>([&](int i) { return wa[i * 64]; },
                                           [&](int i, uint4 a) { u[i % K::UB] = mfma_bf16_16(a, x[i / K::UB], u[i % K::UB]); });
}

// Second half of Eq. 5, up to the normalisers ip, im, which go into the factors of what is linear in phi.
template <int D>
__device__ __forceinline__ void softmax16(const f32x4 (&u)[Tok16<D>::UB], float (&ep)[D / 8], float (&em)[D / 8], float& ip, float& im) {
  float mx = u[0][0], mn = -u[0][0];
#pragma unroll
  for (int j = 0; j < D / 8; ++j) { mx = fmaxf(mx, u[j / 4][j % 4]); mn = fmaxf(mn, -u[j / 4][j % 4]); }
  quad2<MaxOp>(mx, mn);
  ip = im = 0.f;
#pragma unroll
  for (int j = 0; j < D / 8; ++j) {
    ep[j] = __builtin_amdgcn_exp2f(fmaf(u[j / 4][j % 4], kLog2e, -mx * kLog2e));
    em[j] = __builtin_amdgcn_exp2f(fmaf(u[j / 4][j % 4], -kLog2e, -mn * kLog2e));
    ip += ep[j]; im += em[j];
  }
  quad2<SumOp>(ip, im);
  ip = __builtin_amdgcn_rcpf(ip); im = __builtin_amdgcn_rcpf(im);
}

// dx = du W~^T for 16 tokens, tokens on the accumulator rows: du enters as fp16, scaled by one power of two that brings the wavefront's largest into
// [1, 2) (dub; zero for tokens that do not exist), and acc is to be multiplied by its, the inverse.  blk_its: the same, 0 where all are zero.
template <int D, int AHEAD>
__device__ __forceinline__ void du_to_dx16(const float (&du)[D / 8], const uint4* sWB, int lane, bool valid, float zero, f32x4 (&acc)[D / 16],
                                           float& its, uint32_t (&dub)[D / 16], float& blk_its) {
  using K = Tok16<D>;
  float m = 0.f;
#pragma unroll
  for (int j = 0; j < K::FL; ++j) m = fmaxf(m, fabsf(du[j]));
  m = row_max_mag(quad<MagOp>(valid ? m : 0.f));
  const float s = pow2_normaliser(m), ts = valid ? s : 0.f;
#pragma unroll
  for (int j = 0; j < K::FL / 2; ++j) dub[j] = mul_pack_f16x2(du[2 * j], du[2 * j + 1], ts, zero);
  its = __builtin_amdgcn_rcpf(s);      // exact: a power of two
  blk_its = m > 0.f ? its : 0.f;
#pragma unroll
  for (int mb = 0; mb < K::MB; ++mb) acc[mb] = f32x4{0.f, 0.f, 0.f, 0.f};
  const uint4* wb = sWB + lane + opaque_zero();
  pipelined_operands<K::DK * K::MB, AHEAD>(
      [&](int i) { return wb[i * 64]; },
      [&](int i, uint4 b) {
        const uint32_t* a = dub + 4 * (i / K::MB);
        acc[i % K::MB] = mfma_f16_16(make_uint4(a[0], a[1], a[2], a[3]), b, acc[i % K::MB]);
      });
}

// What the dW~ contraction reads (DwTile): the rows x as fp16 into rows 16*slot .. of the tile sX [kTile][D], du (as du_to_dx16 packs it) into sU
// [kTile][D/2], its inverse scale into sIts[slot].
template <int D>
__device__ __forceinline__ void park_dw16(const uint4 (&x)[D / 32], const uint32_t (&dub)[D / 16], float blk_its, char* sX, char* sU, float* sIts,
                                          int slot, int lane) {
  using K = Tok16<D>;
  const unsigned lz = opaque_lane(lane), q = lz / 16, t = lz % 16;
  const int row = 16 * slot + (int)t;
  char* rowp = sX + row * (D * 2);
#pragma unroll
  for (int ks = 0; ks < K::KS; ++ks)
    *reinterpret_cast<uint4*>(rowp + (((4 * ks + q) ^ (unsigned)swz<D>((int)t)) * 16)) =
        make_uint4(bf16x2_to_f16x2(x[ks].x), bf16x2_to_f16x2(x[ks].y), bf16x2_to_f16x2(x[ks].z), bf16x2_to_f16x2(x[ks].w));
  char* urow = sU + row * D;
#pragma unroll
  for (int c = 0; c < K::DK; ++c)
    *reinterpret_cast<uint4*>(urow + (((q * K::DK + c) ^ (unsigned)swz<D / 2>((int)t)) * 16)) =
        make_uint4(dub[4 * c], dub[4 * c + 1], dub[4 * c + 2], dub[4 * c + 3]);
  if (lane == 0) sIts[slot] = blk_its;
}

}  // namespace linattn
