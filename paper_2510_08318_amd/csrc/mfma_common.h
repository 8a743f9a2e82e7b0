// Device-side building blocks shared by the bf16-I/O forward and backward kernels (gfx950 MFMA,
// tokens along the N dimension): operand images in LDS, the two halves of Eq. 5, transposing
// LDS reads.  Header-only; include after kernels.h.
#pragma once
#include "mfma_layout.h"

namespace linattn {

constexpr float kLog2e = 1.4426950408889634f;
constexpr int NT = 256;          // 4 wavefronts (tile-synchronised kernels)

template <int D>
struct Cfg {
  static constexpr int HALF = D / 2;     // pre-softmax features u = x W~
  static constexpr int UM = HALF / 32;   // row blocks of U^T
  static constexpr int UK = D / 16;      // k-steps over the d input channels
  static constexpr int LOC = HALF / 2;   // pre-softmax features a lane owns
  static constexpr int NPK = D / 4;      // packed fp16 pairs of phi a lane owns (d/2 values)
  static constexpr int CH = D / 8;       // 16-byte chunks per tile row
  static constexpr int W_IMG = UK * UM * 64;   // uint4 entries of the W~^T operand image
};

// XOR swizzle of the 16-byte chunk index inside a tile row: makes the transposing 8-byte reads
// (4 consecutive rows x 32 bytes per 16 lanes) and the 16-byte row writes hit distinct banks.
// Depends on r % 16 only, so it is the same for every 16-row k-step of a tile.
template <int D>
__device__ __forceinline__ int swz(int r) {
  if (D == 128) return ((r & 3) << 2) | ((r >> 2) & 3);
  if (D == 32) return r & 3;                               // 4 chunks per row
  return (((r & 3) << 1) ^ ((r >> 2) & 3)) & 7;
}

// A zero the optimiser cannot see through: added to an LDS index it keeps loop-invariant
// operand reads inside the loop (hoisted, they would not fit the register file and spill).
__device__ __forceinline__ int opaque_zero() {
  int z = 0;
  asm volatile("" : "+v"(z));
  return z;
}

typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
// Streaming (non-temporal) 16-byte global load / store, for fully coalesced accesses only: with
// the operand-layout loads (two 16-byte pieces of a row per instruction, four instructions per
// 128-byte line) the hint makes the line be fetched again and costs 20 % of the bandwidth.
__device__ __forceinline__ uint4 ld_nt(const uint4* p) {
  return __builtin_bit_cast(uint4, __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(p)));
}
__device__ __forceinline__ void st_nt(uint4* p, uint4 v) {
  __builtin_nontemporal_store(__builtin_bit_cast(u32x4, v), reinterpret_cast<u32x4*>(p));
}

// Exchange with lane^32: returns (value of the low-half lane, value of the high-half lane),
// identical in both lanes of a pair.
__device__ __forceinline__ void pair32(float x, float& lo, float& hi) {
  const uint32_t u = __builtin_bit_cast(uint32_t, x);
  auto r = __builtin_amdgcn_permlane32_swap(u, u, false, false);
  lo = __builtin_bit_cast(float, (uint32_t)r[0]);
  hi = __builtin_bit_cast(float, (uint32_t)r[1]);
}

// W~ [D][D/2] bf16 (one head) -> LDS image of the A operands of U^T = W~^T X^T:
// entry (ks, mb, lane=(m,g)) holds W~[16ks + 8g + e][owned_row<HALF>(mb, m)], e = 0..7.  A thread reads four adjacent features of
// eight channels (8 bytes a load, all in flight together) and writes the four entries they fill; the two halves are apart so that what else a
// prologue reads can be requested before the first of it is waited for.
// The four entries from eight channels x four features.
__device__ __forceinline__ void write_w_entries(const uint2 (&r)[8], uint4* dst) {
  auto lo = [](uint32_t a, uint32_t b) { return (a & 0xffffu) | (b << 16); };
  auto hi = [](uint32_t a, uint32_t b) { return (a >> 16) | (b & 0xffff0000u); };
  dst[0] = make_uint4(lo(r[0].x, r[1].x), lo(r[2].x, r[3].x), lo(r[4].x, r[5].x), lo(r[6].x, r[7].x));
  dst[1] = make_uint4(hi(r[0].x, r[1].x), hi(r[2].x, r[3].x), hi(r[4].x, r[5].x), hi(r[6].x, r[7].x));
  dst[2] = make_uint4(lo(r[0].y, r[1].y), lo(r[2].y, r[3].y), lo(r[4].y, r[5].y), lo(r[6].y, r[7].y));
  dst[3] = make_uint4(hi(r[0].y, r[1].y), hi(r[2].y, r[3].y), hi(r[4].y, r[5].y), hi(r[6].y, r[7].y));
}
template <int D>
struct WImage {
  using C = Cfg<D>;
  uint2 r[8];
  __device__ __forceinline__ void load(const uint16_t* __restrict__ w, int tid) {
    const int mq = tid % 8, mb = (tid / 8) % C::UM, g = (tid / (8 * C::UM)) % 2, ks = tid / (16 * C::UM);
    const uint16_t* src = w + (16 * ks + 8 * g) * C::HALF + owned_row<C::HALF>(mb, 4 * mq);
    if (tid >= C::W_IMG / 4) return;
#pragma unroll
    for (int e = 0; e < 8; ++e) r[e] = *reinterpret_cast<const uint2*>(src + e * C::HALF);
  }
  __device__ __forceinline__ void write(uint4* sWA, int tid) const {      // at least W_IMG/4 threads
    const int mq = tid % 8, mb = (tid / 8) % C::UM, g = (tid / (8 * C::UM)) % 2, ks = tid / (16 * C::UM);
    if (tid < C::W_IMG / 4) write_w_entries(r, sWA + (ks * C::UM + mb) * 64 + 32 * g + 4 * mq);
  }
};

// N uses (MFMAs) of 16-byte operands that come from LDS or global memory, each requested AHEAD uses
// before it is needed.  Left to itself the compiler, short of registers, issues read, wait, MFMA,
// read, wait, MFMA: with one wavefront per SIMD nothing hides those waits.  AHEAD = 0 keeps that
// order but fences it, so that a single operand is live at a time.
template <int N, int AHEAD, typename Load, typename Use>
__device__ __forceinline__ void pipelined_operands(Load load, Use use) {
  uint4 op[N];
#pragma unroll
  for (int i = 0; i < AHEAD && i < N; ++i) op[i] = load(i);
#pragma unroll
  for (int i = 0; i < N; ++i) {
    if (i + AHEAD < N) op[i + AHEAD] = load(i + AHEAD);
    __builtin_amdgcn_sched_barrier(0);
    use(i, op[i]);
    __builtin_amdgcn_sched_barrier(0);
  }
}

// First half of Eq. 5 for the 32 tokens of one wavefront: U^T = W~^T X^T on bf16 MFMA.
// xb[ks] is this lane's B operand (8 channels of its token per k-step).  On return the lane holds
// u[mb][r] = pre-softmax feature g*LOC + 16*mb + r of its token.  xb is dead afterwards, so the
// caller can refill it with the next block while the softmax runs.
template <int D>
__device__ __forceinline__ void project(const uint4 (&xb)[Cfg<D>::UK], const uint4* sWA, int lane,
                                        f32x16 (&u)[Cfg<D>::UM]) {
  using C = Cfg<D>;
#pragma unroll
  for (int mb = 0; mb < C::UM; ++mb)
#pragma unroll
    for (int r = 0; r < 16; ++r) u[mb][r] = 0.f;
  const uint4* wa = sWA + lane + opaque_zero();
#pragma unroll
  for (int ks = 0; ks < C::UK; ++ks) {
    const bf16x8 b = as_bf16x8(xb[ks]);
#pragma unroll
    for (int mb = 0; mb < C::UM; ++mb) {
      const bf16x8 a = as_bf16x8(wa[(ks * C::UM + mb) * 64]);
      u[mb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, u[mb], 0, 0, 0);
    }
  }
}

// Sum of the two fp16 halves of a packed pair, added to an fp32 accumulator (v_dot2_f32_f16 against (1, 1):
// exact products, fp32 sum).
__device__ __forceinline__ float add_pair_f16(uint32_t p, float acc) {
  const f16x2 one = {(_Float16)1.0f, (_Float16)1.0f};
  return __builtin_amdgcn_fdot2(__builtin_bit_cast(f16x2, p), one, acc, false);
}

// Second half of Eq. 5: the two softmaxes over the d/2 features (in-lane, plus one exchange with
// lane^32).  pk[] receives the lane's d/2 values of phi as fp16 pairs: first LOC values
// softmax(+u) for features g*LOC .. g*LOC+LOC-1, then LOC values softmax(-u) for the same
// features.  valid == false zeroes the token (tail masking happens after phi: phi(0) is the
// uniform vector, not zero).
// CENTRE: the values are phi - 2/D (phi minus its mean over the features), so that the fp16 rounding
// acts on the deviation from the uniform map; the caller adds (2/D) x the column sums back.
template <int D, bool CENTRE = false>
__device__ __forceinline__ void softmax_pair(const f32x16 (&u)[Cfg<D>::UM], bool valid, uint32_t (&pk)[Cfg<D>::NPK]) {
  using C = Cfg<D>;
  float mx = u[0][0], mn = u[0][0];
#pragma unroll
  for (int mb = 0; mb < C::UM; ++mb)
#pragma unroll
    for (int r = 0; r < 16; ++r) { mx = fmaxf(mx, u[mb][r]); mn = fminf(mn, u[mb][r]); }
  float lo, hi;
  pair32(mx, lo, hi); mx = fmaxf(lo, hi);
  pair32(mn, lo, hi); mn = fminf(lo, hi);
  // one softmax half at a time keeps only LOC exponentials live
#pragma unroll
  for (int half = 0; half < 2; ++half) {
    const float sl = half ? -kLog2e : kLog2e;
    const float c0 = half ? mn * kLog2e : -mx * kLog2e;
    float e[C::LOC];
    float s = 0.f;
#pragma unroll
    for (int mb = 0; mb < C::UM; ++mb)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const float a = __builtin_amdgcn_exp2f(fmaf(u[mb][r], sl, c0));
        e[16 * mb + r] = a;
        s += a;
      }
    pair32(s, lo, hi); s = lo + hi;
    const float inv = valid ? __builtin_amdgcn_rcpf(s) : 0.f;
    if constexpr (CENTRE) {
      const float mc = valid ? -2.0f / D : 0.f;
#pragma unroll
      for (int j = 0; j < C::LOC / 2; ++j)
        pk[half * (C::LOC / 2) + j] = pack_f16x2(fmaf(e[2 * j], inv, mc), fmaf(e[2 * j + 1], inv, mc));
    } else {
#pragma unroll
    for (int j = 0; j < C::LOC / 2; ++j) pk[half * (C::LOC / 2) + j] = pack_f16x2(e[2 * j] * inv, e[2 * j + 1] * inv);
    }
  }
}

// Eq. 5 up to a per-token positive factor, for the query side only: the output of Eq. 3 is a ratio
// that is linear in phi(q_i) above and below, so phi(q_i) may be scaled by any positive number.
// Scaling by the softmax(+u) denominator s+ leaves exp(u - max u) as the first half and
// (s+/s-) exp(min u - u) as the second: one multiply per token-half saved, values stay in (0, 64].
template <int D>
__device__ __forceinline__ void softmax_pair_ratio(const f32x16 (&u)[Cfg<D>::UM], uint32_t (&pk)[Cfg<D>::NPK]) {
  using C = Cfg<D>;
  float mx = u[0][0], mn = u[0][0];
#pragma unroll
  for (int mb = 0; mb < C::UM; ++mb)
#pragma unroll
    for (int r = 0; r < 16; ++r) { mx = fmaxf(mx, u[mb][r]); mn = fminf(mn, u[mb][r]); }
  float lo, hi;
  pair32(mx, lo, hi); mx = fmaxf(lo, hi);
  pair32(mn, lo, hi); mn = fminf(lo, hi);
  float sp = 0.f;
  {
    const float c0 = -mx * kLog2e;
    float e[C::LOC];
#pragma unroll
    for (int mb = 0; mb < C::UM; ++mb)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const float a = __builtin_amdgcn_exp2f(fmaf(u[mb][r], kLog2e, c0));
        e[16 * mb + r] = a;
        sp += a;
      }
#pragma unroll
    for (int j = 0; j < C::LOC / 2; ++j) pk[j] = pack_f16x2(e[2 * j], e[2 * j + 1]);
    pair32(sp, lo, hi); sp = lo + hi;
  }
  {
    const float c0 = mn * kLog2e;
    float e[C::LOC];
    float sm = 0.f;
#pragma unroll
    for (int mb = 0; mb < C::UM; ++mb)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const float a = __builtin_amdgcn_exp2f(fmaf(u[mb][r], -kLog2e, c0));
        e[16 * mb + r] = a;
        sm += a;
      }
    pair32(sm, lo, hi); sm = lo + hi;
    const float ratio = sp * __builtin_amdgcn_rcpf(sm);
#pragma unroll
    for (int j = 0; j < C::LOC / 2; ++j) pk[C::LOC / 2 + j] = pack_f16x2(e[2 * j] * ratio, e[2 * j + 1] * ratio);
  }
}

template <int CTRL>
__device__ __forceinline__ float dpp_move(float v) {
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, 0xf, 0xf, true));
}
// Reductions over the four lanes l, l+16, l+32, l+48 (in 16-token blocks a token), every one of them receives the result.  Two or four at a time: a swap of two quantities
// combines both in one operation.
struct SumOp { static __device__ __forceinline__ float of(float a, float b) { return a + b; } };
struct MaxOp { static __device__ __forceinline__ float of(float a, float b) { return fmaxf(a, b); } };
// a, b -> [a of the low 32 lanes, b of the low 32], [a of the high 32, b of the high 32]
__device__ __forceinline__ void swap32(float& a, float& b) {
  auto r = __builtin_amdgcn_permlane32_swap(__builtin_bit_cast(uint32_t, a), __builtin_bit_cast(uint32_t, b), false, false);
  a = __builtin_bit_cast(float, (uint32_t)r[0]); b = __builtin_bit_cast(float, (uint32_t)r[1]);
}
// rows of 16 lanes: a, b -> [a0, b0, a2, b2], [a1, b1, a3, b3]
__device__ __forceinline__ void swap16(float& a, float& b) {
  auto r = __builtin_amdgcn_permlane16_swap(__builtin_bit_cast(uint32_t, a), __builtin_bit_cast(uint32_t, b), false, false);
  a = __builtin_bit_cast(float, (uint32_t)r[0]); b = __builtin_bit_cast(float, (uint32_t)r[1]);
}
template <typename Op>
__device__ __forceinline__ float quad(float a) {
  float b = a;
  swap32(a, b); a = b = Op::of(a, b);
  swap16(a, b); return Op::of(a, b);
}
template <typename Op>
__device__ __forceinline__ void quad2(float& a, float& b) {
  swap32(a, b);
  float s = Op::of(a, b), t = s;
  swap16(s, t); a = b = Op::of(s, t);
  swap32(a, b);
}
template <typename Op>
__device__ __forceinline__ void quad4(float& a, float& b, float& c, float& d) {
  swap32(a, b); swap32(c, d);
  float s = Op::of(a, b), t = Op::of(c, d);
  swap16(s, t);
  a = b = Op::of(s, t);                  // rows: a, c, b, d
  swap32(a, b);
  c = a; d = b;
  swap16(a, c); swap16(b, d);
}
// Maxima of magnitudes, which compare as integers (a floating-point maximum of exchanged values first quiets both): over the four lanes of a token, and
// over the 16 lanes of a row.
struct MagOp {
  static __device__ __forceinline__ float of(float a, float b) {
    const uint32_t x = __builtin_bit_cast(uint32_t, a), y = __builtin_bit_cast(uint32_t, b);
    return __builtin_bit_cast(float, x > y ? x : y);
  }
};
__device__ __forceinline__ float row_max_mag(float x) {
  x = MagOp::of(x, dpp_move<0xB1>(x));      // quad_perm [1,0,3,2]
  x = MagOp::of(x, dpp_move<0x4E>(x));      // quad_perm [2,3,0,1]
  x = MagOp::of(x, dpp_move<0x124>(x));     // row_ror 4
  return MagOp::of(x, dpp_move<0x128>(x));  // row_ror 8
}

// Sum of x over the 16 lanes of a row, and over the 32 lanes that share lane/32 (every one of them receives it): DPP inside a
// row, then the two rows of a half are exchanged with one permlane16 swap.
__device__ __forceinline__ float row_sum(float x) {
  x += dpp_move<0xB1>(x);      // quad_perm [1,0,3,2]
  x += dpp_move<0x4E>(x);      // quad_perm [2,3,0,1]
  x += dpp_move<0x124>(x);     // row_ror 4
  return x + dpp_move<0x128>(x);     // row_ror 8
}
__device__ __forceinline__ float half_wave_sum(float x) {
  float a = row_sum(x), b = a;
  swap16(a, b);
  return a + b;
}

__device__ __forceinline__ float state_scale(float amax) {
  return (amax >= 0x1p-100f && amax < 3.0e38f) ? ldexpf(1.0f, 13 - ilogbf(amax)) : 1.0f;   // the scale itself stays finite
}
// A state (S, dS) [D][D] fp32 of one head in the registers of a workgroup: thread tid < ITEMS holds features 8*fo .. +7 x channels
// 4*cq .. +3, the others zeros.  Eight 16-byte loads in flight per thread, and every operand image is written from here: the statistics an image
// needs first (means, the largest magnitude) are taken on the registers, with no pass through LDS or memory for the state itself.
template <int D, int NTHREADS>
struct StateRegs {
  using L = ApplyLayout<D>;
  static constexpr int CQ = D / 4, FO = D / 8, ITEMS = CQ * FO;
  static_assert(ITEMS <= NTHREADS, "one item per thread");
  float v[8][4];
  int fo, cq;
  bool active;
  __device__ __forceinline__ void load(const float* __restrict__ S, int tid) {
    active = tid < ITEMS;
    cq = tid % CQ; fo = (tid / CQ) % FO;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const float4 r = active ? *reinterpret_cast<const float4*>(S + (8 * fo + e) * D + 4 * cq) : make_float4(0.f, 0.f, 0.f, 0.f);
      v[e][0] = r.x; v[e][1] = r.y; v[e][2] = r.z; v[e][3] = r.w;
    }
  }
  // part[FO][D]: sums over each octet of features
  __device__ __forceinline__ void octet_sums(float* part) const {
    if (!active) return;
    float s[4];
#pragma unroll
    for (int i = 0; i < 4; ++i)
      s[i] = ((v[0][i] + v[1][i]) + (v[2][i] + v[3][i])) + ((v[4][i] + v[5][i]) + (v[6][i] + v[7][i]));
    *reinterpret_cast<float4*>(part + fo * D + 4 * cq) = make_float4(s[0], s[1], s[2], s[3]);
  }
  // The column block that carries z (column block MB of MBS = MB + 1): entry (ks, MB, lane = (c, g)) holds scale * z[feature(ks, g, e)]
  // whatever c is, so each lane of the product receives phi . z of its own token rows.
  template <int KIND = kPhiHedgehog>
  static __device__ __forceinline__ void write_z_block(const float* z, uint4* img, float sc, int tid) {
    for (int it = tid; it < L::KS * 64; it += NTHREADS) {
      const int ks = it / 64, g = (it / 32) % 2;
      const float* f = z + (KIND == kPhiRelu ? 16 * ks + 8 * g : L::feature(ks, g, 0));
      img[(ks * L::MBZ + L::MB) * 64 + it % 64] = make_uint4(pack_f16x2(sc * f[0], sc * f[1]), pack_f16x2(sc * f[2], sc * f[3]),
                                                             pack_f16x2(sc * f[4], sc * f[5]), pack_f16x2(sc * f[6], sc * f[7]));
    }
  }
  // Power of two that brings the largest magnitude (of amax and the state) into [2^13, 2^14): fp16 operand images of the state are
  // scaled by it; every consumer forms a ratio or divides the scale out again.  red: NTHREADS/64 floats.  Contains a barrier.
  __device__ __forceinline__ float scale(float* red, int tid, float amax = 0.f) const {
#pragma unroll
    for (int e = 0; e < 8; ++e)
#pragma unroll
      for (int i = 0; i < 4; ++i) amax = fmaxf(amax, fabsf(v[e][i]));
    amax = quad<MagOp>(row_max_mag(amax));
    if (tid % 64 == 0) red[tid / 64] = amax;
    __syncthreads();
#pragma unroll
    for (int i = 0; i < NTHREADS / 64; ++i) amax = fmaxf(amax, red[i]);
    return state_scale(amax);
  }
  // B operands of Y = phi S (contraction over the features of phi, tokens on the accumulator rows): entry (ks, mb, lane = (c, g)), MBS
  // column blocks to a k-step, holds scale * S[feature(ks, g, e)][channel_cols(mb, c)].
  // KIND = kPhiRelu: the features are the d channels in their plain order, 16ks + 8g + e.
  template <int MBS, int KIND = kPhiHedgehog>
  __device__ __forceinline__ void write_apply_image(uint4* img, float sc) const {
    if (!active) return;
    const int g = KIND == kPhiRelu ? fo % 2 : (fo / (D / 32)) % 2;
    const int ks = KIND == kPhiRelu ? fo / 2 : fo / (D / 16) * (L::KS / 2) + fo % (D / 32);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int ch = 4 * cq + i;
      img[(ks * MBS + ch % L::MB) * 64 + 32 * g + ch / L::MB] =
          make_uint4(pack_f16x2(sc * v[0][i], sc * v[1][i]), pack_f16x2(sc * v[2][i], sc * v[3][i]),
                     pack_f16x2(sc * v[4][i], sc * v[5][i]), pack_f16x2(sc * v[6][i], sc * v[7][i]));
    }
  }
};

// Transposing LDS read: from a [row][column] fp16 tile, lane l of a wavefront receives
// tile[row0 + 8*(l/32) + 0..7][col0 + l%32] -- an MFMA A or B operand whose contraction index
// is the tile row.  Two ds_read_b64_tr_b16: within each group of 16 lanes, lane s supplies the
// address of row s/4, columns 4*(s%4)..+3, and receives column s of the four rows.
// tr_offset() is the lane's byte offset for row0 = 0 and the first (j = 0) or second (j = 1)
// group of four rows; row0 = 16*ks adds 16*ks*RS bytes (the swizzle repeats every 16 rows).
// The 32-column block and the group enter by exclusive-or: a block's chunk numbers differ from block 0's in bits that the lane's part leaves 0,
// and row r + 4 (r + 8 below) changes one bit of the swizzle.
template <int D, int ROWS>      // ROWS: tile rows between the lane groups of 32
__device__ __forceinline__ int tr_lane(unsigned lane) {
  const unsigned r = ROWS * (lane / 32) + (lane % 16) / 4;
  return (int)(r * (D * 2) + (((2 * (lane / 16 % 2) + lane % 4 / 2) ^ (unsigned)swz<D>((int)r)) * 16) + lane % 2 * 8);
}
template <int D>
__device__ __forceinline__ int tr_offset(int col0, int lane, int j) {      // col0: a multiple of 32
  return (tr_lane<D, 8>((unsigned)lane) ^ (2 * col0) ^ (j && D > 32 ? 16 : 0)) + j * 4 * (D * 2);
}

// Byte offset of this lane's address for a transposing read of an operand of k-step 0 in the
// token order of a turned operand (the 16 tokens behind a lane's accumulator registers):
// j = 0: tile rows 4g .. 4g+3, j = 1: rows 8+4g .. 8+4g+3 (g = lane/32); columns col0 + lane%32.
template <int D>
__device__ __forceinline__ int tr_offset_g4(int col0, int lane, int j) {
  return (tr_lane<D, 4>((unsigned)lane) ^ (2 * col0) ^ (j && D > 32 ? 32 : 0)) + j * 8 * (D * 2);
}

// LDS addresses as 32-bit integers.  tr_base() puts a tile's base into the register that an offset is in, where the optimiser cannot take it out
// again: what is left to add, the k-step, then fits the instruction's 16-bit offset.  With the base (the tiles lie above 64 KB) among the
// constants every read had an addition of its own, 126 in the contractions of a tile of the query-side backward.
__device__ __forceinline__ uint32_t lds_address(const void* p) { return (uint32_t)(uintptr_t)(__attribute__((address_space(3))) const char*)p; }
__device__ __forceinline__ uint32_t tr_base(const char* tile, int off) {
  uint32_t a = lds_address(tile) + (uint32_t)off;
  asm volatile("" : "+v"(a));
  return a;
}
__device__ __forceinline__ f16x8 read_tr(const char* tile, int off0, int off1) {
  struct { s16x4 lo, hi; } v;
  v.lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)(tile + off0));
  v.hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)(tile + off1));
  return __builtin_bit_cast(f16x8, v);
}
__device__ __forceinline__ f16x8 read_tr(uint32_t at0, uint32_t at1) {
  struct { s16x4 lo, hi; } v;
  v.lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)at0);
  v.hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)at1);
  return __builtin_bit_cast(f16x8, v);
}

// power of two p with p * m in [1, 2) for 2^-100 <= m < 3e38; 1 for smaller m (zero included) and
// for non-finite m.  The lower limit keeps p itself finite: for m below 2^-127 (fp32 subnormals, which
// a saturated softmax leaves in du) the exact normaliser is not representable, and such values are
// zero against anything they are added to, so they may flush in the fp16 operand.
__device__ __forceinline__ float pow2_normaliser(float m) {
  // 2^-ilogb(m), from the exponent; 2^-127 for m from 2^127 is subnormal
  const uint32_t e = 0x7f000000u - (__builtin_bit_cast(uint32_t, m) & 0x7f800000u);
  return m >= 0x1p-100f && m < 3.0e38f ? __builtin_bit_cast(float, e > 0x00400000u ? e : 0x00400000u) : 1.0f;
}

// A token's largest gradient is normalised as if it were no larger than this: the scale is then at least 2^-126, a normal number whose
// reciprocal v_rcp_f32 gives exactly (values from 2^127 would ask for 2^-127), and the operand stays below 8 times the unit it is brought to.  At
// that unit, entries down to 2^-24 of the token's largest are normal fp16 numbers; with 1, those from 2^-14 on lost their low bits.
constexpr float kTokenMax = 0x1.8p126f, kTokenUnit = 0x1p10f;

// Running power-of-two scale of a workgroup's sums over tokens (fp16 MFMA operands, fp32
// accumulators).  A tile whose largest operand magnitude is m wants the scale gamma_for(m), which
// puts m into [16, 32).  The workgroup keeps the smallest scale any of its tiles has asked for and,
// when a tile lowers it, multiplies its accumulators by the exact ratio (gamma_step), so a tile far
// larger than every earlier one cannot overflow fp16, and tiles that are all zero (kGammaUnset) leave
// the choice to the first tile that is not.
constexpr float kGammaUnset = 0x1p60f;
__device__ __forceinline__ float gamma_for(float m) {
  return m >= 0x1p-56f && m < 3.0e38f ? 16.f * pow2_normaliser(m) : kGammaUnset;
}
// Returns the factor (a power of two <= 1) the accumulators must be multiplied by; updates gamma.
__device__ __forceinline__ float gamma_step(float& gamma, float wanted) {
  const float next = fminf(gamma, wanted);
  const float ratio = next * __builtin_amdgcn_rcpf(gamma);      // exact: both are powers of two
  gamma = next;
  return ratio;
}

__device__ __forceinline__ void unpack_bf16x8(uint4 v, float* f) {
  f[0] = __builtin_bit_cast(float, v.x << 16); f[1] = __builtin_bit_cast(float, v.x & 0xffff0000u);
  f[2] = __builtin_bit_cast(float, v.y << 16); f[3] = __builtin_bit_cast(float, v.y & 0xffff0000u);
  f[4] = __builtin_bit_cast(float, v.z << 16); f[5] = __builtin_bit_cast(float, v.z & 0xffff0000u);
  f[6] = __builtin_bit_cast(float, v.w << 16); f[7] = __builtin_bit_cast(float, v.w & 0xffff0000u);
}

// max(x, 0) on a packed pair of bf16 (-0 becomes +0).
// As 16-bit integers the negative bf16 values are exactly the negative numbers, so one packed
// signed maximum with 0 does it.
__device__ __forceinline__ uint32_t relu_bf16x2(uint32_t u) {
  typedef short s16x2 __attribute__((ext_vector_type(2)));
  const s16x2 z = {0, 0};
  return __builtin_bit_cast(uint32_t, __builtin_elementwise_max(__builtin_bit_cast(s16x2, u), z));
}
// Eight bf16 of a row -> fp16 of max(x, 0): an MFMA operand piece of the ReLU map.
__device__ __forceinline__ uint4 relu_f16x8(uint4 x) {
  uint4 r;
  r.x = bf16x2_to_f16x2(relu_bf16x2(x.x)); r.y = bf16x2_to_f16x2(relu_bf16x2(x.y));
  r.z = bf16x2_to_f16x2(relu_bf16x2(x.z)); r.w = bf16x2_to_f16x2(relu_bf16x2(x.w));
  return r;
}

// The 32 rows from token t0 of a head of n tokens, as the accumulators with tokens on the rows hold them: lane (c, g), register r has PIECE
// bytes of token t0 + 8*(r/4) + 4g + r%4, at byte PIECE*c of the row, so that every store instruction writes two whole rows.
// The stores are buffer stores bounded to the rows that exist: the hardware drops those past n.  No branch (behind one the compiler cannot count the
// stores in flight, and a later wait for a load that was requested before them, the next block's rows, turns into a wait for the
// stores as well), and one vector instruction for an address.  Choosing between the row and a sink by a select took five, 64 more a block: a pass
// of 4 x 1000 x 64 took 8.5 us in place of 8.0, of 12 x 4133 x 64 7.7 in place of 6.9, the fp32-arithmetic key side (12 x 32760 x 128, bf16 tensors),
// which that kept from spilling, 164 in place of 156, each with the kernel of that time; nothing where the memory or the barriers of dW~ are what is waited for.
// All arguments but the lane are uniform.
template <int PIECE>
struct TokenRows {
  __amdgpu_buffer_rsrc_t rows;
  uint32_t at, pitch;
  __device__ __forceinline__ TokenRows(void* base, size_t pitch_bytes, int t0, int n, int lane) {
    const int left = n - t0 < 32 ? n - t0 : 32;
    pitch = (uint32_t)pitch_bytes;
    rows = __builtin_amdgcn_make_buffer_rsrc(static_cast<char*>(base) + (size_t)t0 * pitch_bytes, 0, left > 0 ? (uint32_t)left * pitch : 0, 0x00020000);
    const int lz = lane + opaque_zero();                   // (the sixteen offsets are not held across a caller's loop)
    at = (uint32_t)(4 * (lz / 32)) * pitch + (uint32_t)(PIECE * (lz % 32));
  }
  template <bool STREAM, typename V>                       // STREAM: non-temporal
  __device__ __forceinline__ void store(int r, V v) const {
    static_assert(sizeof(V) == PIECE, "a lane's piece of a row");
    const uint32_t off = at + (uint32_t)(8 * (r / 4) + r % 4) * pitch;
    constexpr int aux = STREAM ? 2 : 0;
    if constexpr (PIECE == 4) __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, v), rows, off, 0, aux);
    else if constexpr (PIECE == 8) __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2, v), rows, off, 0, aux);
    else __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, v), rows, off, 0, aux);
  }
};

// 32x32x16 MFMA on operands carried as f16x8 registers whose bits are fp16 or (BF16) bf16.
template <bool BF16>
__device__ __forceinline__ f32x16 mfma16(f16x8 a, f16x8 b, f32x16 c) {
  if constexpr (BF16)
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
  else
    return __builtin_amdgcn_mfma_f32_32x32x16_f16(a, b, c, 0, 0, 0);
}

// Wavefront pw (of four) owns D/64 x D/64 blocks of 32 features x 32 channels of a state: feature blocks fblk(0 ..), channel blocks cblk(0 ..).  The
// first of its feature blocks, zblk, is the one whose z it sums (width 64: two wavefronts have it, do_z is one of them).
template <int D>
struct Quadrant {
  static constexpr int WMN = D / 64;
  int mi, ni;
  __device__ __forceinline__ explicit Quadrant(int pw) : mi(pw / 2), ni(pw % 2) {}
  __device__ __forceinline__ int fblk(int i) const { return mi * WMN + (WMN == 2 ? i ^ ni : i); }
  __device__ __forceinline__ int cblk(int j) const { return ni * WMN + j; }
  __device__ __forceinline__ int zblk() const { return fblk(0); }
  __device__ __forceinline__ bool do_z() const { return WMN == 2 || ni == 0; }
};
// Where a lane's transposing reads of k-step 0 of its blocks start (tr_offset): tiles sA (features) and sB (channels).
template <int D>
struct QuadrantReads {
  uint32_t a[D / 64][2], b[D / 64][2];
  __device__ __forceinline__ QuadrantReads(const Quadrant<D>& qd, const char* sA, const char* sB, int lane) {
#pragma unroll
    for (int i = 0; i < D / 64; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        a[i][j] = tr_base(sA, tr_offset<D>(32 * qd.fblk(i), lane, j));
        b[i][j] = tr_base(sB, tr_offset<D>(32 * qd.cblk(i), lane, j));
      }
  }
};

// One 128-token tile of a split-n sum over tokens: s[i][j] += A_i^T B_j and zacc += A_0^T w, with A
// and B fp16 tiles [kTile][D] in LDS (swizzled 16-byte chunks) read by transposing reads, the
// operands of k-step ks+1 requested before the MFMAs of k-step ks.  wop(ks) returns the B operand
// of the z sum for that k-step (per-token weights, the same in every column); do_z whether this wavefront owns a z block at all.
// BF16: the tiles and wop's operands hold bf16 instead of fp16 (same bits per element, bf16 MFMA).
template <int D, bool BF16 = false, typename WOp>
__device__ __forceinline__ void contract_tile(const QuadrantReads<D>& rd, f32x16 (&s)[D / 64][D / 64],
                                              f32x16& zacc, bool do_z, WOp wop) {
  constexpr int RS = D * 2, WMN = D / 64, KSN = kTile / 16;
  f16x8 a[KSN][WMN], b[KSN][WMN], wv[KSN];
  auto request = [&](int kn) {
#pragma unroll
    for (int i = 0; i < WMN; ++i) a[kn][i] = read_tr(rd.a[i][0] + kn * 16 * RS, rd.a[i][1] + kn * 16 * RS);
#pragma unroll
    for (int j = 0; j < WMN; ++j) b[kn][j] = read_tr(rd.b[j][0] + kn * 16 * RS, rd.b[j][1] + kn * 16 * RS);
    wv[kn] = wop(kn);
  };
  request(0);
#pragma unroll
  for (int ks = 0; ks < KSN; ++ks) {
    if (ks + 1 < KSN) request(ks + 1);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i < WMN; ++i)
#pragma unroll
      for (int j = 0; j < WMN; ++j) s[i][j] = mfma16<BF16>(a[ks][i], b[ks][j], s[i][j]);
    if (WMN == 2 || do_z) zacc = mfma16<BF16>(a[ks][0], wv[ks], zacc);
    __builtin_amdgcn_sched_barrier(0);
  }
}

}  // namespace linattn
