// bf16-I/O backward path on gfx950 MFMA.  The paper trains through the converted layers
// (Sec. 5.1) but prints no gradient formula; these kernels apply the chain rule to Eq. 3 and Eq. 5.
// With S, z from the forward, den_i = phi(q_i).z, o_i = phi(q_i) S / den_i, delta_i = dO_i.o_i:
//
//   query side   g_i  = dL/dphi(q_i) = (dO_i S^T - delta_i z) / den_i
//                dS   = sum_i phi(q_i)^T dO_i / den_i          dz = -sum_i phi(q_i) delta_i / den_i
//   key side     g_j  = dL/dphi(k_j) = v_j dS^T + dz           dv_j = phi(k_j) dS
//   through phi  du = p+ (g+ - <g+,p+>) - p- (g- - <g-,p->),   dx = du W~^T,   dW~ = sum x^T du
//
// bwd_q_kernel    : per 128-token tile: phi(Q), G = dO S^T, delta, du, dq; dS, dz partials (split-n); dW~_q partials
// bwd_k_kernel    : per 16-token block: phi(K), g, du, dk, dv; dW~_k partials
// (the partials are reduced in state_reduce.hip)
//
// Precision: every 16-bit MFMA operand except the stored bf16 q, k (projection) is fp16.
// Operands that belong to one token or block only (dO_i for g_i, du_i for dx_i) are scaled by a
// power of two taken from their largest magnitude, so any gradient scale is safe; bf16 values scaled so are exact in fp16 (in dO_i
// with a factor of up to three bits beside it).  In the sums over
// tokens the weight 1/den_i goes into phi_i (where phi's roundings have too much in common into dO_i, see kSharedRounding), with one power of two per
// workgroup that follows the running maximum of |dO_i|/den_i over its tiles (largest magnitude so far in [16, 32)), and du for dW~ is scaled likewise;
// when a tile raises the maximum the fp32 accumulators are rescaled by the exact ratio, so neither a
// late large tile nor leading all-zero tiles can overflow or flush fp16.  delta enters dz in fp32.  Accumulation is fp32 everywhere; partial
// sums are combined in a fixed order.
#pragma once
#include "kernels.h"
#include "mfma16.h"

namespace linattn {
namespace {

// ---- operand images ------------------------------------------------------------------------
// Each workgroup of the two main kernels builds the images it needs in LDS, straight from the fp32 state and W~: the state is held
// in registers (StateRegs) while the statistics below are taken, a microsecond or two of prologue.  As kernels of their own, once
// per head, the images cost 11.5 + 11.5 us per call (12 heads of width 128, latency) and the main kernels as long a prologue to
// copy them in.
// Both sides centre the state before it is rounded to fp16 operands (exact in real arithmetic; the roundings
// then act on what the gradients are made of instead of on a common part that cancels):
//   query side:   S^c = S - z vbar^T with vbar = sum_j v_j / n (the + half of S sums to sum_j v_j, the + half
//                 of z to n).  The kernel then has delta^c = delta - dO . vbar, g is unchanged, and its dz comes
//                 out as dz^c = dz + dS vbar.
//   key side:     dz is completed against the ROUNDED image: dzc[f] = dz^c[f] - vbar . r(dS[f]), so
//                 that v_j . r(dS[f]) + dzc[f] = (v_j - vbar) . r(dS[f]) + dz^c[f] holds exactly and the rounding
//                 of the image acts on v_j - vbar, not on v_j (values with a common offset cost nothing).
//   CENTRE (LINATTN_FLAG_CENTRED): the query-side kernel accumulated dS' = sum (phi - 2/D)^T dO/den and dz' likewise;
//                 (2/D) x its column sums (cs_part) complete them: dS = dS' + (2/D) 1 colsum^T (constant over the
//                 features: it only enters the row that dv gets back), dz^c = dz' + (2/D) wsum.  In addition the
//                 mean over each half's features is taken out of dS' and of dz^c: the softmax Jacobian drops what
//                 is constant over a half, and dv gets the constant row mean_+ + mean_- back.  (Without the flag
//                 this last step is left out: where phi is spiky the rows of dS differ by orders of magnitude and
//                 a common shift only adds rounding error to the small ones.)

// Query side: image of S^c, z in sZ[D]; returns the image's scale.  vbar_out: non-null in one workgroup per head.
// scratch: FO*D + D + NTHREADS/64 floats of LDS.  Ends before the barrier that the caller needs after building its images.
// S: the state, loaded; z: element tid < D of its row z.
template <int D, int NTHREADS>
__device__ __forceinline__ float build_query_state(StateRegs<D, NTHREADS>& S, float z, uint4* sGA, float* sZ, float* scratch,
                                                   float* __restrict__ vbar_out, int tid) {
  using R = StateRegs<D, NTHREADS>;
  float* part = scratch;
  float* vb = part + R::FO * D;                             // (bwd_q_kernel keeps it with DR)
  float* red = vb + D;
  if (tid < D) sZ[tid] = z;
  S.octet_sums(part);
  __syncthreads();
  if (tid < D) {
    // column sums of the + half of S; the + half of z sums to n
    float sv = 0.f, nt = 0.f;
#pragma unroll
    for (int o = 0; o < R::FO / 2; ++o) sv += part[o * D + tid];
#pragma unroll
    for (int q = 0; q < D / 8; ++q) {
      const float4 z = reinterpret_cast<const float4*>(sZ)[q];
      nt += (z.x + z.y) + (z.z + z.w);
    }
    const float c = sv / nt;
    vb[tid] = c;
    if (vbar_out != nullptr) vbar_out[tid] = c;
  }
  __syncthreads();
#pragma unroll
  for (int e = 0; e < 8; ++e)
#pragma unroll
    for (int i = 0; i < 4; ++i) S.v[e][i] -= sZ[8 * S.fo + e] * vb[4 * S.cq + i];
  if (!S.active) {
#pragma unroll
    for (int e = 0; e < 8; ++e)
#pragma unroll
      for (int i = 0; i < 4; ++i) S.v[e][i] = 0.f;
  }
  const float scale = S.scale(red, tid);
  write_grad_image16<D, NTHREADS>(S, sGA, scale);
  return scale;
}

// Key side: the two images of dS, the matched dz in sZ[D], the constant row of dv in sRow[D] (zero without CENTRE); returns the scale.
// scratch: FO*D + 4*D + NTHREADS/64 + 4 floats of LDS.
// S: dS, loaded; dz, vb_own: element tid < D of its row dz and of vbar.
template <int D, int NTHREADS, bool CENTRE>
__device__ __forceinline__ float build_key_state(StateRegs<D, NTHREADS>& S, float dz, float vb_own, uint4* sVA, uint4* sGA, float* sZ, float* sRow,
                                                 float* scratch, const float* __restrict__ cs_part, int P, int tid) {
  using R = StateRegs<D, NTHREADS>;
  float* part = scratch;
  float* vb = part + R::FO * D;
  float* m0 = vb + D;
  float* m1 = m0 + D;
  float* cB = m1 + D;
  float* red = cB + D;                                      // [NTHREADS/64], then wsum and the two means of dz
  float* misc = red + NTHREADS / 64;
  if (tid < D) {
    vb[tid] = vb_own;
    cB[tid] = dz;
  }
  if constexpr (CENTRE) {
    // column sums and wsum of the query-side workgroups, in a fixed order
    float colsum = 0.f;
    if (tid <= D)
      for (int p = 0; p < P; p += 8) {
        float t[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) t[i] = p + i < P ? cs_part[(size_t)(p + i) * (D + 8) + tid] : 0.f;
        colsum += ((t[0] + t[1]) + (t[2] + t[3])) + ((t[4] + t[5]) + (t[6] + t[7]));
      }
    if (tid == D) misc[0] = colsum;
    S.octet_sums(part);
    __syncthreads();
    const float wsum = misc[0];
    if (tid < D) {
      float a = 0.f, b = 0.f;
#pragma unroll
      for (int o = 0; o < R::FO / 2; ++o) { a += part[o * D + tid]; b += part[(R::FO / 2 + o) * D + tid]; }
      a *= 2.0f / D; b *= 2.0f / D;
      m0[tid] = a; m1[tid] = b;
      sRow[tid] = (a + b) + (4.0f / D) * colsum;
      cB[tid] += (2.0f / D) * wsum;
    }
    __syncthreads();
    if (tid < 128) {
      // the mean of each half of dz^c, one wavefront each
      float t = tid % 64 < D / 2 ? cB[(tid / 64) * (D / 2) + tid % 64] : 0.f;
      for (int k = 32; k >= 1; k >>= 1) t += __shfl_xor(t, k, 64);
      if (tid % 64 == 0) misc[1 + tid / 64] = t * (2.0f / D);
    }
    const float* m = S.fo < R::FO / 2 ? m0 : m1;
    if (S.active) {
#pragma unroll
      for (int e = 0; e < 8; ++e)
#pragma unroll
        for (int i = 0; i < 4; ++i) S.v[e][i] -= m[4 * S.cq + i];
    }
  } else {
    if (tid < D) sRow[tid] = 0.f;
  }
  const float scale = S.scale(red, tid);                    // (its barrier covers vb, cB and misc as well)
  write_grad_image16<D, NTHREADS>(S, sGA, scale);
  write_apply_image16<D, NTHREADS>(S, sVA, scale);
  const float inv = __builtin_amdgcn_rcpf(scale);           // exact: a power of two
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    float dot = 0.f;
#pragma unroll
    for (int i = 0; i < 4; ++i) dot = fmaf((float)(_Float16)(scale * S.v[e][i]), vb[4 * S.cq + i], dot);
    dot = D == 128 ? half_wave_sum(dot) : row_sum(dot);     // over the CQ lanes that share the octet of features
    const int f = 8 * S.fo + e;
    if (S.active && S.cq == 0) sZ[f] = cB[f] - (CENTRE ? misc[f < D / 2 ? 1 : 2] : 0.f) - dot * inv;
  }
  return scale;
}

// ---- dW~ = sum_i x_i^T du_i, accumulated inside the kernels that make du ---------------------
// The workgroup parks 128 tokens in LDS as two fp16 tiles, x [kTile][D] and du [kTile][D/2] (rows swizzled
// like the phi tile; a 16-token block of du carries the power-of-two scale du_to_dx16 gave it, with the
// inverse scales beside the tile).  Its NW wavefronts then contract over the tokens with transposing
// reads of both tiles: wavefront w owns the feature block w % NB and RB 32-channel row blocks and brings
// the blocks to one common power-of-two scale that follows the running maximum of the workgroup
// (gamma_step; the accumulators are rescaled by the exact ratio when a tile raises it).  Partials per
// workgroup are reduced in a fixed order afterwards.
template <int D, int NW>
struct DwTile {
  static constexpr int HALF = D / 2;
  static constexpr int RSX = D * 2;                        // bytes per row of the x tile
  static constexpr int RSU = HALF * 2;                     // bytes per row of the du tile
  static constexpr int NB = HALF / 32;                     // 32-column blocks of du
  static constexpr int RB = (D / 32) * NB >= NW ? (D / 32) * NB / NW : 1;   // row blocks per wavefront
  static constexpr int BPT = kTile / 16;                   // du blocks (each with a scale of its own) per parked tile
  static constexpr int KSN = kTile / 16;
  static constexpr int KBATCH = D == 64 ? KSN : KSN / 4;        // k-steps whose operands are in flight together
  static constexpr int DU_BYTES = kTile * RSU;
  f32x16 acc[RB];
  float gamma;
  int fb, row0;
  bool active;

  __device__ __forceinline__ void init(int w) {
    fb = w % NB; row0 = (w / NB) * RB;
    active = row0 < D / 32;
    gamma = kGammaUnset;
#pragma unroll
    for (int i = 0; i < RB; ++i)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][r] = 0.f;
  }
  // lane: pass opaque_lane() from inside the tile loop: the read offsets are then worked out per tile (a few
  // integer operations) instead of being held in registers, or spilled, across the whole loop
  __device__ __forceinline__ void contract(const char* sX, const char* sU, const float* sIts, int lane) {
    float its[BPT];
    float m = 0.f;
#pragma unroll
    for (int i = 0; i < BPT; ++i) { its[i] = sIts[i]; m = fmaxf(m, its[i]); }
    float gnext = gamma;
    float ratio = gamma_step(gnext, gamma_for(m));
    // the same in every lane: kept in scalar registers
    gamma = __builtin_bit_cast(float, __builtin_amdgcn_readfirstlane(__builtin_bit_cast(int, gnext)));
    ratio = __builtin_bit_cast(float, __builtin_amdgcn_readfirstlane(__builtin_bit_cast(int, ratio)));
    if (ratio != 1.f) {
#pragma unroll
      for (int j = 0; j < RB; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[j][r] *= ratio;
    }
    if (!active) return;
    uint32_t offA[RB][2], offB[2];
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      offB[j] = tr_base(sU, tr_offset_g4<HALF>(32 * fb, lane, j));
#pragma unroll
      for (int i = 0; i < RB; ++i) offA[i][j] = tr_base(sX, tr_offset_g4<D>(32 * (row0 + i), lane, j));
    }
    // the operands of KBATCH k-steps are requested before their first MFMA: one LDS latency per batch instead of one per k-step
#pragma unroll
    for (int k0 = 0; k0 < KSN; k0 += KBATCH) {
      f16x8 a[KBATCH][RB], b[KBATCH];
#pragma unroll
      for (int ks = 0; ks < KBATCH; ++ks) {
        b[ks] = read_tr(offB[0] + (k0 + ks) * 16 * RSU, offB[1] + (k0 + ks) * 16 * RSU);
#pragma unroll
        for (int i = 0; i < RB; ++i) a[ks][i] = read_tr(offA[i][0] + (k0 + ks) * 16 * RSX, offA[i][1] + (k0 + ks) * 16 * RSX);
      }
#pragma unroll
      for (int ks = 0; ks < KBATCH; ++ks) {
        const _Float16 f = (_Float16)(gamma * its[k0 + ks]);   // a power of two, or 0 for an all-zero block
        const f16x8 bo = b[ks] * f;
#pragma unroll
        for (int i = 0; i < RB; ++i) acc[i] = __builtin_amdgcn_mfma_f32_32x32x16_f16(a[ks][i], bo, acc[i], 0, 0, 0);
      }
    }
  }
  // part: this workgroup's [D][HALF] partial
  __device__ __forceinline__ void store(float* part, int lane) const {
    if (!active) return;
    const float ig = __builtin_amdgcn_rcpf(gamma);
    const int c = lane % 32, g = lane / 32;
#pragma unroll
    for (int i = 0; i < RB; ++i)
#pragma unroll
      for (int r = 0; r < 16; ++r)
        part[(32 * (row0 + i) + 8 * (r / 4) + 4 * g + (r % 4)) * HALF + 32 * fb + c] = acc[i][r] * ig;
  }
};

// A value that is the same in every lane, in a scalar register.
__device__ __forceinline__ float uniform(float x) { return __builtin_bit_cast(float, __builtin_amdgcn_readfirstlane(__builtin_bit_cast(int, x))); }

// ---- sums over the tokens of a tile ----------------------------------------------------------
// A 128-token tile of dS and dz: s[i][j] += P_i^T Y_j with P = kPhiUnit f phi and Y = y stok dO as fp16 tiles [kTile][D] in LDS (per token f y = (1 - r') / (den stok),
// times the running scale), and z += P_0 . w with w = -y stok delta in fp32, feature lane%32 of the first block over the tokens that the lane
// holds (eight of a k-step; the lane 32 further has the others): as MFMA blocks the z sums took a fifth of the MFMAs and 16 registers.
// The operands of k-step ks+1 are requested before the MFMAs of k-step ks.
// SUMS (centred): also csum[j] += sum f Y, the lane's column of block j, and wsum += sum f w, over the same tokens.
// w, f: the lane's first token of k-step 0.
template <int D, bool SUMS>
__device__ __forceinline__ void contract_tokens(const QuadrantReads<D>& rd, f32x16 (&s)[D / 64][D / 64], float& z, const float* w, const float* f,
                                                float (&csum)[D / 64], float& wsum) {
  constexpr int RS = D * 2, WMN = D / 64, KSN = kTile / 16, AHEAD = D == 64 ? 4 : 1;
  f16x8 a[KSN][WMN], b[KSN][WMN];
  auto request = [&](int kn) {
#pragma unroll
    for (int i = 0; i < WMN; ++i) a[kn][i] = read_tr(rd.a[i][0] + kn * 16 * RS, rd.a[i][1] + kn * 16 * RS);
#pragma unroll
    for (int j = 0; j < WMN; ++j) b[kn][j] = read_tr(rd.b[j][0] + kn * 16 * RS, rd.b[j][1] + kn * 16 * RS);
  };
#pragma unroll
  for (int ks = 0; ks < AHEAD; ++ks) request(ks);
#pragma unroll
  for (int ks = 0; ks < KSN; ++ks) {
    float4 wv[2], fv[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      wv[i] = *reinterpret_cast<const float4*>(w + 16 * ks + 4 * i);
      if constexpr (SUMS) fv[i] = *reinterpret_cast<const float4*>(f + 16 * ks + 4 * i);
    }
    if (ks + AHEAD < KSN) request(ks + AHEAD);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i < WMN; ++i)
#pragma unroll
      for (int j = 0; j < WMN; ++j) s[i][j] = mfma16<false>(a[ks][i], b[ks][j], s[i][j]);
    const float wt[8] = {wv[0].x, wv[0].y, wv[0].z, wv[0].w, wv[1].x, wv[1].y, wv[1].z, wv[1].w};
#pragma unroll
    for (int e = 0; e < 8; ++e) z = fmaf((float)a[ks][0][e], wt[e], z);
    if constexpr (SUMS) {
      const float ft[8] = {fv[0].x, fv[0].y, fv[0].z, fv[0].w, fv[1].x, fv[1].y, fv[1].z, fv[1].w};
#pragma unroll
      for (int e = 0; e < 8; ++e) {
#pragma unroll
        for (int j = 0; j < WMN; ++j) csum[j] = fmaf((float)b[ks][j][e], ft[e], csum[j]);
        wsum = fmaf(wt[e], ft[e], wsum);
      }
#pragma unroll
      for (int j = 0; j < WMN; ++j) asm volatile("" : "+v"(csum[j]));
      asm volatile("" : "+v"(wsum));
    }
    // (the sums are taken here, and not after the branches that follow the tile, with every operand kept until there)
    asm volatile("" : "+v"(z));
    __builtin_amdgcn_sched_barrier(0);
  }
}

// What phi enters that sum with: a power of two that keeps small features out of the fp16 subnormals (f is at most 1, or 32 / kTokenUnit).
constexpr float kPhiUnit = 0x1p14f;
// The relative error of phi . z from rounded phi above which a token's weight is formed with it.  A single feature's rounding gives up to 2^-11; tokens of
// ordinary maps stay below (rms 3e-5, of sharp ones with a feature of 0.2 of den 6e-5), and 1.7e-4 in four ways of rounding is what the other operands'
// roundings leave of tokens with the same query.  dS of such heads, rms: 2e-4 without, 7e-5 now, and 6e-5 with the normaliser from rounded phi for every token,
// which has the weight in dO and rounds both operands.  It costs 1 % of a training step (bwd_q 12 heads x 32760 x 128 with dW~ 92.2 -> 95.7 us; 5 % of
// a backward call of maps so sharp that most tokens are parked twice).
constexpr float kSharedRounding = 0x1.6p-13f;

// z in fp16 pieces, as the A operands of the product that gives the token wavefronts phi . z from phi in fp16: piece r of scale * z, 12 bits
// below the one before it, in the rows 4q + r, so that a lane receives its token's four sums in its four accumulator registers and no exchange is needed.
template <int D>
struct ZPieces {
  using K = Tok16<D>;
  static constexpr int IMG = 2 * K::DK * 16;      // uint4 entries: (ks, q, r), eight features as in Tok16
  // z is at most n in each feature (and a sum of states over a few thousand devices fits)
  static __device__ __forceinline__ float scale(int n) { return 16.f * pow2_normaliser((float)n); }
  static __device__ __forceinline__ void write(const float* z, uint4* img, float sc, int tid) {      // at least 8*IMG threads
    if (tid >= 8 * IMG) return;
    const int e = tid % 8, r = tid / 8 % 4, q = tid / 32 % 4, ks = tid / 128;
    float left = sc * z[ks / K::DK * K::HALF + q * K::FL + 8 * (ks % K::DK) + e], piece = 0.f;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      piece = i <= r ? (float)(_Float16)left : piece;
      left = (left - piece) * 0x1p12f;
    }
    reinterpret_cast<_Float16*>(img)[tid] = (_Float16)piece;
  }
  static __device__ __forceinline__ uint4 operand(const uint4* img, int ks, unsigned lane) { return img[16 * ks + 4 * (lane / 16) + lane % 4]; }
  static __device__ __forceinline__ float sum(const f32x4& s) { return fmaf(fmaf(fmaf(s[3], 0x1p-12f, s[2]), 0x1p-12f, s[1]), 0x1p-12f, s[0]); }
};

// ---- query side --------------------------------------------------------------------------
// LDS operands of the token wavefronts' MFMA phases are requested QAHEAD MFMAs before their use.
constexpr int QAHEAD = 4;
constexpr int NTQ = 768;     // 12 wavefronts, one workgroup per compute unit
// Whether a tile's q rows, which dW~ contracts, have a place of their own in LDS.  Else (width 128, whose images and tiles fill it) they take phi's when dS
// has read it, with one more barrier to a tile.
template <int D>
constexpr bool kOwnX = D == 64;
// BLEND: dout is the gradient of the mixed output of Eq. 6; the linear branch receives (1 - r') dout.  DR: dL/dr = sum dout . (s - o) is
// asked for, and the workgroup's part goes to dr_part: the token wavefronts have dout . (o - vbar) as their delta, and the accumulate
// wavefronts, which wait for phi in the first half of a tile, read s and dout for dout . (s - vbar).  That sum as a streaming kernel of
// its own read dout once more and took 36 us (12 heads x 32760 x 128); here it costs 13 to 20.  An instance of its
// own: as a condition at run time its registers were spilled in blended calls without dL/dr too (centred, width 128, with dW~: 10, no other instance any).
// DW: dW~_q is accumulated here as well (DwTile).
//
// Wavefronts 0-7 ("tok") each own 16 tokens of a 128-token tile: phi, G = dO S^T, delta, du, dq.  o = phi S is not needed: with
// A+- = sum G phi and Z+- = sum z phi over the two halves of the features, den = Z+ + Z-, delta = (A+ + A-) / den and the two sums
// of the softmax Jacobian are combinations of the same four, so dots of what the lane holds in fp32 stand in for 40 of the
// MFMAs and for a second image of S.  Wavefronts 8-11 ("acc") contract the tile's phi, dO and delta into dS, dz
// and its x, du into dW~ meanwhile.  The tiles are single (64 KB of images leave room for
// one phi, dO and du tile).  A tile: phi, G and the sums; phi and dO are parked between two barriers and dS contracts them
// while du and dx are formed; (DW) x takes phi's place and du its tile between two more, and dW~ contracts those beside the next
// tile's first half.
// What bounds it is the issue of vector and matrix instructions, which overlap little: a SIMD has two tok wavefronts (750 vector instructions and 68
// MFMAs a tile each) and one acc (300 and 48), 11 of the tile's 14 thousand cycles.  Four tok wavefronts of 32 tokens, one to a SIMD, left a third of the
// issue slots empty and had 1700 instructions a tile: 111 us, now 96 (12 heads x 32760 x 128 with dW~), 41 / 34 (centred, 12 x 8190), 114 / 108 to 117 with
// dL/dr.  For a 16-token form to gain, nothing may be spilled: nine spilled addresses of the acc wavefronts, a scratch access to a k-step, took back all of it.
template <int D, bool STREAM, bool BLEND, bool DR, bool CENTRE, bool DW>
__global__ __launch_bounds__(NTQ) void bwd_q_kernel(const uint16_t* __restrict__ q, const uint16_t* __restrict__ dout,
                                                    const uint16_t* __restrict__ wq, const float* __restrict__ state,
                                                    float* __restrict__ vbar, uint16_t* __restrict__ dq,
                                                    float* __restrict__ partials, float* __restrict__ dw_part,
                                                    const uint16_t* __restrict__ blend, const float* __restrict__ rptr,
                                                    float* __restrict__ dr_part, float* __restrict__ cs_part,
                                                    int H, int n, int P, Rows rw) {
  using C = Cfg<D>;
  using K = Tok16<D>;
  constexpr int RS = D * 2;
  constexpr int WMN = D / 64;
  constexpr int NTOK = kTile / 16;                         // token wavefronts
  constexpr float mean = CENTRE ? 2.0f / D : 0.f;          // what is taken out of phi before it is rounded: its mean over the features
  using DWT = DwTile<D, 4>;
  extern __shared__ uint4 smem[];
  uint4* sWA = smem;
  uint4* sGA = sWA + K::W_IMG;
  uint4* sWB = sGA + K::G_IMG;
  uint4* sZP = sWB + K::T_IMG;                             // z in fp16 pieces (ZPieces)
  char* sPhi = reinterpret_cast<char*>(sZP + ZPieces<D>::IMG);      // [kTile][D] fp16: kPhiUnit f phi(q) (CENTRE: phi(q) - 2/D), then (DW) the q rows
  char* sDO = sPhi + kTile * RS;                           // [kTile][D] fp16: y stok dO
  float* sW = reinterpret_cast<float*>(sDO + kTile * RS);  // [kTile] -y stok delta
  float* sF = sW + kTile;                                  // [kTile] f (CENTRE)
  float* sVb = sF + kTile;                                 // [D] vbar (DR)
  float* sZ = sVb + D;                                     // [D] z, unscaled
  float* sRed = sZ + D;                                    // [16]: 0..7 the tile's operand maxima, 8..15 the du blocks' inverse scales
  char* sDU = reinterpret_cast<char*>(sRed + 16);          // DW: the tile's du, [kTile][D/2] fp16
  char* sX = kOwnX<D> ? sDU + DWT::DU_BYTES : sPhi;        // DW: its q rows

  const int tid = threadIdx.x, lane = tid % 64;
  const int w = __builtin_amdgcn_readfirstlane(tid / 64);
  const int bh = blockIdx.y, p = blockIdx.x, h = bh % H;
  const float om = BLEND ? 1.f - fminf(fmaxf(*rptr, 0.f), 1.f) : 1.f;      // 1 - r'
  const float* sb = state + (size_t)bh * (D + 1) * D;
  const int ntile = (n + kTile - 1) / kTile;
  float dr_acc = 0.f;

  // Everything the prologue reads is requested before any of it is waited for.  (The first rows as well: registers of the acc wavefronts are spilled.)
  float scale;
  {
    StateRegs<D, NTQ> S;
    WImages16<D, NTQ> W;
    S.load(sb, tid);
    const float z = sb[D * D + (tid < D ? tid : 0)];
    W.load(wq + (size_t)h * D * C::HALF, tid);
    __builtin_amdgcn_sched_barrier(0);
    W.write(sWA, sWB, tid);
    scale = build_query_state<D, NTQ>(S, z, sGA, sZ, reinterpret_cast<float*>(sPhi), p == 0 ? vbar + (size_t)bh * D : nullptr, tid);
  }
  if (DR && tid < D) sVb[tid] = reinterpret_cast<const float*>(sPhi)[D / 8 * D + tid];
  const float zs = ZPieces<D>::scale(n);
  ZPieces<D>::write(sZ, sZP, zs, tid);
  __syncthreads();

  // running power-of-two scale of the sums over tokens, the same in every wavefront; returns the factor for the accumulators
  float gamma = kGammaUnset;
  auto next_gamma = [&]() -> float {
    float m = sRed[0];
#pragma unroll
    for (int i = 1; i < NTOK; ++i) m = fmaxf(m, sRed[i]);
    float gnext = gamma;
    const float ratio = gamma_step(gnext, gamma_for(m));
    // the same in every lane: kept in scalar registers
    gamma = __builtin_bit_cast(float, __builtin_amdgcn_readfirstlane(__builtin_bit_cast(int, gnext)));
    return __builtin_bit_cast(float, __builtin_amdgcn_readfirstlane(__builtin_bit_cast(int, ratio)));
  };

  if (w < NTOK) {
    const int ql = lane / 16;
    uint16_t* dqb = dq + head_base(rw, bh, H);
    uint4 xq[K::KS], xr[K::KS], dor[K::KS];
    const float zero = opaque_zero_scalar();
    const float unit_z = uniform(__builtin_amdgcn_rcpf(kPhiUnit * zs));      // exact
    const LoadRows16<D> qrows(q + head_base(rw, bh, H), rw.sn, n, lane), drows(dout + head_base(rw, bh, H), rw.sn, n, lane);
    qrows.load(xq, p * kTile + 16 * w);
    uint4 zop[2 * K::DK];
#pragma unroll
    for (int ks = 0; ks < 2 * K::DK; ++ks) zop[ks] = ZPieces<D>::operand(sZP, ks, lane);
    float z_mean = 0.f;                                  // mean * the sum of z
    if constexpr (CENTRE) {
      for (int j = 0; j < D / 64; ++j) z_mean += sZ[64 * j + lane];
      z_mean = uniform(mean * quad<SumOp>(row_sum(z_mean)));
    }
    // the first rows have arrived before the loop: with them still out, the compiler's wait at the top of a tile, which has to hold
    // for the first tile too, would be a wait for the previous tile's stores
    qrows.arrived(xq);
    for (int tile = p; tile < ntile; tile += P) {
      const int t0 = tile * kTile + 16 * w;
      const bool valid = t0 + lane % 16 < n;
      drows.load(dor, t0);
      f32x4 u[K::UB];
      project16<D, QAHEAD>(xq, sWA, lane, u);
      if constexpr (DW) {
#pragma unroll
        for (int ks = 0; ks < K::KS; ++ks) xr[ks] = xq[ks];
      }
      float ep[K::FL], em[K::FL], ip, im;
      softmax16<D>(u, ep, em, ip, im);
      __builtin_amdgcn_sched_barrier(0);                   // (nothing waits for dO any earlier)
      // dO scaled by a power of two that brings the token's largest magnitude into [kTokenUnit, 2 kTokenUnit): exact in fp16 down to 2^-27 of that.  (The largest of those that
      // are finite: an infinity or NaN then stays in its own channel of dS.)
      float dmax, stok;
      uint4 bq[K::KS];
      {
        FiniteMax16 most;
#pragma unroll
        for (int ks = 0; ks < K::KS; ++ks) most.take(dor[ks]);
        dmax = quad<MagOp>(most.value());
        // (times 1, 1.25, 1.5 or 1.75, eight bits times three: still exact.  The weight that goes into phi is divided by it, so that tokens whose queries are
        // alike round in four ways)
        stok = pow2_normaliser(fminf(dmax, kTokenMax)) * fmaf((float)(((uint32_t)(t0 + lane % 16) * 0x165667b1u) >> 30), 0.25f * kTokenUnit, kTokenUnit);
#pragma unroll
        for (int ks = 0; ks < K::KS; ++ks) {
          float f[8];
          unpack_bf16x8(dor[ks], f);
          bq[ks] = make_uint4(mul_pack_f16x2(f[0], f[1], stok, zero), mul_pack_f16x2(f[2], f[3], stok, zero),
                              mul_pack_f16x2(f[4], f[5], stok, zero), mul_pack_f16x2(f[6], f[7], stok, zero));
        }
      }
      const float istok = __builtin_amdgcn_rcpf(stok);

      // G = dO S^T (times scale * stok), rows laid out like phi
      f32x4 ga[K::GB];
#pragma unroll
      for (int mb = 0; mb < K::GB; ++mb) ga[mb] = f32x4{0.f, 0.f, 0.f, 0.f};
      const int gl = grad16_lane<D>(opaque_lane(lane));
      pipelined_operands<K::KS * K::GB, QAHEAD>([&](int i) { return sGA[i * 64 + (gl ^ (4 * (i / K::GB)))]; },
                                                [&](int i, uint4 a) { ga[i % K::GB] = mfma_f16_16(a, bq[i / K::GB], ga[i % K::GB]); });
      // (dO stays packed until it is parked)
#pragma unroll
      for (int ks = 0; ks < K::KS; ++ks) asm volatile("" : "+v"(bq[ks].x), "+v"(bq[ks].y), "+v"(bq[ks].z), "+v"(bq[ks].w));
      // A+-, Z+-; feature ql*FL + j of each half
      const int z_at = ql * K::FL / 4 + opaque_zero();
      auto z4 = [&](int i) { return reinterpret_cast<const float4*>(sZ)[z_at + i]; };
      float ap = 0.f, am = 0.f, Zp = 0.f, Zm = 0.f;
#pragma unroll
      for (int i4 = 0; i4 < K::FL / 4; ++i4) {
        const float4 vp = z4(i4), vm = z4(C::HALF / 4 + i4);
        const float zp[4] = {vp.x, vp.y, vp.z, vp.w}, zm[4] = {vm.x, vm.y, vm.z, vm.w};
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int j = 4 * i4 + i;
          ap = fmaf(ga[i4][i], ep[j], ap); am = fmaf(ga[K::GB / 2 + i4][i], em[j], am);
          Zp = fmaf(zp[i], ep[j], Zp); Zm = fmaf(zm[i], em[j], Zm);
        }
      }
      ap *= ip; am *= im; Zp *= ip; Zm *= im;
      float own = ap + am;                                 // this lane's share
      quad4<SumOp>(ap, am, Zp, Zm);
      const float inv_den = __builtin_amdgcn_rcpf(Zp + Zm);
      // 1 / (scale * stok * den), in an order that keeps in range what is; scale is a power of two
      const float r0 = inv_den * __builtin_amdgcn_rcpf(scale) * istok;
      if constexpr (DR) {
        // the -dout . o part of dout . (s - o), this lane's share; the images are centred, so o here is
        // o - vbar: the other part of the sum is taken as dout . (s - vbar) to match
        if (valid) dr_acc -= own * r0;
      }
      const float delta = (ap + am) * r0;
      {
        // the tile's largest |dO_i| / den_i
        const float m = row_max_mag(fmaxf(valid ? dmax * inv_den * om : 0.f, 0.f));
        if (lane == 0) sRed[w] = m;
      }
      __syncthreads();                                   // the previous tile has been read
      next_gamma();
      {
        // (addresses from a lane index that the optimiser cannot hoist: held across the loop they end up in scratch memory)
        const unsigned lz = opaque_lane(lane);
        const int row = 16 * w + lz % 16, psw = swz<D>(lz % 16), qz = lz / 16;
        char* rowp = sPhi + row * RS;
        // The weight of the token, (1 - r') / den times the running scale, goes into phi, which is rounded anyway, and dO enters exactly.  (With the weight in
        // dO both operands are rounded, twice the variance of dS.)  A token whose dO vanishes or flushes in fp16 has none.
        const float wt = dmax < 0x1p-100f ? 0.f : inv_den * om * gamma * istok;
        auto park_phi = [&](float f) {                   // the packed features; returns their sum over z / f
          // CENTRE: phi minus its mean over the features, rounded after the subtraction: the fp16 rounding then acts
          // on the deviation from the uniform map; (2/D) x the column sums are added back on the key side
          const float fu = kPhiUnit * f, up = fu * ip, um = fu * im, c0 = CENTRE ? -mean * fu : zero;
          auto pack8 = [&](const float* e, float m) {
            return make_uint4(mul_pack_f16x2(e[0], e[1], m, c0), mul_pack_f16x2(e[2], e[3], m, c0), mul_pack_f16x2(e[4], e[5], m, c0),
                              mul_pack_f16x2(e[6], e[7], m, c0));
          };
          f32x4 zr = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
          for (int c = 0; c < K::DK; ++c) {
            const uint4 a = pack8(ep + 8 * c, up), b = pack8(em + 8 * c, um);
            *reinterpret_cast<uint4*>(rowp + (((qz * K::DK + c) ^ psw) * 16)) = a;
            *reinterpret_cast<uint4*>(rowp + (((C::CH / 2 + qz * K::DK + c) ^ psw) * 16)) = b;
            zr = mfma_f16_16(zop[c], a, zr);
            zr = mfma_f16_16(zop[K::DK + c], b, zr);
          }
          return fmaf(ZPieces<D>::sum(zr), unit_z, f * z_mean);
        };
        char* drowp = sDO + row * RS;
#pragma unroll
        for (int ks = 0; ks < K::KS; ++ks) *reinterpret_cast<uint4*>(drowp + (((4 * ks + qz) ^ psw) * 16)) = bq[ks];
        float y = 1.f, f = wt;
        const float den = Zp + Zm, all = wt * den;
        const bool off = fabsf(park_phi(wt) - all) > kSharedRounding * all;
        if (__any(off)) {
          // What the roundings of a token's features have in common does not average out over tokens whose queries are alike.  Where it is large, phi is
          // rounded without the weight, and the weight, in dO, has the normaliser of phi as it was rounded.  (One that is off by a factor of two is of a token
          // whose features with a key behind them round to next to nothing.)
          f = off ? 1.f : wt;
          const float den_r = park_phi(f);
          if (off) y = wt * (den_r > 0.5f * den && den_r < 2.f * den ? den * __builtin_amdgcn_rcpf(den_r) : 1.f);
#pragma unroll
          for (int ks = 0; ks < K::KS; ++ks)
            *reinterpret_cast<uint4*>(drowp + (((4 * ks + qz) ^ psw) * 16)) =
                make_uint4(mul_pack_f16x2(bq[ks].x, y, zero), mul_pack_f16x2(bq[ks].y, y, zero), mul_pack_f16x2(bq[ks].z, y, zero),
                           mul_pack_f16x2(bq[ks].w, y, zero));
        }
        if (lane < 16) {
          sW[row] = -delta * stok * y;
          if constexpr (CENTRE) sF[row] = f;
        }
      }
      __syncthreads();
      // g = (1 - r') (G - delta z) / den, its sums cp, cm against phi, and du
      const float r1 = om * r0, r2 = om * inv_den * delta;
      const float cp = ap * r1 - r2 * Zp, cm = am * r1 - r2 * Zm;
      const float r1p = r1 * ip, r2p = r2 * ip, cpp = cp * ip, r1m = r1 * im, r2m = r2 * im, cmm = cm * im;
      float du[K::FL];
#pragma unroll
      for (int i4 = 0; i4 < K::FL / 4; ++i4) {
        const float4 vp = z4(i4), vm = z4(C::HALF / 4 + i4);
        const float zp[4] = {vp.x, vp.y, vp.z, vp.w}, zm[4] = {vm.x, vm.y, vm.z, vm.w};
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int j = 4 * i4 + i;
          const float gp = fmaf(ga[i4][i], r1p, fmaf(-r2p, zp[i], -cpp));
          const float gm = fmaf(ga[K::GB / 2 + i4][i], r1m, fmaf(-r2m, zm[i], -cmm));
          du[j] = ep[j] * gp - em[j] * gm;
        }
      }
      // The next tile's rows go out before the dq stores: loads and stores retire in order, and a wait for a load issued behind
      // the stores would wait for the stores as well.
      qrows.load(xq, t0 + P * kTile);
      uint32_t dub[K::FL / 2];
      float blk_its;
      {
        f32x4 xa[K::MB];
        float its;
        du_to_dx16<D, QAHEAD>(du, sWB, lane, valid, zero, xa, its, dub, blk_its);
        const float none[K::MB] = {};
        store_token_rows16<D, STREAM, false>(dqb, rw.sn, t0, n, lane, xa, its, none);
      }
      if constexpr (DW) {
        if constexpr (!kOwnX<D>) __syncthreads();        // dS has read the tile's phi
        park_dw16<D>(xr, dub, blk_its, sX, sDU, sRed + 8, w, lane);
        __syncthreads();
      }
    }
  } else {
    float csum[WMN], wsum = 0.f;                         // column sums of the dO/den operand, sum of the -delta/den operand
#pragma unroll
    for (int j = 0; j < WMN; ++j) csum[j] = 0.f;
    f32x16 s[WMN][WMN];
    float zacc = 0.f;
#pragma unroll
    for (int r = 0; r < 16; ++r)
#pragma unroll
      for (int i = 0; i < WMN; ++i)
#pragma unroll
        for (int j = 0; j < WMN; ++j) s[i][j][r] = 0.f;
    const int pw = w - NTOK, g = lane / 32;
    const Quadrant<D> qd(pw);
    DWT dwt;
    if constexpr (DW) dwt.init(pw);
    // DR: the thread's chunk column of s and dout
    constexpr int PER = kTile * C::CH / 256;
    const int crow = (tid - 64 * NTOK) / C::CH, ccol = (tid - 64 * NTOK) % C::CH;
    for (int tile = p; tile < ntile; tile += P) {
      // (blend is never null here: as a branch the section keeps its registers to itself; without one, 97 are spilled with CENTRE and DW where 3
      // are, and 75 with DW alone where none is)
      if (DR && blend != nullptr) {
        const uint16_t* srow = blend + head_base(rw, bh, H) + 8 * ccol;
        const uint16_t* drow = dout + head_base(rw, bh, H) + 8 * ccol;
        // (width 128: two batches, all at once they are spilled)
        constexpr int BATCH = D == 128 ? PER / 2 : PER;
#pragma unroll
        for (int i0 = 0; i0 < PER; i0 += BATCH) {
          uint4 sv[BATCH], dv[BATCH];
#pragma unroll
          for (int i = 0; i < BATCH; ++i) {
            const int t = tile * kTile + crow + (i0 + i) * (256 / C::CH);
            const size_t at = (size_t)(t < n ? t : n - 1) * rw.sn;
            sv[i] = ld_nt(reinterpret_cast<const uint4*>(srow + at));
            dv[i] = *reinterpret_cast<const uint4*>(drow + at);
          }
#pragma unroll
          for (int i = 0; i < BATCH; ++i) {
            const float4 v0 = reinterpret_cast<const float4*>(sVb)[2 * ccol], v1 = reinterpret_cast<const float4*>(sVb)[2 * ccol + 1];
            const float vb[8] = {v0.x, v0.y, v0.z, v0.w, v1.x, v1.y, v1.z, v1.w};
            float a[8], b[8], t = 0.f;
            unpack_bf16x8(sv[i], a);
            unpack_bf16x8(dv[i], b);
#pragma unroll
            for (int e = 0; e < 8; ++e) t = fmaf(b[e], a[e] - vb[e], t);
            if (tile * kTile + crow + (i0 + i) * (256 / C::CH) < n) dr_acc += t;
          }
          __builtin_amdgcn_sched_barrier(0);
        }
      }
      __syncthreads();
      const float ratio = next_gamma();
      if (ratio != 1.f) {                                // this tile is larger than every earlier one
        if constexpr (CENTRE) {
          wsum *= ratio;
#pragma unroll
          for (int j = 0; j < WMN; ++j) csum[j] *= ratio;
        }
        zacc *= ratio;
#pragma unroll
        for (int r = 0; r < 16; ++r)
#pragma unroll
          for (int i = 0; i < WMN; ++i)
#pragma unroll
            for (int j = 0; j < WMN; ++j) s[i][j][r] *= ratio;
      }
      // (worked out per tile: held across the loop these addresses end up in scratch memory, and every k-step waits for one)
      const int lz = opaque_lane(lane);
      const QuadrantReads<D> rd(qd, sPhi, sDO, lz);
      __syncthreads();
      contract_tokens<D, CENTRE>(rd, s, zacc, sW + 8 * (lz / 32), sF + 8 * (lz / 32), csum, wsum);
      if constexpr (DW) {
        if constexpr (!kOwnX<D>) __syncthreads();
        __syncthreads();
        dwt.contract(sX, sDU, sRed + 8, opaque_lane(lane));
      }
    }
    if constexpr (DW) dwt.store(dw_part + ((size_t)bh * P + p) * (size_t)D * C::HALF, lane);

    const float ig = __builtin_amdgcn_rcpf(gamma), ip = ig * (1.f / kPhiUnit);      // exact: gamma is a power of two
    if constexpr (CENTRE) {
      // column sums of dO/den (the wavefronts qd.mi = 0 hold every channel block once) and the sum of -delta/den
      float* cs = cs_part + ((size_t)bh * P + p) * (D + 8);
#pragma unroll
      for (int j = 0; j < WMN; ++j) {
        float lo, hi;
        pair32(csum[j], lo, hi);
        if (qd.mi == 0 && g == 0) cs[32 * qd.cblk(j) + (lane % 32)] = (lo + hi) * ig;
      }
      float lo, hi;
      pair32(wsum, lo, hi);
      if (pw == 0 && lane == 0) cs[D] = (lo + hi) * ig;
    }
    float* dst = partials + ((size_t)bh * P + p) * (size_t)(D + 1) * D;
    const int c = lane % 32;
#pragma unroll
    for (int i = 0; i < WMN; ++i)
#pragma unroll
      for (int j = 0; j < WMN; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int f = 32 * qd.fblk(i) + 8 * (r / 4) + 4 * g + (r % 4);
          dst[f * D + 32 * qd.cblk(j) + c] = s[i][j][r] * ip;
        }
    {
      float lo, hi;
      pair32(zacc, lo, hi);
      if (qd.do_z() && g == 0) dst[D * D + 32 * qd.zblk() + c] = (lo + hi) * ip;
    }
  }
  if constexpr (DR) {
    for (int k = 32; k >= 1; k >>= 1) dr_acc += __shfl_xor(dr_acc, k, 64);
    __syncthreads();                                       // the last tile's slots have been read
    if (lane == 0) sRed[w] = dr_acc;
    __syncthreads();
    if (tid == 0)
      dr_part[(size_t)bh * P + p] = (((sRed[0] + sRed[1]) + (sRed[2] + sRed[3])) + ((sRed[4] + sRed[5]) + (sRed[6] + sRed[7])))
                                    + ((sRed[8] + sRed[9]) + (sRed[10] + sRed[11]));
  }
}

// ---- key side ----------------------------------------------------------------------------
// LDS operands of the MFMA phases are requested KAHEAD MFMAs before their use.
constexpr int KAHEAD = 3;
// One workgroup per compute unit: with dW~ 12 wavefronts, without 8, whose prologue is shorter and whose rows arrive no later: 12 / 8 wavefronts, us, 4 heads x
// 1000 x 128 11.7 / 9.9, 12 x 2000 13.3 / 11.8, 12 x 4133 20.8 / 18.3, 12 x 16000 40.7 / 40.2, 24 x 20000 x 64 47.4 / 46.2 (8 of 32 tokens: 47.2).
template <bool DW>
constexpr int kKeyThreads = DW ? 768 : 512;

// Every wavefront takes blocks of 16 tokens.  DW: dW~_k is accumulated here as well (DwTile): wavefronts 0-7 walk 128-token tiles in step and park their
// k rows (kept in registers: read again at the end of a block they came from beyond the L2, whose 4 MB a round of 32 compute
// units passes) and du, and wavefronts 8-11 contract those over the tokens while the next tile is under way.
// STREAM: dv is stored non-temporally, as dk always is (stream_gradients).
// Eight wavefronts of 32 tokens, two to a SIMD, filled 40 % of its vector issue: 107 us, now 87 (12 heads x 32760 x 128 with dW~; 403 MB of rows, 4.6
// TB/s), in [B,n,H,d] 118 / 90, centred 12 x 8190 36 / 31, 12 x 1000 16.1 / 13.5.
template <int D, bool STREAM, bool CENTRE, bool DW>
__global__ __launch_bounds__(kKeyThreads<DW>) void bwd_k_kernel(const uint16_t* __restrict__ k, const uint16_t* __restrict__ v,
                                                    const uint16_t* __restrict__ wk, const float* __restrict__ dstate,
                                                    uint16_t* __restrict__ dk, uint16_t* __restrict__ dv,
                                                    float* __restrict__ dw_part,
                                                    const float* __restrict__ vbar, const float* __restrict__ cs_part,
                                                    int H, int n, int P, Rows rw) {
  using K = Tok16<D>;
  constexpr int NTK = kKeyThreads<DW>, NW = NTK / 64, NTOK = DW ? kTile / 16 : NW;
  using DWT = DwTile<D, NW - kTile / 16>;
  extern __shared__ uint4 smem[];
  uint4* sWA = smem;
  uint4* sVA = sWA + K::W_IMG;             // image of dS for dv (contraction over features)
  uint4* sGA = sVA + K::A_IMG;             // image of dS for g (contraction over channels)
  uint4* sWB = sGA + K::G_IMG;
  float* sZ = reinterpret_cast<float*>(sWB + K::T_IMG); // [D] dz, unscaled
  float* sIts = sZ + D;                                 // [8]: DW: the parked du blocks' inverse scales
  float* sRow = sIts + 8;                               // [D] constant row of dv, then the scratch of the prologue
  char* sX = reinterpret_cast<char*>(sRow + D);         // DW: [kTile][D] fp16, a tile's k rows
  char* sU = sX + kTile * D * 2;                        // DW: [kTile][D/2] fp16, their du

  const int tid = threadIdx.x, lane = tid % 64;
  const int w = __builtin_amdgcn_readfirstlane(tid / 64);
  const int bh = blockIdx.y, h = bh % H;
  const uint16_t* wkh = wk + (size_t)h * D * K::HALF;

  const int step = 16 * NTOK * gridDim.x;
  int t0 = 16 * (blockIdx.x * NTOK + w);
  // Everything the prologue reads, and the first rows, is requested before any of it is waited for: one memory latency instead of three (with the
  // exchanges of the reductions as DPP steps and swaps, not through LDS: 12 x 1000 x 64 9.7 -> 6.6 us, 12 x 4133 x 64 11.3 -> 10.1).
  const LoadRows16<D> krows(k + head_base(rw, bh, H), rw.sn, n, lane);
  uint4 xk[K::KS];
  float scale;
  {
    StateRegs<D, NTK> S;
    WImages16<D, NTK> W;
    const float* ds = dstate + (size_t)bh * (D + 1) * D;
    S.load(ds, tid);
    const int own = tid < D ? tid : 0;
    const float dz = ds[D * D + own], vb_own = vbar[(size_t)bh * D + own];
    W.load(wkh, tid);
    krows.load(xk, w < NTOK ? t0 : n);
    __builtin_amdgcn_sched_barrier(0);
    W.write(sWA, sWB, tid);
    // sZ: dz matched to the rounded image of dS (and, with LINATTN_FLAG_CENTRED, to its centring over the features)
    scale = build_key_state<D, NTK, CENTRE>(S, dz, vb_own, sVA, sGA, sZ, sRow, sRow + D, CENTRE ? cs_part + (size_t)bh * P * (D + 8) : nullptr, P, tid);
  }
  __syncthreads();

  if (w < NTOK) {
    const float inv_scale = __builtin_amdgcn_rcpf(scale);    // exact: power of two
    const int ql = lane / 16;
    uint16_t* dkb = dk + head_base(rw, bh, H);
    uint16_t* dvb = dv + head_base(rw, bh, H);
    const float zero = opaque_zero_scalar();
    const LoadRows16<D> vrows(v + head_base(rw, bh, H), rw.sn, n, lane);
    float dv_add[K::MB];
#pragma unroll
    for (int mb = 0; mb < K::MB; ++mb) dv_add[mb] = CENTRE ? sRow[K::MB * (lane % 16) + mb] : 0.f;
    uint4 xr[K::KS], vr[K::KS];
    // DW: every token wavefront makes the same number of rounds (there are barriers inside); one whose block does not exist works on zeros
    for (; (DW ? t0 - 16 * w : t0) < n; t0 += step) {
      const bool valid = t0 + lane % 16 < n;
      vrows.load(vr, t0);                               // wanted after the projection, the softmax and dv
      f32x4 u[K::UB];
      project16<D, KAHEAD>(xk, sWA, lane, u);
      if constexpr (DW) {
#pragma unroll
        for (int ks = 0; ks < K::KS; ++ks) xr[ks] = xk[ks];
      } else {
        krows.load(xk, t0 + step);                      // the next block's k flies during this one
      }
      float ep[K::FL], em[K::FL], ip, im;
      softmax16<D>(u, ep, em, ip, im);

      // dv = phi(k) dS, tokens on the accumulator rows
      {
        uint32_t pk[K::FL];
#pragma unroll
        for (int j = 0; j < K::FL / 2; ++j) {
          pk[j] = mul_pack_f16x2(ep[2 * j], ep[2 * j + 1], ip, zero);
          pk[K::FL / 2 + j] = mul_pack_f16x2(em[2 * j], em[2 * j + 1], im, zero);
        }
        f32x4 va[K::MB];
#pragma unroll
        for (int mb = 0; mb < K::MB; ++mb) va[mb] = f32x4{0.f, 0.f, 0.f, 0.f};
        const uint4* sva = sVA + lane + opaque_zero();
        pipelined_operands<2 * K::DK * K::MB, KAHEAD>(
            [&](int i) { return sva[i * 64]; },
            [&](int i, uint4 b) {
              const uint32_t* a = pk + 4 * (i / K::MB);
              va[i % K::MB] = mfma_f16_16(make_uint4(a[0], a[1], a[2], a[3]), b, va[i % K::MB]);
            });
        store_token_rows16<D, STREAM, CENTRE>(dvb, rw.sn, t0, n, lane, va, inv_scale, dv_add);
      }

      // g = v dS^T + dz, rows laid out like phi, and its sums against phi
      float gp[K::FL], gm[K::FL], cp = 0.f, cm = 0.f;
      {
        uint4 bq[K::KS];
#pragma unroll
        for (int ks = 0; ks < K::KS; ++ks)
          bq[ks] = make_uint4(bf16x2_to_f16x2(vr[ks].x), bf16x2_to_f16x2(vr[ks].y), bf16x2_to_f16x2(vr[ks].z), bf16x2_to_f16x2(vr[ks].w));
        f32x4 ga[K::GB];
#pragma unroll
        for (int mb = 0; mb < K::GB; ++mb) ga[mb] = f32x4{0.f, 0.f, 0.f, 0.f};
        const int gl = grad16_lane<D>(opaque_lane(lane));
        pipelined_operands<K::KS * K::GB, KAHEAD>([&](int i) { return sGA[i * 64 + (gl ^ (4 * (i / K::GB)))]; },
                                                  [&](int i, uint4 a) { ga[i % K::GB] = mfma_f16_16(a, bq[i / K::GB], ga[i % K::GB]); });
        const int z_at = ql * K::FL / 4 + opaque_zero();
#pragma unroll
        for (int i4 = 0; i4 < K::FL / 4; ++i4) {
          const float4 vp = reinterpret_cast<const float4*>(sZ)[z_at + i4], vm = reinterpret_cast<const float4*>(sZ)[z_at + K::HALF / 4 + i4];
          const float zp[4] = {vp.x, vp.y, vp.z, vp.w}, zm[4] = {vm.x, vm.y, vm.z, vm.w};
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const int j = 4 * i4 + i;
            gp[j] = fmaf(ga[i4][i], inv_scale, zp[i]);
            gm[j] = fmaf(ga[K::GB / 2 + i4][i], inv_scale, zm[i]);
            cp = fmaf(gp[j], ep[j], cp); cm = fmaf(gm[j], em[j], cm);
          }
        }
      }
      quad2<SumOp>(cp, cm);
      cp *= ip * ip; cm *= im * im;
      float du[K::FL];
#pragma unroll
      for (int j = 0; j < K::FL; ++j) du[j] = ep[j] * fmaf(gp[j], ip, -cp) - em[j] * fmaf(gm[j], im, -cm);
      uint32_t dub[K::FL / 2];
      float blk_its;
      {
        f32x4 xa[K::MB];
        float its;
        du_to_dx16<D, KAHEAD>(du, sWB, lane, valid, zero, xa, its, dub, blk_its);
        // DW: the next block's k rows, before the dk stores: a wait for them must not wait for the stores
        if constexpr (DW) krows.load(xk, t0 + step);
        store_token_rows16<D, true, false>(dkb, rw.sn, t0, n, lane, xa, its, dv_add);
      }
      if constexpr (DW) {
        __syncthreads();                                // the tiles' previous readers are done
        park_dw16<D>(xr, dub, blk_its, sX, sU, sIts, w, lane);
        __syncthreads();
      }
    }
  } else if constexpr (DW) {
    DWT dwt;
    dwt.init(w - NTOK);
    for (t0 = 16 * NTOK * blockIdx.x; t0 < n; t0 += step) {
      __syncthreads();
      __syncthreads();
      dwt.contract(sX, sU, sIts, opaque_lane(lane));
    }
    dwt.store(dw_part + ((size_t)bh * gridDim.x + blockIdx.x) * (size_t)D * K::HALF, lane);
  }
}

template <int D, bool DW>
constexpr size_t q_smem() {
  return sizeof(uint4) * (Tok16<D>::W_IMG + Tok16<D>::G_IMG + Tok16<D>::T_IMG + ZPieces<D>::IMG)
       + 2 * (size_t)kTile * D * 2 + (2 * kTile + 2 * D + 16) * sizeof(float) + (DW ? DwTile<D, 4>::DU_BYTES + (kOwnX<D> ? (size_t)kTile * D * 2 : 0) : 0);
}
template <int D, bool DW>
constexpr size_t k_smem() {
  // the prologue's scratch lies where the DW tiles are afterwards
  constexpr size_t scratch = ((size_t)(D / 8) * D + 4 * D + kKeyThreads<DW> / 64 + 4) * sizeof(float);
  constexpr size_t tiles = DW ? (size_t)kTile * D * 2 + DwTile<D, 4>::DU_BYTES : 0;
  return sizeof(uint4) * (Tok16<D>::W_IMG + Tok16<D>::A_IMG + Tok16<D>::G_IMG + Tok16<D>::T_IMG) + (2 * D + 8) * sizeof(float)
       + (scratch > tiles ? scratch : tiles);
}
template <int D, bool CENTRE, bool STREAM>
hipError_t run_bwd_as(const BwdArgs& a, const Plan& p, hipStream_t s) {
  hipError_t e;
  // dW~ partials: [BH][P] blocks of the query side, then as many of the key side
  const size_t side_elems = (size_t)p.BH * p.P * D * (D / 2);
  auto launch_q = [&](auto kernel) -> hipError_t {
    const size_t smem = a.dwq ? q_smem<D, true>() : q_smem<D, false>();
    hipError_t e2 = set_smem_once<decltype(kernel)::value>(smem);
    if (e2 != hipSuccess) return e2;
    decltype(kernel)::value<<<dim3(p.P, p.BH), NTQ, smem, s>>>(
        (const uint16_t*)a.q, (const uint16_t*)a.dout, (const uint16_t*)a.wq, a.state, a.vbar, (uint16_t*)a.dq, a.partials, a.dw_part,
        (const uint16_t*)a.blend_in, a.blend_r, a.dr_part, a.cs_part, p.H, p.n, p.P, p.rows);
    return hipGetLastError();
  };
  if (a.blend_in && a.blend_dr)
    e = a.dwq ? launch_q(KernelTag<bwd_q_kernel<D, STREAM, true, true, CENTRE, true>>{}) : launch_q(KernelTag<bwd_q_kernel<D, STREAM, true, true, CENTRE, false>>{});
  else if (a.blend_in)
    e = a.dwq ? launch_q(KernelTag<bwd_q_kernel<D, STREAM, true, false, CENTRE, true>>{}) : launch_q(KernelTag<bwd_q_kernel<D, STREAM, true, false, CENTRE, false>>{});
  else
    e = a.dwq ? launch_q(KernelTag<bwd_q_kernel<D, STREAM, false, false, CENTRE, true>>{}) : launch_q(KernelTag<bwd_q_kernel<D, STREAM, false, false, CENTRE, false>>{});
  if (e != hipSuccess) return e;
  if ((e = launch_state_reduce(a.partials, a.dstate, p, DrSum{a.dr_part, p.BH * p.P, a.blend_r, a.blend_dr}, s)) != hipSuccess) return e;
  // with dW~_k a workgroup takes 128-token tiles, and the partials are laid out like the query side's; else 16 tokens a wavefront
  constexpr int UNIT = kKeyThreads<false> / 4;
  const int units = (p.n + UNIT - 1) / UNIT, per_head = p.BH < kCUs ? kCUs / p.BH : 1;
  const int groups = a.dwk ? p.P : units < per_head ? units : per_head;
  auto launch_k = [&](auto kernel, int threads, size_t smem) -> hipError_t {
    hipError_t e2 = set_smem_once<decltype(kernel)::value>(smem);
    if (e2 != hipSuccess) return e2;
    decltype(kernel)::value<<<dim3(groups, p.BH), threads, smem, s>>>(
        (const uint16_t*)a.k, (const uint16_t*)a.v, (const uint16_t*)a.wk, a.dstate, (uint16_t*)a.dk, (uint16_t*)a.dv,
        a.dw_part + side_elems, a.vbar, a.cs_part, p.H, p.n, p.P, p.rows);
    return hipGetLastError();
  };
  e = a.dwk ? launch_k(KernelTag<bwd_k_kernel<D, STREAM, CENTRE, true>>{}, kKeyThreads<true>, k_smem<D, true>()) :
      launch_k(KernelTag<bwd_k_kernel<D, STREAM, CENTRE, false>>{}, kKeyThreads<false>, k_smem<D, false>());
  if (e != hipSuccess) return e;
  if (a.dwq || a.dwk) {
    if ((e = launch_dw_reduce2(a.dwq ? a.dw_part : nullptr, a.dwq, p.P, a.dwk ? a.dw_part + side_elems : nullptr, a.dwk, groups, p, s)) != hipSuccess) return e;
  }
  return hipSuccess;
}
template <bool STREAM>
hipError_t run_bwd(const BwdArgs& a, const Plan& p, hipStream_t s) {
  if (p.centred) return p.d == 128 ? run_bwd_as<128, true, STREAM>(a, p, s) : run_bwd_as<64, true, STREAM>(a, p, s);
  return p.d == 128 ? run_bwd_as<128, false, STREAM>(a, p, s) : run_bwd_as<64, false, STREAM>(a, p, s);
}

}  // namespace

}  // namespace linattn
