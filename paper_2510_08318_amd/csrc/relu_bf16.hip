// ReLU feature map, bf16 I/O: phi(x) = max(x, 0) on the d channels of a head (the "ReLU" row of
// the paper's ablation of kernel functions), put into Eq. 3 with kReluEps in the denominator.
// This file holds the state pass and the backward; the query pass is apply_bf16_kernel<.., kPhiRelu>
// in fwd_bf16.hip.
//
// With no projection and no softmax the map costs a sign test, so every kernel here is the plain
// contraction of Eq. 3 (or of its chain rule) on MFMA with fp32 accumulation -- bf16 operands in
// the state pass (K and V as stored: exact products, no conversion), fp16 where a state or a
// gradient is an operand (the query pass and the backward):
//   relu_state_kernel  : S_p = sum_j phi(k_j)^T v_j, z_p = sum_j phi(k_j) over the tiles of a split
//   relu_bwd_q_kernel  : den, G = dO S^T, delta, dq; split-n partials of dS, dz
//   relu_bwd_k_kernel  : dv = phi(k) dS, dk = (v dS^T + dz) where k > 0
// Gradients (chain rule through Eq. 3, then the mask of max(x, 0), whose derivative at 0 is taken as 0):
//   den_i = phi(q_i).z + eps, o_i = phi(q_i) S / den_i, delta_i = dO_i . o_i
//   dphi(q_i) = (S dO_i - delta_i z) / den_i;  dS = sum_i phi(q_i)^T dO_i / den_i;  dz = -sum_i phi(q_i) delta_i / den_i
//   dphi(k_j) = dS v_j + dz;  dv_j = dS^T phi(k_j)
// Operands that are gradients are scaled by powers of two before the cast to fp16, as in bwd_bf16.h.
#include "kernels.h"
#include "mfma16.h"

namespace linattn {
namespace {

// ---- state pass -------------------------------------------------------------------------------
// 4 wavefronts.  One segment = the 128-token tiles tile0 .. tile0+nt-1 of one (b,h): K (through
// max(.,0)) and V are parked in LDS as they are, bf16 (no conversion: the kernel's time is its own
// instruction stream, not HBM), and contracted over the tokens with transposing reads on bf16 MFMA;
// wavefront (mi, ni) owns the feature rows 32*WMN*mi .. and the channel columns 32*WMN*ni .. of S.
// z = phi(K)^T 1 rides along as one more MFMA per k-step against an operand of ones.  Every thread
// of the workgroup calls it (it contains workgroup barriers).
template <int D>
__device__ __forceinline__ void relu_state_segment(const uint16_t* __restrict__ kb, const uint16_t* __restrict__ vb,
                                                   float* __restrict__ dst, int tile0, int nt, int n, Rows rw) {
  constexpr int RS = D * 2;
  constexpr int WMN = D / 64;
  constexpr int XPT = (kTile * (D / 8)) / NT;   // 16-byte chunks of a tile per thread
  extern __shared__ uint4 smem[];
  char* sK = reinterpret_cast<char*>(smem);      // [kTile][D] bf16, swizzled chunks
  char* sV = sK + kTile * RS;

  const int tid = threadIdx.x, lane = tid % 64;
  const int w = __builtin_amdgcn_readfirstlane(tid / 64);
  const int g = lane / 32;
  const Quadrant<D> qd(w);
  const int tile_end = tile0 + nt;

  f32x16 s[WMN][WMN], zacc;
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    zacc[r] = 0.f;
#pragma unroll
    for (int i = 0; i < WMN; ++i)
#pragma unroll
      for (int j = 0; j < WMN; ++j) s[i][j][r] = 0.f;
  }
  const QuadrantReads<D> rd(qd, sK, sV, lane);
  uint4 ones;
  ones.x = ones.y = ones.z = ones.w = 0x3F803F80u;      // bf16 1.0
  const f16x8 one_op = as_f16x8(ones);

  // Loads are branch-free (rows past n read row n-1 and are zeroed on their way into LDS; after the
  // last tile of a segment that tile is requested once more and ignored): a load behind a branch
  // makes the compiler wait for every outstanding load at the join.
  // Tiles kept in flight per workgroup, and how often the loop body repeats them.  Measured at the
  // Wan-14B 720p shape: one tile 287 us, two 276 us, three 295 us, four 290 us.  The compiler waits
  // for every outstanding load at the top of the loop, so only an unrolled body overlaps them.
  constexpr int DEPTH = 2, UNROLL = 2;
  uint4 kr[DEPTH][XPT], vr[DEPTH][XPT];
  // Addresses: a wavefront-uniform tile pointer (scalar registers) plus a 32-bit byte offset per
  // thread and piece that is computed once (15 vector instructions per load otherwise, a quarter
  // of this kernel's instruction stream).  Rows past n are redirected to row n-1 with one minimum
  // per load.
  static_assert(NT % (D / 8) == 0, "a thread keeps its chunk column");
  uint32_t voff[XPT];
#pragma unroll
  for (int i = 0; i < XPT; ++i)
    voff[i] = (uint32_t)(((tid + NT * i) / (D / 8)) * rw.sn + (tid % (D / 8)) * 8) * 2u;
  int loff[XPT];                                   // LDS byte offsets of the thread's pieces
#pragma unroll
  for (int i = 0; i < XPT; ++i) {
    const int r = (tid + NT * i) / (D / 8), c = tid % (D / 8);
    loff[i] = r * RS + ((c ^ swz<D>(r)) * 16);
  }
  auto load_tile = [&](uint4 (&kx)[XPT], uint4 (&vx)[XPT], int tile) {
    tile = tile < tile_end ? tile : tile_end - 1;
    const int t0 = tile * kTile;
    const char* kt = reinterpret_cast<const char*>(kb + (size_t)t0 * rw.sn);
    const char* vt = reinterpret_cast<const char*>(vb + (size_t)t0 * rw.sn);
    const int last = n - 1 - t0;                  // last row of the tile that exists (>= kTile-1: all do)
    const uint32_t last_off = (uint32_t)(last * rw.sn + (tid % (D / 8)) * 8) * 2u;
#pragma unroll
    for (int i = 0; i < XPT; ++i) {
      const uint32_t off = voff[i] < last_off ? voff[i] : last_off;      // same column: offsets grow with the row
      kx[i] = ld_nt(reinterpret_cast<const uint4*>(kt + off));
      vx[i] = ld_nt(reinterpret_cast<const uint4*>(vt + off));
    }
  };
  auto consume = [&](uint4 (&kx)[XPT], uint4 (&vx)[XPT], int tile, bool real) {
    __syncthreads();                              // previous tile's operand reads are done
    // the tiles stay bf16 (the products of a bf16 MFMA are exact): K through the sign test, V as it
    // is.  Rows that do not exist hold copies of row n-1: zeroing their K is enough (phi = 0 adds
    // nothing to S or z); only a head's last tile and padding steps pay for that.
    const bool full = real && (tile + 1) * kTile <= n;      // uniform
#pragma unroll
    for (int i = 0; i < XPT; ++i) {
      uint4 hk;
      hk.x = relu_bf16x2(kx[i].x); hk.y = relu_bf16x2(kx[i].y); hk.z = relu_bf16x2(kx[i].z); hk.w = relu_bf16x2(kx[i].w);
      if (!full) {
        const int r = (tid + NT * i) / (D / 8);
        if (!(real && tile * kTile + r < n)) hk = make_uint4(0, 0, 0, 0);
      }
      *reinterpret_cast<uint4*>(sK + loff[i]) = hk;
      *reinterpret_cast<uint4*>(sV + loff[i]) = vx[i];
    }
    load_tile(kx, vx, tile + DEPTH);
    __syncthreads();
    contract_tile<D, true>(rd, s, zacc, qd.do_z(), [&](int) { return one_op; });
  };
#pragma unroll
  for (int j = 0; j < DEPTH; ++j) load_tile(kr[j], vr[j], tile0 + j);
  for (int tile = tile0; tile < tile_end; tile += UNROLL * DEPTH) {
#pragma unroll
    for (int u = 0; u < UNROLL; ++u)
#pragma unroll
      for (int j = 0; j < DEPTH; ++j) {
        const int tl = tile + u * DEPTH + j;
        consume(kr[j], vr[j], tl, tl < tile_end);     // a padding step adds zeros
      }
  }
  const int c = lane % 32;
#pragma unroll
  for (int i = 0; i < WMN; ++i)
#pragma unroll
    for (int j = 0; j < WMN; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int f = 32 * qd.fblk(i) + 8 * (r / 4) + 4 * g + (r % 4);
        dst[f * D + 32 * qd.cblk(j) + c] = s[i][j][r];
      }
  if (qd.do_z() && c == 0) {
#pragma unroll
    for (int r = 0; r < 16; ++r) dst[D * D + 32 * qd.zblk() + 8 * (r / 4) + 4 * g + (r % 4)] = zacc[r];
  }
  __syncthreads();                               // the next segment reuses the LDS tiles
}

// Grid: Split::G workgroups; workgroup g takes the tiles [lo(g), lo(g+1)) of the call's (b,h)-major
// tile sequence, one segment per head it touches (at most two), so every compute unit gets the same
// share whatever B*H is.  Partials: [BH][Split::PS][(d+1)*d], summed by the split reduction.
template <int D>
__global__ __launch_bounds__(NT) void relu_state_kernel(const uint16_t* __restrict__ k, const uint16_t* __restrict__ v,
                                                        float* __restrict__ partials, int H, int n, Split sp, Rows rw) {
  const int gi = blockIdx.x;
  long long lo = split_lo(sp, gi);
  const long long hi = split_lo(sp, gi + 1);
  while (lo < hi) {
    const int bh = split_head(sp, lo);
    const long long head0 = (long long)bh * sp.ntile;
    const long long seg_hi = hi < head0 + sp.ntile ? hi : head0 + sp.ntile;
    const int slot = gi - split_owner(sp, head0);
    relu_state_segment<D>(k + head_base(rw, bh, H), v + head_base(rw, bh, H),
                          partials + ((size_t)bh * sp.PS + slot) * (size_t)(D + 1) * D,
                          (int)(lo - head0), (int)(seg_hi - lo), n, rw);
    lo = seg_hi;
  }
}

// ---- backward ----------------------------------------------------------------------------------
// Both sides work with the head's phi-weighted mean value row c = sum_f S[f] / sum_f z[f] taken out (exact in real arithmetic, any row
// would do; values with a common offset then cost the gradients nothing):
//   query side: S^c = S - z c^T; o - c and delta - dO . c take the places of o and delta, dq is unchanged up to eps / den, and its dz
//     comes out as dz + dS c;
//   key side: dzc[f] = dz[f] - c . r(dS[f]) with r the fp16 rounding of the image, so that
//     v_j . r(dS[f]) + dzc[f] = (v_j - c) . r(dS[f]) + (dz + dS c)[f] holds exactly.
// Each workgroup builds the operand images it needs in its prologue, from the state in registers (StateRegs).  Built by a kernel
// of their own and copied, they cost two launches of 9.4 us more (12 heads x 32760 x 128).
//
// The image of S^c in sG, z in sZ[D]; returns the scale.  scratch: FO*D + D + NTHREADS/64 floats of LDS.
template <int D, int NTHREADS>
__device__ __forceinline__ float build_relu_query_state(const float* __restrict__ state, uint4* sG, float* sZ, float* scratch,
                                                        float* __restrict__ mean_out, int tid) {
  using R = StateRegs<D, NTHREADS>;
  R S;
  S.load(state, tid);
  const float z_own = state[D * D + (tid < D ? tid : 0)];
  float* part = scratch;
  float* mean = part + R::FO * D;
  float* red = mean + D;
  if (tid < D) sZ[tid] = z_own;
  S.octet_sums(part);
  __syncthreads();
  if (tid < D) {
    float sv = 0.f, zt = 0.f;
#pragma unroll
    for (int o = 0; o < R::FO; ++o) sv += part[o * D + tid];
#pragma unroll
    for (int q = 0; q < D / 4; ++q) {
      const float4 z = reinterpret_cast<const float4*>(sZ)[q];
      zt += (z.x + z.y) + (z.z + z.w);
    }
    const float c = zt > 0.f ? sv / zt : 0.f;
    mean[tid] = c;
    if (mean_out != nullptr) mean_out[tid] = c;
  }
  __syncthreads();
  if (S.active) {
#pragma unroll
    for (int e = 0; e < 8; ++e)
#pragma unroll
      for (int i = 0; i < 4; ++i) S.v[e][i] -= sZ[8 * S.fo + e] * mean[4 * S.cq + i];
  }
  const float scale = S.scale(red, tid);
  write_grad_image16<D, NTHREADS, kPhiRelu>(S, sG, scale);
  return scale;
}

// The two images of dS and dzc in sZ[D]; returns the scale.  red: NTHREADS/64 floats of LDS.
template <int D, int NTHREADS>
__device__ __forceinline__ float build_relu_key_state(const float* __restrict__ dstate, uint4* sC, uint4* sG, float* sZ, float* red,
                                                      const float* __restrict__ mean, int tid) {
  using R = StateRegs<D, NTHREADS>;
  R S;
  S.load(dstate, tid);
  const float4 cm = *reinterpret_cast<const float4*>(mean + 4 * S.cq);
  float dz[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) dz[e] = dstate[D * D + 8 * S.fo + e];
  const float scale = S.scale(red, tid);
  write_grad_image16<D, NTHREADS, kPhiRelu>(S, sG, scale);
  write_apply_image16<D, NTHREADS, kPhiRelu>(S, sC, scale);
  const float inv = __builtin_amdgcn_rcpf(scale);           // exact: a power of two
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    auto img = [&](int i) { return (float)(_Float16)(scale * S.v[e][i]); };
    float dot = fmaf(img(3), cm.w, fmaf(img(2), cm.z, fmaf(img(1), cm.y, img(0) * cm.x)));
    dot = D == 128 ? half_wave_sum(dot) : row_sum(dot);     // over the CQ lanes that share the octet of features
    if (S.active && S.cq == 0) sZ[8 * S.fo + e] = dz[e] - dot * inv;
  }
  return scale;
}

// G^T = M Y^T for the 16 tokens of a wavefront: y[ks] is the lane's piece of its token's row (fp16, channels 32ks + 8q ..) and img an
// image of write_grad_image16<.., kPhiRelu>; register r of ga[2*ks + h] is then feature 32ks + 8q + 4h + r of the lane's token, element 4h + r of piece ks.
template <int D, int AHEAD>
__device__ __forceinline__ void relu_grad(const uint4* img, int lane, const uint4 (&y)[D / 32], f32x4 (&ga)[D / 16]) {
  using K = Tok16<D>;
#pragma unroll
  for (int mb = 0; mb < K::GB; ++mb) ga[mb] = f32x4{0.f, 0.f, 0.f, 0.f};
  const int gl = grad16_lane<D>(opaque_lane(lane));
  pipelined_operands<K::KS * K::GB, AHEAD>([&](int i) { return img[i * 64 + (gl ^ (4 * (i / K::GB)))]; },
                                           [&](int i, uint4 a) { ga[i % K::GB] = mfma_f16_16(a, y[i / K::GB], ga[i % K::GB]); });
}

// A lane's row pieces (bf16, channels 32ks + 8q .. of its token) -> 16 rows of base, a wavefront's tokens t0 ..: through `buf`
// ([16][D] bf16 of LDS, the wavefront's own), so that an instruction stores 1 KB of whole rows, with bounded buffer stores as in TokenRows.
template <int D>
struct RowStore {
  static constexpr int CH = D / 8, RPI = 64 / CH;          // 16-byte chunks of a row, rows per store
  char* buf;
  int lane;
  __device__ __forceinline__ void put(int ks, uint4 x) const {
    const int row = lane % 16;
    *reinterpret_cast<uint4*>(buf + row * D * 2 + (((4 * ks + lane / 16) ^ swz<D>(row)) * 16)) = x;
  }
  template <bool STREAM>                                    // non-temporal
  __device__ __forceinline__ void flush(uint16_t* base, size_t sn, int t0, int n) const {
    __builtin_amdgcn_wave_barrier();
    const int left = n - t0 < 16 ? n - t0 : 16;
    const uint32_t pitch = (uint32_t)sn * 2;
    const __amdgpu_buffer_rsrc_t rows = __builtin_amdgcn_make_buffer_rsrc(reinterpret_cast<char*>(base) + (size_t)t0 * pitch, 0,
                                                                          left > 0 ? (uint32_t)left * pitch : 0, 0x00020000);
    const int c = lane % CH;
#pragma unroll
    for (int i = 0; i < 16 / RPI; ++i) {
      const int row = i * RPI + lane / CH;
      const uint4 x = *reinterpret_cast<const uint4*>(buf + row * D * 2 + ((c ^ swz<D>(row)) * 16));
      __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, x), rows, (uint32_t)row * pitch + 16 * c, 0, STREAM ? 2 : 0);
    }
    __builtin_amdgcn_wave_barrier();
  }
};

// ---- query side of the backward -------------------------------------------------------------------
// grid (P, BH), 12 wavefronts, one workgroup per compute unit.  Wavefronts 0-7 ("tok") each own 16 tokens of a 128-token tile, four
// lanes a token: G = dO S^T with the tokens on the accumulator columns and the features in the order in which the lane holds
// its token's channels, so den = phi . z and delta = phi . G / den are dots of registers, the mask of dq is the lane's own row and dq
// leaves in the pieces in which q came.  They park phi(q) and gamma * dO / den as fp16 and form dq while wavefronts 8-11 ("acc") contract
// the tile over its tokens into dS (dz: one more MFMA per k-step).  Bound by its instruction stream (its rows take 51 us
// at the memory's rate): 75 us at 12 heads x 32760 x 128, 11.5 at 12 x 4133 x 64; with four token wavefronts of 32 tokens 89 and 12.6.
constexpr int NTQ = 768;
template <int D, bool STREAM>
__global__ __launch_bounds__(NTQ) void relu_bwd_q_kernel(const uint16_t* __restrict__ q, const uint16_t* __restrict__ dout,
                                                         const float* __restrict__ state, float* __restrict__ mean_row,
                                                         uint16_t* __restrict__ dq, float* __restrict__ partials,
                                                         int H, int n, int P, Rows rw) {
  using K = Tok16<D>;
  constexpr int RS = D * 2;
  constexpr int WMN = D / 64;
  constexpr int NTOK = kTile / 16;
  extern __shared__ uint4 smem[];
  uint4* sG = smem;                                        // image of S^c
  char* sPhi = reinterpret_cast<char*>(sG + K::G_IMG);     // [kTile][D] fp16: phi(q)
  char* sDO = sPhi + kTile * RS;                           // [kTile][D] fp16: gamma * dO / den
  uint16_t* sW16 = reinterpret_cast<uint16_t*>(sDO + kTile * RS);   // [kTile] fp16: -gamma * delta / den
  float* sZ = reinterpret_cast<float*>(sW16 + kTile);      // [D] z, unscaled
  float* sRed = sZ + D;                                    // [8] the tile's operand maxima
  char* sOut = reinterpret_cast<char*>(sRed + NTOK);       // [8][16][D] bf16: RowStore

  const int tid = threadIdx.x, lane = tid % 64;
  const int w = __builtin_amdgcn_readfirstlane(tid / 64);
  const int bh = blockIdx.y, p = blockIdx.x;
  const int ntile = (n + kTile - 1) / kTile;

  const float scale = build_relu_query_state<D, NTQ>(state + (size_t)bh * (D + 1) * D, sG, sZ, reinterpret_cast<float*>(sPhi),
                                                     p == 0 ? mean_row + (size_t)bh * D : nullptr, tid);
  __syncthreads();

  // running power-of-two scale of the sums over tokens (see gamma_for), the same in every wavefront; returns the factor for the
  // accumulators
  float gamma = kGammaUnset;
  auto next_gamma = [&]() -> float {
    float m = sRed[0];
#pragma unroll
    for (int i = 1; i < NTOK; ++i) m = fmaxf(m, sRed[i]);
    float gnext = gamma;
    const float ratio = gamma_step(gnext, gamma_for(m));
    gamma = __builtin_bit_cast(float, __builtin_amdgcn_readfirstlane(__builtin_bit_cast(int, gnext)));
    return __builtin_bit_cast(float, __builtin_amdgcn_readfirstlane(__builtin_bit_cast(int, ratio)));
  };

  if (w < NTOK) {
    const int ql = lane / 16;
    uint16_t* dqb = dq + head_base(rw, bh, H);
    const float zero = opaque_zero_scalar();
    const LoadRows16<D> qrows(q + head_base(rw, bh, H), rw.sn, n, lane), drows(dout + head_base(rw, bh, H), rw.sn, n, lane);
    uint4 xq[K::KS], dor[K::KS], xn[K::KS];
    qrows.load(xn, p * kTile + 16 * w);
    drows.load(dor, p * kTile + 16 * w);
    // the first rows have arrived before the loop: with them still out, the compiler's wait at the top of a tile, which has to hold
    // for the first tile too, would be a wait for the previous tile's stores
    qrows.arrived(xn);
    drows.arrived(dor);
    for (int tile = p; tile < ntile; tile += P) {
      const int t0 = tile * kTile + 16 * w;                // (rows past n are zeros)
      // phi(q); whether it has any feature above zero; the token's largest finite |dO|
      uint32_t any = 0;
      FiniteMax16 most;
#pragma unroll
      for (int ks = 0; ks < K::KS; ++ks) {
        xq[ks] = make_uint4(relu_bf16x2(xn[ks].x), relu_bf16x2(xn[ks].y), relu_bf16x2(xn[ks].z), relu_bf16x2(xn[ks].w));
        any |= (xq[ks].x | xq[ks].y) | (xq[ks].z | xq[ks].w);
        most.take(dor[ks]);
      }
      float dmax = most.value(), any_of = __builtin_bit_cast(float, any);
      quad2<MagOp>(dmax, any_of);
      const float stok = kTokenUnit * pow2_normaliser(fminf(dmax, kTokenMax)), istok = __builtin_amdgcn_rcpf(stok);
      // a query with phi(q) = 0 adds nothing to dS and dz, but its 1 / den = 1 / eps would set the
      // common scale gamma and push every other token's operand into the fp16 subnormals
      const bool live = __builtin_bit_cast(uint32_t, any_of) != 0;
      // dO scaled by a power of two: exact in fp16 down to 2^-27 of the token's largest
      uint4 bq[K::KS];
#pragma unroll
      for (int ks = 0; ks < K::KS; ++ks) {
        float f[8];
        unpack_bf16x8(dor[ks], f);
        bq[ks] = make_uint4(mul_pack_f16x2(f[0], f[1], stok, zero), mul_pack_f16x2(f[2], f[3], stok, zero),
                            mul_pack_f16x2(f[4], f[5], stok, zero), mul_pack_f16x2(f[6], f[7], stok, zero));
      }

      // G (times scale * stok)
      f32x4 ga[K::GB];
      relu_grad<D, 4>(sG, lane, bq, ga);
      // the rows stay packed until their next use: seen as the same values, their unpacked form would be kept (and spilled)
      auto repack = [&](uint4 (&x)[K::KS]) {
#pragma unroll
        for (int ks = 0; ks < K::KS; ++ks) asm volatile("" : "+v"(x[ks].x), "+v"(x[ks].y), "+v"(x[ks].z), "+v"(x[ks].w));
      };
      repack(bq);
      const int z_at = 2 * ql + opaque_zero();
      auto z8 = [&](int ks, float (&z)[8]) {
        const float4 a = reinterpret_cast<const float4*>(sZ)[z_at + 8 * ks], b = reinterpret_cast<const float4*>(sZ)[z_at + 8 * ks + 1];
        z[0] = a.x; z[1] = a.y; z[2] = a.z; z[3] = a.w; z[4] = b.x; z[5] = b.y; z[6] = b.z; z[7] = b.w;
      };
      float a_sum = 0.f, Z = 0.f;
#pragma unroll
      for (int ks = 0; ks < K::KS; ++ks) {
        float f[8], z[8];
        unpack_bf16x8(xq[ks], f);
        z8(ks, z);
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          a_sum = fmaf(ga[2 * ks + e / 4][e % 4], f[e], a_sum);
          Z = fmaf(z[e], f[e], Z);
        }
      }
      repack(xq);
      quad2<SumOp>(a_sum, Z);
      const float inv_den = __builtin_amdgcn_rcpf(Z + kReluEps);
      // 1 / (scale * stok * den); scale and stok are powers of two
      const float r1 = (inv_den * __builtin_amdgcn_rcpf(scale)) * istok;
      const float delta = a_sum * r1;
      {
        // the tile's largest operand of the two sums, |dO_i| / den_i or |delta_i| / den_i, of those that are finite
        const float ad = fabsf(delta);
        const float m = row_max_mag(fmaxf(live ? fmaxf(dmax, ad < __builtin_inff() ? ad : 0.f) * inv_den : 0.f, 0.f));
        if (lane == 0) sRed[w] = m;
      }
      __syncthreads();                                   // the previous tile has been read
      next_gamma();
      {
        const unsigned lz = opaque_lane(lane);
        const int row = 16 * w + lz % 16, psw = swz<D>(lz % 16), qz = lz / 16;
        char* rowp = sPhi + row * RS;
        char* drowp = sDO + row * RS;
        const float sc = live ? inv_den * gamma : 0.f, so = sc * istok;
#pragma unroll
        for (int ks = 0; ks < K::KS; ++ks) {
          *reinterpret_cast<uint4*>(rowp + (((4 * ks + qz) ^ psw) * 16)) =
              make_uint4(bf16x2_to_f16x2(xq[ks].x), bf16x2_to_f16x2(xq[ks].y), bf16x2_to_f16x2(xq[ks].z), bf16x2_to_f16x2(xq[ks].w));
          *reinterpret_cast<uint4*>(drowp + (((4 * ks + qz) ^ psw) * 16)) =
              make_uint4(mul_pack_f16x2(bq[ks].x, so, zero), mul_pack_f16x2(bq[ks].y, so, zero), mul_pack_f16x2(bq[ks].z, so, zero),
                         mul_pack_f16x2(bq[ks].w, so, zero));
        }
        if (lane < 16) sW16[row] = (uint16_t)(pack_f16x2(live ? -delta * sc : 0.f, 0.f) & 0xffffu);
      }
      repack(xq);
      // the next tile's rows, before the dq stores: loads and stores retire in order
      qrows.load(xn, t0 + P * kTile);
      drows.load(dor, t0 + P * kTile);
      __syncthreads();
      // dq = (G - delta z) / den where q > 0
      const float r2 = inv_den * delta;
      const RowStore<D> out{sOut + w * 16 * RS, (int)opaque_lane(lane)};
#pragma unroll
      for (int ks = 0; ks < K::KS; ++ks) {
        float f[8], z[8], v[8];
        unpack_bf16x8(xq[ks], f);
        z8(ks, z);
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] = f[e] > 0.f ? fmaf(ga[2 * ks + e / 4][e % 4], r1, -(r2 * z[e])) : 0.f;
        out.put(ks, make_uint4(pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3]), pack_bf16x2(v[4], v[5]), pack_bf16x2(v[6], v[7])));
      }
      out.template flush<STREAM>(dqb, rw.sn, t0, n);
    }
  } else {
    f32x16 s[WMN][WMN], zacc;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      zacc[r] = 0.f;
#pragma unroll
      for (int i = 0; i < WMN; ++i)
#pragma unroll
        for (int j = 0; j < WMN; ++j) s[i][j][r] = 0.f;
    }
    const int g = lane / 32;
    const Quadrant<D> qd(w - NTOK);
    const QuadrantReads<D> rd(qd, sPhi, sDO, lane);
    for (int tile = p; tile < ntile; tile += P) {
      __syncthreads();
      const float ratio = next_gamma();
      if (ratio != 1.f) {                                // this tile is larger than every earlier one
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          zacc[r] *= ratio;
#pragma unroll
          for (int i = 0; i < WMN; ++i)
#pragma unroll
            for (int j = 0; j < WMN; ++j) s[i][j][r] *= ratio;
        }
      }
      __syncthreads();
      contract_tile<D>(rd, s, zacc, qd.do_z(),
                       [&](int ks) { return as_f16x8(*reinterpret_cast<const uint4*>(sW16 + 16 * ks + 8 * g)); });
    }
    const float ig = __builtin_amdgcn_rcpf(gamma);    // exact: gamma is a power of two
    float* dst = partials + ((size_t)bh * P + p) * (size_t)(D + 1) * D;
    const int c = lane % 32;
#pragma unroll
    for (int i = 0; i < WMN; ++i)
#pragma unroll
      for (int j = 0; j < WMN; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int f = 32 * qd.fblk(i) + 8 * (r / 4) + 4 * g + (r % 4);
          dst[f * D + 32 * qd.cblk(j) + c] = s[i][j][r] * ig;
        }
    if (qd.do_z() && c == 0) {
#pragma unroll
      for (int r = 0; r < 16; ++r) dst[D * D + 32 * qd.zblk() + 8 * (r / 4) + 4 * g + (r % 4)] = zacc[r] * ig;
    }
  }
}

// ---- key side of the backward ---------------------------------------------------------------------
// Wavefronts on 16-token blocks of their own: dv = phi(k) dS with the tokens on the accumulator rows, and
// g = v dS^T + dz with the tokens on the columns (relu_grad), dk = g where k > 0 in the pieces in which k came.
// NTK: 12 wavefronts where a workgroup has several rounds of width 128, else 8, whose prologue is the shorter: 8 / 12 / 16 wavefronts, us, 12 heads x 32760 x
// 128 80.4 / 77.5 / 82.6, 4 x 1000 x 128 8.3 / 9.6 / 11.3, 12 x 16000 x 64 21.7 / 22.3 / 22.7, 12 x 4133 x 64 9.7 / 9.95 / 9.75.  (Eight wavefronts of 32 tokens: 88.6,
// 15.1, 23.7 and 10.8; the rows take 69 at 12 x 32760 x 128.)
template <int D, bool STREAM, int NTK>
__global__ __launch_bounds__(NTK) void relu_bwd_k_kernel(const uint16_t* __restrict__ k, const uint16_t* __restrict__ v,
                                                         const float* __restrict__ dstate, const float* __restrict__ mean_row,
                                                         uint16_t* __restrict__ dk, uint16_t* __restrict__ dv,
                                                         int H, int n, Rows rw) {
  using K = Tok16<D>;
  constexpr int NW = NTK / 64;
  extern __shared__ uint4 smem[];
  uint4* sC = smem;                                        // image of dS for dv
  uint4* sG = sC + K::A_IMG;                               // image of dS for g
  float* sZ = reinterpret_cast<float*>(sG + K::G_IMG);     // [D] dzc
  float* sRed = sZ + D;                                    // [NW]
  char* sOut = reinterpret_cast<char*>(sRed + NW);         // [NW][16][D] bf16: RowStore

  const int tid = threadIdx.x, lane = tid % 64;
  const int w = __builtin_amdgcn_readfirstlane(tid / 64);
  const int ql = lane / 16;
  const int bh = blockIdx.y;
  uint16_t* dkb = dk + head_base(rw, bh, H);
  uint16_t* dvb = dv + head_base(rw, bh, H);
  const LoadRows16<D> krows(k + head_base(rw, bh, H), rw.sn, n, lane), vrows(v + head_base(rw, bh, H), rw.sn, n, lane);
  const float scale = build_relu_key_state<D, NTK>(dstate + (size_t)bh * (D + 1) * D, sC, sG, sZ, sRed, mean_row + (size_t)bh * D, tid);
  const float inv_scale = __builtin_amdgcn_rcpf(scale);    // exact: power of two
  __syncthreads();

  const int step = 16 * NW * gridDim.x;
  for (int t0 = 16 * (blockIdx.x * NW + w); t0 < n; t0 += step) {
    uint4 xk[K::KS], xv[K::KS];
    krows.load(xk, t0);
    vrows.load(xv, t0);
    {
      f32x4 va[K::MB];
#pragma unroll
      for (int mb = 0; mb < K::MB; ++mb) va[mb] = f32x4{0.f, 0.f, 0.f, 0.f};
      const uint4* sc = sC + lane + opaque_zero();
      uint4 a;
      pipelined_operands<K::KS * K::MB, 3>([&](int i) { return sc[i * 64]; },
                                           [&](int i, uint4 b) {
                                             if (i % K::MB == 0) a = relu_f16x8(xk[i / K::MB]);
                                             va[i % K::MB] = mfma_f16_16(a, b, va[i % K::MB]);
                                           });
      const float none[K::MB] = {};
      store_token_rows16<D, false, false>(dvb, rw.sn, t0, n, lane, va, inv_scale, none);
    }
    {
      uint4 y[K::KS];
#pragma unroll
      for (int ks = 0; ks < K::KS; ++ks)
        y[ks] = make_uint4(bf16x2_to_f16x2(xv[ks].x), bf16x2_to_f16x2(xv[ks].y), bf16x2_to_f16x2(xv[ks].z), bf16x2_to_f16x2(xv[ks].w));
      f32x4 ga[K::GB];
      relu_grad<D, 3>(sG, lane, y, ga);
      const RowStore<D> out{sOut + w * 16 * D * 2, (int)opaque_lane(lane)};
      const int z_at = 2 * ql + opaque_zero();
#pragma unroll
      for (int ks = 0; ks < K::KS; ++ks) {
        const float4 za = reinterpret_cast<const float4*>(sZ)[z_at + 8 * ks], zb = reinterpret_cast<const float4*>(sZ)[z_at + 8 * ks + 1];
        const float z[8] = {za.x, za.y, za.z, za.w, zb.x, zb.y, zb.z, zb.w};
        float f[8], u[8];
        unpack_bf16x8(xk[ks], f);
#pragma unroll
        for (int e = 0; e < 8; ++e) u[e] = f[e] > 0.f ? fmaf(ga[2 * ks + e / 4][e % 4], inv_scale, z[e]) : 0.f;
        out.put(ks, make_uint4(pack_bf16x2(u[0], u[1]), pack_bf16x2(u[2], u[3]), pack_bf16x2(u[4], u[5]), pack_bf16x2(u[6], u[7])));
      }
      out.template flush<STREAM>(dkb, rw.sn, t0, n);
    }
  }
}

template <int D>
constexpr size_t state_smem() { return 2 * (size_t)kTile * D * 2; }
template <int D>
constexpr size_t q_smem() {
  return sizeof(uint4) * Tok16<D>::G_IMG + 3 * (size_t)kTile * D * 2 + kTile * 2 + (D + kTile / 16) * sizeof(float);
}
template <int D, int NTK>
constexpr size_t k_smem() {
  return sizeof(uint4) * (Tok16<D>::A_IMG + Tok16<D>::G_IMG) + (D + NTK / 64) * sizeof(float) + (NTK / 64) * 16 * (size_t)D * 2;
}

template <int D>
hipError_t run_state(const void* k, const void* v, float* partials, const Plan& p, hipStream_t s) {
  hipError_t e;
  if ((e = set_smem_once<relu_state_kernel<D>>(state_smem<D>())) != hipSuccess) return e;
  relu_state_kernel<D><<<dim3(p.split.G), NT, state_smem<D>(), s>>>((const uint16_t*)k, (const uint16_t*)v, partials,
                                                                   p.H, p.n, p.split, p.rows);
  return hipGetLastError();
}

template <int D, bool STREAM, int NTK>
hipError_t run_bwd_k(const BwdArgs& a, const Plan& p, int per_head, hipStream_t s) {
  constexpr size_t smem = k_smem<D, NTK>();
  const hipError_t e = set_smem_once<relu_bwd_k_kernel<D, STREAM, NTK>>(smem);
  if (e != hipSuccess) return e;
  const int units = (p.n + NTK / 4 - 1) / (NTK / 4);       // 16 tokens a wavefront
  relu_bwd_k_kernel<D, STREAM, NTK><<<dim3(units < per_head ? units : per_head, p.BH), NTK, smem, s>>>(
      (const uint16_t*)a.k, (const uint16_t*)a.v, a.dstate, a.vbar, (uint16_t*)a.dk, (uint16_t*)a.dv, p.H, p.n, p.rows);
  return hipGetLastError();
}

template <int D, bool STREAM>
hipError_t run_bwd(const BwdArgs& a, const Plan& p, hipStream_t s) {
  hipError_t e;
  if ((e = set_smem_once<relu_bwd_q_kernel<D, STREAM>>(q_smem<D>())) != hipSuccess) return e;
  relu_bwd_q_kernel<D, STREAM><<<dim3(p.P, p.BH), NTQ, q_smem<D>(), s>>>((const uint16_t*)a.q, (const uint16_t*)a.dout, a.state, a.vbar,
                                                                (uint16_t*)a.dq, a.partials, p.H, p.n, p.P, p.rows);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  if ((e = launch_state_reduce(a.partials, a.dstate, p, DrSum{}, s)) != hipSuccess) return e;
  const int per_head = p.BH < kCUs ? kCUs / p.BH : 1;
  if constexpr (D == 128)
    if ((p.n + 191) / 192 > per_head) return run_bwd_k<D, STREAM, 768>(a, p, per_head, s);
  return run_bwd_k<D, STREAM, 512>(a, p, per_head, s);
}

}  // namespace

hipError_t launch_relu_state_bf16(const void* k, const void* v, float* partials, const Plan& p, hipStream_t s) {
  return p.d == 128 ? run_state<128>(k, v, partials, p, s) : run_state<64>(k, v, partials, p, s);
}

hipError_t launch_relu_bwd_bf16(const BwdArgs& a, const Plan& p, hipStream_t s) {
  if (stream_gradients(p)) return p.d == 128 ? run_bwd<128, true>(a, p, s) : run_bwd<64, true>(a, p, s);
  return p.d == 128 ? run_bwd<128, false>(a, p, s) : run_bwd<64, false>(a, p, s);
}

}  // namespace linattn
