// bf16-I/O forward path on gfx950 MFMA (fp32 accumulation), tokens along the N dimension.
//
// Precision: the projections u = x W~ multiply the stored bf16 values exactly (bf16 MFMA).
// phi, and the state it is contracted with, are carried as fp16 (11-bit significand): phi lies
// in [0,1] and a few entries near 1 (sharp softmaxes of large-magnitude tokens) dominate sums
// that otherwise cancel, so 8-bit significands miss the 1e-2 accuracy contract by 2-4x while
// fp16 operands leave the bf16 rounding of the output as the largest error.  V is widened
// bf16 -> fp16 on its way into LDS (exact for 2^-14 <= |v| < 65520).
//
// state_partials_ws_kernel   : phi(K) (Eq. 5) fused with the split-n partial state
//                              S_p = sum_j phi(k_j)^T v_j, z_p = sum_j phi(k_j)  (Eq. 3)
// apply_bf16_kernel          : phi(Q), out = phi(Q) S / (phi(Q) . z), bf16 store (Eq. 3)
//
// Both start from U^T = W~^T X^T with X rows loaded straight into the MFMA B operand
// (16 bytes per lane), so a lane owns one token and d/4 of its d/2 pre-softmax features; the
// softmax reductions are in-lane plus one exchange with lane^32.
#include "kernels.h"
#include "mfma_common.h"

namespace linattn {
namespace {

// ------------------------------------------------------------------------------------------
// Query pass.  Units of 32-token blocks, one to a wavefront, are dealt to one workgroup per compute unit (make_deal_of_blocks), and
// the workgroups of a head sweep its tokens together (next_share).  Per block: load Q rows straight into the
// B operand of the projection (a lane owns a token), phi; phi then is the A operand of
// out = phi S, which puts the tokens on the accumulator rows and the channels on the lanes: a lane
// holds MB adjacent channels of 16 tokens and every store instruction writes two whole rows.  One
// more column block of the S image carries z in every column, so the same lanes get phi . z.
template <int MB> struct RowPiece;
template <> struct RowPiece<4> { typedef uint2 type; };
template <> struct RowPiece<2> { typedef uint32_t type; };
__device__ __forceinline__ uint32_t piece_word(const uint2& p, int i) { return i ? p.y : p.x; }
__device__ __forceinline__ uint32_t piece_word(const uint32_t& p, int) { return p; }
__device__ __forceinline__ void set_piece_word(uint2& p, int i, uint32_t v) { if (i) p.y = v; else p.x = v; }
__device__ __forceinline__ void set_piece_word(uint32_t& p, int, uint32_t v) { p = v; }

// The state of head bh as the sum of its workgroups' partials, pairwise, to sum[(D+1)*D/4] in LDS and, if given, to dst.  Up to 20 loads of
// a thread are in flight; those of a missing slot repeat the last one's and count as zero (branch-free).
template <int D> constexpr int kSumSlots = D == 64 ? 8 : 2;      // see sum_in_apply
template <int N, int NTHREADS, int NS>
__device__ __forceinline__ void sum_slots_of(const float4* __restrict__ src, int cnt, float4* sum, float4* __restrict__ dst, int tid) {
  constexpr int ALL = (N + NTHREADS - 1) / NTHREADS, EB = ALL * NS <= 20 ? ALL : 16 / NS;      // elements at a time: all of a thread's, if they fit
  auto add = [](float4 a, float4 b) { return make_float4(a.x + b.x, a.y + b.y, a.z + b.z, a.w + b.w); };
#pragma unroll 1
  for (int e0 = tid; e0 < N; e0 += EB * NTHREADS) {
    float4 t[EB][NS];
#pragma unroll
    for (int j = 0; j < EB; ++j) {
      const int e = e0 + j * NTHREADS < N ? e0 + j * NTHREADS : N - 1;
#pragma unroll
      for (int p = 0; p < NS; ++p) t[j][p] = src[(size_t)(p < cnt ? p : cnt - 1) * N + e];
    }
#pragma unroll
    for (int j = 0; j < EB; ++j) {
#pragma unroll
      for (int p = 1; p < NS; ++p)
        if (p >= cnt) t[j][p] = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
      for (int m = 1; m < NS; m *= 2)
#pragma unroll
        for (int p = 0; p < NS; p += 2 * m) t[j][p] = add(t[j][p], t[j][p + m]);
      if (e0 + j * NTHREADS < N) {
        sum[e0 + j * NTHREADS] = t[j][0];
        if (dst != nullptr) dst[e0 + j * NTHREADS] = t[j][0];
      }
    }
  }
}
template <int D, int NTHREADS>
__device__ __forceinline__ void sum_slots(const float* __restrict__ partials, float4* sum, float4* __restrict__ dst, const Split& sp,
                                          int bh, int tid) {
  constexpr int N = (D + 1) * D / 4;
  const int cnt = split_owner(sp, (long long)(bh + 1) * sp.ntile - 1) - split_owner(sp, (long long)bh * sp.ntile) + 1;
  const float4* src = reinterpret_cast<const float4*>(partials) + (size_t)bh * sp.PS * N;
  if constexpr (kSumSlots<D> > 2) {
    if (cnt > 4) { sum_slots_of<N, NTHREADS, kSumSlots<D>>(src, cnt, sum, dst, tid); return; }
    if (cnt > 2) { sum_slots_of<N, NTHREADS, 4>(src, cnt, sum, dst, tid); return; }
  }
  sum_slots_of<N, NTHREADS, 2>(src, cnt, sum, dst, tid);
}

// Which query passes may have their units dealt evenly (run_apply): not those that sum, with few units a head.  Those that have take the instance with a loop over a workgroup's heads (EVEN);
// carried by the others it cost them 0.2 to 0.6 us: 12 heads x 4133 x 64 18.4 us a call, 18.1 without, 12 x 8190 x 128 37.3 / 36.8, 30 x 1000 x 64 15.5 /
// 15.0.
template <bool SUM>
constexpr bool apply_even = !SUM;

// Wavefronts to a SIMD that the register limit leaves room for: those of the workgroup, two or three.  Four at width 64: the
// limit keeps the loop's schedule from spreading into the prologue's registers (without it the CogVideoX-2B shape
// loses 2 us).  Not with blend, whose pieces of s need the registers (they spill), nor where 12 wavefronts sum the state (so does their
// prologue).  Five (96 registers) for long calls of the Hedgehog map without the loop over heads: as scheduled for four, with 99, 24 heads x 20000 x 64
// [B,n,H,d] takes 65.4 us a call, so 63.0; 30 x 17550 63.8 / 62.6; 12 x 8190 22.1 / 22.3; ReLU 55.8 / 56.3.
template <int D, bool BLEND, int KIND, bool SUM, int NW, bool EVEN>
constexpr int kApplyOccupancy = D == 128 || BLEND || (SUM && NW == 12) ? NW / 4 : KIND == kPhiHedgehog && !SUM && NW == 8 && !EVEN ? 5 : 4;

// The prologue holds the state in registers (StateRegs): staged in LDS first, the pass took 2-3 us longer per launch (57.5 -> 54.5
// us at 12 heads x 32760 x 128, 7.6 -> 7.2 at 4 x 1000 x 64).
// BLEND: mixed attention (Sec. 4.1, Eq. 6): out = r' s + (1 - r') o with the softmax-branch output
// s read in the same pieces as out is stored, and r' = clip(*rptr, 0, 1).
// KIND = kPhiRelu: phi(q) = max(q, 0) straight from the loaded rows (no projection, no W~), features
// in channel order, kReluEps in the denominator.
// SUM: the state is summed here, from the partials of at most kSumSlots<D> state-pass workgroups a head (the rule is at
// sum_in_apply); the first workgroup of a head writes it to `state`.
template <int D, bool BLEND, int KIND, bool SUM, int NW, bool EVEN>
__global__ __launch_bounds__(64 * NW, (kApplyOccupancy<D, BLEND, KIND, SUM, NW, EVEN>)) void apply_bf16_kernel(const uint16_t* __restrict__ q, const uint16_t* __restrict__ wq,
                                                         const float* __restrict__ partials, float* __restrict__ state,
                                                         uint16_t* __restrict__ out,
                                                         const uint16_t* __restrict__ blend, const float* __restrict__ rptr,
                                                         int H, int n, Split deal, Split sp, Rows rw) {
  using C = Cfg<D>;
  using L = ApplyLayout<D>;
  constexpr int NT3 = 64 * NW;
  constexpr int SA_IMG = L::KS * L::MBZ * 64;
  constexpr int HB = L::MB / 2;             // channel column blocks per accumulation pass (two passes)
  using Piece = typename RowPiece<L::MB>::type;   // a lane's MB adjacent bf16 channels of one token
  extern __shared__ uint4 smem[];
  uint4* sWA = smem;
  uint4* sSA = sWA + C::W_IMG;
  char* sStage = reinterpret_cast<char*>(sSA + SA_IMG); // z and reduction slots of the prologue

  const int tid = threadIdx.x, lane = tid % 64;
  const int w = __builtin_amdgcn_readfirstlane(tid / 64);
  const int g = lane / 32;
  for (Share sh = EVEN ? first_share(deal, blockIdx.x, blockIdx.y) : head_share(deal, blockIdx.x, blockIdx.y); sh.there;
       sh = EVEN ? next_share(deal, blockIdx.x, sh) : Share{}) {
    const int bh = sh.bh, h = bh % H;
    const uint16_t* qb = q + head_base(rw, bh, H);
    uint16_t* ob = out + head_base(rw, bh, H);
    const uint16_t* bb = BLEND ? blend + head_base(rw, bh, H) : nullptr;
    const float rb = BLEND ? fminf(fmaxf(*rptr, 0.f), 1.f) : 0.f;

    const Blocks own = blocks_of(deal, sh, w, (n + 31) / 32);
    const int nblk = own.end, stride = own.stride;
    const int c = lane % 32;
    const uint32_t lane_off = ((uint32_t)(4 * g) * (uint32_t)rw.sn + (uint32_t)(L::MB * c)) * 2u;   // bytes

    uint4 x[C::UK];
    auto load_block = [&](int b) {
      const int t = b * 32 + (lane % 32);
      const int tc = t < n ? t : (n - 1);
      const uint4* row = reinterpret_cast<const uint4*>(qb + (size_t)tc * rw.sn);
#pragma unroll
      for (int ks = 0; ks < C::UK; ++ks) x[ks] = row[2 * ks + g];
    };
    // the first block's rows are requested before the prologue, so that they arrive under it
    int b = own.first;
    if (b < nblk) load_block(b);

    float scale;
    {
      using R = StateRegs<D, NT3>;
      float* sb = state + (size_t)bh * (D + 1) * D;
      float* sZ = reinterpret_cast<float*>(sStage);
      R S;
      WImage<D> W;
      if constexpr (KIND == kPhiHedgehog) W.load(wq + (size_t)h * D * C::HALF, tid);
      float zv;
      if constexpr (SUM) {
        float4* sSum = reinterpret_cast<float4*>(sZ + D + 64);
        sum_slots<D, NT3>(partials, sSum, sh.u == 0 ? reinterpret_cast<float4*>(sb) : nullptr, sp, bh, tid);
        __syncthreads();
        const float* sum = reinterpret_cast<const float*>(sSum);
        S.load(sum, tid);
        zv = tid < D ? sum[D * D + tid] : 0.f;
      } else {
        S.load(sb, tid);
        zv = tid < D ? sb[D * D + tid] : 0.f;
      }
      if (tid < D) sZ[tid] = zv;
      if constexpr (KIND == kPhiHedgehog) W.write(sWA, tid);
      scale = S.scale(sZ + D, tid, fabsf(zv));            // (its barrier covers z as well)
      S.template write_apply_image<L::MBZ, KIND>(sSA, scale);
      R::template write_z_block<KIND>(sZ, sSA, scale, tid);
    }
    __syncthreads();
    const float den_eps = KIND == kPhiRelu ? scale * kReluEps : 0.f;    // the image carries scale * z

    for (; b < nblk; b += stride) {
      uint32_t pk[C::NPK];
      if constexpr (KIND == kPhiRelu) {
        static_assert(C::NPK == 4 * C::UK, "one 16-byte piece of phi per piece of the row");
#pragma unroll
        for (int ks = 0; ks < C::UK; ++ks) {
          const uint4 f = relu_f16x8(x[ks]);
          pk[4 * ks] = f.x; pk[4 * ks + 1] = f.y; pk[4 * ks + 2] = f.z; pk[4 * ks + 3] = f.w;
        }
        if constexpr (!BLEND) load_block(b + stride < nblk ? b + stride : b);
      } else {
        f32x16 u[C::UM];
        project<D>(x, sWA, lane, u);
        // next block's rows fly during the rest of this one (BLEND: the pieces of s take their
        // registers, so each 16-byte piece of the next rows is requested in the second pass as the
        // k-step that frees a piece of phi has been issued)
        if constexpr (!BLEND) load_block(b + stride < nblk ? b + stride : b);
        softmax_pair_ratio<D>(u, pk);
      }
      // register r of an accumulator is token b*32 + 8*(r/4) + 4g + r%4; the lane's MB channels of it
      // are MB*c .. MB*c + MB-1, two bytes each
      const bool full = b * 32 + 32 <= n;
      Piece sv[BLEND ? 16 : 1];               // the same pieces of the softmax branch
      if constexpr (BLEND) {
        const char* sb = reinterpret_cast<const char*>(bb + (size_t)(b * 32) * rw.sn) + lane_off;
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int row = 8 * (r / 4) + (r % 4);
          const bool there = full || b * 32 + row + 4 * g < n;
          sv[r] = there ? *reinterpret_cast<const Piece*>(sb + (size_t)row * rw.sn * 2) : Piece{};
        }
      }

      const uint4* next_row = nullptr;
      if constexpr (BLEND) {
        const int bn = b + stride < nblk ? b + stride : b;
        const int t = bn * 32 + (lane % 32);
        next_row = reinterpret_cast<const uint4*>(qb + (size_t)(t < n ? t : n - 1) * rw.sn);
      }
      // out = phi S in two passes over the lane's channels; the first also carries the block whose
      // every column is z, so each lane gets the normalisers of its 16 tokens
      const uint4* ssa = sSA + lane + opaque_zero();
      float inv[16], keep[16];
      Piece word[16];
#pragma unroll
      for (int pass = 0; pass < 2; ++pass) {
        f32x16 o[HB], dn;
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          dn[r] = 0.f;
#pragma unroll
          for (int i = 0; i < HB; ++i) o[i][r] = 0.f;
        }
#pragma unroll
        for (int ks = 0; ks < L::KS; ++ks) {
          uint4 aq; aq.x = pk[4 * ks]; aq.y = pk[4 * ks + 1]; aq.z = pk[4 * ks + 2]; aq.w = pk[4 * ks + 3];
          const f16x8 aop = as_f16x8(aq);
#pragma unroll
          for (int i = 0; i < HB; ++i)
            o[i] = __builtin_amdgcn_mfma_f32_32x32x16_f16(aop, as_f16x8(ssa[(ks * L::MBZ + pass * HB + i) * 64]), o[i], 0, 0, 0);
          if (pass == 0) dn = __builtin_amdgcn_mfma_f32_32x32x16_f16(aop, as_f16x8(ssa[(ks * L::MBZ + L::MB) * 64]), dn, 0, 0, 0);
          if constexpr (BLEND) {
            static_assert(C::UK == L::KS, "one piece of x per k-step");
            if (pass == 1) x[ks] = next_row[2 * ks + g];
          }
        }
        if (pass == 0) {
#pragma unroll
          for (int r = 0; r < 16; ++r) inv[r] = __builtin_amdgcn_rcpf(KIND == kPhiRelu ? dn[r] + den_eps : dn[r]);
        }
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          float y[HB];
#pragma unroll
          for (int i = 0; i < HB; ++i) {
            y[i] = o[i][r] * inv[r];
            if constexpr (BLEND) {
              const int ch = pass * HB + i;                         // which of the lane's MB channels
              const uint32_t sw = piece_word(sv[r], ch / 2);
              const float sf = (ch % 2) ? __builtin_bit_cast(float, sw & 0xffff0000u) : __builtin_bit_cast(float, sw << 16);
              y[i] = fmaf(rb, sf - y[i], y[i]);
            }
          }
          if constexpr (HB == 2) {
            set_piece_word(word[r], pass, pack_bf16x2(y[0], y[1]));
          } else {
            if (pass == 0) keep[r] = y[0];
            else set_piece_word(word[r], 0, pack_bf16x2(keep[r], y[0]));
          }
        }
      }
      {
        // Every store instruction writes two whole rows.  The stores are non-temporal: with ordinary
        // stores the tail of out stays dirty in the last-level cache and is written back under
        // whatever kernel runs next (measured: the next call's state pass loses 30 us, this pass
        // gains 20 us)
        const TokenRows<sizeof(Piece)> rows(ob, rw.sn * 2, b * 32, n, lane);
#pragma unroll
        for (int r = 0; r < 16; ++r) rows.template store<true>(r, word[r]);
      }
    }
    if (EVEN && sh.rest < sh.hi) __syncthreads();        // the next head's images take the place of these
  }
}

// State pass, wavefront-specialised: 8 wavefronts, one workgroup per compute unit.  Wavefronts
// 0-3 ("phi") turn the K rows of tile i+1 into phi and park it in one of two LDS buffers;
// wavefronts 4-7 ("acc") park the V tile there and meanwhile accumulate S = phi^T V, z = phi^T 1
// from the other buffer (tile i).  Each SIMD hosts one wavefront of each kind, so the softmax
// arithmetic of one tile overlaps the MFMA phase of the previous one; a single barrier per tile
// swaps the buffers.
constexpr int NT1 = 512;
constexpr int OPA = 1;           // k-steps of operand read-ahead in the accumulate phase (1, 2, 3 measured alike)

// Feature of phi (order of Eq. 5) behind feature slot n (0..31) of 32-row block fb of the turned
// phi (see state_partials_ws_kernel): fb = half*(D/64) + b, jj = n/16, g' = (n%16)/8, e = n%8
//   feature = half*D/2 + g'*D/4 + 8*(2b + jj) + e.
template <int D>
__device__ __forceinline__ int turned_feature(int fb, int n) {
  const int half = fb / (D / 64), b = fb % (D / 64);
  return half * (D / 2) + ((n % 16) / 8) * (D / 4) + 8 * (2 * b + n / 16) + (n % 8);
}

// One segment of a workgroup's tile range: tiles tile0 .. tile0+nt-1 of one (b,h), whose K and V
// rows start at kb, vb and whose W~_k is wkh; the partial state goes to dst.  Every thread of the
// workgroup calls it (it contains workgroup barriers).
// CENTRE (LINATTN_FLAG_CENTRED): the phi wavefronts produce phi - 2/D, so that the fp16 rounding acts on the
// deviation from the uniform map; the accumulate wavefronts sum the columns of V from the operands they read
// anyway (a lane of a transposed V operand holds 8 tokens of one channel) and the segment's partial state is
// completed in fp32: S += (2/D) 1 (sum v)^T, z += (2/D) x the number of tokens.
template <int D, bool CENTRE>
__device__ __forceinline__ void state_segment(const uint16_t* __restrict__ kb, const uint16_t* __restrict__ vb,
                                              const uint16_t* __restrict__ wkh, float* __restrict__ dst,
                                              int tile0, int nt, int n, Rows rw) {
  using C = Cfg<D>;
  constexpr int RS = D * 2;
  constexpr int WMN = D / 64;
  constexpr int VPT = (kTile * C::CH) / 256;     // 16-byte chunks of the V tile per acc thread
  constexpr int BUF = 2 * kTile * RS;            // one buffer: turned-phi operand image, then V tile
  constexpr int FB = D / 32;                     // 32-row blocks of S over the features
  extern __shared__ uint4 smem[];
  uint4* sWA = smem;
  char* sBuf = reinterpret_cast<char*>(sWA + C::W_IMG);
  float* zred = reinterpret_cast<float*>(sBuf + 2 * BUF);      // [4][D] z of the four phi wavefronts

  const int tid = threadIdx.x, lane = tid % 64;
  const int w = __builtin_amdgcn_readfirstlane(tid / 64);
  const int role = w / 4, pw = w % 4;            // role 0: phi, role 1: acc
  const int g = lane / 32;

  {
    WImage<D> W;
    W.load(wkh, tid);
    W.write(sWA, tid);
  }
  __syncthreads();

  if (role == 0) {
    // ---- phi wavefronts ------------------------------------------------------------------
    const int prow = 32 * pw + (lane % 32);
    // selection operands: B[k = 8g+e][n] = 1 iff n == 16*jj + 8g + e
    f16x8 sel[2];
#pragma unroll
    for (int jj = 0; jj < 2; ++jj) {
      uint32_t q[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int e0 = 16 * jj + 8 * g + 2 * i;
        q[i] = ((lane % 32) == e0 ? 0x3C00u : 0u) | ((lane % 32) == e0 + 1 ? 0x3C000000u : 0u);
      }
      uint4 t; t.x = q[0]; t.y = q[1]; t.z = q[2]; t.w = q[3];
      sel[jj] = as_f16x8(t);
    }
    float zs[FB];
#pragma unroll
    for (int i = 0; i < FB; ++i) zs[i] = 0.f;
    auto load_k = [&](uint4 (&x)[C::UK], int tile) {
      const int t = tile * kTile + prow;
      const int tc = t < n ? t : (n - 1);
      const uint4* row = reinterpret_cast<const uint4*>(kb + (size_t)tc * rw.sn);
#pragma unroll
      for (int ks = 0; ks < C::UK; ++ks) x[ks] = row[2 * ks + g];
    };
    // one tile: x holds its K rows and is refilled with the tile two steps ahead as soon as the
    // projection has consumed it
    auto phi_step = [&](uint4 (&x)[C::UK], int it) {
      if (it < nt) {
        const int tile = tile0 + it;
        const bool valid = (tile * kTile + prow) < n;
        f32x16 u[C::UM];
        project<D>(x, sWA, lane, u);
        if (it + 2 < nt) load_k(x, tile + 2);
        uint32_t pk[C::NPK];
        softmax_pair<D, CENTRE>(u, valid, pk);
        // turn phi from "token per lane" to "feature slot per lane" with an MFMA against the 0/1
        // selection operands: the accumulator is then (after an exact repack to fp16) the A operand
        // of S = phi^T V with the tokens of a 16-token k-step in the order {4g..4g+3, 8+4g..8+4g+3};
        // z is the in-lane sum.  The operands go to LDS ready-made: entry (pw, fb, kb, lane).
        uint4* img = reinterpret_cast<uint4*>(sBuf + (it & 1) * BUF) + (pw * FB * 2) * 64 + lane;
#pragma unroll
        for (int fb = 0; fb < FB; ++fb) {
          const int half = fb / (D / 64), b = fb % (D / 64);
          f32x16 t;
#pragma unroll
          for (int r = 0; r < 16; ++r) t[r] = 0.f;
#pragma unroll
          for (int jj = 0; jj < 2; ++jj) {
            const int base = half * (C::LOC / 2) + 4 * (2 * b + jj);
            uint4 a; a.x = pk[base]; a.y = pk[base + 1]; a.z = pk[base + 2]; a.w = pk[base + 3];
            t = __builtin_amdgcn_mfma_f32_32x32x16_f16(as_f16x8(a), sel[jj], t, 0, 0, 0);
          }
          float zsum = 0.f;
#pragma unroll
          for (int r = 0; r < 16; ++r) zsum += t[r];
          zs[fb] += zsum;
#pragma unroll
          for (int kb = 0; kb < 2; ++kb) {
            uint4 a;
            a.x = pack_f16x2(t[8 * kb], t[8 * kb + 1]);     a.y = pack_f16x2(t[8 * kb + 2], t[8 * kb + 3]);
            a.z = pack_f16x2(t[8 * kb + 4], t[8 * kb + 5]); a.w = pack_f16x2(t[8 * kb + 6], t[8 * kb + 7]);
            img[(fb * 2 + kb) * 64] = a;
          }
        }
      }
      __syncthreads();
    };
    uint4 xa[C::UK], xc[C::UK];
    load_k(xa, tile0);
    if (nt > 1) load_k(xc, tile0 + 1);
    for (int it = 0; it <= nt; it += 2) {       // nt + 1 barriers in total, as in the acc branch
      phi_step(xa, it);
      if (it + 1 <= nt) phi_step(xc, it + 1);
    }
    // z of this wavefront's tokens: both lane groups of a slot
#pragma unroll
    for (int fb = 0; fb < FB; ++fb) {
      float lo, hi;
      pair32(zs[fb], lo, hi);
      if (g == 0) zred[pw * D + 32 * fb + lane] = lo + hi;
    }
    if constexpr (CENTRE) {
      __syncthreads();      // the two barriers of the accumulate branch's column-sum reduction
      __syncthreads();
    }
  } else {
    // ---- acc wavefronts ------------------------------------------------------------------
    const int mi = pw / 2, ni = pw % 2;
    const int atid = tid - 256;
    f32x16 s[WMN][WMN];
#pragma unroll
    for (int r = 0; r < 16; ++r)
#pragma unroll
      for (int i = 0; i < WMN; ++i)
#pragma unroll
        for (int j = 0; j < WMN; ++j) s[i][j][r] = 0.f;
    auto fblk = [&](int i) { return mi * WMN + ((WMN == 2) ? (i ^ ni) : i); };
    // (tr_offset_g4 by its definition: from its exclusive-or form the accumulate loop has 28 vector instructions fewer a tile, the phi wavefronts of its SIMD
    // fall behind, and the pass takes 294 us in place of 289 at 40 heads x 75600 x 128, 50.3 / 49.6 at 12 x 32760)
    int offB[WMN][2];
#pragma unroll
    for (int i = 0; i < WMN; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        const int r = 4 * (lane / 32) + ((lane % 16) / 4) + 8 * j;
        const int col = 32 * (ni * WMN + i) + 16 * ((lane / 16) % 2) + 4 * (lane % 4);
        offB[i][j] = r * RS + (((col / 8) ^ swz<D>(r)) * 16) + (col % 8) * 2 + kTile * RS;
      }
    auto load_v = [&](uint4 (&vr)[VPT], int tile) {
      const int t0 = tile * kTile;
#pragma unroll
      for (int i = 0; i < VPT; ++i) {
        const int idx = atid + 256 * i;
        const int r = idx / C::CH, c = idx % C::CH;
        const int tv = (t0 + r) < n ? (t0 + r) : (n - 1);
        vr[i] = ld_nt(reinterpret_cast<const uint4*>(vb + (size_t)tv * rw.sn) + c);
      }
    };
    float csum[WMN];                                 // CENTRE: column sums of V over the lane's tokens
#pragma unroll
    for (int j = 0; j < WMN; ++j) csum[j] = 0.f;
    // one step: park V tile `it` (held in vr, refilled with the tile two steps ahead), then
    // accumulate tile it-1 from the other buffer
    auto acc_step = [&](uint4 (&vr)[VPT], int it) {
      if (it < nt) {
        char* sV = sBuf + (it & 1) * BUF + kTile * RS;
#pragma unroll
        for (int i = 0; i < VPT; ++i) {
          const int idx = atid + 256 * i;
          const int rv = idx / C::CH, c = idx % C::CH;
          uint4 hv;
          hv.x = bf16x2_to_f16x2(vr[i].x); hv.y = bf16x2_to_f16x2(vr[i].y);
          hv.z = bf16x2_to_f16x2(vr[i].z); hv.w = bf16x2_to_f16x2(vr[i].w);
          *reinterpret_cast<uint4*>(sV + rv * RS + ((c ^ swz<D>(rv)) * 16)) = hv;
        }
        if (it + 2 < nt) load_v(vr, tile0 + it + 2);
      }
      if (it >= 1) {
        // operands are requested OPA k-steps before the MFMAs that use them.
        // k-step ks = tokens 16ks .. 16ks+15 = phi wavefront ks/2, half kb = ks%2 of its block.
        const char* buf = sBuf + ((it - 1) & 1) * BUF;
        const uint4* img = reinterpret_cast<const uint4*>(buf) + lane + opaque_zero();
        constexpr int KSN = kTile / 16;
        f16x8 a[KSN][WMN], b[KSN][WMN];
        auto request = [&](int kn) {
#pragma unroll
          for (int i = 0; i < WMN; ++i) a[kn][i] = as_f16x8(img[(((kn / 2) * FB + fblk(i)) * 2 + (kn % 2)) * 64]);
#pragma unroll
          for (int j = 0; j < WMN; ++j) b[kn][j] = read_tr(buf + kn * 16 * RS, offB[j][0], offB[j][1]);
        };
#pragma unroll
        for (int ks = 0; ks < OPA; ++ks) request(ks);
#pragma unroll
        for (int ks = 0; ks < KSN; ++ks) {
          if (ks + OPA < KSN) request(ks + OPA);
          __builtin_amdgcn_sched_barrier(0);
#pragma unroll
          for (int i = 0; i < WMN; ++i)
#pragma unroll
            for (int j = 0; j < WMN; ++j)
              s[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_f16(a[ks][i], b[ks][j], s[i][j], 0, 0, 0);
          if constexpr (CENTRE) {
#pragma unroll
            for (int j = 0; j < WMN; ++j) {
              const uint4 q = __builtin_bit_cast(uint4, b[ks][j]);
              csum[j] = add_pair_f16(q.x, csum[j]); csum[j] = add_pair_f16(q.y, csum[j]);
              csum[j] = add_pair_f16(q.z, csum[j]); csum[j] = add_pair_f16(q.w, csum[j]);
            }
          }
          __builtin_amdgcn_sched_barrier(0);
        }
      }
      __syncthreads();
    };
    uint4 va[VPT], vc[VPT];
    load_v(va, tile0);
    if (nt > 1) load_v(vc, tile0 + 1);
    for (int it = 0; it <= nt; it += 2) {
      acc_step(va, it);
      if (it + 1 <= nt) acc_step(vc, it + 1);
    }
    const int c = lane % 32;
    float corr[WMN];
#pragma unroll
    for (int j = 0; j < WMN; ++j) corr[j] = 0.f;
    if constexpr (CENTRE) {
      // column sums of v: the two lane groups of the wavefronts mi = 0 (mi = 1 holds the same sums), in a
      // fixed order; every step has ended with a barrier, so the tile buffers are free.  Rows past n
      // were parked as copies of row n - 1: their share is taken out again.
      float* svp = reinterpret_cast<float*>(sBuf);            // [D] sums, then [D] (2/D) x sums
#pragma unroll
      for (int j = 0; j < WMN; ++j) {
        float lo, hi;
        pair32(csum[j], lo, hi);
        if (mi == 0 && g == 0) svp[32 * (ni * WMN + j) + c] = lo + hi;
      }
      __syncthreads();
      float* svs = svp + D;
      if (atid < D) {
        const int t_hi = (tile0 + nt) * kTile;
        const int dup = t_hi > n ? t_hi - n : 0;
        float t = svp[atid];
        if (dup > 0) {
          const uint32_t last = bf16x2_to_f16x2((uint32_t)vb[(size_t)(n - 1) * rw.sn + atid]) & 0xffffu;
          t -= (float)dup * (float)__builtin_bit_cast(_Float16, (uint16_t)last);
        }
        svs[atid] = t * (2.0f / D);
      }
      __syncthreads();
#pragma unroll
      for (int j = 0; j < WMN; ++j) corr[j] = svs[32 * (ni * WMN + j) + c];
    }
#pragma unroll
    for (int i = 0; i < WMN; ++i)
#pragma unroll
      for (int j = 0; j < WMN; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int f = turned_feature<D>(fblk(i), 8 * (r / 4) + 4 * g + (r % 4));
          dst[f * D + 32 * (ni * WMN + j) + c] = CENTRE ? s[i][j][r] + corr[j] : s[i][j][r];
        }
  }
  // z: the four phi wavefronts, in a fixed order (CENTRE: plus 2/D per token of the segment)
  __syncthreads();
  if (tid < D) {
    float zv = (zred[tid] + zred[2 * D + tid]) + (zred[D + tid] + zred[3 * D + tid]);
    if constexpr (CENTRE) {
      const int t_lo = tile0 * kTile, t_hi = (tile0 + nt) * kTile < n ? (tile0 + nt) * kTile : n;
      zv += (2.0f / D) * (float)(t_hi - t_lo);
    }
    dst[D * D + turned_feature<D>(tid / 32, tid % 32)] = zv;
  }
  __syncthreads();                               // the next segment reuses every LDS region
}

// Grid: Split::G workgroups; workgroup g takes the tiles [lo(g), lo(g+1)) of the call's (b,h)-major
// tile sequence, one segment per head it touches (at most two).
template <int D, bool CENTRE>
__global__ __launch_bounds__(NT1) void state_partials_ws_kernel(const uint16_t* __restrict__ k, const uint16_t* __restrict__ v,
                                                                const uint16_t* __restrict__ wk, float* __restrict__ partials,
                                                                int H, int n, Split sp, Rows rw) {
  const int g = blockIdx.x;
  long long lo = split_lo(sp, g);
  const long long hi = split_lo(sp, g + 1);
  while (lo < hi) {
    const int bh = split_head(sp, lo);
    const long long head0 = (long long)bh * sp.ntile;
    const long long seg_hi = hi < head0 + sp.ntile ? hi : head0 + sp.ntile;
    const int slot = g - split_owner(sp, head0);
    state_segment<D, CENTRE>(k + head_base(rw, bh, H), v + head_base(rw, bh, H), wk + (size_t)(bh % H) * D * (D / 2),
                     partials + ((size_t)bh * sp.PS + slot) * (size_t)(D + 1) * D,
                     (int)(lo - head0), (int)(seg_hi - lo), n, rw);
    lo = seg_hi;
  }
}

template <int D>
constexpr size_t state_ws_smem() { return sizeof(uint4) * Cfg<D>::W_IMG + 4 * (size_t)kTile * D * 2 + 4 * D * sizeof(float); }

template <int D>
constexpr size_t apply_smem(bool sum) {
  // the images, then z and a few reduction slots of the prologue, then (sum) the state
  return sizeof(uint4) * (Cfg<D>::W_IMG + ApplyLayout<D>::KS * ApplyLayout<D>::MBZ * 64) + (D + 64) * sizeof(float)
       + (sum ? (size_t)(D + 1) * D * sizeof(float) : 0);
}

}  // namespace

namespace {
template <int D, bool CENTRE>
hipError_t run_state_ws(const void* k, const void* v, const void* wk, float* partials, const Plan& p, hipStream_t s) {
  hipError_t e;
  if ((e = set_smem_once<state_partials_ws_kernel<D, CENTRE>>(state_ws_smem<D>())) != hipSuccess) return e;
  state_partials_ws_kernel<D, CENTRE><<<dim3(p.split.G), dim3(NT1), state_ws_smem<D>(), s>>>(
      (const uint16_t*)k, (const uint16_t*)v, (const uint16_t*)wk, partials, p.H, p.n, p.split, p.rows);
  return hipGetLastError();
}
}  // namespace

hipError_t launch_state_partials_bf16(const void* k, const void* v, const void* wk, float* partials,
                                      const Plan& p, hipStream_t s) {
  if (p.d == 128)
    return p.centred ? run_state_ws<128, true>(k, v, wk, partials, p, s) : run_state_ws<128, false>(k, v, wk, partials, p, s);
  return p.centred ? run_state_ws<64, true>(k, v, wk, partials, p, s) : run_state_ws<64, false>(k, v, wk, partials, p, s);
}

namespace {

// 8 wavefronts to a workgroup, one workgroup per compute unit: a unit is small enough for an even deal.  12 where the call is so short that they
// save a round, since few rounds are bound by the latency of each.  Rounds with 8 / 12, and us: 1 head x 75600 x 128 2 / 1, 14.5 / 12.9, with blend
// 19.4 / 17.2; 5 x 15000 x 128 2 / 1, 14.6 / 13.2; 7 x 20000 x 64 3 / 2, 10.3 / 10.3, with blend 14.6 / 13.9; but 12 x 8190 x 128 2 / 2, 15.5 / 15.4;
// 26 x 2222 x 64 1 / 1, 7.2 / 7.7; 3 x 500 x 128 1 / 1, 9.7 / 11.7; 4 x 1000 x 64 1 / 1, 8.0 / 8.8; 12 x 32760 x 128 6 / 5, with blend 67 / 73,
// ReLU 36.7 / 37.7.
// The costs of the deal lose least, among 960 sets of them, over 355 calls of 1 to 255 heads with every form timed.  Calls, head by head / evenly, us:
// 153 heads x 763 x 128 47.0 / 50.0 (3 rounds for 153 compute units, 2 for all), 40 x 20000 x 128 179.9 / 181.9, 30 x 17550 x 64 61.1 / 62.4; but 12 x 32760 x
// 128 99.8 / 97.6, 160 x 4000 x 128 158.9 / 154.5, 40 x 75600 x 128 631 / 626.  The blended pass of width 128, whose rounds are the longest, gains
// more: 138 x 1563 89.6 / 79.9, 154 x 1102 73.9 / 69.1.
// 12 wavefronts with an even deal, two prologues around one round each, pay where a head's last unit is short and 8 would be dealt evenly too, in the
// blended pass of width 128 also where they would not: evenly with 8 / with 12, last unit of up to 8 of 12 blocks, 6 x 32283 56.4 / 54.2, 30 x 6203
// 60.4 / 57.2, 46 x 3931 61.5 / 57.8; of 9 or more, 24 x 7995 58.3 / 61.5, with blend 144 x 1051 65.9 / 68.8; head by head with 8 / evenly with 12, with
// blend 155 x 1019 69.5 / 66.2, but without 136 x 827 47.1 / 48.8.
template <int D, bool BLEND>
constexpr DealCost kApplyCost = D == 128 && BLEND ? DealCost{3} : DealCost{4, 2, 5, 240};
template <int D, bool BLEND, int KIND, bool SUM, int NW, bool EVEN>
hipError_t run_apply_as(const void* q, const void* wq, const float* partials, float* state, void* out, const void* blend_in,
                           const float* blend_r, const Plan& p, const Split& deal, hipStream_t s) {
  hipError_t e;
  constexpr size_t smem = apply_smem<D>(SUM);
  if ((e = set_smem_once<apply_bf16_kernel<D, BLEND, KIND, SUM, NW, EVEN>>(smem)) != hipSuccess) return e;
  apply_bf16_kernel<D, BLEND, KIND, SUM, NW, EVEN><<<grid_of(deal), 64 * NW, smem, s>>>(
      (const uint16_t*)q, (const uint16_t*)wq, partials, state, (uint16_t*)out, (const uint16_t*)blend_in, blend_r, p.H, p.n, deal, p.split, p.rows);
  return hipGetLastError();
}
template <int D, bool BLEND, int KIND, bool SUM, int NW>
hipError_t run_apply_waves(const void* q, const void* wq, const float* partials, float* state, void* out, const void* blend_in,
                           const float* blend_r, const Plan& p, const Split& deal, hipStream_t s) {
  if constexpr (apply_even<SUM>)
    if (!deal.share) return run_apply_as<D, BLEND, KIND, SUM, NW, true>(q, wq, partials, state, out, blend_in, blend_r, p, deal, s);
  return run_apply_as<D, BLEND, KIND, SUM, NW, false>(q, wq, partials, state, out, blend_in, blend_r, p, deal, s);
}
template <int D, bool BLEND, int KIND, bool SUM>
hipError_t run_apply(const void* q, const void* wq, const float* partials, float* state, void* out, const void* blend_in,
                     const float* blend_r, const Plan& p, hipStream_t s) {
  const int blocks = (p.n + 31) / 32;
  // Every workgroup of a pass that sums reads all of its head's partials.  A call, us, units of 8 / 4 / 2: width 64, 24 heads x 500 (4 partials) 11.5 / 11.3 / 12.4, 48
  // x 500 13.6 / 14.1 / 14.1, 4 x 500 10.1 / 9.5 / 9.4, 24 x 768 (6) 13.4 / 13.9 / 13.9, 12 x 768 11.9 / 11.5 / 11.6, and one tile 32 x 100 8.7 / 8.8 / 9.2; width 128, 128 x 100 (1)
  // 18.2 / 18.1 / 22.8, 12 x 100 14.4 / 14.4 / 14.5, 4 x 100 14.2 / 14.4 / 14.0, 64 x 256 (2) 22.7 / 20.8 / 26.1, 4 x 256 17.0 / 15.1 / 14.6, 128 x 256 23.6 / 24.2.
  const UnitLimits most = SUM ? UnitLimits{240, D == 128 ? 16 : p.split.ntile > 1 ? 64 : 0} : UnitLimits();
  const int read = SUM ? p.split.PS : 1;
  const Split d8 = make_deal_of_blocks(p.BH, blocks, 8, kApplyCost<D, BLEND>, apply_even<SUM>, read, most);
  if constexpr (!SUM || kSumSlots<D> * kTile > 8 * 32) {   // (at most 8 blocks a head otherwise)
    const bool even12 = apply_even<SUM> && ((D == 128 && BLEND) || !d8.share) && (blocks + 11) % 12 < 8;
    const Split d12 = make_deal_of_blocks(p.BH, blocks, 12, kApplyCost<D, BLEND>, even12, read, most);
    const int r8 = split_rounds(d8);
    if (r8 <= 3 && split_rounds(d12) < r8)
      return run_apply_waves<D, BLEND, KIND, SUM, 12>(q, wq, partials, state, out, blend_in, blend_r, p, d12, s);
  }
  return run_apply_waves<D, BLEND, KIND, SUM, 8>(q, wq, partials, state, out, blend_in, blend_r, p, d8, s);
}

template <int D, bool SUM>
hipError_t pick_apply(const void* q, const void* wq, const float* partials, float* state, void* out,
                      const void* blend_in, const float* blend_r, const Plan& p, hipStream_t s) {
  if (p.kind == kPhiRelu)      // the dispatch has refused a blend with this map
    return run_apply<D, false, kPhiRelu, SUM>(q, nullptr, partials, state, out, nullptr, nullptr, p, s);
  return blend_in ? run_apply<D, true, kPhiHedgehog, SUM>(q, wq, partials, state, out, blend_in, blend_r, p, s)
                  : run_apply<D, false, kPhiHedgehog, SUM>(q, wq, partials, state, out, nullptr, nullptr, p, s);
}

}  // namespace

// Short calls, where a launch is a fifth of the time: the query pass sums the partials itself, up to six tiles a head at width 64 and two at 128 (at least
// as many as partials), and up to eight where the heads are few or so many that each has few partials.  Every workgroup of a head, up to
// sixteen (four at 128), reads all of them.  A call, reduction launched / summed here, with the units that each takes, us: width 64, 1 head x 100 9.7 / 8.0, 32 x 300
// 12.4 / 10.7, 64 x 500 16.0 / 15.2, 12 x 768 12.1 / 11.5, 32 x 768 14.7 / 14.5, but 48 x 640 15.1 / 15.5; seven and eight tiles 4 x 1000 10.9 / 10.7, 8 x 1000 11.5 / 11.8, 12 x
// 1000 12.0 / 12.7, 48 x 900 17.8 / 18.8, 64 x 1000 18.4 / 18.4, 100 x 1000 22.2 / 19.5, 200 x 1024 33.9 / 30.3.  Width 128: 1 x 100 14.2 / 13.7, 128 x 100 25.4 /
// 18.1, 48 x 256 22.7 / 19.7, 200 x 256 31.4 / 26.1.  With units of eight blocks: nine to sixteen tiles 12 x 2000 x 64 15.1 / 17.1, 128 x 2000 x 64 33.1 / 31.4, three
// or four at 128, a state of 66 KB each, 4 x 500 17.9 / 18.5, 128 x 500 32.8 / 30.1.
bool sum_in_apply(const Plan& p) {
  if (p.d == 128) return p.split.ntile <= kSumSlots<128>;
  return p.split.ntile <= 6 || (p.split.ntile <= kSumSlots<64> && (p.BH <= 4 || p.split.T > 2 * kSlots));
}

hipError_t launch_apply_bf16(const void* q, const void* wq, const float* partials, float* state, void* out,
                             const void* blend_in, const float* blend_r, const Plan& p, hipStream_t s) {
  if (sum_in_apply(p))
    return p.d == 128 ? pick_apply<128, true>(q, wq, partials, state, out, blend_in, blend_r, p, s)
                      : pick_apply<64, true>(q, wq, partials, state, out, blend_in, blend_r, p, s);
  return p.d == 128 ? pick_apply<128, false>(q, wq, partials, state, out, blend_in, blend_r, p, s)
                    : pick_apply<64, false>(q, wq, partials, state, out, blend_in, blend_r, p, s);
}

}  // namespace linattn
