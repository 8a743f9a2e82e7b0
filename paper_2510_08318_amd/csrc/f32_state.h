// Sum over tokens of phi(x_j)^T y_j and of phi(x_j), in fp32 arithmetic on the bf16 matrix cores (f32_split.h): the state pass of
// the forward (x = k, y = v) and, with per-token weights, the sums dS and dz of the backward (x = q, y = dO).
#pragma once
#include "f32_split.h"
#include "f32_plain.h"

namespace linattn {
namespace f32 {

// 8 wavefronts, one workgroup per compute unit, 128-token tiles.  Wavefronts 0-3 ("phi") turn the rows of tile i+1 into phi and
// split it while wavefronts 4-7 ("acc") contract tile i; then phi is parked in LDS as
// three row-major bf16 tiles, read back by transposing reads.  The three tiles (96 KB at d = 128) leave no room for a second
// buffer, so two barriers per tile fence the parking; everything else of one role runs beside the other's.  y reaches the
// acc wavefronts straight from memory where it is stored as fp32 (a lane holds 8 tokens of one column and splits them itself;
// its three tiles would not fit beside phi's) and through an LDS tile where it is stored as bf16.
// z (sum of phi) is summed in the phi wavefronts' lanes, which own their tokens, and combined once per segment.
// WEIGHTED: weights[bh][t] = {a, b}: S = sum a phi^T y, z = sum b phi.
template <int D, int KIND, typename T, bool WEIGHTED>
struct StatePass {
  using C = Cfg<D>;
  static constexpr int NX = kPieces<T>;
  static constexpr int NP = KIND == kPhiRelu && NX == 1 && !WEIGHTED ? 1 : 3;     // pieces of phi (max(x, 0) of a bf16 is a bf16)
  static constexpr int RS = D * 2;
  // blocks of S of an acc wavefront, FW feature blocks x CW column blocks: y through LDS wants a square (fewest operand reads), y
  // from memory one column block, whose y then is read and split by one wavefront only
  static constexpr int FW = NX == 1 ? D / 64 : D / 64 * (D / 64), CW = NX == 1 ? D / 64 : 1;
  static constexpr int PT = kTile * RS;                            // bytes of one piece tile
  static constexpr int W_BYTES = KIND == kPhiRelu ? 0 : NX * C::W_IMG * 16;
  static constexpr int Y_BYTES = NX == 1 ? PT : 0;
  static constexpr size_t SMEM = (size_t)W_BYTES + NP * PT + Y_BYTES + (4 * D + 4) * sizeof(float);

  // Tiles tile0 .. tile0+nt-1 of one (b,h); xb, yb: its first rows; every thread of the workgroup calls it.
  static __device__ __forceinline__ void segment(const T* __restrict__ xb, const T* __restrict__ yb, const T* __restrict__ wh,
                                                 const float2* __restrict__ weights, float* __restrict__ dst, int tile0, int nt,
                                                 int n, Rows rw) {
    extern __shared__ uint4 smem[];
    uint4* sW = smem;
    char* sPhi = reinterpret_cast<char*>(smem) + W_BYTES;
    char* sY = sPhi + NP * PT;
    float* zred = reinterpret_cast<float*>(sY + Y_BYTES);          // [4][D]
    int* sPlain = reinterpret_cast<int*>(zred + 4 * D);            // [4] the acc wavefront's sum is not finite
    const int tid = threadIdx.x, lane = tid % 64;
    const int w = __builtin_amdgcn_readfirstlane(tid / 64);
    const int role = w / 4, pw = w % 4, g = lane / 32, c = lane % 32;
    if constexpr (KIND == kPhiHedgehog) {
      build_w_pieces<D, T, NT8>(wh, sW, tid);
      __syncthreads();
    }
    if (role == 0) {
      const int prow = 32 * pw + c;
      RowOctets<D, T> x;
      float2 wt;
      // a tile's rows are requested while the previous one is worked on: fp32 rows half before and half behind the parking (the
      // pieces of phi take their registers in between)
      constexpr int EARLY = NX == 1 ? D / 16 : D / 32;
      auto row_of = [&](int it) {
        const int t = (tile0 + (it < nt ? it : nt - 1)) * kTile + prow;
        return t < n ? t : n - 1;
      };
      auto load_early = [&](int it) {
        const int tc = row_of(it);
        x.template load<0, EARLY>(xb + (size_t)tc * rw.sn, g);
        if constexpr (WEIGHTED) wt = weights[tc];
      };
      auto load_late = [&](int it) { x.template load<EARLY, D / 16>(xb + (size_t)row_of(it) * rw.sn, g); };
      float z[D / 2];
#pragma unroll
      for (int i = 0; i < D / 2; ++i) z[i] = 0.f;
      load_early(0);
      load_late(0);
      for (int it = 0; it < nt; ++it) {
        const bool valid = (tile0 + it) * kTile + prow < n;
        float f[D / 2];
        phi_octets<D, KIND, T>(x, sW, lane, f);
        // odd tiles are summed negated (see the head of f32_split.h)
        const float wa = (valid ? (WEIGHTED ? wt.x : 1.f) : 0.f) * ((tile0 + it) % 2 ? -1.f : 1.f), wb = valid ? (WEIGHTED ? wt.y : 1.f) : 0.f;
        load_early(it + 1);
        uint4 pk[D / 16][3];
#pragma unroll
        for (int ks = 0; ks < D / 16; ++ks) {
          float v[8];
#pragma unroll
          for (int e = 0; e < 8; ++e) {
            const int i = 8 * ks + e;
            z[i] = fmaf(f[i], wb, z[i]);
            v[e] = f[i] * wa;
          }
          split8(v, pk[ks]);
        }
        __syncthreads();                                           // the previous tile has been read
        // (addresses worked out here, from a lane index the optimiser cannot hoist: held across the loop they end up in scratch
        // memory, and a wait for a scratch load waits for the rows requested before it as well)
        const int lrow = 32 * pw + (lane + opaque_zero()) % 32;
        const int psw = swz<D>(lrow);
        char* rowp = sPhi + lrow * RS;
#pragma unroll
        for (int ks = 0; ks < D / 16; ++ks) {
          const int chunk = phi_feature<D, KIND>(ks, g) / 8;
#pragma unroll
          for (int p = 0; p < NP; ++p) *reinterpret_cast<uint4*>(rowp + p * PT + ((chunk ^ psw) * 16)) = pk[ks][p];
        }
        load_late(it + 1);
        __syncthreads();
      }
#pragma unroll
      for (int ks = 0; ks < D / 16; ++ks)
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const float sum = half_wave_sum(z[8 * ks + e]);
          if (c == 0) zred[pw * D + phi_feature<D, KIND>(ks, g) + e] = sum;
        }
    } else {
      const int fb0 = NX == 1 ? FW * (pw / 2) : FW == 4 ? 0 : pw / 2;            // first feature block
      const int cb0 = NX == 1 ? CW * (pw % 2) : FW == 4 ? pw : pw % 2;           // first column block
      // a tile is summed by itself and then added, odd ones subtracted: the piece products then round a sum over 128 tokens and not
      // the whole segment's (12 heads of 32 760 tokens, fp32 tensors: error of out 7.4e-7 with one running sum, 4.1e-7 with
      // tiles added, 2.4e-7 with the sign alternating; scalar FMAs 3.9e-7)
      f32x16 s[FW][CW];
      auto clear = [](f32x16 (&t)[FW][CW]) {
#pragma unroll
        for (int i = 0; i < FW; ++i)
#pragma unroll
          for (int j = 0; j < CW; ++j) t[i][j] = zero16();
      };
      auto add_tile = [&](const f32x16 (&t)[FW][CW], int it) {
        const float sign = (tile0 + it) % 2 ? -1.f : 1.f;
#pragma unroll
        for (int i = 0; i < FW; ++i)
#pragma unroll
          for (int j = 0; j < CW; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) s[i][j][r] = fmaf(t[i][j][r], sign, s[i][j][r]);
      };
      clear(s);
      int offA[FW][2];
#pragma unroll
      for (int i = 0; i < FW; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) offA[i][j] = tr_offset<D>(32 * (fb0 + i), lane, j);
      auto phi_operand = [&](int ks, int i, uint4 (&a)[NP]) {
#pragma unroll
        for (int p = 0; p < NP; ++p)
          a[p] = __builtin_bit_cast(uint4, read_tr(sPhi + p * PT + ks * 16 * RS, offA[i][0], offA[i][1]));
      };
      constexpr int KSN = kTile / 16;
      if constexpr (NX == 1) {
        // y through LDS
        constexpr int YPT = kTile * C::CH / 256;
        const int atid = tid - 256;
        int offB[CW][2];
#pragma unroll
        for (int j = 0; j < CW; ++j)
#pragma unroll
          for (int h = 0; h < 2; ++h) offB[j][h] = tr_offset<D>(32 * (cb0 + j), lane, h);
        uint4 y[YPT];
        auto load_y = [&](int it) {
          const int t0 = (tile0 + (it < nt ? it : nt - 1)) * kTile;
#pragma unroll
          for (int i = 0; i < YPT; ++i) {
            const int idx = atid + 256 * i, r = idx / C::CH, ch = idx % C::CH;
            const int t = t0 + r < n ? t0 + r : n - 1;
            y[i] = ld_nt(reinterpret_cast<const uint4*>(yb + (size_t)t * rw.sn) + ch);
          }
        };
        auto contract = [&](int it) {
          const int z0 = opaque_zero();
          f32x16 t[FW][CW];
          clear(t);
#pragma unroll
          for (int ks = 0; ks < KSN; ++ks) {
            uint4 a[FW][NP], b[CW][1];
#pragma unroll
            for (int i = 0; i < FW; ++i) phi_operand(ks, i, a[i]);
#pragma unroll
            for (int j = 0; j < CW; ++j)
              b[j][0] = __builtin_bit_cast(uint4, read_tr(sY + ks * 16 * RS + z0, offB[j][0], offB[j][1]));
            mfma_pieces<NP, 1>(a, b, t);
          }
          add_tile(t, it);
        };
        load_y(0);
        for (int it = 0; it < nt; ++it) {
          __syncthreads();
#pragma unroll
          for (int i = 0; i < YPT; ++i) {
            const int idx = atid + 256 * i, r = idx / C::CH, ch = idx % C::CH;
            *reinterpret_cast<uint4*>(sY + r * RS + ((ch ^ swz<D>(r)) * 16)) = y[i];
          }
          load_y(it + 1);
          __syncthreads();
          contract(it);
        }
      } else {
        // y from memory: k-step kg of the segment (16 tokens), the lane's 8 tokens of its column, AHEAD k-steps ahead
        constexpr int AHEAD = 4;
        static_assert(KSN % AHEAD == 0, "a k-step keeps its slot");
        float y[AHEAD][8];
        const uint32_t sn4 = (uint32_t)rw.sn * 4u;
        const uint32_t col4 = (uint32_t)(32 * cb0 + c) * 4u;
        auto load_y = [&](float (&slot)[8], int kg) {
          int row0 = tile0 * kTile + 16 * kg;
          row0 = row0 < n ? row0 : n - 1;
          const int last = n - 1 - row0 < 15 ? n - 1 - row0 : 15;    // rows past n read row n - 1: their phi is zero
          const char* base = reinterpret_cast<const char*>(yb + (size_t)row0 * rw.sn);
          const uint32_t last4 = (uint32_t)last * sn4 + col4;
#pragma unroll
          for (int e = 0; e < 8; ++e) {
            const uint32_t off = (uint32_t)(8 * g + e) * sn4 + col4;
            slot[e] = *reinterpret_cast<const float*>(base + (off < last4 ? off : last4));
          }
        };
        auto contract = [&](int it) {
          f32x16 t[FW][CW];
          clear(t);
          // fenced: left to itself the compiler moves the requests for k-step ks + AHEAD down to their use
#pragma unroll
          for (int ks = 0; ks < KSN; ++ks) {
            uint4 b[1][NX];
            split8(y[ks % AHEAD], b[0]);
            load_y(y[ks % AHEAD], it * KSN + ks + AHEAD);
            __builtin_amdgcn_sched_barrier(0);
            constexpr int PAIR = FW < 2 ? 1 : 2;
#pragma unroll
            for (int i = 0; i < FW; i += PAIR) {
              uint4 a[PAIR][NP];
#pragma unroll
              for (int q = 0; q < PAIR; ++q) phi_operand(ks, i + q, a[q]);
              mfma_pieces<NP, NX>(a, b, reinterpret_cast<f32x16(&)[PAIR][1]>(t[i]));
            }
            __builtin_amdgcn_sched_barrier(0);
          }
          add_tile(t, it);
        };
#pragma unroll
        for (int i = 0; i < AHEAD; ++i) load_y(y[i], i);
        for (int it = 0; it < nt; ++it) {
          __syncthreads();
          __syncthreads();
          contract(it);
        }
      }
      // a y that does not split makes its column NaN or Inf; so does, for both halves of the Hedgehog map, an x: one row of a block
      // tells (ReLU: an x that does not split makes its feature's row so)
      float chk = 0.f;
#pragma unroll
      for (int i = 0; i < FW; ++i)
#pragma unroll
        for (int r = 0; r < (KIND == kPhiRelu ? 16 : 1); ++r)
#pragma unroll
          for (int j = 0; j < CW; ++j) chk = fmaf(s[i][j][r], 0.f, chk);
      const bool bad = __any(chk != chk);
      if (lane == 0) sPlain[pw] = bad;
#pragma unroll
      for (int i = 0; i < FW; ++i)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          float* row = dst + (32 * (fb0 + i) + 8 * (r / 4) + 4 * g + (r % 4)) * D + 32 * cb0 + c;
#pragma unroll
          for (int j = 0; j < CW; ++j) row[32 * j] = s[i][j][r];
        }
    }
    __syncthreads();
    if (tid < D) dst[D * D + tid] = (zred[tid] + zred[2 * D + tid]) + (zred[D + tid] + zred[3 * D + tid]);
    const int4 bad4 = *reinterpret_cast<const int4*>(sPlain);
    const bool plain = __builtin_amdgcn_readfirstlane((bad4.x | bad4.y) | (bad4.z | bad4.w)) != 0;       // the same in every wavefront
    if (__builtin_expect(plain, 0)) __threadfence();                                    // what is stored above is written again, by other wavefronts
    __syncthreads();                                               // the next segment reuses every LDS region
    if (__builtin_expect(plain, 0)) {
      const int t1 = (tile0 + nt) * kTile;
      Plain<D, KIND, T>::template state<WEIGHTED>(xb, yb, wh, weights, dst, tile0 * kTile, t1 < n ? t1 : n, rw.sn,
                                                    reinterpret_cast<float*>(sPhi), w, lane);
    }
  }
};

// Grid: Split::G workgroups, each a contiguous range of the call's tiles (at most two heads), as in state_partials_ws_kernel.
// weights: [BH][n] (WEIGHTED).
template <int D, int KIND, typename T, bool WEIGHTED>
__global__ __launch_bounds__(NT8) void state_f32_kernel(const T* __restrict__ x, const T* __restrict__ y, const T* __restrict__ wx,
                                                        const float2* __restrict__ weights, float* __restrict__ partials,
                                                        int H, int n, Split sp, Rows rw) {
  const int gi = blockIdx.x;
  long long lo = split_lo(sp, gi);
  const long long hi = split_lo(sp, gi + 1);
  while (lo < hi) {
    const int bh = split_head(sp, lo);
    const long long head0 = (long long)bh * sp.ntile;
    const long long seg_hi = hi < head0 + sp.ntile ? hi : head0 + sp.ntile;
    const int slot = gi - split_owner(sp, head0);
    StatePass<D, KIND, T, WEIGHTED>::segment(x + head_base(rw, bh, H), y + head_base(rw, bh, H), wx + (size_t)(bh % H) * D * (D / 2),
                                             WEIGHTED ? weights + (size_t)bh * n : nullptr,
                                             partials + ((size_t)bh * sp.PS + slot) * (size_t)(D + 1) * D,
                                             (int)(lo - head0), (int)(seg_hi - lo), n, rw);
    lo = seg_hi;
  }
}

template <int D, int KIND, typename T, bool WEIGHTED>
hipError_t run_state_pass(const void* x, const void* y, const void* wx, const float2* weights, float* partials, const Plan& p, hipStream_t s) {
  constexpr size_t smem = StatePass<D, KIND, T, WEIGHTED>::SMEM;
  const hipError_t e = set_smem_once<state_f32_kernel<D, KIND, T, WEIGHTED>>(smem);
  if (e != hipSuccess) return e;
  state_f32_kernel<D, KIND, T, WEIGHTED><<<dim3(p.split.G), NT8, smem, s>>>((const T*)x, (const T*)y, (const T*)wx, weights, partials,
                                                                           p.H, p.n, p.split, p.rows);
  return hipGetLastError();
}

}  // namespace f32
}  // namespace linattn
