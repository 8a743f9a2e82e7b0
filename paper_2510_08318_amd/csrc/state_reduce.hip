// Cross-workgroup reductions in a fixed order (no atomics, so the results are bitwise
// reproducible): the split-n partial states, and the weight gradient dW~ = sum x^T du.
#include "kernels.h"

namespace linattn {
namespace {

// The parts of dL/dr (Eq. 6) summed in a fixed order by one workgroup of 256; zero outside the clip's range [0, 1].
__device__ __forceinline__ void sum_dr(const DrSum& d) {
  __shared__ float red[256];
  float acc = 0.f;
  for (int i = threadIdx.x; i < d.count; i += 256) acc += d.part[i];
  red[threadIdx.x] = acc;
  __syncthreads();
  for (int m = 128; m >= 1; m >>= 1) {
    if ((int)threadIdx.x < m) red[threadIdx.x] += red[threadIdx.x + m];
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    const float rv = *d.r;
    *d.dr = (rv >= 0.f && rv <= 1.f) ? red[0] : 0.f;
  }
}

// state[bh][e] = sum over the slots p of partials[bh][p][e], four adjacent elements per thread.  GROUPS threads share an element:
// each sums a contiguous share of the slots, eight loads in flight and added pairwise, and the shares are combined pairwise
// through LDS; the order is fixed by the shape, so the result is reproducible, and the longest chain of roundings is short
// (256 slots: 2 + 3 + 4 levels where one running sum has 256).
// SPLIT: the slots of head bh are those of the workgroups whose tile ranges touch it (Split), of sp.PS allocated; otherwise P.
// Workgroup (columns, 0), if there is one, takes dL/dr (as a launch of its own 4.7 us).
template <int GROUPS, bool SPLIT>
__global__ __launch_bounds__(256) void state_reduce_kernel(const float4* __restrict__ partials, float4* __restrict__ state,
                                                           Split sp, int P, int elems4, int columns, DrSum dr) {
  constexpr int EL = 256 / GROUPS;
  if ((int)blockIdx.x == columns) {
    if (blockIdx.y == 0) sum_dr(dr);
    return;
  }
  __shared__ float4 red[GROUPS > 1 ? 256 : 1];
  const int el = threadIdx.x % EL, grp = threadIdx.x / EL;
  const int e = blockIdx.x * EL + el;
  const int bh = blockIdx.y;
  int cnt = P;
  if constexpr (SPLIT) {
    __shared__ int s_cnt;
    if (threadIdx.x == 0)
      s_cnt = split_owner(sp, (long long)(bh + 1) * sp.ntile - 1) - split_owner(sp, (long long)bh * sp.ntile) + 1;
    __syncthreads();
    cnt = s_cnt;
  }
  const int p_lo = cnt * grp / GROUPS, p_hi = cnt * (grp + 1) / GROUPS;
  const float4* src = partials + (size_t)bh * (SPLIT ? sp.PS : P) * elems4 + (e < elems4 ? e : 0);
  auto add = [](float4 a, float4 b) { return make_float4(a.x + b.x, a.y + b.y, a.z + b.z, a.w + b.w); };
  const float4 zero = make_float4(0.f, 0.f, 0.f, 0.f);
  float4 acc = zero;
  auto sum8 = [&](const float4 (&t)[8]) {
    acc = add(acc, add(add(add(t[0], t[1]), add(t[2], t[3])), add(add(t[4], t[5]), add(t[6], t[7]))));
  };
  int p = p_lo;
  for (; p + 8 <= p_hi; p += 8) {
    float4 t[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) t[i] = src[(size_t)(p + i) * elems4];
    sum8(t);
  }
  if (p + 4 <= p_hi) {
    float4 t[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) t[i] = src[(size_t)(p + i) * elems4];
    acc = add(acc, add(add(t[0], t[1]), add(t[2], t[3])));
    p += 4;
  }
  for (; p < p_hi; ++p) acc = add(acc, src[(size_t)p * elems4]);
  if constexpr (GROUPS > 1) {
    red[threadIdx.x] = acc;
#pragma unroll
    for (int m = GROUPS / 2; m >= 1; m >>= 1) {
      __syncthreads();
      if (grp < m) red[threadIdx.x] = add(red[threadIdx.x], red[threadIdx.x + m * EL]);
    }
    acc = red[threadIdx.x];
  }
  if (grp == 0 && e < elems4) state[(size_t)bh * elems4 + e] = acc;
}

// ---- dW~ = sum_{b, i} x_i^T du_i ------------------------------------------------------------
// dw[h][e] = sum_b sum_p part[(b*H + h)][p][e], b then p ascending.
// blockIdx.z picks one of up to two (partials, output, partials per (b,h)) triples; a triple without output is skipped.
__global__ __launch_bounds__(256) void dw_reduce_kernel(const float* __restrict__ part0, float* __restrict__ dw0, int P0,
                                                        const float* __restrict__ part1, float* __restrict__ dw1, int P1,
                                                        int B, int H, int elems) {
  const float* part = blockIdx.z ? part1 : part0;
  float* dw = blockIdx.z ? dw1 : dw0;
  const int P = blockIdx.z ? P1 : P0;
  const int e = blockIdx.x * 256 + threadIdx.x, h = blockIdx.y;
  if (e >= elems || dw == nullptr) return;
  // eight partials are requested together and added pairwise (a missing one adds 0): one memory latency per eight terms
  float acc = 0.f;
  for (int b = 0; b < B; ++b) {
    const float* src = part + ((size_t)(b * H + h) * P) * elems + e;
    for (int p0 = 0; p0 < P; p0 += 8) {
      float v[8];
#pragma unroll
      for (int j = 0; j < 8; ++j) v[j] = p0 + j < P ? src[(size_t)(p0 + j) * elems] : 0.f;
      acc += ((v[0] + v[1]) + (v[2] + v[3])) + ((v[4] + v[5]) + (v[6] + v[7]));
    }
  }
  dw[(size_t)h * elems + e] = acc;
}

}  // namespace

namespace {
template <int GROUPS, bool SPLIT>
void run_state_reduce(const float* partials, float* state, const Plan& p, const DrSum& dr, hipStream_t s) {
  const int elems4 = (int)(p.state_elems / 4);      // (d+1) d is a multiple of 4; both buffers are 16-byte aligned
  constexpr int EL = 256 / GROUPS;
  const int columns = (elems4 + EL - 1) / EL;
  state_reduce_kernel<GROUPS, SPLIT><<<dim3(columns + (dr.dr != nullptr), p.BH), 256, 0, s>>>(
      reinterpret_cast<const float4*>(partials), reinterpret_cast<float4*>(state), p.split, p.P, elems4, columns, dr);
}
// One thread per four elements while its slots fit one batch of loads, more threads with more slots.  Measured after a fresh
// write of the partials, with about 4 us of event overhead, one / four / sixteen threads, width 128: 40 heads of 8 slots 7.9 /
// 8.8 / 15.6 us; 20 of 14: 8.0 / 7.7 / 10.4; 12 of 22: 7.8 / 7.4 / 9.1; 4 of 64: 8.6 / 7.6 / 7.5; 2 of 128: 11.9 / 8.3 / 7.3;
// 1 of 256: 18.0 / 9.1 / 7.5.
template <bool SPLIT>
hipError_t state_reduce_any(const float* partials, float* state, const Plan& p, const DrSum& dr, hipStream_t s) {
  const int slots = SPLIT ? p.split.PS : p.P;
  if (slots <= 8) run_state_reduce<1, SPLIT>(partials, state, p, dr, s);
  else if (slots <= 32) run_state_reduce<4, SPLIT>(partials, state, p, dr, s);
  else run_state_reduce<16, SPLIT>(partials, state, p, dr, s);
  return hipGetLastError();
}
}  // namespace

hipError_t launch_state_reduce(const float* partials, float* state, const Plan& p, const DrSum& dr, hipStream_t s) {
  return state_reduce_any<false>(partials, state, p, dr, s);
}

hipError_t launch_state_reduce_split(const float* partials, float* state, const Plan& p, const DrSum& dr, hipStream_t s) {
  return state_reduce_any<true>(partials, state, p, dr, s);
}

hipError_t launch_dw_reduce2(const float* part0, float* dw0, int P0, const float* part1, float* dw1, int P1, const Plan& p, hipStream_t s) {
  const int elems = p.d * (p.d / 2);
  dw_reduce_kernel<<<dim3((elems + 255) / 256, p.H, 2), 256, 0, s>>>(part0, dw0, P0, part1, dw1, P1, p.B, p.H, elems);
  return hipGetLastError();
}

}  // namespace linattn
