// Internal interface between the host dispatch (api.cpp) and the gfx950 kernels.
// Nothing here is exported from the shared library.
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>
#include <atomic>

namespace linattn {

// Tokens a workgroup of the bf16 kernels consumes per iteration (4 waves x 32 tokens).
constexpr int kTile = 128;
// Workgroup slots the split-n plan aims to fill: one resident workgroup per compute unit.
constexpr int kSlots = 256;
// Compute units of the gfx950 parts this library targets (MI355X / MI350X).
constexpr int kCUs = 256;
// Feature maps (the values of LINATTN_PHI_*): Eq. 5, and the weight-free phi(x) = max(x, 0) of the
// kernel-function ablation.  The ReLU map can give phi(q) . z = 0, so its denominator carries
// kReluEps.
constexpr int kPhiHedgehog = 1, kPhiRelu = 2;
constexpr float kReluEps = 1e-6f;
// Workgroups (= partial sums) of the streaming dot product sum(dout * s) of the mixed attention's dL/dr.
constexpr int kDotParts = 1024;

// Where the rows of q, k, v, out (and dout, dq, dk, dv) sit in memory, in elements: element
// (b, h, t, c) is at b*sb + h*sh + t*sn + c.  [B,H,n,d]: sb = H*n*d, sh = n*d, sn = d;
// [B,n,H,d] (heads interleaved per token, what a transformer block's projection emits):
// sb = n*H*d, sh = d, sn = H*d.
struct Rows {
  size_t sb, sh, sn;
};
__host__ __device__ inline size_t head_base(const Rows& r, int bh, int H) {
  return (size_t)(bh / H) * r.sb + (size_t)(bh % H) * r.sh;
}

// Split of the bf16 state pass: the T = B*H*ntile 128-token tiles of a call, in (b,h)-major order,
// are dealt to G workgroups in contiguous ranges [lo(g), lo(g+1)), lo(g) = floor(g*T/G), so that
// every compute unit gets the same share whatever B*H is (a per-head split leaves
// 256 mod B*H units idle).  T/G <= ntile, so a range touches at most two heads; a workgroup
// writes one partial state per head it touches, into slot g - owner(first tile of the head).
struct Split {
  int G;            // workgroups
  int ntile;        // tiles per (b,h)
  long long T;      // tiles in all
  int PS;           // partial slots per (b,h) (the largest number of workgroups touching one head)
  bool small;       // T * G < 2^31: the index arithmetic fits 32 bits (a 64-bit division is a hundred dependent instructions, in
                    // the prologue of every workgroup)
};
// a * b / c, all positive
__host__ __device__ inline long long split_muldiv(const Split& s, long long a, long long b, long long c) {
  if (s.small) return (long long)((unsigned)a * (unsigned)b / (unsigned)c);
  return a * b / c;
}
__host__ __device__ inline long long split_lo(const Split& s, int g) { return split_muldiv(s, g, s.T, s.G); }
// the head that tile x belongs to
__host__ __device__ inline int split_head(const Split& s, long long x) {
  return s.small ? (int)((unsigned)x / (unsigned)s.ntile) : (int)(x / s.ntile);
}
// the workgroup whose range holds tile x
__host__ __device__ inline int split_owner(const Split& s, long long x) {
  int g = (int)split_muldiv(s, x, s.G, s.T);
  while (g + 1 < s.G && split_lo(s, g + 1) <= x) ++g;
  while (g > 0 && split_lo(s, g) > x) --g;
  return g;
}

// How one call is cut into workgroups and where its scratch regions sit in the workspace.
struct Plan {
  int B, H, n, d;
  int kind;         // kPhiHedgehog or kPhiRelu (set by the dispatch, not by make_plan)
  bool bf16_storage; // the fp32-arithmetic kernels read and write bf16 tensors (LINATTN_BF16_F32MATH)
  bool centred;      // LINATTN_FLAG_CENTRED (set by the dispatch): phi minus its mean in the sums over tokens, centred operand images
  int BH;
  Rows rows;        // memory layout of the token tensors
  Split split;      // state passes (and the weighted one of the fp32-arithmetic backward)
  int P;            // split-n factor (partials per (b,h)) of the query-side backward and of dW~
  int QP;           // workgroups per (b,h) of the bf16 query pass
  size_t state_elems;     // (d+1)*d
  size_t off_partials;    // fp32 [BH][max(P, split.PS)][(d+1)*d]
  size_t off_state;       // fp32 [BH][(d+1)*d]   (used when the caller gave no state buffer)
  size_t fwd_bytes;       // end of the two regions above: all the scratch a forward call touches
  // backward only
  int KP;                 // workgroups per (b,h) of the passes with 8 wavefronts, each on its own 32-token blocks
  size_t off_dstate;      // fp32 [BH][(d+1)*d]   dS, dz
  size_t off_centre;      // bf16 backward: fp32 [BH][3][d] (mean value row vbar; the other two rows unused), then
                          // [BH][P][d+8] per-workgroup column sums of dO/den (d) and the sum of -delta/den (1)
  size_t off_drpart;      // fp32 [BH][P] + [kDotParts]: per-workgroup parts of dL/dr (mixed attention, Eq. 6)
  size_t off_dwpart;      // fp32 [BH][P][d*d/2] partial dW~_q, then [BH][max(P, KP)][d*d/2] partial dW~_k (weight gradients only)
  size_t du_bytes;        // bytes of one dL/du region (0 in bf16 mode: dW~ is accumulated where du is made)
  size_t off_du_q;        // dL/du of the query side (weight gradients, fp32 arithmetic only): fp32 [BH][n][d/2]
  size_t off_du_k;        // the same for the key side
  size_t bytes_no_wgrads; // workspace needed by forward and by backward without dW~
  size_t total_bytes;
};

// Pure host arithmetic; returns false if the shape is unsupported or overflows.
// total_bytes includes the weight-gradient regions, bytes_no_wgrads does not.
bool make_plan(int B, int H, int n, int d, int dtype, int layout, Plan* p);

// Everything one backward call touches (device pointers; workspace regions already resolved).
struct BwdArgs {
  const void *q, *k, *v, *dout, *wq, *wk;
  void *dq, *dk, *dv;
  const float* state;     // [BH][d+1][d] from the forward
  float *dwq, *dwk;       // nullable
  float *partials, *dstate, *dw_part, *du_q, *du_k;
  float *vbar, *cs_part;   // Plan::off_centre
  // mixed attention (Eq. 6): softmax-branch output, the layer's r, dL/dr; all null when off
  const void* blend_in;
  const float* blend_r;
  float* blend_dr;
  float* dr_part;
};

// A kernel instantiation as a value, for launch code shared by several.
template <auto Kernel>
struct KernelTag {
  static constexpr auto value = Kernel;
};

// Raises a kernel's dynamic-LDS limit to `bytes`, once per kernel instantiation and device: the
// attribute call is a driver call, and the launchers sit on the enqueue path of every step.
template <auto Kernel>
hipError_t set_smem_once(size_t bytes) {
  static std::atomic<uint64_t> done{0};
  int dev = -1;
  const bool tracked = hipGetDevice(&dev) == hipSuccess && dev >= 0 && dev < 64;
  if (tracked && (done.load(std::memory_order_acquire) >> dev & 1)) return hipSuccess;
  const hipError_t e = hipFuncSetAttribute((const void*)Kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
  if (e == hipSuccess && tracked) done.fetch_or(uint64_t(1) << dev, std::memory_order_release);
  return e;
}

// ---- forward launchers (enqueue only) ---------------------------------------------------
// phi(K) fused with the split-n partial state (Eq. 5 + the two sums of Eq. 3).
hipError_t launch_state_partials_f32(const void* k, const void* v, const void* wk, float* partials,
                                     const Plan& p, hipStream_t s);
hipError_t launch_state_partials_bf16(const void* k, const void* v, const void* wk, float* partials,
                                      const Plan& p, hipStream_t s);
// The same for the ReLU map (bf16); partial slots per head follow Plan::split as well.
hipError_t launch_relu_state_bf16(const void* k, const void* v, float* partials, const Plan& p, hipStream_t s);
// Fixed-order sum of the partials into the exported state layout [BH][d+1][d] fp32.
hipError_t launch_state_reduce(const float* partials, float* state, const Plan& p, hipStream_t s);
// The same for the partials of the bf16 forward state pass (slots per head follow Plan::split).
hipError_t launch_state_reduce_split(const float* partials, float* state, const Plan& p, hipStream_t s);
// phi(Q) S / (phi(Q) . z) and the store of out (Eq. 3, right-hand side).
hipError_t launch_apply_f32(const void* q, const void* wq, const float* state, void* out,
                            const void* blend_in, const float* blend_r, const Plan& p, hipStream_t s);
// bf16: from the state, or (sum_in_apply) from the partials of the state pass, writing the state as well.
bool sum_in_apply(const Plan& p);
hipError_t launch_apply_bf16(const void* q, const void* wq, const float* partials, float* state, void* out,
                             const void* blend_in, const float* blend_r, const Plan& p, hipStream_t s);

// ---- backward launchers (enqueue only) --------------------------------------------------
// dw0[h][e] = sum over b, then over the P0 splits, of part0[(b*H+h)][p][e], and the same for the second triple in one launch; a
// triple whose output is null is skipped.
hipError_t launch_dw_reduce2(const float* part0, float* dw0, int P0, const float* part1, float* dw1, int P1, const Plan& p, hipStream_t s);
hipError_t launch_bwd_bf16(const BwdArgs& a, const Plan& p, hipStream_t s);
hipError_t launch_bwd_f32(const BwdArgs& a, const Plan& p, hipStream_t s);
hipError_t launch_relu_bwd_bf16(const BwdArgs& a, const Plan& p, hipStream_t s);
// part[0 .. kDotParts-1] = partial sums of sum_i a[i] * (b[i] - vbar[bh(i)][channel(i)]) over two bf16 token tensors in the
// plan's layout; vbar fp32 [BH][d].
hipError_t launch_dot_centred_bf16(const void* a, const void* b, const float* vbar, float* part, const Plan& p, hipStream_t s);
// dr = sum of the count parts in a fixed order if 0 <= *r <= 1, else 0 (Eq. 6, clipped r).
hipError_t launch_dr_reduce(const float* part, int count, const float* r, float* dr, hipStream_t s);

}  // namespace linattn
