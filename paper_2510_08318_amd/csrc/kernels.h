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
// Parts of dL/dr beyond one per workgroup of the bf16 query side: the fp32-arithmetic gradient kernel may have more workgroups.
constexpr int kDrSlack = 1024;

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
  // The index arithmetic runs in the prologue of every workgroup.  It has no division: as 64-bit divisions (a hundred dependent
  // instructions each, thousands with their copies, which the instruction cache has to bring in) it took 0.5 us of a state pass and
  // 1.3 us of a kernel that calls next_share.
  int share;        // not 0: G = B*H*share and no workgroup has tiles of two heads (next_share)
  int blocks;       // make_deal_of_blocks: 32-token blocks to a unit, the first wavefronts of the workgroup one each
  int quot, rem;    // T / G, T % G
  float inv_G, per_T, inv_ntile;      // 1 / G, G / T, 1 / ntile
};
inline void finish_split(Split& s) {
  s.quot = (int)(s.T / s.G); s.rem = (int)(s.T % s.G);
  s.inv_G = 1.0f / (float)s.G; s.per_T = (float)s.G / (float)s.T; s.inv_ntile = 1.0f / (float)s.ntile;
}
// floor(g T / G).  The quotient of g * rem (below 2^18: rem is 0 where G exceeds 512) is estimated in fp32 to within one and corrected.
__host__ __device__ inline long long split_lo(const Split& s, int g) {
  const int x = g * s.rem;
  int q = (int)((float)x * s.inv_G);
  if (q * s.G > x) --q;
  if ((q + 1) * s.G <= x) ++q;
  return (long long)g * s.quot + q;
}
// the head that tile x belongs to (the estimate is off by at most one: at most 65535 heads)
__host__ __device__ inline int split_head(const Split& s, long long x) {
  int h = (int)((float)x * s.inv_ntile);
  if ((long long)h * s.ntile > x) --h;
  if ((long long)(h + 1) * s.ntile <= x) ++h;
  return h;
}
// the workgroup whose range holds tile x
__host__ __device__ inline int split_owner(const Split& s, long long x) {
  int g = (int)((float)x * s.per_T);
  g = g < s.G ? g : s.G - 1;
  if (split_lo(s, g) > x) --g;
  if (g + 1 < s.G && split_lo(s, g + 1) <= x) ++g;
  return g;
}

// A workgroup's share of one head: units u, u + step, .. below end (head-relative).  The workgroups that have units of this head
// alone take them in turn, so that they sweep the head together (in one piece each, the query pass of 40 heads x 75600 x 128 took 340
// us where it takes 327); those at its ends, which have units of two heads, take theirs in one piece.
// for (Share sh = first_share(s, blockIdx.x, blockIdx.y); sh.there; sh = next_share(s, blockIdx.x, sh)) visits the one or two shares of
// a workgroup.
struct Share {
  bool there;
  int bh, u, step, end;
  long long rest, hi;      // the workgroup's tiles beyond this share
};
__host__ __device__ inline Share next_share(const Split& s, int g, const Share& prev) {
  Share r = prev;
  r.there = prev.rest < prev.hi;
  if (!r.there) return r;
  const long long lo = prev.rest, hi = prev.hi;
  r.bh = split_head(s, lo);
  const long long head0 = (long long)r.bh * s.ntile, head1 = head0 + s.ntile;
  if (hi <= head1 && lo == split_lo(s, g)) {
    int g0 = split_owner(s, head0), g1 = split_owner(s, head1 - 1);
    if (split_lo(s, g0) < head0) ++g0;
    if (split_lo(s, g1 + 1) > head1) --g1;
    r.u = (int)(split_lo(s, g0) - head0) + (g - g0);
    r.step = g1 - g0 + 1;
    r.end = (int)(split_lo(s, g1 + 1) - head0);
    r.rest = hi;
  } else {
    const long long stop = hi < head1 ? hi : head1;
    r.u = (int)(lo - head0);
    r.step = 1;
    r.end = (int)(stop - head0);
    r.rest = stop;
  }
  return r;
}
// gx, gy: the workgroup's place in the grid that grid_of(s) is.  (With one grid dimension, and the head divided out of it, a pass of 8 us takes 0.4
// us longer.)
__host__ __device__ inline Share head_share(const Split& s, int gx, int gy) {      // where s.share is known not to be 0
  Share r{};
  r.there = true;
  r.bh = gy; r.u = gx; r.step = s.share; r.end = s.ntile;
  return r;
}
__host__ __device__ inline Share first_share(const Split& s, int gx, int gy) {
  if (s.share) return head_share(s, gx, gy);
  Share r{};
  r.rest = split_lo(s, gx); r.hi = split_lo(s, gx + 1);
  return next_share(s, gx, r);
}
// the most units a workgroup gets
inline int split_rounds(const Split& s) {
  return s.share ? (s.ntile + s.share - 1) / s.share : (int)((s.T + s.G - 1) / s.G);
}
inline dim3 grid_of(const Split& s) { return s.share ? dim3(s.share, s.G / s.share) : dim3(s.G); }

// The deal of a kernel that builds a head's operand images in its prologue: `per_head` units of each head to one workgroup per compute
// unit (one per head where there are more heads), either the same number of workgroups to every head (each then has one head) or the
// units of all heads evenly (a workgroup may then have the end of one head and the start of the next, and builds images twice).
// may_even = false: always the first form, for kernels without a loop over a workgroup's heads.
// What the forms cost, in eighths of a round in which every compute unit has a unit: a prologue; a round with units for a part of the compute
// units, `fixed` and in proportion to that part up to `full` of them, at least `least` (the memory system serves fewer faster; the defaults,
// 8 for any part, where arithmetic bounds a round).
struct DealCost {
  int prologue, fixed = 8, least = 8, full = kCUs;
};
inline Split make_deal(int BH, int per_head, DealCost cost, bool may_even = true) {
  Split s{};
  s.ntile = per_head;
  s.T = (long long)BH * per_head;
  s.PS = 1;
  s.share = kCUs / BH < per_head ? (BH < kCUs ? kCUs / BH : 1) : per_head;
  s.G = BH * s.share;
  if (may_even && s.T > kCUs && BH < kCUs) {
    auto round = [&](long long units) {                    // times full
      const long long t = cost.fixed * cost.full + (8 - cost.fixed) * (units < cost.full ? units : cost.full);
      return t > cost.least * cost.full ? t : (long long)cost.least * cost.full;
    };
    const long long rounds = (per_head + s.share - 1) / s.share, whole = (s.T - 1) / kCUs;
    const long long by_head = (rounds - 1) * round(s.G) + round(BH * (per_head - (rounds - 1) * s.share)) + cost.prologue * cost.full;
    const long long even = whole * round(kCUs) + round(s.T - whole * kCUs) + 2 * cost.prologue * cost.full;
    if (even < by_head) { s.G = kCUs; s.share = 0; }
  }
  finish_split(s);
  return s;
}

// The deal of `blocks` 32-token blocks a head to workgroups of `waves` wavefronts, a block to a wavefront.  Units are of four or two blocks where every unit
// gets a compute unit of its own: in so short a call most of the chip is empty, its time is the latency of a block, and a wavefront that shares its SIMD
// (or the LDS) with fewer others is done with it sooner.  Us, units of 8 / 4 / 2: bf16 query pass 4 heads x 1000 x 64 7.2 / 6.0 / 5.85, 3 x
// 300 x 128 9.3 / 7.3 / 6.7, ReLU 4 x 2000 x 64 5.0 / 4.1; fp32 arithmetic, 2 x 1024 x 64: query pass 8.9 / 7.4 / 6.8, gradients 15.1 + 12.8 / 12.2 + 10.7 / 10.2 +
// 10.4.
// More workgroups also bring more copies of a head's state into the eight L2s, one to each XCD (workgroups are dealt to them in turn) or to each workgroup
// of a head that has fewer.  With many heads of few blocks that costs more than the smaller unit saves: a call, bf16, 48 heads x 300 x 128 25.2 / 23.1 / 23.9 (96
// copies more for units of two), 32 x 300 x 128 22.7 / 21.0 / 21.5 (64), 16 x 300 x 128 20.0 / 18.3 / 18.2 (32); bf16 tensors in fp32 arithmetic 64 x 128 x 128 26.5 /
// 26.4 / 27.8 (64), 16 x 256 x 128 25.3 / 22.6 / 22.4 (32).  Units of four pay wherever they fit.  A query pass that sums reads `partials` states a copy and has limits of its
// own (run_apply).
constexpr int kXCDs = 8;
struct UnitLimits {
  long long four = 1 << 30, two = 48;      // the most states more than with the next larger unit, for units of four and of two
};
constexpr UnitLimits kNoUnitLimits{1 << 30, 1 << 30};
inline Split make_deal_of_blocks(int BH, int blocks, int waves, DealCost cost, bool may_even = true, int partials = 1, UnitLimits most = UnitLimits()) {
  auto states = [&](int u) {
    const int per_head = (blocks + u - 1) / u;
    return (long long)BH * (per_head < kXCDs ? per_head : kXCDs) * partials;
  };
  int unit = waves;
  for (int u = 4; u >= 2; u /= 2) {
    if ((long long)BH * ((blocks + u - 1) / u) > kCUs || states(u) - states(unit) > (u == 4 ? most.four : most.two)) break;
    unit = u;
  }
  Split s = make_deal(BH, (blocks + unit - 1) / unit, cost, may_even);
  s.blocks = unit;
  return s;
}
// A wavefront's blocks of a share: first, stride and end (of `all` blocks a head); a wavefront beyond the unit's blocks has none.
struct Blocks {
  int first, stride, end;
};
__host__ __device__ inline Blocks blocks_of(const Split& s, const Share& sh, int w, int all) {
  Blocks r;
  r.end = all < sh.end * s.blocks ? all : sh.end * s.blocks;
  r.stride = sh.step * s.blocks;
  r.first = w < s.blocks ? sh.u * s.blocks + w : r.end;
  return r;
}

// How one call is cut into workgroups and where its scratch regions sit in the workspace.
struct Plan {
  int B, H, n, d;
  int kind;         // kPhiHedgehog or kPhiRelu (set by the dispatch, not by make_plan)
  bool bf16_math;    // bf16 arithmetic (set by the dispatch)
  bool bf16_storage; // the fp32-arithmetic kernels read and write bf16 tensors (LINATTN_BF16_F32MATH)
  bool centred;      // LINATTN_FLAG_CENTRED (set by the dispatch): phi minus its mean in the sums over tokens, centred operand images
  int BH;
  Rows rows;        // memory layout of the token tensors
  Split split;      // state passes (and the weighted one of the fp32-arithmetic backward)
  int P;            // split-n factor (partials per (b,h)) of the query-side backward and of dW~
  size_t state_elems;     // (d+1)*d
  size_t off_partials;    // fp32 [BH][max(P, split.PS)][(d+1)*d]
  size_t off_state;       // fp32 [BH][(d+1)*d]   (used when the caller gave no state buffer)
  size_t fwd_bytes;       // end of the two regions above: all the scratch a forward call touches
  // backward only
  size_t off_dstate;      // fp32 [BH][(d+1)*d]   dS, dz
  size_t off_centre;      // bf16 backward: fp32 [BH][3][d] (mean value row vbar; the other two rows unused), then
                          // [BH][P][d+8] per-workgroup column sums of dO/den (d) and the sum of -delta/den (1)
  size_t off_drpart;      // fp32 [BH][P] + [kDrSlack]: per-workgroup parts of dL/dr (mixed attention, Eq. 6)
  size_t off_dwpart;      // fp32 [BH][P][d*d/2] partial dW~_q, then as many of dW~_k, in room for 256 / BH of them a head (weight gradients only)
  size_t du_bytes;        // bytes of one dL/du region (0 in bf16 mode: dW~ is accumulated where du is made)
  size_t off_du_q;        // dL/du of the query side (weight gradients, fp32 arithmetic only): fp32 [BH][n][d/2]
  size_t off_du_k;        // the same for the key side
  size_t bytes_no_wgrads; // workspace needed by forward and by backward without dW~
  size_t total_bytes;
};

// Pure host arithmetic; returns false if the shape is unsupported or overflows.
// total_bytes includes the weight-gradient regions, bytes_no_wgrads does not.
bool make_plan(int B, int H, int n, int d, int dtype, int layout, Plan* p);
// The workgroups of the state passes.  The split of make_plan, by which the workspace is sized, gives every workgroup the same number of tiles, and some
// of them tiles of two heads: two prologues, two partial states, the loads in flight drained between them.  Head by head no workgroup has two, and
// no head more partials; it is taken where the busiest workgroup has no more tiles for it, or, of four and more in the bf16 Hedgehog pass, one more.  Evenly /
// head by head, us a pass: 12 heads x 4133 x 64 (2 tiles either way) 8.6 / 7.55, x 128 14.9 / 13.5, 30 x 3000 x 64 (3) 10.4 / 9.4, 7 x 20000 x
// 128 (5) 25.4 / 21.9, 30 x 17550 x 64 (17 / 18) 29.4 / 27.7, 12 x 32760 x 128 (12 / 13) 50.9 / 48.8.  Of 364 forward calls of 5 to 200 heads with one tile more, all
// 28 of four tiles gain (0.1 to 4 us of 23 to 51), those of five to ten 0.9 to 2.7 us on average, of three at width 128 6 of 12 (12 x 8190 loses 0.75 of 40); but ReLU
// 12 x 32760 x 128 44.2 / 47.3, a forward call of fp32 tensors there 271 / 275.
// Where the even split gives no workgroup tiles of two heads there is nothing to save, and the head-wise one, if its workgroups to a head are odd, ends the
// pass later at width 64: those with a tile more, the last of each head, then lie on all XCDs and not on one of them.  A forward call, us, evenly / head by head:
// 13 heads x 2560 x 64 16.9 / 18.3, 12 x 2816 17.1 / 18.3, 48 x 768 16.0 / 17.1, 26 x 1280 16.7 / 17.9, 5 x 6656 17.1 / 17.6; but even numbers 30 x 1152 17.7 / 16.4, 52 x
// 640 16.2 / 15.0, 9 x 3712 17.7 / 17.1, and at width 128 48 x 768 29.6 / 29.0, 13 x 2560 29.2 / 29.2.
inline void deal_state_pass(Plan* p) {
  const int m = p->BH < kSlots ? kSlots / p->BH : 1, G = p->split.G;
  if (m > p->split.ntile) return;
  const bool hedgehog = p->kind == kPhiHedgehog && p->bf16_math;
  const int even = split_rounds(p->split), by_head = (p->split.ntile + m - 1) / m;
  if (by_head > even + (even >= 4 && hedgehog)) return;
  if (p->d == 64 && hedgehog && m % 2 && p->BH < G) {
    // head h starts at workgroup ceil(h G / BH), which starts at its first tile if (-h G mod BH) tiles-a-head are below G
    int a = G, b = p->BH;
    while (b) { const int r = a % b; a = b; b = r; }
    if ((long long)(p->BH - a) * p->split.ntile < G) return;
  }
  p->split.G = p->BH * m;
  p->split.PS = m;
  finish_split(p->split);
}

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

// Whether the bf16 backward stores dq and dv non-temporally (the ReLU map: dq and dk, dv never): where the three gradients take more than half of
// the last-level cache (256 MB).  Left dirty there, large ones are written back under the kernels that follow and displace the rows these
// read; small ones serve whoever reads them next.  dk of the Hedgehog map is always non-temporal: written last together with dv, it makes room for
// the next kernel's rows, which is worth what its reader loses.  Us, all non-temporal / dk alone / none: a training step and then one pass over each
// gradient, 12 heads x 4133 x 64 (6 MB a gradient) 69.1 / 65.3 / 64.1, 12 x 8190 x 128 (25 MB) 160 / 155 / 153; the step alone, whose forward is then the
// next to run, 50.1 / 50.0 / 50.7 and 124 / 122 / 124.  All / none: 12 x 16000 (49 MB) 231 / 234 and 175 / 184; 12 x 32760 (100 MB) 423 / 428 and 324 / 340;
// 40 x 20000 (205 MB) 809 / 812 and 587 / 603.  ReLU, dq and dk / none: 12 x 4133 x 64 65.6 / 62.8 and 47.4 / 47.8; 12 x 8190 151 / 147 and 117 / 119; 12 x
// 16000 209 / 210 and 158 / 165; 12 x 32760 374 / 377 and 279 / 284, with dv too 382 and 280 (relu_bwd_k 87 -> 94); 40 x 20000 728 / 737 and 509 / 519.
inline bool stream_gradients(const Plan& p) { return (size_t)p.BH * p.n * p.d * 2 * 3 > ((size_t)128 << 20); }

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
// dL/dr of the mixed attention: *dr = the count parts summed in a fixed order if 0 <= *r <= 1, else 0 (Eq. 6, clipped r); off where dr is null.
struct DrSum {
  const float* part;
  int count;
  const float* r;
  float* dr;
};
// Fixed-order sum of the partials into the exported state layout [BH][d+1][d] fp32, and (one workgroup more) dL/dr.
hipError_t launch_state_reduce(const float* partials, float* state, const Plan& p, const DrSum& dr, hipStream_t s);
// The same for the partials of the bf16 forward state pass (slots per head follow Plan::split).
hipError_t launch_state_reduce_split(const float* partials, float* state, const Plan& p, const DrSum& dr, hipStream_t s);
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
hipError_t launch_bwd_bf16_stream(const BwdArgs& a, const Plan& p, hipStream_t s);      // its form with non-temporal gradients
hipError_t launch_bwd_f32(const BwdArgs& a, const Plan& p, hipStream_t s);
hipError_t launch_relu_bwd_bf16(const BwdArgs& a, const Plan& p, hipStream_t s);

}  // namespace linattn
