// Shared declarations of the backward sweeps (gfx950).
#pragma once

#include "sweep.hpp"

namespace infcl {

constexpr int kBwdBN = kSweepBN;  // swept rows per tile

// One side of the backward: own rows get a gradient, the other modality is swept.
struct BwdSide {
  const void* own;    // [b, d] rows whose gradient is produced
  const void* swept;  // [b, d] the other modality
  const float* lse_own;     // [b]  natural-log log-sum-exp of the own side
  const float* lse2_swept;  // [b]  log-sum-exp of the swept side times log2(e)
  const float* ell_own;     // [b]  r_i - x_ii of the own side
  const float* ell_swept;   // [b]
  void* dOwn;               // [own_end - own_off, d], by own row - own_off: fp32, or with gdt = 1 the
                            // input's 16-bit type
};

struct BwdParams {
  BwdSide side[2];  // image rows owned, text rows owned
  int64_t b, d;
  const float* scale;
  const float* udiag;  // [b]  <img_i, txt_i>
  const float* dloss;  // device scalar or nullptr (= 1)
  int64_t own_off, own_end;  // own rows [own_off, own_end) of both sides (a shard; 0 and b for the whole batch)
  double* ds_part;           // [gridDim.x]
  const float* g16;          // fp16 inputs: block maxima for the scale of G' (g16_scale)
  int gdt;                   // gradient type, which chooses the kernel instantiation: 0 fp32, 1 16-bit
  // Work split (plan_bwd): of the 2 nblk row blocks (image side first) the
  // first nfull are swept whole, one workgroup each; each of the others is
  // swept by ns workgroups, a contiguous range of whole groups of gran tiles each, whose unscaled
  // fp32 sums go to part[(block - nfull) ns + k][rows][d] for bwd_reduce.
  int nblk, nfull, ns, gran;
  float* part;
};

// A workgroup's share of the plan: its side, row block and swept rows
// [row0, row0 + rows), row0 a multiple of the tile, and with ns > 1 the slot
// of its partial sums (nullptr: final gradients).  The sweeps count tiles and
// rows from row0.
struct BwdTask {
  int sd, rb, row0, rows;
  float* part;
};
__device__ __forceinline__ BwdTask bwd_task(const BwdParams& p, int bm_d) {
  // (readfirstlane: the compiler divides on the vector unit and would keep the
  // wave-uniform results in vector registers for the whole sweep)
  BwdTask t;
  const int wg = blockIdx.x;
  int blk = wg;
  t.row0 = 0;
  t.rows = (int)p.b;  // at most 2^30
  t.part = nullptr;
  if (p.ns > 1 && wg >= p.nfull) {
    const uint32_t ntile = ((uint32_t)p.b + kBwdBN - 1) / kBwdBN;
    const uint32_t r = wg - p.nfull, ns = p.ns;
    const uint32_t q = __builtin_amdgcn_readfirstlane(r / ns), k = r - q * ns;
    blk = p.nfull + (int)q;
    const uint32_t g = p.gran, nunit = (ntile + g - 1) / g;
    // nunit (k + 1) <= 2^31: ntile <= 2^25, k < ns <= 64
    const uint32_t t0 = __builtin_amdgcn_readfirstlane(nunit * k / ns * g);
    const uint32_t t1 = __builtin_amdgcn_readfirstlane(nunit * (k + 1) / ns * g);
    t.row0 = (int)t0 * kBwdBN;
    t.rows = (t1 >= ntile ? (int)p.b : (int)t1 * kBwdBN) - t.row0;
    t.part = p.part + (int64_t)r * bm_d;
  }
  t.sd = blk >= p.nblk ? 1 : 0;
  t.rb = t.sd ? blk - p.nblk : blk;
  return t;
}

// How a backward call is split over workgroups (see plan_bwd in bwd.hip).
struct BwdPlan {
  int bm;           // own rows per row block
  int nblk;         // row blocks per side
  int nfull, ns;    // blocks swept whole; parts of each other block
  int gran;         // tiles that a part's range is a multiple of (what the sweep's loop unrolls)
  int nwg;          // workgroups
  size_t part_bytes;  // partial sums and dscale partials (0 when nothing is split)
};

constexpr int kWideBM = 64;  // own rows per workgroup of the wide-row sweeps

// fp16 inputs: G' is rounded to fp16 after multiplication by a power of two
// alpha, and the fp32 accumulators are multiplied by 1/alpha at the end (exact
// scaling, the role loss scaling plays in mixed-precision training): without
// it the G' of a well-separated batch (loss near zero) lies below fp16's
// smallest subnormal, 2^-24, and the gradients would vanish.  alpha maps a
// bound B on every |G'| to at most 2^14 (fp16's largest finite value is about
// 2^16): off the diagonal P^r_ij <= 1 - P^r_ii = -expm1(-l^r_i) and
// P^c_ij <= -expm1(-l^c_j), and |G'_ii| <= -expm1(-l^r_i) - expm1(-l^c_i), so
// B = max_i(-expm1(-l^r_i)) + max_j(-expm1(-l^c_j)).
// bwd_prep leaves the two maxima of each of its kPrepBlocks blocks; every wave
// that needs alpha reduces them itself (one pair per lane).
constexpr int kPrepBlocks = 64;
// TOP: alpha B lies in [2^(TOP-1), 2^TOP).  fp32 inputs scale G' too, for its
// bf16 parts (the third is 2^-17 of a weight or less), and take TOP = 0: with
// bf16's exponents there is nothing to gain above 1, and larger weights would
// take the sums of large entries past the largest float.
template <int TOP = 14>
__device__ __forceinline__ int g16_exponent(const float* part) {
  const int lane = __lane_id();
  float mr = part[2 * lane], mc = part[2 * lane + 1];
#pragma unroll
  for (int k = 1; k < 64; k <<= 1) {
    mr = fmaxf(mr, shfl_xor(mr, k));
    mc = fmaxf(mc, shfl_xor(mc, k));
  }
  const float B = mr + mc;
  int k = 0;
  if (B > 0.f) {
    int e;
    (void)frexpf(B, &e);  // B = m 2^e, m in [0.5, 1): alpha B = m 2^TOP < 2^TOP
    k = TOP - e;
    k = k > 100 ? 100 : k;
  }
  return __builtin_amdgcn_readfirstlane(k);
}

// Gradient element type of a sweep: fp32, or with G16 the 16-bit input type
// (fp16 with F16, else bf16), rounded to nearest even from the fp32 gradient
// when stored.  The fp32 value is materialised first: the compiler would
// otherwise fuse the final scaling into an fp16 conversion (a mixed-precision
// multiply that rounds the exact product once), whose result differs from a
// cast of the fp32 gradient by one unit where that lands on a tie.
template <bool G16, bool F16>
struct GradOut {
  using type = float;
  static __device__ __forceinline__ float cvt(float v) { return v; }
};
template <bool F16>
struct GradOut<true, F16> {
  using type = __bf16;
  static __device__ __forceinline__ __bf16 cvt(float v) {
    asm volatile("" : "+v"(v));
    return to16<F16>(v);
  }
};

}  // namespace infcl
