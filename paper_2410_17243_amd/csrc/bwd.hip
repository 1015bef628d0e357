// Backward sweeps of the tiled symmetric InfoNCE loss (gfx950).
//
// What is computed (paper Sec. 3.1, Eq. 6-8, completed for both halves of the
// symmetric loss, the text side and the scale; the appendix's in-GPU backward
// algorithm recomputes every tile from the saved log-sum-exp vectors):
//   dL/dx_ij = (1/2b) (P^r_ij + P^c_ij) - (1/b) delta_ij,
//   P^r_ij = exp(x_ij - r_i),  P^c_ij = exp(x_ij - c_j),
//   dimg = k * G' txt,   dtxt = k * G'^T img,
//   with G' = P^r + P^c off the diagonal, G'_ii = expm1(-(r_i-x_ii)) + expm1(-(c_i-x_ii)),
//   k = dloss * s / (2b), and
//   ds = dloss/(2b) * sum_{i != j} [P^r_ij (u_ij - u_ii) + P^c_ij (u_ij - u_jj)],  u = <img_i, txt_j>.
//
// Design (differs from the paper's single pass that read-modify-writes the text
// gradient tile in HBM for every tile): one kernel, two kinds of row block.
// A block that "owns" image rows keeps their dimg rows in registers and sweeps
// all text rows; a block of text rows swaps the roles.  The similarity tile is
// recomputed for each side, but no gradient leaves the registers before the
// sweep ends and no atomics are used.  A workgroup owns 128 rows (32 per wave)
// and sweeps 32-row tiles of the other side.  Per tile and wave:
//   GEMM1  S^T(32 swept x 32 own) = swept_tile * own^T   (own operand held in
//          registers for the whole sweep, swept rows read from LDS with a
//          row permutation that makes the accumulator usable as GEMM2's operand)
//   G'     two exp2 per entry (log2 domain), the diagonal from expm1 terms
//   GEMM2  the four waves' G' blocks are exchanged through LDS and each wave
//          multiplies all 128 own rows by its quarter of the features.
// This file: 16-bit inputs, d = 128 to 512; wider rows are in bwd_wide.hip,
// fp32 inputs in bwd_f32.hip.
//
// Memory pipeline.  Tiles arrive by LDS DMA (buffer loads that write LDS).
// Each tile buffer, its log-sum-exp slot and the G' buffers are separate LDS
// objects and the tile loop is unrolled over the buffer rotation, so every
// LDS address is tied to one object at compile time: the compiler can then
// see that the reads of the current tiles never alias the DMA in flight and
// does not stall them on it.  The DMA instructions of the next tile are
// spread over the MFMAs of GEMM1 (a burst fills the address queue and stalls
// every wave at issue).
#include <type_traits>

#include "bwd.hpp"

namespace infcl {

constexpr int kBwdBM = 128;  // own rows per workgroup (32 per wave)
constexpr int kGpBytes = kBwdBM * kBwdBN * 2;  // one 16-bit G' exchange buffer

// LDS read-ahead (steps) of GEMM1 (build-time tuning knob).
#ifndef INFCL_BWD_G1_PRE
#define INFCL_BWD_G1_PRE 4
#endif

template <bool F16, int D, bool G16>
__global__ void __launch_bounds__(256, 1) bwd_sweep(BwdParams p) {
  using GO = GradOut<G16, F16>;  // gradient element type
  constexpr int KS = D / 16;            // 16-wide contraction steps of GEMM1
  constexpr int ROWG = D * 2;           // bytes per row in HBM
  constexpr int TILEB = kBwdBN * ROWG;  // bytes per swept tile
  constexpr int NIW = TILEB / 4096;     // 1 KiB DMA instructions per wave and tile
  constexpr int FBW = D / 128;          // 32-feature blocks per wave
  constexpr int NACC = 4 * FBW;
  static_assert(D % 128 == 0 && KS % NIW == 0, "tile DMA layout");
  static_assert(3 * TILEB + 3 * 1024 + 2 * kGpBytes + 2048 <= 160 * 1024, "LDS budget");
  __shared__ __attribute__((aligned(1024))) char tA_[TILEB];
  __shared__ __attribute__((aligned(1024))) char tB_[TILEB];
  __shared__ __attribute__((aligned(1024))) char tC_[TILEB];
  // log-sum-exp slots: 32 values used; the rest of the 1 KiB catches the zeros
  // that the other lanes of the (branch-free) slot DMA write
  __shared__ __attribute__((aligned(1024))) float lA_[256];
  __shared__ __attribute__((aligned(1024))) float lB_[256];
  __shared__ __attribute__((aligned(1024))) float lC_[256];
  __shared__ __attribute__((aligned(1024))) char gp_[2 * kGpBytes];
  __shared__ double red[256];
  INFCL_LDS char* const tA = (INFCL_LDS char*)tA_;
  INFCL_LDS char* const tB = (INFCL_LDS char*)tB_;
  INFCL_LDS char* const tC = (INFCL_LDS char*)tC_;
  INFCL_LDS float* const lA = (INFCL_LDS float*)lA_;
  INFCL_LDS float* const lB = (INFCL_LDS float*)lB_;
  INFCL_LDS float* const lC = (INFCL_LDS float*)lC_;
  INFCL_LDS char* const gp = (INFCL_LDS char*)gp_;

  const int lane = __lane_id();
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);  // wave-uniform (SGPR)
  const int l32 = lane & 31, h = lane >> 5;
  const int64_t b = p.b;
  const BwdTask task = bwd_task(p, kBwdBM * D);
  const BwdSide& sd = p.side[task.sd];
  const char* const swept = (const char*)sd.swept + (int64_t)task.row0 * ROWG;
  const float* const lse2_swept = sd.lse2_swept + task.row0;
  const int rows = task.rows, ntile = (rows + kBwdBN - 1) / kBwdBN;
  const int64_t wg0 = p.own_off + (int64_t)task.rb * kBwdBM;  // own_off is a multiple of 32
  const int64_t own0 = wg0 + 32 * wave;                            // this wave's first own row
  const int64_t iown = own0 + l32;                                 // this lane's own row
  const bool own_ok = iown < p.own_end;
  const int64_t irow = own_ok ? iown : p.own_end - 1;
  const int own0_t = (int)(own0 - task.row0);  // counted from the first swept row

  const float s = p.scale[0];
  const float k2 = s * kLog2e;
  const float dl = p.dloss ? p.dloss[0] : 1.0f;
  // fp16: G' is rounded after scaling by alpha = 2^g16e, divided out at the end
  const int g16e = F16 ? g16_exponent(p.g16) : 0;
  const float g16a = F16 ? ldexpf(1.f, g16e) : 1.0f;
  const float kfin = dl * s / (2.0f * (float)b) * (F16 ? ldexpf(1.f, -g16e) : 1.0f);

  // own operand of GEMM1, held for the whole sweep: row irow, slots 8h..8h+7 of each step
  bf16x8 ownf[KS];
  {
    const __bf16* src = (const __bf16*)sd.own + irow * D + 8 * h;
#pragma unroll
    for (int s2 = 0; s2 < KS; ++s2) ownf[s2] = *(const bf16x8*)(src + 16 * s2);
  }
  const float aO = own_ok ? sd.lse_own[iown] * kLog2e : 0.f;
  const float uO = own_ok ? p.udiag[iown] : 0.f;
  const float gdiag = own_ok ? expm1f(-sd.ell_own[iown]) + expm1f(-sd.ell_swept[iown]) : 0.f;

  auto opaque_lane = [&]() {
    int lo = lane;
    asm volatile("" : "+v"(lo));
    return lo;
  };

  // ---- DMA of swept tile jt into the segment-blocked layout of dst.
  // Instruction k = wave + 4 kk fills LDS bytes [1024 k, 1024 k + 1024): segment
  // k >> 3, rows 4 (k & 7) .. +3; lane L fills row 4 (k & 7) + (L >> 4), physical
  // chunk L & 15, i.e. logical chunk (L & 15) ^ g(row).  Since g(row) =
  // 4 (L >> 4) + (k & 3) and k & 3 = wave, the per-lane part of every source
  // offset is one constant and the rest is wave-uniform.  The DMA lane offsets
  // are rebuilt from an opaque lane id at each use: all 512 registers are in
  // use at d = 512, a value held across the loop would be spilled, and a
  // scratch reload waits for all DMA in flight.  Rows past the
  // end of the sweep fall outside the resource and load as zeros (their G' is masked).
  // (The wave-uniform rest is the wave's 4 rows, added to the lane part, plus a
  // compile-time constant, the scalar operand.)
  auto dma_lane_off = [&]() { return sweep_dma_lane_off(opaque_lane(), wave, ROWG) + 4 * wave * ROWG; };
  auto dma_kk_off = [&](int kk) { return sweep_dma_kk_off(kk, 0, ROWG); };
  auto tile_rsrc = [&](int jt) {
    return sweep_tile_rsrc(swept + (int64_t)jt * TILEB, rows - jt * kBwdBN, ROWG);
  };
  auto lse_rsrc = [&](int jt) {
    return sweep_tile_rsrc(lse2_swept + (int64_t)jt * kBwdBN, rows - jt * kBwdBN, 4);
  };
  // The log-sum-exp slot of a tile is loaded by every wave with the full wave
  // (no divergent branch in the middle of GEMM1): lanes 8k..8k+7 all fetch the
  // tile's 32 values, so the 1 KiB slot holds 8 copies (the first is read).
  // All waves write the same bytes.
  auto lse_lane_off = [&]() { return 16u * (uint32_t)(opaque_lane() & 7); };
  auto issue_tile = [&](int jt, INFCL_LDS char* dst, INFCL_LDS float* ldst) {
    const u32x4 rs = tile_rsrc(jt);
    const uint32_t lo = dma_lane_off();
#pragma unroll
    for (int kk = 0; kk < NIW; ++kk) dma16_asm(rs, dst + 1024 * (wave + 4 * kk), lo, dma_kk_off(kk));
    dma16_asm(lse_rsrc(jt), ldst, lse_lane_off());
  };

  // ---- per-lane LDS offsets of GEMM1's swept fragments; every read is one
  // of these plus an immediate
  auto make_offA = [&](int lo, int (&offA)[8]) {
    const int l32o = lo & 31, ho = lo >> 5;
    const int rA = sweep_perm(l32o);
#pragma unroll
    for (int k = 0; k < 8; ++k) offA[k] = sweep_seg_off(rA, 2 * k + ho);
  };

  double ds_acc = 0.0;

  // ---- GEMM1 of the tile in cur: S^T block, MFMA row m <-> swept row perm(m).
  // LDS fragments are read kPre steps ahead of their MFMA through a register
  // ring.  With with_dma, the loads of tile dtile into (ddst, dlse) are issued
  // between the MFMAs, one 1 KiB instruction per KS / NIW steps.
  // GEMM1's fragment offsets are computed once and held in registers (rebuilt
  // per tile they cost about 2.5% of the backward at d = 512)
  int offA[8];
  make_offA(lane, offA);
  auto gemm1 = [&](const INFCL_LDS char* cur, bool with_dma, int dtile, INFCL_LDS char* ddst,
                   INFCL_LDS float* dlse) {
    u32x4 drs = tile_rsrc(0), drl = lse_rsrc(0);
    uint32_t dlo = 0;
    if (with_dma) {
      drs = tile_rsrc(dtile);
      drl = lse_rsrc(dtile);
      dlo = dma_lane_off();
    }
    auto dma_step = [&](int s2) {
      if (!with_dma) return;
      constexpr int SPI = KS / NIW;  // steps per DMA instruction
      if ((s2 + 1) % SPI == 0) {
        const int kk = (s2 + 1) / SPI - 1;
        dma16_asm(drs, ddst + 1024 * (wave + 4 * kk), dlo, dma_kk_off(kk));
      }
      if (s2 == (KS > 1 ? 1 : 0)) dma16_asm(drl, dlse, lse_lane_off());
    };
    f32x16 sacc;
    constexpr int kPre = KS < INFCL_BWD_G1_PRE ? KS : INFCL_BWD_G1_PRE;
    bf16x8 ring[kPre];
#pragma unroll
    for (int i = 0; i < kPre; ++i) ring[i] = *(const INFCL_LDS bf16x8*)(cur + offA[i & 7] + kSeg * (i >> 3));
    __builtin_amdgcn_sched_group_barrier(0x100, kPre, 0);
#pragma unroll
    for (int s2 = 0; s2 < KS; ++s2) {
      // no leading padding (its sources are LDS loads and the own
      // rows, never restored just before; the build's scan checks it)
      mfma16_vgpr<F16, false>(sacc, ring[s2 % kPre], ownf[s2], s2 == 0, s2 == KS - 1);
      dma_step(s2);
      if (s2 + kPre < KS) {
        const int n = s2 + kPre;
        ring[s2 % kPre] = *(const INFCL_LDS bf16x8*)(cur + offA[n & 7] + kSeg * (n >> 3));
        __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
      }
    }
    return sacc;
  };

  // ---- G' of swept tile jt from its S^T block (log2 domain); entry r <->
  // swept row j = 16 (r>>3) + 8h + (r&7) of the tile.  Returns the dscale
  // contribution.  Tiles touching the diagonal or the end of the sweep take
  // the masked path (uniform branch).  Own rows past the end need no mask:
  // each own row feeds its own gradient row only, which is not stored, and
  // its dscale sum is dropped after the sweep.
  auto tile_special = [&](int jt) {
    const int j0 = jt * kBwdBN;
    return (j0 == own0_t) || (j0 + kBwdBN > rows);
  };
  auto epilogue = [&](int jt, const INFCL_LDS float* lsep, const f32x16& sacc, float (&gv)[16]) -> float {
    const int j0 = jt * kBwdBN;
    const bool special = tile_special(jt);
    const int lo = opaque_lane();  // (the masks' lane parts are rebuilt per use: held, they would spill)
    const int jl = j0 + 8 * (lo >> 5), iown_t = own0_t + (lo & 31);
    float ds_tile = 0.f;
    const INFCL_LDS char* lp = (const INFCL_LDS char*)lsep + 32 * h;
#pragma unroll
    for (int q4 = 0; q4 < 4; ++q4) {
      const f32x4 v = *(const INFCL_LDS f32x4*)(lp + 64 * (q4 >> 1) + 16 * (q4 & 1));
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        const int r = 4 * q4 + c;
        const float pO = exp2_hw(__builtin_fmaf(sacc[r], k2, -aO));
        const float pS = exp2_hw(__builtin_fmaf(sacc[r], k2, -v[c]));
        gv[r] = pO + pS;
        if (!special) {
          ds_tile = __builtin_fmaf(pO, sacc[r] - uO, ds_tile);
        } else {
          const int j = jl + 16 * (r >> 3) + (r & 7);
          const bool jok = j < rows;
          const bool dg = j == iown_t;
          gv[r] = jok ? (dg ? gdiag : gv[r]) : 0.f;
          ds_tile += (bool)(jok & !dg) ? pO * (sacc[r] - uO) : 0.f;
        }
      }
    }
    return ds_tile;
  };
  auto to_h16 = [&](const float (&gv)[16], bf16x8 (&ga)[2]) {
#pragma unroll
    for (int r = 0; r < 16; ++r) ga[r >> 3][r & 7] = to16<F16>(F16 ? gv[r] * g16a : gv[r]);
  };

  // G' exchange buffer (the input's 16-bit type): [128 own rows][32 swept rows], 64-byte rows whose
  // four 16-byte chunks are XOR-swizzled by (row >> 2) & 3.
  auto put_gp = [&](INFCL_LDS char* gpb, const bf16x8 (&ga)[2]) {
    const int lo = opaque_lane();
    const int row = 32 * wave + (lo & 31);
#pragma unroll
    for (int s2 = 0; s2 < 2; ++s2)
      *(INFCL_LDS bf16x8*)(gpb + gp_chunk_off(row, 2 * s2 + (lo >> 5))) = ga[s2];
  };

  // GEMM2's per-lane offsets, computed once: another 2.5% at d = 512
  int offBh[2][FBW], offGh[2];
#pragma unroll
  for (int t = 0; t < 2; ++t)
#pragma unroll
    for (int fbw = 0; fbw < FBW; ++fbw) offBh[t][fbw] = sweep_tr_off(lane, t, wave * FBW + fbw);
#pragma unroll
  for (int s2 = 0; s2 < 2; ++s2) offGh[s2] = gp_chunk_off(l32, 2 * s2 + h);
  {
    // dacc[ob * FBW + fbw] holds own block ob (rows 32 ob .. of the workgroup)
    // x feature block wave FBW + fbw
    f32x16 dacc[NACC];
#pragma unroll
    for (int i = 0; i < NACC; ++i)
#pragma unroll
      for (int r = 0; r < 16; ++r) dacc[i][r] = 0.f;

    // ---- GEMM2 of the tile in cur with the G' in gpb, as an explicit
    // software pipeline over its 2 FBW groups (contraction half s2, feature
    // block fbw; 4 MFMAs each, one per own block): stage g issues the LDS reads
    // of group g + 2 and then the MFMAs of group g.  The stages also
    // compute the G' of the next tile (sacc, log-sum-exp values in lnext), a
    // share per stage, into ga.  The stages are separate scheduling regions.
    auto gemm2_staged = [&](const INFCL_LDS char* cur, const INFCL_LDS char* gpb,
                            const INFCL_LDS float* lnext, const f32x16& sacc, bf16x8 (&ga)[2]) -> float {
      constexpr int NG = 2 * FBW;
      constexpr int PD = 2;
      constexpr int EPS = (16 + NG - 1) / NG;  // G' entries per stage
      constexpr int NL = EPS > 2 ? 4 : 2;      // live log-sum-exp blocks
      const int lo = opaque_lane();
      const int ho = lo >> 5;
      const INFCL_LDS char* lp = (const INFCL_LDS char*)lnext + 32 * ho;
      auto readL = [&](int q4) { return *(const INFCL_LDS f32x4*)(lp + 64 * (q4 >> 1) + 16 * (q4 & 1)); };
      auto first_stage = [](int q) { return (4 * q) / EPS; };  // first stage using LSE block q
      auto readA = [&](int s2, bf16x8 (&A)[4]) {
#pragma unroll
        for (int ob = 0; ob < 4; ++ob)
          A[ob] = *(const INFCL_LDS bf16x8*)(gpb + 2048 * ob + offGh[s2]);
      };
      auto readB = [&](int g, s16x4 (&bq)[2]) {
        const int s2 = g / FBW, fbw = g % FBW;
#pragma unroll
        for (int t = 0; t < 2; ++t)
          bq[t] = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
              (INFCL_LDS s16x4*)(cur + offBh[t][fbw] + 16 * s2 * kSegRow));
      };
      // A holds G' of contraction half 0 until the last stage of that half has
      // issued its MFMAs, then half 1 (read straight after).
      bf16x8 A[4];
      s16x4 Bq[PD + 1][2];
      f32x4 Lq[NL];
      readA(0, A);
#pragma unroll
      for (int q = 0; q < 4; ++q)
        if (first_stage(q) == 0) Lq[q % NL] = readL(q);
#pragma unroll
      for (int g = 0; g < PD && g < NG; ++g) readB(g, Bq[g]);
      __builtin_amdgcn_sched_barrier(0);
      float ds_tile = 0.f;
#pragma unroll
      for (int g = 0; g < NG; ++g) {
        if (g + PD < NG) readB(g + PD, Bq[(g + PD) % (PD + 1)]);
#pragma unroll
        for (int q = 0; q < 4; ++q)
          if (first_stage(q) == g + 1) Lq[q % NL] = readL(q);
#pragma unroll
        for (int i = 0; i < EPS; ++i) {
          const int r = g * EPS + i;
          if (r < 16) {
            const float x = sacc[r];
            const float pO = exp2_hw(__builtin_fmaf(x, k2, -aO));
            const float pS = exp2_hw(__builtin_fmaf(x, k2, -Lq[(r >> 2) % NL][r & 3]));
            ga[r >> 3][r & 7] = to16<F16>(F16 ? (pO + pS) * g16a : pO + pS);
            ds_tile = __builtin_fmaf(pO, x - uO, ds_tile);
          }
        }
        const int fbw = g % FBW;
        const s16x4* bq = Bq[g % (PD + 1)];
        const s16x8 bb = {bq[0][0], bq[0][1], bq[0][2], bq[0][3], bq[1][0], bq[1][1], bq[1][2], bq[1][3]};
#pragma unroll
        for (int ob = 0; ob < 4; ++ob)
          dacc[ob * FBW + fbw] = mfma16<F16>(A[ob], __builtin_bit_cast(bf16x8, bb), dacc[ob * FBW + fbw]);
        if (g == FBW - 1) readA(1, A);
        __builtin_amdgcn_sched_barrier(0);
      }
      return ds_tile;
    };

    {
      // Software pipeline over tiles: iteration jt runs GEMM1 of tile jt+1
      // (issuing the loads of tile jt+2), then GEMM2 of tile jt together with
      // the G' of tile jt+1.  Three tile buffers rotate; G' buffers alternate.
      // Past the last tile, GEMM1 runs on a stale buffer and the G' step takes
      // the masked path (rows past the sweep's end), so it yields zeros.
      issue_tile(0, tA, lA);
      issue_tile(1, tB, lB);
      wait_dma();
      __syncthreads();
      {
        const f32x16 sacc = gemm1(tA, false, 0, tC, lC);
        float gv[16];
        const float d0 = epilogue(0, lA, sacc, gv);
        ds_acc += (double)d0;
        bf16x8 ga[2];
        to_h16(gv, ga);
        put_gp(gp, ga);
      }
      __syncthreads();
      auto body = [&](int jt, const INFCL_LDS char* cur, INFCL_LDS char* nxt, const INFCL_LDS float* lnxt,
                      INFCL_LDS char* fre, INFCL_LDS float* lfre) {
        const bool next = jt + 1 < ntile;
        const f32x16 sacc = gemm1(nxt, true, jt + 2, fre, lfre);
        __builtin_amdgcn_sched_barrier(0);
        bf16x8 ga[2];
        float dn = gemm2_staged(cur, gp + (jt & 1) * kGpBytes, lnxt, sacc, ga);
        // pin the unmasked G' here: otherwise it is sunk into the not-special
        // branch below and computed after GEMM2 instead of alongside it
        asm volatile("" : "+v"(ga[0]), "+v"(ga[1]), "+v"(dn));
        __builtin_amdgcn_sched_barrier(0);
        if (tile_special(jt + 1)) {
          float gv[16];
          dn = epilogue(jt + 1, lnxt, sacc, gv);
          to_h16(gv, ga);
        }
        if (next) ds_acc += (double)dn;
        put_gp(gp + ((jt + 1) & 1) * kGpBytes, ga);
        wait_dma();
        __syncthreads();
      };
      // Unrolled over the buffer rotation without tests in between (with them
      // the accumulators spill): a tile index past the end is a tile of rows past
      // the end, fully masked (zero G').  Parts of a split block are multiples of
      // three tiles (BwdPlan::gran).
      for (int jt = 0; jt < ntile; jt += 3) {
        body(jt, tA, tB, lB, tC, lC);
        body(jt + 1, tB, tC, lC, tA, lA);
        body(jt + 2, tC, tA, lA, tB, lB);
      }
    }

    // ---- write dOwn (or this part's unscaled sums): lane holds feature l32 of
    // a 32-feature block, rows 8(r>>2)+4h+(r&3)
    const int rl0 = 4 * h, f0 = 32 * wave * FBW + l32;
    if (task.part) {
#pragma unroll
      for (int ob = 0; ob < 4; ++ob) {
        float* dst = task.part + (32 * ob + rl0) * D + f0;
#pragma unroll
        for (int fbw = 0; fbw < FBW; ++fbw)
#pragma unroll
          for (int r = 0; r < 16; ++r) dst[(8 * (r >> 2) + (r & 3)) * D + 32 * fbw] = dacc[ob * FBW + fbw][r];
      }
    } else {
      const bool all_ok = wg0 + kBwdBM <= p.own_end;
#pragma unroll
      for (int ob = 0; ob < 4; ++ob) {
        auto* dst = (typename GO::type*)sd.dOwn + (wg0 - p.own_off + 32 * ob + rl0) * D + f0;
#pragma unroll
        for (int fbw = 0; fbw < FBW; ++fbw)
#pragma unroll
          for (int r = 0; r < 16; ++r) {
            const int64_t row = wg0 + 32 * ob + 8 * (r >> 2) + rl0 + (r & 3);
            if (all_ok || row < p.own_end)
              dst[(8 * (r >> 2) + (r & 3)) * D + 32 * fbw] = GO::cvt(kfin * dacc[ob * FBW + fbw][r]);
          }
      }
    }
  }

  // ---- dscale partial of this workgroup: fixed-order reduction
  red[threadIdx.x] = own_ok ? ds_acc : 0.0;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if ((int)threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x == 0) p.ds_part[blockIdx.x] = red[0];
}

// dscale = dloss / (2b) * (sum of the sweeps' partials), fixed order, by one
// workgroup of 256; into dscale (fp32) and/or dscale64 (fp64), whichever is given
__device__ __forceinline__ void dscale_sum(const double* part, int64_t n, int64_t b, const float* dloss, float* dscale,
                                           double* dscale64) {
  __shared__ double red[256];
  double s = 0.0;
  for (int64_t k = threadIdx.x; k < n; k += 256) s += part[k];
  red[threadIdx.x] = s;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if ((int)threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    const double dl = dloss ? (double)dloss[0] : 1.0;
    const double v = red[0] * dl / (2.0 * (double)b);
    if (dscale) *dscale = (float)v;
    if (dscale64) *dscale64 = v;
  }
}
__global__ void __launch_bounds__(256) dscale_finish(const double* part, int64_t n, int64_t b, const float* dloss,
                                                     float* dscale, double* dscale64) {
  dscale_sum(part, n, b, dloss, dscale, dscale64);
}

// Gradients of the split row blocks: the ns partial sums of each element in
// fixed order, scaled as the sweeps scale theirs and rounded once to the
// gradient type.  Bound by memory (the partials are read once, 16 bytes per
// lane; at most 64 MiB of them, which stay in the last-level cache: 12 us).
// One more workgroup (the last grid row) sums dscale: as a launch of its own
// that took 4.7 us.  F32: the sums of fp32 inputs, whose alpha is divided out
// of them as bwd_f32 does (with F16 it is part of the factor).
template <bool G16, bool F16, bool F32 = false>
__global__ void __launch_bounds__(256) bwd_reduce(BwdParams p, int bm, int nwg, float* dscale, double* dscale64) {
  using GO = GradOut<G16, F16>;
  if (blockIdx.y == gridDim.y - 1) {
    if (blockIdx.x == 0) dscale_sum(p.ds_part, nwg, p.b, p.dloss, dscale, dscale64);
    return;
  }
  const int c4 = (int)(p.d >> 2);  // 4-feature groups per row
  const int per = bm * c4;         // ... per block
  const int q = blockIdx.y;
  const int e = blockIdx.x * 256 + threadIdx.x;
  const int blk = p.nfull + q;
  const int sd = blk >= p.nblk ? 1 : 0;
  const int rl = e / c4;
  const int64_t row = (int64_t)(sd ? blk - p.nblk : blk) * bm + rl;  // own row - own_off
  const float s = p.scale[0];
  const float dl = p.dloss ? p.dloss[0] : 1.0f;
  const float g16inv = F16 || F32 ? ldexpf(1.f, -g16_exponent<F32 ? 0 : 14>(p.g16)) : 1.0f;
  const float kfin = dl * s / (2.0f * (float)p.b) * (F16 ? g16inv : 1.0f);
  if (e >= per || row >= p.own_end - p.own_off) return;
  const f32x4* src = (const f32x4*)(p.part + (int64_t)q * p.ns * per * 4) + e;
  f32x4 a = {0.f, 0.f, 0.f, 0.f};
  int k = 0;
  for (; k + 4 <= p.ns; k += 4) {  // four loads in flight, added in order
    f32x4 v[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) v[u] = src[(int64_t)(k + u) * per];
#pragma unroll
    for (int u = 0; u < 4; ++u) a += v[u];
  }
  for (; k < p.ns; ++k) a += src[(int64_t)k * per];
  typedef typename GO::type out4 __attribute__((ext_vector_type(4)));
  out4 o;
#pragma unroll
  for (int u = 0; u < 4; ++u) o[u] = GO::cvt(kfin * (F32 ? g16inv * a[u] : a[u]));
  *(out4*)((typename GO::type*)p.side[sd].dOwn + row * p.d + 4 * (e - rl * c4)) = o;
}

template <bool F16>
static int launch_bwd_sweep(const BwdParams& p, int nwg, hipStream_t stream) {
  auto go = [&](auto dc) {
    constexpr int D = decltype(dc)::value;
    if (p.gdt)
      hipLaunchKernelGGL((bwd_sweep<F16, D, true>), dim3(nwg), dim3(256), 0, stream, p);
    else
      hipLaunchKernelGGL((bwd_sweep<F16, D, false>), dim3(nwg), dim3(256), 0, stream, p);
    return hipGetLastError() == hipSuccess ? 0 : 1;
  };
  switch (p.d) {
    case 128: return go(std::integral_constant<int, 128>{});
    case 256: return go(std::integral_constant<int, 256>{});
    case 384: return go(std::integral_constant<int, 384>{});
    case 512: return go(std::integral_constant<int, 512>{});
  }
  return 2;
}

// Before the sweeps: the log-sum-exp vectors rescaled to base 2 (the swept
// side is streamed through LDS next to every tile and used as is), and for
// fp16 (g16 given) the maxima behind the scale of G' (see g16_exponent).
// kPrepBlocks workgroups for any b, so that the maxima are one pair per lane.
__global__ void __launch_bounds__(256) bwd_prep(const float* lse_r, const float* lse_c, const float* aux, float* l2r,
                                                float* l2c, float* g16, int64_t b) {
  float mr = 0.f, mc = 0.f;
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < b; i += (int64_t)kPrepBlocks * 256) {
    l2r[i] = lse_r[i] * kLog2e;
    l2c[i] = lse_c[i] * kLog2e;
    if (g16) {
      mr = fmaxf(mr, -expm1f(-aux[i]));
      mc = fmaxf(mc, -expm1f(-aux[b + i]));
    }
  }
  if (g16) {
    __shared__ float sr[4], sc[4];
#pragma unroll
    for (int k = 1; k < 64; k <<= 1) {
      mr = fmaxf(mr, shfl_xor(mr, k));
      mc = fmaxf(mc, shfl_xor(mc, k));
    }
    if ((threadIdx.x & 63) == 0) {
      sr[threadIdx.x >> 6] = mr;
      sc[threadIdx.x >> 6] = mc;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
      g16[2 * blockIdx.x] = fmaxf(fmaxf(sr[0], sr[1]), fmaxf(sr[2], sr[3]));
      g16[2 * blockIdx.x + 1] = fmaxf(fmaxf(sc[0], sc[1]), fmaxf(sc[2], sc[3]));
    }
  }
}

bool bwd_wide_supported(int64_t d, int dtype);
int launch_bwd_wide(const BwdParams& p, int nwg, bool f16, hipStream_t stream);
int launch_bwd_f32(const BwdParams& p, int nwg, hipStream_t stream);

// Split of the backward over workgroups, for nrows own rows of each side
// against b swept rows: both sides' row blocks run in one launch, and the
// blocks beyond the last whole round of kCUs are swept in ns parts each, so
// that a batch of few blocks, or the remainder of a larger one, still fills
// the chip (measured, one launch per side before, step with the forward:
// b = 1024, d = 512 fp32 1834 -> 179 us, b = 4096, d = 768 fp16 456 -> 202 us,
// b = 8192, d = 256 fp32 4.60 -> 1.44 ms).  ns minimises (rounds of parts) / ns
// block times plus the cost of a part (prologue, epilogue) and of the reduction,
// which reads and writes bm x d floats per part; the partial sums take at most
// cap bytes.
// The model's constants are rough.  Per tile and feature 3.7e-3 us is the
// 128-row sweep's (3.6e-3 at b = 32768, d = 512, 4.1e-3 at 256, 4.9e-3 at 128, of
// two workgroups per CU there) and 0.011 the fp32 sweep's (0.0106 at b = 8192,
// d = 512, 0.0119 at 256); the wide sweeps' blocks of half the rows take
// 1.9e-3 (b = 131072, d = 768), so that they split a little further.  A part's
// fixed 8 us is about half of what kernel traces show at small batches (15 us at
// b = 256 and 18 at 1000, d = 512), and 2e6 bytes per us about half the rate of
// the writes and the reduction's reads together (4 to 14 us for 3 to 50 MB).  One
// workgroup per compute unit is counted at every width, although at 16-bit
// d = 128 and fp32 d up to 192 two or three are resident.
constexpr int kCUs = 256;
BwdPlan plan_bwd(int64_t b, int64_t nrows, int64_t d, int dtype, size_t cap) {
  BwdPlan pl;
  pl.bm = bwd_wide_supported(d, dtype) ? kWideBM : kBwdBM;
  pl.nblk = (int)((nrows + pl.bm - 1) / pl.bm);
  const int total = 2 * pl.nblk;
  const int64_t ntile = (b + kBwdBN - 1) / kBwdBN;
  pl.gran = dtype != 1 && pl.bm == kBwdBM ? 3 : 1;
  const int64_t nunit = (ntile + pl.gran - 1) / pl.gran;
  pl.nfull = total / kCUs * kCUs;
  pl.ns = 1;
  pl.part_bytes = 0;
  const int rem = total - pl.nfull;
  if (rem > 0) {
    // microseconds: a tile, a part's fixed cost, a part's bytes through the reduction
    const double t_tile = (dtype == 1 ? 0.011 : 3.7e-3) * (double)d;
    const double blk_bytes = (double)pl.bm * (double)d * 4.0;
    double best = 0.0;
    for (int ns = 1; ns <= 64 && ns <= nunit; ++ns) {
      const int64_t parts = (int64_t)rem * ns;
      const double bytes = (double)parts * blk_bytes;
      if (ns > 1 && bytes + 8.0 * (double)(pl.nfull + parts) > (double)cap) break;
      const double rounds = (double)((parts + kCUs - 1) / kCUs);
      double t = rounds * (8.0 + t_tile * (double)((nunit + ns - 1) / ns * pl.gran));
      if (ns > 1) t += 6.0 + bytes / 2.0e6;
      if (ns == 1 || t < best) {
        best = t;
        pl.ns = ns;
      }
    }
  }
  pl.nwg = pl.nfull + rem * pl.ns;
  if (pl.ns > 1) {
    const size_t sums = (size_t)rem * pl.ns * (size_t)pl.bm * (size_t)d * sizeof(float);
    pl.part_bytes = sums + (size_t)pl.nwg * sizeof(double);  // the sums, then the dscale partials
  } else {
    pl.nfull = total;
  }
  return pl;
}

// Backward: 16-bit inputs take the 128-row sweep above up to d = 512 and the
// wide-row sweeps (64 own rows per workgroup) beyond; fp32 inputs have their own.  Own
// rows are [r0, r0 + nrows) of both sides (all b for the whole batch; a
// shard's samples otherwise, with dimg/dtxt [nrows, d]: fp32, or with gdt = 1
// the 16-bit input type); lse_r, lse_c and aux cover all b samples.  dscale
// (fp32) and/or dscale64 (fp64) receive this call's share, dloss/(2b) times its
// partial sums.  part: the partial sums of split row blocks, part_cap bytes.
int launch_bwd(const void* img, const void* txt, int64_t b, int64_t d, int dtype, int64_t r0, int64_t nrows,
               const float* scale, const float* lse_r, const float* lse_c, const float* aux, const float* dloss,
               void* dimg, void* dtxt, int gdt, float* dscale, double* dscale64, float* lse2, double* ds_part,
               float* g16, float* part, size_t part_cap, hipStream_t stream) {
  const bool wide = bwd_wide_supported(d, dtype);
  const BwdPlan pl = plan_bwd(b, nrows, d, dtype, part_cap);
  float* l2r = lse2;
  float* l2c = lse2 + b;
  hipLaunchKernelGGL(bwd_prep, dim3(kPrepBlocks), dim3(256), 0, stream, lse_r, lse_c, aux, l2r, l2c,
                     dtype != 0 ? g16 : nullptr, b);
  if (hipGetLastError() != hipSuccess) return 1;
  BwdParams p;
  p.g16 = g16;
  p.b = b;
  p.d = d;
  p.scale = scale;
  p.udiag = aux + 2 * b;
  p.dloss = dloss;
  p.own_off = r0;
  p.own_end = r0 + nrows;
  p.gdt = gdt;
  p.side[0] = BwdSide{img, txt, lse_r, l2c, aux, aux + b, dimg};
  p.side[1] = BwdSide{txt, img, lse_c, l2r, aux + b, aux, dtxt};
  p.nblk = pl.nblk;
  p.nfull = pl.nfull;
  p.ns = pl.ns;
  p.gran = pl.gran;
  p.part = part;
  const int64_t split = 2 * (int64_t)pl.nblk - pl.nfull;  // split row blocks
  p.ds_part = pl.ns > 1 ? (double*)(part + split * pl.ns * pl.bm * d) : ds_part;
  int rc;
  if (dtype == 1)
    rc = launch_bwd_f32(p, pl.nwg, stream);
  else if (wide)
    rc = launch_bwd_wide(p, pl.nwg, dtype == 2, stream);
  else if (dtype == 2)
    rc = launch_bwd_sweep<true>(p, pl.nwg, stream);
  else
    rc = launch_bwd_sweep<false>(p, pl.nwg, stream);
  if (rc) return rc;
  if (pl.ns > 1) {
    const dim3 grid((unsigned)((pl.bm * (d >> 2) + 255) / 256), (unsigned)split + 1);
    if (dtype == 2 && gdt)
      hipLaunchKernelGGL((bwd_reduce<true, true>), grid, dim3(256), 0, stream, p, pl.bm, pl.nwg, dscale,
                         dscale64);
    else if (dtype == 2)
      hipLaunchKernelGGL((bwd_reduce<false, true>), grid, dim3(256), 0, stream, p, pl.bm, pl.nwg, dscale,
                         dscale64);
    else if (dtype == 1)
      hipLaunchKernelGGL((bwd_reduce<false, false, true>), grid, dim3(256), 0, stream, p, pl.bm, pl.nwg, dscale,
                         dscale64);
    else if (gdt)
      hipLaunchKernelGGL((bwd_reduce<true, false>), grid, dim3(256), 0, stream, p, pl.bm, pl.nwg, dscale,
                         dscale64);
    else
      hipLaunchKernelGGL((bwd_reduce<false, false>), grid, dim3(256), 0, stream, p, pl.bm, pl.nwg, dscale,
                         dscale64);
    return hipGetLastError() == hipSuccess ? 0 : 1;
  }
  hipLaunchKernelGGL(dscale_finish, dim3(1), dim3(256), 0, stream, (const double*)p.ds_part, (int64_t)pl.nwg, b,
                     dloss, dscale, dscale64);
  return hipGetLastError() == hipSuccess ? 0 : 1;
}

bool bwd_supported(int64_t d, int dtype) {
  if (dtype == 0 || dtype == 2) return d % 128 == 0 && d >= 128 && d <= 1024;
  return d % 64 == 0 && d >= 64 && d <= 512;
}

}  // namespace infcl
