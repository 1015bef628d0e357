// Forward sweep of the tiled symmetric InfoNCE loss for fp32 inputs (gfx950),
// and the finalize shared by both forward sweeps.  (16-bit inputs take the
// resident-rows sweep of fwd2.hip.)
//
// What is computed (paper Sec. 3.1, Eq. 2-5; the in-GPU forward algorithm of
// Sec. 3.2): for every row i and column j of S = s * img * txt^T, the
// off-diagonal log-sum-exp of row i and of column j, without storing S.
//
// Work decomposition (differs from the paper's one-row-block-per-thread-block
// design: here a persistent 2-D grid of workgroups shares the column
// statistics without atomics):
//   - A workgroup tile covers 64 rows i (image rows) x 256 columns j (text
//     rows), or 32 x 128 where few tiles would leave compute units idle.  The
//     MFMA computes the transposed block S^T (M = j, N = i), so each lane owns a
//     fixed i and 16 consecutive-ish j's per 32x32 block.
//   - The products run on the bf16 MFMA, every fp32 operand in three exact
//     bf16 parts (split3 in common.hpp): b = 8192, d = 512 558 -> 423 us against
//     the fp32 MFMA, d = 256 310 -> 234 us, at a smaller error.
//   - Workgroup (q, g) of a P_r x P_c grid sweeps row tiles q, q+P_r, ... and,
//     for each, the column tiles of column group g.  Row statistics stay in
//     registers across the sweep (one running pair per lane and row, merged
//     across lanes only when the row tile is done); column statistics are
//     reduced across lanes every tile and merged into the group's own slice
//     colR/colL[q][j] in global memory (only this workgroup touches it).
//   - The finalize kernel merges the partial pairs of every row and column in
//     a fixed order and evaluates the per-sample terms in fp64.
//   - Workgroups of one column group are launched with the same index modulo
//     8, so they run on one XCD and share its L2 for the text tiles.
//
// Online log-sum-exp (Eq. 4-5) with lazy references: each running pair keeps a
// reference R (a value actually seen, so l >= 1 after the first one) and adds
// exp2(y - R) for new values y; a tile whose partial sum exceeds 2^64 (or is
// not finite, e.g. while R is still -inf) is redone with the exact max-rescaled
// merge.  The paper's merge starts from 0; the identity of the merge is the
// empty sum (R = -inf, l = 0), which is what is used here.
#include "common.hpp"

namespace infcl {

struct FwdParams {
  const void* img;  // rows i, [b, d]
  const void* txt;  // rows j, [b, d]
  int64_t b, d;
  const float* scale;
  float* rowR;  // [Pc * 4][rstride]   per (column group, wave) partial row pairs, by own row - r0
  float* rowL;
  float* colR;  // [Pr][b]       per row group partial column pairs
  float* colL;
  float* udiag;  // [b]  <img_i, txt_i>
  int Pr, Pc;
  int nRT, nCT;
  int64_t r0, rend;  // own rows [r0, rend) (a shard of the batch; 0 and b for the whole batch)
  int64_t rstride;   // rend - r0
};

// Shape of a workgroup tile: MB 32-column blocks per wave (four waves), NB
// 32-row blocks; 128 bytes of every row per stage.
template <int MB, int NB>
struct FwdTile {
  static constexpr int BI = 32 * NB;   // rows i
  static constexpr int BJ = 128 * MB;  // columns j
  static constexpr int Rows = BI + BJ;
  static constexpr int StageBytes = Rows * 128;
  static constexpr int NIW = Rows / 32;  // 1 KiB DMA instructions per wave and stage
};

// Chunk swizzle for 128-byte rows: 16 consecutive rows reading the same logical
// 16-byte chunk hit 16 distinct bank groups.
__device__ __forceinline__ int fwd_swz(int r, int c) { return c ^ ((r >> 1) & 7); }

// Per-lane source offsets of the K-stage DMA: instruction k (= wave + 4 kk)
// fills tile rows 8k..8k+7; lane L copies logical chunk fwd_swz(r, L & 7) of row
// r = 8k + L/8 to physical chunk L & 7.  The first BI rows are image rows, the others text rows.
template <int NIW>
struct FwdDmaOffsets {
  uint32_t off[NIW];
};

template <int MB, int NB>
__device__ __forceinline__ FwdDmaOffsets<FwdTile<MB, NB>::NIW> fwd_dma_offsets(int64_t d, int es, int wave, int lane) {
  using T = FwdTile<MB, NB>;
  FwdDmaOffsets<T::NIW> o;
#pragma unroll
  for (int kk = 0; kk < T::NIW; ++kk) {
    const int k = wave + 4 * kk;
    const int r = 8 * k + (lane >> 3);
    const int rl = kk < NB ? r : r - T::BI;  // row within the image or the text tile
    o.off[kk] = (uint32_t)(rl * d * es + 16 * fwd_swz(r, lane & 7));
  }
  return o;
}

// Issue the DMA of one K-stage (128 bytes of each of the tile's rows).  Rows
// past b fall outside the buffer resources and load as zeros (they are masked).
template <int MB, int NB>
__device__ __forceinline__ void fwd_stage_dma(const FwdParams& p, const FwdDmaOffsets<FwdTile<MB, NB>::NIW>& o,
                                              int64_t i0, int64_t j0, int st, INFCL_LDS char* buf, int wave) {
  const int64_t b = p.b, rowb = p.d * (int64_t)sizeof(float);
  const u32x4 ri = rsrc_words((const char*)p.img + i0 * rowb, (p.rend - i0) * rowb);
  const u32x4 rt = rsrc_words((const char*)p.txt + j0 * rowb, (b - j0) * rowb);
  const uint32_t soff = (uint32_t)st * 128u;
#pragma unroll
  for (int kk = 0; kk < FwdTile<MB, NB>::NIW; ++kk)
    dma16_asm(kk < NB ? ri : rt, buf + 1024 * (wave + 4 * kk), o.off[kk], soff);
}

// MFMA work of one K-stage: acc[mb][nb] += S^T block (j block mb, i block nb).
// A 16-wide contraction step is 64 bytes; lane half h holds floats 8h..8h+7.
// The products run on the bf16 MFMA with every operand in three exact bf16
// parts (split3): 24 MFMAs of 32 cycles per step and wave instead of 32 of 64,
// next to 176 vector instructions that split the fragments (two waves share a
// SIMD, so one's splitting overlaps the other's MFMAs).
template <int MB, int NB>
__device__ __forceinline__ void fwd_stage_mfma(const INFCL_LDS char* buf, f32x16 (&acc)[MB][NB], int wave, int lane) {
  const int l32 = lane & 31, h = lane >> 5;
#pragma unroll
  for (int s = 0; s < 2; ++s) {
    split3 a[MB], bb[NB];
    auto frag = [&](int r) {
      const int c = 4 * s + 2 * h;
      return split_f32(*(const INFCL_LDS f32x4*)(buf + r * 128 + fwd_swz(r, c) * 16),
                       *(const INFCL_LDS f32x4*)(buf + r * 128 + fwd_swz(r, c + 1) * 16));
    };
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) a[mb] = frag(FwdTile<MB, NB>::BI + 32 * MB * wave + 32 * mb + l32);
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) bb[nb] = frag(32 * nb + l32);
    constexpr int qa[6] = {2, 0, 1, 1, 0, 0}, qb[6] = {0, 2, 1, 0, 1, 0};
#pragma unroll
    for (int t = 0; t < 6; ++t)
#pragma unroll
      for (int mb = 0; mb < MB; ++mb)
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) acc[mb][nb] = mfma_bf16(a[mb].p[qa[t]], bb[nb].p[qb[t]], acc[mb][nb]);
  }
}

// One butterfly step of the reduce-scatter below: lanes exchange the half of
// their HALF*2 live values that the partner keeps (partner = lane ^ HALF).
template <bool kMax, int HALF, int N>
__device__ __forceinline__ void rs_step(float (&v)[N], int l32) {
  const bool bit = (l32 & HALF) != 0;
#pragma unroll
  for (int t = 0; t < HALF; ++t) {
    const float send = bit ? v[t] : v[t + HALF];
    const float keep = bit ? v[t + HALF] : v[t];
    const float recv = shfl_xor(send, HALF);
    v[t] = kMax ? fmaxf(keep, recv) : keep + recv;
  }
}

// Reduce-scatter over the 32 lanes of each wave half: on entry v[t] is this
// lane's partial for value index t (0..N-1, N = 32 or 16); on exit the result
// is the total over the 32 lanes for index fwd_rs_index<N>(lane) (sum, or max
// when kMax); with N = 16 lanes l and l ^ 8 hold the same one.
template <int N>
__device__ __forceinline__ int fwd_rs_index(int l32) {
  return N == 32 ? l32 : ((l32 >> 4) << 3) | (l32 & 7);
}
template <int N>
__device__ __forceinline__ int fwd_rs_lane(int t) {
  return N == 32 ? t : ((t >> 3) << 4) | (t & 7);
}
template <bool kMax, int N>
__device__ __forceinline__ float half_reduce_scatter(float (&v)[N], int lane) {
  const int l32 = lane & 31;
#pragma unroll
  for (int t = 0; t < N / 2; ++t) {
    // odd 16-lane rows of x swap with even rows of y: lanes with bit 4 clear end
    // with (own v[t], partner v[t]); lanes with bit 4 set with (partner v[t+N/2], own v[t+N/2])
    auto sw = __builtin_amdgcn_permlane16_swap(__float_as_uint(v[t]), __float_as_uint(v[t + N / 2]), false, false);
    const float x = __uint_as_float(sw[0]), y = __uint_as_float(sw[1]);
    v[t] = kMax ? fmaxf(x, y) : x + y;
  }
  if constexpr (N == 32) rs_step<kMax, 8>(v, l32);
  rs_step<kMax, 4>(v, l32);
  rs_step<kMax, 2>(v, l32);
  rs_step<kMax, 1>(v, l32);
  if constexpr (N == 16) {
    const float o = shfl_xor(v[0], 8);
    v[0] = kMax ? fmaxf(v[0], o) : v[0] + o;
  }
  return v[0];
}

// Epilogue of one workgroup tile.  acc[mb][nb][r] <-> column
// j = jw + 32 mb + 8 (r>>2) + (r&3), row i = i0 + 32 nb + l32, jw = j0 + 32 MB wave + 4 h.
// The exponent of an entry is fma(acc, kk, -reference): unmasked tiles pass the
// raw dot products with kk = s log2(e); tiles touching the diagonal or the
// ragged end pass y = s log2(e) <.,.> with excluded entries set to -inf and kk = 1.
template <bool MASKED, int MB, int NB>
__device__ __forceinline__ void fwd_epilogue(const FwdParams& p, const f32x16 (&acc)[MB][NB], float (&rowR)[NB],
                                             float (&rowL)[NB], int64_t j0, int q, bool first_row_tile, float k2,
                                             int wave, int lane) {
  const int l32 = lane & 31, h = lane >> 5;
  const int64_t b = p.b;
  const int64_t jw = j0 + 32 * MB * wave + 4 * h;
  const float ninf = -__builtin_inff();
  const float kk = MASKED ? 1.0f : k2;
  auto jof = [&](int mb, int r) -> int64_t { return jw + 32 * mb + 8 * (r >> 2) + (r & 3); };

  // ---- row statistics: per lane and row, lazy reference with an exact fallback
  {
    float t[NB];
    bool bad = false;
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) {
      float s = 0.f;
#pragma unroll
      for (int mb = 0; mb < MB; ++mb)
#pragma unroll
        for (int r = 0; r < 16; ++r) s += exp2_hw(__builtin_fmaf(acc[mb][nb][r], kk, -rowR[nb]));
      t[nb] = s;
      bad |= !lazy_ok(s);
    }
    if (!wave_any(bad)) {
#pragma unroll
      for (int nb = 0; nb < NB; ++nb) rowL[nb] += t[nb];
    } else {
#pragma unroll
      for (int nb = 0; nb < NB; ++nb) {
        float m = rowR[nb];
#pragma unroll
        for (int mb = 0; mb < MB; ++mb)
#pragma unroll
          for (int r = 0; r < 16; ++r) m = fmaxf(m, acc[mb][nb][r] * kk);
        const float ms = m == ninf ? 0.f : m;
        float s2 = rowL[nb] * exp2_hw(rowR[nb] - ms);
#pragma unroll
        for (int mb = 0; mb < MB; ++mb)
#pragma unroll
          for (int r = 0; r < 16; ++r) s2 += exp2_hw(__builtin_fmaf(acc[mb][nb][r], kk, -ms));
        rowL[nb] = m == ninf ? 0.f : s2;
        rowR[nb] = m;
      }
    }
  }

  // ---- column statistics: reference = the group's running pair for column j
  {
    constexpr int NV = 16 * MB;  // columns per lane
    const int tmine = fwd_rs_index<NV>(l32);
    const int64_t jmine = jof(tmine >> 4, tmine & 15);  // the column this lane reduces to
    float* cR = p.colR + (int64_t)q * b;
    float* cL = p.colL + (int64_t)q * b;
    float Rold = ninf, Lold = 0.f;
    float ref[NV];
    if (first_row_tile) {
#pragma unroll
      for (int t = 0; t < NV; ++t) ref[t] = ninf;
    } else if constexpr (!MASKED) {
#pragma unroll
      for (int mb = 0; mb < MB; ++mb)
#pragma unroll
        for (int a = 0; a < 4; ++a) {
          const f32x4 v = *(const f32x4*)(cR + jw + 32 * mb + 8 * a);
#pragma unroll
          for (int c = 0; c < 4; ++c) ref[16 * mb + 4 * a + c] = v[c];
        }
      Rold = cR[jmine];
      Lold = cL[jmine];
    } else {
#pragma unroll
      for (int t = 0; t < NV; ++t) {
        const int64_t j = jof(t >> 4, t & 15);
        const float v = cR[j < b ? j : b - 1];
        ref[t] = j < b ? v : ninf;
      }
      const int64_t jc = jmine < b ? jmine : b - 1;
      const float r0 = cR[jc], l0 = cL[jc];
      Rold = jmine < b ? r0 : ninf;
      Lold = jmine < b ? l0 : 0.f;
    }
    float v[NV];
#pragma unroll
    for (int t = 0; t < NV; ++t) {
      const int mb = t >> 4, r = t & 15;
      float s = 0.f;
#pragma unroll
      for (int nb = 0; nb < NB; ++nb) s += exp2_hw(__builtin_fmaf(acc[mb][nb][r], kk, -ref[t]));
      // a column whose entries are all excluded so far has ref = -inf and sums
      // exp2(-inf + inf) = NaN here; that sends the tile to the exact path
      v[t] = s;
    }
    const float tot = half_reduce_scatter<false>(v, lane);
    float Rnew = Rold, Lnew = Lold + tot;
    if (wave_any(!lazy_ok(tot))) {
      // exact path: per-column max over this tile, broadcast, rescaled sums
#pragma unroll
      for (int t = 0; t < NV; ++t) {
        const int mb = t >> 4, r = t & 15;
        float m = acc[mb][0][r] * kk;
        if constexpr (NB == 2) m = fmaxf(m, acc[mb][1][r] * kk);
        v[t] = m;
      }
      const float mt = half_reduce_scatter<true>(v, lane);
      const float Rn = fmaxf(Rold, mt);
#pragma unroll
      for (int t = 0; t < NV; ++t) {
        const float rn = shfl_idx(Rn, (lane & 32) | fwd_rs_lane<NV>(t));
        const float rs = rn == ninf ? 0.f : rn;
        const int mb = t >> 4, r = t & 15;
        float s = 0.f;
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) s += exp2_hw(__builtin_fmaf(acc[mb][nb][r], kk, -rs));
        v[t] = s;
      }
      const float tot2 = half_reduce_scatter<false>(v, lane);
      Rnew = Rn;
      Lnew = Rn == ninf ? 0.f : Lold * exp2_hw(Rold - Rn) + tot2;
    }
    if (!MASKED || jmine < b) {
      cR[jmine] = Rnew;
      cL[jmine] = Lnew;
    }
  }
}

template <int MB, int NB>
__global__ void __launch_bounds__(256, 2) fwd_sweep(FwdParams p) {
  using T = FwdTile<MB, NB>;
  __shared__ __attribute__((aligned(1024))) char lds_[2 * T::StageBytes];
  INFCL_LDS char* lds0 = (INFCL_LDS char*)lds_;
  INFCL_LDS char* lds1 = lds0 + T::StageBytes;
  split_limit_parts();
  const int lane = __lane_id();
  const int wave = threadIdx.x >> 6;
  const int l32 = lane & 31, h = lane >> 5;
  const int64_t b = p.b;
  const int nst = (int)((p.d * (int64_t)sizeof(float)) / 128);  // K-stages per tile (even)

  const int g = blockIdx.x % p.Pc;
  const int q = blockIdx.x / p.Pc;
  const int ct_lo = (int)(((int64_t)g * p.nCT) / p.Pc);
  const int ct_hi = (int)(((int64_t)(g + 1) * p.nCT) / p.Pc);
  const int ncol = ct_hi - ct_lo;
  const int nrow = q < p.nRT ? (p.nRT - 1 - q) / p.Pr + 1 : 0;
  const int ntile = ncol * nrow;
  if (ntile <= 0) return;

  const float k2 = p.scale[0] * kLog2e;
  const float ninf = -__builtin_inff();

  float rowR[NB], rowL[NB];
#pragma unroll
  for (int nb = 0; nb < NB; ++nb) {
    rowR[nb] = ninf;
    rowL[nb] = 0.f;
  }

  const auto dmo = fwd_dma_offsets<MB, NB>(p.d, (int)sizeof(float), wave, lane);
  int rr = 0, cc = 0;  // position of the current tile in this workgroup's (row, column) sweep
  fwd_stage_dma<MB, NB>(p, dmo, p.r0 + (int64_t)q * T::BI, (int64_t)ct_lo * T::BJ, 0, lds0, wave);
  wait_dma();
  __syncthreads();

  for (int tau = 0; tau < ntile; ++tau) {
    const int64_t i0 = p.r0 + (int64_t)(q + rr * p.Pr) * T::BI;
    const int64_t j0 = (int64_t)(ct_lo + cc) * T::BJ;
    const bool has_next = tau + 1 < ntile;
    const int nrr = cc + 1 == ncol ? rr + 1 : rr;
    const int ncc = cc + 1 == ncol ? 0 : cc + 1;
    const int64_t ni0 = p.r0 + (int64_t)(q + nrr * p.Pr) * T::BI;
    const int64_t nj0 = (int64_t)(ct_lo + ncc) * T::BJ;

    f32x16 acc[MB][NB];
#pragma unroll
    for (int mb = 0; mb < MB; ++mb)
#pragma unroll
      for (int nb = 0; nb < NB; ++nb)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[mb][nb][r] = 0.f;

    // The diagonal <img_i, txt_i> of the tile's rows, from the staged chunks by
    // fp32 FMAs (256 / BI threads per row): swapping the modalities gives the
    // same bits, which the split products' order does not.
    const bool diag = j0 < i0 + T::BI && i0 < j0 + T::BJ;
    constexpr int TPR = 256 / T::BI;
    const int il = threadIdx.x / TPR;
    const int jl = (int)(i0 - j0) + il;  // the row's own column, if in the tile
    const bool dhas = diag && jl >= 0 && jl < T::BJ;
    float dsum = 0.f;
    auto diag_stage = [&](const INFCL_LDS char* buf) {
      if (dhas) {
#pragma unroll
        for (int u = 0; u < 8 / TPR; ++u) {
          const int c = (threadIdx.x % TPR) + TPR * u, rt = T::BI + jl;
          const f32x4 x = *(const INFCL_LDS f32x4*)(buf + il * 128 + fwd_swz(il, c) * 16);
          const f32x4 y = *(const INFCL_LDS f32x4*)(buf + rt * 128 + fwd_swz(rt, c) * 16);
#pragma unroll
          for (int e = 0; e < 4; ++e) dsum = __builtin_fmaf(x[e], y[e], dsum);
        }
      }
    };
    for (int st = 0; st < nst; st += 2) {
      fwd_stage_dma<MB, NB>(p, dmo, i0, j0, st + 1, lds1, wave);
      fwd_stage_mfma<MB, NB>(lds0, acc, wave, lane);
      diag_stage(lds0);
      wait_dma();
      __syncthreads();
      if (st + 2 < nst)
        fwd_stage_dma<MB, NB>(p, dmo, i0, j0, st + 2, lds0, wave);
      else if (has_next)
        fwd_stage_dma<MB, NB>(p, dmo, ni0, nj0, 0, lds0, wave);
      fwd_stage_mfma<MB, NB>(lds1, acc, wave, lane);
      diag_stage(lds1);
      if (st + 2 < nst) {
        wait_dma();
        __syncthreads();
      }
    }

    // the next tile's first stage is in flight while the epilogue runs
    const bool special = diag || (i0 + T::BI > p.rend) || (j0 + T::BJ > b);
    if (special) {
      const int64_t jw = j0 + 32 * MB * wave + 4 * h;
      if (diag) {
#pragma unroll
        for (int k = 1; k < TPR; k <<= 1) dsum += shfl_xor(dsum, k);
        if (dhas && threadIdx.x % TPR == 0 && i0 + il < p.rend) p.udiag[i0 + il] = dsum;
      }
      // scaled exponents, -inf for the diagonal and for rows/columns past b
#pragma unroll
      for (int mb = 0; mb < MB; ++mb)
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) {
          const int64_t i = i0 + 32 * nb + l32;
#pragma unroll
          for (int r = 0; r < 16; ++r) {
            const int64_t j = jw + 32 * mb + 8 * (r >> 2) + (r & 3);
            const bool ok = i < p.rend && j < b && i != j;
            acc[mb][nb][r] = ok ? acc[mb][nb][r] * k2 : ninf;
          }
        }
      fwd_epilogue<true, MB, NB>(p, acc, rowR, rowL, j0, q, rr == 0, k2, wave, lane);
    } else {
      fwd_epilogue<false, MB, NB>(p, acc, rowR, rowL, j0, q, rr == 0, k2, wave, lane);
    }

    // end of a row tile: merge the two lane halves and publish one pair per wave
    if (cc + 1 == ncol) {
#pragma unroll
      for (int nb = 0; nb < NB; ++nb) {
        float R = rowR[nb], L = rowL[nb];
        lse2_merge(R, L, shfl_xor(rowR[nb], 32), shfl_xor(rowL[nb], 32));
        const int64_t i = i0 + 32 * nb + l32;
        if (h == 0 && i < p.rend) {
          const int64_t slot = (int64_t)(g * 4 + wave) * p.rstride + (i - p.r0);
          p.rowR[slot] = R;
          p.rowL[slot] = L;
        }
        rowR[nb] = ninf;
        rowL[nb] = 0.f;
      }
    }
    rr = nrr;
    cc = ncc;

    if (has_next) {
      wait_dma();
      __syncthreads();
    }
  }
}

// ---------------------------------------------------------------- finalize
// Per-sample terms of samples [r0, r0 + n) (all b for the whole batch, a
// shard's own samples otherwise).  Sample r0 + t takes its row pair from the
// nrowpart partials at rowR/rowL[k rstride + t] and its column pair from the
// ncolpart partials at colR/colL[k cstride + t].
struct FinParams {
  int64_t r0, n;
  const float* scale;
  const float* rowR;
  const float* rowL;
  int nrowpart;
  int64_t rstride;
  const float* colR;
  const float* colL;
  int ncolpart;
  int64_t cstride;
  const float* udiag;  // [b], by sample index
  float* lse_r;        // [n]
  float* lse_c;        // [n]
  float* aux;          // [3n]: l^r, l^c, u_ii
  double* partial;     // [gridDim.x]
};

// One workgroup finishes 32 samples: thread (t, g) of 32 x 8 takes every eighth
// partial pair of sample t from pair g on (32 samples' pairs of one slot are
// one 128-byte line), and the eight parts meet in LDS.  With one thread per
// sample the 16 to 96 fp64 exponentials of a sample were one serial chain:
// 12 us at 40 pairs and 21 us at 96 whatever the batch, against 7 and 10 us
// (25 against 17 us at b = 131072, where it is 1e-4 of the forward).
constexpr int kFinT = 32, kFinG = 8;

// Level M and sum S (log2 S + M the merged value) of the n base-2 partial pairs
// (R, l) of sample t at R/L[k stride + t], in every thread of the sample; an
// empty pair (R = -inf) weighs zero.  Each thread keeps up to eight pairs in
// registers.  The order of the additions is fixed by n alone.
__device__ __forceinline__ void merge_parts(const float* R, const float* L, int n, int64_t stride, int64_t t, bool ok,
                                            int tl, int g, float (*sm)[kFinT], double (*ss)[kFinT], float& M,
                                            double& S) {
  M = -__builtin_inff();
  float r[8], l[8];
#pragma unroll
  for (int u = 0; u < 8; ++u) {
    const int k = g + kFinG * u;
    const bool in = ok && k < n;
    r[u] = in ? R[(int64_t)k * stride + t] : -__builtin_inff();
    l[u] = in ? L[(int64_t)k * stride + t] : 0.f;
    M = fmaxf(M, r[u]);
  }
  for (int k = g + kFinG * 8; k < n; k += kFinG)
    if (ok) M = fmaxf(M, R[(int64_t)k * stride + t]);
  sm[g][tl] = M;
  __syncthreads();
#pragma unroll
  for (int k = 0; k < kFinG; ++k) M = fmaxf(M, sm[k][tl]);
  S = 0.0;
  if (M != -__builtin_inff()) {
#pragma unroll
    for (int u = 0; u < 8; ++u)
      if (r[u] != -__builtin_inff()) S += (double)l[u] * exp2((double)r[u] - (double)M);
    for (int k = g + kFinG * 8; k < n; k += kFinG)
      if (ok) {
        const float rk = R[(int64_t)k * stride + t];
        if (rk != -__builtin_inff()) S += (double)L[(int64_t)k * stride + t] * exp2((double)rk - (double)M);
      }
  }
  ss[g][tl] = S;
  __syncthreads();
  S = 0.0;
#pragma unroll
  for (int k = 0; k < kFinG; ++k) S += ss[k][tl];
}
// ... as a natural-log log-sum-exp over the off-diagonal entries
__device__ __forceinline__ double merged_lse(float M, double S) {
  return M == -__builtin_inff() ? -__builtin_inf() : ((double)M + log2(S)) * 0.6931471805599453;
}

__device__ __forceinline__ double softplus64(double z) {
  if (z == -__builtin_inf()) return 0.0;
  return fmax(z, 0.0) + log1p(exp(-fabs(z)));
}

__global__ void __launch_bounds__(256) fwd_finalize(FinParams p) {
  __shared__ float smr[kFinG][kFinT], smc[kFinG][kFinT];
  __shared__ double ssr[kFinG][kFinT], ssc[kFinG][kFinT], red[kFinT];
  const int tl = threadIdx.x & (kFinT - 1), g = threadIdx.x / kFinT;
  const int64_t t = (int64_t)blockIdx.x * kFinT + tl;
  const bool ok = t < p.n;
  float Mr, Mc;
  double Sr, Sc;
  merge_parts(p.rowR, p.rowL, p.nrowpart, p.rstride, t, ok, tl, g, smr, ssr, Mr, Sr);
  merge_parts(p.colR, p.colL, p.ncolpart, p.cstride, t, ok, tl, g, smc, ssc, Mc, Sc);
  if (g == 0) {
    const double offr = merged_lse(Mr, Sr), offc = merged_lse(Mc, Sc);
    double contrib = 0.0;
    if (ok) {
      const double u = (double)p.udiag[p.r0 + t];
      const double x = (double)p.scale[0] * u;
      const double er = softplus64(offr - x);  // r_i - x_ii, cancellation-free
      const double ec = softplus64(offc - x);
      p.lse_r[t] = (float)(x + er);
      p.lse_c[t] = (float)(x + ec);
      p.aux[t] = (float)er;
      p.aux[p.n + t] = (float)ec;
      p.aux[2 * p.n + t] = (float)u;
      contrib = er + ec;
    }
    red[tl] = contrib;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    double c = 0.0;
    for (int k = 0; k < kFinT; ++k) c += red[k];
    p.partial[blockIdx.x] = c;
  }
}

// Sharded forward: one base-2 pair per column j in [0, b) over this shard's
// rows, merged from the ncolpart row-group partials (colR/colL[k b + j]) in a
// fixed order: out[j] = R, out[b + j] = l.  This is what the column owner
// receives from every shard.
__global__ void __launch_bounds__(256) fwd_col_pairs(const float* colR, const float* colL, int ncolpart, int64_t b,
                                                     float* out) {
  __shared__ float sm[kFinG][kFinT];
  __shared__ double ss[kFinG][kFinT];
  const int tl = threadIdx.x & (kFinT - 1), g = threadIdx.x / kFinT;
  const int64_t j = (int64_t)blockIdx.x * kFinT + tl;
  float M;
  double S;
  merge_parts(colR, colL, ncolpart, b, j, j < b, tl, g, sm, ss, M, S);
  if (g == 0 && j < b) {
    out[j] = M;
    out[b + j] = (float)S;
  }
}

// Fixed-order sum of `n` fp64 partials, times `mul`; one workgroup.
__global__ void __launch_bounds__(256) sum_partials(const double* part, int64_t n, double mul, float* out32,
                                                    double* out64) {
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
    double v = red[0] * mul;
    if (out32) *out32 = (float)v;
    if (out64) *out64 = v;
  }
}

// ------------------------------------------------------------ host launchers
bool fwd2_supported(int64_t d, int dtype);
void fwd2_grid(int64_t b, int64_t nrows, int64_t d, int* Pr, int* Pc);
int launch_fwd2(const void* img, const void* txt, int64_t b, int64_t d, int dtype, int64_t r0, int64_t nrows,
                const float* scale, float* rowR, float* rowL, float* colR, float* colL, float* udiag, float* ref2,
                hipStream_t stream);

// Tile shape of the streamed-tiles sweep for nrows own rows against b columns:
// 64 x 256, unless so few tiles leave compute units idle (a tile's K-stages are
// a serial chain: b = 1024, d = 512 takes 44 us in 64 tiles of 64 x 256, 20
// in 256 of 32 x 128).
static int fwd1_shape(int64_t b, int64_t nrows) {
  return ((nrows + 63) / 64) * ((b + 255) / 256) >= 192 ? 2 : 1;  // MB = NB
}

// Grid of the streamed-tiles sweep: Pc column groups (one per XCD when there
// are enough column tiles) times Pr row groups, about two workgroups per
// compute unit.
void fwd1_grid(int64_t b, int64_t nrows, int* Pr, int* Pc) {
  const int64_t s = fwd1_shape(b, nrows);
  const int64_t nRT = (nrows + 32 * s - 1) / (32 * s), nCT = (b + 128 * s - 1) / (128 * s);
  *Pc = (int)(nCT < 8 ? nCT : 8);
  *Pr = (int)(nRT < 64 ? nRT : 64);
}

// Most partial pairs per sample that the grid of any nrows <= b leaves.
int fwd1_pairs(int64_t b) {
  const int64_t r = (b + 31) / 32, c = (b + 127) / 128;
  return (int)((r < 64 ? r : 64) + 4 * (c < 8 ? c : 8));
}

static int launch_fwd1(const void* img, const void* txt, int64_t b, int64_t d, int dtype, int64_t r0, int64_t nrows,
                       const float* scale, hipStream_t stream, float* rowR, float* rowL, float* colR, float* colL,
                       float* udiag) {
  FwdParams p;
  p.img = img;
  p.txt = txt;
  p.b = b;
  p.d = d;
  p.scale = scale;
  p.rowR = rowR;
  p.rowL = rowL;
  p.colR = colR;
  p.colL = colL;
  p.udiag = udiag;
  fwd1_grid(b, nrows, &p.Pr, &p.Pc);
  const int64_t s = fwd1_shape(b, nrows);
  p.nRT = (int)((nrows + 32 * s - 1) / (32 * s));
  p.nCT = (int)((b + 128 * s - 1) / (128 * s));
  p.r0 = r0;
  p.rend = r0 + nrows;
  p.rstride = nrows;
  if (dtype != 1) return 2;  // every supported 16-bit width takes the resident-rows sweep
  if (s == 2)
    hipLaunchKernelGGL((fwd_sweep<2, 2>), dim3(p.Pr * p.Pc), dim3(256), 0, stream, p);
  else
    hipLaunchKernelGGL((fwd_sweep<1, 1>), dim3(p.Pr * p.Pc), dim3(256), 0, stream, p);
  return hipGetLastError() == hipSuccess ? 0 : 1;
}

// Partial pairs per own row and per column that the sweep over nrows own rows
// leaves.
static void sweep_parts(int64_t b, int64_t d, int dtype, int64_t nrows, int* nrowpart, int* ncolpart) {
  int Pr = 0, Pc = 0;
  if (fwd2_supported(d, dtype)) {
    fwd2_grid(b, nrows, d, &Pr, &Pc);
    *nrowpart = Pc;
  } else {
    fwd1_grid(b, nrows, &Pr, &Pc);
    *nrowpart = Pc * 4;
  }
  *ncolpart = Pr;
}

// The four arrays of partial pairs inside their region: nrowpart x nrows row
// pairs, ncolpart x b column pairs, each array on a 256-byte boundary.
struct PairPtrs {
  float *rowR, *rowL, *colR, *colL;
};
static PairPtrs pair_ptrs(float* pairs, int nrowpart, int64_t nrows, int ncolpart, int64_t b) {
  const int64_t nr = ((int64_t)nrowpart * nrows + 63) / 64 * 64, nc = ((int64_t)ncolpart * b + 63) / 64 * 64;
  return PairPtrs{pairs, pairs + nr, pairs + 2 * nr, pairs + 2 * nr + nc};
}

// The sweep over own rows [r0, r0 + nrows) against all b columns: 16-bit
// inputs with d a multiple of 128 up to 1024 take the resident-rows sweep, everything else the
// streamed-tiles sweep above.  Both leave partial pairs: nrowpart per own row
// (stride nrows, by row - r0) and ncolpart per column (stride b).
static int launch_sweep(const void* img, const void* txt, int64_t b, int64_t d, int dtype, int64_t r0, int64_t nrows,
                        const float* scale, float* pairs, float* udiag, float* ref2, hipStream_t stream,
                        int* nrowpart, int* ncolpart, PairPtrs* pp) {
  sweep_parts(b, d, dtype, nrows, nrowpart, ncolpart);
  *pp = pair_ptrs(pairs, *nrowpart, nrows, *ncolpart, b);
  if (fwd2_supported(d, dtype))
    return launch_fwd2(img, txt, b, d, dtype, r0, nrows, scale, pp->rowR, pp->rowL, pp->colR, pp->colL, udiag, ref2,
                       stream);
  return launch_fwd1(img, txt, b, d, dtype, r0, nrows, scale, stream, pp->rowR, pp->rowL, pp->colR, pp->colL, udiag);
}

static int launch_finalize(int64_t r0, int64_t n, double loss_mul, const float* scale, float* loss, double* loss64,
                           float* lse_r, float* lse_c, float* aux, const float* rowR, const float* rowL, int nrowpart,
                           int64_t rstride, const float* colR, const float* colL, int ncolpart, int64_t cstride,
                           const float* udiag, double* partial, hipStream_t stream) {
  FinParams f;
  f.r0 = r0;
  f.n = n;
  f.scale = scale;
  f.rowR = rowR;
  f.rowL = rowL;
  f.nrowpart = nrowpart;
  f.rstride = rstride;
  f.colR = colR;
  f.colL = colL;
  f.ncolpart = ncolpart;
  f.cstride = cstride;
  f.udiag = udiag;
  f.lse_r = lse_r;
  f.lse_c = lse_c;
  f.aux = aux;
  f.partial = partial;
  const int nfin = (int)((n + kFinT - 1) / kFinT);
  hipLaunchKernelGGL(fwd_finalize, dim3(nfin), dim3(256), 0, stream, f);
  if (hipGetLastError() != hipSuccess) return 1;
  hipLaunchKernelGGL(sum_partials, dim3(1), dim3(256), 0, stream, (const double*)partial, (int64_t)nfin, loss_mul,
                     loss, loss64);
  return hipGetLastError() == hipSuccess ? 0 : 1;
}

// Forward over the whole batch: the sweep over all rows, then the finalize of
// every sample and the loss.
int launch_fwd(const void* img, const void* txt, int64_t b, int64_t d, int dtype, const float* scale, float* loss,
               double* loss64, float* lse_r, float* lse_c, float* aux, hipStream_t stream, float* pairs, float* udiag,
               float* ref2, double* partial) {
  int nrowpart = 0, ncolpart = 0;
  PairPtrs pp;
  const int rc =
      launch_sweep(img, txt, b, d, dtype, 0, b, scale, pairs, udiag, ref2, stream, &nrowpart, &ncolpart, &pp);
  if (rc != 0) return rc;
  return launch_finalize(0, b, 1.0 / (2.0 * (double)b), scale, loss, loss64, lse_r, lse_c, aux, pp.rowR, pp.rowL,
                         nrowpart, b, pp.colR, pp.colL, ncolpart, b, udiag, partial, stream);
}

// Sharded forward, local part: the sweep over own rows [r0, r0 + nrows), row
// partials left in the workspace, and one base-2 pair per column over the own
// rows written to colpair ([2b]: R then l).
int launch_fwd_shard(const void* img, const void* txt, int64_t b, int64_t d, int dtype, int64_t r0, int64_t nrows,
                     const float* scale, float* colpair, hipStream_t stream, float* pairs, float* udiag, float* ref2) {
  int nrowpart = 0, ncolpart = 0;
  PairPtrs pp;
  const int rc =
      launch_sweep(img, txt, b, d, dtype, r0, nrows, scale, pairs, udiag, ref2, stream, &nrowpart, &ncolpart, &pp);
  if (rc != 0) return rc;
  hipLaunchKernelGGL(fwd_col_pairs, dim3((unsigned)((b + kFinT - 1) / kFinT)), dim3(256), 0, stream, (const float*)pp.colR,
                     (const float*)pp.colL, ncolpart, b, colpair);
  return hipGetLastError() == hipSuccess ? 0 : 1;
}

// Sharded forward, owner part: the per-sample terms of own samples [r0, r0 +
// nrows) from the row partials of launch_fwd_shard and the nparts column pairs
// received for the own columns (colpairs: [nparts][2 nrows], R then l), and
// this shard's share of the loss, sum of (l^r + l^c) / (2b), into loss_part.
int launch_fwd_shard_finish(int64_t b, int64_t d, int dtype, int64_t r0, int64_t nrows, int64_t nparts,
                            const float* colpairs, const float* scale, float* lse_r, float* lse_c, float* aux,
                            double* loss_part, hipStream_t stream, float* pairs, const float* udiag, double* partial) {
  int nrowpart = 0, ncolpart = 0;
  sweep_parts(b, d, dtype, nrows, &nrowpart, &ncolpart);
  const PairPtrs pp = pair_ptrs(pairs, nrowpart, nrows, ncolpart, b);
  return launch_finalize(r0, nrows, 1.0 / (2.0 * (double)b), scale, nullptr, loss_part, lse_r, lse_c, aux, pp.rowR,
                         pp.rowL, nrowpart, nrows, colpairs, colpairs + nrows, (int)nparts, 2 * nrows, udiag, partial,
                         stream);
}

}  // namespace infcl
