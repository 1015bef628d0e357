// Backward sweep for fp32 rows in a single pass (gfx950).
//
// Same quantities as the 16-bit sweeps (bwd.hip, bwd_wide.hip).  The products
// run on the bf16 MFMA with every fp32 operand as three bf16 parts (split3 in
// common.hpp: exact parts, products dropped below fp32's own rounding), fp32
// accumulation throughout: six 32-cycle MFMAs where the fp32 MFMA needs eight
// of 64 cycles.  A workgroup owns 64 rows; the wave pair (2 ob, 2 ob + 1) shares
// own block ob (32 rows): each wave contracts every other 16-feature step of
// GEMM1 (its own rows' parts held in registers) and owns every other
// 32-feature block of the gradient.  Per tile of 32 swept rows, whose parts lie
// in LDS as three bf16 planes in the swept-tile layout:
//   loads  of the next tile into registers (plain range-checked loads);
//   GEMM1  partial S^T (32 swept x 32 own) over the wave's steps;
//   join   each wave hands its partner the 8 accumulator entries per lane the
//          partner finishes and adds the partner's half of its own 8;
//   G'     two exp2 per entry, the diagonal from expm1 terms; the 8 values are
//          handed to the partner lane by lane: a lane's 8 + 8 values, split, are
//          the A operand of GEMM2 as they are;
//   GEMM2  32 own rows x the wave's feature blocks (transposing reads);
//   split  of the next tile, once per workgroup, written to the planes between
//          two barriers.
// The step's figures (backward, both sides): with 128 own rows on the fp32 MFMA
// d = 512 b = 8192 took 3.78 ms (two passes, spilling) and d = 256 1.07 ms;
// this form with the fp32 MFMA 2.05 ms at d = 512 (86% of its rate); split
// products, every wave splitting the fragments it reads, 1.69 and 0.91 ms (2000
// vector instructions per tile beside 192 MFMAs); split once per tile 1.53 and
// 0.81 ms; the split interleaved with GEMM2 1.40 and 0.78 ms.  The gradients'
// error against fp64 fell from 3.3e-6 to 5.5e-7 (d = 512, b = 1024).
#include "bwd.hpp"

namespace infcl {

template <int D>
__global__ void __launch_bounds__(256, 1) bwd_f32(BwdParams p) {
  constexpr int KH = D / 32;            // 16-feature steps of GEMM1 per wave
  constexpr int ROWG = D * 4;           // bytes per row
  constexpr int TILEB = kBwdBN * ROWG;  // bytes per swept tile
  constexpr int NLD = D / 64;           // 8-feature chunks a lane loads and splits per tile
  constexpr int PLANEB = kSeg * ((D + 127) / 128);  // one bf16 plane of a tile
  constexpr int FBW = D / 64;           // 32-feature gradient blocks per wave
  static_assert(D % 64 == 0 && 3 * PLANEB + 2 * 8192 <= 160 * 1024, "LDS budget");
  __shared__ __attribute__((aligned(1024))) char planes_[3 * PLANEB];
  __shared__ __attribute__((aligned(16))) float xs_[4][64][8];  // join
  __shared__ __attribute__((aligned(16))) float xg_[4][64][8];  // G'
  INFCL_LDS char* const planes = (INFCL_LDS char*)planes_;

  split_limit_parts();
  const int lane = __lane_id();
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int ob = wave >> 1, kh = wave & 1;
  const int l32 = lane & 31, h = lane >> 5;
  const BwdTask task = bwd_task(p, kWideBM * D);
  const BwdSide& sd = p.side[task.sd];
  const char* const swept = (const char*)sd.swept + (int64_t)task.row0 * ROWG;
  const float* const lse2_swept = sd.lse2_swept + task.row0;
  const int rows = task.rows, ntile = (rows + kBwdBN - 1) / kBwdBN;
  const int64_t wg0 = p.own_off + (int64_t)task.rb * kWideBM;  // own_off is a multiple of 32
  const int64_t own0 = wg0 + 32 * ob;
  const int64_t iown = own0 + l32;
  const bool own_ok = iown < p.own_end;
  const int64_t irow = own_ok ? iown : p.own_end - 1;
  const int own0_t = (int)(own0 - task.row0);  // counted from the first swept row

  const float s = p.scale[0];
  const float k2 = s * kLog2e;
  const float dl = p.dloss ? p.dloss[0] : 1.0f;

  // G' is split into bf16 parts too: scaled by alpha = 2^g16e before, so that
  // the low parts of small weights stay normal.  alpha is divided out of the
  // sums and not of kfin, which is small by itself (dloss, 1/2b) and could
  // leave the normal numbers where the gradients do not.
  const int g16e = g16_exponent<0>(p.g16);
  const float g16a = ldexpf(1.f, g16e), g16inv = ldexpf(1.f, -g16e);
  const float kfin = dl * s / (2.0f * (float)p.b);

  // own operand: row irow, features 16 (2 s2 + kh) + 8h .. +8
  split3 ownf[KH];
  {
    const float* src = (const float*)sd.own + irow * D + 16 * kh + 8 * h;
#pragma unroll
    for (int s2 = 0; s2 < KH; ++s2)
      ownf[s2] = split_f32(*(const f32x4*)(src + 32 * s2), *(const f32x4*)(src + 32 * s2 + 4));
  }
  const float aO = own_ok ? sd.lse_own[iown] * kLog2e : 0.f;
  const float uO = own_ok ? p.udiag[iown] : 0.f;
  const float gdiag = own_ok ? expm1f(-sd.ell_own[iown]) + expm1f(-sd.ell_swept[iown]) : 0.f;

  // a tile's loads: lane of thread tid takes row tid >> 3, chunks (tid & 7) + 8 k
  f32x4 raw[NLD][2];
  const int ldv = (int)(threadIdx.x >> 3) * ROWG + 32 * (int)(threadIdx.x & 7);
  auto load_tile = [&](int jt) {
    int n = rows - jt * kBwdBN < kBwdBN ? rows - jt * kBwdBN : kBwdBN;
    asm("" : "+s"(n));  // (scalar clamp, as in sweep_tile_rsrc)
    const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc(
        (void*)(swept + (int64_t)jt * TILEB), (short)0, n > 0 ? n * ROWG : 0, 0x00020000);
#pragma unroll
    for (int k = 0; k < NLD; ++k)
#pragma unroll
      for (int u = 0; u < 2; ++u)
        raw[k][u] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(r, ldv + 256 * k + 16 * u, 0, 0));
  };
  // ... split and written to the planes: chunk (tid & 7) + 8 k of the row
  int offW[2];
#pragma unroll
  for (int k = 0; k < 2; ++k) offW[k] = sweep_seg_off(threadIdx.x >> 3, (threadIdx.x & 7) + 8 * k);
  auto put_tile = [&](const u32x4 (&t)[NLD][3]) {
#pragma unroll
    for (int k = 0; k < NLD; ++k)
#pragma unroll
      for (int q = 0; q < 3; ++q)
        *(INFCL_LDS u32x4*)(planes + PLANEB * q + kSeg * (k >> 1) + offW[k & 1]) = t[k][q];
  };
  // GEMM1's swept fragments: step s2 at plane + kSeg (s2 >> 2) + offA[s2 & 3].
  // The kh = 1 wave takes the tile's row halves swapped, so that accumulator
  // entries 0..7 of either wave are the ones it finishes (tile rows 16 kh + 8 h + i).
  int offA[4];
#pragma unroll
  for (int k = 0; k < 4; ++k) offA[k] = sweep_seg_off(sweep_perm(l32) ^ (16 * kh), 2 * (2 * k + kh) + h);
  // GEMM2's transposing reads of block 2 fb + kh, rows 16 kk ..:
  // plane + kSeg (fb >> 1) + 16 kSegRow kk + offB[fb & 1][tt]
  int offB[2][2];
#pragma unroll
  for (int k = 0; k < 2; ++k)
#pragma unroll
    for (int tt = 0; tt < 2; ++tt) offB[k][tt] = sweep_tr_off(lane, tt, 2 * k + kh);
  // base-2 log-sum-exp of the 8 swept rows whose entries the lane forms
  auto load_L = [&](int jt, f32x4& A, f32x4& B) {
    const int j0 = jt * kBwdBN;
    int n = rows - j0 < kBwdBN ? rows - j0 : kBwdBN;
    asm("" : "+s"(n));  // (scalar clamp, as in sweep_tile_rsrc)
    const __amdgpu_buffer_rsrc_t r =
        __builtin_amdgcn_make_buffer_rsrc((void*)(lse2_swept + j0), (short)0, n > 0 ? 4 * n : 0, 0x00020000);
    const int vo = 4 * (16 * kh + 8 * h);
    A = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(r, vo, 0, 0));
    B = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(r, vo + 16, 0, 0));
  };

  double ds_acc = 0.0;
  f32x16 dacc[FBW];
#pragma unroll
  for (int i = 0; i < FBW; ++i)
#pragma unroll
    for (int r = 0; r < 16; ++r) dacc[i][r] = 0.f;
  auto gp_entry = [&](float x, float Lj, float& ds) {
    const float pO = exp2_hw(__builtin_fmaf(x, k2, -aO));
    const float pS = exp2_hw(__builtin_fmaf(x, k2, -Lj));
    ds = __builtin_fmaf(pO, x - uO, ds);
    return (pO + pS) * g16a;
  };

  auto body = [&](int jt) {
    f32x4 L0, L1;
    load_L(jt, L0, L1);
    load_tile(jt + 1);
    // ---- GEMM1, two accumulation chains
    f32x16 s0, s1;
#pragma unroll
    for (int r = 0; r < 16; ++r) s0[r] = s1[r] = 0.f;
    // (fragments read one step ahead; each step a scheduling region)
    split3 ring[2];
    auto readA = [&](int s2, split3& a) {
#pragma unroll
      for (int q = 0; q < 3; ++q)
        a.p[q] = *(const INFCL_LDS bf16x8*)(planes + PLANEB * q + kSeg * (s2 >> 2) + offA[s2 & 3]);
    };
    readA(0, ring[0]);
#pragma unroll
    for (int s2 = 0; s2 < KH; ++s2) {
      if (s2 + 1 < KH) readA(s2 + 1, ring[(s2 + 1) & 1]);
      mfma_split(ring[s2 & 1], ownf[s2], s0, s1);
      __builtin_amdgcn_sched_barrier(0);
    }
    // ---- join
    float x[8];
    {
      f32x4 o0, o1;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        x[i] = s0[i] + s1[i];
        x[4 + i] = s0[4 + i] + s1[4 + i];
        o0[i] = s0[8 + i] + s1[8 + i];
        o1[i] = s0[12 + i] + s1[12 + i];
      }
      *(INFCL_LDS f32x4*)&xs_[wave][lane][0] = o0;
      *(INFCL_LDS f32x4*)&xs_[wave][lane][4] = o1;
    }
    __syncthreads();
    {
      const f32x4 q0 = *(const INFCL_LDS f32x4*)&xs_[wave ^ 1][lane][0];
      const f32x4 q1 = *(const INFCL_LDS f32x4*)&xs_[wave ^ 1][lane][4];
#pragma unroll
      for (int i = 0; i < 8; ++i) x[i] += i < 4 ? q0[i] : q1[i - 4];
    }
    // ---- G' (entry i <-> tile row 16 kh + 8 h + i)
    float gv[8], ds_t = 0.f;
#pragma unroll
    for (int i = 0; i < 8; ++i) gv[i] = gp_entry(x[i], i < 4 ? L0[i] : L1[i - 4], ds_t);
    const int j0 = jt * kBwdBN;
    if ((j0 == own0_t) || (j0 + kBwdBN > rows)) {
      // tile on the diagonal or past the end: masked entries
      ds_t = 0.f;
      const int jl = j0 + 16 * kh + 8 * h, iown_t = own0_t + l32;
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        float dsv = 0.f;
        const float gg = gp_entry(x[i], i < 4 ? L0[i] : L1[i - 4], dsv);
        const bool ok = jl + i < rows;
        const bool dg = jl + i == iown_t;
        gv[i] = ok ? (dg ? gdiag * g16a : gg) : 0.f;
        ds_t += (ok & !dg) ? dsv : 0.f;
      }
    }
    ds_acc += (double)ds_t;
    *(INFCL_LDS f32x4*)&xg_[wave][lane][0] = f32x4{gv[0], gv[1], gv[2], gv[3]};
    *(INFCL_LDS f32x4*)&xg_[wave][lane][4] = f32x4{gv[4], gv[5], gv[6], gv[7]};
    __syncthreads();
    split3 A[2];  // A[kk]: G' of the lane's own row against tile rows 16 kk + 8 h + (0 .. 7)
    {
      const f32x4 q0 = *(const INFCL_LDS f32x4*)&xg_[wave ^ 1][lane][0];
      const f32x4 q1 = *(const INFCL_LDS f32x4*)&xg_[wave ^ 1][lane][4];
      float A0[8], A1[8];
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const float o = i < 4 ? q0[i] : q1[i - 4];
        A0[i] = kh ? o : gv[i];
        A1[i] = kh ? gv[i] : o;
      }
      A[0] = split_f32(A0);
      A[1] = split_f32(A1);
    }
    // ---- GEMM2: fragments read one group ahead; between a group's six MFMAs,
    // half a chunk of the next tile's split (22 instructions)
    u32x4 nt[NLD][3];
    auto readB = [&](int g, bf16x8 (&B)[3]) {
      const int fb = g >> 1, kk = g & 1;
#pragma unroll
      for (int q = 0; q < 3; ++q) {
        s16x4 t[2];
#pragma unroll
        for (int tt = 0; tt < 2; ++tt)
          t[tt] = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
              (INFCL_LDS s16x4*)(planes + PLANEB * q + kSeg * (fb >> 1) + 16 * kSegRow * kk + offB[fb & 1][tt]));
        const s16x8 bb = {t[0][0], t[0][1], t[0][2], t[0][3], t[1][0], t[1][1], t[1][2], t[1][3]};
        B[q] = __builtin_bit_cast(bf16x8, bb);
      }
    };
    bf16x8 Bq[2][3];
    readB(0, Bq[0]);
#pragma unroll
    for (int g = 0; g < 2 * FBW; ++g) {
      const int fb = g >> 1, kk = g & 1;
      if (g + 1 < 2 * FBW) readB(g + 1, Bq[(g + 1) & 1]);
      const bf16x8(&B)[3] = Bq[g & 1];
      split_pair(raw[fb][kk][0], raw[fb][kk][1], 2 * kk, nt[fb]);
      split_pair(raw[fb][kk][2], raw[fb][kk][3], 2 * kk + 1, nt[fb]);
      dacc[fb] = mfma_bf16(A[kk].p[2], B[0], dacc[fb]);
      dacc[fb] = mfma_bf16(A[kk].p[0], B[2], dacc[fb]);
      dacc[fb] = mfma_bf16(A[kk].p[1], B[1], dacc[fb]);
      dacc[fb] = mfma_bf16(A[kk].p[1], B[0], dacc[fb]);
      dacc[fb] = mfma_bf16(A[kk].p[0], B[1], dacc[fb]);
      dacc[fb] = mfma_bf16(A[kk].p[0], B[0], dacc[fb]);
#pragma unroll
      for (int i = 0; i < 6; ++i) {
        __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);  // LDS read
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);  // MFMA
        __builtin_amdgcn_sched_group_barrier(0x002, 4, 0);  // VALU
      }
      __builtin_amdgcn_sched_barrier(0);
    }
    __syncthreads();  // every wave has read the planes and the exchange areas
    put_tile(nt);
    __syncthreads();
  };
  {
    load_tile(0);
    u32x4 nt[NLD][3];
#pragma unroll
    for (int k = 0; k < NLD; ++k)
#pragma unroll
      for (int e = 0; e < 4; ++e) split_pair(raw[k][e >> 1][2 * (e & 1)], raw[k][e >> 1][2 * (e & 1) + 1], e, nt[k]);
    put_tile(nt);
  }
  __syncthreads();
  for (int jt = 0; jt < ntile; ++jt) body(jt);

  // ---- write dOwn (or this part's unscaled sums): lane holds feature l32 of
  // block 2 fb + kh, rows 8 (r >> 2) + 4 h + (r & 3) of own block ob
  const int f0 = 32 * kh + l32;
  if (task.part) {
    float* dst = task.part + (32 * ob + 4 * h) * D + f0;
#pragma unroll
    for (int fb = 0; fb < FBW; ++fb)
#pragma unroll
      for (int r = 0; r < 16; ++r) dst[(8 * (r >> 2) + (r & 3)) * D + 64 * fb] = dacc[fb][r];
  } else {
    const bool all_ok = own0 + 32 <= p.own_end;
    float* dst = (float*)sd.dOwn + (own0 - p.own_off + 4 * h) * D + f0;
#pragma unroll
    for (int fb = 0; fb < FBW; ++fb)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int64_t row = own0 + 8 * (r >> 2) + 4 * h + (r & 3);
        if (all_ok || row < p.own_end) dst[(8 * (r >> 2) + (r & 3)) * D + 64 * fb] = kfin * (g16inv * dacc[fb][r]);
      }
  }

  // ---- dscale partial: fixed-order reduction in the (now free) join area
  double* red = (double*)&xs_[0][0][0];
  red[threadIdx.x] = own_ok ? ds_acc : 0.0;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if ((int)threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x == 0) p.ds_part[blockIdx.x] = red[0];
}

int launch_bwd_f32(const BwdParams& p, int nwg, hipStream_t stream) {
  switch (p.d) {
    case 64: hipLaunchKernelGGL(bwd_f32<64>, dim3(nwg), dim3(256), 0, stream, p); break;
    case 128: hipLaunchKernelGGL(bwd_f32<128>, dim3(nwg), dim3(256), 0, stream, p); break;
    case 192: hipLaunchKernelGGL(bwd_f32<192>, dim3(nwg), dim3(256), 0, stream, p); break;
    case 256: hipLaunchKernelGGL(bwd_f32<256>, dim3(nwg), dim3(256), 0, stream, p); break;
    case 320: hipLaunchKernelGGL(bwd_f32<320>, dim3(nwg), dim3(256), 0, stream, p); break;
    case 384: hipLaunchKernelGGL(bwd_f32<384>, dim3(nwg), dim3(256), 0, stream, p); break;
    case 448: hipLaunchKernelGGL(bwd_f32<448>, dim3(nwg), dim3(256), 0, stream, p); break;
    case 512: hipLaunchKernelGGL(bwd_f32<512>, dim3(nwg), dim3(256), 0, stream, p); break;
    default: return 2;
  }
  return hipGetLastError() == hipSuccess ? 0 : 1;
}

}  // namespace infcl
