// e4m3 and MXFP4 grouped expert GEMMs of batches with few rows per expert
// (row alignment 128: fewer than 256 pairs per local expert on average, up to
// 1024 where 256-row tiles would leave half the CUs idle).
//
// Such a batch reads every touched expert's weights once for a few rows.  A CU
// requests some 25 to 31 GB/s here, rows (from L2) and weights (from HBM) alike
// (24 GB/s when everything streams from HBM), so a launch lasts as long as the
// bytes its busiest CU requests:
//   * rows are loaded and multiplied in the pieces that hold rows (8-row load
//     segments, 16-row MFMA fragments): a tile of 20 rows requests 3 KB of
//     rows per K step where a whole 128-row tile requested 16 KB;
//   * tiles are 128 columns wide (MXFP4, whose columns are half the bytes, 256
//     from 64 pairs per expert on), so that a batch of a few experts has
//     several work items per CU, and two to four workgroups share a CU: the
//     loads of one proceed while another waits at its step's barrier;
//   * the work order (deal_item) keeps an expert's tiles of one column slice on
//     one XCD at one time, which then reads that weight slice once, and deals
//     the slices round to the XCDs: with contiguous shares a hot expert's
//     tiles fell to one XCD (e4m3, Zipf(1.2) routing, 130 rows per expert:
//     167 -> 138 us GEMM1; equal on balanced routing).  The 64-row MXFP4 tiles
//     keep contiguous shares: a little faster beside another batch's GEMMs
//     (64 batches of 24 rows per expert on two streams: 6.22 against 6.40 ms),
//     equal under skewed routing.  All M tiles of a slice in a row (column
//     major) was slower in both (6.52 ms).
// BM 64, or 160 (e4m3) or 128 (MXFP4) rows: batch_plan.  160 rows are the most
// that let two workgroups share a CU; a batch of 130 rows per expert then needs
// one tile per expert where 128 rows need two, the second of them a pass over
// the weights for a few rows (16 experts, d 7168, I 2048, 133 rows: GEMM1 + GEMM2
// 227 -> 189 us).  A 160 x 256 MXFP4 tile spills registers.
// Measured against the 128 x 256 tiles of whole rows that this file replaced
// (16 experts, GEMM1 + GEMM2):
//   e4m3  d 7168, I 2048: 33 rows per expert 165 -> 148 us, 133: 259 -> 189;
//         d 6144, I 2560: 20 rows 230 -> 157 us; d 2048, I 1024: 32 rows
//         49 -> 28 us
//   MXFP4 d 7168, I 2048: 29 rows 106 -> 93 us; d 2048, I 1024: 32 rows
//         35 -> 23 us
// and 64-column e4m3 tiles (158 us at 33 rows, 157 us at d 6144), two stages
// of 64 x 128 by four waves (148, 167 us), 256 x 128 row-skipping tiles (153 us
// at 33, 209 at 133).
//
// Same LDS rows, swizzles, operand layouts and per-output K order as the
// 256-row kernels (gemm_fp8.hip, gemm_mx.hip), so a row's result does not
// depend on the kernel its batch used.
#include "gemm_common.h"

#include <algorithm>

namespace cep {
namespace {

__device__ inline int b_swz_mx(int r) { return (r & 1) | ((r >> 1) & 2); }

// FP8: e4m3 weights (float32 block scales, promoted per K block), else MXFP4
// (E8M0 scales applied by the MFMA).  WGM x WGN waves; wave row wm owns the
// 16-row fragments wm, wm + WGM, ...; wave column wn the columns
// [wn*WN, wn*WN + WN), whole 64-column gate/up groups for SWIGLU.
template <bool FP8, int BM, int BN, int NW, int WGM, int STAGES, int OCC, bool SWIGLU>
__global__ __launch_bounds__(64 * NW, OCC) void k_gemm_rows(GemmArgs g) {
  constexpr int WGN = NW / WGM, WN = BN / WGN;
  constexpr int FM = BM / 16 / WGM, FN = WN / 16;
  constexpr int BB = FP8 ? 128 : 64;      // bytes of a weight row per K step
  constexpr int CHB = BB / 16;            // 16-byte chunks of it
  constexpr int A_LD = BM / 8 / NW;       // row load segments per wave, at most
  constexpr int B_LD = BN * BB / 1024 / NW;
  constexpr int AG = BM > 128 ? 2 : 1;  // 128-row scale groups a tile touches
  constexpr int PER_MAX = A_LD + B_LD + 1;
  static_assert(B_LD * 1024 * NW == BN * BB, "weight loads split evenly over the waves");
  static_assert(STAGES == 2 || STAGES == 3, "wait counts below");
  static_assert(WN % 64 == 0, "a wave's columns hold whole gate/up groups");
  static_assert(BM % (16 * WGM) == 0 && BM % (8 * NW) == 0 && BM <= 160, "whole fragments, two scale groups");
  int mt, nt;
  constexpr bool SPREAD = FP8 || BM != 64;
  if (!(SPREAD ? deal_item(*g.n_tiles, g.N / BN, &mt, &nt)
               : work_item<kGroupM, false>(0, *g.n_tiles, g.N / BN, &mt, &nt)))
    return;
  const Tile t = g.tiles[mt];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wid = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wid / WGN, wn = wid % WGN;
  const int K = g.K, nkb = K / 128;
  const int rows = __builtin_amdgcn_readfirstlane(t.rows);
  const int row0 = __builtin_amdgcn_readfirstlane(t.row0);
  const uint8_t *blob = blob_of(g.bt, __builtin_amdgcn_readfirstlane(t.expert));
  const char *Ag = (const char *)(g.A + (size_t)row0 * K);
  const char *Bg = (const char *)(blob + g.b_off) +
                   (FP8 ? (size_t)nt * BN * K : (size_t)nt * (BN / 16) * (K / 128) * 1024);
  // row scales of K step kb: 512 bytes per 128-row group
  const char *Asg = (const char *)g.As + (size_t)(row0 >> 7) * 512;
  const size_t as_step = (size_t)(g.s_ld >> 7) * 512;
  const int n_as = 32 * (AG > 1 ? mx_row_groups(row0, rows) : 1);  // lanes that load them
  // MXFP4 weight scales: per K step the tile's 4 * BN bytes of the 1 KB record
  const char *Bsg = (const char *)(blob + g.bs_off) + (size_t)(nt * BN / 256) * nkb * 1024 +
                    (nt * BN % 256) * 4;

  __shared__ u32x4 sA[STAGES][BM * 8];
  __shared__ u32x4 sB[STAGES][BN * CHB];
  __shared__ u32x4 sAs[STAGES][AG * 32];
  __shared__ u32x4 sBs[FP8 ? 1 : STAGES][FP8 ? 1 : BN / 4];
  // e4m3: block scales of the tile's columns, [32-column group][K block]
  // (GEMM2: one 128-column block)
  constexpr int NBS = SWIGLU ? BN / kInterleave : (BN > 128 ? BN / 128 : 1);
  __shared__ float sF[FP8 ? NBS * (kMaxDim / 128) : 1];

  const int n_seg = (rows + 7) >> 3;  // 8-row segments that hold rows
  const int n_a = n_seg > wid ? (n_seg - wid + NW - 1) / NW : 0;
  const int per = n_a + B_LD + (wid == 0) + (!FP8 && wid == 1);  // loads a step
  auto stage = [&](int kb, int buf) {
#pragma unroll
    for (int i = 0; i < A_LD; ++i) {
      const int seg = wid + NW * i, r = seg * 8 + (lane >> 3);
      if (i < n_a)
        dma16_s(Ag + (size_t)kb * 128,
                (uint32_t)r * K + (uint32_t)(((lane & 7) ^ ((r >> 1) & 7)) * 16),
                __builtin_amdgcn_readfirstlane(lds_offset(&sA[buf][seg * 64])));
    }
#pragma unroll
    for (int i = 0; i < B_LD; ++i) {
      const int seg = wid * B_LD + i;
      uint32_t off;
      if constexpr (FP8) {
        const int r = seg * 8 + (lane >> 3);
        off = (uint32_t)r * K + (uint32_t)(((lane & 7) ^ ((r >> 1) & 7)) * 16);
      } else {
        const int r = lane >> 2;  // column of the segment's 1 KB block
        off = (uint32_t)seg * nkb * 1024 + r * 64 + (((lane & 3) ^ b_swz_mx(r)) * 16);
      }
      dma16_s(Bg + (size_t)kb * (FP8 ? 128 : 1024), off,
              __builtin_amdgcn_readfirstlane(lds_offset(&sB[buf][seg * 64])));
    }
    if (wid == 0 && lane < n_as)
      dma16_s(Asg + (size_t)kb * as_step, lane * 16,
              __builtin_amdgcn_readfirstlane(lds_offset(&sAs[buf][0])));
    if (!FP8 && wid == 1 && lane < BN / 4)
      dma16_s(Bsg + (size_t)kb * 1024, lane * 16,
              __builtin_amdgcn_readfirstlane(lds_offset(&sBs[FP8 ? 0 : buf][0])));
  };

#pragma unroll
  for (int s = 0; s < STAGES - 1; ++s)
    if (s < nkb) stage(s, s);

  const int r16 = lane & 15, grp = lane >> 4;
  // GEMM2: coefficient and output row of the lane's rows, loaded before the
  // K loop
  float wr[FM];
  int yd[FM];
  if constexpr (!SWIGLU) {
#pragma unroll
    for (int i = 0; i < FM; ++i) {
      const int rt = (i * WGM + wm) * 16 + r16;
      wr[i] = rt < rows ? g.wrow[(size_t)row0 + rt] : 0.0f;
      yd[i] = g.ydst && rt < rows ? g.ydst[(size_t)row0 + rt] : -1;
    }
  }
  if constexpr (FP8) {
    // GEMM1: NBS consecutive rows of [N/32][nkb]; GEMM2: row nt*BN/128 of
    // [N/128][nkb]
    const float *bs = (const float *)(blob + g.bs_off) +
                      (SWIGLU || BN > 128 ? (size_t)nt * NBS : (size_t)(nt * BN / 128)) * nkb;
    for (int i = tid; i < NBS * nkb; i += 64 * NW) sF[i] = bs[i];
    wait_lgkm0();  // in LDS before the first step's barrier
  }

  f32x4 acc[FM][FN];
#pragma unroll
  for (int i = 0; i < FM; ++i)
#pragma unroll
    for (int j = 0; j < FN; ++j) acc[i][j] = f32x4{};

  const int asw = (r16 >> 1) & 7, bsw = FP8 ? asw : b_swz_mx(r16);
  const int f0 = (row0 & 127) >> 4;  // first fragment of the tile in its 128-row group
  auto read8 = [&](const u32x4 *s, int row) {  // a 128-byte LDS row
    const u32x4 lo = s[row * 8 + (grp ^ asw)];
    const u32x4 hi = s[row * 8 + ((grp + 4) ^ asw)];
    return __builtin_bit_cast(i32x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
  };
  for (int kb = 0; kb < nkb; ++kb) {
    // this wave's loads of step kb are done when at most the loads of the
    // STAGES-2 steps issued after it are outstanding
    if (STAGES == 3 && kb + 1 < nkb)
      wait_vmcnt_upto<0, PER_MAX>(per);
    else
      wait_vmcnt<0>();
    // every wave's loads of step kb landed; step kb-1 fully consumed
    __builtin_amdgcn_s_barrier();
    if (kb + STAGES - 1 < nkb) stage(kb + STAGES - 1, (kb + STAGES - 1) % STAGES);
    const int buf = kb % STAGES;
    if (wm * 16 >= rows) continue;  // a wave without rows only loads
    uint2 sa[AG];
#pragma unroll
    for (int a = 0; a < AG; ++a) sa[a] = ((const uint2 *)&sAs[buf][0])[a * 64 + lane];
    i32x8 b[FN];
    uint32_t sb[FN / 4];
    float sf[FN / 2];
#pragma unroll
    for (int j = 0; j < FN; ++j) {
      const int row = wn * WN + j * 16 + r16;
      if constexpr (FP8) {
        b[j] = read8(sB[buf], row);
        if (j % 2 == 0) sf[j / 2] = sF[(SWIGLU ? wn * (WN / 32) + j / 2 : (wn * WN + j * 16) / 128) * nkb + kb];
      } else {
        const u32x4 v = sB[buf][row * 4 + (grp ^ bsw)];
        b[j] = __builtin_bit_cast(i32x8, __builtin_shufflevector(v, v, 0, 1, 2, 3, -1, -1, -1, -1));
        if (j % 4 == 0)
          sb[j / 4] = ((const uint32_t *)&sBs[FP8 ? 0 : buf][0])[(wn * (WN / 64) + j / 4) * 64 + lane];
      }
    }
#pragma unroll
    for (int i = 0; i < FM; ++i) {
      if ((i * WGM + wm) * 16 >= rows) break;  // uniform over the wave
      const i32x8 a = read8(sA[buf], (i * WGM + wm) * 16 + r16);
      const int fg = f0 + i * WGM + wm, f = fg & 7;
      const uint2 sai = sa[AG > 1 && fg >= 8 ? AG - 1 : 0];
      const int sx = (int)((f < 4 ? sai.x : sai.y) >> (8 * (f & 3)));  // byte 0: this fragment's scale
#pragma unroll
      for (int j = 0; j < FN; ++j) {
        if constexpr (FP8) {
          const f32x4 p = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(b[j], a, f32x4{}, 0, 0,
                                                                           0, 127, 0, sx);
          acc[i][j] += p * sf[j / 2];
        } else {
          const int sw = (int)sb[j / 4];
          switch (j % 4) {
            case 0: acc[i][j] = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(b[j], a, acc[i][j], 4, 0, 0, sw, 0, sx); break;
            case 1: acc[i][j] = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(b[j], a, acc[i][j], 4, 0, 1, sw, 0, sx); break;
            case 2: acc[i][j] = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(b[j], a, acc[i][j], 4, 0, 2, sw, 0, sx); break;
            default: acc[i][j] = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(b[j], a, acc[i][j], 4, 0, 3, sw, 0, sx); break;
          }
        }
      }
    }
  }

  // acc[i][j][r]: row (i*WGM + wm)*16 + l%16, column wn*WN + j*16 +
  // 4*(l/16) + r of the tile
#pragma unroll
  for (int i = 0; i < FM; ++i) {
    if ((i * WGM + wm) * 16 >= rows) break;
    const int rt = (i * WGM + wm) * 16 + r16;
    const size_t row = (size_t)row0 + rt;
    if constexpr (SWIGLU) {
      const int I = g.N / 2;
#pragma unroll
      for (int q = 0; q < FN / 4; ++q) {
        float h[2][4], m = 0.0f;
#pragma unroll
        for (int jj = 0; jj < 2; ++jj)
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            h[jj][r] = silu_mul(acc[i][4 * q + jj][r], acc[i][4 * q + jj + 2][r]);
            m = fmaxf(m, fabsf(h[jj][r]));
          }
        m = fmaxf(m, __shfl_xor(m, 16));
        m = fmaxf(m, __shfl_xor(m, 32));
        const int code = max((int)((__float_as_uint(m) >> 23) & 0xff) - 8, 0);
        const int hblk = (nt * BN + wn * WN) / 64 + q;  // MX block of h columns
        uint32_t v[2];
#pragma unroll
        for (int jj = 0; jj < 2; ++jj) {
          float qv[4];
#pragma unroll
          for (int r = 0; r < 4; ++r)
            qv[r] = fminf(fmaxf(ldexpf(h[jj][r], 127 - code), -448.0f), 448.0f);
          int u = __builtin_amdgcn_cvt_pk_fp8_f32(qv[0], qv[1], 0, false);
          v[jj] = (uint32_t)__builtin_amdgcn_cvt_pk_fp8_f32(qv[2], qv[3], u, true);
        }
        if (rt < rows) {
          uint8_t *H = (uint8_t *)g.out + row * I + hblk * 32 + 4 * grp;
          *(uint32_t *)H = v[0];
          *(uint32_t *)(H + 16) = v[1];
          if (grp == 0)
            ((uint8_t *)g.out_s)[mx_row_scale_offset((int)row, hblk, g.s_ld)] = (uint8_t)code;
        }
      }
    } else if (rt < rows) {
      // y = coefficient * acc in bf16; a row with yd >= 0 goes to that
      // output row as float32
      const size_t col = (size_t)nt * BN + wn * WN + 4 * grp;
      __bf16 *yrow = (__bf16 *)g.out + row * g.N + col;
      uint32_t *orow = yd[i] >= 0 ? (uint32_t *)g.yout + (size_t)yd[i] * g.N + col : nullptr;
#pragma unroll
      for (int j = 0; j < FN; ++j) {
        uint32_t v[2];
#pragma unroll
        for (int r = 0; r < 2; ++r)
          v[r] = (uint32_t)__builtin_bit_cast(uint16_t, (__bf16)(acc[i][j][2 * r] * wr[i])) |
                 ((uint32_t)__builtin_bit_cast(uint16_t, (__bf16)(acc[i][j][2 * r + 1] * wr[i]))
                  << 16);
        if (orow)
          *(u32x4 *)(orow + j * 16) = u32x4{plus_zero(v[0] << 16), plus_zero(v[0] & 0xffff0000u),
                                            plus_zero(v[1] << 16), plus_zero(v[1] & 0xffff0000u)};
        else
          *(uint2 *)(yrow + j * 16) = make_uint2(v[0], v[1]);
      }
    }
  }
}

template <bool FP8, int BM, int BN, int NW, int WGM, int STAGES, int OCC, bool SWIGLU>
hipError_t launch_as(const GemmArgs &g, int grid_tiles, hipStream_t s) {
  const int grid = deal_grid(grid_tiles, g.N / BN);
  hipLaunchKernelGGL((k_gemm_rows<FP8, BM, BN, NW, WGM, STAGES, OCC, SWIGLU>), dim3(grid),
                     dim3(64 * NW), 0, s, g);
  return hipGetLastError();
}

}  // namespace

template <bool SWIGLU>
hipError_t launch_rows(const GemmArgs &g, int grid_tiles, bool fp8, bool small, hipStream_t s) {
  if (g.N % 256 || g.K % 128 || g.K > kMaxDim || g.s_ld % 256) return hipErrorInvalidValue;
  if (fp8) {
    if (small) return launch_as<true, 64, 128, 8, 4, 3, 2, SWIGLU>(g, grid_tiles, s);
    return launch_as<true, 160, 128, 4, 2, 2, 2, SWIGLU>(g, grid_tiles, s);
  }
  if (small) return launch_as<false, 64, 128, 4, 4, 2, 4, SWIGLU>(g, grid_tiles, s);
  return launch_as<false, 128, 256, 4, 2, 2, 2, SWIGLU>(g, grid_tiles, s);
}
template hipError_t launch_rows<true>(const GemmArgs &, int, bool, bool, hipStream_t);
template hipError_t launch_rows<false>(const GemmArgs &, int, bool, bool, hipStream_t);

}  // namespace cep
