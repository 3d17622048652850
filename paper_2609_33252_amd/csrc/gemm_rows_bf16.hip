// bf16 grouped expert GEMMs of mid-size batches for gfx950 (CDNA4) MFMA: tiles
// of up to 128 rows x 128 columns (batch_plan, kListVar).
//
// Bound by the bytes a CU requests, rows and weights alike, as the e4m3 and
// MXFP4 tiles of gemm_rows.hip are: a tile loads the 8-row segments that hold
// rows, two workgroups share a CU, and the work order deals an expert's tiles to
// all XCDs.  Each of the four waves owns 32 rows and all columns of the tile, so
// that the gate and up columns of a fused SwiGLU meet in one lane's registers
// and a wave without rows only loads.  Against 128-row tiles that loaded whole
// 64-row halves, weights three stages deep, in contiguous XCD shares (GEMM1 +
// GEMM2): 8 experts of d 4096, I 2048, 132 rows each 150 -> 129 us, 16 experts
// of 64 rows 172 -> 161, 8 experts of d 7168 under Zipf(1.2) routing 229 -> 209,
// 12 experts of d 2304, I 1408, 88 rows 73 -> 66; 193 rows of d 4096 141 -> 141.
// 160 and 192 rows with five and six waves: +10 to +40 % (fewer items than
// slots); 64 columns: +10 %.
//
// LDS rows, swizzle, operand layout and K order (ascending 16-wide steps of
// v_mfma_f32_32x32x16_bf16) as in gemm_bf16.hip: a row's result does not depend
// on the kernel.
#include "gemm_common.h"

#include <algorithm>

namespace cep {
namespace {

template <bool SWIGLU, bool GATHER>
__global__ __launch_bounds__(256, 2) void k_rows_bf16(GemmArgs g) {
  constexpr int BM = kBf16VarTileM, BN = 128, STAGES = 2, NW = 4, FN = BN / 32;
  static_assert(BM == 32 * NW, "a wave owns 32 rows");
  constexpr int A_LD = BM / 8 / NW, B_LD = BN / 8 / NW;
  static_assert(FN % 2 == 0, "gate/up pairs");
  int mt, nt;
  if (!deal_item(*g.n_tiles, g.N / BN, &mt, &nt)) return;
  const Tile t = g.tiles[mt];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wid = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int K = g.K, nk = K / 64;
  const int rows = __builtin_amdgcn_readfirstlane(t.rows);
  const int row0 = __builtin_amdgcn_readfirstlane(t.row0);
  const uint8_t *blob = blob_of(g.bt, __builtin_amdgcn_readfirstlane(t.expert));
  // first column's place in the blocked weight layout (bf16_block_index)
  const int n0 = nt * BN;
  const char *Bg = (const char *)(blob + g.b_off) + (size_t)(n0 >> 7) * (K >> 6) * 16384 +
                   ((n0 >> 4) & 7) * 1024;
  const char *Ag = GATHER ? nullptr : (const char *)(g.A + (size_t)row0 * K * 2);

  __shared__ u32x4 sA[STAGES][BM * 8];
  __shared__ u32x4 sB[STAGES][BN * 8];

  // A load fills 8 LDS rows of 8 chunks; lane l fills slot l % 8 of row l / 8,
  // which holds chunk (l % 8) ^ ((row >> 1) & 7)
  const int n_seg = (rows + 7) >> 3;
  const int n_a = n_seg > wid ? (n_seg - wid + NW - 1) / NW : 0;
  const int ch = (lane & 7) ^ ((lane >> 4) & 3);  // chunk in an even segment; odd: ch ^ 4
  const char *arow[A_LD];
  if constexpr (GATHER) {
#pragma unroll
    for (int i = 0; i < A_LD; ++i) {
      const int seg = wid + NW * i, r = seg * 8 + (lane >> 3);
      const int p = r < rows ? g.perm[row0 + r] : -1;
      arow[i] = (const char *)g.xrow[g.arow0 + (p >= 0 ? p / g.k : 0)] + (ch ^ ((seg & 1) * 4)) * 16;
    }
  }
  // byte offset of the lane's weight chunk in segment seg: column row%16 of its
  // 16-column group, 32-wide K half chunk/4
  auto b_off = [&](int seg) {
    const int r = seg * 8 + (lane >> 3), c = ch ^ ((seg & 1) * 4);
    return (uint32_t)((c >> 2) * 8192 + (r >> 4) * 1024 + (r & 15) * 64 + (c & 3) * 16);
  };
  auto stage = [&](int kt, int buf) {
#pragma unroll
    for (int i = 0; i < A_LD; ++i) {
      const int seg = wid + NW * i;
      if (i >= n_a) break;
      const uint32_t lds = __builtin_amdgcn_readfirstlane(lds_offset(&sA[buf][seg * 64]));
      if constexpr (GATHER)
        dma16(arow[i] + (size_t)kt * 128, lds);
      else
        dma16_s(Ag + (size_t)kt * 128,
                (uint32_t)(seg * 8 + (lane >> 3)) * K * 2 + (ch ^ ((seg & 1) * 4)) * 16, lds);
    }
#pragma unroll
    for (int i = 0; i < B_LD; ++i) {
      const int seg = wid * B_LD + i;
      dma16_s(Bg + (size_t)kt * 16384, b_off(seg),
              __builtin_amdgcn_readfirstlane(lds_offset(&sB[buf][seg * 64])));
    }
  };
  stage(0, 0);

  const bool mine = wid * 32 < rows;
  f32x16 acc[FN];
#pragma unroll
  for (int j = 0; j < FN; ++j) acc[j] = f32x16{};
  const int rsw = ((lane & 31) >> 1) & 7;
  for (int kt = 0; kt < nk; ++kt) {
    // this wave's loads of step kt are its only ones outstanding
    wait_vmcnt<0>();
    // every wave's loads of step kt landed; step kt-1 fully consumed
    __builtin_amdgcn_s_barrier();
    if (kt + 1 < nk) stage(kt + 1, (kt + 1) % STAGES);
    if (!mine) continue;
    const int buf = kt % STAGES;
    bf16x8 a[4], b[4][FN];
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) {
      const int slot = (kk * 2 + (lane >> 5)) ^ rsw;
      a[kk] = __builtin_bit_cast(bf16x8, sA[buf][(wid * 32 + (lane & 31)) * 8 + slot]);
#pragma unroll
      for (int j = 0; j < FN; ++j)
        b[kk][j] = __builtin_bit_cast(bf16x8, sB[buf][(j * 32 + (lane & 31)) * 8 + slot]);
    }
#pragma unroll
    for (int kk = 0; kk < 4; ++kk)
#pragma unroll
      for (int j = 0; j < FN; ++j)
        acc[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[kk], b[kk][j], acc[j], 0, 0, 0);
  }
  if (!mine) return;
  // lane l, element r: column l % 32, row 8*(r/4) + 4*(l/32) + r%4
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    const int rt = wid * 32 + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3);
    if (rt >= rows) continue;
    const size_t row = (size_t)row0 + rt;
    if constexpr (SWIGLU) {
      __bf16 *H = (__bf16 *)g.out + row * (g.N / 2) + n0 / 2 + (lane & 31);
#pragma unroll
      for (int q = 0; q < FN / 2; ++q)
        H[q * 32] = (__bf16)silu_mul(acc[2 * q][r], acc[2 * q + 1][r]);
    } else {
      const float w = g.wrow[row];
      const int yd = g.ydst ? g.ydst[row] : -1;
      float *yr = (yd >= 0 ? g.yout + (size_t)yd * g.N : (float *)g.out + row * g.N) + n0 +
                  (lane & 31);
#pragma unroll
      for (int j = 0; j < FN; ++j) {
        const float v = acc[j][r] * w;
        yr[j * 32] = yd >= 0 ? __uint_as_float(plus_zero(__float_as_uint(v))) : v;
      }
    }
  }
}

template <bool SWIGLU, bool GATHER>
hipError_t launch_as(const GemmArgs &g, int grid_tiles, hipStream_t s) {
  if (g.N % 128 || g.K % 64) return hipErrorInvalidValue;
  hipLaunchKernelGGL((k_rows_bf16<SWIGLU, GATHER>), dim3(deal_grid(grid_tiles, g.N / 128)),
                     dim3(256), 0, s, g);
  return hipGetLastError();
}

}  // namespace

template <bool SWIGLU>
hipError_t launch_bf16_mid(const GemmArgs &g, int grid_tiles, hipStream_t s) {
  if constexpr (SWIGLU) {
    if (g.A == nullptr) {
      if (!g.xrow || !g.perm || g.k < 1) return hipErrorInvalidValue;
      return launch_as<true, true>(g, grid_tiles, s);
    }
  }
  return launch_as<SWIGLU, false>(g, grid_tiles, s);
}
template hipError_t launch_bf16_mid<true>(const GemmArgs &, int, hipStream_t);
template hipError_t launch_bf16_mid<false>(const GemmArgs &, int, hipStream_t);

}  // namespace cep
