// Dispatch of the GEMM kernel that loads straight into LDS: which problems, which tile.
#include "gemm_dma.h"

namespace hfta {

// The kernel is for launches that leave about one workgroup per compute unit, with a reduction long enough to
// be worth a pipeline: up to 256 workgroups of the smallest tile that keeps the count there (a workgroup alone
// on its compute unit spends 0.18 / 0.29 / 0.37 us per 64-element k-tile with 64 x 64 / 128 x 64 / 128 x 128,
// so the smaller tile wins as long as it costs no second round), 320 of the largest.  Measured per call, against
// the register-staged kernels with their split reductions:
//   forward  8 x 2048 x 256, K = 1024     20.3 -> 15.9 us       5 x 693 x 384, K = 1536    24.9 -> 13.6 us
//   data     8 x 2048 x 256, K = 8192      147 -> 101 us        4 x 3000 x 256, K = 5000     85 -> 57 us
//   weights  8 x 256 x 768, K = 2048      33.7 -> 18.2 us       5 x 384 x 1536, K = 693     36 -> 13.1 us
//   few rows 8 x 32 x 1024, K = 512        10.6 -> 5.8 us
// With four k-tiles or fewer both take the same time (8 x 2048 x 256, K = 256: 9.1 and 9.3 us), and with many more
// workgroups than compute units the smaller stages of the register-staged kernels hide more (4 x 3000 x 768,
// K = 256: 16 against 19 us; 256 x 256 tiles: 180 us both at 16 x 4096 x 512, K = 2048).
// Reductions past 128 k-tiles keep their split over k: this kernel walks them in sequence.
int gemm_dma_tile(const GemmDesc& d) {
  if (d.dtype != HFTA_BF16 || (!d.a_kc && d.b_kc)) return -1;
  if ((d.a_kc || d.b_kc) && d.K % 8 != 0) return -1;
  if ((!d.a_kc && d.M % 8 != 0) || (!d.b_kc && d.N % 8 != 0)) return -1;
  const int64_t kt = (int64_t)d.S * ((d.K + 63) / 64), G = (int64_t)d.G0 * d.G1;
  if (kt < 5 || kt > 128) return -1;
  auto tiles = [&](int bm, int bn) { return (int64_t)((d.M + bm - 1) / bm) * ((d.N + bn - 1) / bn) * G; };
  if (tiles(64, 64) <= 256) return 0;
  if (tiles(128, 64) <= 256) return 1;
  if (tiles(128, 128) <= 320) return 2;
  return -1;
}

template <int WM, int WN, int MI, int NI, int OCC, bool A_KC, bool B_KC, typename OutT>
static void launch(const GemmDesc& d, GemmArgs a, hipStream_t st) {
  constexpr int BM = WM * MI * 32, BN = WN * NI * 32, BK = 64;
  a.tiles_m = (d.M + BM - 1) / BM;
  a.tiles_n = (d.N + BN - 1) / BN;
  a.tiles_per_seg = (d.K + BK - 1) / BK;
  a.total_tiles = d.S * a.tiles_per_seg;
  const dim3 grid((unsigned)(a.tiles_m * a.tiles_n), 1, (unsigned)(d.G0 * d.G1 * a.splits));
  hipLaunchKernelGGL((gemm_dma_kernel<WM, WN, MI, NI, BK, A_KC, B_KC, OutT, 3, OCC>), grid, dim3(WM * WN * 64), 0, st, a);
}

template <bool A_KC, bool B_KC, typename OutT>
static int launch_tile(const GemmDesc& d, const GemmArgs& a, hipStream_t st) {
  switch (gemm_dma_tile(d)) {
    case 0: launch<2, 2, 1, 1, 3, A_KC, B_KC, OutT>(d, a, st); break;      // 64 x 64
    case 1: launch<2, 2, 2, 1, 2, A_KC, B_KC, OutT>(d, a, st); break;      // 128 x 64
    case 2: launch<2, 4, 2, 1, 2, A_KC, B_KC, OutT>(d, a, st); break;      // 128 x 128
    default: return HFTA_EUNSUPPORTED;
  }
  return launch_status();
}

// `a`: operand extents set, operands loadable in whole 16-byte pieces, no split.
int gemm_dma_launch(const GemmDesc& d, const GemmArgs& a, hipStream_t st) {
  if (a.splits != 1) return HFTA_EUNSUPPORTED;
  if (d.a_kc && !d.b_kc) return d.out_f32 ? launch_tile<true, false, float>(d, a, st) : launch_tile<true, false, bf16_raw>(d, a, st);
  if (d.a_kc && d.b_kc) return d.out_f32 ? launch_tile<true, true, float>(d, a, st) : launch_tile<true, true, bf16_raw>(d, a, st);
  if (!d.out_f32) return launch_tile<false, false, bf16_raw>(d, a, st);
  GemmArgs s = a;
  s.bsum = d.bsum;
  const int rc = launch_tile<false, false, float>(d, s, st);
  if (rc == HFTA_OK && d.bsum && d.bsum_done) *d.bsum_done = true;
  return rc;
}

template <int MW, int MX>
static void launch_pair(GemmPair p, hipStream_t st) {
  auto tiles = [](GemmArgs& a, int bm, int batches, int& x, int& total) {
    a.tiles_m = (a.M + bm - 1) / bm;
    a.tiles_n = (a.N + 63) / 64;
    a.tiles_per_seg = (a.K + 63) / 64;
    a.total_tiles = a.tiles_per_seg;
    x = a.tiles_m * a.tiles_n;
    total = x * batches;
  };
  tiles(p.dw, MW * 64, p.dw_total, p.dw_x, p.dw_total);
  tiles(p.dx, MX * 64, p.dx_total, p.dx_x, p.dx_total);
  p.first = (p.dw_total + 7) / 8 * 8;
  hipLaunchKernelGGL((gemm_dma_pair_kernel<MW, MX>), dim3((unsigned)(p.first + p.dx_total)), dim3(256), 0, st, p);
}

static int64_t tiles64(const GemmDesc& d, int bm) { return (int64_t)((d.M + bm - 1) / bm) * ((d.N + 63) / 64) * d.G0; }

// Two launches of a few hundred workgroups each are a wait of 4 us, two prologues and two tails that leave compute units idle; in one
// launch the data gradient's tiles fill the places that the weight gradient's long chains leave, two or three workgroups to a compute
// unit.  us, two launches -> one (256 -> 1024 etc. are Fx -> Fy):
//   8 x 2048 rows, 256 -> 768 34.0 -> 24.5, 256 -> 1024 36.9 -> 28.4, 256 -> 256 25.8 -> 18.2   4 x 3000, 256 -> 1024 37.0 -> 26.7,
//   1024 -> 256 36.2 -> 31.6   5 x 693, 384 -> 1536 25.4 -> 21.2   1 x 64, 256 -> 768 15.3 -> 6.7   8 x 3000, 256 -> 1000 56.9 -> 51.0
// Up to 3 1/4 rounds of the 512 places and 24.8 GFLOP; more work is faster on larger tiles: 3 x 2048, 512 -> 2048 (25.8 GFLOP)
// 43.8 -> 46.0, 4 x 2048, 256 -> 3000 (25.2) 51.6 -> 52.7, 16 x 693, 1024 -> 256 (1920 tiles) 26.3 -> 28.3, 8 x 2048, 1024 -> 256
// (2304 tiles) 34.5 -> 35.2, 16 x 4096, 512 -> 2048 292 -> 496.  Reductions past 128 k-tiles of the weight gradient stay split.
// Not widths that are no whole tiles of 128 where each product alone is one round of 128 x 128 tiles under a long reduction: those read
// less than the pair's 64 columns.  102 such shapes of 40 k-tiles together and more (9 x 2138, 104 -> 2912 56.7 -> 66.7,
// 5 x 2433, 232 -> 1944 52.8 -> 61.5) take 1.08 times as long in one launch at the median, the same with whole tiles 0.91 times
// (121 shapes), with shorter reductions 0.89 (200).
bool gemm_dma_pair_takes(const GemmDesc& dw, const GemmDesc& dx) {
  auto round128 = [](const GemmDesc& d) {
    return gemm_dma_tile(d) == 2 && (int64_t)((d.M + 127) / 128) * ((d.N + 127) / 128) * d.G0 <= 256;
  };
  if ((dw.M % 128 || dw.N % 128) && (dw.K + 63) / 64 + (dx.K + 63) / 64 >= 40 && round128(dw) && round128(dx)) return false;
  return dw.dtype == HFTA_BF16 && dw.M % 8 == 0 && dw.N % 8 == 0 && dw.K >= 64 && dw.K <= 128 * 64 &&
         tiles64(dw, 128) + tiles64(dx, 128) <= 1664 && 4.0 * dw.G0 * dw.K * dw.M * dw.N <= 24.8e9;
}

// The weight gradient's tile as for a launch of its own; data gradients of few tiles take the smaller one too (5 x 693, 384 -> 1536
// 23.2 -> 21.2; with 512 tiles, 8 x 1024, 256 -> 1024, 17.0 -> 20.8).
int gemm_dma_pair_launch(const GemmDesc& dw, const GemmArgs& aw, const GemmDesc& dx, const GemmArgs& ax, hipStream_t st) {
  GemmPair p;
  p.dw = aw; p.dx = ax;
  p.dw.bsum = dw.bsum;
  p.dw_total = dw.G0; p.dx_total = dx.G0;
  const bool w64 = tiles64(dw, 64) <= 256, x64 = tiles64(dx, 64) <= 384;
  if (w64 && x64) launch_pair<1, 1>(p, st);
  else if (w64) launch_pair<1, 2>(p, st);
  else if (x64) launch_pair<2, 1>(p, st);
  else launch_pair<2, 2>(p, st);
  const int rc = launch_status();
  if (rc == HFTA_OK && dw.bsum && dw.bsum_done) *dw.bsum_done = true;
  return rc;
}

}  // namespace hfta
