// Dispatch of the 256x256 GEMM kernel on a ring of LDS slots.
#include "gemm_ring.h"

namespace hfta {

template <bool A_KC, bool B_KC, typename OutT, bool COLB, int ACT, int VB>
static void launch(const GemmArgs& a, dim3 grid, int blocks, hipStream_t st) {
  const int tiles = (int)(grid.x * grid.z);
  // the order in which a bias is added: see the kernel
  if constexpr (A_KC && !B_KC && sizeof(OutT) == 2) {
    if (a.bias && tiles <= blocks) {
      hipLaunchKernelGGL((gemm_ring_kernel<A_KC, B_KC, OutT, COLB, ACT, VB, true>), dim3((unsigned)blocks), dim3(RING_THREADS), 0, st, a,
                         (int)grid.x, tiles);
      return;
    }
  }
  hipLaunchKernelGGL((gemm_ring_kernel<A_KC, B_KC, OutT, COLB, ACT, VB>), dim3((unsigned)blocks), dim3(RING_THREADS), 0, st, a, (int)grid.x,
                     tiles);
}

template <bool A_KC, bool B_KC, bool COLB, int ACT>
static void launch_bf16(const GemmArgs& a, dim3 grid, int blocks, hipStream_t st) {
  if (a.c_vec == 16) launch<A_KC, B_KC, bf16_raw, COLB, ACT, 16>(a, grid, blocks, st);
  else launch<A_KC, B_KC, bf16_raw, COLB, ACT, 8>(a, grid, blocks, st);
}

// `a` carries tile counts for 256x256 tiles of 64-element k-tiles and operand extents; every operand loads in whole 16-byte pieces,
// aligned, or (contiguous along m / n) aligned to 8 bytes with m_last / n_last set where the extent is no multiple of eight.
// HFTA_EUNSUPPORTED: not a launch this kernel is built for.
int gemm_ring_launch(const GemmDesc& d, const GemmArgs& a0, dim3 grid, hipStream_t st) {
  const bool partial = a0.splits > 1, f32 = d.out_f32 || partial;
  const bool colb = d.bias && d.bias_mode == 2;
  const int64_t tiles = (int64_t)grid.x * grid.z;
  const int blocks = (int)(tiles < persistent_blocks() ? tiles : persistent_blocks());
  if (blocks < 1 || tiles > (1 << 30)) return HFTA_EUNSUPPORTED;
  if (a0.total_tiles / a0.splits < RING_MIN_T) return HFTA_EUNSUPPORTED;
  if (d.act != HFTA_ACT_NONE && d.act != HFTA_ACT_RELU && d.act != HFTA_ACT_LEAKY) return HFTA_EUNSUPPORTED;
  if (colb && (reinterpret_cast<uintptr_t>(d.bias) % 8 != 0 || d.bias_g0 % 4 != 0 || d.bias_g1 % 4 != 0 || d.N % 4 != 0))
    return HFTA_EUNSUPPORTED;
  const int vb = partial ? a0.p_vec : a0.c_vec;
  if (f32 ? vb != 16 : vb != 16 && vb != 8) return HFTA_EUNSUPPORTED;
  if (d.N % (vb / (f32 ? 4 : 2)) != 0) return HFTA_EUNSUPPORTED;
  if (partial ? (int64_t)d.M * d.N * 4 >= (int64_t)1 << 31 : a0.c_extent == 0) return HFTA_EUNSUPPORTED;
  if (d.bias && tiles <= blocks && (f32 || !d.a_kc || d.b_kc)) return HFTA_EUNSUPPORTED;      // forms that no bias comes with
  GemmArgs a = a0;
  a.slope = d.act == HFTA_ACT_NONE ? 1.f : d.act == HFTA_ACT_RELU ? 0.f : d.slope;
  const bool ident = d.act == HFTA_ACT_NONE;
  if (f32) {
    if (colb || !ident) return HFTA_EUNSUPPORTED;
    if (d.a_kc && !d.b_kc) launch<true, false, float, false, BIG_NONE, 16>(a, grid, blocks, st);
    else if (d.a_kc && d.b_kc) launch<true, true, float, false, BIG_NONE, 16>(a, grid, blocks, st);
    else if (!d.a_kc && !d.b_kc) launch<false, false, float, false, BIG_NONE, 16>(a, grid, blocks, st);
    else return HFTA_EUNSUPPORTED;
  } else if (d.a_kc && !d.b_kc) {
    if (colb && ident) launch_bf16<true, false, true, BIG_NONE>(a, grid, blocks, st);
    else if (colb) launch_bf16<true, false, true, BIG_SEL>(a, grid, blocks, st);
    else if (ident) launch_bf16<true, false, false, BIG_NONE>(a, grid, blocks, st);
    else launch_bf16<true, false, false, BIG_SEL>(a, grid, blocks, st);
  } else if (colb || !ident) {
    return HFTA_EUNSUPPORTED;
  } else if (d.a_kc && d.b_kc) {
    launch_bf16<true, true, false, BIG_NONE>(a, grid, blocks, st);
  } else if (!d.a_kc && !d.b_kc) {
    launch_bf16<false, false, false, BIG_NONE>(a, grid, blocks, st);
  } else {
    return HFTA_EUNSUPPORTED;
  }
  return launch_status();
}

}  // namespace hfta
