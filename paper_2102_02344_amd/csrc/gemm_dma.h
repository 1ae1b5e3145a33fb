// bf16 GEMM on operand tiles that travel from memory straight into LDS.
//
// The register-staged kernels (gemm_pf.h, gemm_big.h) keep two k-tiles in flight, all that their registers
// hold.  A launch with no more than about one workgroup per compute unit has nothing else to hide the
// latency of a load behind: its k-loop ran at one 32-element k-tile per 0.8 us (128 x 128 tile, 2 us for 64
// elements) where the matrix instructions need 0.12.  Here a load writes LDS itself (buffer_load ... lds,
// 16 bytes a lane), so ST - 1 k-tiles of 64 elements are in flight in ST LDS stages and no vector register
// or ds_write is spent on them.
//
// Such a load fills 1 KB of LDS in lane order, so rows cannot be padded; what a lane fetches is permuted
// instead (DmaOp): 16-byte pieces of neighbouring rows land on different banks, both for the 16-byte reads of
// k-contiguous tiles ([row][64 k]) and for the transpose reads of m/n-contiguous ones ([64 k][column]).
//
// Synchronisation: one barrier per k-tile.  A wave waits until its own loads of the tile about to be read have
// landed (vmcnt: the ST - 2 tiles behind it may stay in flight) and its reads of the tile before have returned
// (lgkmcnt), then the barrier makes both true for all waves, and the stage that was read last is refilled.
// Loads past the end of the reduction are out of range for their buffer (zeros, no memory request), which
// keeps the counts fixed.
//
// Host side guarantees: bf16 operands, every 16-byte piece wholly inside or outside its operand (rows 16-byte
// aligned, extent along the contiguous dimension a multiple of 8), each operand slice below 2 GiB.
#pragma once
#include "gemm_pf.h"

namespace hfta {

typedef int dma_i32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ dma_i32x4 dma_rsrc(const void* p, uint32_t bytes) {
  const uint64_t a = reinterpret_cast<uint64_t>(p);
  dma_i32x4 r;
  r.x = __builtin_amdgcn_readfirstlane((int)(uint32_t)a);
  r.y = __builtin_amdgcn_readfirstlane((int)(uint32_t)(a >> 32) & 0xffff);   // stride 0
  r.z = __builtin_amdgcn_readfirstlane((int)bytes);
  r.w = 0x00020000;
  return r;
}
// 64 lanes x 16 bytes from rsrc + voff (per lane) to LDS bytes lds .. lds + 1023 in lane order
__device__ __forceinline__ void dma_load(uint32_t lds, uint32_t voff, dma_i32x4 rsrc) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds"
               :: "s"(lds), "v"(voff), "s"(rsrc) : "memory", "m0");
}
template <int N> __device__ __forceinline__ void dma_wait_barrier() {
  asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" :: "n"(N) : "memory");
}

// One operand's tile of R rows (k-contiguous) or columns (m/n-contiguous) x BK k, fetched by WAVES waves in
// 1 KB chunks, NC per wave.
template <int R, int BK, bool KC, int WAVES> struct DmaOp {
  static constexpr int BYTES = R * BK * 2;
  static constexpr int NC = BYTES / 1024 / WAVES;
  static constexpr int W = KC ? BK / 8 : R / 8;          // pieces per row / k-row of the tile
  static constexpr int KR = 64 / W;                      // rows / k-rows per chunk
  static_assert(NC >= 1 && KR >= 1 && BYTES % (1024 * WAVES) == 0, "whole chunks per wave");
  uint32_t off[NC];
  uint32_t step;                                         // bytes per unit of k
  // piece p of row (k-row) r sits at position p ^ swz(r): the 16 rows a quarter-wave reads together (k-contiguous)
  // or the four k-rows of a transpose read (m/n-contiguous) cover all 64 banks once
  static __device__ __forceinline__ int swz(int r) {
    if (KC) return W == 8 ? (r ^ (r >> 3)) & 7 : (r >> 2) & 3;
    return R >= 128 ? (r & 3) << 2 : ((r >> 1) & 1) << 2;
  }
  // k (within the tile) of the piece this lane fetches in chunk c
  static __device__ __forceinline__ int k_of(int c, int lane) {
    const int r = c * KR + lane / W;
    return KC ? ((lane % W) ^ swz(r)) * 8 : r;
  }
  __device__ __forceinline__ void init(int r0, int rows, int64_t ld, int wave, int lane) {
    step = KC ? 2u : (uint32_t)(ld * 2);
#pragma unroll
    for (int i = 0; i < NC; ++i) {
      const int c = wave * NC + i;
      if (KC) {
        const int r = r0 + c * KR + lane / W;
        off[i] = r < rows ? (uint32_t)((int64_t)r * ld * 2) + (uint32_t)k_of(c, lane) * 2u : PF_OOB;
      } else {
        const int k = k_of(c, lane), col = r0 + ((lane % W) ^ swz(k)) * 8;
        off[i] = col < rows ? (uint32_t)k * step + (uint32_t)col * 2u : PF_OOB;
      }
    }
  }
  __device__ __forceinline__ void load(int i, uint32_t lds, dma_i32x4 rs, int k0, int K, int wave, int lane) const {
    const int c = wave * NC + i;
    dma_load(lds + (uint32_t)c * 1024u, k0 + k_of(c, lane) < K ? off[i] + (uint32_t)k0 * step : PF_OOB, rs);
  }
  // matrix-instruction fragment: lane l holds row (column) base + l%32 and k = 16s + 8(l/32) + 0..7
  static __device__ __forceinline__ bf16x8_t frag(const unsigned char* tile, int base, int s, int lane) {
    if (KC) {
      const int r = base + (lane & 31);
      return *reinterpret_cast<const bf16x8_t*>(tile + r * (BK * 2) + (((2 * s + (lane >> 5)) ^ swz(r)) << 4));
    }
    const int r16 = lane & 15, k = 8 * (lane >> 5) + (r16 >> 2);           // + 16s: the same position pattern
    const int piece = (base >> 3) + 2 * ((lane >> 4) & 1) + ((r16 & 3) >> 1);
    const unsigned char* a0 = tile + (16 * s + k) * (R * 2) + ((piece ^ swz(k)) << 4) + (r16 & 1) * 8;
    typedef __attribute__((address_space(3))) pf_v4s* lds_v4s;
    union { pf_v4s h[2]; bf16x8_t v; } u;
    u.h[0] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4s)(a0));
    u.h[1] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4s)(a0 + 4 * (R * 2)));
    return u.v;
  }
};

// Epilogue (see store_tile in gemm.h): waves with `mine` put their MI x NI blocks, staged row r0 and column c0
// on, into LDS in the output type; then 16- or 8-byte pieces of rows go out.
template <int BN, typename OutT> constexpr int dma_pitch() { return BN * (int)sizeof(OutT) + (sizeof(OutT) == 2 ? 8 : 16); }

template <int MI, int NI, int BN, typename OutT, int KIND, bool COLB>
__device__ __forceinline__ void dma_stage(const f32x16_t (&acc)[MI][NI], unsigned char* lds, int r0, int c0, int M, int N, int m0,
                                          int n0, const bf16_raw* bias, int act, float slope, int lane) {
  constexpr int ES = sizeof(OutT), PITCH = dma_pitch<BN, OutT>();
  const int ml = lane & 31, nq = (lane >> 5) * 4;
#pragma unroll
  for (int j = 0; j < NI; ++j)
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int nl = c0 + j * 32 + 8 * q + nq;
      float cb[4] = {0.f, 0.f, 0.f, 0.f};
      if (COLB) col_bias4(cb, bias, n0 + nl, N);
#pragma unroll
      for (int i = 0; i < MI; ++i) {
        const int rl = r0 + i * 32 + ml;
        float bm = 0.f;
        if (!COLB && bias && m0 + rl < M) bm = bf16_to_f32(bias[m0 + rl]);
        float x[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) x[e] = epi_act<KIND>(acc[i][j][4 * q + e] + (COLB ? cb[e] : bm), act, slope);
        unsigned char* dst = lds + rl * PITCH + nl * ES;
        if (ES == 2) *reinterpret_cast<uint2*>(dst) = make_uint2(pack_bf16x2(x[0], x[1]), pack_bf16x2(x[2], x[3]));
        else *reinterpret_cast<float4*>(dst) = make_float4(x[0], x[1], x[2], x[3]);
      }
    }
}

template <int RP, int BN, int THREADS, typename OutT, int VB>
__device__ __forceinline__ void dma_store_rows(const unsigned char* lds, OutT* Cb, int64_t c_ld, int M, int N, int m0, int n0,
                                               int t, int c_seg, int64_t c_seg_stride) {
  constexpr int ES = sizeof(OutT), PITCH = dma_pitch<BN, OutT>();
  constexpr int EPV = VB / ES, PPR = BN / EPV, RPI = THREADS / PPR;
  static_assert(RPI >= 1 && RP % RPI == 0, "whole rows per pass");
  const int r0 = t / PPR, c = t % PPR, n = n0 + c * EPV;
  const unsigned char* src = lds + r0 * PITCH + c * VB;
  OutT* dst = Cb + (int64_t)(m0 + r0) * c_ld + col_offset(n, c_seg, c_seg_stride);
#pragma unroll 4
  for (int it = 0; it < RP / RPI; ++it) {
    typedef typename std::conditional<VB == 16, uint4, typename std::conditional<VB == 8, uint2, OutT>::type>::type V;
    if (m0 + r0 + it * RPI >= M) break;
    const V v = *reinterpret_cast<const V*>(src + it * RPI * PITCH);
    OutT* d = dst + (int64_t)it * RPI * c_ld;
    if (n + EPV <= N) {
      *reinterpret_cast<V*>(d) = v;
    } else {
      const OutT* e = reinterpret_cast<const OutT*>(&v);
#pragma unroll
      for (int k = 0; k < EPV; ++k)
        if (n + k < N) d[k] = e[k];
    }
  }
}

// Column sums of an operand tile (GemmDesc::bsum), in the order of the stand-alone column sum (colsum_vec_kernel): row r
// belongs to chain r % 64, a chain adds its rows in order, the chains are added in order.  So a bias gradient does not
// depend on which kernel took the weight gradient, and with it on the number of models.  A tile is 64 rows: a thread keeps
// eight columns of its rows of a tile, each a chain of its own.
constexpr int SUM_CHAINS = 64;
__device__ __forceinline__ void add_bf16x8(float (&s)[8], const uint4& q) {
  const uint32_t w[4] = {q.x, q.y, q.z, q.w};
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    s[2 * i] += __uint_as_float(w[i] << 16);
    s[2 * i + 1] += __uint_as_float(w[i] & 0xffff0000u);
  }
}
// PPR eight-column pieces per row; thread t holds chains t / PPR + k * (SUM_CHAINS / C), k < C, of piece t % PPR
template <int PPR, int C>
__device__ __forceinline__ void store_colsums(const float (&s)[C][8], float* lds, float* out, int n0, int N, int t) {
#pragma unroll
  for (int k = 0; k < C; ++k) {
    float* d = lds + (t / PPR + k * (SUM_CHAINS / C)) * (PPR * 8) + (t % PPR) * 8;
    *reinterpret_cast<float4*>(d) = make_float4(s[k][0], s[k][1], s[k][2], s[k][3]);
    *reinterpret_cast<float4*>(d + 4) = make_float4(s[k][4], s[k][5], s[k][6], s[k][7]);
  }
  __syncthreads();
  if (t < PPR * 8 && n0 + t < N) {
    float v = 0.f;
#pragma unroll 16
    for (int r = 0; r < SUM_CHAINS; ++r) v += lds[r * (PPR * 8) + t];
    out[n0 + t] = v;
  }
}

// What one instantiation keeps in LDS: WM x WN waves, MI x NI matrix-instruction blocks each
template <int WM, int WN, int MI, int NI, int BK, bool A_KC, bool B_KC, typename OutT, int ST> struct DmaTile {
  static constexpr int BM = WM * MI * 32, BN = WN * NI * 32, WAVES = WM * WN;
  typedef DmaOp<BM, BK, A_KC, WAVES> OpA;
  typedef DmaOp<BN, BK, B_KC, WAVES> OpB;
  static constexpr int STAGE = OpA::BYTES + OpB::BYTES;
  // rows staged per epilogue pass: as many whole wave rows as fit
  static constexpr int ROWB = dma_pitch<BN, OutT>();
  static constexpr int STAGES = ST * STAGE;
  static constexpr int WPP = BM * ROWB <= STAGES + 4096 ? WM : WM / 2;   // wave rows per pass
  static constexpr int RP = WPP * MI * 32;
  static_assert(WPP >= 1 && RP * ROWB <= STAGES + 4096, "the staged output must fit");
  static constexpr int SMEM = RP * ROWB > STAGES ? RP * ROWB : STAGES;
};

// workgroup `lin` of tiles_x x batches: a contiguous range of (batch, tile) per XCD, as in gemm_kernel
__device__ __forceinline__ void dma_renumber(int lin, int tiles_x, int total, int& bx, int& bz) {
  const int per = total >> 3;
  const int l2 = lin < (per << 3) ? (lin & 7) * per + (lin >> 3) : lin;
  bz = l2 / tiles_x;
  bx = l2 - bz * tiles_x;
}

// Tile bx of batch bz
template <int WM, int WN, int MI, int NI, int BK, bool A_KC, bool B_KC, typename OutT, int ST>
__device__ __forceinline__ void gemm_dma_body(const GemmArgs& p, int bx, int bz, unsigned char* smem) {
  typedef DmaTile<WM, WN, MI, NI, BK, A_KC, B_KC, OutT, ST> T;
  constexpr int BM = T::BM, BN = T::BN, WAVES = T::WAVES;
  typedef typename T::OpA OpA;
  typedef typename T::OpB OpB;
  constexpr int STAGE = T::STAGE, SMEM = T::STAGES;
  constexpr int PER = OpA::NC + OpB::NC, KS = BK / 16;
  constexpr int FLIGHT = (ST - 2) * PER;                  // loads of the tiles that stay in flight at a barrier
  constexpr int WPP = T::WPP, RP = T::RP;
  const int t = threadIdx.x, lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const int wm = wave / WN, wn = wave % WN;
  const int m0 = (bx % p.tiles_m) * BM, n0 = (bx / p.tiles_m) * BN;
  const int g0 = bz / p.G1, g1 = bz % p.G1;
  const bf16_raw* Ab = reinterpret_cast<const bf16_raw*>(p.A) + g0 * p.a_g0 + g1 * p.a_g1;
  const bf16_raw* Bb = reinterpret_cast<const bf16_raw*>(p.Bm) + g0 * p.b_g0 + g1 * p.b_g1;
  const int kt = p.total_tiles;

  OpA oa;
  OpB ob;
  oa.init(m0, p.M, p.a_ld, wave, lane);
  ob.init(n0, p.N, p.b_ld, wave, lane);
  typedef __attribute__((address_space(3))) unsigned char* lds_ptr;
  const uint32_t lds0 = (uint32_t)(uintptr_t)(lds_ptr)smem;
  // k-tile tt: its operand slices and k range, and chunks [c0, c1) of this wave's PER loads of it
  struct Tile { dma_i32x4 ra, rb; int k0, K; };
  auto aim = [&](int tt) {
    const bool live = tt < kt;
    const int tc = live ? tt : 0;
    const int seg = tc / p.tiles_per_seg;
    Tile x;
    x.k0 = (tc - seg * p.tiles_per_seg) * BK;
    x.K = live ? p.K : 0;
    x.ra = dma_rsrc(Ab + seg * p.a_ss, p.a_extent);
    x.rb = dma_rsrc(Bb + seg * p.b_ss, p.b_extent);
    return x;
  };
  auto issue = [&](const Tile& x, int stage, int c0, int c1) {
    const uint32_t lds = lds0 + (uint32_t)(stage * STAGE);
#pragma unroll
    for (int i = 0; i < PER; ++i)
      if (i >= c0 && i < c1) {
        if (i < OpA::NC) oa.load(i, lds, x.ra, x.k0, x.K, wave, lane);
        else ob.load(i - OpA::NC, lds + OpA::BYTES, x.rb, x.k0, x.K, wave, lane);
      }
  };

  f32x16_t acc[MI][NI];
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int j = 0; j < NI; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;

#pragma unroll
  for (int d = 0; d < ST - 1; ++d) issue(aim(d), d, 0, PER);
  // column sums of B, by the workgroups of the first row tile: 8 columns of every (threads / pieces)-th k-row a thread
  constexpr bool SUMS = !A_KC && !B_KC && sizeof(OutT) == 4;
  constexpr int SPPR = BN / 8, SROWS = WAVES * 64 / SPPR, SC = SUMS ? SUM_CHAINS / SROWS : 1;
  static_assert(!SUMS || (BK == SUM_CHAINS && SUM_CHAINS * BN * 4 <= SMEM), "a tile's rows are the chains");
  const bool sums = SUMS && p.bsum && m0 == 0;
  float cs[SC][8];
#pragma unroll
  for (int k = 0; k < SC; ++k)
#pragma unroll
    for (int e = 0; e < 8; ++e) cs[k][e] = 0.f;
  bool done = false;
  for (int base = 0; !done; base += ST) {
#pragma unroll
    for (int d = 0; d < ST; ++d) {
      dma_wait_barrier<FLIGHT>();
      const Tile nx = aim(base + d + ST - 1);
      const unsigned char* As = smem + d * STAGE;
      const unsigned char* Bs = As + OpA::BYTES;
      // The refill's loads are spread over the k-steps: issued in one go, the texture path takes them at 64 bytes
      // per clock and the wave would stand still before its first matrix instruction.
      bf16x8_t a[2][MI], b[2][NI];
#pragma unroll
      for (int i = 0; i < MI; ++i) a[0][i] = OpA::frag(As, (wm * MI + i) * 32, 0, lane);
#pragma unroll
      for (int j = 0; j < NI; ++j) b[0][j] = OpB::frag(Bs, (wn * NI + j) * 32, 0, lane);
#pragma unroll
      for (int s = 0; s < KS; ++s) {
        if (s + 1 < KS) {
#pragma unroll
          for (int i = 0; i < MI; ++i) a[(s + 1) & 1][i] = OpA::frag(As, (wm * MI + i) * 32, s + 1, lane);
#pragma unroll
          for (int j = 0; j < NI; ++j) b[(s + 1) & 1][j] = OpB::frag(Bs, (wn * NI + j) * 32, s + 1, lane);
        }
        issue(nx, (d + ST - 1) % ST, PER * s / KS, PER * (s + 1) / KS);
#pragma unroll
        for (int i = 0; i < MI; ++i)
#pragma unroll
          for (int j = 0; j < NI; ++j)
            acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(b[s & 1][j], a[s & 1][i], acc[i][j], 0, 0, 0);
      }
      if constexpr (SUMS) {
        if (sums) {
#pragma unroll
          for (int k = 0; k < SC; ++k) {
            const int r = t / SPPR + k * SROWS;
            add_bf16x8(cs[k], *reinterpret_cast<const uint4*>(Bs + r * (BN * 2) + (((t % SPPR) ^ OpB::swz(r)) << 4)));
          }
        }
      }
      if (base + d + 1 >= kt) { done = true; break; }
    }
  }
  dma_wait_barrier<0>();                                   // nothing may land in the stages any more
  if constexpr (SUMS) {
    if (sums) {
      store_colsums<SPPR, SC>(cs, reinterpret_cast<float*>(smem), p.bsum + (int64_t)g0 * p.N, n0, p.N, t);
      __syncthreads();
    }
  }

  OutT* Cb = reinterpret_cast<OutT*>(p.C) + g0 * p.c_g0 + g1 * p.c_g1;
  const bf16_raw* bias = p.bias ? reinterpret_cast<const bf16_raw*>(p.bias) + g0 * p.bias_g0 + g1 * p.bias_g1 : nullptr;
  const bool colb = bias && p.bias_mode == 2;
#pragma unroll
  for (int pass = 0; pass < WM / WPP; ++pass) {
    const int mp = m0 + pass * RP;
    if (pass) __syncthreads();
    if (wm / WPP == pass) {
      const int r0 = wm % WPP * MI * 32, c0 = wn * NI * 32;
#define DMA_STAGE(KIND, COLB) dma_stage<MI, NI, BN, OutT, KIND, COLB>(acc, smem, r0, c0, p.M, p.N, mp, n0, bias, p.act, p.slope, lane)
      if (sizeof(OutT) == 2 && (colb || p.act == HFTA_ACT_TANH || p.act == HFTA_ACT_GELU)) {
        if (colb && p.act == HFTA_ACT_NONE) DMA_STAGE(EPI_NONE, true);
        else if (colb && p.act == HFTA_ACT_RELU) DMA_STAGE(EPI_RELU, true);
        else if (colb) DMA_STAGE(EPI_ANY, true);
        else DMA_STAGE(EPI_ANY, false);
      } else if (p.act == HFTA_ACT_RELU) DMA_STAGE(EPI_RELU, false);
      else if (p.act == HFTA_ACT_LEAKY) DMA_STAGE(EPI_LEAKY, false);
      else DMA_STAGE(EPI_NONE, false);
#undef DMA_STAGE
    }
    __syncthreads();
    if (p.c_vec == 16) dma_store_rows<RP, BN, WAVES * 64, OutT, 16>(smem, Cb, p.c_ld, p.M, p.N, mp, n0, t, p.c_seg, p.c_seg_stride);
    else if (p.c_vec == 8) dma_store_rows<RP, BN, WAVES * 64, OutT, 8>(smem, Cb, p.c_ld, p.M, p.N, mp, n0, t, p.c_seg, p.c_seg_stride);
    else dma_store_rows<RP, BN, WAVES * 64, OutT, sizeof(OutT)>(smem, Cb, p.c_ld, p.M, p.N, mp, n0, t, p.c_seg, p.c_seg_stride);
  }
}

template <int WM, int WN, int MI, int NI, int BK, bool A_KC, bool B_KC, typename OutT, int ST, int OCC>
__global__ __launch_bounds__(WM * WN * 64, OCC) void gemm_dma_kernel(GemmArgs p) {
  __shared__ __attribute__((aligned(1024))) unsigned char smem[DmaTile<WM, WN, MI, NI, BK, A_KC, B_KC, OutT, ST>::SMEM];
  int bx, bz;
  dma_renumber(blockIdx.x + gridDim.x * blockIdx.z, gridDim.x, gridDim.x * gridDim.z, bx, bz);
  gemm_dma_body<WM, WN, MI, NI, BK, A_KC, B_KC, OutT, ST>(p, bx, bz, smem);
}

// Both gradients of a Linear in one launch: workgroups below `first` (a multiple of 8, those past the tiles have nothing to do) take
// the weight gradient X^T dY, the longer reduction, the others the data gradient dY W^T.  MW, MX: matrix-instruction blocks of 32 rows
// per wavefront.
struct GemmPair { GemmArgs dw, dx; int first, dw_x, dw_total, dx_x, dx_total; };
template <int MW, int MX>
__global__ __launch_bounds__(256, 2) void gemm_dma_pair_kernel(GemmPair p) {
  constexpr int SW = DmaTile<2, 2, MW, 1, 64, false, false, float, 3>::SMEM, SX = DmaTile<2, 2, MX, 1, 64, true, true, bf16_raw, 3>::SMEM;
  __shared__ __attribute__((aligned(1024))) unsigned char smem[SW > SX ? SW : SX];
  int bx, bz;
  if ((int)blockIdx.x < p.first) {
    if ((int)blockIdx.x >= p.dw_total) return;
    dma_renumber(blockIdx.x, p.dw_x, p.dw_total, bx, bz);
    gemm_dma_body<2, 2, MW, 1, 64, false, false, float, 3>(p.dw, bx, bz, smem);
  } else {
    dma_renumber((int)blockIdx.x - p.first, p.dx_x, p.dx_total, bx, bz);
    gemm_dma_body<2, 2, MX, 1, 64, true, true, bf16_raw, 3>(p.dx, bx, bz, smem);
  }
}

int gemm_dma_tile(const GemmDesc& d);      // rows x columns of the tile the kernel would take, as an index; -1: not for it
int gemm_dma_launch(const GemmDesc& d, const GemmArgs& a, hipStream_t st);
bool gemm_dma_pair_takes(const GemmDesc& dw, const GemmDesc& dx);      // from the shapes alone
int gemm_dma_pair_launch(const GemmDesc& dw, const GemmArgs& aw, const GemmDesc& dx, const GemmArgs& ax, hipStream_t st);

}  // namespace hfta
