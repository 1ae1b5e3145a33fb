// fp32 form of the batched GEMM core (same descriptor, same operand kinds as gemm.h).
//
// The limit is the fp32 matrix instruction (157 TFLOP/s nominal; a library product of 8192 x 8192 x 8192 reaches 154 on
// this card); the short reductions it mostly gets (K = 64 and 128) run at 80-120, the rest being a tile's first loads and
// its epilogue.  One 32x32x2 instruction takes 64 cycles, so LDS and the vector ALU have room and what a k-tile
// must not do is wait for memory.  Hence: two k-tiles in flight in registers behind the one being
// multiplied, every load a raw buffer load without control flow (out of range = zeros, see gemm_pf.h);
// 16-byte pieces whatever the row pitch (a multi-dword access needs 4-byte alignment only, and an fp32 row
// has that), the piece that straddles a row's end read from where the row's last four elements start and
// moved into place on its way into LDS.  An operand contiguous along m / n stays in its natural [k][n]
// layout in LDS: a lane's fragment is one float, so 32 lanes read 32 neighbouring banks.
//
// NB: matrix blocks per wavefront and dimension.  NB = 2 (128x128 tile): the throughput form.  NB = 1 (64x64
// tile): four times the workgroups, a quarter of the matrix instructions per k-tile, for problems that would
// leave compute units idle.  VEC = false: single-element loads, for operands with fewer than four elements
// along their contiguous dimension.
#include "gemm_pf.h"

namespace hfta {

namespace {

constexpr int F32_BK = GemmT<float>::BK;                   // 16 floats of k per tile
constexpr int F32_SMALL_TILES = 512;                       // fewer 128x128 tiles than this: 64x64 tiles
typedef uint32_t pf_u32x4_a4 __attribute__((ext_vector_type(4), aligned(4)));

// rotates a four-element piece that was read `sh` elements early into place; what lies past the end becomes zero
__device__ __forceinline__ float4 shift_piece(float4 v, int sh) {
  if (sh & 1) v = make_float4(v.y, v.z, v.w, 0.f);
  if (sh & 2) v = make_float4(v.z, v.w, 0.f, 0.f);
  return v;
}

__device__ __forceinline__ float4 ld_f4(__amdgpu_buffer_rsrc_t rs, uint32_t off) {
  const pf_u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(rs, (int)off, 0, 0);
  return make_float4(__uint_as_float(v.x), __uint_as_float(v.y), __uint_as_float(v.z), __uint_as_float(v.w));
}
__device__ __forceinline__ float ld_f1(__amdgpu_buffer_rsrc_t rs, uint32_t off) {
  return __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rs, (int)off, 0, 0));
}

template <bool KC, int NB, bool VEC> struct F32Operand;

// k-contiguous: LDS [row][16 k + 4 pad]; thread t stages 4-float group t%4 of rows t/4 (+ 64)
template <int NB, bool VEC> struct F32Operand<true, NB, VEC> {
  static constexpr int BYTES = 64 * NB * GEMM_PITCH;
  typedef float4 Regs[NB];
  uint32_t off[NB];
  int kg;
  __device__ __forceinline__ void init(int row0, int rows, int64_t ld, int t) {
    kg = (t & 3) * 4;
#pragma unroll
    for (int h = 0; h < NB; ++h) {
      const int r = row0 + (t >> 2) + 64 * h;
      off[h] = r < rows ? (uint32_t)((int64_t)r * ld * 4) : PF_OOB;
    }
  }
  __device__ __forceinline__ void load(Regs& q, __amdgpu_buffer_rsrc_t rs, int k0, int K) const {
    const int k = k0 + kg;
#pragma unroll
    for (int h = 0; h < NB; ++h) {
      if (VEC) {
        q[h] = ld_f4(rs, k < K ? off[h] + (uint32_t)min(k, K - 4) * 4u : PF_OOB);
      } else {
        float e[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) e[i] = ld_f1(rs, k + i < K ? off[h] + (uint32_t)(k + i) * 4u : PF_OOB);
        q[h] = make_float4(e[0], e[1], e[2], e[3]);
      }
    }
  }
  // tail: the k-tile reaches past K (the same for the whole workgroup)
  __device__ __forceinline__ void store(unsigned char* tile, Regs& q, int t, int k0, int K) const {
    if (VEC && k0 + F32_BK > K) {
      const int k = k0 + kg, sh = k < K ? k - min(k, K - 4) : 0;
#pragma unroll
      for (int h = 0; h < NB; ++h) q[h] = shift_piece(q[h], sh);
    }
#pragma unroll
    for (int h = 0; h < NB; ++h) *reinterpret_cast<float4*>(tile + ((t >> 2) + 64 * h) * GEMM_PITCH + kg * 4) = q[h];
  }
  // the four k of step s for row base + lane%32: k = 8 s + 4 (lane/32) + j
  static __device__ __forceinline__ void frag(float (&f)[4], const unsigned char* tile, int base, int s, int lane) {
    const float4 v = *reinterpret_cast<const float4*>(tile + (base + (lane & 31)) * GEMM_PITCH + (2 * s + (lane >> 5)) * 16);
    f[0] = v.x; f[1] = v.y; f[2] = v.z; f[3] = v.w;
  }
};

// m/n-contiguous: LDS [16 k][64 NB columns + 8 pad]; k-rows four apart (the two lane halves of a fragment read)
// are 32 banks apart.  NB = 2: thread t stages columns 4 (t % 32) .. of k-rows t/32 and t/32 + 8; NB = 1: columns
// 4 (t % 16) .. of k-row t/16.
template <int NB, bool VEC> struct F32Operand<false, NB, VEC> {
  static constexpr int PITCH = (64 * NB + 8) * 4;          // 4 rows = 4 * 136 (or 72) dwords = 32 banks mod 64
  static constexpr int BYTES = F32_BK * PITCH;
  static constexpr int CG = 16 * NB, RS = GEMM_THREADS / CG;
  typedef float4 Regs[NB];
  uint32_t ldb;
  uint32_t coff;                                           // byte offset of the piece's column, or PF_OOB
  int kr, sh;
  __device__ __forceinline__ void init(int col0, int cols, int64_t ld, int t) {
    ldb = (uint32_t)(ld * 4);
    kr = t / CG;
    const int c = col0 + (t % CG) * 4;
    if (VEC) {
      const int cc = min(c, cols - 4);
      coff = c < cols ? (uint32_t)cc * 4u : PF_OOB;
      sh = c < cols ? c - cc : 0;
    } else {
      coff = (uint32_t)c * 4u;
      sh = cols - c;                                       // elements of the piece that exist (may exceed four)
    }
  }
  __device__ __forceinline__ void load(Regs& q, __amdgpu_buffer_rsrc_t rs, int k0, int K) const {
#pragma unroll
    for (int h = 0; h < NB; ++h) {
      const int k = k0 + kr + RS * h;
      if (VEC) {
        q[h] = ld_f4(rs, k < K && coff != PF_OOB ? (uint32_t)k * ldb + coff : PF_OOB);
      } else {
        float e[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) e[i] = ld_f1(rs, k < K && i < sh ? (uint32_t)k * ldb + coff + 4u * i : PF_OOB);
        q[h] = make_float4(e[0], e[1], e[2], e[3]);
      }
    }
  }
  __device__ __forceinline__ void store(unsigned char* tile, Regs& q, int t, int, int) const {
    if (VEC && __any(sh != 0)) {
#pragma unroll
      for (int h = 0; h < NB; ++h) q[h] = shift_piece(q[h], sh);
    }
#pragma unroll
    for (int h = 0; h < NB; ++h) *reinterpret_cast<float4*>(tile + (kr + RS * h) * PITCH + (t % CG) * 16) = q[h];
  }
  static __device__ __forceinline__ void frag(float (&f)[4], const unsigned char* tile, int base, int s, int lane) {
    const unsigned char* a = tile + (8 * s + 4 * (lane >> 5)) * PITCH + (base + (lane & 31)) * 4;
#pragma unroll
    for (int j = 0; j < 4; ++j) f[j] = *reinterpret_cast<const float*>(a + j * PITCH);
  }
};

template <int NB>
constexpr int f32_smem_bytes(int tiles) {
  const int epi = 64 * (64 * NB + 4) * 4; // the epilogue's staging: 64 rows at a time
  return tiles > epi ? tiles : epi;
}

template <bool A_KC, bool B_KC, int NB, bool VEC>
__global__ __launch_bounds__(GEMM_THREADS, 3) void gemm_f32_kernel(GemmArgs p) {
  typedef F32Operand<A_KC, NB, VEC> OA;
  typedef F32Operand<B_KC, NB, VEC> OB;
  constexpr int T = 64 * NB, PF = 2;
  __shared__ __attribute__((aligned(16))) unsigned char smem[f32_smem_bytes<NB>(2 * (OA::BYTES + OB::BYTES))];
  auto at = [&](int buf) { return smem + buf * OA::BYTES; };
  auto bt = [&](int buf) { return smem + 2 * OA::BYTES + buf * OB::BYTES; };

  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  const int wm = wave >> 1, wn = wave & 1;
  int bx = blockIdx.x, bz = blockIdx.z;
  {  // XCD-aware renumbering, as in gemm_kernel
    const int total = gridDim.x * gridDim.z, per = total >> 3;
    const int lin = blockIdx.x + gridDim.x * blockIdx.z;
    if (lin < (per << 3)) {
      const int l2 = (lin & 7) * per + (lin >> 3);
      bz = l2 / gridDim.x;
      bx = l2 - bz * gridDim.x;
    }
  }
  const int tile_m = bx % p.tiles_m, tile_n = bx / p.tiles_m;
  const int m0 = tile_m * T, n0 = tile_n * T;
  const int split = bz % p.splits, g = bz / p.splits;
  const int g0 = g / p.G1, g1 = g % p.G1;
  const float* Ab = reinterpret_cast<const float*>(p.A) + g0 * p.a_g0 + g1 * p.a_g1;
  const float* Bb = reinterpret_cast<const float*>(p.Bm) + g0 * p.b_g0 + g1 * p.b_g1;
  const int t_begin = (int)((int64_t)p.total_tiles * split / p.splits);
  const int t_end = (int)((int64_t)p.total_tiles * (split + 1) / p.splits);

  f32x16_t acc[NB][NB];
#pragma unroll
  for (int i = 0; i < NB; ++i)
#pragma unroll
    for (int j = 0; j < NB; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;

  OA oa;
  OB ob;
  oa.init(m0, p.M, p.a_ld, t);
  ob.init(n0, p.N, p.b_ld, t);
  typename OA::Regs ra[PF];
  typename OB::Regs rb[PF];
  auto k_of = [&](int tt) { return (tt % p.tiles_per_seg) * F32_BK; };
  auto issue = [&](int set, int tt) {
    const bool live = tt < t_end;
    const int Ke = live ? p.K : 0;                         // a dead tile has no valid k: nothing is requested
    const int tc = live ? tt : t_begin;
    const int seg = tc / p.tiles_per_seg;
    const int k0 = (tc - seg * p.tiles_per_seg) * F32_BK;
    oa.load(ra[set], pf_rsrc(Ab + seg * p.a_ss, p.a_extent), k0, Ke);
    ob.load(rb[set], pf_rsrc(Bb + seg * p.b_ss, p.b_extent), k0, Ke);
  };

  if (t_begin < t_end) {
#pragma unroll
    for (int d = 0; d < PF; ++d) issue(d, t_begin + d);
    oa.store(at(0), ra[0], t, k_of(t_begin), p.K);
    ob.store(bt(0), rb[0], t, k_of(t_begin), p.K);
    __syncthreads();
    int buf = 0;
    bool done = false;
    for (int base = t_begin; !done; base += PF) {
#pragma unroll
      for (int d = 0; d < PF; ++d) {
        const int cur = base + d;
        issue(d, cur + PF);
        const unsigned char* As = at(buf);
        const unsigned char* Bs = bt(buf);
#pragma unroll
        for (int s = 0; s < 2; ++s) {
          float a[NB][4], b[NB][4];
#pragma unroll
          for (int i = 0; i < NB; ++i) {
            OA::frag(a[i], As, wm * 32 * NB + i * 32, s, lane);
            OB::frag(b[i], Bs, wn * 32 * NB + i * 32, s, lane);
          }
#pragma unroll
          for (int k = 0; k < 4; ++k)
#pragma unroll
            for (int i = 0; i < NB; ++i)
#pragma unroll
              for (int j = 0; j < NB; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(b[j][k], a[i][k], acc[i][j], 0, 0, 0);
        }
        if (cur + 1 >= t_end) { done = true; break; }
        oa.store(at(buf ^ 1), ra[(d + 1) % PF], t, k_of(cur + 1), p.K);
        ob.store(bt(buf ^ 1), rb[(d + 1) % PF], t, k_of(cur + 1), p.K);
        __syncthreads();
        buf ^= 1;
      }
    }
    __syncthreads();
  }

  // ---- epilogue: 64 rows at a time through LDS, 16-byte pieces of whole row segments out ----
  const bool part = p.splits > 1;
  float* Cb = part ? p.partial + ((int64_t)split * (gridDim.z / p.splits) + g) * (int64_t)p.M * p.N
                   : reinterpret_cast<float*>(p.C) + g0 * p.c_g0 + g1 * p.c_g1;
  const int64_t c_ld = part ? p.N : p.c_ld;
  const float* bias = p.bias && !part ? reinterpret_cast<const float*>(p.bias) + g0 * p.bias_g0 + g1 * p.bias_g1 : nullptr;
  const int act = part ? HFTA_ACT_NONE : p.act;
  float* st = reinterpret_cast<float*>(smem);
  constexpr int SP = T + 4;                                // staging pitch, floats
  const int ml = lane & 31, nq = (lane >> 5) * 4;
#pragma unroll
  for (int pass = 0; pass < NB; ++pass) {
    if (NB == 1 || wm == pass) {
#pragma unroll
      for (int i = 0; i < NB; ++i) {
        const int rl = NB == 1 ? wm * 32 + ml : i * 32 + ml;
        const int m = m0 + pass * 64 + rl;
        float bm = 0.f;
        if (bias && p.bias_mode == 1 && m < p.M) bm = bias[m];
#pragma unroll
        for (int j = 0; j < NB; ++j)
#pragma unroll
          for (int q = 0; q < 4; ++q)
            *reinterpret_cast<float4*>(st + rl * SP + wn * 32 * NB + j * 32 + 8 * q + nq) =
                make_float4(acc[i][j][4 * q] + bm, acc[i][j][4 * q + 1] + bm, acc[i][j][4 * q + 2] + bm, acc[i][j][4 * q + 3] + bm);
      }
    }
    __syncthreads();
    constexpr int PPR = T / 4, RPI = GEMM_THREADS / PPR;   // pieces per row, rows per iteration
    const int c = t % PPR, n = n0 + c * 4;
    float cb[4] = {0.f, 0.f, 0.f, 0.f};
    if (bias && p.bias_mode == 2) {
#pragma unroll
      for (int e = 0; e < 4; ++e) cb[e] = n + e < p.N ? bias[n + e] : 0.f;
    }
#pragma unroll 4
    for (int it = 0; it < 64 / RPI; ++it) {
      const int rl = t / PPR + it * RPI, m = m0 + pass * 64 + rl;
      const float4 v = *reinterpret_cast<const float4*>(st + rl * SP + c * 4);
      float e[4] = {v.x + cb[0], v.y + cb[1], v.z + cb[2], v.w + cb[3]};
      if (act != HFTA_ACT_NONE) {
#pragma unroll
        for (int k = 0; k < 4; ++k) e[k] = apply_act(e[k], act, p.slope);
      }
      if (m >= p.M) continue;
      if (n + 4 <= p.N && (part || p.c_seg <= 0)) {
        *reinterpret_cast<pf_u32x4_a4*>(Cb + (int64_t)m * c_ld + n) =
            pf_u32x4_a4{__float_as_uint(e[0]), __float_as_uint(e[1]), __float_as_uint(e[2]), __float_as_uint(e[3])};
      } else {
#pragma unroll
        for (int k = 0; k < 4; ++k)
          if (n + k < p.N) Cb[(int64_t)m * c_ld + (part ? (int64_t)(n + k) : col_offset(n + k, p.c_seg, p.c_seg_stride))] = e[k];
      }
    }
    if (pass + 1 < NB) __syncthreads();
  }
}

template <int NB, bool VEC>
int f32_layout(const GemmDesc& d, const GemmArgs& a, dim3 grid, hipStream_t st) {
  if (d.a_kc && !d.b_kc) hipLaunchKernelGGL((gemm_f32_kernel<true, false, NB, VEC>), grid, dim3(GEMM_THREADS), 0, st, a);
  else if (d.a_kc && d.b_kc) hipLaunchKernelGGL((gemm_f32_kernel<true, true, NB, VEC>), grid, dim3(GEMM_THREADS), 0, st, a);
  else if (!d.a_kc && !d.b_kc) hipLaunchKernelGGL((gemm_f32_kernel<false, false, NB, VEC>), grid, dim3(GEMM_THREADS), 0, st, a);
  else return HFTA_EUNSUPPORTED;
  return launch_status();
}

}  // namespace

// HFTA_EUNSUPPORTED: an operand slice does not fit a buffer descriptor (nothing has been launched).
int gemm_f32_launch(const GemmDesc& d, const GemmArgs& base, hipStream_t st) {
  GemmArgs a = base;
  const int64_t a_ext = ((d.a_kc ? (int64_t)(d.M - 1) * d.a_ld + d.K : (int64_t)(d.K - 1) * d.a_ld + d.M)) * 4;
  const int64_t b_ext = ((d.b_kc ? (int64_t)(d.N - 1) * d.b_ld + d.K : (int64_t)(d.K - 1) * d.b_ld + d.N)) * 4;
  if (a_ext >= (int64_t)1 << 31 || b_ext >= (int64_t)1 << 31 || d.a_ld <= 0 || d.b_ld <= 0) return HFTA_EUNSUPPORTED;
  a.a_extent = (uint32_t)a_ext;
  a.b_extent = (uint32_t)b_ext;
  const int64_t G = (int64_t)d.G0 * d.G1;
  const int64_t t128 = (int64_t)((d.M + 127) / 128) * ((d.N + 127) / 128) * G * a.splits;
  const bool small = t128 < F32_SMALL_TILES || d.M <= 64 || d.N <= 64;
  const int T = small ? 64 : 128;
  a.tiles_m = (d.M + T - 1) / T;
  a.tiles_n = (d.N + T - 1) / T;
  dim3 grid((unsigned)(a.tiles_m * a.tiles_n), 1, (unsigned)(G * a.splits));
  const bool vec = d.K >= 4 && (d.a_kc || d.M >= 4) && (d.b_kc || d.N >= 4);
  if (small) return vec ? f32_layout<1, true>(d, a, grid, st) : f32_layout<1, false>(d, a, grid, st);
  return vec ? f32_layout<2, true>(d, a, grid, st) : f32_layout<2, false>(d, a, grid, st);
}

}  // namespace hfta
