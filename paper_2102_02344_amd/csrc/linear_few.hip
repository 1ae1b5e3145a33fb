// Linear layers of few rows with the operators that stand beside them: the fully connected head of a point-cloud model.
//
// A head of three layers on 32 rows a model ran as 26 launches (split products, their sums, BatchNorm, dropout, cross-entropy,
// and the way back), each as long as a launch that waits for the one before it takes: 4.5-10 us, 134 us of a bf16 step of 8 models
// whose weights are 10 MB.  With at most 32 rows a column of a layer's output is one column of one matrix-instruction tile, so
// everything that works by columns -- BatchNorm over the rows, its activation, the dropout behind it, and all of it backwards --
// is done by the workgroup that has the product in hand: six launches, 51 us of that step (12, 8 and 7 forward, 8, 7 and 9 back; 1376 ->
// 1310 a step), and on 3 models of 13 clouds 114 -> 40 us (411 -> 351 a step).  In fp32 two models of 4 clouds
// (1024 -> 256 -> 16, no BatchNorm) 58 -> 30 us (185 -> 161 a step), four of 32 clouds 2026 -> 1979 a step.  With many models the single
// operators are the sooner way: few_pays, few_ws_pays.
//
// Bound: the wait for one launch, one load of the operands (all of a workgroup's in flight at once) and the chain of the matrix
// instructions and the row sums behind them.  Hence 32-column tiles, as many workgroups as that gives, and the forward's
// reduction cut over the wavefronts of a workgroup in the pieces that the split product cuts it in.
//
// The bits are those of the single operators: the same split of the reduction added in the same order, the same instruction (fp32:
// the fp32 one up to 64 k, the product of three bf16 parts above, see gemm_f32.hip), BatchNorm's sums over 16 row lanes, every
// stored tensor rounded where it was.  (The heads of the transform sub-networks turn a last-bit difference into percents a few
// layers on.)
#include "gemm_pf.h"
#include "bn_common.h"
#include "f32_split.h"

namespace hfta {
int linear_row_splits(int B, int M, int Fx, int Fy, int dtype);
bool gemm_f32_big_tiles(int M, int N, int64_t G);
}

using namespace hfta;

namespace {

constexpr int FEW_ROWS = 32;                             // one matrix-instruction tile
constexpr int FEW_LANES = 16;                            // row lanes of BatchNorm's sums (bn_fwd_linear_kernel)
constexpr int FWD_WAVES = 16;                            // most wavefronts of a workgroup
constexpr int PART_PITCH = 36;                           // floats: 32 columns and a pad
constexpr int PART_BYTES = FEW_ROWS * PART_PITCH * 4;    // one piece of the reduction
// bf16: W's columns in LDS, 64 bytes per k, and the partial sums over them; two workgroups a compute unit (82,048 bytes with the
// cross-entropy's tile, one: there is one a model).  fp32: the partial sums of 32 pieces, one workgroup a compute unit whatever the split;
// two of 128 registers spill beside BatchNorm and the cross-entropy.
template <typename T> struct FewFwd;
template <> struct FewFwd<bf16_raw> { static constexpr int LDS = 76 * 1024, MAX_K = LDS / 64, SPLITS = 16; };
template <> struct FewFwd<float> { static constexpr int SPLITS = 32, LDS = SPLITS * PART_BYTES; };
static_assert(FewFwd<bf16_raw>::SPLITS * PART_BYTES <= FewFwd<bf16_raw>::LDS && FewFwd<bf16_raw>::SPLITS <= FWD_WAVES, "the partial sums");

struct FewFwdArgs {
  const void* X; const void* W; const void* bias; void* Z;
  int M, Fx, Fy, splits;
  const float* gamma; const float* beta; float* rm; float* rv; float* save_mean; float* save_invstd; void* Y;
  const uint8_t* mask; void* Yd;
  float eps, momentum, slope, scale;
  int act;
  const int32_t* labels; float* loss; void* dlogits;
};

// matrix-instruction fragment of a [16 k][columns] tile kept as it lies in memory (see pf_frag)
template <int PITCH> __device__ __forceinline__ bf16x8_t nat_frag(const unsigned char* tile, int base, int s, int lane) {
  const int r16 = lane & 15;
  const unsigned char* a0 = tile + (16 * s + 8 * (lane >> 5) + (r16 >> 2)) * PITCH + (base + 16 * ((lane >> 4) & 1) + 4 * (r16 & 3)) * 2;
  typedef __attribute__((address_space(3))) pf_v4s* lds_v4s;
  union { pf_v4s h[2]; bf16x8_t v; } u;
  u.h[0] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4s)(a0));
  u.h[1] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4s)(a0 + 4 * PITCH));
  return u.v;
}

__device__ __forceinline__ uint4 load16(__amdgpu_buffer_rsrc_t rs, bool ok, int64_t elem) {
  const pf_u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(rs, (int)(ok ? (uint32_t)(elem * 2) : PF_OOB), 0, 0);
  return make_uint4(v.x, v.y, v.z, v.w);
}

// sum over the 16 row lanes of a column, in order
__device__ __forceinline__ float lane_sum(float (*red)[FEW_ROWS], int c) {
  float s = 0.f;
#pragma unroll
  for (int j = 0; j < FEW_LANES; ++j) s += red[j][c];
  return s;
}

__device__ __forceinline__ float4 load16f(__amdgpu_buffer_rsrc_t rs, bool ok, int64_t elem) {
  const pf_u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(rs, (int)(ok ? (uint32_t)(elem * 4) : PF_OOB), 0, 0);
  return make_float4(__uint_as_float(v.x), __uint_as_float(v.y), __uint_as_float(v.z), __uint_as_float(v.w));
}
__device__ __forceinline__ float load4f(__amdgpu_buffer_rsrc_t rs, bool ok, int64_t elem) {
  return __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rs, (int)(ok ? (uint32_t)(elem * 4) : PF_OOB), 0, 0));
}
__device__ __forceinline__ void mfma_f32x4(f32x16_t& acc, const float4& first, const float4& second) {
  acc = __builtin_amdgcn_mfma_f32_32x32x2f32(first.x, second.x, acc, 0, 0, 0);
  acc = __builtin_amdgcn_mfma_f32_32x32x2f32(first.y, second.y, acc, 0, 0, 0);
  acc = __builtin_amdgcn_mfma_f32_32x32x2f32(first.z, second.z, acc, 0, 0, 0);
  acc = __builtin_amdgcn_mfma_f32_32x32x2f32(first.w, second.w, acc, 0, 0, 0);
}
// lane l holds row l % 32, columns 8q + 4(l / 32) .. + 3
__device__ __forceinline__ void put_tile(float* part, const f32x16_t& acc, int lane) {
#pragma unroll
  for (int q = 0; q < 4; ++q)
    *reinterpret_cast<float4*>(part + (lane & 31) * PART_PITCH + 8 * q + 4 * (lane >> 5)) =
        make_float4(acc[4 * q], acc[4 * q + 1], acc[4 * q + 2], acc[4 * q + 3]);
}

// The products of the forward: wavefront w takes the k-tiles that split w (fp32: also w + wavefronts) of the split product takes
// (linear_fwd_splits) and leaves its sums in smem.
template <typename T> __device__ __forceinline__ void few_fwd_product(const FewFwdArgs& p, unsigned char* smem, int n0, int b, int wave, int lane);

template <> __device__ __forceinline__ void few_fwd_product<bf16_raw>(const FewFwdArgs& p, unsigned char* smem, int n0, int b, int wave, int lane) {
  const int tt = (p.Fx + 31) / 32;                       // k-tiles of 32
  f32x16_t acc;
#pragma unroll
  for (int v = 0; v < 16; ++v) acc[v] = 0.f;
  if (wave < p.splits) {
    const int t0 = tt * wave / p.splits, t1 = tt * (wave + 1) / p.splits;
    const __amdgpu_buffer_rsrc_t rx = pf_rsrc((const bf16_raw*)p.X + (int64_t)b * p.M * p.Fx, (uint32_t)p.M * p.Fx * 2u);
    const __amdgpu_buffer_rsrc_t rw = pf_rsrc((const bf16_raw*)p.W + (int64_t)b * p.Fx * p.Fy, (uint32_t)p.Fx * p.Fy * 2u);
    const int row = lane & 31, xk = 8 * (lane >> 5), wk = lane >> 2, wc = n0 + (lane & 3) * 8;
    for (int tb = t0; tb < t1; tb += 4) {                // 128 k in flight
      uint4 xa[8], wv[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const int k0 = tb * 32 + u * 16;
        const bool live = tb + u / 2 < t1;
        wv[u] = load16(rw, live && k0 + wk < p.Fx && wc < p.Fy, (int64_t)(k0 + wk) * p.Fy + wc);
        xa[u] = load16(rx, live && row < p.M && k0 + xk < p.Fx, (int64_t)row * p.Fx + k0 + xk);
      }
#pragma unroll
      for (int u = 0; u < 8; ++u)
        if (tb + u / 2 < t1) *reinterpret_cast<uint4*>(smem + (tb * 2 + u) * 1024 + lane * 16) = wv[u];
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");  // a wavefront reads its own k-tiles alone
#pragma unroll
      for (int u = 0; u < 8; ++u)
        if (tb + u / 2 < t1)
          acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(nat_frag<64>(smem + (tb * 2 + u) * 1024, 0, 0, lane),
                                                        *reinterpret_cast<const bf16x8_t*>(&xa[u]), acc, 0, 0, 0);
    }
  }
  __syncthreads();                                       // the sums lie over the operand
  if (wave < p.splits) put_tile(reinterpret_cast<float*>(smem + wave * PART_BYTES), acc, lane);
}

// The fp32 instruction takes one k of a column per lane: both operands come from memory in its layout, W by whole 128-byte rows.
template <> __device__ __forceinline__ void few_fwd_product<float>(const FewFwdArgs& p, unsigned char* smem, int n0, int b, int wave, int lane) {
  const int tt = (p.Fx + 15) / 16;                       // k-tiles of 16
  const __amdgpu_buffer_rsrc_t rx = pf_rsrc((const float*)p.X + (int64_t)b * p.M * p.Fx, (uint32_t)p.M * p.Fx * 4u);
  const __amdgpu_buffer_rsrc_t rw = pf_rsrc((const float*)p.W + (int64_t)b * p.Fx * p.Fy, (uint32_t)p.Fx * p.Fy * 4u);
  const int row = lane & 31, hk = 4 * (lane >> 5), c = n0 + row;
  for (int sp = wave; sp < p.splits; sp += (int)(blockDim.x >> 6)) {
    const int t0 = tt * sp / p.splits, t1 = tt * (sp + 1) / p.splits;
    f32x16_t acc;
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[v] = 0.f;
    for (int k0 = t0 * 16; k0 < t1 * 16; k0 += 64) {     // 64 k in flight
      float4 x[8], w[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const int k = k0 + 8 * u + hk;
        const bool live = k < t1 * 16 && k < p.Fx;       // Fx is a multiple of 4
        x[u] = load16f(rx, live && row < p.M, (int64_t)row * p.Fx + k);
        float e[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) e[j] = load4f(rw, live && c < p.Fy, (int64_t)(k + j) * p.Fy + c);
        w[u] = make_float4(e[0], e[1], e[2], e[3]);
      }
#pragma unroll
      for (int u = 0; u < 8; ++u)
        if (k0 + 8 * u < t1 * 16) mfma_f32x4(acc, w[u], x[u]);
    }
    put_tile(reinterpret_cast<float*>(smem + sp * PART_BYTES), acc, lane);
  }
}

// Z = X W + bias for 32 columns of one model, then
//   FEW_ACT   the activation
//   FEW_BN    BatchNorm over the rows, activation, dropout (mask given)
//   FEW_XENT  softmax cross-entropy over the columns (at most 32: one workgroup holds them all)
enum { FEW_ACT, FEW_BN, FEW_XENT };
template <typename T, int KIND>
__global__ __launch_bounds__(64 * FWD_WAVES) void linear_few_fwd_kernel(FewFwdArgs p) {
  __shared__ __attribute__((aligned(16))) unsigned char smem[FewFwd<T>::LDS];
  __shared__ float red[KIND == FEW_BN ? FEW_LANES : 1][FEW_ROWS];
  const int t = threadIdx.x, lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const int n0 = blockIdx.x * 32, b = blockIdx.y;
  few_fwd_product<T>(p, smem, n0, b, wave, lane);
  const float* part = reinterpret_cast<const float*>(smem);
  __syncthreads();
  const int col = t & 31, ty = (t >> 5) & (FEW_LANES - 1), c = n0 + col;
  const bool mine = t < 32 * FEW_LANES, live = mine && c < p.Fy;
  const float bias = p.bias && live ? Elem<T>::load((const T*)p.bias + (int64_t)b * p.Fy + c) : 0.f;
  float z[2] = {0.f, 0.f};                               // rows ty and ty + 16, as stored
  T* zrow = (T*)p.Z + ((int64_t)b * p.M) * p.Fy + c;
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const int r = ty + FEW_LANES * h;
    float s = 0.f;
    for (int k = 0; k < p.splits; ++k) s += part[(k * FEW_ROWS + r) * PART_PITCH + col];
    if (p.bias) s += bias;
    if (KIND == FEW_ACT) s = bn_act(s, p.act, p.slope);
    const T o = Elem<T>::from_f32(s);
    z[h] = Elem<T>::to_f32(o);
    if (live && r < p.M) zrow[(int64_t)r * p.Fy] = o;
  }
  if constexpr (KIND == FEW_BN) {
    auto column_sum = [&](float v) {
      __syncthreads();
      if (mine) red[ty][col] = v;
      __syncthreads();
      return lane_sum(red, col);
    };
    const bool has[2] = {ty < p.M, ty + FEW_LANES < p.M};
    float s = 0.f;
#pragma unroll
    for (int h = 0; h < 2; ++h)
      if (has[h]) s += z[h];
    const float m = (float)p.M, mean = column_sum(s) / m;
    float q = 0.f;
#pragma unroll
    for (int h = 0; h < 2; ++h)
      if (has[h]) { const float d = z[h] - mean; q = fmaf(d, d, q); }
    const float var = column_sum(q) / m, invstd = 1.0f / sqrtf(var + p.eps);
    if (!live) return;
    const int k = b * p.Fy + c;
    const float g = p.gamma[k], bt = p.beta[k];
    if (ty == 0) {
      p.save_mean[k] = mean;
      p.save_invstd[k] = invstd;
      if (p.rm) {
        const float unb = m > 1.f ? var * (m / (m - 1.f)) : var;
        p.rm[k] = (1.f - p.momentum) * p.rm[k] + p.momentum * mean;
        p.rv[k] = (1.f - p.momentum) * p.rv[k] + p.momentum * unb;
      }
    }
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      if (!has[h]) continue;
      const int64_t i = ((int64_t)b * p.M + ty + FEW_LANES * h) * p.Fy + c;
      const T y = Elem<T>::from_f32(bn_act(fmaf(g, (z[h] - mean) * invstd, bt), p.act, p.slope));
      ((T*)p.Y)[i] = y;
      if (p.mask) Elem<T>::store((T*)p.Yd + i, p.mask[i] ? Elem<T>::to_f32(y) * p.scale : 0.f);
    }
  } else if constexpr (KIND == FEW_XENT) {
    __shared__ float zt[FEW_ROWS][33];
    if (mine) { zt[ty][col] = z[0]; zt[ty + FEW_LANES][col] = z[1]; }
    __syncthreads();
    if (wave != 0) return;
    // a lane per row, as softmax_xent_kernel
    const int K = p.Fy;
    float a = 0.f;
    const float invR = 1.f / (float)p.M;
    if (lane < p.M) {
      const float* zr = zt[lane];
      T* dz = (T*)p.dlogits + ((int64_t)b * p.M + lane) * K;
      const int lab = p.labels[(int64_t)b * p.M + lane];
      float mx = -INFINITY;
      for (int k = 0; k < K; ++k) mx = fmaxf(mx, zr[k]);
      float se = 0.f;
      for (int k = 0; k < K; ++k) se += expf(zr[k] - mx);
      const float lse = mx + logf(se);
      a += lse - label_score(zr, lab, K);
      for (int k = 0; k < K; ++k) {
        const float pk = expf(zr[k] - lse);
        Elem<T>::store(dz + k, (pk - (k == lab ? 1.f : 0.f)) * invR);
      }
    }
    const float s = wave_sum(a);
    if (lane == 0) p.loss[b] = s * invR;
  }
}

constexpr int DW_BM = 128, DW_BN = 64, DW_XP = DW_BM * 2 + 64, DW_YP = DW_BN * 2 + 64;
// k of dX's product in LDS at a time; bytes of an operand's row there (fp32: of one of its three planes)
template <typename T> struct FewBwd;
template <> struct FewBwd<bf16_raw> { static constexpr int K = 512, PITCH = K * 2 + 16, LDS = 2 * FEW_ROWS * PITCH; };
template <> struct FewBwd<float> { static constexpr int K = 256, PITCH = K * 2 + 16, PLANE = FEW_ROWS * PITCH, LDS = 6 * PLANE; };
static_assert(FEW_ROWS * (DW_XP + DW_YP) <= FewBwd<bf16_raw>::LDS, "the weight gradient's operands");
constexpr int FEW_F32_EXACT_K = 64;                      // up to here the fp32 instruction, as gemm_f32_launch

struct FewBwdArgs {
  const void* X; const void* W; const void* dY; void* dX; float* dW; float* dbias;
  int M, Fx, Fy, dx_tiles, dw_m;
  const void* Z; const float* gamma; const float* beta; const float* save_mean; const float* save_invstd;
  const uint8_t* mask; float* dgamma; float* dbeta; float* dx_sum;
  float slope, scale;
  int act;
};

__device__ __forceinline__ void clear_tile(f32x16_t& acc) {
#pragma unroll
  for (int v = 0; v < 16; ++v) acc[v] = 0.f;
}

// 128 x 64 of dW = X^T dY at (m0, n0), 32 rows a wavefront; lane l ends with column l % 32 of either half and rows
// 8(v / 4) + 4(l / 32) + v % 4, so that a store is whole 128-byte row segments
template <typename T> __device__ __forceinline__ void few_dw_product(const FewBwdArgs& p, unsigned char* smem, int m0, int n0, int b, int wave,
                                                                     int lane, f32x16_t (&acc)[2]);
template <> __device__ __forceinline__ void few_dw_product<bf16_raw>(const FewBwdArgs& p, unsigned char* smem, int m0, int n0, int b, int wave,
                                                                     int lane, f32x16_t (&acc)[2]) {
  const int t = threadIdx.x;
  const __amdgpu_buffer_rsrc_t rx = pf_rsrc((const bf16_raw*)p.X + (int64_t)b * p.M * p.Fx, (uint32_t)p.M * p.Fx * 2u);
  const __amdgpu_buffer_rsrc_t ry = pf_rsrc((const bf16_raw*)p.dY + (int64_t)b * p.M * p.Fy, (uint32_t)p.M * p.Fy * 2u);
  unsigned char* xs = smem;
  unsigned char* ys = smem + FEW_ROWS * DW_XP;
  uint4 x[2];
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int r = (t >> 4) + 16 * i, c = m0 + (t & 15) * 8;
    x[i] = load16(rx, r < p.M && c < p.Fx, (int64_t)r * p.Fx + c);
  }
  const int yr = t >> 3, yc = n0 + (t & 7) * 8;
  const uint4 y = load16(ry, yr < p.M && yc < p.Fy, (int64_t)yr * p.Fy + yc);
#pragma unroll
  for (int i = 0; i < 2; ++i) *reinterpret_cast<uint4*>(xs + ((t >> 4) + 16 * i) * DW_XP + (t & 15) * 16) = x[i];
  *reinterpret_cast<uint4*>(ys + yr * DW_YP + (t & 7) * 16) = y;
  __syncthreads();
#pragma unroll
  for (int s = 0; s < 2; ++s) {
    const bf16x8_t a = nat_frag<DW_XP>(xs, wave * 32, s, lane);
#pragma unroll
    for (int j = 0; j < 2; ++j) acc[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, nat_frag<DW_YP>(ys, j * 32, s, lane), acc[j], 0, 0, 0);
  }
}
template <> __device__ __forceinline__ void few_dw_product<float>(const FewBwdArgs& p, unsigned char*, int m0, int n0, int b, int wave, int lane,
                                                                  f32x16_t (&acc)[2]) {
  const __amdgpu_buffer_rsrc_t rx = pf_rsrc((const float*)p.X + (int64_t)b * p.M * p.Fx, (uint32_t)p.M * p.Fx * 4u);
  const __amdgpu_buffer_rsrc_t ry = pf_rsrc((const float*)p.dY + (int64_t)b * p.M * p.Fy, (uint32_t)p.M * p.Fy * 4u);
  const int c = lane & 31, hk = 4 * (lane >> 5), m = m0 + wave * 32 + c;
  float x[4][4], y[2][4][4];
#pragma unroll
  for (int s = 0; s < 4; ++s)
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const int r = 8 * s + hk + k;
      x[s][k] = load4f(rx, r < p.M && m < p.Fx, (int64_t)r * p.Fx + m);
#pragma unroll
      for (int j = 0; j < 2; ++j) y[j][s][k] = load4f(ry, r < p.M && n0 + 32 * j + c < p.Fy, (int64_t)r * p.Fy + n0 + 32 * j + c);
    }
#pragma unroll
  for (int s = 0; s < 4; ++s)
#pragma unroll
    for (int k = 0; k < 4; ++k)
#pragma unroll
      for (int j = 0; j < 2; ++j) acc[j] = __builtin_amdgcn_mfma_f32_32x32x2f32(x[s][k], y[j][s][k], acc[j], 0, 0, 0);
}

// 32 columns of dX = dY W^T from f0 on, over the whole reduction, in the first wavefront's accumulators: all of a chunk's loads in
// flight, one chain of matrix instructions.  Lane l ends with row l % 32 and columns 8q + 4(l / 32) .. + 3.
template <typename T> __device__ __forceinline__ void few_dx_product(const FewBwdArgs& p, unsigned char* smem, int f0, int b, int wave, int lane,
                                                                     f32x16_t& acc);
template <> __device__ __forceinline__ void few_dx_product<bf16_raw>(const FewBwdArgs& p, unsigned char* smem, int f0, int b, int wave, int lane,
                                                                     f32x16_t& acc) {
  typedef FewBwd<bf16_raw> F;
  const int t = threadIdx.x;
  const __amdgpu_buffer_rsrc_t ry = pf_rsrc((const bf16_raw*)p.dY + (int64_t)b * p.M * p.Fy, (uint32_t)p.M * p.Fy * 2u);
  const __amdgpu_buffer_rsrc_t rw = pf_rsrc((const bf16_raw*)p.W + (int64_t)b * p.Fx * p.Fy, (uint32_t)p.Fx * p.Fy * 2u);
  unsigned char* ds = smem;
  unsigned char* ws = smem + FEW_ROWS * F::PITCH;
  for (int k0 = 0; k0 < p.Fy; k0 += F::K) {
    const int kc = min(F::K, p.Fy - k0), ppr = (kc + 15) / 16 * 2, steps = ppr / 2;    // 16-byte pieces of a row
    uint4 d[8], w[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int e = t + 256 * i, r = e / ppr, k = k0 + (e - r * ppr) * 8;
      d[i] = load16(ry, r < p.M && k < p.Fy, (int64_t)r * p.Fy + k);
      w[i] = load16(rw, r < FEW_ROWS && f0 + r < p.Fx && k < p.Fy, (int64_t)(f0 + r) * p.Fy + k);
    }
    if (k0) __syncthreads();                             // the chunk before has been read
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int e = t + 256 * i, r = e / ppr, at = r * F::PITCH + (e - r * ppr) * 16;
      if (r < FEW_ROWS) {
        *reinterpret_cast<uint4*>(ds + at) = d[i];
        *reinterpret_cast<uint4*>(ws + at) = w[i];
      }
    }
    __syncthreads();
    if (wave == 0) {
      const int at = (lane & 31) * F::PITCH + (lane >> 5) * 16;
#pragma unroll 8
      for (int s = 0; s < steps; ++s)
        acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(*reinterpret_cast<const bf16x8_t*>(ws + at + s * 32),
                                                      *reinterpret_cast<const bf16x8_t*>(ds + at + s * 32), acc, 0, 0, 0);
    }
  }
}
template <> __device__ __forceinline__ void few_dx_product<float>(const FewBwdArgs& p, unsigned char* smem, int f0, int b, int wave, int lane,
                                                                  f32x16_t& acc) {
  typedef FewBwd<float> F;
  const int t = threadIdx.x;
  const __amdgpu_buffer_rsrc_t ry = pf_rsrc((const float*)p.dY + (int64_t)b * p.M * p.Fy, (uint32_t)p.M * p.Fy * 4u);
  const __amdgpu_buffer_rsrc_t rw = pf_rsrc((const float*)p.W + (int64_t)b * p.Fx * p.Fy, (uint32_t)p.Fx * p.Fy * 4u);
  // the fp32 instruction from memory in its own layout
  auto exact = [&]() {
    if (wave != 0) return;
    clear_tile(acc);
    const int row = lane & 31, hk = 4 * (lane >> 5);
    for (int k0 = 0; k0 < p.Fy; k0 += 64) {
      float4 d[8], w[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const int k = k0 + 8 * u + hk;                   // Fy is a multiple of 4
        d[u] = load16f(ry, row < p.M && k < p.Fy, (int64_t)row * p.Fy + k);
        w[u] = load16f(rw, f0 + row < p.Fx && k < p.Fy, (int64_t)(f0 + row) * p.Fy + k);
      }
#pragma unroll
      for (int u = 0; u < 8; ++u)
        if (k0 + 8 * u < p.Fy) mfma_f32x4(acc, w[u], d[u]);
    }
  };
  if (p.Fy <= FEW_F32_EXACT_K) { exact(); return; }
  f32x16_t low;
  clear_tile(low);
  SplitSeen seen;
  for (int k0 = 0; k0 < p.Fy; k0 += F::K) {
    const int kc = min(F::K, p.Fy - k0), ppr = (kc + 15) / 16 * 4, steps = ppr / 4;    // four-element pieces of a row
    float4 d[8], w[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int e = t + 256 * i, r = e / ppr, k = k0 + (e - r * ppr) * 4;
      d[i] = load16f(ry, r < p.M && k < p.Fy, (int64_t)r * p.Fy + k);
      w[i] = load16f(rw, r < FEW_ROWS && f0 + r < p.Fx && k < p.Fy, (int64_t)(f0 + r) * p.Fy + k);
    }
    if (k0) __syncthreads();                             // the chunk before has been read
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int e = t + 256 * i, r = e / ppr, at = r * F::PITCH + (e - r * ppr) * 8;
      if (r < FEW_ROWS) {
        uint2 o[3];
        split4(d[i], o, seen);
#pragma unroll
        for (int pl = 0; pl < 3; ++pl) *reinterpret_cast<uint2*>(smem + pl * F::PLANE + at) = o[pl];
        split4(w[i], o, seen);
#pragma unroll
        for (int pl = 0; pl < 3; ++pl) *reinterpret_cast<uint2*>(smem + (3 + pl) * F::PLANE + at) = o[pl];
      }
    }
    __syncthreads();
    if (wave == 0) {
      const int at = (lane & 31) * F::PITCH + (lane >> 5) * 16;
#pragma unroll 2
      for (int s = 0; s < steps; ++s) {
        bf16x8_t x[3], y[3];
#pragma unroll
        for (int pl = 0; pl < 3; ++pl) {
          x[pl] = *reinterpret_cast<const bf16x8_t*>(smem + pl * F::PLANE + at + s * 32);
          y[pl] = *reinterpret_cast<const bf16x8_t*>(smem + (3 + pl) * F::PLANE + at + s * 32);
        }
        constexpr int PA[6] = {2, 1, 0, 1, 0, 0}, PB[6] = {0, 1, 2, 0, 1, 0};
#pragma unroll
        for (int q = 0; q < 6; ++q) {
          f32x16_t& c = q < 5 ? low : acc;
          c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(y[PB[q]], x[PA[q]], c, 0, 0, 0);
        }
      }
    }
  }
#pragma unroll
  for (int v = 0; v < 16; ++v) acc[v] += low[v];
  if (__syncthreads_or(seen.bad())) exact();
}

// Both gradients of one Linear.  Workgroups below dx_tiles take 32 columns of dX and carry them on: FEW_BN through the dropout,
// activation and BatchNorm of the layer below (Z: what that BatchNorm normalised), FEW_ACT through its dropout and activation (Z: the
// activation's output), FEW_PLAIN not.  The others take 128 x 64 of dW, the first of them per column block the column sums of dY.
enum { FEW_PLAIN = 2 };
template <typename T, int KIND>
__global__ __launch_bounds__(256) void linear_few_bwd_kernel(FewBwdArgs p) {
  __shared__ __attribute__((aligned(16))) unsigned char smem[FewBwd<T>::LDS];
  __shared__ float red[FEW_LANES][FEW_ROWS];
  const int t = threadIdx.x, lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const int b = blockIdx.y;
  f32x16_t acc[2];
  clear_tile(acc[0]);
  clear_tile(acc[1]);

  if ((int)blockIdx.x >= p.dx_tiles) {                   // ---- dW
    const int q = (int)blockIdx.x - p.dx_tiles, m0 = (q % p.dw_m) * DW_BM, n0 = (q / p.dw_m) * DW_BN;
    few_dw_product<T>(p, smem, m0, n0, b, wave, lane, acc);
    float* out = p.dW + (int64_t)b * p.Fx * p.Fy;
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const int n = n0 + 32 * j + (lane & 31);
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const int m = m0 + wave * 32 + 8 * (v >> 2) + 4 * (lane >> 5) + (v & 3);
        if (m < p.Fx && n < p.Fy) out[(int64_t)m * p.Fy + n] = acc[j][v];
      }
    }
    if (p.dbias && m0 == 0) {                            // as colsum_kernel: four row slices
      float (*sl)[DW_BN] = reinterpret_cast<float (*)[DW_BN]>(&red[0][0]);
      const int c = t & 63, slice = t >> 6;
      float s = 0.f;
      if (n0 + c < p.Fy) {
        const T* y = (const T*)p.dY + (int64_t)b * p.M * p.Fy + n0 + c;
        for (int r = slice; r < p.M; r += 4) s += Elem<T>::load(y + (int64_t)r * p.Fy);
      }
      sl[slice][c] = s;
      __syncthreads();
      if (slice == 0 && n0 + c < p.Fy) p.dbias[(int64_t)b * p.Fy + n0 + c] = (sl[0][c] + sl[1][c]) + (sl[2][c] + sl[3][c]);
    }
    return;
  }

  const int f0 = blockIdx.x * 32;
  few_dx_product<T>(p, smem, f0, b, wave, lane, acc[0]);
  __syncthreads();
  float* tile = reinterpret_cast<float*>(smem);          // [32 rows][32 columns]
  if (wave == 0) put_tile(tile, acc[0], lane);
  __syncthreads();
  const int col = t & 31, ty = t >> 5, c = f0 + col;     // row lanes ty and ty + 8
  const bool live = c < p.Fx;
  const int64_t at0 = (int64_t)b * p.M * p.Fx + c;
  T dx[4];                                               // rows ty, ty + 16 (lane ty), ty + 8, ty + 24 (lane ty + 8)
#pragma unroll
  for (int i = 0; i < 4; ++i) dx[i] = Elem<T>::from_f32(tile[(ty + 8 * (i >> 1) + 16 * (i & 1)) * PART_PITCH + col]);
  T* out = (T*)p.dX;
  if constexpr (KIND == FEW_PLAIN) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int r = ty + 8 * (i >> 1) + 16 * (i & 1);
      if (live && r < p.M) out[at0 + (int64_t)r * p.Fx] = dx[i];
    }
    return;
  }
  // the dropout below, and what its activation and BatchNorm work on
  float dy[4], z[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int r = ty + 8 * (i >> 1) + 16 * (i & 1);
    const bool on = live && r < p.M;
    const int64_t at = at0 + (int64_t)r * p.Fx;
    dy[i] = Elem<T>::to_f32(dx[i]);
    if (p.mask) dy[i] = Elem<T>::to_f32(Elem<T>::from_f32(on && p.mask[at] ? dy[i] * p.scale : 0.f));
    z[i] = on ? Elem<T>::load((const T*)p.Z + at) : 0.f;
  }
  if constexpr (KIND == FEW_ACT) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int r = ty + 8 * (i >> 1) + 16 * (i & 1);
      if (live && r < p.M) Elem<T>::store(out + at0 + (int64_t)r * p.Fx, dy[i] * act_grad(z[i], p.act, p.slope));
    }
  } else {
    const int k = b * p.Fx + (live ? c : p.Fx - 1);
    const float mean = p.save_mean[k], invstd = p.save_invstd[k], g = p.gamma[k], bt = p.beta[k];
    float xh[4], gr[4];
    float s1[2] = {0.f, 0.f}, s2[2] = {0.f, 0.f};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int r = ty + 8 * (i >> 1) + 16 * (i & 1);
      xh[i] = (z[i] - mean) * invstd;
      gr[i] = dy[i] * act_grad(fmaf(g, xh[i], bt), p.act, p.slope);
      if (r < p.M) {
        s1[i >> 1] += gr[i];
        s2[i >> 1] = fmaf(gr[i], xh[i], s2[i >> 1]);
      }
    }
    auto column_sum = [&](const float (&v)[2]) {
      __syncthreads();
      red[ty][col] = v[0];
      red[ty + 8][col] = v[1];
      __syncthreads();
      return lane_sum(red, col);
    };
    const float t1 = column_sum(s1), t2 = column_sum(s2);
    if (live && ty == 0) {
      p.dbeta[k] = t1;
      p.dgamma[k] = t2;
    }
    const float m = (float)p.M, mb = t1 / m, mg = t2 / m, sc = g * invstd;
    float s3[2] = {0.f, 0.f};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int r = ty + 8 * (i >> 1) + 16 * (i & 1);
      if (r >= p.M) continue;
      const T o = Elem<T>::from_f32(sc * (gr[i] - mb - xh[i] * mg));
      if (live) out[at0 + (int64_t)r * p.Fx] = o;
      s3[i >> 1] += Elem<T>::to_f32(o);
    }
    if (p.dx_sum) {                                      // uniform over the grid
      const float t3 = column_sum(s3);
      if (live && ty == 0) p.dx_sum[k] = t3;
    }
  }
}

bool al16(const void* q) { return reinterpret_cast<uintptr_t>(q) % 16 == 0; }
bool bn_act_ok(int act) { return act == HFTA_ACT_NONE || act == HFTA_ACT_RELU || act == HFTA_ACT_LEAKY; }
// rows of whole pieces; operand slices below 2 GiB; channels of all models counted in 31 bits
bool few_ok(int B, int M, int Fx, int Fy, int dtype) {
  const int q = dtype == HFTA_BF16 ? 8 : 4;
  return B > 0 && B <= 65535 && M > 0 && M <= FEW_ROWS && Fx > 0 && Fy > 0 && valid_dtype(dtype) && Fx % q == 0 && Fy % q == 0 &&
         (int64_t)Fx * Fy < (int64_t)1 << 29 && Fx < 1 << 24 && Fy < 1 << 24 &&
         (int64_t)B * Fx < (int64_t)1 << 31 && (int64_t)B * Fy < (int64_t)1 << 31;
}
// fp32: pieces of the reduction that the fp32 instruction takes in the split product too
bool few_fwd_ok(int B, int M, int Fx, int Fy, int dtype) {
  if (!few_ok(B, M, Fx, Fy, dtype)) return false;
  const int splits = linear_row_splits(B, M, Fx, Fy, dtype);
  if (dtype == HFTA_BF16) return Fx <= FewFwd<bf16_raw>::MAX_K && splits <= FewFwd<bf16_raw>::SPLITS;
  return splits <= FewFwd<float>::SPLITS && (Fx + splits - 1) / splits <= FEW_F32_EXACT_K;
}

// Whether a layer of such shapes is sooner in these launches than in the single operators.  A launch of few workgroups costs the wait
// for it; one of many costs what its workgroups do, and there the single operators' larger tiles read less.  us, single operators ->
// these, BatchNorm and dropout forward and backward, 32 rows a model:
//   bf16, 1024 -> 512    16 models 20 -> 12, 28 -> 20     32: 24 -> 18, 37 -> 33     64: 24 -> 36, 60 -> 59    256: 89 -> 155, 257 -> 285
//         512 -> 256     64: 20 -> 13, 32 -> 28     96: 26 -> 20, 40 -> 40    128: 19 -> 26, 45 -> 51    512: 58 -> 83, 170 -> 268
//   fp32, 64 -> 64       32: 13 -> 6, 17 -> 6    256: 13 -> 11, 20 -> 15 (without BatchNorm 12 -> 14)   512: 18 -> 21, 29 -> 34
//         28 -> 436      500: 51 -> 133, 47 -> 162
// The forward's time in bf16 goes with its workgroups times the k that a wavefront walks (one wavefront the whole reduction where it is
// not split), the backward's with its workgroups: six rounds of two a compute unit; in fp32 a compute unit holds one.  Both calls of a
// layer, 497 shapes of 1 to 622 models: 0.98 to 3.0 times as fast within these lines (2.2 at the median), 0.33 to 1.6 past them (0.90).
bool few_pays(int B, int M, int Fx, int Fy, int dtype) {
  const int64_t fwd = (int64_t)((Fy + 31) / 32) * B, splits = linear_row_splits(B, M, Fx, Fy, dtype);
  const int64_t bwd = (int64_t)((Fx + 31) / 32 + (Fx + DW_BM - 1) / DW_BM * ((Fy + DW_BN - 1) / DW_BN)) * B;
  if (dtype == HFTA_BF16) return fwd * ((Fx + splits - 1) / splits) <= 1 << 18 && bwd <= 3072;
  return fwd <= 512 && bwd <= 640;
}
// The forward alone against the split product and the sum of its parts, two launches.  bf16, 32 rows, 1024 -> 512: 8 models 12 -> 6 us,
// 24 18 -> 14, 48 22 -> 24; 53 models 776 -> 376 20 -> 22.  fp32, more pieces than wavefronts (1024 -> 512, 1 model 9.4 -> 12.3, 2 11.4 ->
// 12.6; 4, of 16 pieces, 11.7 -> 10.3).
bool few_ws_pays(int B, int Fx, int Fy, int dtype, int splits) {
  const int64_t fwd = (int64_t)((Fy + 31) / 32) * B;
  return dtype == HFTA_BF16 ? fwd * ((Fx + splits - 1) / splits) <= 3 << 16 : splits <= FWD_WAVES && fwd <= 512;
}

template <int KIND> int few_fwd_launch(int B, int dtype, FewFwdArgs a, hipStream_t st) {
  // 512 threads for the 32 columns x 16 row lanes, more where the reduction is cut finer
  const int waves = a.splits < 8 ? 8 : a.splits > FWD_WAVES ? FWD_WAVES : a.splits;
  const dim3 grid((unsigned)((a.Fy + 31) / 32), (unsigned)B), block(64 * waves);
  if (dtype == HFTA_BF16) hipLaunchKernelGGL((linear_few_fwd_kernel<bf16_raw, KIND>), grid, block, 0, st, a);
  else hipLaunchKernelGGL((linear_few_fwd_kernel<float, KIND>), grid, block, 0, st, a);
  return launch_status();
}

int few_fwd_args(FewFwdArgs& a, int B, int M, int Fx, int Fy, int dtype, const void* X, const void* W, const void* bias, void* Z) {
  if (B <= 0 || M <= 0 || Fx <= 0 || Fy <= 0 || !valid_dtype(dtype) || !X || !W || !Z) return HFTA_EINVAL;
  if (!few_fwd_ok(B, M, Fx, Fy, dtype) || !al16(X) || !al16(W)) return HFTA_EUNSUPPORTED;
  a = FewFwdArgs{};
  a.X = X; a.W = W; a.bias = bias; a.Z = Z;
  a.M = M; a.Fx = Fx; a.Fy = Fy; a.splits = linear_row_splits(B, M, Fx, Fy, dtype);
  return HFTA_OK;
}

template <int KIND> int few_bwd_launch(int B, int dtype, const FewBwdArgs& a, hipStream_t st) {
  const dim3 grid((unsigned)(a.dx_tiles + a.dw_m * ((a.Fy + DW_BN - 1) / DW_BN)), (unsigned)B);
  if (dtype == HFTA_BF16) hipLaunchKernelGGL((linear_few_bwd_kernel<bf16_raw, KIND>), grid, dim3(256), 0, st, a);
  else hipLaunchKernelGGL((linear_few_bwd_kernel<float, KIND>), grid, dim3(256), 0, st, a);
  return launch_status();
}

int few_bwd_args(FewBwdArgs& a, int B, int M, int Fx, int Fy, int dtype, const void* X, const void* W, const void* dY, void* dX, float* dW,
                 float* dbias) {
  if (B <= 0 || M <= 0 || Fx <= 0 || Fy <= 0 || !valid_dtype(dtype) || !X || !W || !dY || !dX || !dW) return HFTA_EINVAL;
  if (!few_ok(B, M, Fx, Fy, dtype) || !al16(X) || !al16(W) || !al16(dY)) return HFTA_EUNSUPPORTED;
  // the weight gradient is the fp32 instruction's: gemm_f32_launch takes it for all small tiles of so few rows, for large ones up to 16
  // (the shapes of the forward are far below those)
  if (dtype == HFTA_F32 && M > 16 && gemm_f32_big_tiles(Fx, Fy, B)) return HFTA_EUNSUPPORTED;
  a = FewBwdArgs{};
  a.X = X; a.W = W; a.dY = dY; a.dX = dX; a.dW = dW; a.dbias = dbias;
  a.M = M; a.Fx = Fx; a.Fy = Fy; a.dx_tiles = (Fx + 31) / 32; a.dw_m = (Fx + DW_BM - 1) / DW_BM;
  return HFTA_OK;
}

}  // namespace

namespace hfta {
// the split forward of a Linear (linear_row_splits > 1) in one launch, where that is sooner; HFTA_EUNSUPPORTED: not a shape, alignment
// or activation for it
int linear_few_fwd(int B, int M, int Fx, int Fy, int dtype, const void* X, const void* W, const void* bias, void* Y, int act, float slope,
                   hipStream_t st) {
  FewFwdArgs a;
  const int rc = few_fwd_args(a, B, M, Fx, Fy, dtype, X, W, bias, Y);
  if (rc != HFTA_OK) return rc;
  if (!bn_act_ok(act) || !few_ws_pays(B, Fx, Fy, dtype, a.splits)) return HFTA_EUNSUPPORTED;
  a.act = act; a.slope = slope;
  return few_fwd_launch<FEW_ACT>(B, dtype, a, st);
}
}

extern "C" {

int hfta_linear_few_supported(int B, int M, int Fx, int Fy, int dtype) {
  return few_fwd_ok(B, M, Fx, Fy, dtype) && few_pays(B, M, Fx, Fy, dtype) ? 1 : 0;
}

int hfta_linear_bn_fwd(int B, int M, int Fx, int Fy, int dtype, const void* X, const void* W, const void* bias, const float* gamma,
                       const float* beta, float eps, float momentum, float* running_mean, float* running_var, float* save_mean,
                       float* save_invstd, void* Z, void* Y, int act, float act_slope, const uint8_t* mask, float p, void* Yd, void* stream) {
  if (!gamma || !beta || !save_mean || !save_invstd || !Y || !(eps >= 0.f) || (running_mean == nullptr) != (running_var == nullptr) ||
      (mask == nullptr) != (Yd == nullptr) || (mask && (!(p >= 0.f) || !(p < 1.f))))
    return HFTA_EINVAL;
  FewFwdArgs a;
  const int rc = few_fwd_args(a, B, M, Fx, Fy, dtype, X, W, bias, Z);
  if (rc != HFTA_OK) return rc;
  if (!bn_act_ok(act)) return HFTA_EUNSUPPORTED;
  a.gamma = gamma; a.beta = beta; a.rm = running_mean; a.rv = running_var; a.save_mean = save_mean; a.save_invstd = save_invstd;
  a.Y = Y; a.mask = mask; a.Yd = Yd;
  a.eps = eps; a.momentum = momentum; a.act = act; a.slope = act_slope; a.scale = 1.f / (1.f - p);
  return few_fwd_launch<FEW_BN>(B, dtype, a, as_stream(stream));
}

int hfta_linear_xent(int B, int M, int Fx, int K, int dtype, const void* X, const void* W, const void* bias, void* logits,
                     const int32_t* labels, float* loss, void* dlogits, void* stream) {
  if (!labels || !loss || !dlogits) return HFTA_EINVAL;
  FewFwdArgs a;
  const int rc = few_fwd_args(a, B, M, Fx, K, dtype, X, W, bias, logits);
  if (rc != HFTA_OK) return rc;
  if (K > 32) return HFTA_EUNSUPPORTED;
  a.labels = labels; a.loss = loss; a.dlogits = dlogits;
  return few_fwd_launch<FEW_XENT>(B, dtype, a, as_stream(stream));
}

int hfta_linear_bwd_bn(int B, int M, int Fx, int Fy, int dtype, const void* X, const void* W, const void* dY, void* dX, float* dW,
                       float* dbias, const void* Z, const float* gamma, const float* beta, const float* save_mean,
                       const float* save_invstd, int act, float act_slope, const uint8_t* mask, float p, float* dgamma, float* dbeta,
                       float* dx_sum, void* stream) {
  if (Z ? (!gamma || !beta || !save_mean || !save_invstd || !dgamma || !dbeta || (mask && (!(p >= 0.f) || !(p < 1.f)))) : (mask || dx_sum))
    return HFTA_EINVAL;
  FewBwdArgs a;
  const int rc = few_bwd_args(a, B, M, Fx, Fy, dtype, X, W, dY, dX, dW, dbias);
  if (rc != HFTA_OK) return rc;
  if (!Z) return few_bwd_launch<FEW_PLAIN>(B, dtype, a, as_stream(stream));
  if (!bn_act_ok(act)) return HFTA_EUNSUPPORTED;
  a.Z = Z; a.gamma = gamma; a.beta = beta; a.save_mean = save_mean; a.save_invstd = save_invstd;
  a.mask = mask; a.dgamma = dgamma; a.dbeta = dbeta; a.dx_sum = dx_sum; a.slope = act_slope; a.act = act; a.scale = 1.f / (1.f - p);
  return few_bwd_launch<FEW_BN>(B, dtype, a, as_stream(stream));
}

int hfta_linear_bwd_act(int B, int M, int Fx, int Fy, int dtype, const void* X, const void* W, const void* dY, void* dX, float* dW,
                        float* dbias, const void* H, int act, float act_slope, const uint8_t* mask, float p, void* stream) {
  if (!H || (mask && (!(p >= 0.f) || !(p < 1.f)))) return HFTA_EINVAL;
  FewBwdArgs a;
  const int rc = few_bwd_args(a, B, M, Fx, Fy, dtype, X, W, dY, dX, dW, dbias);
  if (rc != HFTA_OK) return rc;
  if (!bn_act_ok(act)) return HFTA_EUNSUPPORTED;
  a.Z = H; a.mask = mask; a.slope = act_slope; a.act = act; a.scale = 1.f / (1.f - p);
  return few_bwd_launch<FEW_ACT>(B, dtype, a, as_stream(stream));
}

}  // extern "C"
