// Linear layers of few rows with the operators that stand beside them, bf16: the fully connected head of a point-cloud model.
//
// A head of three layers on 32 rows a model ran as 26 launches (split products, their sums, BatchNorm, dropout, cross-entropy,
// and the way back), each as long as a launch that waits for the one before it takes: 4.5-10 us, 134 us of a step of 8 models
// whose weights are 10 MB.  With at most 32 rows a column of a layer's output is one column of one matrix-instruction tile, so
// everything that works by columns -- BatchNorm over the rows, its activation, the dropout behind it, and all of it backwards --
// is done by the workgroup that has the product in hand: six launches, 50 us of that step (1376 -> 1310), and on 3 models of 13
// clouds 114 -> 40 us (411 -> 351 a step).
//
// Bound: the wait for one launch, one load of the operands (all of a workgroup's in flight at once) and the chain of the matrix
// instructions and the row sums behind them.  Hence 32-column tiles, as many workgroups as that gives, and the forward's
// reduction cut over the wavefronts of a workgroup in the pieces that the split product cuts it in.
//
// The bits are those of the single operators: the same split of the reduction added in the same order, BatchNorm's sums over 16
// row lanes, every stored tensor rounded where it was.  (The heads of the transform sub-networks turn a last-bit difference into
// percents a few layers on.)
#include "gemm_pf.h"
#include "bn_common.h"

namespace hfta {
int linear_row_splits(int B, int M, int Fx, int Fy, int dtype);
}

using namespace hfta;

namespace {

constexpr int FEW_ROWS = 32;                             // one matrix-instruction tile
constexpr int FEW_LANES = 16;                            // row lanes of BatchNorm's sums (bn_fwd_linear_kernel)
constexpr int FWD_LDS = 76 * 1024;                       // W's columns: 64 bytes per k; two workgroups a compute unit
constexpr int FWD_MAX_K = FWD_LDS / 64;
constexpr int FWD_MAX_SPLITS = 16;                       // wavefronts of a workgroup
constexpr int PART_PITCH = 36;                           // floats: 32 columns and a pad
static_assert(FWD_MAX_SPLITS * FEW_ROWS * PART_PITCH * 4 <= FWD_LDS, "the partial sums lie over the operand");

struct FewFwdArgs {
  const bf16_raw* X; const bf16_raw* W; const bf16_raw* bias; bf16_raw* Z;
  int M, Fx, Fy, splits;
  const float* gamma; const float* beta; float* rm; float* rv; float* save_mean; float* save_invstd; bf16_raw* Y;
  const uint8_t* mask; bf16_raw* Yd;
  float eps, momentum, slope, scale;
  int act;
  const int32_t* labels; float* loss; bf16_raw* dlogits;
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

// Z = X W + bias for 32 columns of one model, then
//   XENT == false  BatchNorm over the rows, activation, dropout (mask given)
//   XENT == true   softmax cross-entropy over the columns (at most 32: one workgroup holds them all)
// Wavefront w < splits takes the k-tiles that split w of the split product takes (linear_fwd_splits).
template <bool XENT>
__global__ __launch_bounds__(64 * FWD_MAX_SPLITS) void linear_few_fwd_kernel(FewFwdArgs p) {
  __shared__ __attribute__((aligned(16))) unsigned char smem[FWD_LDS];
  __shared__ float red[FEW_LANES][FEW_ROWS];
  const int t = threadIdx.x, lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const int n0 = blockIdx.x * 32, b = blockIdx.y;
  const int tt = (p.Fx + 31) / 32;                       // k-tiles of 32
  f32x16_t acc;
#pragma unroll
  for (int v = 0; v < 16; ++v) acc[v] = 0.f;
  if (wave < p.splits) {
    const int t0 = tt * wave / p.splits, t1 = tt * (wave + 1) / p.splits;
    const __amdgpu_buffer_rsrc_t rx = pf_rsrc(p.X + (int64_t)b * p.M * p.Fx, (uint32_t)p.M * p.Fx * 2u);
    const __amdgpu_buffer_rsrc_t rw = pf_rsrc(p.W + (int64_t)b * p.Fx * p.Fy, (uint32_t)p.Fx * p.Fy * 2u);
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
  __syncthreads();
  float* part = reinterpret_cast<float*>(smem);
  if (wave < p.splits) {                                 // lane l holds row l % 32, columns 8q + 4(l / 32) .. + 3
#pragma unroll
    for (int q = 0; q < 4; ++q)
      *reinterpret_cast<float4*>(part + (wave * FEW_ROWS + (lane & 31)) * PART_PITCH + 8 * q + 4 * (lane >> 5)) =
          make_float4(acc[4 * q], acc[4 * q + 1], acc[4 * q + 2], acc[4 * q + 3]);
  }
  __syncthreads();
  const int col = t & 31, ty = (t >> 5) & (FEW_LANES - 1), c = n0 + col;
  const bool mine = t < 32 * FEW_LANES, live = mine && c < p.Fy;
  const float bias = p.bias && live ? bf16_to_f32(p.bias[(int64_t)b * p.Fy + c]) : 0.f;
  float z[2] = {0.f, 0.f};                               // rows ty and ty + 16, as stored
  bf16_raw* zrow = p.Z + ((int64_t)b * p.M) * p.Fy + c;
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const int r = ty + FEW_LANES * h;
    float s = 0.f;
    for (int k = 0; k < p.splits; ++k) s += part[(k * FEW_ROWS + r) * PART_PITCH + col];
    if (p.bias) s += bias;
    const bf16_raw o = f32_to_bf16(s);
    z[h] = bf16_to_f32(o);
    if (live && r < p.M) zrow[(int64_t)r * p.Fy] = o;
  }
  if constexpr (!XENT) {
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
      const bf16_raw y = f32_to_bf16(bn_act(fmaf(g, (z[h] - mean) * invstd, bt), p.act, p.slope));
      p.Y[i] = y;
      if (p.mask) p.Yd[i] = f32_to_bf16(p.mask[i] ? bf16_to_f32(y) * p.scale : 0.f);
    }
  } else {
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
      bf16_raw* dz = p.dlogits + ((int64_t)b * p.M + lane) * K;
      const int lab = p.labels[(int64_t)b * p.M + lane];
      float mx = -INFINITY;
      for (int k = 0; k < K; ++k) mx = fmaxf(mx, zr[k]);
      float se = 0.f;
      for (int k = 0; k < K; ++k) se += expf(zr[k] - mx);
      const float lse = mx + logf(se);
      // a label past the classes is read where the stored form reads it
      a += lse - (lab >= 0 && lab < K ? zr[lab] : bf16_to_f32(p.Z[((int64_t)b * p.M + lane) * K + lab]));
      for (int k = 0; k < K; ++k) {
        const float pk = expf(zr[k] - lse);
        dz[k] = f32_to_bf16((pk - (k == lab ? 1.f : 0.f)) * invR);
      }
    }
    const float s = wave_sum(a);
    if (lane == 0) p.loss[b] = s * invR;
  }
}

constexpr int BWD_K = 512;                               // k of dX's product in LDS at a time
constexpr int BWD_PITCH = BWD_K * 2 + 16;
constexpr int DW_BM = 128, DW_BN = 64, DW_XP = DW_BM * 2 + 64, DW_YP = DW_BN * 2 + 64;
static_assert(FEW_ROWS * (DW_XP + DW_YP) <= 2 * FEW_ROWS * BWD_PITCH, "the weight gradient's operands");

struct FewBwdArgs {
  const bf16_raw* X; const bf16_raw* W; const bf16_raw* dY; bf16_raw* dX; float* dW; float* dbias;
  int M, Fx, Fy, dx_tiles, dw_m;
  const bf16_raw* Z; const float* gamma; const float* beta; const float* save_mean; const float* save_invstd;
  const uint8_t* mask; float* dgamma; float* dbeta; float* dx_sum;
  float slope, scale;
  int act;
};

// Both gradients of one Linear.  Workgroups below dx_tiles take 32 columns of dX = dY W^T over the whole reduction and, with BN,
// carry them on through the dropout, activation and BatchNorm of the layer below (Z: what that BatchNorm normalised); the others
// 128 x 64 of dW = X^T dY, the first of them per column block the column sums of dY.
template <bool BN>
__global__ __launch_bounds__(256) void linear_few_bwd_kernel(FewBwdArgs p) {
  __shared__ __attribute__((aligned(16))) unsigned char smem[2 * FEW_ROWS * BWD_PITCH];
  __shared__ float red[FEW_LANES][FEW_ROWS];
  const int t = threadIdx.x, lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const int b = blockIdx.y;
  const __amdgpu_buffer_rsrc_t ry = pf_rsrc(p.dY + (int64_t)b * p.M * p.Fy, (uint32_t)p.M * p.Fy * 2u);
  f32x16_t acc[2];
#pragma unroll
  for (int j = 0; j < 2; ++j)
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[j][v] = 0.f;

  if ((int)blockIdx.x >= p.dx_tiles) {                   // ---- dW
    const int q = (int)blockIdx.x - p.dx_tiles, m0 = (q % p.dw_m) * DW_BM, n0 = (q / p.dw_m) * DW_BN;
    const __amdgpu_buffer_rsrc_t rx = pf_rsrc(p.X + (int64_t)b * p.M * p.Fx, (uint32_t)p.M * p.Fx * 2u);
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
    // lane l holds column l % 32 and rows 8(v / 4) + 4(l / 32) + v % 4: whole 128-byte row segments per store
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
      for (int r = slice; r < p.M; r += 4) s += bf16_to_f32(*reinterpret_cast<const bf16_raw*>(ys + r * DW_YP + c * 2));
      sl[slice][c] = s;
      __syncthreads();
      if (slice == 0 && n0 + c < p.Fy) p.dbias[(int64_t)b * p.Fy + n0 + c] = (sl[0][c] + sl[1][c]) + (sl[2][c] + sl[3][c]);
    }
    return;
  }

  // ---- dX: all of a chunk's loads in flight, the chain of matrix instructions on the first wavefront
  const int f0 = blockIdx.x * 32;
  const __amdgpu_buffer_rsrc_t rw = pf_rsrc(p.W + (int64_t)b * p.Fx * p.Fy, (uint32_t)p.Fx * p.Fy * 2u);
  unsigned char* ds = smem;
  unsigned char* ws = smem + FEW_ROWS * BWD_PITCH;
  for (int k0 = 0; k0 < p.Fy; k0 += BWD_K) {
    const int kc = min(BWD_K, p.Fy - k0), ppr = (kc + 15) / 16 * 2, steps = ppr / 2;   // 16-byte pieces of a row
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
      const int e = t + 256 * i, r = e / ppr, at = r * BWD_PITCH + (e - r * ppr) * 16;
      if (r < FEW_ROWS) {
        *reinterpret_cast<uint4*>(ds + at) = d[i];
        *reinterpret_cast<uint4*>(ws + at) = w[i];
      }
    }
    __syncthreads();
    if (wave == 0) {
      const int at = (lane & 31) * BWD_PITCH + (lane >> 5) * 16;
#pragma unroll 8
      for (int s = 0; s < steps; ++s)
        acc[0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(*reinterpret_cast<const bf16x8_t*>(ws + at + s * 32),
                                                         *reinterpret_cast<const bf16x8_t*>(ds + at + s * 32), acc[0], 0, 0, 0);
    }
  }
  __syncthreads();
  float* tile = reinterpret_cast<float*>(smem);          // [32 rows][32 columns]
  if (wave == 0) {
#pragma unroll
    for (int q = 0; q < 4; ++q)
      *reinterpret_cast<float4*>(tile + (lane & 31) * PART_PITCH + 8 * q + 4 * (lane >> 5)) =
          make_float4(acc[0][4 * q], acc[0][4 * q + 1], acc[0][4 * q + 2], acc[0][4 * q + 3]);
  }
  __syncthreads();
  const int col = t & 31, ty = t >> 5, c = f0 + col;     // row lanes ty and ty + 8
  const bool live = c < p.Fx;
  const int64_t at0 = (int64_t)b * p.M * p.Fx + c;
  bf16_raw dx[4];                                        // rows ty, ty + 16 (lane ty), ty + 8, ty + 24 (lane ty + 8)
#pragma unroll
  for (int i = 0; i < 4; ++i) dx[i] = f32_to_bf16(tile[(ty + 8 * (i >> 1) + 16 * (i & 1)) * PART_PITCH + col]);
  if constexpr (!BN) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int r = ty + 8 * (i >> 1) + 16 * (i & 1);
      if (live && r < p.M) p.dX[at0 + (int64_t)r * p.Fx] = dx[i];
    }
  } else {
    const int k = b * p.Fx + (live ? c : p.Fx - 1);
    const float mean = p.save_mean[k], invstd = p.save_invstd[k], g = p.gamma[k], bt = p.beta[k];
    float xh[4], gr[4];
    float s1[2] = {0.f, 0.f}, s2[2] = {0.f, 0.f};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int r = ty + 8 * (i >> 1) + 16 * (i & 1);
      const bool on = live && r < p.M;
      const int64_t at = at0 + (int64_t)r * p.Fx;
      float dy = bf16_to_f32(dx[i]);
      if (p.mask) dy = bf16_to_f32(f32_to_bf16(on && p.mask[at] ? dy * p.scale : 0.f));
      xh[i] = ((on ? bf16_to_f32(p.Z[at]) : 0.f) - mean) * invstd;
      gr[i] = dy * act_grad(fmaf(g, xh[i], bt), p.act, p.slope);
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
      const bf16_raw o = f32_to_bf16(sc * (gr[i] - mb - xh[i] * mg));
      if (live) p.dX[at0 + (int64_t)r * p.Fx] = o;
      s3[i >> 1] += bf16_to_f32(o);
    }
    if (p.dx_sum) {                                      // uniform over the grid
      const float t3 = column_sum(s3);
      if (live && ty == 0) p.dx_sum[k] = t3;
    }
  }
}

bool al16(const void* q) { return reinterpret_cast<uintptr_t>(q) % 16 == 0; }
bool bn_act_ok(int act) { return act == HFTA_ACT_NONE || act == HFTA_ACT_RELU || act == HFTA_ACT_LEAKY; }
bool few_ok(int B, int M, int Fx, int Fy, int dtype) {
  return B > 0 && B <= 65535 && M > 0 && M <= FEW_ROWS && Fx > 0 && Fy > 0 && dtype == HFTA_BF16 && Fx % 8 == 0 && Fy % 8 == 0 &&
         (int64_t)Fx * Fy < (int64_t)1 << 30;            // operand slices below 2 GiB
}

}  // namespace

extern "C" {

int hfta_linear_few_supported(int B, int M, int Fx, int Fy, int dtype) {
  return few_ok(B, M, Fx, Fy, dtype) && Fx <= FWD_MAX_K && linear_row_splits(B, M, Fx, Fy, dtype) <= FWD_MAX_SPLITS ? 1 : 0;
}

static int few_fwd_args(FewFwdArgs& a, int B, int M, int Fx, int Fy, int dtype, const void* X, const void* W, const void* bias, void* Z) {
  if (B <= 0 || M <= 0 || Fx <= 0 || Fy <= 0 || !valid_dtype(dtype) || !X || !W || !Z) return HFTA_EINVAL;
  if (!hfta_linear_few_supported(B, M, Fx, Fy, dtype) || !al16(X) || !al16(W)) return HFTA_EUNSUPPORTED;
  a = FewFwdArgs{};
  a.X = (const bf16_raw*)X; a.W = (const bf16_raw*)W; a.bias = (const bf16_raw*)bias; a.Z = (bf16_raw*)Z;
  a.M = M; a.Fx = Fx; a.Fy = Fy; a.splits = linear_row_splits(B, M, Fx, Fy, dtype);
  return HFTA_OK;
}
// 512 threads for the 32 columns x 16 row lanes, more where the reduction is cut finer
static int few_fwd_threads(int splits) { return 64 * (splits < 8 ? 8 : splits); }

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
  a.Y = (bf16_raw*)Y; a.mask = mask; a.Yd = (bf16_raw*)Yd;
  a.eps = eps; a.momentum = momentum; a.act = act; a.slope = act_slope; a.scale = 1.f / (1.f - p);
  hipLaunchKernelGGL(linear_few_fwd_kernel<false>, dim3((unsigned)((Fy + 31) / 32), (unsigned)B), dim3(few_fwd_threads(a.splits)), 0,
                     as_stream(stream), a);
  return launch_status();
}

int hfta_linear_xent(int B, int M, int Fx, int K, int dtype, const void* X, const void* W, const void* bias, void* logits,
                     const int32_t* labels, float* loss, void* dlogits, void* stream) {
  if (!labels || !loss || !dlogits) return HFTA_EINVAL;
  FewFwdArgs a;
  const int rc = few_fwd_args(a, B, M, Fx, K, dtype, X, W, bias, logits);
  if (rc != HFTA_OK) return rc;
  if (K > 32) return HFTA_EUNSUPPORTED;
  a.labels = labels; a.loss = loss; a.dlogits = (bf16_raw*)dlogits;
  hipLaunchKernelGGL(linear_few_fwd_kernel<true>, dim3(1, (unsigned)B), dim3(few_fwd_threads(a.splits)), 0, as_stream(stream), a);
  return launch_status();
}

int hfta_linear_bwd_bn(int B, int M, int Fx, int Fy, int dtype, const void* X, const void* W, const void* dY, void* dX, float* dW,
                       float* dbias, const void* Z, const float* gamma, const float* beta, const float* save_mean,
                       const float* save_invstd, int act, float act_slope, const uint8_t* mask, float p, float* dgamma, float* dbeta,
                       float* dx_sum, void* stream) {
  if (B <= 0 || M <= 0 || Fx <= 0 || Fy <= 0 || !valid_dtype(dtype) || !X || !W || !dY || !dX || !dW) return HFTA_EINVAL;
  if (Z ? (!gamma || !beta || !save_mean || !save_invstd || !dgamma || !dbeta || (mask && (!(p >= 0.f) || !(p < 1.f)))) : (mask || dx_sum))
    return HFTA_EINVAL;
  if (!few_ok(B, M, Fx, Fy, dtype) || !al16(X) || !al16(W) || !al16(dY) || (Z && !bn_act_ok(act))) return HFTA_EUNSUPPORTED;
  FewBwdArgs a{};
  a.X = (const bf16_raw*)X; a.W = (const bf16_raw*)W; a.dY = (const bf16_raw*)dY; a.dX = (bf16_raw*)dX; a.dW = dW; a.dbias = dbias;
  a.M = M; a.Fx = Fx; a.Fy = Fy; a.dx_tiles = (Fx + 31) / 32; a.dw_m = (Fx + DW_BM - 1) / DW_BM;
  a.Z = (const bf16_raw*)Z; a.gamma = gamma; a.beta = beta; a.save_mean = save_mean; a.save_invstd = save_invstd;
  a.mask = mask; a.dgamma = dgamma; a.dbeta = dbeta; a.dx_sum = dx_sum; a.slope = act_slope; a.act = act; a.scale = 1.f / (1.f - p);
  const dim3 grid((unsigned)(a.dx_tiles + a.dw_m * ((Fy + DW_BN - 1) / DW_BN)), (unsigned)B);
  if (Z) hipLaunchKernelGGL(linear_few_bwd_kernel<true>, grid, dim3(256), 0, as_stream(stream), a);
  else hipLaunchKernelGGL(linear_few_bwd_kernel<false>, grid, dim3(256), 0, as_stream(stream), a);
  return launch_status();
}

}  // extern "C"
