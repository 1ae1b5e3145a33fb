// BatchNorm + activation + max over the point axis as ONE operator, forward and backward.
//
// PointNet's global feature is max_l act(BN(z))[., l].  Fused, the activated tensor is never
// written and never read back: the forward streams z twice (statistics, then normalise-and-max)
// and writes only [B][Nb][C] values and indices; the backward needs z once, because the
// gradient arriving from the pool is non-zero at exactly one point per (sample, channel), so the
// two BatchNorm sums collapse to Nb gathered elements per channel.
//
// The forward is bit-identical to hfta_bn_fwd followed by hfta_maxpool_points (the maximum is
// taken over the activated values rounded to the storage type, lowest index on ties); the
// backward equals hfta_maxpool_points_bwd followed by hfta_bn_bwd up to fp32 summation order.
//
// One workgroup per channel (b, c); each wavefront owns whole rows (samples) in the second pass
// so that the argmax reduction stays inside a wave.
#include "bn_common.h"

using namespace hfta;

namespace {

struct BnPoolFwdArgs {
  const void* X; void* V; int32_t* idx;
  const float* gamma; const float* beta;
  float* running_mean; float* running_var; float* save_mean; float* save_invstd;
  int64_t xsb, xsn, xsc, vsb, vsn, vsc;
  int Nb, C, L, act;
  float eps, momentum, slope;
};

template <typename T, int VEC, int NT>
__global__ __launch_bounds__(NT) void bn_fwd_maxpool_kernel(BnPoolFwdArgs p) {
  constexpr int NW = NT / 64, UN = bn_unroll(VEC);
  __shared__ float sh[NW][2];
  const int c = blockIdx.x, b = blockIdx.y;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const T* x = reinterpret_cast<const T*>(p.X) + b * p.xsb + c * p.xsc;
  const int chunks = p.L / VEC;
  const float shift = Elem<T>::load(x);
  float s1 = 0.f, s2 = 0.f;
  // same element -> thread assignment and reduction order as the stand-alone BatchNorm forward,
  // so the statistics (and with them every activated value) come out bit-identical
  for (RowWalk w(chunks, NT); w.n < p.Nb;) {
    float v[UN][VEC];
    bool ok[UN];
#pragma unroll
    for (int u = 0; u < UN; ++u) {
      ok[u] = w.n < p.Nb;
      load_vec<T, VEC>(ok[u] ? x + w.n * p.xsn + w.ch * VEC : x, v[u]);
      w.step();
    }
#pragma unroll
    for (int u = 0; u < UN; ++u)
      if (ok[u]) {
#pragma unroll
        for (int e = 0; e < VEC; ++e) { const float d = v[u][e] - shift; s1 += d; s2 = fmaf(d, d, s2); }
      }
  }
  block_sum2<NW>(s1, s2, sh);
  const float m = (float)p.Nb * (float)p.L;
  const float dm = s1 / m;
  const float mean = shift + dm;
  float var = s2 / m - dm * dm;
  var = var < 0.f ? 0.f : var;
  const float invstd = 1.0f / sqrtf(var + p.eps);
  const int k = b * p.C + c;
  const float g = p.gamma[k], bt = p.beta[k];
  if (threadIdx.x == 0) {
    p.save_mean[k] = mean;
    p.save_invstd[k] = invstd;
    if (p.running_mean) {
      const float unb = m > 1.f ? var * (m / (m - 1.f)) : var;
      p.running_mean[k] = (1.f - p.momentum) * p.running_mean[k] + p.momentum * mean;
      p.running_var[k] = (1.f - p.momentum) * p.running_var[k] + p.momentum * unb;
    }
  }
  for (int n = wave; n < p.Nb; n += NW) {
    const T* row = x + n * p.xsn;
    float best = -INFINITY;
    int bi = 0x7fffffff;
    for (int c0 = lane; c0 < chunks; c0 += 64 * UN) {
      float v[UN][VEC];
#pragma unroll
      for (int u = 0; u < UN; ++u) load_vec<T, VEC>(row + min(c0 + 64 * u, chunks - 1) * VEC, v[u]);
#pragma unroll
      for (int u = 0; u < UN; ++u) {
        const int ch = c0 + 64 * u;
        if (ch < chunks) {
#pragma unroll
          for (int e = 0; e < VEC; ++e) {
            // the activated value exactly as hfta_bn_fwd would have stored it
            const float y = Elem<T>::to_f32(Elem<T>::from_f32(bn_act(fmaf(g, (v[u][e] - mean) * invstd, bt), p.act, p.slope)));
            if (y > best || bi == 0x7fffffff) { best = y; bi = ch * VEC + e; }
          }
        }
      }
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
      const float ov = __shfl_xor(best, o, 64);
      const int oi = __shfl_xor(bi, o, 64);
      if (oi != 0x7fffffff && (bi == 0x7fffffff || ov > best || (ov == best && oi < bi))) { best = ov; bi = oi; }
    }
    if (lane == 0) {
      const int64_t o = b * p.vsb + n * p.vsn + c * p.vsc;
      reinterpret_cast<T*>(p.V)[o] = Elem<T>::from_f32(best);
      p.idx[o] = bi;
    }
  }
}

// Normalise, activate, store AND take each row's maximum of the stored values: the pass that writes the activated tensor
// is the one that would be read again for the maximum (512 -> 2048 channels, 6 x 16 x 2500 points: 400 + 204 us apart,
// 404 here).  A wavefront per row; the maximum as hfta_maxpool_points takes it, lowest index on ties.
template <typename T>
__global__ __launch_bounds__(256) void bn_apply_maxpool_kernel(BnPoolFwdArgs p, T* Y, int64_t ysb, int64_t ysn, int64_t ysc, int64_t rows) {
  constexpr int U = 5;                                     // pieces in flight: a 2500-point row is two rounds
  const int lane = threadIdx.x & 63;
  const int64_t r = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (r >= rows) return;
  const int c = (int)(r % p.C);
  const int64_t bn = r / p.C;
  const int n = (int)(bn % p.Nb), b = (int)(bn / p.Nb), k = b * p.C + c;
  const T* x = reinterpret_cast<const T*>(p.X) + b * p.xsb + n * p.xsn + c * p.xsc;
  T* y = Y + b * ysb + n * ysn + c * ysc;
  const float mean = p.save_mean[k], invstd = p.save_invstd[k], g = p.gamma[k], bt = p.beta[k];
  const int chunks = p.L / 4;
  float best = -INFINITY;
  int bi = 0x7fffffff;
  for (int c0 = lane; c0 < chunks; c0 += 64 * U) {
    float v[U][4];
#pragma unroll
    for (int u = 0; u < U; ++u) load_vec<T, 4>(x + min(c0 + 64 * u, chunks - 1) * 4, v[u]);
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int ch = c0 + 64 * u;
      if (ch < chunks) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          v[u][e] = Elem<T>::to_f32(Elem<T>::from_f32(bn_act(fmaf(g, (v[u][e] - mean) * invstd, bt), p.act, p.slope)));
          if (v[u][e] > best || bi == 0x7fffffff) { best = v[u][e]; bi = ch * 4 + e; }
        }
        store_vec<T, 4>(y + ch * 4, v[u]);
      }
    }
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    const float ov = __shfl_xor(best, o, 64);
    const int oi = __shfl_xor(bi, o, 64);
    if (oi != 0x7fffffff && (bi == 0x7fffffff || ov > best || (ov == best && oi < bi))) { best = ov; bi = oi; }
  }
  if (lane == 0) {
    const int64_t o = b * p.vsb + n * p.vsn + c * p.vsc;
    reinterpret_cast<T*>(p.V)[o] = Elem<T>::from_f32(best);
    p.idx[o] = bi;
  }
}

// Statistics and pooled values from what the fp32 convolution's epilogue left per (sample, column tile, channel): sum, sum
// of squares about the tile's mean, extreme of z (largest, or smallest where gamma < 0) and where it is.  BatchNorm is
// monotone in z per channel and the activations taken here do not decrease, so the extreme's normalised value is the row's
// maximum; a row whose activated values are all equal (clipped, or gamma = 0) or no numbers has its maximum at point 0.  The 1.3 GB of z
// are not read (4 x 32 x 2500 points, 1024 channels: bn_fwd_maxpool_kernel 402 us, this 23 and the epilogue 122 more).
// 16 channels a workgroup: 16 lanes read 256 contiguous bytes of a part, 64 parts in flight.
// p.X == nullptr: z was not stored.  Then z at point 0, where it is asked for, is the product again, from `at0`; and the z that
// was pooled goes to at0.zhit, [B][Nb][C], for the backward.
struct PoolAt0 { const float* x; const float* w; const float* bias; int64_t xsb, xsn, xsc; int Ci; float* zhit; };
constexpr int PP_C = 16, PP_P = 64;
__global__ __launch_bounds__(PP_C * PP_P) void bn_pool_parts_kernel(BnPoolFwdArgs p, const float4* __restrict__ part, int tiles, int cols,
                                                                    PoolAt0 at0) {
  __shared__ double red[PP_P][PP_C][2];
  const int cl = threadIdx.x % PP_C, pl = threadIdx.x / PP_C;
  const int c = blockIdx.x * PP_C + cl, b = blockIdx.y, k = b * p.C + c;
  const bool live = c < p.C;
  const float4* pp = part + (int64_t)b * p.Nb * tiles * p.C + (live ? c : 0);
  const double full = 1.0 / cols, last = 1.0 / (p.L - (tiles - 1) * cols);
  double s1 = 0.0, s2 = 0.0;
#pragma unroll 4
  for (int i = pl; i < p.Nb * tiles; i += PP_P) {
    const float4 v = pp[(int64_t)i * p.C];
    s1 += (double)v.x;
    s2 += (double)v.y + (double)v.x * (double)v.x * ((i + 1) % tiles ? full : last);
  }
  red[pl][cl][0] = s1;
  red[pl][cl][1] = s2;
  __syncthreads();
  for (int h = PP_P / 2; h > 0; h >>= 1) {
    if (pl < h) {
      red[pl][cl][0] += red[pl + h][cl][0];
      red[pl][cl][1] += red[pl + h][cl][1];
    }
    __syncthreads();
  }
  if (!live) return;
  const double m = (double)p.Nb * (double)p.L, mz = red[0][cl][0] / m;
  double var = red[0][cl][1] / m - mz * mz;
  var = var < 0.0 ? 0.0 : var;
  const float mean = (float)mz, invstd = (float)(1.0 / sqrt(var + (double)p.eps));
  const float g = p.gamma[k], bt = p.beta[k];
  if (pl == 0) {
    p.save_mean[k] = mean;
    p.save_invstd[k] = invstd;
    if (p.running_mean) {
      const float unb = (float)(m > 1.0 ? var * (m / (m - 1.0)) : var);
      p.running_mean[k] = (1.f - p.momentum) * p.running_mean[k] + p.momentum * mean;
      p.running_var[k] = (1.f - p.momentum) * p.running_var[k] + p.momentum * unb;
    }
  }
  const bool clips = p.act == HFTA_ACT_RELU || (p.act == HFTA_ACT_LEAKY && p.slope == 0.f);
  for (int n = pl; n < p.Nb; n += PP_P) {
    float best = -INFINITY;
    int at = 0x7fffffff;
#pragma unroll 4
    for (int q = 0; q < tiles; ++q) {
      const float4 v = pp[(int64_t)(n * tiles + q) * p.C];
      if (v.z > best || at == 0x7fffffff) { best = v.z; at = __float_as_int(v.w); }
    }
    float z = g < 0.f ? -best : best;
    float pre = fmaf(g, (z - mean) * invstd, bt);
    const bool clipped = clips && !(pre > 0.f);
    if (g == 0.f || clipped || pre != pre) {
      at = 0;
      if (p.X) {
        z = reinterpret_cast<const float*>(p.X)[b * p.xsb + n * p.xsn + c * p.xsc];
        pre = fmaf(g, (z - mean) * invstd, bt);
        if (clipped && pre > 0.f) pre = 0.f;               // the row's maximum was not positive
      } else if (clipped && pre == pre) {
        pre = 0.f;                                         // its gradient is zero: any z of the row will do for the backward
      } else {
        const float* x = at0.x + b * at0.xsb + n * at0.xsn;
        const float* w = at0.w + (int64_t)k * at0.Ci;
        z = at0.bias ? at0.bias[k] : 0.f;
        for (int i = 0; i < at0.Ci; ++i) z = fmaf(w[i], x[i * at0.xsc], z);
        pre = fmaf(g, (z - mean) * invstd, bt);
        if (clipped && pre > 0.f) pre = 0.f;
      }
    }
    if (at0.zhit) at0.zhit[((int64_t)b * p.Nb + n) * p.C + c] = z;
    const int64_t o = b * p.vsb + n * p.vsn + c * p.vsc;
    reinterpret_cast<float*>(p.V)[o] = bn_act(pre, p.act, p.slope);
    p.idx[o] = at;
  }
}

struct BnPoolBwdArgs {
  const void* X; const void* dV; const int32_t* idx; void* dX;
  const float* gamma; const float* beta; const float* save_mean; const float* save_invstd;
  float* dgamma; float* dbeta; float* dx_sum;
  int64_t xsb, xsn, xsc, vsb, vsn, vsc, dxsb, dxsn, dxsc;
  int Nb, C, L, act;
  float slope;
};

template <typename T, int VEC, int NT>
__global__ __launch_bounds__(NT) void bn_bwd_maxpool_kernel(BnPoolBwdArgs p) {
  constexpr int NW = NT / 64, UN = bn_unroll(VEC);
  __shared__ float sh[NW][2];
  const int c = blockIdx.x, b = blockIdx.y, k = b * p.C + c;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const T* x = reinterpret_cast<const T*>(p.X) + b * p.xsb + c * p.xsc;
  const T* dv = reinterpret_cast<const T*>(p.dV) + b * p.vsb + c * p.vsc;
  const int32_t* ix = p.idx + b * p.vsb + c * p.vsc;
  T* dx = reinterpret_cast<T*>(p.dX) + b * p.dxsb + c * p.dxsc;
  const float mean = p.save_mean[k], invstd = p.save_invstd[k], g = p.gamma[k], bt = p.beta[k];
  // the incoming gradient is dV at the argmax point of each sample and zero elsewhere
  float s1 = 0.f, s2 = 0.f;
  for (int n = threadIdx.x; n < p.Nb; n += NT) {
    const int hit = min(max(ix[n * p.vsn], 0), p.L - 1);     // never address outside the row
    const float xh = (Elem<T>::load(x + n * p.xsn + hit) - mean) * invstd;
    const float gr = Elem<T>::load(dv + n * p.vsn) * act_grad(fmaf(g, xh, bt), p.act, p.slope);
    s1 += gr;
    s2 = fmaf(gr, xh, s2);
  }
  block_sum2<NW>(s1, s2, sh);
  if (threadIdx.x == 0) { p.dbeta[k] = s1; p.dgamma[k] = s2; }
  const float m = (float)p.Nb * (float)p.L;
  const float mb = s1 / m, mg = s2 / m, sc = g * invstd;
  const int chunks = p.L / VEC;
  float s3 = 0.f;
  for (int n = wave; n < p.Nb; n += NW) {
    const T* row = x + n * p.xsn;
    T* drow = dx + n * p.dxsn;
    const int hit = min(max(ix[n * p.vsn], 0), p.L - 1);
    const float gv = Elem<T>::load(dv + n * p.vsn);
    for (int c0 = lane; c0 < chunks; c0 += 64 * UN) {
      float v[UN][VEC];
#pragma unroll
      for (int u = 0; u < UN; ++u) load_vec<T, VEC>(row + min(c0 + 64 * u, chunks - 1) * VEC, v[u]);
#pragma unroll
      for (int u = 0; u < UN; ++u) {
        const int ch = c0 + 64 * u;
        if (ch < chunks) {
#pragma unroll
          for (int e = 0; e < VEC; ++e) {
            const float xh = (v[u][e] - mean) * invstd;
            float gr = 0.f;
            if (ch * VEC + e == hit) gr = gv * act_grad(fmaf(g, xh, bt), p.act, p.slope);
            v[u][e] = sc * (gr - mb - xh * mg);
            s3 += Elem<T>::to_f32(Elem<T>::from_f32(v[u][e]));
          }
          store_vec<T, VEC>(drow + ch * VEC, v[u]);
        }
      }
    }
  }
  if (p.dx_sum) {
    float dummy = 0.f;
    block_sum2<NW>(s3, dummy, sh);
    if (threadIdx.x == 0) p.dx_sum[k] = s3;
  }
}

constexpr int POOL_MIN_COLS = 128;                         // narrowest column tile that comes with sums

bool act_ok(int act) { return act == HFTA_ACT_NONE || act == HFTA_ACT_RELU || act == HFTA_ACT_LEAKY; }

}  // namespace

namespace hfta {
int conv1x1_fwd_pool_part(int B, int Nb, int Ci, int Co, int L, const void* X, const int64_t xs[4], const void* W, const void* bias,
                          void* Z, const int64_t zs[4], const float* gamma, float4* part, int* cols, hipStream_t st);
// the same product's partial sums for a tail that stores no output (conv_pool_f32_fwd.hip): 128-column tiles
size_t pool32_pack_bytes(int B, int Co);
int pool32_main(int B, int Nb, int Ci, int Co, int L, const float* X, const int64_t xs[4], const float* W, const float* bias,
                const float* gamma, float4* part, void* scratch, hipStream_t st);
// workspace of hfta_conv1x1_bn_maxpool_f32_fwd: the partial sums, then what that product wants
static size_t pool32_part_bytes(int B, int Nb, int Ci, int Co, int L) {
  return (hfta_conv1x1_bn_pool_fwd_workspace_bytes(B, Nb, Ci, Co, L, HFTA_F32) + 255) & ~(size_t)255;
}
size_t pool32_least_bytes(int B, int Nb, int Ci, int Co, int L);
size_t pool32_fwd_bytes(int B, int Nb, int Ci, int Co, int L) { return pool32_part_bytes(B, Nb, Ci, Co, L) + pool32_pack_bytes(B, Co); }
}

extern "C" {

size_t hfta_conv1x1_bn_pool_fwd_workspace_bytes(int B, int Nb, int Ci, int Co, int L, int dtype) {
  if (B <= 0 || Nb <= 0 || Ci <= 0 || Co <= 0 || L <= 0 || !valid_dtype(dtype)) return 0;
  if (dtype == HFTA_BF16) return hfta_conv1x1_bn_fwd_workspace_bytes(B, Nb, Ci, Co, L, dtype);
  return (size_t)B * Nb * ((L + POOL_MIN_COLS - 1) / POOL_MIN_COLS) * Co * sizeof(float4);
}

int hfta_conv1x1_bn_pool_fwd(int B, int Nb, int Ci, int Co, int L, int dtype, const void* X, const int64_t xs[4], const void* W,
                             const void* bias, const float* gamma, const float* beta, float eps, float momentum,
                             float* running_mean, float* running_var, float* save_mean, float* save_invstd, void* Z,
                             const int64_t zs[4], void* Y, const int64_t ys[4], void* V, int32_t* idx, const int64_t vs[3], int act,
                             float act_slope, void* workspace, size_t ws_bytes, void* stream) {
  if (B <= 0 || Nb <= 0 || Ci <= 0 || Co <= 0 || L <= 0 || !valid_dtype(dtype) || !X || !xs || !W || !gamma || !beta ||
      !save_mean || !save_invstd || !Z || !zs || (Y && !ys) || !V || !idx || !vs || !(eps >= 0.f))
    return HFTA_EINVAL;
  if ((running_mean == nullptr) != (running_var == nullptr)) return HFTA_EINVAL;
  if (!act_ok(act) || xs[3] != 1 || zs[3] != 1 || (Y && ys[3] != 1) || B > 65535) return HFTA_EUNSUPPORTED;
  hipStream_t st = as_stream(stream);
  BnPoolFwdArgs a{Z, V, idx, gamma, beta, running_mean, running_var, save_mean, save_invstd,
                  zs[0], zs[1], zs[2], vs[0], vs[1], vs[2], Nb, Co, L, act, eps, momentum, act_slope};
  if (Y) {                       // the activated tensor is wanted too: statistics, then one pass for both
    const bool pieces = bn_vec4_ok(Z, zs, L, dtype) && bn_vec4_ok(Y, ys, L, dtype);
    // Rows of partial pieces take that in two passes, and small ones are better off with one launch less, BatchNorm's own kernel
    // and the maximum: that, and here, in us: 64 channels on 2 x 4 x 129 points 13.8 15.4, 128 on 2 x 8 x 257 17.0 18.1, 256 on
    // 1 x 16 x 333 29.8 28.4, 2048 on 1 x 2 x 333 33.1 33.5, on 6 x 4 x 513 170 151, on 6 x 16 x 2499 3298 2654.
    if (!pieces && (int64_t)B * Nb * Co * L < (int64_t)1 << 20) {
      const int rc = hfta_conv1x1_bn_fwd(B, Nb, Ci, Co, L, dtype, X, xs, W, bias, gamma, beta, eps, momentum, running_mean, running_var,
                                         save_mean, save_invstd, Z, zs, Y, ys, act, act_slope, workspace, ws_bytes, stream);
      return rc != HFTA_OK ? rc : hfta_maxpool_points(B, Nb, Co, L, dtype, Y, ys, V, idx, vs, stream);
    }
    int rc = hfta_conv1x1_bn_fwd(B, Nb, Ci, Co, L, dtype, X, xs, W, bias, gamma, beta, eps, momentum, running_mean, running_var,
                                 save_mean, save_invstd, Z, zs, nullptr, nullptr, act, act_slope, workspace, ws_bytes, stream);
    if (rc != HFTA_OK) return rc;
    if (pieces) {
      const int64_t rows = (int64_t)B * Nb * Co;
      const dim3 grid((unsigned)((rows + 3) / 4));
      if (dtype == HFTA_BF16)
        hipLaunchKernelGGL(bn_apply_maxpool_kernel<bf16_raw>, grid, dim3(256), 0, st, a, (bf16_raw*)Y, ys[0], ys[1], ys[2], rows);
      else
        hipLaunchKernelGGL(bn_apply_maxpool_kernel<float>, grid, dim3(256), 0, st, a, (float*)Y, ys[0], ys[1], ys[2], rows);
      return launch_status();
    }
    rc = hfta_bn_apply_fwd(B, Nb, Co, L, dtype, Z, zs, gamma, beta, save_mean, save_invstd, Y, ys, act, act_slope, stream);
    return rc != HFTA_OK ? rc : hfta_maxpool_points(B, Nb, Co, L, dtype, Y, ys, V, idx, vs, stream);
  }
  // fp32: statistics and maxima from the convolution's epilogue; needs an activation that does not decrease
  if (dtype == HFTA_F32 && !(act == HFTA_ACT_LEAKY && !(act_slope >= 0.f)) && workspace &&
      ws_bytes >= hfta_conv1x1_bn_pool_fwd_workspace_bytes(B, Nb, Ci, Co, L, dtype) && reinterpret_cast<uintptr_t>(workspace) % 16 == 0 &&
      (int64_t)B * Nb <= 65535) {
    int cols = 0;
    const int rc = conv1x1_fwd_pool_part(B, Nb, Ci, Co, L, X, xs, W, bias, Z, zs, gamma, (float4*)workspace, &cols, st);
    if (rc != HFTA_OK) return rc;
    if (cols > 0) {
      hipLaunchKernelGGL(bn_pool_parts_kernel, dim3((unsigned)((Co + PP_C - 1) / PP_C), (unsigned)B), dim3(PP_C * PP_P), 0, st, a,
                         (const float4*)workspace, (L + cols - 1) / cols, cols, PoolAt0{});
      return launch_status();
    }
  } else {
    const int rc = hfta_conv1x1_fwd(B, Nb, Ci, Co, L, dtype, X, xs, W, bias, Z, zs, HFTA_ACT_NONE, 0.f, stream);
    if (rc != HFTA_OK) return rc;
  }
  return hfta_bn_fwd_maxpool(B, Nb, Co, L, dtype, Z, zs, gamma, beta, eps, momentum, running_mean, running_var, save_mean,
                             save_invstd, V, idx, vs, act, act_slope, stream);
}

// The same in fp32 without Z (backward: conv_pool_f32.hip)
int hfta_conv1x1_bn_maxpool_f32_fwd(int B, int Nb, int Ci, int Co, int L, const float* X, const int64_t xs[4], const float* W,
                                    const float* bias, const float* gamma, const float* beta, float eps, float momentum,
                                    float* running_mean, float* running_var, float* save_mean, float* save_invstd, float* V,
                                    int32_t* idx, const int64_t vs[3], float* zhit, int act, float act_slope, void* workspace,
                                    size_t ws_bytes, void* stream) {
  if (B <= 0 || Nb <= 0 || Ci <= 0 || Co <= 0 || L <= 0 || !X || !xs || !W || !gamma || !beta || !save_mean || !save_invstd || !V ||
      !idx || !vs || !zhit || !(eps >= 0.f))
    return HFTA_EINVAL;
  if ((running_mean == nullptr) != (running_var == nullptr)) return HFTA_EINVAL;
  if (!(act == HFTA_ACT_NONE || act == HFTA_ACT_RELU || (act == HFTA_ACT_LEAKY && act_slope >= 0.f))) return HFTA_EUNSUPPORTED;
  const size_t need = pool32_least_bytes(B, Nb, Ci, Co, L);
  if (xs[3] != 1 || need == 0) return HFTA_EUNSUPPORTED;
  if (!workspace || reinterpret_cast<uintptr_t>(workspace) % 256 != 0 ||
      ws_bytes < need)
    return HFTA_EWORKSPACE;
  hipStream_t st = as_stream(stream);
  BnPoolFwdArgs a{nullptr, V, idx, gamma, beta, running_mean, running_var, save_mean, save_invstd,
                  0, 0, 0, vs[0], vs[1], vs[2], Nb, Co, L, act, eps, momentum, act_slope};
  const int64_t zs[4] = {(int64_t)Co * L, (int64_t)B * Co * L, L, 1};
  int cols = POOL_MIN_COLS;
  int rc = HFTA_EUNSUPPORTED;
  if (ws_bytes >= pool32_fwd_bytes(B, Nb, Ci, Co, L))
    rc = pool32_main(B, Nb, Ci, Co, L, X, xs, W, bias, gamma, (float4*)workspace, (char*)workspace + pool32_part_bytes(B, Nb, Ci, Co, L), st);
  if (rc == HFTA_EUNSUPPORTED) rc = conv1x1_fwd_pool_part(B, Nb, Ci, Co, L, X, xs, W, bias, nullptr, zs, gamma, (float4*)workspace, &cols, st);
  if (rc != HFTA_OK) return rc;
  if (cols <= 0) return HFTA_EUNSUPPORTED;
  hipLaunchKernelGGL(bn_pool_parts_kernel, dim3((unsigned)((Co + PP_C - 1) / PP_C), (unsigned)B), dim3(PP_C * PP_P), 0, st, a,
                     (const float4*)workspace, (L + cols - 1) / cols, cols,
                     PoolAt0{X, W, bias, xs[0], xs[1], xs[2], Ci, zhit});
  return launch_status();
}

int hfta_bn_fwd_maxpool(int B, int Nb, int C, int L, int dtype, const void* X, const int64_t xs[4], const float* gamma,
                        const float* beta, float eps, float momentum, float* running_mean, float* running_var,
                        float* save_mean, float* save_invstd, void* V, int32_t* idx, const int64_t vs[3], int act,
                        float act_slope, void* stream) {
  if (B <= 0 || Nb <= 0 || C <= 0 || L <= 0 || !valid_dtype(dtype) || !X || !xs || !gamma || !beta || !save_mean ||
      !save_invstd || !V || !idx || !vs || !(eps >= 0.f))
    return HFTA_EINVAL;
  if ((running_mean == nullptr) != (running_var == nullptr)) return HFTA_EINVAL;
  if (!act_ok(act) || xs[3] != 1 || B > 65535) return HFTA_EUNSUPPORTED;
  BnPoolFwdArgs a{X, V, idx, gamma, beta, running_mean, running_var, save_mean, save_invstd,
                  xs[0], xs[1], xs[2], vs[0], vs[1], vs[2], Nb, C, L, act, eps, momentum, act_slope};
  dim3 grid((unsigned)C, (unsigned)B);
  hipStream_t st = as_stream(stream);
  const bool v4 = bn_vec4_ok(X, xs, L, dtype);
  const bool big = bn_wide_block((int64_t)Nb * L * dtype_size(dtype));
#define HFTA_LAUNCH(T, V_) \
  do { if (big) hipLaunchKernelGGL((bn_fwd_maxpool_kernel<T, V_, 1024>), grid, dim3(1024), 0, st, a); \
       else hipLaunchKernelGGL((bn_fwd_maxpool_kernel<T, V_, 256>), grid, dim3(256), 0, st, a); } while (0)
  if (dtype == HFTA_BF16) { if (v4) HFTA_LAUNCH(bf16_raw, 4); else HFTA_LAUNCH(bf16_raw, 1); }
  else { if (v4) HFTA_LAUNCH(float, 4); else HFTA_LAUNCH(float, 1); }
#undef HFTA_LAUNCH
  return launch_status();
}

int hfta_bn_bwd_maxpool(int B, int Nb, int C, int L, int dtype, const void* X, const int64_t xs[4], const void* dV,
                        const int32_t* idx, const int64_t vs[3], const float* gamma, const float* beta,
                        const float* save_mean, const float* save_invstd, void* dX, const int64_t dxs[4],
                        float* dgamma, float* dbeta, float* dx_sum, int act, float act_slope, void* stream) {
  if (B <= 0 || Nb <= 0 || C <= 0 || L <= 0 || !valid_dtype(dtype) || !X || !xs || !dV || !idx || !vs || !gamma || !beta ||
      !save_mean || !save_invstd || !dX || !dxs || !dgamma || !dbeta)
    return HFTA_EINVAL;
  if (!act_ok(act) || xs[3] != 1 || dxs[3] != 1 || B > 65535) return HFTA_EUNSUPPORTED;
  BnPoolBwdArgs a{X, dV, idx, dX, gamma, beta, save_mean, save_invstd, dgamma, dbeta, dx_sum,
                  xs[0], xs[1], xs[2], vs[0], vs[1], vs[2], dxs[0], dxs[1], dxs[2], Nb, C, L, act, act_slope};
  dim3 grid((unsigned)C, (unsigned)B);
  hipStream_t st = as_stream(stream);
  const bool v4 = bn_vec4_ok(X, xs, L, dtype) && bn_vec4_ok(dX, dxs, L, dtype);
  const bool big = bn_wide_block((int64_t)Nb * L * dtype_size(dtype));
#define HFTA_LAUNCH(T, V_) \
  do { if (big) hipLaunchKernelGGL((bn_bwd_maxpool_kernel<T, V_, 1024>), grid, dim3(1024), 0, st, a); \
       else hipLaunchKernelGGL((bn_bwd_maxpool_kernel<T, V_, 256>), grid, dim3(256), 0, st, a); } while (0)
  if (dtype == HFTA_BF16) { if (v4) HFTA_LAUNCH(bf16_raw, 4); else HFTA_LAUNCH(bf16_raw, 1); }
  else { if (v4) HFTA_LAUNCH(float, 4); else HFTA_LAUNCH(float, 1); }
#undef HFTA_LAUNCH
  return launch_status();
}

}  // extern "C"
