// Fused Adam: one coalesced pass over the parameter arena [B][P] of all models.
//
// grid.y is the model index, so a workgroup only ever touches one model: its
// five hyper-parameters are read once from the device arrays and the two bias
// corrections 1 - beta^t are formed once per workgroup in double precision
// (1 - 0.999^t loses most of its bits in fp32 for small t), then broadcast
// through LDS.  Each thread updates four consecutive parameters with 16-byte
// accesses.  HBM-bound: reads theta, g, m, v and writes theta, m, v (+ the bf16
// copy the GEMMs read).
#include <algorithm>
#include "common.h"

using namespace hfta;

namespace {

struct AdamArgs {
  float* theta; const void* grad; float* m; float* v; bf16_raw* lowp;
  const float* lr; const float* beta1; const float* beta2; const float* eps; const float* wd;
  int64_t P;
  int t, decoupled;
};

// The state passes through once a step: non-temporal, so that it does not push what the next forward reads -- the bf16 weights
// written here, the batch -- out of the Infinity Cache.  Steps, us: residual MLP 10514 -> 10415, its small sweep 612 -> 604, language
// model 1286 -> 1266, transforms 3898 -> 3863, small GAN 1242 -> 1223, classification 1384 -> 1374.
template <bool NT> __device__ __forceinline__ float4 adam_ld(const float* p) {
  typedef float f4v __attribute__((ext_vector_type(4)));
  const f4v* q = reinterpret_cast<const f4v*>(p);
  const f4v v = NT ? __builtin_nontemporal_load(q) : *q;
  return make_float4(v.x, v.y, v.z, v.w);
}
template <bool NT> __device__ __forceinline__ void adam_st(float* p, float4 a) {
  typedef float f4v __attribute__((ext_vector_type(4)));
  const f4v v = {a.x, a.y, a.z, a.w};
  if (NT) __builtin_nontemporal_store(v, reinterpret_cast<f4v*>(p));
  else *reinterpret_cast<f4v*>(p) = v;
}
// from 1.5 M parameters, 18 MB in three arrays: 0.8 M lose by it (185.2 -> 186.7 us a step), 2.4 M gain (422.6 -> 418.6)
constexpr int64_t ADAM_NT_MIN = (int64_t)3 << 19;

struct AdamHp { float lr, b1, b2, eps, wd, inv_bc1, inv_bc2; };

__device__ __forceinline__ void adam_one(float& th, float g, float& m, float& v, const AdamHp& h, int decoupled) {
  if (decoupled) th = th * (1.f - h.lr * h.wd);
  else g = fmaf(h.wd, th, g);
  m = h.b1 * m + (1.f - h.b1) * g;
  v = h.b2 * v + (1.f - h.b2) * (g * g);
  const float mhat = m * h.inv_bc1;
  const float vhat = v * h.inv_bc2;
  th = th - h.lr * mhat / (sqrtf(vhat) + h.eps);
}

template <typename G, bool VEC4>
__global__ __launch_bounds__(256) void adam_kernel(AdamArgs p) {
  __shared__ AdamHp sh;
  const int b = blockIdx.y;
  if (threadIdx.x == 0) {
    AdamHp h;
    h.lr = p.lr[b]; h.b1 = p.beta1[b]; h.b2 = p.beta2[b]; h.eps = p.eps[b]; h.wd = p.wd[b];
    h.inv_bc1 = (float)(1.0 / (1.0 - pow((double)h.b1, (double)p.t)));
    h.inv_bc2 = (float)(1.0 / (1.0 - pow((double)h.b2, (double)p.t)));
    sh = h;
  }
  __syncthreads();
  const AdamHp h = sh;
  const int64_t base = (int64_t)b * p.P;
  const G* gr = reinterpret_cast<const G*>(p.grad) + base;
  if (VEC4) {
    const int64_t i = ((int64_t)blockIdx.x * 256 + threadIdx.x) * 4;
    if (i >= p.P) return;
    float4 th = *reinterpret_cast<float4*>(p.theta + base + i);
    float4 m = *reinterpret_cast<float4*>(p.m + base + i);
    float4 v = *reinterpret_cast<float4*>(p.v + base + i);
    float g[4];
    if (sizeof(G) == 4) {
      *reinterpret_cast<float4*>(g) = *reinterpret_cast<const float4*>(gr + i);
    } else {
      const uint2 raw = *reinterpret_cast<const uint2*>(gr + i);
      g[0] = __uint_as_float(raw.x << 16); g[1] = __uint_as_float(raw.x & 0xffff0000u);
      g[2] = __uint_as_float(raw.y << 16); g[3] = __uint_as_float(raw.y & 0xffff0000u);
    }
    adam_one(th.x, g[0], m.x, v.x, h, p.decoupled);
    adam_one(th.y, g[1], m.y, v.y, h, p.decoupled);
    adam_one(th.z, g[2], m.z, v.z, h, p.decoupled);
    adam_one(th.w, g[3], m.w, v.w, h, p.decoupled);
    *reinterpret_cast<float4*>(p.theta + base + i) = th;
    *reinterpret_cast<float4*>(p.m + base + i) = m;
    *reinterpret_cast<float4*>(p.v + base + i) = v;
    if (p.lowp) {
      uint2 o;
      o.x = pack_bf16x2(th.x, th.y);
      o.y = pack_bf16x2(th.z, th.w);
      *reinterpret_cast<uint2*>(p.lowp + base + i) = o;
    }
  } else {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= p.P) return;
    float th = p.theta[base + i], m = p.m[base + i], v = p.v[base + i];
    const float g = Elem<G>::load(gr + i);
    adam_one(th, g, m, v, h, p.decoupled);
    p.theta[base + i] = th; p.m[base + i] = m; p.v[base + i] = v;
    if (p.lowp) p.lowp[base + i] = f32_to_bf16(th);
  }
}

struct AdamMultiArgs {
  float* theta; const void* grad; float* m; float* v; bf16_raw* lowp;
  const float* lr; const float* beta1; const float* beta2; const float* eps; const float* wd;
  int64_t total;                                  // B * P
  int B, nseg, t, decoupled;
  int64_t off[HFTA_ADAM_MAX_SEGMENTS + 1];        // per-model element offsets
};

// Parameter-major arena: thread -> flat index -> (segment, model).  The bias
// corrections of all B models are formed once per workgroup in double.
template <typename G, bool VEC4, bool NT>
__global__ __launch_bounds__(256) void adam_multi_kernel(AdamMultiArgs p) {
  extern __shared__ float bc[];                   // [B][2]
  for (int b = threadIdx.x; b < p.B; b += 256) {
    bc[2 * b] = (float)(1.0 / (1.0 - pow((double)p.beta1[b], (double)p.t)));
    bc[2 * b + 1] = (float)(1.0 / (1.0 - pow((double)p.beta2[b], (double)p.t)));
  }
  __syncthreads();
  constexpr int W = VEC4 ? 4 : 1;
  const int64_t i = ((int64_t)blockIdx.x * 256 + threadIdx.x) * W;
  if (i >= p.total) return;
  // binary search: largest j with B*off[j] <= i
  int lo = 0, hi = p.nseg;
  while (hi - lo > 1) {
    const int mid = (lo + hi) >> 1;
    if ((int64_t)p.B * p.off[mid] <= i) lo = mid; else hi = mid;
  }
  const int64_t n = p.off[lo + 1] - p.off[lo];
  const int b = (int)((i - (int64_t)p.B * p.off[lo]) / n);
  AdamHp h;
  h.lr = p.lr[b]; h.b1 = p.beta1[b]; h.b2 = p.beta2[b]; h.eps = p.eps[b]; h.wd = p.wd[b];
  h.inv_bc1 = bc[2 * b]; h.inv_bc2 = bc[2 * b + 1];
  const G* gr = reinterpret_cast<const G*>(p.grad);
  if (VEC4) {
    float4 th = adam_ld<NT>(p.theta + i);
    float4 m = adam_ld<NT>(p.m + i);
    float4 v = adam_ld<NT>(p.v + i);
    float g[4];
    if (sizeof(G) == 4) {
      *reinterpret_cast<float4*>(g) = adam_ld<NT>((const float*)(gr + i));
    } else {
      const uint2 raw = *reinterpret_cast<const uint2*>(gr + i);
      g[0] = __uint_as_float(raw.x << 16); g[1] = __uint_as_float(raw.x & 0xffff0000u);
      g[2] = __uint_as_float(raw.y << 16); g[3] = __uint_as_float(raw.y & 0xffff0000u);
    }
    adam_one(th.x, g[0], m.x, v.x, h, p.decoupled);
    adam_one(th.y, g[1], m.y, v.y, h, p.decoupled);
    adam_one(th.z, g[2], m.z, v.z, h, p.decoupled);
    adam_one(th.w, g[3], m.w, v.w, h, p.decoupled);
    adam_st<NT>(p.theta + i, th);
    adam_st<NT>(p.m + i, m);
    adam_st<NT>(p.v + i, v);
    if (p.lowp) {
      uint2 o;
      o.x = pack_bf16x2(th.x, th.y);
      o.y = pack_bf16x2(th.z, th.w);
      *reinterpret_cast<uint2*>(p.lowp + i) = o;
    }
  } else {
    float th = p.theta[i], m = p.m[i], v = p.v[i];
    const float g = Elem<G>::load(gr + i);
    adam_one(th, g, m, v, h, p.decoupled);
    p.theta[i] = th; p.m[i] = m; p.v[i] = v;
    if (p.lowp) p.lowp[i] = f32_to_bf16(th);
  }
}

// where element i of the arena lies: its model, and the end of that model's part of the segment
__device__ __forceinline__ void adam_locate(const AdamMultiArgs& p, int64_t i, int& b, int64_t& end) {
  int lo = 0, hi = p.nseg;                        // largest j with B * off[j] <= i
  while (hi - lo > 1) {
    const int mid = (lo + hi) >> 1;
    if ((int64_t)p.B * p.off[mid] <= i) lo = mid; else hi = mid;
  }
  const int64_t n = p.off[lo + 1] - p.off[lo], base = (int64_t)p.B * p.off[lo];
  const int64_t q = i - base;
  b = q < 0x7fffffffLL && n < 0x7fffffffLL ? (int)((uint32_t)q / (uint32_t)n) : (int)(q / n);
  end = base + (int64_t)(b + 1) * n;
}

// The same for arenas with segments of any length (9 biases, 50 classes): 16-byte accesses need the arrays' alignment alone.
// A workgroup's elements mostly lie in one model's part of one segment: that is looked up once for the workgroup; only
// workgroups with a boundary in them look up per thread, and only groups of four across a boundary per element.  HBM-bound:
// 27.8 M parameters 340 (element-wise) -> 147 us, 15.1 M 190 -> 78.  Arenas of whole groups keep the kernel above: 268 M
// parameters 1450 us there, 1477 here (1640 with the loads ahead of the lookup).  Small arenas are bound by the chain of two
// lookups, of many parts (a model's share of a segment) by their boundaries, and keep the kernel above too, element by element.
// Element-wise and here, in us: parts of similar length, 1 part, 600 k parameters 8.5 7.2, 64 parts 600 k 9.7 9.9, 1.0 M 13.1
// 11.3, 240 parts 800 k 12.4 13.4, 1.2 M 15.8 14.9, 960 parts 1.0 M 14.7 17.2, 1.3 M 16.8 17.3, 2.0 M 23.6 18.5, 9600 parts
// 1.3 M 18.5 21.2, 2.0 M 25.2 24.6; lengths over all magnitudes, 36 parts 727 k 10.7 12.3, 63 parts 914 k 12.7 14.4, 156 parts
// 1.0 M 13.7 14.8.  More than 128 models cost the element-wise kernel's workgroups their bias corrections: 256 models, 30
// segments 700 k 15.6 15.9, 1.0 M 20.5 17.8.
int64_t adam_odd_min(int B, int nseg) {
  return (14 << 16) + (B > 128 ? 0 : std::min((int64_t)B * nseg * 768, (int64_t)18 << 16));
}
template <typename G, bool NT>
__global__ __launch_bounds__(256, 8) void adam_multi_odd_kernel(AdamMultiArgs p) {
  extern __shared__ float bc[];                   // [B][2]
  const int64_t i0 = (int64_t)blockIdx.x * 1024, i = i0 + threadIdx.x * 4;
  for (int b = threadIdx.x; b < p.B; b += 256) {
    bc[2 * b] = (float)(1.0 / (1.0 - pow((double)p.beta1[b], (double)p.t)));
    bc[2 * b + 1] = (float)(1.0 / (1.0 - pow((double)p.beta2[b], (double)p.t)));
  }
  __syncthreads();
  if (i >= p.total) return;
  auto params = [&](int b) {
    AdamHp h;
    h.lr = p.lr[b]; h.b1 = p.beta1[b]; h.b2 = p.beta2[b]; h.eps = p.eps[b]; h.wd = p.wd[b];
    h.inv_bc1 = bc[2 * b]; h.inv_bc2 = bc[2 * b + 1];
    return h;
  };
  int b;
  int64_t end;
  adam_locate(p, i0, b, end);
  if (end < i0 + 1024) adam_locate(p, i, b, end);
  const G* gr = reinterpret_cast<const G*>(p.grad);
  if (i + 4 > end) {                              // across a boundary, or fewer than four at the arena's end
    for (int64_t j = i; j < i + 4 && j < p.total; ++j) {
      adam_locate(p, j, b, end);
      float th = p.theta[j], m = p.m[j], v = p.v[j];
      adam_one(th, Elem<G>::load(gr + j), m, v, params(b), p.decoupled);
      p.theta[j] = th; p.m[j] = m; p.v[j] = v;
      if (p.lowp) p.lowp[j] = f32_to_bf16(th);
    }
    return;
  }
  float4 th = adam_ld<NT>(p.theta + i);
  float4 m = adam_ld<NT>(p.m + i);
  float4 v = adam_ld<NT>(p.v + i);
  float g[4];
  if (sizeof(G) == 4) {
    *reinterpret_cast<float4*>(g) = adam_ld<NT>((const float*)(gr + i));
  } else {
    const uint2 raw = *reinterpret_cast<const uint2*>(gr + i);
    g[0] = __uint_as_float(raw.x << 16); g[1] = __uint_as_float(raw.x & 0xffff0000u);
    g[2] = __uint_as_float(raw.y << 16); g[3] = __uint_as_float(raw.y & 0xffff0000u);
  }
  const AdamHp h = params(b);
  adam_one(th.x, g[0], m.x, v.x, h, p.decoupled);
  adam_one(th.y, g[1], m.y, v.y, h, p.decoupled);
  adam_one(th.z, g[2], m.z, v.z, h, p.decoupled);
  adam_one(th.w, g[3], m.w, v.w, h, p.decoupled);
  adam_st<NT>(p.theta + i, th);
  adam_st<NT>(p.m + i, m);
  adam_st<NT>(p.v + i, v);
  if (p.lowp) *reinterpret_cast<uint2*>(p.lowp + i) = make_uint2(pack_bf16x2(th.x, th.y), pack_bf16x2(th.z, th.w));
}

}  // namespace

extern "C" int hfta_adam_step_multi(int B, int nseg, const int64_t* seg_offsets, int grad_dtype, float* theta,
                                    const void* grad, float* m, float* v, void* theta_lowp, const float* lr,
                                    const float* beta1, const float* beta2, const float* eps,
                                    const float* weight_decay, int step_t, int decoupled_wd, void* stream) {
  if (B <= 0 || nseg <= 0 || !seg_offsets || !valid_dtype(grad_dtype) || !theta || !grad || !m || !v || !lr || !beta1 ||
      !beta2 || !eps || !weight_decay || step_t < 1)
    return HFTA_EINVAL;
  if (nseg > HFTA_ADAM_MAX_SEGMENTS || B > HFTA_ADAM_MAX_MODELS) return HFTA_EUNSUPPORTED;
  if (seg_offsets[0] != 0) return HFTA_EINVAL;
  AdamMultiArgs a;
  bool all4 = true;
  for (int j = 0; j <= nseg; ++j) {
    if (j > 0 && seg_offsets[j] <= seg_offsets[j - 1]) return HFTA_EINVAL;
    a.off[j] = seg_offsets[j];
    if (seg_offsets[j] % 4 != 0) all4 = false;
  }
  for (int j = nseg + 1; j <= HFTA_ADAM_MAX_SEGMENTS; ++j) a.off[j] = seg_offsets[nseg];
  auto al = [](const void* q, size_t k) { return reinterpret_cast<uintptr_t>(q) % k == 0; };
  const bool aligned = al(theta, 16) && al(m, 16) && al(v, 16) && al(grad, grad_dtype == HFTA_BF16 ? 8 : 16) &&
                  (!theta_lowp || al(theta_lowp, 8));
  a.theta = theta; a.grad = grad; a.m = m; a.v = v; a.lowp = (bf16_raw*)theta_lowp;
  a.lr = lr; a.beta1 = beta1; a.beta2 = beta2; a.eps = eps; a.wd = weight_decay;
  a.total = (int64_t)B * seg_offsets[nseg];
  a.B = B; a.nseg = nseg; a.t = step_t; a.decoupled = decoupled_wd ? 1 : 0;
  const bool v4 = aligned && all4, odd = aligned && !all4 && a.total >= adam_odd_min(B, nseg);
  const int64_t per_block = v4 || odd ? 1024 : 256;
  const int64_t blocks = (a.total + per_block - 1) / per_block;
  if (blocks > 0x7fffffffLL) return HFTA_EINVAL;
  const size_t shm = (size_t)B * 2 * sizeof(float);
  hipStream_t st = as_stream(stream);
  dim3 grid((unsigned)blocks);
  const bool nt = a.total >= ADAM_NT_MIN;
#define HFTA_ADAM(K) hipLaunchKernelGGL((K), grid, dim3(256), shm, st, a)
#define HFTA_ADAM_BY_SIZE(G) \
  do { if (odd) { if (nt) HFTA_ADAM((adam_multi_odd_kernel<G, true>)); else HFTA_ADAM((adam_multi_odd_kernel<G, false>)); } \
       else if (v4) { if (nt) HFTA_ADAM((adam_multi_kernel<G, true, true>)); else HFTA_ADAM((adam_multi_kernel<G, true, false>)); } \
       else HFTA_ADAM((adam_multi_kernel<G, false, false>)); } while (0)
  if (grad_dtype == HFTA_BF16) HFTA_ADAM_BY_SIZE(bf16_raw);
  else HFTA_ADAM_BY_SIZE(float);
#undef HFTA_ADAM_BY_SIZE
#undef HFTA_ADAM
  return launch_status();
}

extern "C" int hfta_adam_step(int B, int64_t P, int grad_dtype, float* theta, const void* grad, float* m, float* v,
                              void* theta_lowp, const float* lr, const float* beta1, const float* beta2,
                              const float* eps, const float* weight_decay, int step_t, int decoupled_wd,
                              void* stream) {
  if (B <= 0 || P <= 0 || !valid_dtype(grad_dtype) || !theta || !grad || !m || !v || !lr || !beta1 || !beta2 || !eps ||
      !weight_decay || step_t < 1)
    return HFTA_EINVAL;
  if (B > 65535) return HFTA_EUNSUPPORTED;
  auto al = [](const void* q, size_t a) { return reinterpret_cast<uintptr_t>(q) % a == 0; };
  const bool v4 = P % 4 == 0 && al(theta, 16) && al(m, 16) && al(v, 16) && al(grad, grad_dtype == HFTA_BF16 ? 8 : 16) &&
                  (!theta_lowp || al(theta_lowp, 8));
  const int64_t per_block = v4 ? 1024 : 256;
  const int64_t blocks = (P + per_block - 1) / per_block;
  if (blocks > 0x7fffffffLL) return HFTA_EINVAL;
  AdamArgs a{theta, grad, m, v, (bf16_raw*)theta_lowp, lr, beta1, beta2, eps, weight_decay, P, step_t, decoupled_wd ? 1 : 0};
  dim3 grid((unsigned)blocks, (unsigned)B);
  hipStream_t st = as_stream(stream);
  if (grad_dtype == HFTA_BF16) {
    if (v4) hipLaunchKernelGGL((adam_kernel<bf16_raw, true>), grid, dim3(256), 0, st, a);
    else hipLaunchKernelGGL((adam_kernel<bf16_raw, false>), grid, dim3(256), 0, st, a);
  } else {
    if (v4) hipLaunchKernelGGL((adam_kernel<float, true>), grid, dim3(256), 0, st, a);
    else hipLaunchKernelGGL((adam_kernel<float, false>), grid, dim3(256), 0, st, a);
  }
  return launch_status();
}
