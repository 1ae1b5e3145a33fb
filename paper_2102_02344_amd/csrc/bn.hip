// Fused BatchNorm (training mode) over the channels of all B models.
//
// Conv-family layout (stride_l == 1): one workgroup per channel (b, c), which needs the channel's Nb rows of L
// contiguous elements twice -- for the sums, and to form the result.  The first H pieces of four elements per
// thread stay in registers in between (held_pieces() below); what a channel has beyond that is read again,
// from L2 / Infinity Cache for all but the largest channels.  Statistics use sums shifted by the channel's
// first element, which keeps fp32 accurate when |mean| >> std.
// Reductions: per-lane partials -> wave64 shuffle reduction -> 4-entry LDS.
//
// Linear layout (L == 1, stride_c == 1, the table's [N, B, C] case): one thread
// per channel, coalesced across channels, two passes over the Nb samples.
#include <type_traits>
#include "bn_common.h"

namespace hfta { int persistent_blocks(); }     // compute units

using namespace hfta;

namespace {

constexpr int BN_UNROLL = 4;   // pieces a thread loads before it uses the first (conv layout)

struct BnFwdArgs {
  const void* X; void* Y;
  const float* gamma; const float* beta;
  float* running_mean; float* running_var; float* save_mean; float* save_invstd;
  int64_t xsb, xsn, xsc, ysb, ysn, ysc;
  int Nb, C, L, act;
  float eps, momentum, slope;
};

// What bounds these kernels is the memory system behind L2: two workgroups of a 160 KB channel pair on each of 32 units are
// more than an XCD's 4 MB, so a second read travels the fabric again.  With the pieces in registers the forward moves two
// tensors instead of three, the backward three instead of five.
//
// held_waves: wavefronts per SIMD for `words` held registers (1024 threads: 8 or 4; 8 take up to `most`; nothing held: what the
// kernel comes to, 7 or 8).
constexpr int held_waves(int words, int most, int nt) { return words == 0 ? 4 : words <= most ? 8 : nt == 1024 || words > 56 ? 4 : 5; }

// the words of a piece (element offsets from the channel's start in 32 bits: a scalar base and one register a load; held_rows_ok)
template <typename T>
__device__ __forceinline__ void held_load(const T* x, uint32_t row, int ch, uint32_t (&w)[sizeof(T)]) {
  typedef uint32_t V __attribute__((ext_vector_type(sizeof(T))));
  const uint32_t at = (row + (uint32_t)ch * 4u) * (uint32_t)sizeof(T);
  const V raw = *reinterpret_cast<const V*>(reinterpret_cast<const char*>(x) + at);
#pragma unroll
  for (int i = 0; i < (int)sizeof(T); ++i) w[i] = raw[i];
}
template <typename T>
__device__ __forceinline__ void held_values(const uint32_t (&w)[sizeof(T)], float (&v)[4]) {
  if (sizeof(T) == 2) {
    v[0] = __uint_as_float(w[0] << 16); v[1] = __uint_as_float(w[0] & 0xffff0000u);
    v[2] = __uint_as_float(w[1] << 16); v[3] = __uint_as_float(w[1] & 0xffff0000u);
  } else {
#pragma unroll
    for (int e = 0; e < 4; ++e) v[e] = __uint_as_float(w[e & (sizeof(T) - 1)]);
  }
}
// The walk again from the start: what the last one computed along the way is not kept in registers.
__device__ __forceinline__ RowWalk held_walk(const RowWalk& start) {
  RowWalk w = start;
  asm volatile("" : "+v"(w.n), "+v"(w.ch));
  return w;
}
// keeps the words, not the values made from them, in registers
template <int W> __device__ __forceinline__ void held_keep(uint32_t (&w)[W]) {
#pragma unroll
  for (int i = 0; i < W; ++i) asm volatile("" : "+v"(w[i]));
}

template <typename T, int VEC, int NT, int H>
__global__ __launch_bounds__(NT, VEC == 1 ? 4 : held_waves(H * (int)sizeof(T), NT == 1024 ? 40 : 20, NT)) void bn_fwd_conv_kernel(BnFwdArgs p, int per) {
  constexpr int UN = H ? 2 : bn_unroll(VEC), W = sizeof(T);
  static_assert(H == 0 || VEC == 4, "pieces are held whole");
  __shared__ float sh[NT / 64][2];
  const int c = blockIdx.x, b = blockIdx.y;
  const T* x = reinterpret_cast<const T*>(p.X) + b * p.xsb + c * p.xsc;
  T* y = reinterpret_cast<T*>(p.Y) + b * p.ysb + c * p.ysc;
  const int chunks = p.L / VEC;
  uint32_t held[H ? H : 1][W];
  const RowWalk start(chunks, NT);
  RowWalk rest = held_walk(start);                                  // where the pieces that are not held begin
#pragma unroll
  for (int u = 0; u < H; ++u) {
    if (u % 4 == 0 && u >= per) break;                   // `per` pieces exist for some thread
    const bool ok = rest.n < p.Nb;                       // a piece past the end re-reads the channel's first and is not used
    held_load<T>(x, ok ? (uint32_t)rest.n * (uint32_t)p.xsn : 0u, ok ? rest.ch : 0, held[u]);
    rest.step();
  }
  const float shift = Elem<T>::load(x);
  float s1 = 0.f, s2 = 0.f;
  auto add = [&](const float (&v)[VEC]) {
#pragma unroll
    for (int e = 0; e < VEC; ++e)
      { const float d = v[e] - shift; s1 += d; s2 = fmaf(d, d, s2); }
  };
  if constexpr (H > 0) {
    RowWalk w = held_walk(start);
#pragma unroll
    for (int u = 0; u < H; ++u) {
      if (u % 4 == 0 && u >= per) break;
      float v[VEC];
      held_values<T>(held[u], v);
      if (w.n < p.Nb) add(v);
      held_keep(held[u]);
      w.step();
    }
  }
  for (RowWalk w = rest; w.n < p.Nb;) {
    // UN pieces per trip, their loads issued together: the bytes in flight per thread set the bandwidth
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
      if (ok[u]) add(v[u]);
  }
  block_sum2<NT / 64>(s1, s2, sh);
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
  if (!p.Y) return;                      // statistics only: a consumer normalises on load
  auto write = [&](float (&v)[VEC], int n, int ch) {
#pragma unroll
    for (int e = 0; e < VEC; ++e) v[e] = bn_act(fmaf(g, (v[e] - mean) * invstd, bt), p.act, p.slope);
    store_vec<T, VEC>(y + n * p.ysn + ch * VEC, v);
  };
  if constexpr (H > 0) {
    RowWalk w = held_walk(start);
#pragma unroll
    for (int u = 0; u < H; ++u) {
      if (u % 4 == 0 && u >= per) break;
      float v[VEC];
      held_values<T>(held[u], v);
      if (w.n < p.Nb) write(v, w.n, w.ch);
      w.step();
    }
  }
  for (RowWalk w = rest; w.n < p.Nb;) {
    float v[UN][VEC];
    int n[UN], ch[UN];
#pragma unroll
    for (int u = 0; u < UN; ++u) {
      n[u] = w.n; ch[u] = w.ch;
      load_vec<T, VEC>(n[u] < p.Nb ? x + n[u] * p.xsn + ch[u] * VEC : x, v[u]);
      w.step();
    }
#pragma unroll
    for (int u = 0; u < UN; ++u)
      if (n[u] < p.Nb) write(v[u], n[u], ch[u]);
  }
}

// Rows that are no multiple of four elements: the sums run over single elements in order (the walk of VEC == 1: thread t adds
// the channel's elements t, t + NT, ...), whatever the loads are, because sums in another order move the outputs of the
// segmentation and the transform array by 0.01 to 0.1 after three steps, more than two correct forms may differ by.  Single
// elements from memory reach a quarter of the bandwidth, so a channel travels in four-element pieces into LDS, rows at a pitch
// of whole pieces, and is added up from there, 2 or 4 bytes a lane.
// Stages rows of L elements at pitch 4 * chunks; the caller's barrier makes them visible.
template <typename T, int NT>
__device__ __forceinline__ void bn_stage(T* lds, const T* x, int64_t sn, int Nb, int L, int chunks) {
  constexpr int UN = 4, W = sizeof(T);
  typedef uint32_t Words __attribute__((ext_vector_type(W)));
  for (RowWalk w(chunks, NT); w.n < Nb;) {
    Words q[UN];
    int n[UN], ch[UN];
#pragma unroll
    for (int u = 0; u < UN; ++u) {
      n[u] = w.n; ch[u] = w.ch;
      const bool ok = w.n < Nb;
      const typename PieceAt<T>::type raw = *reinterpret_cast<const typename PieceAt<T>::type*>((ok ? x + w.n * sn : x) + (ok ? min(w.ch * 4, L - 4) : 0));
#pragma unroll
      for (int i = 0; i < W; ++i) q[u][i] = raw[i];
      w.step();
    }
#pragma unroll
    for (int u = 0; u < UN; ++u)
      if (n[u] < Nb) {
        uint32_t v[W];
#pragma unroll
        for (int i = 0; i < W; ++i) v[i] = q[u][i];
        piece_shift(v, ch[u] * 4 - min(ch[u] * 4, L - 4));
#pragma unroll
        for (int i = 0; i < W; ++i) q[u][i] = v[i];
        *reinterpret_cast<Words*>(lds + (n[u] * chunks + ch[u]) * 4) = q[u];
      }
  }
}
constexpr int STAGE_SMALL = 20 * 1024 - 256, STAGE_MID = 40 * 1024 - 256, STAGE_HALF = 80 * 1024 - 256, STAGE_FULL = 160 * 1024 - 256;

template <typename T, int NT, int BYTES>
__global__ __launch_bounds__(NT) void bn_fwd_odd_kernel(BnFwdArgs p) {
  __shared__ float sh[NT / 64][2];
  __shared__ __attribute__((aligned(16))) unsigned char smem[BYTES];
  T* lds = reinterpret_cast<T*>(smem);
  const int c = blockIdx.x, b = blockIdx.y;
  const T* x = reinterpret_cast<const T*>(p.X) + b * p.xsb + c * p.xsc;
  T* y = reinterpret_cast<T*>(p.Y) + b * p.ysb + c * p.ysc;
  const int chunks = (p.L + 3) / 4, pitch = chunks * 4;
  const float shift = Elem<T>::load(x);
  bn_stage<T, NT>(lds, x, p.xsn, p.Nb, p.L, chunks);
  __syncthreads();
  float s1 = 0.f, s2 = 0.f;
#pragma unroll 8
  for (RowWalk w(p.L, NT); w.n < p.Nb; w.step()) {
    const float d = Elem<T>::load(lds + w.n * pitch + w.ch) - shift;
    s1 += d;
    s2 = fmaf(d, d, s2);
  }
  block_sum2<NT / 64>(s1, s2, sh);
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
  if (!p.Y) return;
  for (RowWalk w(chunks, NT); w.n < p.Nb; w.step()) {
    float v[4];
    load_vec<T, 4>(lds + (w.n * chunks + w.ch) * 4, v);
#pragma unroll
    for (int e = 0; e < 4; ++e) v[e] = bn_act(fmaf(g, (v[e] - mean) * invstd, bt), p.act, p.slope);
    store_piece<T, 4, true>(y + w.n * p.ysn, w.ch, p.L, v);
  }
}

// Normalisation with given statistics (the forward kernel's second pass alone): what a consumer that
// normalises on load computes, written out.
template <typename T, int VEC, int NT, bool RAG>
__global__ __launch_bounds__(NT) void bn_apply_conv_kernel(BnFwdArgs p) {
  const int c = blockIdx.x, b = blockIdx.y, k = b * p.C + c;
  const T* x = reinterpret_cast<const T*>(p.X) + b * p.xsb + c * p.xsc;
  T* y = reinterpret_cast<T*>(p.Y) + b * p.ysb + c * p.ysc;
  const int chunks = RAG ? (p.L + VEC - 1) / VEC : p.L / VEC;
  const float mean = p.save_mean[k], invstd = p.save_invstd[k], g = p.gamma[k], bt = p.beta[k];
  for (RowWalk w(chunks, NT); w.n < p.Nb;) {
    float v[BN_UNROLL][VEC];
    int n[BN_UNROLL], ch[BN_UNROLL];
#pragma unroll
    for (int u = 0; u < BN_UNROLL; ++u) {
      n[u] = w.n; ch[u] = w.ch;
      load_piece<T, VEC, RAG>(n[u] < p.Nb ? x + n[u] * p.xsn : x, n[u] < p.Nb ? ch[u] : 0, p.L, v[u]);
      w.step();
    }
#pragma unroll
    for (int u = 0; u < BN_UNROLL; ++u)
      if (n[u] < p.Nb) {
#pragma unroll
        for (int e = 0; e < VEC; ++e) v[u][e] = bn_act(fmaf(g, (v[u][e] - mean) * invstd, bt), p.act, p.slope);
        store_piece<T, VEC, RAG>(y + n[u] * p.ysn, ch[u], p.L, v[u]);
      }
  }
}

// Training statistics from partial sums that the producing convolution left behind (sums of (x - shift) and
// (x - shift)^2 per slice, shift = the channel's conv bias or 0), so that the tensor is read once, for the
// normalisation (bn_apply_conv_kernel), or not at all (a consumer normalises on load).  The partials lie
// [part][channel], so a workgroup takes 16 neighbouring channels -- 16 lanes read 128 contiguous bytes of one
// part, 64 such rows are in flight per step -- instead of one channel whose parts are a channel count apart.
// Per-lane sums in a fixed order, then a fixed-order tree over the 64 part lanes.
constexpr int BNS_C = 16, BNS_P = 64;
__global__ __launch_bounds__(BNS_C * BNS_P) void bn_stats_part_kernel(BnFwdArgs p, const float* __restrict__ part, int parts,
                                                                      const bf16_raw* __restrict__ shift_v) {
  __shared__ float2 red[BNS_P][BNS_C];
  const int cl = threadIdx.x & (BNS_C - 1), pl = threadIdx.x / BNS_C;
  const int c = blockIdx.x * BNS_C + cl, b = blockIdx.y;
  const bool live = c < p.C;
  const float2* pp = reinterpret_cast<const float2*>(part) + (int64_t)b * parts * p.C + (live ? c : 0);
  float s1 = 0.f, s2 = 0.f;
#pragma unroll 4
  for (int i = pl; i < parts; i += BNS_P) {
    const float2 v = pp[(int64_t)i * p.C];
    s1 += v.x; s2 += v.y;
  }
  red[pl][cl] = make_float2(s1, s2);
  __syncthreads();
  for (int h = BNS_P / 2; h > 0; h >>= 1) {
    if (pl < h) {
      const float2 a = red[pl][cl], o = red[pl + h][cl];
      red[pl][cl] = make_float2(a.x + o.x, a.y + o.y);
    }
    __syncthreads();
  }
  if (pl != 0 || !live) return;
  const int k = b * p.C + c;
  const float shift = shift_v ? bf16_to_f32(shift_v[k]) : 0.f;
  const float m = (float)p.Nb * (float)p.L;
  const float dm = red[0][cl].x / m;
  const float mean = shift + dm;
  float var = red[0][cl].y / m - dm * dm;
  var = var < 0.f ? 0.f : var;
  p.save_mean[k] = mean;
  p.save_invstd[k] = 1.0f / sqrtf(var + p.eps);
  if (p.running_mean) {
    const float unb = m > 1.f ? var * (m / (m - 1.f)) : var;
    p.running_mean[k] = (1.f - p.momentum) * p.running_mean[k] + p.momentum * mean;
    p.running_var[k] = (1.f - p.momentum) * p.running_var[k] + p.momentum * unb;
  }
}

// Linear layout [.., Nb, C] (channel stride 1, the fully connected head): a workgroup owns 64
// channels x 16 sample lanes, so the loads of a column are spread over lanes instead of walking one
// after the other through the memory latency; per-lane partial sums meet in LDS in a fixed order.
constexpr int BNL_C = 64, BNL_N = 16;

__device__ __forceinline__ float bnl_reduce(float v, float (*red)[BNL_C], int tx, int ty) {
  __syncthreads();                       // the previous reduction's readers are done
  red[ty][tx] = v;
  __syncthreads();
  float s = 0.f;
#pragma unroll
  for (int j = 0; j < BNL_N; ++j) s += red[j][tx];
  return s;
}

template <typename T>
__global__ __launch_bounds__(BNL_C * BNL_N) void bn_fwd_linear_kernel(BnFwdArgs p) {
  __shared__ float red[BNL_N][BNL_C];
  const int tx = threadIdx.x % BNL_C, ty = threadIdx.x / BNL_C;
  const int c = blockIdx.x * BNL_C + tx, b = blockIdx.y;
  const bool live = c < p.C;
  const int cc = live ? c : p.C - 1;
  const T* x = reinterpret_cast<const T*>(p.X) + b * p.xsb + cc;
  T* y = reinterpret_cast<T*>(p.Y) + b * p.ysb + cc;
  float s = 0.f;
  for (int n = ty; n < p.Nb; n += BNL_N) s += Elem<T>::load(x + n * p.xsn);
  const float m = (float)p.Nb;
  const float mean = bnl_reduce(s, red, tx, ty) / m;
  float q = 0.f;
  for (int n = ty; n < p.Nb; n += BNL_N) { const float d = Elem<T>::load(x + n * p.xsn) - mean; q = fmaf(d, d, q); }
  const float var = bnl_reduce(q, red, tx, ty) / m;
  const float invstd = 1.0f / sqrtf(var + p.eps);
  const int k = b * p.C + cc;
  const float g = p.gamma[k], bt = p.beta[k];
  if (live && ty == 0) {
    p.save_mean[k] = mean;
    p.save_invstd[k] = invstd;
    if (p.running_mean) {
      const float unb = m > 1.f ? var * (m / (m - 1.f)) : var;
      p.running_mean[k] = (1.f - p.momentum) * p.running_mean[k] + p.momentum * mean;
      p.running_var[k] = (1.f - p.momentum) * p.running_var[k] + p.momentum * unb;
    }
  }
  if (!live) return;
  for (int n = ty; n < p.Nb; n += BNL_N) {
    const float v = Elem<T>::load(x + n * p.xsn);
    Elem<T>::store(y + n * p.ysn, bn_act(fmaf(g, (v - mean) * invstd, bt), p.act, p.slope));
  }
}

struct BnBwdArgs {
  const void* X; const void* dY; void* dX;
  const float* gamma; const float* beta; const float* save_mean; const float* save_invstd;
  float* dgamma; float* dbeta; float* dx_sum;
  int64_t xsb, xsn, xsc, dysb, dysn, dysc, dxsb, dxsn, dxsc;
  int Nb, C, L, act;
  float slope;
};

// XL: the pieces of X wait in LDS and only those of dY in registers, so that two 1024-thread workgroups fit a compute unit
// (80 KB and 64 registers each) and one loads while the other writes.
template <typename T, int VEC, int NT, int H, bool XL>
__global__ __launch_bounds__(NT, VEC == 1 ? 4 : XL ? 8 : held_waves(2 * H * (int)sizeof(T), 20, NT)) void bn_bwd_conv_kernel(BnBwdArgs p, int per) {
  constexpr int UN = H ? 2 : bn_unroll(VEC), W = sizeof(T), G = H > 4 ? (H + 1) / 2 : 4;    // G: pieces loaded at a time
  static_assert(H == 0 || VEC == 4, "pieces are held whole");
  __shared__ float sh[NT / 64][2];
  const int c = blockIdx.x, b = blockIdx.y, k = b * p.C + c;
  const T* x = reinterpret_cast<const T*>(p.X) + b * p.xsb + c * p.xsc;
  const T* dy = reinterpret_cast<const T*>(p.dY) + b * p.dysb + c * p.dysc;
  T* dx = reinterpret_cast<T*>(p.dX) + b * p.dxsb + c * p.dxsc;
  const int chunks = p.L / VEC;
  typedef uint32_t Words __attribute__((ext_vector_type(W)));
  constexpr int HL = XL ? H - 1 : 0;                     // pieces of X in LDS: the last one's place is left to the sums
  __shared__ Words xl[XL ? HL : 1][XL ? NT : 1];
  uint32_t hx[H ? H - HL : 1][W], hd[H ? H : 1][W];
  const RowWalk start(chunks, NT);
  const float mean = p.save_mean[k], invstd = p.save_invstd[k], g = p.gamma[k], bt = p.beta[k];
  float s1 = 0.f, s2 = 0.f;
  auto add = [&](const float (&v)[VEC], const float (&d)[VEC]) {
#pragma unroll
    for (int e = 0; e < VEC; ++e) {
      const float xh = (v[e] - mean) * invstd;
      const float gr = d[e] * act_grad(fmaf(g, xh, bt), p.act, p.slope);
      s1 += gr;
      s2 = fmaf(gr, xh, s2);
    }
  };
  RowWalk rest = held_walk(start);                       // where the pieces that are not held begin
  if constexpr (H > 0) {
#pragma unroll
    for (int u0 = 0; u0 < H; u0 += G) {
      if (u0 >= per) break;
      uint32_t tx[G][W];
      RowWalk w = rest;
#pragma unroll
      for (int i = 0; i < G; ++i) {
        if (u0 + i >= H) continue;
        const bool ok = rest.n < p.Nb;                   // a piece past the end re-reads the channel's first and is not used
        const int ch = ok ? rest.ch : 0;
        held_load<T>(x, ok ? (uint32_t)rest.n * (uint32_t)p.xsn : 0u, ch, tx[i]);
        held_load<T>(dy, ok ? (uint32_t)rest.n * (uint32_t)p.dysn : 0u, ch, hd[u0 + i]);
        rest.step();
      }
      w = held_walk(w);
#pragma unroll
      for (int i = 0; i < G; ++i) {
        const int u = u0 + i;
        if (u >= H) continue;
        float v[VEC], d[VEC];
        held_values<T>(tx[i], v);
        held_values<T>(hd[u], d);
        if (w.n < p.Nb) add(v, d);
        if (u < HL) {
          Words q;
#pragma unroll
          for (int j = 0; j < W; ++j) q[j] = tx[i][j];
          xl[u < HL ? u : 0][XL ? threadIdx.x : 0] = q;              // read by this thread alone
        } else {
#pragma unroll
          for (int j = 0; j < W; ++j) hx[u < HL ? 0 : u - HL][j] = tx[i][j];
          held_keep(hx[u < HL ? 0 : u - HL]);
        }
        held_keep(hd[u]);
        w.step();
      }
    }
  }
  for (RowWalk w = rest; w.n < p.Nb;) {
    float v[UN][VEC], d[UN][VEC];
    bool ok[UN];
#pragma unroll
    for (int u = 0; u < UN; ++u) {
      ok[u] = w.n < p.Nb;
      load_vec<T, VEC>(ok[u] ? x + w.n * p.xsn + w.ch * VEC : x, v[u]);
      load_vec<T, VEC>(ok[u] ? dy + w.n * p.dysn + w.ch * VEC : dy, d[u]);
      w.step();
    }
#pragma unroll
    for (int u = 0; u < UN; ++u)
      if (ok[u]) add(v[u], d[u]);
  }
  block_sum2<NT / 64>(s1, s2, sh);
  if (threadIdx.x == 0) { p.dbeta[k] = s1; p.dgamma[k] = s2; }
  const float m = (float)p.Nb * (float)p.L;
  const float mb = s1 / m, mg = s2 / m, sc = g * invstd;
  float s3 = 0.f;
  auto write = [&](float (&v)[VEC], const float (&d)[VEC], int n, int ch) {
#pragma unroll
    for (int e = 0; e < VEC; ++e) {
      const float xh = (v[e] - mean) * invstd;
      const float gr = d[e] * act_grad(fmaf(g, xh, bt), p.act, p.slope);
      v[e] = sc * (gr - mb - xh * mg);
      s3 += Elem<T>::to_f32(Elem<T>::from_f32(v[e]));     // the value as it is stored
    }
    store_vec<T, VEC>(dx + n * p.dxsn + ch * VEC, v);
  };
  if constexpr (H > 0) {
    RowWalk w = held_walk(start);
#pragma unroll
    for (int u = 0; u < H; ++u) {
      if (u % G == 0 && u >= per) break;
      float v[VEC], d[VEC];
      uint32_t tx[W];
      if (u < HL) {
        const Words q = xl[u < HL ? u : 0][XL ? threadIdx.x : 0];
#pragma unroll
        for (int j = 0; j < W; ++j) tx[j] = q[j];
      } else {
#pragma unroll
        for (int j = 0; j < W; ++j) tx[j] = hx[u < HL ? 0 : u - HL][j];
      }
      held_values<T>(tx, v);
      held_values<T>(hd[u], d);
      if (w.n < p.Nb) write(v, d, w.n, w.ch);
      w.step();
    }
  }
  for (RowWalk w = rest; w.n < p.Nb;) {
    float v[UN][VEC], d[UN][VEC];
    int n[UN], ch[UN];
#pragma unroll
    for (int u = 0; u < UN; ++u) {
      n[u] = w.n; ch[u] = w.ch;
      const bool ok = n[u] < p.Nb;
      load_vec<T, VEC>(ok ? x + n[u] * p.xsn + ch[u] * VEC : x, v[u]);
      load_vec<T, VEC>(ok ? dy + n[u] * p.dysn + ch[u] * VEC : dy, d[u]);
      w.step();
    }
#pragma unroll
    for (int u = 0; u < UN; ++u)
      if (n[u] < p.Nb) write(v[u], d[u], n[u], ch[u]);
  }
  if (p.dx_sum) {
    float dummy = 0.f;
    block_sum2<NT / 64>(s3, dummy, sh);
    if (threadIdx.x == 0) p.dx_sum[k] = s3;
  }
}

// Rows that are no multiple of four elements (see bn_fwd_odd_kernel): X and dY staged, the sums and that of the stored dX over
// single elements in order.
template <typename T, int NT, int BYTES>
__global__ __launch_bounds__(NT) void bn_bwd_odd_kernel(BnBwdArgs p) {
  __shared__ float sh[NT / 64][2];
  __shared__ __attribute__((aligned(16))) unsigned char smem[BYTES];
  const int c = blockIdx.x, b = blockIdx.y, k = b * p.C + c;
  const T* x = reinterpret_cast<const T*>(p.X) + b * p.xsb + c * p.xsc;
  const T* dy = reinterpret_cast<const T*>(p.dY) + b * p.dysb + c * p.dysc;
  T* dx = reinterpret_cast<T*>(p.dX) + b * p.dxsb + c * p.dxsc;
  const int chunks = (p.L + 3) / 4, pitch = chunks * 4;
  T* lx = reinterpret_cast<T*>(smem);
  T* ld = lx + p.Nb * pitch;
  bn_stage<T, NT>(lx, x, p.xsn, p.Nb, p.L, chunks);
  bn_stage<T, NT>(ld, dy, p.dysn, p.Nb, p.L, chunks);
  const float mean = p.save_mean[k], invstd = p.save_invstd[k], g = p.gamma[k], bt = p.beta[k];
  __syncthreads();
  float s1 = 0.f, s2 = 0.f;
#pragma unroll 8
  for (RowWalk w(p.L, NT); w.n < p.Nb; w.step()) {
    const int at = w.n * pitch + w.ch;
    const float xh = (Elem<T>::load(lx + at) - mean) * invstd;
    const float gr = Elem<T>::load(ld + at) * act_grad(fmaf(g, xh, bt), p.act, p.slope);
    s1 += gr;
    s2 = fmaf(gr, xh, s2);
  }
  block_sum2<NT / 64>(s1, s2, sh);
  if (threadIdx.x == 0) { p.dbeta[k] = s1; p.dgamma[k] = s2; }
  const float m = (float)p.Nb * (float)p.L;
  const float mb = s1 / m, mg = s2 / m, sc = g * invstd;
  for (RowWalk w(chunks, NT); w.n < p.Nb; w.step()) {
    T* at = lx + (w.n * chunks + w.ch) * 4;
    float v[4], d[4];
    load_vec<T, 4>(at, v);
    load_vec<T, 4>(ld + (w.n * chunks + w.ch) * 4, d);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const float xh = (v[e] - mean) * invstd;
      const float gr = d[e] * act_grad(fmaf(g, xh, bt), p.act, p.slope);
      v[e] = sc * (gr - mb - xh * mg);
    }
    store_piece<T, 4, true>(dx + w.n * p.dxsn, w.ch, p.L, v);
    if (p.dx_sum) store_vec<T, 4>(at, v);
  }
  if (p.dx_sum) {                        // uniform over the grid
    __syncthreads();
    float s3 = 0.f, dummy = 0.f;
#pragma unroll 8
    for (RowWalk w(p.L, NT); w.n < p.Nb; w.step()) s3 += Elem<T>::load(lx + w.n * pitch + w.ch);
    block_sum2<NT / 64>(s3, dummy, sh);
    if (threadIdx.x == 0) p.dx_sum[k] = s3;
  }
}

// The reduction half of the backward pass alone: dbeta, dgamma, and per channel the eight constants
// a consumer needs to form dX = sc * (g - mb - xhat * mg) by itself while it streams x and dY:
// coef[k] = {mean, invstd, gamma, beta, mb, mg, sc, 0}.  Nothing of size [Nb, C, L] is written.
template <typename T, int VEC, int NT, bool RAG>
__global__ __launch_bounds__(NT) void bn_bwd_conv_coef_kernel(BnBwdArgs p, float* __restrict__ coef) {
  __shared__ float sh[NT / 64][2];
  const int c = blockIdx.x, b = blockIdx.y, k = b * p.C + c;
  const T* x = reinterpret_cast<const T*>(p.X) + b * p.xsb + c * p.xsc;
  const T* dy = reinterpret_cast<const T*>(p.dY) + b * p.dysb + c * p.dysc;
  const float mean = p.save_mean[k], invstd = p.save_invstd[k], g = p.gamma[k], bt = p.beta[k];
  const int chunks = RAG ? (p.L + VEC - 1) / VEC : p.L / VEC;
  float s1 = 0.f, s2 = 0.f;
  for (RowWalk w(chunks, NT); w.n < p.Nb;) {
    float v[BN_UNROLL][VEC], d[BN_UNROLL][VEC];
    bool ok[BN_UNROLL];
#pragma unroll
    for (int u = 0; u < BN_UNROLL; ++u) {
      ok[u] = w.n < p.Nb;
      load_piece<T, VEC, RAG>(ok[u] ? x + w.n * p.xsn : x, ok[u] ? w.ch : 0, p.L, v[u]);
      load_piece<T, VEC, RAG>(ok[u] ? dy + w.n * p.dysn : dy, ok[u] ? w.ch : 0, p.L, d[u]);   // past a row's end dY is zero: adds nothing
      w.step();
    }
#pragma unroll
    for (int u = 0; u < BN_UNROLL; ++u)
      if (ok[u]) {
#pragma unroll
        for (int e = 0; e < VEC; ++e) {
          const float xh = (v[u][e] - mean) * invstd;
          const float gr = d[u][e] * act_grad(fmaf(g, xh, bt), p.act, p.slope);
          s1 += gr;
          s2 = fmaf(gr, xh, s2);
        }
      }
  }
  block_sum2<NT / 64>(s1, s2, sh);
  if (threadIdx.x == 0) {
    p.dbeta[k] = s1;
    p.dgamma[k] = s2;
    const float m = (float)p.Nb * (float)p.L;
    float4* o = reinterpret_cast<float4*>(coef + (int64_t)k * 8);
    o[0] = make_float4(mean, invstd, g, bt);
    o[1] = make_float4(s1 / m, s2 / m, g * invstd, 0.f);
  }
}

// The same constants from the two sums handed over by the kernel that produced dY (sums[k] = {sum g, sum g xhat}).
__global__ __launch_bounds__(256) void bn_bwd_coef_sums_kernel(const float* __restrict__ sums, const float* __restrict__ gamma,
                                                               const float* __restrict__ beta, const float* __restrict__ mean,
                                                               const float* __restrict__ invstd, float* __restrict__ dgamma,
                                                               float* __restrict__ dbeta, float* __restrict__ coef, int n, float m) {
  const int k = blockIdx.x * 256 + threadIdx.x;
  if (k >= n) return;
  const float2 s = *reinterpret_cast<const float2*>(sums + (int64_t)k * 2);
  dbeta[k] = s.x;
  dgamma[k] = s.y;
  float4* o = reinterpret_cast<float4*>(coef + (int64_t)k * 8);
  o[0] = make_float4(mean[k], invstd[k], gamma[k], beta[k]);
  o[1] = make_float4(s.x / m, s.y / m, gamma[k] * invstd[k], 0.f);
}

template <typename T>
__global__ __launch_bounds__(BNL_C * BNL_N) void bn_bwd_linear_kernel(BnBwdArgs p) {
  __shared__ float red[BNL_N][BNL_C];
  const int tx = threadIdx.x % BNL_C, ty = threadIdx.x / BNL_C;
  const int c = blockIdx.x * BNL_C + tx, b = blockIdx.y;
  const bool live = c < p.C;
  const int cc = live ? c : p.C - 1;
  const int k = b * p.C + cc;
  const T* x = reinterpret_cast<const T*>(p.X) + b * p.xsb + cc;
  const T* dy = reinterpret_cast<const T*>(p.dY) + b * p.dysb + cc;
  T* dx = reinterpret_cast<T*>(p.dX) + b * p.dxsb + cc;
  const float mean = p.save_mean[k], invstd = p.save_invstd[k], g = p.gamma[k], bt = p.beta[k];
  float s1 = 0.f, s2 = 0.f;
  for (int n = ty; n < p.Nb; n += BNL_N) {
    const float xh = (Elem<T>::load(x + n * p.xsn) - mean) * invstd;
    const float gr = Elem<T>::load(dy + n * p.dysn) * act_grad(fmaf(g, xh, bt), p.act, p.slope);
    s1 += gr;
    s2 = fmaf(gr, xh, s2);
  }
  s1 = bnl_reduce(s1, red, tx, ty);
  s2 = bnl_reduce(s2, red, tx, ty);
  if (live && ty == 0) {
    p.dbeta[k] = s1;
    p.dgamma[k] = s2;
  }
  const float m = (float)p.Nb, mb = s1 / m, mg = s2 / m, sc = g * invstd;
  float s3 = 0.f;
  for (int n = ty; n < p.Nb; n += BNL_N) {
    const float xh = (Elem<T>::load(x + n * p.xsn) - mean) * invstd;
    const float gr = Elem<T>::load(dy + n * p.dysn) * act_grad(fmaf(g, xh, bt), p.act, p.slope);
    const T o = Elem<T>::from_f32(sc * (gr - mb - xh * mg));
    if (live) dx[n * p.dxsn] = o;
    s3 += Elem<T>::to_f32(o);
  }
  if (p.dx_sum) {                        // uniform over the grid
    s3 = bnl_reduce(s3, red, tx, ty);
    if (live && ty == 0) p.dx_sum[k] = s3;
  }
}

// Pieces of a channel per thread.
int held_pieces(int Nb, int L, int nt) { return (int)(((int64_t)Nb * ((L + 3) / 4) + nt - 1) / nt); }

// Byte offsets within a channel fit 32 bits.
template <typename T> bool held_rows_ok(int Nb, int L, int64_t sn0, int64_t sn1) {
  const int64_t limit = (int64_t)1 << 32, far = (sn0 > sn1 ? sn0 : sn1);
  return sn0 >= 0 && sn1 >= 0 && far < limit / Nb && ((int64_t)(Nb - 1) * far + L) * (int64_t)sizeof(T) < limit;
}

// How many pieces a thread holds.  All of a channel if they fit with two 1024-thread workgroups per compute unit, else what
// does: us with nothing held -> now, and what the other choice takes:
//   forward   bf16 6 x 16 x 2500, 2048 channels 538 -> 446, 128 channels 31 -> 26; 8 x 32 x 2500, 64 channels 39 -> 28; fp32 4 x 32 x 2500, 128 channels 81 -> 69 with 9 of
//             20 held, 76 with all 20 and one workgroup per unit, which wins where all channels run at once: 64 channels
//             38 -> 27, 34 with 9.
//   backward  the same tensors: 741 -> 588 (777 with both operands in registers and one workgroup per unit), 50 -> 38,
//             62 -> 54; fp32 62 -> 52 and 155 -> 126 with 10 of 20 held in registers, 56 and 137 with 5 in LDS,
//             which wins where 5 are most of the channel (32 x 1024: 41 against 43).
// Past 40 pieces too little of a channel is held to pay for the wavefronts (2 x 64 channels of 100 x 4096 bf16: forward
// 77 us with nothing held, 95 with 20 of 100, backward 125 and 131; elsewhere 61 and 108 with nothing held, 80 and 117 with
// the general activation in the loop).
constexpr int HELD_MOST = 40;
template <typename T, int NT>
void launch_bn_fwd(const BnFwdArgs& a, dim3 grid, hipStream_t st) {
  constexpr int HALF = sizeof(T) == 2 ? 20 : 9, FULL = sizeof(T) == 2 ? HALF : 20;
  const int per = a.Y ? held_pieces(a.Nb, a.L, NT) : 0;            // statistics alone: read once
#define HFTA_HELD(N) hipLaunchKernelGGL((bn_fwd_conv_kernel<T, 4, NT, N>), grid, dim3(NT), 0, st, a, per)
  if (per == 0 || per > HELD_MOST || !held_rows_ok<T>(a.Nb, a.L, a.xsn, 0)) HFTA_HELD(0);
  else if (per <= 4) HFTA_HELD(4);
  else if (per <= HALF / 2) HFTA_HELD(HALF / 2);
  else if (NT == 256 || per <= HALF || (int)(grid.x * grid.y) > persistent_blocks()) HFTA_HELD(HALF);
  else HFTA_HELD((NT == 256 ? HALF : FULL));
#undef HFTA_HELD
}
template <typename T, int NT>
void launch_bn_bwd(const BnBwdArgs& a, dim3 grid, hipStream_t st) {
  constexpr int W = (int)sizeof(T), REGS = 10;
  const int per = held_pieces(a.Nb, a.L, NT);
#define HFTA_HELD(N, XL) hipLaunchKernelGGL((bn_bwd_conv_kernel<T, 4, NT, N, XL>), grid, dim3(NT), 0, st, a, per)
  if (per > HELD_MOST || !held_rows_ok<T>(a.Nb, a.L, a.xsn, a.dysn)) HFTA_HELD(0, false);
  else if constexpr (NT == 256) {
    if (per <= 4) HFTA_HELD(4, false);
    else if (per <= 20 / W) HFTA_HELD(20 / W, false);
    else HFTA_HELD(32 / W, false);
  } else if constexpr (W == 2) {
    if (per <= 4) HFTA_HELD(4, false);
    else HFTA_HELD(10, true);
  } else {
    if (per <= REGS) HFTA_HELD(5, true);
    else HFTA_HELD(REGS, false);
  }
#undef HFTA_HELD
}
// The kernel of the row form: aligned four-element pieces (v4); single elements in order, staged in LDS where the channel fits,
// else from memory.  us with the element loads from memory -> staged: 6 x 16 x 2497 points bf16, 2048 channels forward 1766 -> 605,
// backward 2435 -> 1294, 128 channels 116 -> 45 and 157 -> 87, 6 x 24 x 607, 128 channels 49 -> 24 and 69 -> 48.  Memory stays where
// a thread has few elements (2 x 5 x 331 backward 9.5, staged 11.7) and for the fp32 backward, whose elements are a lane's four
// bytes either way (3 x 13 x 1023, 128 channels 28.2, staged 29.0; the forward, which reads them twice, 21.4 -> 18.4).
constexpr int ODD_MIN = 8;                               // elements per thread from which a channel is staged
template <typename T>
void launch_bn_fwd_rows(const BnFwdArgs& a, int B, bool v4, hipStream_t st) {
  const dim3 grid((unsigned)a.C, (unsigned)B);
  const int64_t bytes = (int64_t)a.Nb * ((a.L + 3) / 4) * 4 * (int64_t)sizeof(T);      // staged
  const bool big = bn_wide_block((int64_t)a.Nb * a.L * (int64_t)sizeof(T));
  if (v4) big ? launch_bn_fwd<T, 1024>(a, grid, st) : launch_bn_fwd<T, 256>(a, grid, st);
  else if (a.L >= 4 && bytes <= STAGE_FULL && (int64_t)a.Nb * a.L >= ODD_MIN * (big ? 1024 : 256)) {
#define HFTA_ODD(NT, N) hipLaunchKernelGGL((bn_fwd_odd_kernel<T, NT, N>), grid, dim3(NT), 0, st, a)
    if (big && bytes <= STAGE_HALF) HFTA_ODD(1024, STAGE_HALF);
    else if (big) HFTA_ODD(1024, STAGE_FULL);
    else if (bytes <= STAGE_SMALL) HFTA_ODD(256, STAGE_SMALL);
    else if (bytes <= STAGE_MID) HFTA_ODD(256, STAGE_MID);
    else HFTA_ODD(256, STAGE_HALF);                      // 32 KB at most; rows of five elements take eight places: 52
#undef HFTA_ODD
  } else if (big) hipLaunchKernelGGL((bn_fwd_conv_kernel<T, 1, 1024, 0>), grid, dim3(1024), 0, st, a, 0);
  else hipLaunchKernelGGL((bn_fwd_conv_kernel<T, 1, 256, 0>), grid, dim3(256), 0, st, a, 0);
}
template <typename T>
void launch_bn_bwd_rows(const BnBwdArgs& a, int B, bool v4, hipStream_t st) {
  const dim3 grid((unsigned)a.C, (unsigned)B);
  const int64_t bytes = 2 * (int64_t)a.Nb * ((a.L + 3) / 4) * 4 * (int64_t)sizeof(T);      // staged
  const bool big = bn_wide_block((int64_t)a.Nb * a.L * (int64_t)sizeof(T));
  if (v4) {
    big ? launch_bn_bwd<T, 1024>(a, grid, st) : launch_bn_bwd<T, 256>(a, grid, st);
    return;
  }
  if constexpr (sizeof(T) == 2) {
    if (a.L >= 4 && bytes <= STAGE_FULL && (int64_t)a.Nb * a.L >= ODD_MIN * (big ? 1024 : 256)) {
#define HFTA_ODD(NT, N) hipLaunchKernelGGL((bn_bwd_odd_kernel<T, NT, N>), grid, dim3(NT), 0, st, a)
      // (rows of five elements take eight places: a small channel can need more than its 2 x 32 KB)
      if (big && bytes <= STAGE_HALF) HFTA_ODD(1024, STAGE_HALF);
      else if (big) HFTA_ODD(1024, STAGE_FULL);
      else if (bytes <= STAGE_SMALL) HFTA_ODD(256, STAGE_SMALL);
      else if (bytes <= STAGE_MID) HFTA_ODD(256, STAGE_MID);
      else if (bytes <= STAGE_HALF) HFTA_ODD(256, STAGE_HALF);
      else HFTA_ODD(256, STAGE_FULL);
#undef HFTA_ODD
      return;
    }
  }
  if (big) hipLaunchKernelGGL((bn_bwd_conv_kernel<T, 1, 1024, 0, false>), grid, dim3(1024), 0, st, a, 0);
  else hipLaunchKernelGGL((bn_bwd_conv_kernel<T, 1, 256, 0, false>), grid, dim3(256), 0, st, a, 0);
}

bool vec_ok(const void* p, const int64_t* s, int L, int dtype) {
  const int es = (int)dtype_size(dtype);
  const size_t bytes = 4 * es;
  return L % 4 == 0 && reinterpret_cast<uintptr_t>(p) % bytes == 0 && s[0] % 4 == 0 && s[1] % 4 == 0 && s[2] % 4 == 0;
}

// Evaluation mode: y = act(gamma (x - running_mean) / sqrt(running_var + eps) + beta), one read and one
// write; the channel's scale and shift are formed once per workgroup.
struct BnEvalArgs {
  const void* X; void* Y;
  const float* gamma; const float* beta; const float* running_mean; const float* running_var;
  int64_t xsb, xsn, xsc, ysb, ysn, ysc;
  int Nb, C, L, act;
  float eps, slope;
};

template <typename T, int VEC, int NT, bool RAG>
__global__ __launch_bounds__(NT) void bn_eval_conv_kernel(BnEvalArgs p) {
  const int c = blockIdx.x, b = blockIdx.y, k = b * p.C + c;
  const T* x = reinterpret_cast<const T*>(p.X) + b * p.xsb + c * p.xsc;
  T* y = reinterpret_cast<T*>(p.Y) + b * p.ysb + c * p.ysc;
  const float mean = p.running_mean[k];
  const float scale = p.gamma[k] * (1.0f / sqrtf(p.running_var[k] + p.eps)), bt = p.beta[k];
  const int chunks = RAG ? (p.L + VEC - 1) / VEC : p.L / VEC;
  for (RowWalk w(chunks, NT); w.n < p.Nb; w.step()) {
    float v[VEC];
    load_piece<T, VEC, RAG>(x + w.n * p.xsn, w.ch, p.L, v);
#pragma unroll
    for (int e = 0; e < VEC; ++e) v[e] = bn_act(fmaf(scale, v[e] - mean, bt), p.act, p.slope);
    store_piece<T, VEC, RAG>(y + w.n * p.ysn, w.ch, p.L, v);
  }
}

template <typename T>
__global__ __launch_bounds__(BNL_C * BNL_N) void bn_eval_linear_kernel(BnEvalArgs p) {
  const int tx = threadIdx.x % BNL_C, ty = threadIdx.x / BNL_C;
  const int c = blockIdx.x * BNL_C + tx, b = blockIdx.y;
  if (c >= p.C) return;
  const int k = b * p.C + c;
  const T* x = reinterpret_cast<const T*>(p.X) + b * p.xsb + c;
  T* y = reinterpret_cast<T*>(p.Y) + b * p.ysb + c;
  const float mean = p.running_mean[k];
  const float scale = p.gamma[k] * (1.0f / sqrtf(p.running_var[k] + p.eps)), bt = p.beta[k];
  for (int n = ty; n < p.Nb; n += BNL_N)
    Elem<T>::store(y + n * p.ysn, bn_act(fmaf(scale, Elem<T>::load(x + n * p.xsn) - mean, bt), p.act, p.slope));
}

int layout_kind(const int64_t* s, int L) {
  if (s[3] == 1) return 1;                 // conv family
  if (L == 1 && s[2] == 1) return 2;       // linear family
  return 0;
}

}  // namespace


namespace hfta {
// see bn_stats_part_kernel; conv layout only, bf16 (the producer is the streaming convolution)
int bn_fwd_from_partials(int B, int Nb, int C, int L, int dtype, const void* X, const int64_t xs[4], const float* gamma,
                         const float* beta, float eps, float momentum, float* running_mean, float* running_var,
                         float* save_mean, float* save_invstd, void* Y, const int64_t ys[4], int act, float slope,
                         const float* part, int parts, const void* shift, hipStream_t st) {
  // Y == nullptr: statistics only (mean, invstd, running statistics); nothing of size [Nb, C, L] is touched
  if (dtype != HFTA_BF16 || B > 65535 || layout_kind(xs, L) != 1 || (Y && layout_kind(ys, L) != 1)) return HFTA_EUNSUPPORTED;
  BnFwdArgs a{X, Y, gamma, beta, running_mean, running_var, save_mean, save_invstd,
              xs[0], xs[1], xs[2], Y ? ys[0] : 0, Y ? ys[1] : 0, Y ? ys[2] : 0, Nb, C, L, act, eps, momentum, slope};
  const bf16_raw* sv = (const bf16_raw*)shift;
  hipLaunchKernelGGL(bn_stats_part_kernel, dim3((unsigned)((C + BNS_C - 1) / BNS_C), (unsigned)B), dim3(BNS_C * BNS_P), 0, st, a, part,
                     parts, sv);
  const int rc = launch_status();
  if (!Y || rc != HFTA_OK) return rc;
  const dim3 grid((unsigned)C, (unsigned)B);
  const bool v4 = vec_ok(X, xs, L, dtype) && vec_ok(Y, ys, L, dtype);
  const bool big = bn_wide_block((int64_t)Nb * L * dtype_size(dtype));
#define HFTA_BN_NORM(T, V, R) \
  do { if (big) hipLaunchKernelGGL((bn_apply_conv_kernel<T, V, 1024, R>), grid, dim3(1024), 0, st, a); \
       else hipLaunchKernelGGL((bn_apply_conv_kernel<T, V, 256, R>), grid, dim3(256), 0, st, a); } while (0)
  if (v4) HFTA_BN_NORM(bf16_raw, 4, false);
  else if (L >= 4) HFTA_BN_NORM(bf16_raw, 4, true);
  else HFTA_BN_NORM(bf16_raw, 1, false);
#undef HFTA_BN_NORM
  return launch_status();
}

// Training statistics of a conv-layout tensor alone (mean, invstd, running statistics): the first pass of
// the forward kernel, for a consumer that normalises on load.
int bn_stats_conv(int B, int Nb, int C, int L, int dtype, const void* X, const int64_t xs[4], const float* gamma,
                  const float* beta, float eps, float momentum, float* running_mean, float* running_var,
                  float* save_mean, float* save_invstd, hipStream_t st) {
  if (B > 65535 || layout_kind(xs, L) != 1) return HFTA_EUNSUPPORTED;
  BnFwdArgs a{X, nullptr, gamma, beta, running_mean, running_var, save_mean, save_invstd,
              xs[0], xs[1], xs[2], 0, 0, 0, Nb, C, L, HFTA_ACT_NONE, eps, momentum, 0.f};
  const bool v4 = vec_ok(X, xs, L, dtype);
  if (dtype == HFTA_BF16) launch_bn_fwd_rows<bf16_raw>(a, B, v4, st);
  else launch_bn_fwd_rows<float>(a, B, v4, st);
  return launch_status();
}

// Reduction half of the training backward pass over the [Nb, B*C, L] layout: dgamma, dbeta and the
// per-channel constants (eight floats, see the kernel) for a consumer that applies them itself.
int bn_bwd_coef(int B, int Nb, int C, int L, int dtype, const void* X, const int64_t xs[4], const void* dY,
                const int64_t dys[4], const float* gamma, const float* beta, const float* save_mean,
                const float* save_invstd, float* dgamma, float* dbeta, float* coef, int act, float slope, hipStream_t st) {
  if (B > 65535 || layout_kind(xs, L) != 1 || layout_kind(dys, L) != 1) return HFTA_EUNSUPPORTED;
  BnBwdArgs a{X, dY, nullptr, gamma, beta, save_mean, save_invstd, dgamma, dbeta, nullptr,
              xs[0], xs[1], xs[2], dys[0], dys[1], dys[2], 0, 0, 0, Nb, C, L, act, slope};
  const dim3 grid((unsigned)C, (unsigned)B);
  const bool v4 = vec_ok(X, xs, L, dtype) && vec_ok(dY, dys, L, dtype);
  const bool big = bn_wide_block((int64_t)Nb * L * dtype_size(dtype));
#define HFTA_BN_COEF(T, V, R) \
  do { if (big) hipLaunchKernelGGL((bn_bwd_conv_coef_kernel<T, V, 1024, R>), grid, dim3(1024), 0, st, a, coef); \
       else hipLaunchKernelGGL((bn_bwd_conv_coef_kernel<T, V, 256, R>), grid, dim3(256), 0, st, a, coef); } while (0)
  HFTA_BN_BY_ROWS(HFTA_BN_COEF);
#undef HFTA_BN_COEF
  return launch_status();
}
int bn_bwd_coef_from_sums(int B, int Nb, int C, int L, const float* sums, const float* gamma, const float* beta,
                          const float* save_mean, const float* save_invstd, float* dgamma, float* dbeta, float* coef,
                          hipStream_t st) {
  const int n = B * C;
  hipLaunchKernelGGL(bn_bwd_coef_sums_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, sums, gamma, beta, save_mean,
                     save_invstd, dgamma, dbeta, coef, n, (float)Nb * (float)L);
  return launch_status();
}
}  // namespace hfta

extern "C" {

int hfta_bn_fwd(int B, int Nb, int C, int L, int dtype, const void* X, const int64_t xs[4], const float* gamma,
                const float* beta, float eps, float momentum, float* running_mean, float* running_var,
                float* save_mean, float* save_invstd, void* Y, const int64_t ys[4], int act, float act_slope,
                void* stream) {
  if (B <= 0 || Nb <= 0 || C <= 0 || L <= 0 || !valid_dtype(dtype) || !X || !xs || !gamma || !beta || !save_mean ||
      !save_invstd || !Y || !ys || !(eps >= 0.f))
    return HFTA_EINVAL;
  if ((running_mean == nullptr) != (running_var == nullptr)) return HFTA_EINVAL;
  if (act != HFTA_ACT_NONE && act != HFTA_ACT_RELU && act != HFTA_ACT_LEAKY) return HFTA_EUNSUPPORTED;
  if (B > 65535) return HFTA_EUNSUPPORTED;
  const bool lin = (L == 1 && xs[2] == 1 && ys[2] == 1);
  const int kx = lin ? 2 : layout_kind(xs, L), ky = lin ? 2 : layout_kind(ys, L);
  if (kx == 0 || kx != ky) return HFTA_EUNSUPPORTED;
  BnFwdArgs a{X, Y, gamma, beta, running_mean, running_var, save_mean, save_invstd,
              xs[0], xs[1], xs[2], ys[0], ys[1], ys[2], Nb, C, L, act, eps, momentum, act_slope};
  hipStream_t st = as_stream(stream);
  if (kx == 2) {
    dim3 grid((unsigned)((C + BNL_C - 1) / BNL_C), (unsigned)B);
    if (dtype == HFTA_BF16) hipLaunchKernelGGL(bn_fwd_linear_kernel<bf16_raw>, grid, dim3(BNL_C * BNL_N), 0, st, a);
    else hipLaunchKernelGGL(bn_fwd_linear_kernel<float>, grid, dim3(BNL_C * BNL_N), 0, st, a);
    return launch_status();
  }
  const bool v4 = vec_ok(X, xs, L, dtype) && vec_ok(Y, ys, L, dtype);
  if (dtype == HFTA_BF16) launch_bn_fwd_rows<bf16_raw>(a, B, v4, st);
  else launch_bn_fwd_rows<float>(a, B, v4, st);
  return launch_status();
}

int hfta_bn_apply_fwd(int B, int Nb, int C, int L, int dtype, const void* X, const int64_t xs[4], const float* gamma,
                      const float* beta, const float* mean, const float* invstd, void* Y, const int64_t ys[4], int act,
                      float act_slope, void* stream) {
  if (B <= 0 || Nb <= 0 || C <= 0 || L <= 0 || !valid_dtype(dtype) || !X || !xs || !gamma || !beta || !mean || !invstd ||
      !Y || !ys)
    return HFTA_EINVAL;
  if (act != HFTA_ACT_NONE && act != HFTA_ACT_RELU && act != HFTA_ACT_LEAKY) return HFTA_EUNSUPPORTED;
  if (B > 65535 || layout_kind(xs, L) != 1 || layout_kind(ys, L) != 1) return HFTA_EUNSUPPORTED;
  BnFwdArgs a{X, Y, gamma, beta, nullptr, nullptr, const_cast<float*>(mean), const_cast<float*>(invstd),
              xs[0], xs[1], xs[2], ys[0], ys[1], ys[2], Nb, C, L, act, 0.f, 0.f, act_slope};
  hipStream_t st = as_stream(stream);
  const dim3 grid((unsigned)C, (unsigned)B);
  const bool v4 = vec_ok(X, xs, L, dtype) && vec_ok(Y, ys, L, dtype);
  const bool big = bn_wide_block((int64_t)Nb * L * dtype_size(dtype));
#define HFTA_BN_APPLY(T, V, R) \
  do { if (big) hipLaunchKernelGGL((bn_apply_conv_kernel<T, V, 1024, R>), grid, dim3(1024), 0, st, a); \
       else hipLaunchKernelGGL((bn_apply_conv_kernel<T, V, 256, R>), grid, dim3(256), 0, st, a); } while (0)
  HFTA_BN_BY_ROWS(HFTA_BN_APPLY);
#undef HFTA_BN_APPLY
  return launch_status();
}

int hfta_bn_eval_fwd(int B, int Nb, int C, int L, int dtype, const void* X, const int64_t xs[4], const float* gamma,
                     const float* beta, const float* running_mean, const float* running_var, float eps, void* Y,
                     const int64_t ys[4], int act, float act_slope, void* stream) {
  if (B <= 0 || Nb <= 0 || C <= 0 || L <= 0 || !valid_dtype(dtype) || !X || !xs || !gamma || !beta || !running_mean ||
      !running_var || !Y || !ys || !(eps >= 0.f))
    return HFTA_EINVAL;
  if (act != HFTA_ACT_NONE && act != HFTA_ACT_RELU && act != HFTA_ACT_LEAKY) return HFTA_EUNSUPPORTED;
  if (B > 65535) return HFTA_EUNSUPPORTED;
  const bool lin = (L == 1 && xs[2] == 1 && ys[2] == 1);
  const int kx = lin ? 2 : layout_kind(xs, L), ky = lin ? 2 : layout_kind(ys, L);
  if (kx == 0 || kx != ky) return HFTA_EUNSUPPORTED;
  BnEvalArgs a{X, Y, gamma, beta, running_mean, running_var, xs[0], xs[1], xs[2], ys[0], ys[1], ys[2],
               Nb, C, L, act, eps, act_slope};
  hipStream_t st = as_stream(stream);
  if (kx == 2) {
    dim3 grid((unsigned)((C + BNL_C - 1) / BNL_C), (unsigned)B);
    if (dtype == HFTA_BF16) hipLaunchKernelGGL(bn_eval_linear_kernel<bf16_raw>, grid, dim3(BNL_C * BNL_N), 0, st, a);
    else hipLaunchKernelGGL(bn_eval_linear_kernel<float>, grid, dim3(BNL_C * BNL_N), 0, st, a);
    return launch_status();
  }
  dim3 grid((unsigned)C, (unsigned)B);
  const bool v4 = vec_ok(X, xs, L, dtype) && vec_ok(Y, ys, L, dtype);
  const bool big = bn_wide_block((int64_t)Nb * L * dtype_size(dtype));
#define HFTA_BN_EVAL(T, V, R) \
  do { if (big) hipLaunchKernelGGL((bn_eval_conv_kernel<T, V, 1024, R>), grid, dim3(1024), 0, st, a); \
       else hipLaunchKernelGGL((bn_eval_conv_kernel<T, V, 256, R>), grid, dim3(256), 0, st, a); } while (0)
  HFTA_BN_BY_ROWS(HFTA_BN_EVAL);
#undef HFTA_BN_EVAL
  return launch_status();
}

int hfta_bn_bwd(int B, int Nb, int C, int L, int dtype, const void* X, const int64_t xs[4], const void* dY,
                const int64_t dys[4], const float* gamma, const float* beta, const float* save_mean,
                const float* save_invstd, void* dX, const int64_t dxs[4], float* dgamma, float* dbeta, float* dx_sum,
                int act, float act_slope, void* stream) {
  if (B <= 0 || Nb <= 0 || C <= 0 || L <= 0 || !valid_dtype(dtype) || !X || !xs || !dY || !dys || !gamma || !beta ||
      !save_mean || !save_invstd || !dX || !dxs || !dgamma || !dbeta)
    return HFTA_EINVAL;
  if (act != HFTA_ACT_NONE && act != HFTA_ACT_RELU && act != HFTA_ACT_LEAKY) return HFTA_EUNSUPPORTED;
  if (B > 65535) return HFTA_EUNSUPPORTED;
  const bool lin = (L == 1 && xs[2] == 1 && dys[2] == 1 && dxs[2] == 1);
  const int kx = lin ? 2 : layout_kind(xs, L);
  if (kx == 0 || (!lin && (layout_kind(dys, L) != kx || layout_kind(dxs, L) != kx))) return HFTA_EUNSUPPORTED;
  BnBwdArgs a{X, dY, dX, gamma, beta, save_mean, save_invstd, dgamma, dbeta, dx_sum,
              xs[0], xs[1], xs[2], dys[0], dys[1], dys[2], dxs[0], dxs[1], dxs[2], Nb, C, L, act, act_slope};
  hipStream_t st = as_stream(stream);
  if (kx == 2) {
    dim3 grid((unsigned)((C + BNL_C - 1) / BNL_C), (unsigned)B);
    if (dtype == HFTA_BF16) hipLaunchKernelGGL(bn_bwd_linear_kernel<bf16_raw>, grid, dim3(BNL_C * BNL_N), 0, st, a);
    else hipLaunchKernelGGL(bn_bwd_linear_kernel<float>, grid, dim3(BNL_C * BNL_N), 0, st, a);
    return launch_status();
  }
  const bool v4 = vec_ok(X, xs, L, dtype) && vec_ok(dY, dys, L, dtype) && vec_ok(dX, dxs, L, dtype);
  if (dtype == HFTA_BF16) launch_bn_bwd_rows<bf16_raw>(a, B, v4, st);
  else launch_bn_bwd_rows<float>(a, B, v4, st);
  return launch_status();
}

}  // extern "C"
