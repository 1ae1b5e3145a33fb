// Backward of  k=1 Conv1d -> BatchNorm (+ activation) -> max over points  in fp32, without the convolution's output or its
// gradient: what conv_bn_pool.hip does for bf16, with every product and sum at fp32 or better.
//
// With hits (the argmax of each sample and channel, where the pooled gradient enters) and, per channel, sc = gamma invstd,
// mb = dbeta / m, mg = dgamma / m, m = Nb L, BatchNorm's backward is  dz = [hits s] - sc mb - p1 (z - mean),  p1 = sc mg invstd.
// With z = W x + bias:
//   dX = [hits s W] - v - G x,   G = sum_c p1 W_c W_c^T,   v = sum_c W_c (sc mb - p1 (mean - bias))
//   dW_c = sum_hits s x - m (sc mb E[x] + p1 Cov(x) W_c)
// G, v, Cov(x) W_c and the channel sums are formed in double; G x is the fp32 product of gemm_f32.hip, with the hits added
// while its output is staged; Cov(x) is a product of the same kind over the points.  Against the chain of stored operators the
// 1024-channel tensors of a 128 -> 1024 layer (1.3 GB each on 4 x 32 x 2500 points) are neither written nor read.
// On 4 x 32 x 2500 points, 128 -> 1024 channels: forward 858 -> 598 us (the product without its stores), backward 1567 -> 314
// (moments 107, dX 123, the rest 84); dX 2.2e-7 -> 5.7e-8 and dW 5.9e-7 -> 6.6e-8 off float64.
// Bound: x read twice and dX written once; the hits, a chain of loads per tile, and the moments' phases take longer.
#include <algorithm>
#include "gemm_pf.h"
#include "f32_split.h"
#include "bn_common.h"
#include "hit_sort.h"

namespace hfta {
bool gemm_f32_big_tiles(int M, int N, int64_t G);
size_t pool32_fwd_bytes(int B, int Nb, int Ci, int Co, int L);
}

using namespace hfta;

namespace {

typedef float f32x4_u __attribute__((ext_vector_type(4), aligned(4)));

struct Pool32Args {
  const float* X; const float* W; const float* bias; const float* zhit; const float* dV; const int32_t* idx;
  const float* gamma; const float* beta; const float* mean; const float* invstd;
  float* dW; float* dbias; float* dgamma; float* dbeta;
  int64_t xsb, xsn, xsc, vsb, vsn, vsc;
  int B, Nb, Ci, Co, L, act, tiles;
  float slope;
  uint32_t x_extent;  // bytes of one sample's x
  // workspace
  double* c1;         // [B][Co] p1
  double* c0;         // [B][Co] sc mb
  double* cv;         // [B][Co] sc mb - p1 (mean - bias)
  float* s;           // [B][Nb][Co] a hit's weight
  uint32_t* skey; float* sval; int* toff;
  float* negG;        // [B][Ci][Ci]
  float* negv;        // [B][Ci]
  float* XXpart;      // [chunks][B][Ci][Ci] sums of products about the means of groups of 64 tiles and less
  double* gm;         // [chunks * groups][B][Ci] those means
  double* gn;         // [chunks * groups][B] a group's points
  double* cov;        // [B][Ci][Ci] Cov(x)
  double* ex;         // [B][Ci] E[x]
  int chunks, groups; // groups: of a chunk, the last may be empty
  float* xg;          // [B][Nb][Co][Ci] the input at each hit
};

// ---- per channel: dbeta, dgamma and what follows from them.  64 channels a workgroup, samples over the wavefronts ----
constexpr int C32_WAVES = 8;
__global__ __launch_bounds__(C32_WAVES * 64) void pool32_coef_kernel(Pool32Args p) {
  __shared__ double red[C32_WAVES][2][64];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int c = blockIdx.x * 64 + lane, b = blockIdx.y, k = b * p.Co + c;
  const bool live = c < p.Co;
  float mean = 0.f, invstd = 0.f, g = 0.f, bt = 0.f;
  if (live) { mean = p.mean[k]; invstd = p.invstd[k]; g = p.gamma[k]; bt = p.beta[k]; }
  const float sc = g * invstd;
  double s1 = 0.0, s2 = 0.0;
  if (live) {
#pragma unroll 4
    for (int n = wave; n < p.Nb; n += C32_WAVES) {
      const int64_t o = ((int64_t)b * p.Nb + n) * p.Co + c;
      const float xh = (p.zhit[o] - mean) * invstd;
      const float gr = p.dV[b * p.vsb + n * p.vsn + c * p.vsc] * act_grad(fmaf(g, xh, bt), p.act, p.slope);
      s1 += (double)gr;
      s2 += (double)gr * (double)xh;
      p.s[o] = gr * sc;
    }
  }
  red[wave][0][lane] = s1;
  red[wave][1][lane] = s2;
  __syncthreads();
  if (wave != 0 || !live) return;
  for (int w = 1; w < C32_WAVES; ++w) { s1 += red[w][0][lane]; s2 += red[w][1][lane]; }
  p.dbeta[k] = (float)s1;
  p.dgamma[k] = (float)s2;
  if (p.dbias) p.dbias[k] = 0.f;                          // a bias in front of a BatchNorm: gradient exactly zero
  const double m = (double)p.Nb * (double)p.L;
  p.c0[k] = (double)sc * s1 / m;
  p.c1[k] = (double)sc * (double)invstd * s2 / m;
  p.cv[k] = p.c0[k] - p.c1[k] * ((double)mean - (p.bias ? (double)p.bias[k] : 0.0));
}

// ---- workgroups 0 .. B Nb - 1: the hits of a sample sorted by point; then -G by 32 x 32 tiles, sixteen shares of the channels
// ---- added in a fixed order; then -v.  Chains of loads: many channels in flight (four shares, two loads a channel: 87 us) ----
__global__ __launch_bounds__(HIT_THREADS) void pool32_prep_kernel(Pool32Args p, int P) {
  __shared__ union { uint32_t key[2][HIT_THREADS]; double g[8][16][64]; double v[8][128]; } sh;
  const int t = threadIdx.x;
  int id = (int)blockIdx.x - p.B * p.Nb;
  if (id < 0) {
    const int n = (int)blockIdx.x % p.Nb, b = (int)blockIdx.x / p.Nb;
    const int64_t row = (int64_t)b * p.Nb + n;
    sort_hits(p.idx + b * p.vsb + n * p.vsn, p.vsc, p.s + row * p.Co, p.skey + row * p.Co, p.sval + row * p.Co, p.toff + row * (p.tiles + 1),
              p.Co, p.L, sh.key, P, p.tiles);
    return;
  }
  const int T = (p.Ci + 31) / 32, b = id % p.B;
  id /= p.B;
  const float* W = p.W + (int64_t)b * p.Co * p.Ci;
  if (id < T * T) {
    const double* c1 = p.c1 + (int64_t)b * p.Co;
    const int lane = t & 63, w = t >> 6, i = id / T * 32 + (lane >> 3) * 4, j = id % T * 32 + (lane & 7) * 4;   // Ci % 4 == 0
    const bool in = i < p.Ci && j < p.Ci;
    double a[4][4];
#pragma unroll
    for (int e = 0; e < 16; ++e) a[e >> 2][e & 3] = 0.0;
    if (in) {
#pragma unroll 8
      for (int c = w; c < p.Co; c += 16) {
        const f32x4_u wi = *reinterpret_cast<const f32x4_u*>(W + (int64_t)c * p.Ci + i), wj = *reinterpret_cast<const f32x4_u*>(W + (int64_t)c * p.Ci + j);
        const double k = c1[c];
#pragma unroll
        for (int x = 0; x < 4; ++x) {
          const double kx = k * (double)wi[x];
#pragma unroll
          for (int y = 0; y < 4; ++y) a[x][y] = fma(kx, (double)wj[y], a[x][y]);
        }
      }
    }
    for (int half = 8; half > 0; half >>= 1) {             // shares w and w + half
      if (w >= half && w < 2 * half) {
#pragma unroll
        for (int e = 0; e < 16; ++e) sh.g[w - half][e][lane] = a[e >> 2][e & 3];
      }
      __syncthreads();
      if (w < half) {
#pragma unroll
        for (int e = 0; e < 16; ++e) a[e >> 2][e & 3] += sh.g[w][e][lane];
      }
      __syncthreads();
    }
    if (w == 0 && in) {
      float* G = p.negG + (int64_t)b * p.Ci * p.Ci;
#pragma unroll
      for (int e = 0; e < 16; ++e) G[(int64_t)(i + (e >> 2)) * p.Ci + j + (e & 3)] = (float)-a[e >> 2][e & 3];
    }
    return;
  }
  const int i = t & 127, q = t >> 7;                       // Ci <= 128; eight shares of the channels
  double a = 0.0;
  if (i < p.Ci) {
#pragma unroll 16
    for (int c = q; c < p.Co; c += 8) a = fma((double)W[(int64_t)c * p.Ci + i], p.cv[(int64_t)b * p.Co + c], a);
  }
  sh.v[q][i] = a;
  __syncthreads();
  if (q == 0 && i < p.Ci) {
    for (int w = 1; w < 8; ++w) a += sh.v[w][i];
    p.negv[(int64_t)b * p.Ci + i] = (float)-a;
  }
}

// ---- second moments of x, and the input at each hit, in one pass over x.  A workgroup takes a share of a model's 64-point
// ---- tiles; each is loaded once (16-byte pieces, the next tile's in flight), parked as it is for the hits (a column of x is
// ---- Ci cache lines in memory) and, about its own mean, as three bf16 planes that are both operands of the product.  The means of
// ---- 64 tiles, or of what the share has left, about their own mean and times the root of their points, are one more tile.  So the
// ---- sums never hold more than the points' own spread, whatever their order: XX / m - E[x]^2 loses what a mean that is large
// ---- against the spread has in digits (dW's error 8e-5 for 3e-5 of the stored operators at a mean of ten spreads), and one
// ---- reference for a model, its first 64 points, what the others lie off by (64 x 8 clouds padded in front with a point five
// ---- spreads away: 7.5e-6 for 5.3e-7 of the stored operators, now 1.4e-7).  The six products of two splits as in gemm_f32.hip.
// ---- 4 x 32 x 2500 x 128: 107 us (98 about one reference), of 5.3 a tile 1.9 are its bytes and 1.4 its matrix instructions: the
// ---- phases of the one workgroup per compute unit (eight wavefronts, 248 registers) follow each other.  Two workgroups spill
// ---- (136-317 us); a pass for the hits and the product over the points on the general kernel took 150. ----
constexpr int MM_PTS = 64, MM_THREADS = 512, MM_WN = MM_THREADS / 128, MM_NJ = 4 / MM_WN, MM_ROWS = MM_THREADS / 16, MM_H = 128 / MM_ROWS, MM_PLANE = 128 * MM_PTS * 2;
__device__ __forceinline__ int mm_swz(int r) { return (r ^ (r >> 3)) & 7; }
// the sum over sixteen lanes, the same bits in each
template <int N> __device__ __forceinline__ float mm_ror(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x120 + N, 0xf, 0xf, false));
}
__device__ __forceinline__ float mm_sum16(float v) {
  v += mm_ror<8>(v);
  v += mm_ror<4>(v);
  v += mm_ror<2>(v);
  return v + mm_ror<1>(v);
}
constexpr int MM_GROUP = MM_PTS, MM_PITCH = 129;           // means: tiles of a group, floats a tile
// tiles added up before they join the others: on channels correlated at 0.99, 66 tiles to a workgroup, dW is 8.9e-7 off float64
// (1.8e-6 without, the stored operators 1.0e-6), in the same time
constexpr int MM_RUN = 8;
__global__ __launch_bounds__(MM_THREADS, 2) void pool32_moments_kernel(Pool32Args p) {
  __shared__ __attribute__((aligned(16))) unsigned char planes[3 * MM_PLANE];
  __shared__ __attribute__((aligned(16))) float raw[128 * MM_PTS];     // 16-byte piece q of row r at q ^ (r & 15)
  __shared__ float means[MM_GROUP * MM_PITCH], count[MM_GROUP];        // of a group's tiles
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6, wm = wave / MM_WN, wn = wave % MM_WN;   // 2 x 4 wavefronts, 64 x 32 each
  const int chunk = blockIdx.x, b = blockIdx.y;
  const int per = (p.L + MM_PTS - 1) / MM_PTS, total = p.Nb * per;
  const int t0 = (int)((int64_t)total * chunk / p.chunks), t1 = (int)((int64_t)total * (chunk + 1) / p.chunks);
  const int row = t >> 4, piece = t & 15;                  // 32 rows x 16 pieces a pass, 4 passes
  // Pieces are loaded whole: what lies behind a row's end is the next row's or, out of range, zero, and takes no part.
  const float* xb = p.X + b * p.xsb;
  const uint32_t ldb = (uint32_t)(p.xsc * 4);
  float4 q[MM_H];
  auto fetch = [&](const float* src, int l) {
    const __amdgpu_buffer_rsrc_t rs = pf_rsrc(src, p.x_extent);
    const uint32_t off = l < p.L ? (uint32_t)row * ldb + (uint32_t)l * 4u : PF_OOB;
#pragma unroll
    for (int h = 0; h < MM_H; ++h) {
      const pf_u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(rs, (int)(row + MM_ROWS * h < p.Ci ? off + (uint32_t)(MM_ROWS * h) * ldb : PF_OOB), 0, 0);
      q[h] = make_float4(__uint_as_float(v.x), __uint_as_float(v.y), __uint_as_float(v.z), __uint_as_float(v.w));
    }
  };
  auto load = [&](int tile) {
    const int n = tile / per;
    fetch(xb + n * p.xsn, tile < t1 ? (tile - n * per) * MM_PTS + piece * 4 : p.L);
  };
  f32x16_t acc[2][MM_NJ], sum[2][MM_NJ];                   // of up to MM_RUN tiles, of all
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < MM_NJ; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[i][j][v] = sum[i][j][v] = 0.f;
  auto gather = [&]() {
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < MM_NJ; ++j)
#pragma unroll
        for (int v = 0; v < 16; ++v) { sum[i][j][v] += acc[i][j][v]; acc[i][j][v] = 0.f; }
  };
  int hlo, hhi;
  auto range = [&](int tile) {                             // of the hits of the 128-point tile that `tile` is half of
    const int tc = min(tile, t1 - 1), n = tc / per;
    const int* off = p.toff + ((int64_t)b * p.Nb + n) * (p.tiles + 1) + (((tc - n * per) * MM_PTS) >> 7);
    hlo = off[0];
    hhi = off[1];
  };
  load(t0);
  range(t0);
  auto park = [&](int r, const float4& c) {
    SplitSeen seen;                                        // (an infinity or a NaN reaches every result through the statistics)
    uint2 o[3];
    split4(c, o, seen);
    unsigned char* d = planes + r * (MM_PTS * 2) + (((piece >> 1) ^ mm_swz(r)) << 4) + (piece & 1) * 8;
#pragma unroll
    for (int i = 0; i < 3; ++i) *reinterpret_cast<uint2*>(d + i * MM_PLANE) = o[i];
  };
  auto frag = [&](int pl, int r0, int s) {
    const int r = r0 + (lane & 31);
    return *reinterpret_cast<const bf16x8_t*>(planes + pl * MM_PLANE + r * (MM_PTS * 2) + (((2 * s + (lane >> 5)) ^ mm_swz(r)) << 4));
  };
  // one block after the other, a tile's accumulators for one block only: registers.  A tile's sums start from zero, and so do
  // those of MM_RUN tiles: few roundings at the size of all.
  auto products = [&]() {
#pragma unroll
    for (int ij = 0; ij < 2 * MM_NJ; ++ij) {
      const int i = ij / MM_NJ, j = ij % MM_NJ;
      f32x16_t low, top;
#pragma unroll
      for (int v = 0; v < 16; ++v) low[v] = top[v] = 0.f;
#pragma unroll
      for (int s = 0; s < MM_PTS / 16; ++s) {
        bf16x8_t x[3], y[3];
#pragma unroll
        for (int pl = 0; pl < 3; ++pl) {
          x[pl] = frag(pl, wm * 64 + i * 32, s);
          y[pl] = frag(pl, (wn * MM_NJ + j) * 32, s);
        }
        constexpr int PA[5] = {2, 1, 0, 1, 0}, PB[5] = {0, 1, 2, 0, 1};
#pragma unroll
        for (int k = 0; k < 5; ++k) low = __builtin_amdgcn_mfma_f32_32x32x16_bf16(y[PB[k]], x[PA[k]], low, 0, 0, 0);
        top = __builtin_amdgcn_mfma_f32_32x32x16_bf16(y[0], x[0], top, 0, 0, 0);
      }
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[i][j][v] += top[v] + low[v];
    }
  };
  for (int tile = t0, group = 0; group < p.groups; ++group) {
    const int g0 = tile, g1 = min(tile + MM_GROUP, t1);
    for (; tile < g1; ++tile) {
      const int n = tile / per, l0 = (tile - n * per) * MM_PTS, have = p.L - (l0 + piece * 4);
      const float pts = (float)min(p.L - l0, MM_PTS), inv = __builtin_amdgcn_rcpf(pts);
      __syncthreads();                                     // the last tile is read
#pragma unroll
      for (int h = 0; h < MM_H; ++h) {
        const int r = row + MM_ROWS * h;
        *reinterpret_cast<float4*>(raw + r * MM_PTS + (piece ^ (r & 15)) * 4) = q[h];
        // (what is out of range has been loaded as zeros; the mean but for its rounding, 2^-23 of it)
        const float y = have > 1 ? q[h].y : 0.f, z = have > 2 ? q[h].z : 0.f, w = have > 3 ? q[h].w : 0.f;
        const float ref = mm_sum16((q[h].x + y) + (z + w)) * inv;
        if (piece == 0) means[(tile - g0) * MM_PITCH + r] = ref;
        park(r, make_float4(have > 0 ? q[h].x - ref : 0.f, have > 1 ? y - ref : 0.f, have > 2 ? z - ref : 0.f, have > 3 ? w - ref : 0.f));
      }
      if (t == 0) count[tile - g0] = pts;
      __syncthreads();
      load(tile + 1);
      const int64_t smp = (int64_t)b * p.Nb + n;
      const int h_lo = hlo, h_hi = hhi;                    // this tile's range of hits, and the first of them
      const uint32_t first = h_lo + lane < h_hi ? p.skey[smp * p.Co + h_lo + lane] : 0xffffffffu;
      range(tile + 1);
      products();
      if ((tile - g0) % MM_RUN == MM_RUN - 1) gather();
      // this tile's hits: those of its 128-point tile whose point is in it, in turn over the wavefronts
      for (int h0 = h_lo; h0 < h_hi; h0 += 64) {
        const uint32_t kl = h0 == h_lo ? first : h0 + lane < h_hi ? p.skey[smp * p.Co + h0 + lane] : 0xffffffffu;
        unsigned long long todo = __ballot((int)(kl >> 10) - l0 >= 0 && (int)(kl >> 10) - l0 < MM_PTS);
        for (int k = 0; todo; ++k, todo &= todo - 1) {
          if (k % (MM_THREADS / 64) != wave) continue;
          const uint32_t key = (uint32_t)__builtin_amdgcn_readlane((int)kl, __builtin_ctzll(todo));
          const int col = (int)(key >> 10) - l0;
          float* out = p.xg + (smp * p.Co + (key & 1023u)) * p.Ci;
#pragma unroll
          for (int r = lane; r < 128; r += 64)
            if (r < p.Ci) out[r] = raw[r * MM_PTS + (((col >> 2) ^ (r & 15)) << 2) + (col & 3)];
        }
      }
    }
    // the group's means as a tile
    const int have = g1 - g0;                              // 0: a chunk of fewer groups
    __syncthreads();
    double* red = reinterpret_cast<double*>(raw);          // [4][128]
    float* mid = raw + 4 * 128 * 2;                        // [128]
    const int i = t & 127, g = t >> 7;
    double s = 0.0;
    for (int k = g; k < have; k += MM_THREADS / 128) s = fma((double)count[k], (double)means[k * MM_PITCH + i], s);
    red[g * 128 + i] = s;
    __syncthreads();
    if (g == 0) {
      double points = 0.0;
      for (int k = 0; k < have; ++k) points += (double)count[k];
      s = have > 0 ? (((s + red[128 + i]) + red[256 + i]) + red[384 + i]) / points : 0.0;
      const int64_t at = ((int64_t)chunk * p.groups + group) * p.B + b;
      if (i < p.Ci) p.gm[at * p.Ci + i] = s;
      if (i == 0) p.gn[at] = points;
      mid[i] = (float)s;
    }
    __syncthreads();
#pragma unroll
    for (int h = 0; h < MM_H; ++h) {
      const int r = row + MM_ROWS * h;
      float c[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int k = piece * 4 + e;
        c[e] = k < have ? (means[k * MM_PITCH + r] - mid[r]) * sqrtf(count[k]) : 0.f;
      }
      park(r, make_float4(c[0], c[1], c[2], c[3]));
    }
    __syncthreads();
    products();
    gather();
  }
  float* XX = p.XXpart + ((int64_t)chunk * p.B + b) * p.Ci * p.Ci;
  // symmetric, element by element the same products in the same order up to the corrections': out as gram_kernel's
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int ci = wm * 64 + i * 32 + (lane & 31);
#pragma unroll
    for (int j = 0; j < MM_NJ; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const int cj = (wn * MM_NJ + j) * 32 + 8 * (v >> 2) + 4 * (lane >> 5) + (v & 3);
        if (ci < p.Ci && cj < p.Ci) XX[(int64_t)cj * p.Ci + ci] = sum[i][j][v];
      }
  }
}

// ---- E[x] and Cov(x) from the workgroups' parts, about the first's mean, in a fixed order: one input channel per workgroup, eight
// ---- shares of the parts ----
__global__ __launch_bounds__(1024, 8) void pool32_cov_kernel(Pool32Args p) {
  constexpr int Q = 256;                                   // groups at a time
  __shared__ double red[8][128], sx[8][128], wn[Q], wi[Q];
  const int i = blockIdx.x, b = blockIdx.y, j = threadIdx.x & 127, g = threadIdx.x >> 7, jc = min(j, p.Ci - 1);
  const int64_t stride = (int64_t)p.B * p.Ci;
  const double* gm = p.gm + (int64_t)b * p.Ci;
  const double ri = gm[i], rj = gm[jc];
  double a = 0.0, s = 0.0;
  const float* XX = p.XXpart + ((int64_t)b * p.Ci + i) * p.Ci + jc;
  for (int q0 = 0; q0 < p.chunks * p.groups; q0 += Q) {
    const int qs = min(Q, p.chunks * p.groups - q0);
    if (q0 > 0) __syncthreads();
    if ((int)threadIdx.x < qs) {
      const int64_t q = q0 + threadIdx.x;
      const double n = p.gn[q * p.B + b];
      wn[threadIdx.x] = n;
      wi[threadIdx.x] = n * (gm[q * stride + i] - ri);
    }
    if (q0 == 0) {
#pragma unroll 8
      for (int q = g; q < p.chunks; q += 8) a += (double)XX[q * stride * p.Ci];
    }
    __syncthreads();
#pragma unroll 8
    for (int q = g; q < qs; q += 8) {
      const double d = gm[(q0 + q) * stride + jc] - rj;
      a = fma(wi[q], d, a);
      s = fma(wn[q], d, s);
    }
  }
  red[g][j] = a;
  sx[g][j] = s;
  __syncthreads();
  if (g == 0) {
    for (int w = 1; w < 8; ++w) { a += red[w][j]; s += sx[w][j]; }
    sx[0][j] = s;
  }
  __syncthreads();
  if (g != 0 || j >= p.Ci) return;
  const double m = (double)p.Nb * (double)p.L;
  p.cov[((int64_t)b * p.Ci + i) * p.Ci + j] = a / m - (sx[0][i] / m) * (s / m);
  if (i == 0) p.ex[(int64_t)b * p.Ci + j] = rj + s / m;
}

// ---- dW: a thread per (channel of eight, input channel) ----
__global__ __launch_bounds__(1024) void pool32_dw_kernel(Pool32Args p) {
  constexpr int CB = 8;
  __shared__ float wrow[CB][128];
  const int c0 = blockIdx.x * CB, b = blockIdx.y, cj = threadIdx.x & 127, e = threadIdx.x >> 7, c = c0 + e;
  if (cj < p.Ci) wrow[e][cj] = c < p.Co ? p.W[((int64_t)b * p.Co + c) * p.Ci + cj] : 0.f;
  __syncthreads();
  if (cj >= p.Ci || c >= p.Co) return;
  const double* cx = p.cov + (int64_t)b * p.Ci * p.Ci + cj;
  double cov = 0.0, sp = 0.0;
#pragma unroll 16
  for (int i = 0; i < p.Ci; ++i) cov = fma((double)wrow[e][i], cx[(int64_t)i * p.Ci], cov);
#pragma unroll 16
  for (int n = 0; n < p.Nb; ++n) {
    const int64_t r = ((int64_t)b * p.Nb + n) * p.Co + c;
    sp = fma((double)p.s[r], (double)p.xg[r * p.Ci + cj], sp);
  }
  const int k = b * p.Co + c;
  const double m = (double)p.Nb * (double)p.L;
  p.dW[(int64_t)k * p.Ci + cj] = (float)(sp - m * (p.c0[k] * p.ex[(int64_t)b * p.Ci + cj] + p.c1[k] * cov));
}

size_t a256(size_t v) { return (v + 255) & ~(size_t)255; }

// the workspace's pieces, from `base` on; returns its size
size_t layout(Pool32Args& a, unsigned char* base) {
  size_t at = 0;
  auto take = [&](auto*& p, size_t n) {
    p = reinterpret_cast<std::remove_reference_t<decltype(p)>>(base + at);
    at += a256(n * sizeof(*p));
  };
  const size_t B = a.B, N = (size_t)a.B * a.Nb, Ci = a.Ci, Co = a.Co;
  take(a.c1, B * Co);
  take(a.c0, B * Co);
  take(a.cv, B * Co);
  take(a.s, N * Co);
  take(a.skey, N * Co);
  take(a.sval, N * Co);
  take(a.toff, N * (a.tiles + 1));
  take(a.negG, B * Ci * Ci);
  take(a.negv, B * Ci);
  const int total = a.Nb * ((a.L + MM_PTS - 1) / MM_PTS), want = (256 + a.B - 1) / a.B;   // a workgroup per compute unit
  a.chunks = want < total ? want : total;
  take(a.XXpart, a.chunks * B * Ci * Ci);
  a.groups = ((total + a.chunks - 1) / a.chunks + MM_GROUP - 1) / MM_GROUP;
  take(a.gm, (size_t)a.chunks * a.groups * B * Ci);
  take(a.gn, (size_t)a.chunks * a.groups * B);
  take(a.cov, B * Ci * Ci);
  take(a.ex, B * Ci);
  take(a.xg, N * Co * Ci);
  return at;
}

bool supported(int B, int Nb, int Ci, int Co, int L) {
  if (B <= 0 || Nb <= 0 || Ci <= 0 || Co <= 0 || L <= 0) return false;
  if (Ci <= 64 || Ci > 128 || Ci % 4 != 0 || Co <= 64 || Co > 1024 || L < 128 || L >= 1 << 21 || (int64_t)B * Nb > 65535) return false;
  return gemm_f32_big_tiles(Ci, L, (int64_t)B * Nb);      // both directions' products in 128 x 128 tiles
}

}  // namespace

namespace hfta {
// least workspace of either direction: the backward's, or the forward's partial sums (whose product is then the general one)
size_t pool32_least_bytes(int B, int Nb, int Ci, int Co, int L) {
  if (!supported(B, Nb, Ci, Co, L)) return 0;
  Pool32Args a{};
  a.B = B; a.Nb = Nb; a.Ci = Ci; a.Co = Co; a.L = L; a.tiles = (L + 127) / 128;
  return std::max(layout(a, nullptr), hfta_conv1x1_bn_pool_fwd_workspace_bytes(B, Nb, Ci, Co, L, HFTA_F32));
}
}  // namespace hfta

extern "C" {

size_t hfta_conv1x1_bn_maxpool_f32_workspace_bytes(int B, int Nb, int Ci, int Co, int L) {
  const size_t least = pool32_least_bytes(B, Nb, Ci, Co, L);
  return least ? std::max(least, pool32_fwd_bytes(B, Nb, Ci, Co, L)) : 0;
}

int hfta_conv1x1_bn_maxpool_f32_bwd(int B, int Nb, int Ci, int Co, int L, const float* X, const int64_t xs[4], const float* W,
                                    const float* bias, const float* zhit, const float* dV, const int32_t* idx, const int64_t vs[3],
                                    const float* gamma, const float* beta, const float* save_mean, const float* save_invstd,
                                    float* dX, const int64_t dxs[4], float* dW, float* dbias, float* dgamma, float* dbeta, int act,
                                    float act_slope, void* workspace, size_t ws_bytes, void* stream) {
  if (B <= 0 || Nb <= 0 || Ci <= 0 || Co <= 0 || L <= 0 || !X || !xs || !W || !zhit || !dV || !idx || !vs || !gamma || !beta ||
      !save_mean || !save_invstd || !dX || !dxs || !dW || !dgamma || !dbeta)
    return HFTA_EINVAL;
  if (!(act == HFTA_ACT_NONE || act == HFTA_ACT_RELU || (act == HFTA_ACT_LEAKY && act_slope >= 0.f))) return HFTA_EUNSUPPORTED;
  if (xs[3] != 1 || dxs[3] != 1 || xs[2] <= 0 || !supported(B, Nb, Ci, Co, L)) return HFTA_EUNSUPPORTED;
  if (!workspace || reinterpret_cast<uintptr_t>(workspace) % 256 != 0 || reinterpret_cast<uintptr_t>(W) % 8 != 0 ||
      ws_bytes < pool32_least_bytes(B, Nb, Ci, Co, L))
    return reinterpret_cast<uintptr_t>(W) % 8 != 0 ? HFTA_EUNSUPPORTED : HFTA_EWORKSPACE;
  const int64_t x_bytes = ((int64_t)(Ci - 1) * xs[2] + L) * 4;
  if (x_bytes >= (int64_t)1 << 31) return HFTA_EUNSUPPORTED;
  hipStream_t st = as_stream(stream);
  Pool32Args a{X, W, bias, zhit, dV, idx, gamma, beta, save_mean, save_invstd, dW, dbias, dgamma, dbeta,
               xs[0], xs[1], xs[2], vs[0], vs[1], vs[2], B, Nb, Ci, Co, L, act, (L + 127) / 128, act_slope,
               (uint32_t)x_bytes};
  layout(a, static_cast<unsigned char*>(workspace));
  hipLaunchKernelGGL(pool32_coef_kernel, dim3((unsigned)((Co + 63) / 64), (unsigned)B), dim3(C32_WAVES * 64), 0, st, a);
  int P = 64;
  while (P < Co) P <<= 1;
  const int T = (Ci + 31) / 32;
  hipLaunchKernelGGL(pool32_prep_kernel, dim3((unsigned)(B * Nb + (T * T + 1) * B)), dim3(HIT_THREADS), 0, st, a, P);
  hipLaunchKernelGGL(pool32_moments_kernel, dim3((unsigned)a.chunks, (unsigned)B), dim3(MM_THREADS), 0, st, a);
  hipLaunchKernelGGL(pool32_cov_kernel, dim3((unsigned)Ci, (unsigned)B), dim3(1024), 0, st, a);
  hipLaunchKernelGGL(pool32_dw_kernel, dim3((unsigned)((Co + 7) / 8), (unsigned)B), dim3(1024), 0, st, a);
  GemmDesc d{};
  d.A = a.negG; d.Bm = X; d.C = dX;
  d.M = Ci; d.N = L; d.K = Ci; d.S = 1; d.G0 = B; d.G1 = Nb;
  d.a_kc = true; d.a_ld = Ci; d.a_g0 = (int64_t)Ci * Ci;
  d.b_kc = false; d.b_ld = xs[2]; d.b_g0 = xs[0]; d.b_g1 = xs[1];
  d.c_ld = dxs[2]; d.c_g0 = dxs[0]; d.c_g1 = dxs[1];
  d.bias = a.negv; d.bias_mode = 1; d.bias_g0 = Ci;
  d.act = HFTA_ACT_NONE; d.dtype = HFTA_F32; d.splits = 1;
  d.hit_key = a.skey; d.hit_val = a.sval; d.hit_off = a.toff; d.hit_w = W; d.hit_co = Co;
  if (launch_status() != HFTA_OK) return HFTA_ELAUNCH;
  return gemm_launch(d, st);
}

}  // extern "C"
