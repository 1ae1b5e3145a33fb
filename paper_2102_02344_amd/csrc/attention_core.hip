// Attention core of one head in one kernel per direction (bf16, heads of at most 64 columns, at most 256 tokens).
//
// As batched GEMMs a 64 x 64 head fills a quarter of a 128 x 128 tile, and the score matrix goes through memory
// four times forward and eight times backward.  Here a head's K and V sit in LDS, scores stay in registers, and
// of the score-sized tensors only P moves: written once forward (the backward's input), read once backward.
// Rounding is that of the batched form, which stores scores, P, dP and dS: each is rounded to bf16 once.
// Per layer of 8 models x 32 x 64 tokens, 4 heads of 64: forward 44 -> 11.5 us, backward 61 -> 22 us;
// 4 x 12 x 250 tokens: 58 -> 23 and 75 -> 35 us.  Bound by latency: a head is 16-row blocks of dependent
// products, reductions and exponentials, two to four wavefronts per SIMD.
//
// Matrix instruction 16 x 16 x 32: operands hold row (column) l%16 and k = 8(l/16) + 0..7, the result column l%16
// and rows 4(l/16) + 0..3.  Products are arranged so that a result is the next product's operand without a
// shuffle: with the keys as the first operand, lane l holds query l%16 and keys 16jb + 4(l/16) + 0..3 of block jb,
// which is an operand of a product over keys if the other side orders k the same way, slots 0..3 from block 2t
// and 4..7 from block 2t + 1.  That order is what two transpose reads of a [token][column] tile deliver: in every
// group of 16 lanes, lane r supplies the address of four neighbouring columns of token r/4, and lane i receives
// column i of the four.
#include "common.h"

namespace hfta {

typedef __bf16 at_bf8 __attribute__((ext_vector_type(8)));
typedef float at_f4 __attribute__((ext_vector_type(4)));
typedef short at_s4 __attribute__((ext_vector_type(4)));

constexpr int AT_PITCH = 144;     // bytes per token row of a staged [token][64] tile: 16 rows' 16-byte reads cover all banks

__device__ __forceinline__ at_bf8 at_row_frag(const unsigned char* tile, int row0, int ks, int lane) {
  return *reinterpret_cast<const at_bf8*>(tile + (row0 + (lane & 15)) * AT_PITCH + ks * 64 + (lane >> 4) * 16);
}
// columns col0 + l%16, tokens tok0 + 4(l/16) + 0..3 and tok0 + 16 + 4(l/16) + 0..3
template <int PITCH>
__device__ __forceinline__ at_bf8 at_tr_frag(const unsigned char* tile, int tok0, int col0, int lane) {
  const int r = lane & 15;
  const unsigned char* a = tile + (tok0 + 4 * (lane >> 4) + (r >> 2)) * PITCH + (col0 + 4 * (r & 3)) * 2;
  typedef __attribute__((address_space(3))) at_s4* lds_s4;
  union { at_s4 h[2]; at_bf8 v; } u;
  u.h[0] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s4)(a));
  u.h[1] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s4)(a + 16 * PITCH));
  return u.v;
}
__device__ __forceinline__ at_bf8 at_pair(uint2 a, uint2 b) {
  union { uint4 q; at_bf8 v; } u;
  u.q = make_uint4(a.x, a.y, b.x, b.y);
  return u.v;
}
// rows tok0 .. of a [token][ld] tensor's 64-column slice, N 16-byte pieces per thread (N NT / 8 rows), through registers
// into LDS; tokens past S and columns past d: zeros.  All loads are in flight before the first is stored.
template <int N, int NT = 256> struct AtRows {
  static constexpr int RP = NT / 8;                              // rows per pass
  uint4 v[N];
  __device__ __forceinline__ void load(const bf16_raw* src, int64_t ld, int tok0, int S, int d) {
    const int r = threadIdx.x >> 3, c = threadIdx.x & 7;
#pragma unroll
    for (int n = 0; n < N; ++n) {
      v[n] = make_uint4(0, 0, 0, 0);
      if (tok0 + r + RP * n < S && c * 8 < d) v[n] = *reinterpret_cast<const uint4*>(src + (int64_t)(tok0 + r + RP * n) * ld + c * 8);
    }
  }
  __device__ __forceinline__ void store(unsigned char* tile) const {
    const int r = threadIdx.x >> 3, c = threadIdx.x & 7;
#pragma unroll
    for (int n = 0; n < N; ++n) *reinterpret_cast<uint4*>(tile + (r + RP * n) * AT_PITCH + c * 16) = v[n];
  }
};
typedef uint32_t at_u2 __attribute__((ext_vector_type(2), aligned(2)));    // P rows start at any element
// entries 16jb + 4g + 0..3 of a P row; only the last block (a uniform branch) can be cut short by S
__device__ __forceinline__ void at_store_p(bf16_raw* row, int jb, int g, int S, uint2 v) {
  const int j = jb * 16 + 4 * g;
  if (jb * 16 + 16 <= S) {
    at_u2 w; w.x = v.x; w.y = v.y;
    *reinterpret_cast<at_u2*>(row + j) = w;
  } else {
    const uint32_t w[2] = {v.x, v.y};
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if (j + e < S) row[j + e] = (bf16_raw)(w[e >> 1] >> (16 * (e & 1)));
  }
}
__device__ __forceinline__ uint2 at_load_p(const bf16_raw* row, int jb, int g, int S) {
  const int j = jb * 16 + 4 * g;
  if (jb * 16 + 16 <= S) {
    const at_u2 w = *reinterpret_cast<const at_u2*>(row + j);
    return make_uint2(w.x, w.y);
  }
  uint32_t w[2] = {0, 0};
#pragma unroll
  for (int e = 0; e < 4; ++e)
    if (j + e < S) w[e >> 1] |= (uint32_t)row[j + e] << (16 * (e & 1));
  return make_uint2(w[0], w[1]);
}
// four columns of a result row as bf16
__device__ __forceinline__ void at_store4(bf16_raw* dst, const at_f4& v) {
  *reinterpret_cast<uint2*>(dst) = make_uint2(pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3]));
}
__device__ __forceinline__ float at_row_sum(float v) {           // over the four lanes that share a query
  v += __shfl_xor(v, 16, 64);
  return v + __shfl_xor(v, 32, 64);
}

// Workgroup (head, part): row blocks part * 4 + wave, stepping by 4 * gridDim.y.  NJ: 16-key blocks held per row.
template <int NJ>
__global__ __launch_bounds__(256) void attn_fwd_kernel(const bf16_raw* __restrict__ QKV, bf16_raw* __restrict__ P,
                                                       bf16_raw* __restrict__ CTX, int S, int E, int H, int d, float scale, int causal) {
  __shared__ __attribute__((aligned(16))) unsigned char sk[NJ * 16 * AT_PITCH];
  __shared__ __attribute__((aligned(16))) unsigned char sv[NJ * 16 * AT_PITCH];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), g = lane >> 4;
  const int bn = blockIdx.x / H, h = blockIdx.x % H;
  const bf16_raw* q = QKV + (int64_t)bn * S * 3 * E + h * d;
  {
    AtRows<NJ / 2> k, v;
    k.load(q + E, 3 * E, 0, S, d);
    v.load(q + 2 * E, 3 * E, 0, S, d);
    k.store(sk);
    v.store(sv);
  }
  __syncthreads();
  const int nb = (S + 15) >> 4;
  for (int rb = blockIdx.y * 4 + wave; rb < nb; rb += 4 * gridDim.y) {
    const int i = rb * 16 + (lane & 15);
    const int nbl = causal ? rb + 1 : nb;                        // key blocks with a valid entry
    const int lim = (causal ? min(i + 1, S) : S) - 4 * g;        // this lane's key 16jb + v is valid below it
    at_bf8 qf[2];
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
      union { uint4 u; at_bf8 v; } x;
      x.u = make_uint4(0, 0, 0, 0);
      if (i < S && ks * 32 + g * 8 < d) x.u = *reinterpret_cast<const uint4*>(q + (int64_t)i * 3 * E + ks * 32 + g * 8);
      qf[ks] = x.v;
    }
    at_f4 s[NJ];
    float mx = -INFINITY;
#pragma unroll
    for (int jb = 0; jb < NJ; ++jb) {
      s[jb] = at_f4{0.f, 0.f, 0.f, 0.f};
      if (jb >= nbl) continue;
#pragma unroll
      for (int ks = 0; ks < 2; ++ks)
        s[jb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(at_row_frag(sk, jb * 16, ks, lane), qf[ks], s[jb], 0, 0, 0);
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        s[jb][v] = jb * 16 + v < lim ? bf16_to_f32(f32_to_bf16(s[jb][v])) * scale : -INFINITY;
        mx = fmaxf(mx, s[jb][v]);
      }
    }
    mx = fmaxf(mx, __shfl_xor(mx, 16, 64));
    mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
    float se = 0.f;
#pragma unroll
    for (int jb = 0; jb < NJ; ++jb) {
      if (jb >= nbl) continue;
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        // masked entries: exp(-inf).  (The native exponential loses a bit per doubling of its argument; it took
        // 21.2 us where this takes 22.8, 4 x 12 x 250 tokens.)
        s[jb][v] = expf(s[jb][v] - mx);
        se += s[jb][v];
      }
    }
    const float inv = 1.f / at_row_sum(se);
    uint2 pk[NJ];
    bf16_raw* prow = P + ((int64_t)blockIdx.x * S + i) * S;
#pragma unroll
    for (int jb = 0; jb < NJ; ++jb) {
      pk[jb] = make_uint2(0, 0);
      if (jb < nbl) pk[jb] = make_uint2(pack_bf16x2(s[jb][0] * inv, s[jb][1] * inv), pack_bf16x2(s[jb][2] * inv, s[jb][3] * inv));
    }
    if (__any(inv != inv)) {                                     // a row that holds a NaN or an infinity: its masked entries stay zero
#pragma unroll
      for (int jb = 0; jb < NJ; ++jb) {
        if (jb != nbl - 1) continue;                             // (the only block with masked entries)
        float x[4];
#pragma unroll
        for (int v = 0; v < 4; ++v) x[v] = jb * 16 + v < lim ? s[jb][v] * inv : 0.f;
        pk[jb] = make_uint2(pack_bf16x2(x[0], x[1]), pack_bf16x2(x[2], x[3]));
      }
    }
    if (i < S) {
#pragma unroll
      for (int jb = 0; jb < NJ; ++jb)
        if (jb < nb) at_store_p(prow, jb, g, S, pk[jb]);
    }
    at_f4 o[4];
#pragma unroll
    for (int cb = 0; cb < 4; ++cb) o[cb] = at_f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int t = 0; t < NJ / 2; ++t) {
      if (2 * t >= nbl) continue;
      const at_bf8 pf = at_pair(pk[2 * t], pk[2 * t + 1]);
#pragma unroll
      for (int cb = 0; cb < 4; ++cb)
        o[cb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(at_tr_frag<AT_PITCH>(sv, t * 32, cb * 16, lane), pf, o[cb], 0, 0, 0);
    }
    if (i < S) {
      bf16_raw* c = CTX + ((int64_t)bn * S + i) * E + h * d + 4 * g;
#pragma unroll
      for (int cb = 0; cb < 4; ++cb)
        if (cb * 16 + 4 * g < d) at_store4(c + cb * 16, o[cb]);
    }
  }
}

// One workgroup per head, 64 queries at a time.  A wavefront takes 16 of them for dP, dS and dQ and leaves its P
// and dS rows in LDS; after a barrier it takes key blocks wave, wave + 4, ... for dK and dV, which it accumulates in
// registers over all queries.  P may come from any caller, so no block is skipped as masked.
// HV = 2: eight wavefronts, two per 16 queries with half the keys each (their halves of sum dP P meet in LDS) and half
// the columns of dQ.  A head of more than 64 tokens fills a compute unit's LDS, so this is what hides its latencies:
// 4 x 12 x 250 tokens 46 -> 35 us.
template <int NJ, int HV>
__global__ __launch_bounds__(256 * HV) void attn_bwd_kernel(const bf16_raw* __restrict__ QKV, const bf16_raw* __restrict__ P,
                                                       const bf16_raw* __restrict__ dCTX, bf16_raw* __restrict__ dQKV, int S, int E,
                                                       int H, int d, float scale) {
  constexpr int PP = NJ * 32 + 32;                               // bytes per row of the P and dS tiles
  __shared__ __attribute__((aligned(16))) unsigned char sk[NJ * 16 * AT_PITCH];
  __shared__ __attribute__((aligned(16))) unsigned char sv[NJ * 16 * AT_PITCH];
  __shared__ __attribute__((aligned(16))) unsigned char sq[64 * AT_PITCH];
  __shared__ __attribute__((aligned(16))) unsigned char sc[64 * AT_PITCH];
  __shared__ __attribute__((aligned(16))) unsigned char sp[64 * PP];
  __shared__ __attribute__((aligned(16))) unsigned char ss[64 * PP];
  __shared__ float sdot[HV][64];
  constexpr int NT = 256 * HV, HB = NJ / HV;                     // threads; key blocks per wavefront
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), g = lane >> 4, li = lane & 15;
  const int half = HV == 2 ? wave >> 2 : 0, qrow = (wave & 3) * 16 + li, j0 = half * HB;
  const int bn = blockIdx.x / H, h = blockIdx.x % H;
  const bf16_raw* q = QKV + (int64_t)bn * S * 3 * E + h * d;
  const bf16_raw* dc = dCTX + (int64_t)bn * S * E + h * d;
  bf16_raw* dq = dQKV + (int64_t)bn * S * 3 * E + h * d;
  const int nb = (S + 15) >> 4;
  // the next 64 queries' Q, dCTX and P rows, fetched while the last are multiplied
  AtRows<2 / HV, NT> rq, rc;
  uint2 pn[HB];
  auto fetch = [&](int i0) {
    rq.load(q, 3 * E, i0, S, d);
    rc.load(dc, E, i0, S, d);
    // (rows past S take the last row's P: their dCTX rows are zeros, so dP, dS and their part of dV are too)
    const bf16_raw* prow = P + ((int64_t)blockIdx.x * S + min(i0 + qrow, S - 1)) * S;
#pragma unroll
    for (int jb = 0; jb < HB; ++jb) {
      pn[jb] = make_uint2(0, 0);
      if (j0 + jb < nb) pn[jb] = at_load_p(prow, j0 + jb, g, S);
    }
  };
  {
    AtRows<NJ / 2 / HV, NT> k, v;
    k.load(q + E, 3 * E, 0, S, d);
    v.load(q + 2 * E, 3 * E, 0, S, d);
    fetch(0);
    k.store(sk);
    v.store(sv);
  }
  constexpr int NW = NJ / (4 * HV);
  at_f4 dk[NW][4], dv[NW][4];
#pragma unroll
  for (int n = 0; n < NW; ++n)
#pragma unroll
    for (int cb = 0; cb < 4; ++cb) { dk[n][cb] = at_f4{0.f, 0.f, 0.f, 0.f}; dv[n][cb] = at_f4{0.f, 0.f, 0.f, 0.f}; }

  for (int i0 = 0; i0 < S; i0 += 64) {
    __syncthreads();                                             // the last group's tiles have been read
    rq.store(sq);
    rc.store(sc);
    const int i = i0 + qrow;
    uint2 pk[HB];
#pragma unroll
    for (int jb = 0; jb < HB; ++jb) pk[jb] = pn[jb];
    __syncthreads();
    at_bf8 cf[2];
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) cf[ks] = at_row_frag(sc, (wave & 3) * 16, ks, lane);
    at_f4 dp[HB];
    float dot = 0.f;
    unsigned char* pt = sp + qrow * PP + j0 * 32 + g * 8;
#pragma unroll
    for (int jb = 0; jb < HB; ++jb) {
      dp[jb] = at_f4{0.f, 0.f, 0.f, 0.f};
      if (j0 + jb >= nb) continue;
#pragma unroll
      for (int ks = 0; ks < 2; ++ks)
        dp[jb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(at_row_frag(sv, (j0 + jb) * 16, ks, lane), cf[ks], dp[jb], 0, 0, 0);
      *reinterpret_cast<uint2*>(pt + jb * 32) = pk[jb];
      const float p[4] = {__uint_as_float(pk[jb].x << 16), __uint_as_float(pk[jb].x & 0xffff0000u),
                          __uint_as_float(pk[jb].y << 16), __uint_as_float(pk[jb].y & 0xffff0000u)};
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        dp[jb][v] = bf16_to_f32(f32_to_bf16(dp[jb][v]));
        dot = fmaf(dp[jb][v], p[v], dot);
      }
    }
    dot = at_row_sum(dot);
    if (HV == 2) {
      if (g == 0) sdot[half][qrow] = dot;
      __syncthreads();
      dot = sdot[0][qrow] + sdot[HV - 1][qrow];
    }
    unsigned char* st = ss + qrow * PP + j0 * 32 + g * 8;
#pragma unroll
    for (int jb = 0; jb < HB; ++jb) {
      if (j0 + jb >= nb) continue;
      const float p[4] = {__uint_as_float(pk[jb].x << 16), __uint_as_float(pk[jb].x & 0xffff0000u),
                          __uint_as_float(pk[jb].y << 16), __uint_as_float(pk[jb].y & 0xffff0000u)};
      float x[4];
#pragma unroll
      for (int v = 0; v < 4; ++v) x[v] = scale * p[v] * (dp[jb][v] - dot);
      pk[jb] = make_uint2(pack_bf16x2(x[0], x[1]), pack_bf16x2(x[2], x[3]));       // dS from here on
      *reinterpret_cast<uint2*>(st + jb * 32) = pk[jb];
    }
    // dQ: all keys, with HV = 2 from the dS rows in LDS (the other half's among them) and half the columns
    if (HV == 2) __syncthreads();
    constexpr int CB = 4 / HV;
    at_f4 o[CB];
#pragma unroll
    for (int cb = 0; cb < CB; ++cb) o[cb] = at_f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int t = 0; t < NJ / 2; ++t) {
      if (2 * t >= nb) continue;
      at_bf8 sf;
      if constexpr (HV == 1) {
        sf = at_pair(pk[2 * t], pk[2 * t + 1]);
      } else {                                                   // (blocks past the last were never written)
        const unsigned char* r = ss + qrow * PP + t * 64 + g * 8;
        sf = at_pair(*reinterpret_cast<const uint2*>(r), 2 * t + 1 < nb ? *reinterpret_cast<const uint2*>(r + 32) : make_uint2(0, 0));
      }
#pragma unroll
      for (int cb = 0; cb < CB; ++cb)
        o[cb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(at_tr_frag<AT_PITCH>(sk, t * 32, (half * CB + cb) * 16, lane), sf, o[cb], 0, 0, 0);
    }
    if (i < S) {
#pragma unroll
      for (int cb = 0; cb < CB; ++cb) {
        const int c = (half * CB + cb) * 16 + 4 * g;
        if (c < d) at_store4(dq + (int64_t)i * 3 * E + c, o[cb]);
      }
    }
    if (i0 + 64 < S) fetch(i0 + 64);
    if (HV == 1) __syncthreads();
#pragma unroll
    for (int kk = 0; kk < 2; ++kk) {
      if (i0 + 32 * kk >= S) continue;
      at_bf8 qf[4], xf[4];
#pragma unroll
      for (int cb = 0; cb < 4; ++cb) {
        qf[cb] = at_tr_frag<AT_PITCH>(sq, kk * 32, cb * 16, lane);
        xf[cb] = at_tr_frag<AT_PITCH>(sc, kk * 32, cb * 16, lane);
      }
#pragma unroll
      for (int n = 0; n < NW; ++n) {
        const int jb = n * 4 * HV + wave;
        if (jb >= nb) continue;
        const at_bf8 pf = at_tr_frag<PP>(sp, kk * 32, jb * 16, lane), sf = at_tr_frag<PP>(ss, kk * 32, jb * 16, lane);
#pragma unroll
        for (int cb = 0; cb < 4; ++cb) {
          dv[n][cb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(xf[cb], pf, dv[n][cb], 0, 0, 0);
          dk[n][cb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(qf[cb], sf, dk[n][cb], 0, 0, 0);
        }
      }
    }
  }
#pragma unroll
  for (int n = 0; n < NW; ++n) {
    const int j = (n * 4 * HV + wave) * 16 + li;
    if (j >= S) continue;
    bf16_raw* row = dq + (int64_t)j * 3 * E + 4 * g;
#pragma unroll
    for (int cb = 0; cb < 4; ++cb)
      if (cb * 16 + 4 * g < d) {
        at_store4(row + E + cb * 16, dk[n][cb]);
        at_store4(row + 2 * E + cb * 16, dv[n][cb]);
      }
  }
}

// Heads this file's kernels take: bf16, whole 16-byte pieces (d a multiple of 8, 16-byte aligned tensors; P at any
// element), at most 64 columns (the staged row) and 256 tokens (scores in registers, P and dS rows in LDS).
bool attn_core_ok(int S, int E, int H, int dtype, const void* a, const void* b, const void* c) {
  const int d = E / H;
  return dtype == HFTA_BF16 && d % 8 == 0 && d <= 64 && S <= 256 &&
         ((reinterpret_cast<uintptr_t>(a) | reinterpret_cast<uintptr_t>(b) | reinterpret_cast<uintptr_t>(c)) & 15) == 0;
}

int attn_core_fwd(int BN, int S, int E, int H, const void* QKV, void* P, void* CTX, int causal, hipStream_t st) {
  const int heads = BN * H, blocks = (S + 63) / 64;             // a workgroup's four wavefronts take 64 rows per pass
  int parts = (512 + heads - 1) / heads;                         // two workgroups per compute unit where the rows allow
  if (parts > blocks) parts = blocks;
  const dim3 grid((unsigned)heads, (unsigned)parts);
  const float scale = 1.f / sqrtf((float)(E / H));
#define HFTA_ATF(NJ) hipLaunchKernelGGL(attn_fwd_kernel<NJ>, grid, dim3(256), 0, st, (const bf16_raw*)QKV, (bf16_raw*)P, \
                                        (bf16_raw*)CTX, S, E, H, E / H, scale, causal)
  if (S <= 64) HFTA_ATF(4);
  else if (S <= 128) HFTA_ATF(8);
  else HFTA_ATF(16);
#undef HFTA_ATF
  return launch_status();
}

int attn_core_bwd(int BN, int S, int E, int H, const void* QKV, const void* P, const void* dCTX, void* dQKV, hipStream_t st) {
  const dim3 grid((unsigned)(BN * H));
  const float scale = 1.f / sqrtf((float)(E / H));
#define HFTA_ATB(NJ, HV) hipLaunchKernelGGL((attn_bwd_kernel<NJ, HV>), grid, dim3(256 * HV), 0, st, (const bf16_raw*)QKV, \
                                            (const bf16_raw*)P, (const bf16_raw*)dCTX, (bf16_raw*)dQKV, S, E, H, E / H, scale)
  if (S <= 64) HFTA_ATB(4, 1);
  else if (S <= 128) HFTA_ATB(8, 2);
  else HFTA_ATB(16, 2);
#undef HFTA_ATB
  return launch_status();
}

}  // namespace hfta
