// Helpers shared by the BatchNorm kernels: vector loads/stores of four elements, fixed-order
// block reductions, activation derivative.
#pragma once
#include "common.h"

namespace hfta {

template <typename T, int VEC> struct Vec;
template <> struct Vec<float, 4> { typedef float4 type; };
template <> struct Vec<float, 1> { typedef float type; };
template <> struct Vec<bf16_raw, 4> { typedef uint2 type; };
template <> struct Vec<bf16_raw, 1> { typedef bf16_raw type; };

template <typename T, int VEC>
__device__ __forceinline__ void load_vec(const T* p, float (&v)[VEC]) {
  typename Vec<T, VEC>::type raw = *reinterpret_cast<const typename Vec<T, VEC>::type*>(p);
  const T* e = reinterpret_cast<const T*>(&raw);
#pragma unroll
  for (int i = 0; i < VEC; ++i) v[i] = Elem<T>::to_f32(e[i]);
}
template <typename T, int VEC>
__device__ __forceinline__ void store_vec(T* p, const float (&v)[VEC]) {
  typename Vec<T, VEC>::type raw;
  T* e = reinterpret_cast<T*>(&raw);
#pragma unroll
  for (int i = 0; i < VEC; ++i) e[i] = Elem<T>::from_f32(v[i]);
  *reinterpret_cast<typename Vec<T, VEC>::type*>(p) = raw;
}

// Rows that are no multiple of four elements, or not aligned to four: the same four-element pieces with
// vector accesses at element alignment (the memory system takes them: a row copy at odd lengths and 2-byte
// alignment moves the bytes at the rate of a 2500-element one, 4.9 TB/s, where single elements reach a
// quarter of it).  The piece that straddles the row's end is read from where the row's last four elements
// start and moved into place; what lies past the end is zero.  Needs L >= 4.
template <typename T> struct PieceAt;
template <> struct PieceAt<bf16_raw> { typedef uint32_t type __attribute__((ext_vector_type(2), aligned(2))); };
template <> struct PieceAt<float> { typedef uint32_t type __attribute__((ext_vector_type(4), aligned(4))); };

__device__ __forceinline__ void piece_shift(uint32_t (&w)[2], int sh) {       // four 16-bit elements, sh of them out
  const uint64_t q = ((uint64_t)w[1] << 32 | w[0]) >> (16 * sh);
  w[0] = (uint32_t)q; w[1] = (uint32_t)(q >> 32);
}
__device__ __forceinline__ void piece_shift(uint32_t (&w)[4], int sh) {       // four 32-bit elements
  if (sh & 1) { w[0] = w[1]; w[1] = w[2]; w[2] = w[3]; w[3] = 0u; }
  if (sh & 2) { w[0] = w[2]; w[1] = w[3]; w[2] = w[3] = 0u; }
}

// piece ch of a row of L elements (VEC == 1: element ch)
template <typename T, int VEC, bool RAG>
__device__ __forceinline__ void load_piece(const T* row, int ch, int L, float (&v)[VEC]) {
  if constexpr (!RAG) {
    load_vec<T, VEC>(row + ch * VEC, v);
  } else {
    constexpr int W = (int)sizeof(T);
    const int at = min(ch * 4, L - 4);
    const typename PieceAt<T>::type raw = *reinterpret_cast<const typename PieceAt<T>::type*>(row + at);
    uint32_t w[W];
#pragma unroll
    for (int i = 0; i < W; ++i) w[i] = raw[i];
    piece_shift(w, ch * 4 - at);
    const T* e = reinterpret_cast<const T*>(w);
#pragma unroll
    for (int i = 0; i < VEC; ++i) v[i] = Elem<T>::to_f32(e[i]);
  }
}
template <typename T, int VEC, bool RAG>
__device__ __forceinline__ void store_piece(T* row, int ch, int L, const float (&v)[VEC]) {
  if constexpr (!RAG) {
    store_vec<T, VEC>(row + ch * VEC, v);
  } else if (ch * 4 + 4 <= L) {
    T e[4];
#pragma unroll
    for (int i = 0; i < VEC; ++i) e[i] = Elem<T>::from_f32(v[i]);
    *reinterpret_cast<typename PieceAt<T>::type*>(row + ch * 4) = *reinterpret_cast<const typename PieceAt<T>::type*>(e);
  } else {
#pragma unroll
    for (int i = 0; i < VEC; ++i)
      if (ch * 4 + i < L) row[ch * 4 + i] = Elem<T>::from_f32(v[i]);
  }
}

// block-wide sum of two values; result valid in every thread
template <int NW>
__device__ __forceinline__ void block_sum2(float& a, float& b, float (*sh)[2]) {
  a = wave_sum(a);
  b = wave_sum(b);
  const int w = threadIdx.x >> 6;
  __syncthreads();
  if ((threadIdx.x & 63) == 0) { sh[w][0] = a; sh[w][1] = b; }
  __syncthreads();
  float ra = 0.f, rb = 0.f;
#pragma unroll
  for (int i = 0; i < NW; i += 4) {          // fixed order, pairwise within groups of four waves
    ra += (sh[i][0] + sh[i + 1][0]) + (sh[i + 2][0] + sh[i + 3][0]);
    rb += (sh[i][1] + sh[i + 1][1]) + (sh[i + 2][1] + sh[i + 3][1]);
    if (NW > 4) __builtin_amdgcn_sched_barrier(0);          // 8 registers at a time: all 32 at once made kernels that hold data spill
  }
  a = ra; b = rb;
}

// The activations a BatchNorm takes: none, ReLU, LeakyReLU.  What is uniform over the launch stays outside the element:
// with the general apply_act a kernel carries tanh and erf for every element it unrolls (the forward kernel 13 KB of code,
// 70 KB with 20 pieces unrolled, fetched anew by each launch) and takes a scalar branch around them.
__device__ __forceinline__ float act_below(int act, float slope) {
  return act == HFTA_ACT_RELU ? 0.f : act == HFTA_ACT_LEAKY ? slope : 1.f;
}
__device__ __forceinline__ float bn_act(float y, int act, float slope) {
  const float lo = act_below(act, slope) * y;
  return y > 0.f ? y : act == HFTA_ACT_RELU ? 0.f : lo;
}
__device__ __forceinline__ float act_grad(float pre, int act, float slope) {
  return pre > 0.f ? 1.f : act_below(act, slope);
}

// Channels whose data is large get one 1024-thread workgroup each (instead of 256 threads):
// 512 channels x 1024 threads fill the chip where 512 x 256 would leave it three quarters empty,
// and fewer channels are in flight at once.
static inline bool bn_wide_block(int64_t channel_bytes) { return channel_bytes >= 32 * 1024; }

// Elements or pieces a thread of the two-pass kernels has in flight.  A row that does not divide into aligned
// pieces is walked element by element: neighbouring lanes read neighbouring elements, so the memory system
// does not mind, but a thread then needs as many loads in flight as the vector form has elements.
constexpr int bn_unroll(int vec) { return vec == 1 ? 16 : 4; }

// Launches LAUNCH(T, VEC, RAG) for `dtype`: aligned four-element pieces (v4), four-element pieces of rows of any
// length and alignment, or, for rows shorter than one piece, single elements.
#define HFTA_BN_BY_ROWS(LAUNCH) \
  do { if (dtype == HFTA_BF16) { if (v4) LAUNCH(bf16_raw, 4, false); else if (L >= 4) LAUNCH(bf16_raw, 4, true); else LAUNCH(bf16_raw, 1, false); } \
       else { if (v4) LAUNCH(float, 4, false); else if (L >= 4) LAUNCH(float, 4, true); else LAUNCH(float, 1, false); } } while (0)

// widest vector access every row of a strided [b][n][c][l] tensor allows: 4 elements or 1
static inline bool bn_vec4_ok(const void* p, const int64_t* s, int L, int dtype) {
  const size_t bytes = 4 * dtype_size(dtype);
  return L % 4 == 0 && reinterpret_cast<uintptr_t>(p) % bytes == 0 && s[0] % 4 == 0 && s[1] % 4 == 0 && s[2] % 4 == 0;
}

}  // namespace hfta
