// bf16 GEMM on 256x256 tiles whose operands travel from memory straight into a ring of LDS slots.
//
// What bounds the products this is for (an MLP block: 16 x 4096 x 512 x 2048) is neither the matrix pipes nor the LDS alone.
// With everything but one part left out, the k-loop on resident tiles takes 81-99 us, the loads alone 107-141 us, and the
// register-staged 256x256 kernel took 141-178 us for both.  So everything here serves the loads:
//  * Operand tiles of 64 k: 128-byte segments.  The L2 hands a compute unit 64-byte segments at half the rate (17-19 TB/s
//    chip-wide against 31-33 TB/s from 128 bytes on, all hits), and a row's 64 bytes now and 64 later open a DRAM page twice.
//  * Five slots of 32 KB, one operand's k-tile each, filled in turn A B A B ...: all 160 KB of LDS.  While a k-tile is read
//    (two slots) two to three operand tiles are in flight, without a register or an LDS store spent on them.
//  * The eight loads of a wavefront per k-tile are spread over its k-steps, two at a time between matrix instructions: issued
//    in one go after the barrier they hold up the wavefront (the texture path takes 64 bytes per clock): 145 -> 131 us.
//  * Results leave by non-temporal stores: left in L2 they displace operands that other tiles read again (154 -> 138 us where
//    K = 512), and tiles run in groups of RING_GM row tiles, so that the 32 tiles an XCD holds at a time are a block of
//    4 x 8 or 4 x 2 instead of a column (191 -> 167 us there with the staging of the old kernel).
// Fragments of a k-step are read one k-step ahead (two register sets), and the barrier of a k-tile stands before its last
// k-step, whose fragments are in registers by then: the matrix instructions run on while the next tile's first reads return.
// Against the register-staged kernels, us: forward 512 -> 2048 178 -> 138, 2048 -> 512 142 -> 125, data gradients 170 -> 138
// and 141 -> 126, weight gradients 142 -> 128; vocabulary 256 -> 8192 on 8 x 2048 rows 114 -> 93.  The same bits.
//
// Tried: two groups of wavefronts a k-step apart, one multiplying while the other reads (two barriers per 32 k: 135-175 us),
// the 16x16x32 instruction (14 % faster alone on random data, the clock drops less; no difference here), 64-byte segments.
//
// Persistent: one workgroup per compute unit walks the tiles; the loader runs one to two k-tiles ahead across tile ends.  The
// epilogue stages 32 rows of a wavefront's block at a time in its own 4 KB of the slot that B's last k-tile has left, so no
// barrier is needed among them, while three operand tiles of the next output tile are on their way.
//
// Host side guarantees (gemm_ring_launch): bf16 operands in whole 16-byte pieces (k-contiguous ones aligned; of others the rows may be
// 8-byte aligned and the last tile start where it ends with the matrix, GemmArgs::m_last / n_last), slices below 2 GiB, RING_MIN_T
// k-tiles or more per output tile, output rows in whole aligned pieces of VB bytes.
#pragma once
#include "gemm_big.h"

namespace hfta {

constexpr int RING_BK = 64, RING_THREADS = 512, RING_SLOTS = 5, RING_GM = 4;
constexpr uint32_t RING_SLOT = 256 * RING_BK * 2;
constexpr uint32_t RING_SMEM = RING_SLOTS * RING_SLOT;
static_assert(RING_SMEM == 160 * 1024, "all of a compute unit's LDS");
constexpr int RING_MIN_T = 3;                            // k-tiles per output tile, see the loader
constexpr int RING_NT = 2;                               // cache policy of the stores: non-temporal

// A lane's fragment addresses (DmaOp::frag) as a few lane offsets and constants, for NB blocks of 32 rows / columns from `base`
template <bool KC, int NB> struct RingFrag {
  typedef DmaOp<256, RING_BK, KC, 8> Op;
  static constexpr int NO = KC ? 4 : NB;
  uint32_t o[NO];
  __device__ __forceinline__ void init(int base, int lane) {
    if (KC) {
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        const int r = base + (lane & 31);
        o[s] = (uint32_t)(r * (RING_BK * 2) + (((2 * s + (lane >> 5)) ^ Op::swz(r)) << 4));
      }
    } else {
      const int r16 = lane & 15, k = 8 * (lane >> 5) + (r16 >> 2);
#pragma unroll
      for (int i = 0; i < NO; ++i) {
        const int piece = ((base + 32 * i) >> 3) + 2 * ((lane >> 4) & 1) + ((r16 & 3) >> 1);
        o[i] = (uint32_t)(k * 512 + ((piece ^ Op::swz(k)) << 4) + (r16 & 1) * 8);
      }
    }
  }
  __device__ __forceinline__ bf16x8_t get(const unsigned char* tile, int i, int s) const {
    // 32 rows on, the high bit of the permutation flips: that of the k-step's piece
    if (KC) return *reinterpret_cast<const bf16x8_t*>(tile + o[(s ^ (2 * (i & 1))) & (NO - 1)] + i * 32 * RING_BK * 2);
    typedef __attribute__((address_space(3))) pf_v4s* lds_v4s;
    union { pf_v4s h[2]; bf16x8_t v; } u;
    const unsigned char* a0 = tile + o[i & (NO - 1)] + s * 16 * 512;
    u.h[0] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4s)(a0));
    u.h[1] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4s)(a0 + 4 * 512));
    return u.v;
  }
};

template <int N> __device__ __forceinline__ void ring_wait_barrier() {
  __builtin_amdgcn_sched_barrier(0);
  dma_wait_barrier<N>();
  __builtin_amdgcn_sched_barrier(0);
}

// LATE: every workgroup has one tile (vtotal <= gridDim.x).
template <bool A_KC, bool B_KC, typename OutT, bool COLB, int ACT, int VB, bool LATE = false>
__global__ __launch_bounds__(RING_THREADS, 2) void gemm_ring_kernel(GemmArgs p, int vgx, int vtotal) {
  __shared__ __attribute__((aligned(1024))) unsigned char smem[RING_SMEM];
  typedef DmaOp<256, RING_BK, A_KC, 8> OpA;
  typedef DmaOp<256, RING_BK, B_KC, 8> OpB;
  constexpr int ES = sizeof(OutT);
  constexpr int NSTORE = 4 * (ES == 2 ? 1 : 2) * (4096 / VB / 64);     // a lane's stores per output tile
  static_assert(OpA::NC == 4 && OpB::NC == 4 && 4 + NSTORE < 64, "the counts of the waits");
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wm = wave >> 2, wn = wave & 3;               // 2 x 4 wavefronts, 128 x 64 each
  typedef __attribute__((address_space(3))) unsigned char* lds_ptr;
  const uint32_t lds0 = (uint32_t)(uintptr_t)(lds_ptr)smem;
  const bool to_partial = ES == 4 && p.splits > 1;
  const int groups = vtotal / vgx / p.splits;

  // tile lin of the (row and column tiles, groups x splits) numbering: a contiguous range per XCD, row tiles in groups
  auto coord = [&](int lin) {
    const int per = vtotal >> 3;
    const int l2 = lin < (per << 3) ? (lin & 7) * per + (lin >> 3) : lin;
    const int bz = l2 / vgx, bx = l2 - bz * vgx;
    const int wid = RING_GM * p.tiles_n, grp = bx / wid, first = grp * RING_GM, rows = min(p.tiles_m - first, RING_GM), in = bx - grp * wid;
    BigCoord c;
    const int tn = in / rows;
    c.n0 = min(tn * 256, p.n_last);
    c.m0 = min((first + in - tn * rows) * 256, p.m_last);
    c.g = bz / p.splits;
    c.split = bz - c.g * p.splits;
    c.g0 = c.g / p.G1;
    c.g1 = c.g - c.g0 * p.G1;
    c.t_begin = (int)((int64_t)p.total_tiles * c.split / p.splits);
    c.t_end = (int)((int64_t)p.total_tiles * (c.split + 1) / p.splits);
    return c;
  };

  // The loader: operand tiles A, B, A, B, ... into the slots in turn.  A is up to a k-tile ahead of B, so each has a position
  // of its own; with three k-tiles or more per output tile B enters a tile after A has and before A leaves it, and the k-loop
  // after B: one set of coordinates does for all.
  OpA oa;
  OpB ob;
  struct Pos { const bf16_raw* base; int k0, left, K; };
  Pos pa, pb;
  int a_lin = blockIdx.x;
  BigCoord nxt = coord(a_lin);                           // of the tile A is in
  auto enter = [&](Pos& q, const bf16_raw* base, int64_t ss) {
    const bool live = a_lin < vtotal;
    const int seg = p.splits > 1 ? nxt.t_begin / p.tiles_per_seg : 0;
    q.k0 = (nxt.t_begin - seg * p.tiles_per_seg) * RING_BK;
    q.base = base + seg * ss;
    q.left = live ? nxt.t_end - nxt.t_begin : 1 << 30;
    q.K = live ? p.K : 0;                                // past the last tile: out of range, zeros, no memory request
  };
  auto enterA = [&]() {
    oa.init(nxt.m0, p.M, p.a_ld, wave, lane);
    enter(pa, reinterpret_cast<const bf16_raw*>(p.A) + nxt.g0 * p.a_g0 + nxt.g1 * p.a_g1, p.a_ss);
  };
  auto enterB = [&]() {
    ob.init(nxt.n0, p.N, p.b_ld, wave, lane);
    enter(pb, reinterpret_cast<const bf16_raw*>(p.Bm) + nxt.g0 * p.b_g0 + nxt.g1 * p.b_g1, p.b_ss);
  };
  auto next_slot = [](uint32_t s) { s += RING_SLOT; return s == RING_SMEM ? 0u : s; };
  uint32_t fill = 0, slotA = 0, slotB = 0;               // byte offset of the next slot to fill, addresses of those being filled
  dma_i32x4 rA, rB;
  // loads [i0, i1) of A's / B's next k-tile
  auto fetchA = [&](int i0, int i1) {
    if (i0 == 0) { rA = dma_rsrc(pa.base, p.a_extent); slotA = lds0 + fill; fill = next_slot(fill); }
#pragma unroll
    for (int i = 0; i < OpA::NC; ++i)
      if (i >= i0 && i < i1) oa.load(i, slotA, rA, pa.k0, pa.K, wave, lane);
    if (i1 == OpA::NC) {
      pa.k0 += RING_BK;
      if (--pa.left == 0) {
        a_lin += gridDim.x;
        if (a_lin < vtotal) nxt = coord(a_lin);
        enterA();
      } else if (pa.k0 >= p.K) {
        pa.k0 = 0;
        pa.base += p.a_ss;
      }
    }
  };
  auto fetchB = [&](int i0, int i1) {
    if (i0 == 0) { rB = dma_rsrc(pb.base, p.b_extent); slotB = lds0 + fill; fill = next_slot(fill); }
#pragma unroll
    for (int i = 0; i < OpB::NC; ++i)
      if (i >= i0 && i < i1) ob.load(i, slotB, rB, pb.k0, pb.K, wave, lane);
    if (i1 == OpB::NC) {
      pb.k0 += RING_BK;
      if (--pb.left == 0) {
        enterB();
      } else if (pb.k0 >= p.K) {
        pb.k0 = 0;
        pb.base += p.b_ss;
      }
    }
  };

  const int ml = lane & 31;
  const bool hi = lane >= 32;                            // lane l holds row l % 32, columns 8q + 4(l / 32) .. + 3 of a block
  RingFrag<A_KC, 4> fa;
  RingFrag<B_KC, 2> fb;
  fa.init(wm * 128, lane);
  fb.init(wn * 64, lane);
  bf16x8_t a[2][4], b[2][2];
  auto read = [&](int set, uint32_t sa, uint32_t sb, int s) {
#pragma unroll
    for (int j = 0; j < 2; ++j) b[set][j] = fb.get(smem + sb, j, s);
#pragma unroll
    for (int i = 0; i < 4; ++i) a[set][i] = fa.get(smem + sa, i, s);
  };
  f32x16_t acc[4][2];
  auto mul = [&](int set, int i0) {                      // two rows of blocks
#pragma unroll
    for (int i = i0; i < i0 + 2; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(b[set][j], a[set][i], acc[i][j], 0, 0, 0);
    __builtin_amdgcn_sched_barrier(0);
  };

  enterA();
  enterB();
  BigCoord cur = nxt;
  fetchA(0, 4);
  fetchB(0, 4);
  fetchA(0, 4);
  fetchB(0, 4);
  ring_wait_barrier<8>();
  uint32_t sa = 0, sb = RING_SLOT;                       // slots of the k-tile being read
  read(0, sa, sb, 0);
  bool after_stores = false;
  for (int lin = blockIdx.x;;) {
    const int T = cur.t_end - cur.t_begin;
    // The bias is the accumulators' initial value where a workgroup walks several tiles and is added to the finished sums where it
    // has one: the order of the kernel that each took the place of (gemm_bigp_kernel, gemm_big_kernel), whose bits these are.  (8 x 2048
    // rows, 256 -> 1024, one tile each: 16.2 us, 16.5 with the bias first.)  Column biases come by scalar loads (the same 64 columns
    // for all lanes).
    auto take_bias = [&]() {
      const bf16_raw* bias = p.bias ? reinterpret_cast<const bf16_raw*>(p.bias) + cur.g0 * p.bias_g0 + cur.g1 * p.bias_g1 : nullptr;
      if (COLB) {
        typedef const __attribute__((address_space(4))) uint2* cptr;
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            const int n = cur.n0 + wn * 64 + j * 32 + 8 * q;
            uint32_t c[4] = {0u, 0u, 0u, 0u};              // N is a multiple of 4
            if (n + 4 <= p.N) { const cptr s = (cptr)(uintptr_t)(bias + n); c[0] = s->x; c[1] = s->y; }
            if (n + 8 <= p.N) { const cptr s = (cptr)(uintptr_t)(bias + n + 4); c[2] = s->x; c[3] = s->y; }
            const uint32_t x = hi ? c[2] : c[0], y = hi ? c[3] : c[1];
            const float v[4] = {__uint_as_float(x << 16), __uint_as_float(x & 0xffff0000u), __uint_as_float(y << 16),
                                __uint_as_float(y & 0xffff0000u)};
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
              for (int e = 0; e < 4; ++e) acc[i][j][4 * q + e] = LATE ? acc[i][j][4 * q + e] + v[e] : v[e];
          }
      } else {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int m = cur.m0 + wm * 128 + i * 32 + ml;
          const float bm = bias && m < p.M ? bf16_to_f32(bias[m]) : 0.f;
#pragma unroll
          for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][j][v] = LATE ? acc[i][j][v] + bm : bm;
        }
      }
    };
    if constexpr (LATE) {
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
          for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;
    } else {
      take_bias();
    }
    __builtin_amdgcn_sched_barrier(0);
    for (int kt = 0;; ++kt) {
      const bool last = kt + 1 == T;
      read(1, sa, sb, 1);
      mul(0, 0);
      if (kt) fetchB(2, 4);                              // the rest of the tile begun at the last barrier
      mul(0, 2);
      read(0, sa, sb, 2);
      mul(1, 0);
      fetchA(0, 2);
      mul(1, 2);
      read(1, sa, sb, 3);
      mul(0, 0);
      fetchA(2, 4);
      mul(0, 2);
      // The next k-tile has landed (what may be out is A's tile behind it, and stores older than that) and this one's slots
      // are read by all: its last k-step is in registers.
      if (after_stores && kt == 0) ring_wait_barrier<4 + NSTORE>();
      else ring_wait_barrier<4>();
      const uint32_t na = next_slot(sb), nb = next_slot(na);
      read(0, na, nb, 0);
      mul(1, 0);
      fetchB(0, 2);
      mul(1, 2);
      if (last) break;
      sa = na;
      sb = nb;
    }
    fetchB(2, 4);
    if constexpr (LATE) take_bias();
    // Epilogue: slot sb, which the loader fills next after the barrier at the end, as staging.
    unsigned char* priv = smem + sb + wave * 4096;
    OutT* Cb = to_partial
        ? reinterpret_cast<OutT*>(p.partial) + ((int64_t)cur.split * groups + cur.g) * (int64_t)p.M * p.N
        : reinterpret_cast<OutT*>(p.C) + cur.g0 * p.c_g0 + cur.g1 * p.c_g1;
    const uint32_t c_ldb = (uint32_t)((to_partial ? (int64_t)p.N : p.c_ld) * ES);
    const __amdgpu_buffer_rsrc_t rc = pf_rsrc(Cb, to_partial ? (uint32_t)((int64_t)p.M * p.N * 4) : p.c_extent);
    // Non-temporal stores where a wavefront's 128 bytes of a row are a cache line and nothing reads them next.  Elsewhere they
    // lose: rows of 10000 bytes 56 -> 70 us (4 x 3000 x 5000, K = 256), partial sums of split products 82 -> 88.
    const bool stream = VB == 16 && !to_partial && ((uint32_t)(uintptr_t)Cb | c_ldb | (uint32_t)p.c_seg) % 128 == 0;
    constexpr int JB = ES == 2 ? 1 : 2;                  // 128 bytes of a row at a time: all 64 columns or half of them
    constexpr int PPR = 128 / VB, RPI = 64 / PPR, NP = 32 / RPI;
    const int rr = lane / PPR, pc = lane % PPR;
#pragma unroll
    for (int jb = 0; jb < JB; ++jb) {
      const int n = cur.n0 + wn * 64 + jb * 32 + pc * (VB / ES);
      const uint32_t colb = n + VB / ES <= p.N
          ? (uint32_t)((to_partial ? (int64_t)n : col_offset(n, p.c_seg, p.c_seg_stride)) * ES) : PF_OOB;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        // 16-byte piece x of row r sits at x ^ (r / 2 % 8): rows of 128 bytes, no bank conflicts either way
#pragma unroll
        for (int j = 0; j < (ES == 2 ? 2 : 1); ++j)
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            float x[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) x[e] = big_act<ACT>(acc[i][ES == 2 ? j : jb][4 * q + e], p.slope);
            unsigned char* row = priv + ml * 128;
            const int sw = (ml >> 1) & 7;
            if (ES == 2)
              *reinterpret_cast<uint2*>(row + (((j * 4 + q) ^ sw) << 4) + (hi ? 8 : 0)) = make_uint2(pack_bf16x2(x[0], x[1]), pack_bf16x2(x[2], x[3]));
            else
              *reinterpret_cast<float4*>(row + (((2 * q + (hi ? 1 : 0)) ^ sw) << 4)) = make_float4(x[0], x[1], x[2], x[3]);
          }
        typedef typename std::conditional<VB == 16, pf_u32x4, pf_u32x2>::type V;
        V v[NP];
#pragma unroll
        for (int h = 0; h < NP; ++h) {
          const int r = rr + h * RPI;
          v[h] = *reinterpret_cast<const V*>(priv + r * 128 + ((((pc * VB) >> 4) ^ ((r >> 1) & 7)) << 4) + ((pc * VB) & 15));
        }
#pragma unroll
        for (int h = 0; h < NP; ++h) {
          const int m = cur.m0 + wm * 128 + i * 32 + rr + h * RPI;
          const uint32_t off = (m < p.M && colb != PF_OOB) ? (uint32_t)m * c_ldb + colb : PF_OOB;
          if constexpr (VB == 16) {
            if (stream) __builtin_amdgcn_raw_buffer_store_b128(v[h], rc, (int)off, 0, RING_NT);
            else __builtin_amdgcn_raw_buffer_store_b128(v[h], rc, (int)off, 0, 0);
          } else {
            __builtin_amdgcn_raw_buffer_store_b64(v[h], rc, (int)off, 0, 0);
          }
        }
      }
    }
    lin += gridDim.x;
    if (LATE || lin >= vtotal) break;
    // every wavefront is through with the staging slot
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
    cur = nxt;
    sa = next_slot(sb);
    sb = next_slot(sa);
    after_stores = true;
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");       // nothing may land in LDS any more
}

int persistent_blocks();     // compute units, in whole XCD rounds
int gemm_ring_launch(const GemmDesc& d, const GemmArgs& a, dim3 grid, hipStream_t st);

}  // namespace hfta
