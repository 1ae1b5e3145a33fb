// Forward product of the fp32 one-operator tail (conv_pool_f32.hip): k=1 convolution of 65 to 128 channels whose output is not
// stored; what leaves are GemmDesc::pool_part's four numbers per (sample, 128-point tile, channel).
//
// In the general fp32 product (gemm_f32.hip) a 128 x 128 tile's operands are split into their three bf16 parts anew for each of the
// eight row tiles that share x and the 2560 column tiles that share W, pass through LDS as six planes, and the tile's output is
// staged to be summed: 690 us for 4 x 32 x 2500 points, 128 -> 1024 channels, where the matrix instructions need 234.  Here a
// wavefront splits its 32 points' x once and keeps the parts in registers (96 of them) while it walks the channels; W is split once
// per call, in the order the instructions read it, and arrives in LDS by loads that go straight there, two blocks of 32 channels
// ahead; and the sums come from the accumulators, whose rows a lane pair holds, between the next block's
// matrix instructions.  Measured: 437 us, and 6 for W's parts (without the interleaving 474); the 4 models' step 2068 -> 1812.
//
// The bits are those of the general product's epilogue: the same instructions in the same order per output, and the same order of
// every sum (a row's 128 columns are four quarters of four interleaved chains).  (Rows with a negative gamma, whose smallest value
// is looked for, keep their signs in the product: the bf16 instruction's sums of negated factors are not always the negated sums.)
//
// Bound: the matrix instructions, 48 of 32 cycles per block and wavefront, beside about 200 vector instructions of the sums, which
// the second wavefront of a SIMD covers (two workgroups per compute unit: 80 KB of LDS, 256 registers).
#include "gemm_dma.h"
#include "f32_split.h"

namespace hfta {

namespace {

constexpr int PM_PTS = 128, PM_ROWS = 32, PM_STEPS = 8, PM_CHUNKS = PM_STEPS * 3;    // 1 KB: one plane's fragments of a k-step
constexpr int PM_BLOCK = PM_CHUNKS * 1024, PM_MAX_CO = 1024;

struct PoolMainArgs {
  const float* X; const float* W; const float* bias; const float* gamma; float4* part;
  unsigned char* pack;            // [B][row blocks][k-step][plane][lane][8 bf16]
  int* bad;                       // [B][row blocks]: W has a value without a split
  int64_t xsb, xsn, xsc;
  int B, Nb, Ci, Co, L, tiles, blocks;
  uint32_t x_extent;
};

// W as three bf16 planes in fragment order: lane l of a k-step holds row l % 32 and k = 16 s + 8 (l / 32) + 0..7.  A workgroup per 32 rows.
__global__ __launch_bounds__(256) void pool32_pack_kernel(PoolMainArgs p) {
  const int blk = blockIdx.x, b = blockIdx.y;
  SplitSeen seen;
#pragma unroll
  for (int u = 0; u < PM_STEPS * 64 / 256; ++u) {
    const int i = threadIdx.x + 256 * u, lane = i & 63, s = i >> 6;
    const int row = blk * PM_ROWS + (lane & 31), k0 = 16 * s + 8 * (lane >> 5);
    float e[8];
    const bool live = row < p.Co;
    const float* w = p.W + ((int64_t)b * p.Co + (live ? row : 0)) * p.Ci;
#pragma unroll
    for (int j = 0; j < 8; ++j) e[j] = live && k0 + j < p.Ci ? w[k0 + j] : 0.f;
    uint2 lo[3], hi[3];
    split4(make_float4(e[0], e[1], e[2], e[3]), lo, seen);
    split4(make_float4(e[4], e[5], e[6], e[7]), hi, seen);
    unsigned char* d = p.pack + ((int64_t)b * p.blocks + blk) * PM_BLOCK + s * 3072 + lane * 16;
#pragma unroll
    for (int pl = 0; pl < 3; ++pl) *reinterpret_cast<uint4*>(d + pl * 1024) = make_uint4(lo[pl].x, lo[pl].y, hi[pl].x, hi[pl].y);
  }
  const int any = __syncthreads_or(seen.bad());
  if (threadIdx.x == 0) p.bad[b * p.blocks + blk] = any;
}

__global__ __launch_bounds__(256, 2) void pool32_main_kernel(PoolMainArgs p) {
  __shared__ __attribute__((aligned(1024))) unsigned char wbuf[3][PM_BLOCK];
  __shared__ float qs[2][4][PM_ROWS], sq[2][4][PM_ROWS], mx[2][4][PM_ROWS], tot[2][PM_ROWS];
  __shared__ uint8_t mat[2][4][PM_ROWS];
  __shared__ float bl[PM_MAX_CO];                        // bias
  __shared__ uint32_t flips[PM_MAX_CO / 32];             // bit per channel: gamma < 0
  const int t = threadIdx.x, lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const int r = lane & 31, h = lane >> 5;
  int tile, g;
  dma_renumber(blockIdx.x, p.tiles, p.tiles * p.Nb * p.B, tile, g);
  const int b = g / p.Nb, n = g - b * p.Nb;
  const int n0 = tile * PM_PTS, c0 = wave * 32;          // the wavefront's quarter of the tile's columns
  const float* xb = p.X + b * p.xsb + n * p.xsn;
  const float* Wb = p.W + (int64_t)b * p.Co * p.Ci;

  // ---- W blocks straight into LDS, six 1 KB chunks a wavefront; past the last block nothing is requested ----
  typedef __attribute__((address_space(3))) unsigned char* lds_ptr;
  const uint32_t lds0 = (uint32_t)(uintptr_t)(lds_ptr)&wbuf[0][0];
  const dma_i32x4 rw = dma_rsrc(p.pack + (int64_t)b * p.blocks * PM_BLOCK, (uint32_t)(p.blocks * PM_BLOCK));
  auto fetch = [&](int blk, int buf) {
#pragma unroll
    for (int i = 0; i < 6; ++i) {
      const uint32_t at = (uint32_t)(wave * 6 + i) * 1024u;
      dma_load(lds0 + (uint32_t)buf * PM_BLOCK + at, blk < p.blocks ? (uint32_t)blk * PM_BLOCK + at + (uint32_t)lane * 16u : PF_OOB, rw);
    }
  };
  fetch(0, 0);
  fetch(1, 1);

  // ---- x of this wavefront's 32 points: lane l holds point l % 32 and k = 16 s + 8 (l / 32) + 0..7 ----
  bf16x8_t xf[PM_STEPS][3];
  bool xbad;
  {
    const __amdgpu_buffer_rsrc_t rx = pf_rsrc(xb, p.x_extent);
    const int col = n0 + c0 + r;
    const uint32_t ld = (uint32_t)(p.xsc * 4);
    SplitSeen seen;
#pragma unroll
    for (int s0 = 0; s0 < PM_STEPS; s0 += 4) {
      float e[4][8];
#pragma unroll
      for (int s = 0; s < 4; ++s)
#pragma unroll
        for (int j = 0; j < 8; ++j) {
          const int k = 16 * (s0 + s) + 8 * h + j;
          e[s][j] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rx, (int)(k < p.Ci && col < p.L ? (uint32_t)k * ld + (uint32_t)col * 4u : PF_OOB), 0, 0));
        }
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        uint2 lo[3], hi[3];
        split4(make_float4(e[s][0], e[s][1], e[s][2], e[s][3]), lo, seen);
        split4(make_float4(e[s][4], e[s][5], e[s][6], e[s][7]), hi, seen);
#pragma unroll
        for (int pl = 0; pl < 3; ++pl) {
          const uint4 v = make_uint4(lo[pl].x, lo[pl].y, hi[pl].x, hi[pl].y);
          xf[s0 + s][pl] = *reinterpret_cast<const bf16x8_t*>(&v);
        }
      }
    }
    for (int c = t; c < p.blocks * PM_ROWS; c += 256) {
      const bool live = c < p.Co;
      bl[c] = live && p.bias ? p.bias[(int64_t)b * p.Co + c] : 0.f;
      const unsigned long long m = __ballot(live && p.gamma[(int64_t)b * p.Co + c] < 0.f);
      if (r == 0) flips[c >> 5] = (uint32_t)(m >> (32 * h));
    }
    xbad = __syncthreads_or(seen.bad());
  }

  const int all = min(p.L - n0, PM_PTS), cnt = min(max(p.L - n0 - c0, 0), 32);
  // A lane pair (l, l + 32) holds a row's 32 columns; after the exchange the lower lane has those = 0, 1 mod 4, the upper those = 2, 3:
  // val[e][q] is column 4 q + 2 h + e
  float val[2][8];
#pragma unroll
  for (int q = 0; q < 8; ++q) val[0][q] = val[1][q] = 0.f;
  auto column = [&](int e, int q) { return 4 * q + 2 * h + e; };
  // a quarter's sum from its four chains, (0 + 1) + (2 + 3)
  auto quarter = [&](const float (&s)[2]) {
    const float pair = s[0] + s[1];
    return pair + __shfl_xor(pair, 32, 64);
  };
  auto write = [&](int i) {
    const int o = i & 1, m = i * PM_ROWS + r;
    if (h != 0 || m >= p.Co) return;
    const float s2 = (sq[o][0][r] + sq[o][1][r]) + (sq[o][2][r] + sq[o][3][r]);
    float best = mx[o][0][r];
    int at = mat[o][0][r];
#pragma unroll
    for (int w = 1; w < 4; ++w)                          // columns ascend: the first of equal ones stays
      if (mx[o][w][r] > best) { best = mx[o][w][r]; at = mat[o][w][r]; }
    p.part[((int64_t)g * p.tiles + tile) * p.Co + m] = make_float4(tot[o][r], s2, best, __int_as_float(n0 + at));
  };

  // EDGE: the row's last tile.  EXACT: some block of this model, or this tile's x, may need the fp32 instruction.
  auto walk = [&](auto edge_c, auto exact_c) {
    constexpr bool EDGE = decltype(edge_c)::value, EXACT = decltype(exact_c)::value;
    // With block i's whole sums known: squares about the tile's mean, largest value and its first column, in eight parts that stand
    // between the next block's matrix instructions
    float mean = 0.f, sum = 0.f, s2[2], best = 0.f;
    int at = 0;
    uint32_t sign = 0;
    auto part = [&](int i, int s) {
      if (s == 0) {
        const int o = i & 1;
        sum = (qs[o][0][r] + qs[o][1][r]) + (qs[o][2][r] + qs[o][3][r]);
        mean = sum / (float)all;
        sign = (flips[max(i, 0)] >> r & 1) << 31;                // gamma < 0: the smallest
        s2[0] = s2[1] = 0.f;
        best = -INFINITY;
        at = 0;
      }
#pragma unroll
      for (int q = 2 * s; q < 2 * s + 2 && s < 4; ++q)
#pragma unroll
        for (int e = 0; e < 2; ++e) {
          const float d = !EDGE || column(e, q) < cnt ? val[e][q] - mean : 0.f;
          s2[e] = fmaf(d, d, s2[e]);
          val[e][q] = __uint_as_float(__float_as_uint(val[e][q]) ^ sign);
          if (EDGE) val[e][q] = column(e, q) < cnt ? val[e][q] : -INFINITY;
          best = fmaxf(best, val[e][q]);
        }
#pragma unroll
      for (int q = 15 - 2 * s; q > 13 - 2 * s && s >= 4; --q)
#pragma unroll
        for (int e = 1; e >= 0; --e) at = val[e][q] == best ? column(e, q) : at;
    };
    auto leave = [&](int i) {
      const int o = i & 1;
      const float sqr = quarter(s2);
      const float ob = __shfl_xor(best, 32, 64);
      const int oa = __shfl_xor(at, 32, 64);
      if (ob > best || (ob == best && oa < at)) { best = ob; at = oa; }
      if (h == 0) {
        sq[o][wave][r] = sqr;
        mx[o][wave][r] = best;
        mat[o][wave][r] = (uint8_t)(c0 + at);
        if (wave == 0) tot[o][r] = sum;
      }
    };
    int buf = 0;
    for (int i = 0; i < p.blocks; ++i) {
      // W's block i has landed (the next one's six loads may be out), the block before and the sums before that are read by all
      dma_wait_barrier<6>();
      fetch(i + 2, buf == 0 ? 2 : buf - 1);
      if (i > 1 && wave == (i & 3)) write(i - 2);
      f32x16_t acc, low;
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[v] = low[v] = 0.f;
      const int* fl = p.bad + b * p.blocks + (i & ~3);
      bool exact = false;
      if constexpr (EXACT) {
        exact = xbad;
        for (int k = 0; k < 4 && (i & ~3) + k < p.blocks; ++k) exact = exact || fl[k];      // 128 rows at a time, as the general product
      }
      if (!EXACT || !exact) {
        const unsigned char* ws = wbuf[buf] + lane * 16;
        bf16x8_t a[2][3];
        auto frags = [&](int s) {
#pragma unroll
          for (int pl = 0; pl < 3; ++pl) a[s & 1][pl] = *reinterpret_cast<const bf16x8_t*>(ws + s * 3072 + pl * 1024);
        };
        frags(0);
#pragma unroll
        for (int s = 0; s < PM_STEPS; ++s) {
          if (s + 1 < PM_STEPS) frags(s + 1);
          constexpr int PA[6] = {2, 1, 0, 1, 0, 0}, PB[6] = {0, 1, 2, 0, 1, 0};
#pragma unroll
          for (int q = 0; q < 6; ++q) {
            f32x16_t& c = q < 5 ? low : acc;
            c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(xf[s][PB[q]], a[s & 1][PA[q]], c, 0, 0, 0);
          }
          part(i - 1, s);                                // (before the first block: of nothing, and not kept)
          __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[v] += low[v];
      } else {
#pragma unroll
        for (int s = 0; s < PM_STEPS; ++s) part(i - 1, s);
        // a value without a split: the fp32 instruction, from memory
        const int row = i * PM_ROWS + r, col = n0 + c0 + r;
        const bool rok = row < p.Co, cok = col < p.L;
        for (int k8 = 0; k8 < p.Ci; k8 += 8) {
          const int k0 = k8 + 4 * h;
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            const bool kok = k0 + j < p.Ci;
            const float w = rok && kok ? Wb[(int64_t)row * p.Ci + k0 + j] : 0.f, x = cok && kok ? xb[(int64_t)(k0 + j) * p.xsc + col] : 0.f;
            acc = __builtin_amdgcn_mfma_f32_32x32x2f32(x, w, acc, 0, 0, 0);
          }
        }
      }
      if (i > 0) leave(i - 1);
      const float bm = bl[i * PM_ROWS + r];
      float s1[2] = {0.f, 0.f};
#pragma unroll
      for (int q = 0; q < 4; ++q) {
#pragma unroll
        for (int e = 0; e < 2; ++e) {
          const float lo = acc[4 * q + e] + bm, hi = acc[4 * q + e + 2] + bm;    // columns 8 q + 4 h + e, + 2
          const auto x = __builtin_amdgcn_permlane32_swap(__float_as_uint(lo), __float_as_uint(hi), false, false);
          val[e][2 * q] = __uint_as_float(x[0]);
          val[e][2 * q + 1] = __uint_as_float(x[1]);
        }
#pragma unroll
        for (int u = 2 * q; u < 2 * q + 2; ++u)
#pragma unroll
          for (int e = 0; e < 2; ++e) s1[e] += !EDGE || column(e, u) < cnt ? val[e][u] : 0.f;
      }
      const float one = quarter(s1);
      if (h == 0) qs[i & 1][wave][r] = one;
      buf = buf == 2 ? 0 : buf + 1;
    }
    dma_wait_barrier<0>();
#pragma unroll
    for (int s = 0; s < PM_STEPS; ++s) part(p.blocks - 1, s);
    leave(p.blocks - 1);
  };
  bool bad = xbad;
  for (int k = lane; k < p.blocks; k += 64) bad = bad || p.bad[b * p.blocks + k];
  bad = __any(bad);
  const bool edge = n0 + PM_PTS > p.L;                   // columns past the end do not take part
  if (bad) walk(std::true_type{}, std::true_type{});
  else if (edge) walk(std::true_type{}, std::false_type{});
  else walk(std::false_type{}, std::false_type{});
  if (p.blocks > 1 && wave == 0) write(p.blocks - 2);
  __syncthreads();
  if (wave == 1) write(p.blocks - 1);
}

}  // namespace

// bytes of W's planes and flags
size_t pool32_pack_bytes(int B, int Co) {
  return (size_t)B * ((Co + 31) / 32) * PM_BLOCK + (((size_t)B * ((Co + 31) / 32) * sizeof(int) + 255) & ~(size_t)255);
}

// pool_part of the product; part: as GemmDesc::pool_part with 128-column tiles.  The caller has checked the shape (65 <= Ci <= 128, Ci % 4
// == 0, Co <= 1024).  HFTA_EUNSUPPORTED: a sample's x does not fit a buffer descriptor (nothing has been launched).
int pool32_main(int B, int Nb, int Ci, int Co, int L, const float* X, const int64_t xs[4], const float* W, const float* bias,
                const float* gamma, float4* part, void* scratch, hipStream_t st) {
  const int64_t x_bytes = ((int64_t)(Ci - 1) * xs[2] + L) * 4;
  if (x_bytes >= (int64_t)1 << 31 || xs[2] <= 0) return HFTA_EUNSUPPORTED;
  PoolMainArgs a{};
  a.X = X; a.W = W; a.bias = bias; a.gamma = gamma; a.part = part;
  a.B = B; a.Nb = Nb; a.Ci = Ci; a.Co = Co; a.L = L; a.tiles = (L + PM_PTS - 1) / PM_PTS; a.blocks = (Co + PM_ROWS - 1) / PM_ROWS;
  a.pack = (unsigned char*)scratch;
  a.bad = (int*)(a.pack + (size_t)B * a.blocks * PM_BLOCK);
  a.xsb = xs[0]; a.xsn = xs[1]; a.xsc = xs[2];
  a.x_extent = (uint32_t)x_bytes;
  const int64_t wgs = (int64_t)a.tiles * Nb * B;
  if (wgs > 0x7fffffff) return HFTA_EUNSUPPORTED;
  hipLaunchKernelGGL(pool32_pack_kernel, dim3((unsigned)a.blocks, (unsigned)B), dim3(256), 0, st, a);
  if (launch_status() != HFTA_OK) return HFTA_ELAUNCH;
  hipLaunchKernelGGL(pool32_main_kernel, dim3((unsigned)wgs), dim3(256), 0, st, a);
  return launch_status();
}

}  // namespace hfta
