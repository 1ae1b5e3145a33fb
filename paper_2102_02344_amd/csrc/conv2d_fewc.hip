// Data gradient of a grouped 4x4 / stride 2 / pad 1 convolution with at most 4 input channels (the
// DCGAN generator's last transposed convolution 64 -> 3 and the discriminator's first layer 3 -> 64;
// fusion rules table, rows "Conv2d" / "ConvTranspose2d").  With 3 rows a matrix-instruction tile is
// 95 % empty and the column-tile gather of the implicit GEMM costs as much as for a full tile, so
// this is plain vector arithmetic:
//     dX[c][2qy+py][2qx+px] = sum_o sum_{(ky,r) in S(py)} sum_{(kx,s) in S(px)} W[o][c][ky][kx] dY[o][qy-1+r][qx-1+s]
//     S(0) = {(1,1), (3,0)},  S(1) = {(0,2), (2,1)}
// One thread owns one q pixel (or two, one above the other: ROWS): the 2x2 output block of every channel (4 Ci accumulators) against the
// 3x3 neighbourhood of dY, 16 Ci multiply-adds per output channel o.  A workgroup covers 32 x 8 ROWS q
// pixels; dY goes through LDS sixteen channels at a time (10 x 36 halo tile; eight of 18 x 36); the weights are the same
// for every thread of a workgroup and are read with scalar loads (they occupy the scalar unit and
// scalar registers, not LDS bandwidth or vector instructions).
//
// The halo travels in pairs of columns (4 bytes) by buffer loads whose addresses are formed once: element by element, with the
// places worked out for each eight channels anew, the staging cost more vector instructions than the multiply-adds, and a
// launch of one workgroup per compute unit waited for eight round trips to memory instead of four, and for the scalar unit in
// every channel (see the loop).  3 x 20 samples of 64 -> 3 channels at 64 x 64: 44 -> 30 us; 10 x 64 fill the chip and are bound by
// LDS reads, multiply-adds and the scalar unit, which takes a bf16 weight apart per use: there a thread owns two rows of q pixels, so that
// 96 multiply-adds stand beside 48 scalar instructions and 12 LDS reads instead of 48 beside 48 and 9: 121 -> 91 us.  Rows of an odd number
// of q pixels, or not on 4 bytes, keep the elements, and one row.
#include "gemm_pf.h"

namespace hfta {

namespace {

constexpr int FC_TX = 32, FC_TY = 8;                       // q tile
constexpr int FC_PW = FC_TX + 2 + 2;                       // halo row pitch (elements): columns -2 .. 33

struct FewcArgs {
  const bf16_raw* Wt; const bf16_raw* dY; bf16_raw* dX;
  int B, Nb, Co, H, W, Hq, Wq, tiles_x;
};

template <int CI, bool PAIR, int ROWS>
__global__ __launch_bounds__(256) void conv_dx_fewc_kernel(FewcArgs p) {
  constexpr int FC_OC = PAIR && ROWS == 1 ? 16 : 8;        // channels of dY per LDS stage
  constexpr int FC_PH = FC_TY * ROWS + 2;                  // halo rows
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  bf16_raw* tile = reinterpret_cast<bf16_raw*>(smem);                           // [2][FC_OC][FC_PH][FC_PW]
  const int t = threadIdx.x, tx = t & (FC_TX - 1), ty = t >> 5;
  const int qx0 = (blockIdx.x % p.tiles_x) * FC_TX, qy0 = (blockIdx.x / p.tiles_x) * FC_TY * ROWS;
  const int n = blockIdx.y, b = blockIdx.z;
  const int P = p.Hq * p.Wq;
  const bf16_raw* dy = p.dY + ((int64_t)n * p.B + b) * p.Co * P;
  const uint32_t* __restrict__ w2 = reinterpret_cast<const uint32_t*>(p.Wt + (int64_t)b * p.Co * CI * 16);   // pairs (kx, kx + 1)

  constexpr int TILE_EL = FC_OC * FC_PH * FC_PW;
  constexpr int COLS = PAIR ? FC_PW / 2 : FC_TX + 2, UNITS = FC_OC * FC_PH * COLS;      // pairs or elements per stage
  constexpr int PER_THREAD = (UNITS + 255) / 256;
  uint32_t stage[PER_THREAD], from[PER_THREAD], to[PER_THREAD];
#pragma unroll
  for (int i = 0; i < PER_THREAD; ++i) {
    const int e = t + 256 * i;
    const int col = e % COLS, r = e / COLS;
    const int row = r % FC_PH, oc = r / FC_PH;
    const int y = qy0 - 1 + row, x = qx0 + (PAIR ? 2 * col - 2 : col - 1);
    const bool ok = oc < FC_OC && y >= 0 && y < p.Hq && x >= 0 && x < p.Wq;
    from[i] = ok ? ((uint32_t)oc * (uint32_t)P + (uint32_t)(y * p.Wq + x)) * 2u : PF_OOB;                 // out of range: zeros, no memory request
    to[i] = (uint32_t)((oc * FC_PH + row) * FC_PW + (PAIR ? 2 * col : col + 1));
  }
  // a buffer per stage; what is read for channels past the last is not used
  auto fetch = [&](int o0) {
    const __amdgpu_buffer_rsrc_t rs = pf_rsrc(dy + (int64_t)o0 * P, (uint32_t)min(FC_OC, p.Co - o0) * (uint32_t)P * 2u);
#pragma unroll
    for (int i = 0; i < PER_THREAD; ++i)
      stage[i] = PAIR ? (uint32_t)__builtin_amdgcn_raw_buffer_load_b32(rs, (int)from[i], 0, 0)
                      : (uint32_t)(uint16_t)__builtin_amdgcn_raw_buffer_load_b16(rs, (int)from[i], 0, 0);
  };
  auto park = [&](int buf) {
#pragma unroll
    for (int i = 0; i < PER_THREAD; ++i)
      if (UNITS % 256 == 0 || t + 256 * i < UNITS) {
        if (PAIR) *reinterpret_cast<uint32_t*>(tile + buf * TILE_EL + to[i]) = stage[i];
        else tile[buf * TILE_EL + to[i]] = (bf16_raw)stage[i];
      }
  };

  float acc[CI][ROWS][2][2];
#pragma unroll
  for (int c = 0; c < CI; ++c)
#pragma unroll
    for (int j = 0; j < ROWS; ++j) acc[c][j][0][0] = acc[c][j][0][1] = acc[c][j][1][0] = acc[c][j][1][1] = 0.f;

  bf16_raw dn[ROWS + 2][3];
  uint32_t wn[CI * 8];
  // the three columns one by one: two neighbours in one 4-byte read are off four bytes in every other lane, which costs launches
  // that fill the chip twice the time
  int at[3] = {tx + 1, tx + 2, tx + 3};
#pragma unroll
  for (int s = 0; s < 3; ++s) asm("" : "+v"(at[s]));
  auto issue = [&](int o0, int buf, int oc) {
    const bf16_raw* tp = tile + buf * TILE_EL + (oc * FC_PH + ty * ROWS) * FC_PW;
#pragma unroll
    for (int r = 0; r < ROWS + 2; ++r)
#pragma unroll
      for (int s = 0; s < 3; ++s) dn[r][s] = tp[r * FC_PW + at[s]];
    const uint32_t* wq = w2 + (size_t)(o0 + oc) * CI * 8;        // uniform address: scalar loads
#pragma unroll
    for (int k = 0; k < CI * 8; ++k) wn[k] = wq[k];
  };

  fetch(0);
  park(0);
  __syncthreads();
  int buf = 0;
  for (int o0 = 0; o0 < p.Co; o0 += FC_OC) {
    const bool more = o0 + FC_OC < p.Co;
    if (more) fetch(o0 + FC_OC);
    // the weights and the neighbourhood of an output channel are on their way while the one before is multiplied: a scalar
    // load's round trip is longer than a channel's multiply-adds
    const int last = min(FC_OC, p.Co - o0) - 1;
    issue(o0, buf, 0);
#pragma unroll 2
    for (int oc = 0; oc <= last; ++oc) {
      float d[ROWS + 2][3];
      uint32_t w[CI * 8];
#pragma unroll
      for (int r = 0; r < ROWS + 2; ++r)
#pragma unroll
        for (int s = 0; s < 3; ++s) d[r][s] = bf16_to_f32(dn[r][s]);
#pragma unroll
      for (int k = 0; k < CI * 8; ++k) w[k] = wn[k];
      issue(o0, buf, min(oc + 1, last));
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int c = 0; c < CI; ++c) {
        float4 k[4];                                            // rows ky = 0..3
#pragma unroll
        for (int ky = 0; ky < 4; ++ky) {
          const uint32_t lo = w[c * 8 + ky * 2], hi = w[c * 8 + ky * 2 + 1];
          k[ky] = make_float4(__uint_as_float(lo << 16), __uint_as_float(lo & 0xffff0000u), __uint_as_float(hi << 16),
                              __uint_as_float(hi & 0xffff0000u));
        }
        const float4 k0 = k[0], k1 = k[1], k2 = k[2], k3 = k[3];
        // py = 0: (ky 1, r 1), (ky 3, r 0);  py = 1: (ky 0, r 2), (ky 2, r 1); the same pairs along x
#define HFTA_FC4(A, w0, x0, w1, x1, w2, x2, w3, x3) A = fmaf(w3, x3, fmaf(w2, x2, fmaf(w1, x1, fmaf(w0, x0, A))))
#pragma unroll
        for (int j = 0; j < ROWS; ++j) {
          float(&o)[2][2] = acc[c][j];
          HFTA_FC4(o[0][0], k1.y, d[j + 1][1], k1.w, d[j + 1][0], k3.y, d[j][1], k3.w, d[j][0]);
          HFTA_FC4(o[0][1], k1.x, d[j + 1][2], k1.z, d[j + 1][1], k3.x, d[j][2], k3.z, d[j][1]);
          HFTA_FC4(o[1][0], k0.y, d[j + 2][1], k0.w, d[j + 2][0], k2.y, d[j + 1][1], k2.w, d[j + 1][0]);
          HFTA_FC4(o[1][1], k0.x, d[j + 2][2], k0.z, d[j + 2][1], k2.x, d[j + 1][2], k2.z, d[j + 1][1]);
        }
#undef HFTA_FC4
      }
      __builtin_amdgcn_sched_barrier(0);
    }
    if (more) park(buf ^ 1);
    __syncthreads();
    buf ^= 1;
  }
#pragma unroll
  for (int j = 0; j < ROWS; ++j) {
    const int qx = qx0 + tx, qy = qy0 + ty * ROWS + j;
    if (qx >= p.Wq || qy >= p.Hq) continue;
    bf16_raw* out = p.dX + (((int64_t)n * p.B + b) * CI) * p.H * p.W + (int64_t)(2 * qy) * p.W + 2 * qx;
#pragma unroll
    for (int c = 0; c < CI; ++c) {
      *reinterpret_cast<uint32_t*>(out + (int64_t)c * p.H * p.W) = pack_bf16x2(acc[c][j][0][0], acc[c][j][0][1]);
      *reinterpret_cast<uint32_t*>(out + (int64_t)c * p.H * p.W + p.W) = pack_bf16x2(acc[c][j][1][0], acc[c][j][1][1]);
    }
  }
}

}  // namespace

// A stage of dY, sixteen channels or what there is, has to lie below 2 GiB: gradients of 2^26 pixels and more take the general path.
bool conv_dx_fewc_supported(int Nb, int B, int Ci, int Co, int H, int W, int kh, int kw, int stride, int pad) {
  return kh == 4 && kw == 4 && stride == 2 && pad == 1 && Ci >= 1 && Ci <= 4 && H % 2 == 0 && W % 2 == 0 && Nb <= 65535 && B <= 65535 &&
         (int64_t)(Co < 16 ? Co : 16) * (H / 2) * (W / 2) * 2 < ((int64_t)1 << 31);
}

int conv_dx_fewc(int B, int Nb, int Ci, int Co, int H, int W, const void* Wt, const void* dY, void* dX, hipStream_t st) {
  if (reinterpret_cast<uintptr_t>(dX) % 4 != 0 || reinterpret_cast<uintptr_t>(Wt) % 4 != 0) return HFTA_EUNSUPPORTED;
  FewcArgs a{(const bf16_raw*)Wt, (const bf16_raw*)dY, (bf16_raw*)dX, B, Nb, Co, H, W, H / 2, W / 2, (W / 2 + FC_TX - 1) / FC_TX};
  const bool pair = a.Wq % 2 == 0 && reinterpret_cast<uintptr_t>(dY) % 4 == 0;
  // two rows of q pixels a thread where that leaves two workgroups per compute unit.  us with one row and with two, 64 -> 3 channels at
  // 64 x 64, workgroups of two rows: 1280 120.6 91.3, 640 68.1 62.3, 400 (60 x 60) 45.3 38.0, 384 46.9 47.9, 120 26.3 33.4; four rows 96.7,
  // 71.8, 39.0, 48.5, 46.9.  Not for images of at most eight rows of q pixels, where it leaves as many workgroups with half of the threads
  // idle: 64 -> 3 channels, 512 images of 16 x 16 35.8 47.6, 1280 of 8 x 8 64.9 85.4; 1280 of 20 x 20 115.6 83.8
  const int64_t two = (int64_t)a.tiles_x * ((a.Hq + 2 * FC_TY - 1) / (2 * FC_TY)) * Nb * B;
  const int rows = pair && two >= 512 && a.Hq > FC_TY ? 2 : 1, ph = FC_TY * rows;
  const size_t lds = 2 * (pair && rows == 1 ? 16 : 8) * (ph + 2) * FC_PW * 2;
  const dim3 grid((unsigned)(a.tiles_x * ((a.Hq + ph - 1) / ph)), (unsigned)Nb, (unsigned)B);
#define HFTA_FEWC(C) \
  do { if (rows == 2) hipLaunchKernelGGL((conv_dx_fewc_kernel<C, true, 2>), grid, dim3(256), lds, st, a); \
       else if (pair) hipLaunchKernelGGL((conv_dx_fewc_kernel<C, true, 1>), grid, dim3(256), lds, st, a); \
       else hipLaunchKernelGGL((conv_dx_fewc_kernel<C, false, 1>), grid, dim3(256), lds, st, a); } while (0)
  switch (Ci) {
    case 1: HFTA_FEWC(1); break;
    case 2: HFTA_FEWC(2); break;
    case 3: HFTA_FEWC(3); break;
    default: HFTA_FEWC(4); break;
  }
#undef HFTA_FEWC
  return launch_status();
}

}  // namespace hfta
