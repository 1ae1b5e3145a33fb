// Forward and weight gradient of the 4x4 / stride 2 / pad 1 convolution with the window operand read straight from image
// rows in LDS: no column tile.
//
// A column tile gathered element by element (conv_ig_gather_kernel, which the tall images of the data gradient keep) costs per
// 32-element k-tile of a 128 x 128 tile 64 two-byte LDS reads and 8 sixteen-byte writes of a wavefront, about 200 of 510 LDS
// clocks against 256 of the matrix instructions, and the LDS is what bounded both kernels.  Image rows need neither:
//   forward: the 8 k of a fragment are two window rows of one channel, i.e. twice four neighbouring pixels 2x - 1 .. 2x + 2
//     of one image row.  Rows are kept shifted by one pixel, so those are two aligned 4-byte words (one ds_read2_b32), and
//     the fragment costs what it cost from the column tile.
//   weight gradient: the 8 k of a fragment are neighbouring output pixels of one tap (ky, kx), i.e. every other pixel of an
//     image row.  Rows are kept as four planes, plane kx holding the pixels 2x + kx - 1: one aligned 16-byte read (two of
//     8 bytes where a row has four output pixels); a piece of 8 pixels is written four times, 8 bytes each.
// Order and operands of the matrix instructions are those of the gathering kernels (k ascending), so results keep their bits
// where k is not split.  A split cuts at multiples of 64 k instead of 32, elsewhere than before unless the channels are a
// multiple of four times the splits.
// 10 models x 64 images, forward: 256 <- 128 channels at 8x8 80 -> 58 us, 128 <- 64 at 16x16 and 512 <- 256 at 4x4 (split over
// k) 85 -> 72 on average, 64 <- 3 40 -> 36; weight gradients of the same layers 75 -> 68, 88 -> 81,
// 70 -> 64 and 46 -> 38 (with k-tiles of 64 and two workgroups per compute unit 73, 83, 67 and 46).  3 models x 20 images:
// forward 26 -> 20 us (12.8 to 20.4 with 64-row tiles, which few_tiles gives it now), weight gradients 22 -> 15.

constexpr int ROWS_PITCH = 144;                          // bytes per row of the plain operand's tile: 64 k + 16 B pad

// the neighbouring lanes' words (0 past the wavefront's ends)
__device__ __forceinline__ uint32_t lane_left(uint32_t v) { return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x138, 0xf, 0xf, false); }
__device__ __forceinline__ uint32_t lane_right(uint32_t v) { return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x130, 0xf, 0xf, false); }

struct __attribute__((aligned(4))) Words2 { uint32_t a, b; };

// TM = 128: four wavefronts of 64 x 64; TM = 64 (layers of at most 64 output rows, launches of few tiles): of 64 x 32.  A k-tile is 64 k = four
// channels; the next one is in flight in registers while this one is multiplied; one barrier per k-tile.
template <int TM>
__global__ __launch_bounds__(256, 3) void conv_rows_fwd_kernel(IgArgs p) {
  constexpr int NT = 256, KC = 4;
  constexpr int NA = TM * 8 / NT;                        // 16-byte weight pieces per thread
  constexpr int FN = TM == 128 ? 2 : 1;
  constexpr int A_BYTES = TM * ROWS_PITCH;
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  const int chan_b = p.NI * p.SP * 2, row_b = p.PW * 2;
  const int stage = A_BYTES + KC * chan_b;
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  int bx, split, b;
  ig_block(p.grid, bx, split, b);
  const int tile_m = bx / p.tiles_n, tile_n = bx % p.tiles_n;
  const int m0 = tile_m * TM, n0 = tile_n * 128;
  const int P = 1 << p.lgP, HW = p.H * p.W;
  const int img0 = n0 >> p.lgP, y0 = (n0 & (P - 1)) >> p.lgWo;
  const int kt0 = split * p.kt_per_split, kt1 = min((p.K + 63) / 64, kt0 + p.kt_per_split);
  const int wm = TM == 128 ? wave >> 1 : 0;
  const int col0 = TM == 128 ? (wave & 1) * 64 : wave * 32;

  const __amdgpu_buffer_rsrc_t rx = pf_rsrc(p.X + (int64_t)b * p.x_model, p.x_bytes);
  const __amdgpu_buffer_rsrc_t rw = pf_rsrc(p.A + (int64_t)b * p.a_model, p.a_bytes);
  // ---- pieces of image rows: fixed over the k-loop up to the channel.  Pieces outside the image or past the batch are zeros.
  // A row has a power of two of at most 32 pieces, so the piece to the left is the neighbouring lane's.
  uint32_t pxo[2];
  int pl[2], pcl[2];                                     // LDS byte offset (-1: no piece), channel inside the k-tile
  bool first[2], last[2];
  const int cpr = p.W >> 3;
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int q = t + NT * i, xc = q % cpr;
    int r = q / cpr;
    const int pr = r % p.PR; r /= p.PR;
    const int il = r % p.NI, c_l = r / p.NI;
    const int iy = 2 * y0 - 1 + pr, img = img0 + il;
    const bool has = q < p.nchunk;
    pxo[i] = PF_OOB; pcl[i] = c_l;
    pl[i] = has ? c_l * chan_b + (il * p.SP + pr * p.PW + xc * 8) * 2 : -1;
    first[i] = xc == 0; last[i] = xc == cpr - 1;
    if (has && iy >= 0 && iy < p.H && img < p.Nb)
      pxo[i] = (uint32_t)(((int64_t)img * p.x_img + (int64_t)c_l * HW + (int64_t)iy * p.W + xc * 8) * 2);
  }
  const uint32_t px_step = (uint32_t)(KC * HW * 2);
  const int ga = t & 7, ra = t >> 3;
  uint32_t wo[NA];
#pragma unroll
  for (int h = 0; h < NA; ++h) {
    const int m = m0 + ra + 32 * h;
    wo[h] = m < p.M ? (uint32_t)(((int64_t)m * p.K + ga * 8) * 2) : PF_OOB;
  }
  pf_u32x4 qa[NA], qp[2];
  auto issue = [&](int kt) {
    const bool in_k = kt * 64 + ga * 8 + 8 <= p.K;
#pragma unroll
    for (int i = 0; i < 2; ++i)
      qp[i] = __builtin_amdgcn_raw_buffer_load_b128(
          rx, (int)((kt * KC + pcl[i] < p.Cx && pxo[i] != PF_OOB) ? pxo[i] + (uint32_t)kt * px_step : PF_OOB), 0, 0);
#pragma unroll
    for (int h = 0; h < NA; ++h)
      qa[h] = __builtin_amdgcn_raw_buffer_load_b128(rw, (int)((in_k && wo[h] != PF_OOB) ? wo[h] + (uint32_t)kt * 128u : PF_OOB), 0, 0);
  };
  auto park = [&](int buf) {
    unsigned char* As = smem + buf * stage;
    unsigned char* Rs = As + A_BYTES;
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const pf_u32x4 v = qp[i];
      const uint32_t left = lane_left(v.w);              // all lanes take part
      if (pl[i] >= 0) {
        *reinterpret_cast<uint4*>(Rs + pl[i]) = make_uint4(v.x << 16 | (first[i] ? 0u : left >> 16), v.y << 16 | v.x >> 16,
                                                           v.z << 16 | v.y >> 16, v.w << 16 | v.z >> 16);
        if (last[i]) *reinterpret_cast<uint32_t*>(Rs + pl[i] + 16) = v.w >> 16;
      }
    }
#pragma unroll
    for (int h = 0; h < NA; ++h) *reinterpret_cast<pf_u32x4*>(As + (ra + 32 * h) * ROWS_PITCH + ga * 16) = qa[h];
  };
  const int r = lane & 31, g = lane >> 5;
  int cb[FN];                                            // byte offset of this lane's window rows 2g of column block j
#pragma unroll
  for (int j = 0; j < FN; ++j) {
    const int n = n0 + col0 + 32 * j + r;
    const int il = (n >> p.lgP) - img0, y = ((n & (P - 1)) >> p.lgWo) - y0, x = n & (p.Wo - 1);
    cb[j] = A_BYTES + il * p.SP * 2 + (2 * y + 2 * g) * row_b + 4 * x;
  }
  const int ab = (wm * 64 + r) * ROWS_PITCH + g * 16;
  f32x16_t acc[2][FN];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < FN; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;

  issue(kt0);
  park(0);
  issue(kt0 + 1);
  __syncthreads();
  int buf = 0;
  for (int kt = kt0; kt < kt1; ++kt, buf ^= 1) {
    park(buf ^ 1);                                       // past the end: buffers nobody reads any more
    issue(kt + 2);
    const unsigned char* Sb = smem + buf * stage;
#pragma unroll
    for (int s = 0; s < KC; ++s) {
      bf16x8_t a[2], bq[FN];
#pragma unroll
      for (int i = 0; i < 2; ++i) a[i] = *reinterpret_cast<const bf16x8_t*>(Sb + ab + i * 32 * ROWS_PITCH + s * 32);
#pragma unroll
      for (int j = 0; j < FN; ++j) {
        const unsigned char* src = Sb + cb[j] + s * chan_b;
        const Words2 lo = *reinterpret_cast<const Words2*>(src), hi = *reinterpret_cast<const Words2*>(src + row_b);
        bq[j] = __builtin_bit_cast(bf16x8_t, make_uint4(lo.a, lo.b, hi.a, hi.b));
      }
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(bq[j], a[i], acc[i][j], 0, 0, 0);
    }
    __syncthreads();
  }
  ig_epilogue<false, TM, FN>(p, acc, smem, b, split, m0, n0, wm, col0, p.cls[0], t, lane);
}

// Pitches in elements; rows hold W + 2 pixels.  The lanes of a half wavefront read one word each of the image rows their 32
// columns lie in (words W / 2 wide, a pitch of PW words apart; of two samples where a sample has 16 pixels): PW = 24 mod 32
// for rows of 4 and 8 words, 16 mod 32 for rows of 16 spread them over all banks (images of more than four 4-word rows: two
// lanes to a bank).  At most 512 pieces, two per thread: 64 + NI Wo / 2 for each of four channels, NI Wo <= 128.
void rows_fwd_geometry(IgArgs& a) {
  const int P = a.Ho * a.Wo;
  if (P >= 128) { a.NI = 1; a.TR = 128 / a.Wo; } else { a.NI = 128 / P; a.TR = a.Ho; }
  a.PR = 2 * a.TR + 2;
  a.nchunk = 4 * a.NI * a.PR * (a.W / 8);
  a.PW = a.W + (a.Wo == 4 || a.Wo == 16 ? 16 : 8);
  a.SP = a.PR * a.PW;
  while (P == 16 && a.SP % 64 != (a.Wo == 4 ? 56 : 32)) a.SP += 8;
}
size_t rows_fwd_lds_bytes(const IgArgs& a, int tm) {
  const size_t k_loop = 2 * ((size_t)tm * ROWS_PITCH + 4 * (size_t)a.NI * a.SP * 2);
  const size_t staging = a.ksplit > 1 ? 64 * (size_t)132 * 4 : 64 * (size_t)IG_EPI_PITCH;
  return k_loop > staging ? k_loop : staging;
}

// ---- weight gradient
//   dW[o][j = (c, ky, kx)] = sum over k = (n, y, x) of dY[n][o][y][x] X[n][c][2 y + ky - 1][2 x + kx - 1]
// Rows are output channels (dY is k-contiguous inside a sample), columns the 128 taps of 8 input channels, a k-tile 32
// consecutive output pixels (of one sample, or of two small ones).  The grid's y splits the k range; partial sums go to fp32
// slices reduced afterwards.  The next two k-tiles are in flight in registers.  k-tiles of 32 rather than 64, so that three
// workgroups fit a compute unit: the split makes 513 to 640 of many layers, which two per unit finish in two rounds.
struct IgDwArgs {
  const bf16_raw* X; const bf16_raw* dY; float* Out;
  int64_t x_img, x_model, y_img, y_model;                // element strides: sample, model
  int64_t o_model, o_split;                              // output strides: model, k split
  int Nb, Ci, Co, H, W, Wo, lgWo, lgP;
  int NI, PR, nchunk;                                    // samples per k-tile, image rows per sample and channel, pieces
  int plane_b, row_b;                                    // bytes between the planes of a row, between rows
  int tiles_n, kt_total, kt_per_split;
  IgGrid grid;                                           // logical grid: x = tiles, y = k split, z = model
  uint32_t x_bytes, y_bytes;                             // extents of one model's slices of X and dY
};

// W4: rows of four output pixels
template <bool W4>
__global__ __launch_bounds__(256, 3) void conv_rows_dw_kernel(IgDwArgs p) {
  constexpr int A_BYTES = GEMM_TILE_BYTES;
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  const int chan_b = p.NI * p.PR * p.row_b;
  const int stage = A_BYTES + 8 * chan_b;
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  const int wm = wave >> 1, wn = wave & 1;
  int bx, by, b;
  ig_block(p.grid, bx, by, b);
  const int tile_m = bx / p.tiles_n, tile_n = bx % p.tiles_n;
  const int m0 = tile_m * 128, c0 = tile_n * 8;
  const int P = 1 << p.lgP, HW = p.H * p.W;
  const int kt_begin = by * p.kt_per_split;
  const int kt_end = min(p.kt_total, kt_begin + p.kt_per_split);

  const __amdgpu_buffer_rsrc_t rx = pf_rsrc(p.X + (int64_t)b * p.x_model, p.x_bytes);
  const __amdgpu_buffer_rsrc_t ry = pf_rsrc(p.dY + (int64_t)b * p.y_model, p.y_bytes);
  // ---- pieces of image rows: channel, sample, row and position are fixed; the image row moves with the k-tile
  const int cpr = p.W >> 3;
  const int xc = t % cpr;
  int q = t / cpr;
  const int prow = q % p.PR; q /= p.PR;
  const int pil = q % p.NI, c_l = q / p.NI;
  const bool first = xc == 0, last = xc == cpr - 1;
  const int pl = t < p.nchunk ? A_BYTES + c_l * chan_b + (pil * p.PR + prow) * p.row_b + xc * 8 : -1;
  // byte offset at sample 0, image row 0
  const uint32_t pxo = t < p.nchunk && c0 + c_l < p.Ci ? (uint32_t)(((int64_t)(c0 + c_l) * HW + xc * 8) * 2) : PF_OOB;
  const int ga = t & 3, ra = t >> 2;
  uint32_t yo[2];                                        // byte offset of the row's pixel 0 in sample 0
#pragma unroll
  for (int h = 0; h < 2; ++h) yo[h] = m0 + ra + 64 * h < p.Co ? (uint32_t)((int64_t)(m0 + ra + 64 * h) * P * 2) : PF_OOB;
  pf_u32x4 qa[2][2], qp[2];
  auto issue = [&](int kt, int set) {
    const int k0 = kt * 32;
    const int img = (k0 >> p.lgP) + pil, iy = 2 * ((k0 & (P - 1)) >> p.lgWo) - 1 + prow;
    const bool ok = pxo != PF_OOB && img < p.Nb && iy >= 0 && iy < p.H;
    qp[set] = __builtin_amdgcn_raw_buffer_load_b128(
        rx, (int)(ok ? pxo + (uint32_t)img * (uint32_t)(p.x_img * 2) + (uint32_t)(iy * p.W * 2) : PF_OOB), 0, 0);
    const int kk = k0 + ga * 8, n = kk >> p.lgP;         // 8 pixels of one sample (P is at least 16)
    const uint32_t yb = (uint32_t)n * (uint32_t)(p.y_img * 2) + (uint32_t)(kk & (P - 1)) * 2u;
#pragma unroll
    for (int h = 0; h < 2; ++h)
      qa[set][h] = __builtin_amdgcn_raw_buffer_load_b128(ry, (int)((n < p.Nb && yo[h] != PF_OOB) ? yo[h] + yb : PF_OOB), 0, 0);
  };
  auto park = [&](int buf, int set) {
    unsigned char* Sb = smem + buf * stage;
    const pf_u32x4 v = qp[set];
    const uint32_t left = lane_left(v.w), right = lane_right(v.x);                                 // all lanes take part
    if (pl >= 0) {
      unsigned char* d = Sb + pl;
      const uint32_t e0 = (v.x & 0xffffu) | v.y << 16, e1 = (v.z & 0xffffu) | v.w << 16;           // pixels 0 2 | 4 6
      const uint32_t o0 = v.x >> 16 | (v.y & 0xffff0000u), o1 = v.z >> 16 | (v.w & 0xffff0000u);   // 1 3 | 5 7
      *reinterpret_cast<uint2*>(d) = make_uint2(o0 << 16 | (first ? 0u : left >> 16), o1 << 16 | o0 >> 16);
      *reinterpret_cast<uint2*>(d + p.plane_b) = make_uint2(e0, e1);
      *reinterpret_cast<uint2*>(d + 2 * p.plane_b) = make_uint2(o0, o1);
      *reinterpret_cast<uint2*>(d + 3 * p.plane_b) = make_uint2(e0 >> 16 | e1 << 16, e1 >> 16 | (last ? 0u : right << 16));
    }
#pragma unroll
    for (int h = 0; h < 2; ++h) *reinterpret_cast<pf_u32x4*>(Sb + (ra + 64 * h) * GEMM_PITCH + ga * 16) = qa[set][h];
  };
  const int r = lane & 31, g = lane >> 5;
  int cb[2], ko[2];                                      // byte offsets: tap of column block j; pixels of k-step s
#pragma unroll
  for (int j = 0; j < 2; ++j) cb[j] = A_BYTES + (wn * 4 + 2 * j + (r >> 4)) * chan_b + ((r >> 2) & 3) * p.row_b + (r & 3) * p.plane_b;
#pragma unroll
  for (int s = 0; s < 2; ++s) {
    const int k = s * 16 + g * 8;
    const int il = k >> p.lgP, y = (k & (P - 1)) >> p.lgWo, x = k & (p.Wo - 1);
    ko[s] = (il * p.PR + 2 * y) * p.row_b + x * 2;
  }
  const int ab = (wm * 64 + r) * GEMM_PITCH + g * 16;
  f32x16_t acc[2][2];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;
  auto mma = [&](int buf) {
    const unsigned char* Sb = smem + buf * stage;
#pragma unroll
    for (int s = 0; s < 2; ++s) {
      bf16x8_t a[2], bq[2];
#pragma unroll
      for (int i = 0; i < 2; ++i) a[i] = *reinterpret_cast<const bf16x8_t*>(Sb + ab + i * 32 * GEMM_PITCH + s * 32);
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        const unsigned char* src = Sb + cb[j] + ko[s];
        if constexpr (W4) {
          const uint2 lo = *reinterpret_cast<const uint2*>(src), hi = *reinterpret_cast<const uint2*>(src + 2 * p.row_b);
          bq[j] = __builtin_bit_cast(bf16x8_t, make_uint4(lo.x, lo.y, hi.x, hi.y));
        } else {
          bq[j] = *reinterpret_cast<const bf16x8_t*>(src);
        }
      }
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(bq[j], a[i], acc[i][j], 0, 0, 0);
    }
  };

  // k-tiles past the end of the split (zeros past the batch) are loaded and parked where nobody reads them any more
  issue(kt_begin, 0);
  issue(kt_begin + 1, 1);
  park(0, 0);
  issue(kt_begin + 2, 0);
  __syncthreads();
  int kt = kt_begin;
  for (; kt + 1 < kt_end; kt += 2) {
    park(1, 1);
    issue(kt + 3, 1);
    mma(0);
    __syncthreads();
    park(0, 0);
    issue(kt + 4, 0);
    mma(1);
    __syncthreads();
  }
  if (kt < kt_end) {
    mma(0);
    __syncthreads();
  }
  const int N = p.Ci * 16;
  float* ob = p.Out + (int64_t)by * p.o_split + (int64_t)b * p.o_model;
  store_tile<float, float, false>(acc, smem, ob, N, p.Co, N, m0, c0 * 16, (const float*)nullptr, 0, HFTA_ACT_NONE, 0.f, 16, t);
}
