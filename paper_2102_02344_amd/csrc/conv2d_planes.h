// Data gradient of the 4x4 / stride 2 / pad 1 convolution from shifted row planes.
//
// Building the column tile element by element (conv_ig_gather_kernel) costs a thread 16 two-byte LDS reads and two
// 16-byte writes per 32-element k-tile, as much LDS time as the matrix instructions' operands.  The transpose
// read (see pf_frag) makes that tile unnecessary: each of its lanes addresses four neighbouring pixels of one
// k-row by itself, so the k-rows of a matrix instruction can be the four taps of a channel's 2x2 window, each at
// its own place in the image rows.  What it needs is that four neighbouring columns of any tap are eight aligned
// bytes, so the rows are kept three times, shifted by -1, 0 and +1 pixels with zeros shifted in: per 16-byte
// piece of input one LDS read and three writes, against 4 x 4 gathered elements per input element.
//
// Memory -> LDS goes by direct loads (dma_load), two 16-channel k-tiles ahead; a wave rebuilds the planes from the
// pieces it fetched itself, so that needs no barrier, and planes are double-buffered: one barrier per 64 k.
// Weights are fragments straight from memory (ig_pack_class_w_kernel), reloaded as they are used up; launches below
// one workgroup per compute unit keep two k-tiles of them (60 workgroups of 128 rows, 32 k-tiles: 33 -> 27 us; 32 of 64
// rows 25.4 -> 24.9), others one
// (a second set costs the third workgroup per compute unit: 60 -> 67 us at 1280).
// 10 models x 64 images: 128 <- 256 channels at 8x8 75 -> 60 us, 256 <- 512 at 4x4 71 -> 53, 64 <- 128 at 16x16 98 -> 66,
// the same products in the same order (a reduction split over k changes bits that a GAN's next layers amplify).

constexpr int DXP_CH = 16;                               // channels per k-tile (64 k)
constexpr int DXP_RAW = 4 * 1024;                        // one slot of raw pieces: 64 per wave

// W4: rows of four pixels, tiles of whole images; a piece is two rows.  Else rows of whole 16-byte pieces.
// AD: k-tiles of weight fragments in registers.
template <int TM, bool W4, int AD>
__global__ __launch_bounds__(256, 2) void conv_dx_planes_kernel(IgArgs p) {
  constexpr int FN = TM == 128 ? 2 : 1;
  extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
  const int t = threadIdx.x, lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6);
  int bx, by, b;
  ig_block(p.grid, bx, by, b);
  const int tile_m = bx / p.tiles_n, tile_n = bx % p.tiles_n;
  const int m0 = tile_m * TM, n0 = tile_n * 64;
  const int py = by;
  const int P = 1 << p.lgP, HW = p.H * p.W;
  const int img0 = n0 >> p.lgP, y0 = (n0 & (P - 1)) >> p.lgWo;
  const int kt1 = (p.Cx + DXP_CH - 1) / DXP_CH;
  const int img_el = p.PR * p.W;                          // elements of an image's rows in a plane
  const int wm = TM == 128 ? wave >> 1 : 0;
  const int col0 = TM == 128 ? (wave & 1) * 64 : wave * 32, px = col0 >> 6;

  // ---- this lane's raw piece
  const int cpr = (W4 ? P : p.W) >> 3;
  int c_l, p_dst;
  uint32_t p_off = PF_OOB;
  bool first = true, last = true;
  {
    int q = t;
    const int xc = q % cpr;
    q /= cpr;
    int pr = 0;
    if (!W4) { pr = q % p.PR; q /= p.PR; first = xc == 0; last = xc == cpr - 1; }
    const int il = q % p.NI, img = img0 + il;
    c_l = q / p.NI;
    const int iy = y0 + py - 1 + pr;
    p_dst = c_l * p.chp + (il * img_el + (W4 ? (2 * xc + 1 - py) * 4 : pr * p.W + xc * 8)) * 2;
    if (c_l < DXP_CH && img < p.Nb && (W4 || (iy >= 0 && iy < p.H)))
      p_off = (uint32_t)(((int64_t)img * p.x_img + (int64_t)c_l * HW + (W4 ? 0 : iy * p.W) + xc * 8) * 2);
  }
  const bool has = c_l < DXP_CH;
  const uint32_t step = (uint32_t)(DXP_CH * HW * 2);
  const dma_i32x4 rx = dma_rsrc(p.X + (int64_t)b * p.x_model, p.x_bytes);
  typedef __attribute__((address_space(3))) unsigned char* lds_ptr;
  const uint32_t raw0 = (uint32_t)(uintptr_t)(lds_ptr)smem + (uint32_t)(wave * 1024);
  auto fetch = [&](int kt, int slot) {
    dma_load(raw0 + (uint32_t)(slot * DXP_RAW), p_off != PF_OOB && kt * DXP_CH + c_l < p.Cx ? p_off + (uint32_t)kt * step : PF_OOB, rx);
  };
  unsigned char* const planes = smem + 2 * DXP_RAW;
  const int buf_bytes = 3 * p.plp;
  uint4 v;
  uint32_t vp, vn;                                        // the elements left and right of the piece
  auto raw_read = [&](int slot) {
    const unsigned char* src = smem + slot * DXP_RAW + wave * 1024 + lane * 16;
    v = *reinterpret_cast<const uint4*>(src);
    vp = vn = 0u;
    if (!W4) {
      if (!first) vp = *reinterpret_cast<const bf16_raw*>(src - 2);
      if (!last) vn = *reinterpret_cast<const bf16_raw*>(src + 16);
    }
  };
  auto plane_write = [&](int buf) {
    if (!has) return;
    unsigned char* d = planes + buf * buf_bytes + p_dst;
    uint4 l, r;
    if (W4) {                                              // two rows of four
      l = make_uint4(v.x << 16, v.y << 16 | v.x >> 16, v.z << 16, v.w << 16 | v.z >> 16);
      r = make_uint4(v.x >> 16 | v.y << 16, v.y >> 16, v.z >> 16 | v.w << 16, v.w >> 16);
    } else {
      l = make_uint4(v.x << 16 | vp, v.y << 16 | v.x >> 16, v.z << 16 | v.y >> 16, v.w << 16 | v.z >> 16);
      r = make_uint4(v.x >> 16 | v.y << 16, v.y >> 16 | v.z << 16, v.z >> 16 | v.w << 16, v.w >> 16 | vn << 16);
    }
    auto put = [&](unsigned char* q, const uint4& x) {
      if (W4) {
        *reinterpret_cast<uint2*>(q) = make_uint2(x.x, x.y);
        *reinterpret_cast<uint2*>(q + 8) = make_uint2(x.z, x.w);
      } else {
        *reinterpret_cast<uint4*>(q) = x;
      }
    };
    put(d, l);
    put(d + p.plp, v);
    put(d + 2 * p.plp, r);
  };

  // ---- weights: fragments [32-row block][k-step] of this wave's class and rows
  const int ktiles32 = (p.K + 31) / 32;
  const __amdgpu_buffer_rsrc_t rw = pf_rsrc(p.A + (int64_t)b * p.a_model, p.a_bytes);
  const uint32_t fo = (uint32_t)((p.cls[2 * py + px].a_off + (int64_t)tile_m * ktiles32 * TM * 32) * 2) + (uint32_t)((wm * 4 * 64 + lane) * 16);
  pf_u32x4 fa[AD][2][4];
  auto load_a = [&](int set, int kt, int i, int s) {
    const int k32 = 2 * kt + (s >> 1);
    fa[set][i][s] = __builtin_amdgcn_raw_buffer_load_b128(
        rw, (int)(k32 < ktiles32 ? fo + (uint32_t)k32 * (uint32_t)(TM * 64) + (uint32_t)((i * 2 + (s & 1)) * 1024) : PF_OOB), 0, 0);
  };
  // ---- columns: where this lane's transpose reads of block j start (channel 2 (lane / 32) of the tile)
  int cb[FN];
#pragma unroll
  for (int j = 0; j < FN; ++j) {
    const int r = lane & 15;
    const int n = n0 + (TM == 128 ? 0 : (wave & 1) * 32) + j * 32 + 16 * ((lane >> 4) & 1) + 4 * (r & 3);
    const int il = (n >> p.lgP) - img0, y = ((n & (P - 1)) >> p.lgWo) - y0, x = n & (p.Wo - 1);
    cb[j] = (px + ((r >> 2) & 1)) * p.plp + 2 * (lane >> 5) * p.chp + (il * img_el + (y + (r >> 3)) * p.W + x) * 2;
  }
  typedef __attribute__((address_space(3))) pf_v4s* lds_v4s;

  f32x16_t acc[2][FN];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < FN; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;

  fetch(0, 0);
  fetch(1, 1);
#pragma unroll
  for (int d = 0; d < AD; ++d)
#pragma unroll
    for (int s = 0; s < 4; ++s)
#pragma unroll
      for (int i = 0; i < 2; ++i) load_a(d, d, i, s);
  if (W4) {                                                // the row above or below the image is never written
    for (int i = t; i < 2 * buf_bytes / 16; i += 256) reinterpret_cast<uint4*>(planes)[i] = make_uint4(0u, 0u, 0u, 0u);
    __syncthreads();
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  raw_read(0);
  plane_write(0);
  bool done = false;
  for (int base = 0; !done; base += 2) {
#pragma unroll
    for (int buf = 0; buf < 2; ++buf) {
      const int kt = base + buf, set = buf % AD;
      // planes of kt written by all waves, those of kt - 1 read; raw pieces of kt + 1 were requested before the last
      // eight fragment loads, so at most eight loads in flight means that they have landed
      asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
      fetch(kt + 2, buf);
      asm volatile("s_waitcnt vmcnt(8)" ::: "memory");
      raw_read(buf ^ 1);
      const unsigned char* pb = planes + buf * buf_bytes;
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        bf16x8_t bq[FN];
#pragma unroll
        for (int j = 0; j < FN; ++j) {
          const unsigned char* a0 = pb + cb[j] + 4 * s * p.chp;
          union { pf_v4s h[2]; bf16x8_t q; } u;
          u.h[0] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4s)(a0));
          u.h[1] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4s)(a0 + p.chp));
          bq[j] = u.q;
        }
#pragma unroll
        for (int i = 0; i < 2; ++i) {
          const bf16x8_t a = __builtin_bit_cast(bf16x8_t, fa[set][i][s]);
#pragma unroll
          for (int j = 0; j < FN; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(bq[j], a, acc[i][j], 0, 0, 0);
          load_a(set, kt + AD, i, s);
        }
        if (s == 1) plane_write(buf ^ 1);
      }
      if (kt + 1 >= kt1) { done = true; break; }
    }
  }
  dma_wait_barrier<0>();
  ig_epilogue<true, TM, FN>(p, acc, smem, b, 0, m0, n0, wm, col0, p.cls[2 * py], t, lane);
}

// Plane geometry of a data gradient's tiles; false for images of four-pixel rows taller than a tile, which the gathering
// kernel keeps.  (Rows of 8 to 64 pixels have 144 to 256 pieces a tile and at most 34 KB of planes.)
bool dxp_geometry(IgArgs& a) {
  const int P = a.Ho * a.Wo;
  const bool w4 = a.W == 4;
  if (w4 ? P > 64 : a.W % 8 != 0) return false;
  const int pieces = DXP_CH * a.NI * (w4 ? P / 8 : a.PR * (a.W / 8));
  if (pieces > 256) return false;                          // one per thread
  a.chp = (a.NI * a.PR * a.W * 2 + 15) & ~15;
  // bank offset between the shifted planes: the four taps' 64-byte stretches of a read cover all banks
  const int want = a.W * 2 == 128 ? 64 : 128;
  a.plp = DXP_CH * a.chp;
  a.plp += (want - a.plp % 256 + 256) % 256;
  return true;
}
size_t dxp_lds_bytes(const IgArgs& a) {
  const size_t k_loop = 2 * (size_t)DXP_RAW + 2 * (size_t)3 * a.plp;
  const size_t staging = 64 * (size_t)IG_EPI_PITCH;
  return k_loop > staging ? k_loop : staging;
}
