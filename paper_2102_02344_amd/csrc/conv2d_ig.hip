// Grouped Conv2d / ConvTranspose2d as an implicit GEMM whose columns run over (sample, output pixel)
// of one model (fusion rules table, rows "Conv2d" and "ConvTranspose2d": one grouped operator with
// G = B; here the model is grid.z and never mixes with the channels).
//
// No column buffer exists in memory: a workgroup brings the raw image rows its output tile needs into LDS and the matrix
// instructions' window operand is read straight from them (conv2d_rows.h, conv2d_planes.h).  Folding the sample index into the
// columns keeps the tiles full for 8x8 and 4x4 images, where a GEMM per sample has 64 or 16 columns.
//
//   forward (and the data gradient of a transposed convolution):
//       Y[o][(n, y, x)] = sum_{(c, ky, kx)} W[o][(c, ky, kx)] X[n][c][s y + ky - p][s x + kx - p]
//   data gradient (and the forward of a transposed convolution), per output-parity class (py, px):
//       dX[c][(n, qy, qx)] = sum_{(o, jy, jx)} Wp[class][c][(o, jy, jx)] dY[n][o][qy + py - 1 + jy][qx + px - 1 + jx]
//     a stride-1 correlation with a 2x2 window and the weights regrouped per class (the taps a class
//     does not see are never multiplied); results land at (2 qy + py, 2 qx + px).
//   weight gradient: dW[o][(c, ky, kx)] = sum_{(n, y, x)} dY[n][o][y][x] X[n][c][...].
//
// bf16 only; output grids whose width and height are powers of two; see ig_*_supported.
#include "gemm_dma.h"

namespace hfta {

namespace {

constexpr int IG_MARGIN = 8;            // gathering kernel: zero columns left of a patch row

// Workgroups are dispatched to the 8 XCDs (each with its own L2) round-robin by their linear id.
// The kernels are launched on a 1-D grid and turn the id into a logical (x, y, z) block such that
// consecutive logical blocks -- the column tiles that share a weight slab, then the row tiles that
// share a patch -- run on the SAME XCD at about the same time, instead of each XCD fetching every
// slab for itself (the 8x8 layer's forward went from a 32 % L2 hit rate to sharing).
struct IgGrid { int gx, gy, gz; };
__device__ __forceinline__ void ig_block(const IgGrid& g, int& bx, int& by, int& bz) {
  const int total = g.gx * g.gy * g.gz, id = blockIdx.x;
  int logical = id;
  if (total % 8 == 0) logical = (id & 7) * (total >> 3) + (id >> 3);
  bx = logical % g.gx;
  const int r = logical / g.gx;
  by = r % g.gy;
  bz = r / g.gy;
}

struct IgClass {
  int oy, ox;                           // patch row / column of tap (0, 0) for output (0, 0), before the margin
  int out_y0, out_x0;                   // where the class's outputs start in the output image
  int64_t a_off;                        // offset of the class's weights inside a model's block
};

struct IgArgs {
  const bf16_raw* X; const bf16_raw* A; bf16_raw* Out; const bf16_raw* bias;
  int64_t x_img, x_model;               // element strides of the view operand: sample, model (channel stride = H * W)
  int64_t a_model;                      // weights: [b][..][m][K], K contiguous
  int64_t o_img, o_model, o_m;          // output element strides: sample, model, GEMM row (channel)
  int Nb, Cx, H, W;                     // view operand: channels per model, image size
  int M, K, N;                          // GEMM sizes per model: rows, reduction, columns = Nb * Ho * Wo
  int Ho, Wo, lgWo, lgP;                // logical output grid per sample (powers of two)
  int OW, oys, oxs;                     // output image width in memory, output step per grid step
  int tap_step;                         // gathering kernel: 1 (patch elements between the taps of a window row)
  int NI, TR, PR, PW, SP;               // samples per tile, grid rows per tile and sample, patch rows, row pitch, sample pitch (elements)
  int nchunk;                           // 16- or (gathering kernel) 8-byte pieces of patch rows per k-tile
  int chp, plp;                         // plane kernels: bytes of a channel's rows in a plane, bytes between planes
  uint32_t x_bytes, a_bytes;            // extent of one model's slice of the view operand / of its weights
  IgGrid grid;                          // logical grid: x = tiles, y = class / k split, z = model
  int ksplit, kt_per_split;             // k range split over the grid's y (> 1: fp32 partial slices instead of Out)
  float* part; int64_t part_split;      // partial slices [split][same indexing as Out]
  int tiles_n, act;
  float slope;
  IgClass cls[4];
};

constexpr int IG_EPI_PITCH = 128 * 2 + 16;   // bytes per staged output row (64 rows at a time)

// accumulators of a wavefront (64 rows x 32 FN columns from column col0) -> staging tile [64][128]
template <int FN>
__device__ __forceinline__ void ig_stage64(f32x16_t (&acc)[2][FN], unsigned char* lds, int M, int mrow0, const bf16_raw* bias,
                                           int act, float slope, int lane, int col0) {
  const int ml = lane & 31, nq = (lane >> 5) * 4;
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int rl = i * 32 + ml, m = mrow0 + rl;
    const float bm = (bias && m < M) ? bf16_to_f32(bias[m]) : 0.f;
#pragma unroll
    for (int j = 0; j < FN; ++j)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int nl = col0 + j * 32 + 8 * q + nq;
        float x[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) x[e] = cheap_act(acc[i][j][4 * q + e] + bm, act, slope);
        *reinterpret_cast<uint2*>(lds + rl * IG_EPI_PITCH + nl * 2) = make_uint2(pack_bf16x2(x[0], x[1]), pack_bf16x2(x[2], x[3]));
      }
  }
}

// Epilogue of a TM x 128 tile: fp32 partial slices when k is split (not with PAIR), else bias + activation and whole
// pieces of the output rows (PAIR: the two classes of a row interleaved).  `smem` is free (behind a barrier).
template <bool PAIR, int TM, int FN>
__device__ __forceinline__ void ig_epilogue(const IgArgs& p, f32x16_t (&acc)[2][FN], unsigned char* smem, int b, int split,
                                            int m0, int n0, int wm, int col0, const IgClass& cl0, int t, int lane) {
  constexpr int NT = 256;
  const int P = 1 << p.lgP;
  if (!PAIR && p.ksplit > 1) {
    // ---- split k: this workgroup's fp32 partial tile goes to its slice, indexed like the output;
    // bias, activation and the conversion happen in ig_split_finish_kernel
    float* lds_f = reinterpret_cast<float*>(smem);
    float* ob = p.part + (int64_t)split * p.part_split + (int64_t)b * p.o_model;
    constexpr int FP = 132;                               // floats per staged row
#pragma unroll 1
    for (int pass = 0; pass < TM / 64; ++pass) {
      const int mp = m0 + 64 * pass;
      if (wm == pass) {
        const int ml = lane & 31, nq = (lane >> 5) * 4;
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
          for (int j = 0; j < FN; ++j)
#pragma unroll
            for (int q = 0; q < 4; ++q)
              *reinterpret_cast<float4*>(lds_f + (i * 32 + ml) * FP + col0 + j * 32 + 8 * q + nq) =
                  make_float4(acc[i][j][4 * q], acc[i][j][4 * q + 1], acc[i][j][4 * q + 2], acc[i][j][4 * q + 3]);
      }
      __syncthreads();
#pragma unroll
      for (int id = t; id < 64 * 32; id += NT) {
        const int rr = id >> 5, pc = id & 31;
        const int m = mp + rr;
        const int n = n0 + pc * 4;
        if (m >= p.M || n >= p.N) continue;
        const int img = n >> p.lgP, pix = n & (P - 1);
        *reinterpret_cast<float4*>(ob + (int64_t)img * p.o_img + (int64_t)m * p.o_m + pix) =
            *reinterpret_cast<const float4*>(lds_f + rr * FP + pc * 4);
      }
      if (pass + 1 < TM / 64) __syncthreads();
    }
    return;
  }

  // ---- epilogue: bias + activation, 64 rows at a time through an LDS staging tile, then whole
  // 16-byte pieces of the output rows
  unsigned char* lds = smem;
  const bf16_raw* bias = p.bias ? p.bias + (int64_t)b * p.M : nullptr;
  bf16_raw* ob = p.Out + (int64_t)b * p.o_model;
#pragma unroll 1
  for (int pass = 0; pass < TM / 64; ++pass) {
    const int mp = m0 + 64 * pass;
    if (wm == pass) ig_stage64<FN>(acc, lds, p.M, mp, bias, p.act, p.slope, lane, col0);
    __syncthreads();
    if (!PAIR) {
      // 8 consecutive columns = 8 consecutive pixels of one sample: one 16-byte piece
#pragma unroll
      for (int id = t; id < 64 * 16; id += NT) {
        const int rr = id >> 4, pc = id & 15;
        const int m = mp + rr, n = n0 + pc * 8;
        if (m >= p.M || n >= p.N) continue;
        const int img = n >> p.lgP, pix = n & (P - 1);
        *reinterpret_cast<uint4*>(ob + (int64_t)img * p.o_img + (int64_t)m * p.o_m + pix) =
            *reinterpret_cast<const uint4*>(lds + rr * IG_EPI_PITCH + pc * 16);
      }
    } else {
      // 4 consecutive pixels x 2 classes = 8 consecutive output elements
#pragma unroll
      for (int id = t; id < 64 * 16; id += NT) {
        const int rr = id >> 4, pc = id & 15;
        const int m = mp + rr, n = n0 + pc * 4;
        if (m >= p.M || n >= p.N) continue;
        const int img = n >> p.lgP, y = (n & (P - 1)) >> p.lgWo, x = n & (p.Wo - 1);
        const uint2 e = *reinterpret_cast<const uint2*>(lds + rr * IG_EPI_PITCH + pc * 8);          // px = 0
        const uint2 o = *reinterpret_cast<const uint2*>(lds + rr * IG_EPI_PITCH + 128 + pc * 8);    // px = 1
        const uint4 v = make_uint4((e.x & 0xffffu) | (o.x << 16), (e.x >> 16) | (o.x & 0xffff0000u),
                                   (e.y & 0xffffu) | (o.y << 16), (e.y >> 16) | (o.y & 0xffff0000u));
        *reinterpret_cast<uint4*>(ob + (int64_t)img * p.o_img + (int64_t)m * p.o_m + (int64_t)(y * p.oys + cl0.out_y0) * p.OW + x * p.oxs) = v;
      }
    }
    if (pass + 1 < TM / 64) __syncthreads();
  }
}

// Data gradient with a gathered column tile, for images of four-pixel rows taller than a tile (conv2d_planes.h has the others).
// Four wavefronts; each computes 64 rows x 64 columns of a TM = 128 row tile, or 64 rows x 32 columns
// of a TM = 64 row tile (layers with at most 64 output rows).  The tile's 128 columns are 64 pixels of the parity class px = 0
// followed by the same 64 pixels of px = 1 (the grid's y = py); a wavefront works on the class its columns belong to, and the
// epilogue interleaves the two classes into whole 16-byte pieces of the output rows.
//
// Column tile and patch are double-buffered and there is one barrier per k-tile.  In iteration kt a thread
//   issues the LDS reads that gather its part of column tile kt+1 from patch kt+1,
//   parks the patch of k-tile kt+2 (registers -> LDS) and issues the loads of the patch of kt+3,
//   runs the matrix instructions on k-tile kt (the gather's reads return meanwhile),
//   issues the loads of the weights of kt+2 (fragments, see below),
//   writes its part of column tile kt+1, and meets the others at the barrier.
// Every load is a raw buffer load whose offset is inside the model's slice or the fixed out-of-range
// value (the hardware returns zeros): no load sits under control flow, so the compiler's wait
// counters let the loads of later k-tiles stay in flight across iterations.  Nothing in the loop
// depends on the k-tile index: loads past the last k-tile are out of range, and what is parked or
// built from them lands in buffers nobody reads any more.
template <int TM>
__global__ __launch_bounds__(256) void conv_ig_gather_kernel(IgArgs p) {
  static_assert(TM == 128 || TM == 64, "row tiles of 128 or 64");
  constexpr int KW = 2, TK = 4, CPT = 8;                 // taps per window row, per channel; channels per k-tile
  constexpr int NT = 256;
  constexpr int KPT = 16;                                // k per thread of the column tile
  constexpr int COLS = 64;                               // pixels per tile
  constexpr int FN = TM == 128 ? 2 : 1;                  // 32-column blocks per wavefront
  constexpr int CH = 4;                                  // elements per patch piece
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  auto Cb = [&](int buf) { return smem + buf * GEMM_TILE_BYTES; };
  const int chan_el = p.NI * p.SP;
  const int patch_el = CPT * chan_el;
  auto Pt = [&](int buf) { return reinterpret_cast<bf16_raw*>(smem + 2 * GEMM_TILE_BYTES) + buf * patch_el; };
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  int bx, by, b;
  ig_block(p.grid, bx, by, b);
  const int tile_m = bx / p.tiles_n, tile_n = bx % p.tiles_n;
  const int m0 = tile_m * TM, n0 = tile_n * COLS;
  const int py2 = 2 * by;                                // first class of the pair
  const IgClass cl0 = p.cls[py2];
  const int P = 1 << p.lgP;
  const int img0 = n0 >> p.lgP;                          // first sample of the tile
  const int y0 = (n0 & (P - 1)) >> p.lgWo;               // first grid row (tiles inside one sample)
  const int HW = p.H * p.W;
  const int rmin = cl0.oy;                               // first patch row's image row for grid row 0 (the same for both classes of a pair)
  const int row_base = y0 + rmin;
  const int ktiles = (p.K + 31) / 32;

  // position of the wavefront's block of the tile
  const int wm = TM == 128 ? wave >> 1 : 0;
  const int col0 = TM == 128 ? (wave & 1) * 64 : wave * 32;

  const __amdgpu_buffer_rsrc_t rx = pf_rsrc(p.X + (int64_t)b * p.x_model, p.x_bytes);
  const __amdgpu_buffer_rsrc_t rw = pf_rsrc(p.A + (int64_t)b * p.a_model, p.a_bytes);
  // ---- patch pieces: fixed over the k-loop up to the channel, which advances CPT per k-tile.
  // Pieces outside the image or past the batch load zeros; threads without a piece park nothing.
  uint32_t pxo[2];                                        // byte offset of the piece at its channel of k-tile 0, or PF_OOB
  int pl[2], pcl[2];                                      // LDS element offset, channel inside the k-tile
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int q = t + NT * i;
    pxo[i] = PF_OOB; pl[i] = -1; pcl[i] = 0;
    if (q < p.nchunk) {
      const int cpr = p.W / CH;                           // pieces per image row
      const int xc = q % cpr;
      int r = q / cpr;
      const int pr = r % p.PR; r /= p.PR;
      const int il = r % p.NI, c_l = r / p.NI;
      const int iy = row_base + pr, img = img0 + il;
      pcl[i] = c_l;
      pl[i] = (c_l * p.NI + il) * p.SP + pr * p.PW + IG_MARGIN + xc * CH;
      if (iy >= 0 && iy < p.H && img < p.Nb)
        pxo[i] = (uint32_t)(((int64_t)img * p.x_img + (int64_t)c_l * HW + (int64_t)iy * p.W + xc * CH) * 2);
    }
  }
  const uint32_t px_step = (uint32_t)(CPT * HW * 2);
  // ---- column of the tile being built: KPT consecutive k of column t % 128
  const int bcol = t & 127, bhalf = t >> 7;
  int boff;                                               // patch element of tap (0, 0), first channel of this half
  {
    const IgClass cl = p.cls[py2 + (bcol >> 6)];
    const int n = n0 + (bcol & 63);
    const int il = (n >> p.lgP) - img0;
    const int y = (n & (P - 1)) >> p.lgWo, x = n & (p.Wo - 1);
    boff = il * p.SP + (y - y0 + (cl.oy - rmin)) * p.PW + x + cl.ox + IG_MARGIN;
    boff += ((bhalf * KPT) / TK) * chan_el;
  }
  // ---- weights: regrouped and stored in the order the matrix instructions consume them
  // ([class][row tile][k-tile][32-row block][k-step][lane][8 k], ig_pack_class_w_kernel), so a
  // wavefront loads its own fragments -- 64 rows of its class, four 16-byte loads per lane, each a
  // contiguous 1 KB per wavefront -- straight into registers: no LDS write, no LDS fragment read.
  const int64_t tile_el = (int64_t)ktiles * TM * 32;      // one (class, row tile): every k-tile's TM x 32 block
  // byte offset of this lane's first fragment of k-tile 0
  const uint32_t fo = (uint32_t)((p.cls[py2 + (col0 >> 6)].a_off + (int64_t)tile_m * tile_el) * 2) + (uint32_t)((wm * 4 * 64 + lane) * 16);
  pf_u32x2 qp[2];
  pf_u32x4 fa_cur[2][2], fa_nxt[2][2];                    // fragments [32-row block][k-step] of this and the next k-tile
  auto issue_a = [&](int kt) {
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int s2 = 0; s2 < 2; ++s2)
        fa_nxt[i][s2] = __builtin_amdgcn_raw_buffer_load_b128(
            rw, (int)(kt < ktiles ? fo + (uint32_t)kt * (uint32_t)(TM * 64) + (uint32_t)((i * 2 + s2) * 1024) : PF_OOB), 0, 0);
  };
  auto issue_p = [&](int kt) {
    const int c0 = kt * CPT;
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const uint32_t off = (c0 + pcl[i] < p.Cx && pxo[i] != PF_OOB) ? pxo[i] + (uint32_t)kt * px_step : PF_OOB;
      qp[i] = __builtin_amdgcn_raw_buffer_load_b64(rx, (int)off, 0, 0);
    }
  };
  auto park_a = [&]() {
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int s2 = 0; s2 < 2; ++s2) fa_cur[i][s2] = fa_nxt[i][s2];
  };
  auto park_p = [&](int buf) {
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      if (pl[i] >= 0) {                                   // a store under a branch; the loads stay branch-free
        *reinterpret_cast<uint2*>(Pt(buf) + pl[i]) = make_uint2(qp[i].x, qp[i].y);
      }
    }
  };
  // column tile from the patch: this thread's 16 consecutive k (the taps of 16 / TK channels) of its column
  // (p.tap_step is 1, passed at run time: with a constant step the compiler merges the KW adjacent
  // elements of a window row into one 2-byte-aligned wide LDS read, which the hardware executes
  // several times slower than the separate 2-byte reads.)
  uint32_t bv[KPT];
  auto build_read = [&](int buf) {
    const bf16_raw* src = Pt(buf) + boff;
#pragma unroll
    for (int kk = 0; kk < KPT; ++kk) {
      const int c_l = kk / TK, tap = kk % TK, ty = tap / KW, tx = tap % KW;
      bv[kk] = src[c_l * chan_el + ty * p.PW + tx * p.tap_step];
    }
  };
  auto build_write = [&](int buf) {
    uint32_t w[KPT / 2];
#pragma unroll
    for (int e = 0; e < KPT / 2; ++e) w[e] = bv[2 * e] | (bv[2 * e + 1] << 16);
    unsigned char* dst = Cb(buf) + bcol * GEMM_PITCH + bhalf * KPT * 2;
    *reinterpret_cast<uint4*>(dst) = make_uint4(w[0], w[1], w[2], w[3]);
    *reinterpret_cast<uint4*>(dst + 16) = make_uint4(w[4], w[5], w[6], w[7]);
  };
  const int r = lane & 31, gsel = lane >> 5;
  f32x16_t acc[2][FN];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < FN; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;
  auto mma = [&](int buf) {
    const unsigned char* Bb = Cb(buf) + (col0 + r) * GEMM_PITCH + gsel * 16;
#pragma unroll
    for (int s = 0; s < 2; ++s) {
      bf16x8_t a[2], bq[FN];
#pragma unroll
      for (int i = 0; i < 2; ++i) a[i] = __builtin_bit_cast(bf16x8_t, fa_cur[i][s]);
#pragma unroll
      for (int j = 0; j < FN; ++j) bq[j] = *reinterpret_cast<const bf16x8_t*>(Bb + j * 32 * GEMM_PITCH + s * 32);
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(bq[j], a[i], acc[i][j], 0, 0, 0);
    }
  };

  issue_a(0);
  issue_p(0);
  // zero both patch buffers once: the margins stay zero
  for (int i = t; i < 2 * patch_el / 2; i += NT) reinterpret_cast<uint32_t*>(Pt(0))[i] = 0u;
  __syncthreads();
  park_a();
  park_p(0);
  issue_a(1);
  issue_p(1);
  __syncthreads();
  build_read(0);
  park_p(1);
  issue_p(2);
  build_write(0);
  __syncthreads();
  for (int kt = 0; kt < ktiles; ++kt) {
    const int buf = kt & 1;
    build_read(buf ^ 1);                                  // gather of column tile kt + 1 (patch kt + 1 was parked an iteration ago)
    park_p(buf);                                          // patch kt + 2
    issue_p(kt + 3);
    mma(buf);
    park_a();                                             // fragments kt + 1 become current, kt + 2 requested
    issue_a(kt + 2);
    build_write(buf ^ 1);
    __syncthreads();
  }

  ig_epilogue<true, TM, FN>(p, acc, smem, b, 0, m0, n0, wm, col0, cl0, t, lane);
}

int ilog2(int v) { int l = 0; while ((1 << l) < v) ++l; return l; }
bool pow2(int v) { return v > 0 && (v & (v - 1)) == 0; }

// Pixels of a data gradient's tile (64 of each class), the rows of dY they need.
void dx_geometry(IgArgs& a, int Ho, int Wo) {
  const int P = Ho * Wo;
  a.Ho = Ho; a.Wo = Wo; a.lgWo = ilog2(Wo); a.lgP = ilog2(P);
  if (P >= 64) { a.NI = 1; a.TR = 64 / Wo; } else { a.NI = 64 / P; a.TR = Ho; }
  a.PR = a.TR + 1;
}

// What the gathering kernel is built for: images of four-pixel rows taller than a tile.  The gather reads 2-byte elements and
// the 32 lanes of a half wavefront are eight rows' pixels: at a row pitch of 12 words no two of the rows share a bank (at the
// natural 8 every fourth does).
bool gather_geometry(IgArgs& a) {
  if (a.W != 4 || a.NI != 1) return false;
  a.PW = 24;
  a.SP = a.PR * a.PW;
  a.nchunk = 8 * a.PR;                                    // pieces: a row of each of eight channels
  return true;
}

// byte extents of one model's slices (buffer-load range checks); false when they do not fit 31 bits
bool ig_extents(IgArgs& a) {
  const int64_t xb = ((int64_t)(a.Nb - 1) * a.x_img + (int64_t)a.Cx * a.H * a.W) * 2, ab = a.a_model * 2;
  if (xb >= ((int64_t)1 << 31) || ab >= ((int64_t)1 << 31)) return false;
  a.x_bytes = (uint32_t)xb; a.a_bytes = (uint32_t)ab;
  return true;
}

size_t ig_lds_bytes(const IgArgs& a) {
  const size_t k_loop = 2 * GEMM_TILE_BYTES + 2 * (size_t)8 * a.NI * a.SP * 2;
  const size_t staging = 64 * (size_t)IG_EPI_PITCH;
  return k_loop > staging ? k_loop : staging;
}

// Weights regrouped per output-parity class for the data gradient of a 4x4 / stride 2 / pad 1
// convolution, Wc[class = 2 py + px][c][k = (o, jy, jx)] = W[o][c][ry + 2 (1 - jy)][rx + 2 (1 - jx)] with
// ry = (py + 1) % 2 (the two taps per axis that reach pixels of that parity, in the order in which
// the gradient rows / columns qy + py - 1 + jy they multiply ascend), and stored in the order the
// matrix instructions consume them:
//   Wp[b][class][row tile][k-tile][32-row block][k-step (16 k)][lane][8 k],
//   lane = 32 (k half) + row inside the block; rows past Ci and k past 4 Co are zeros.
// One thread per 16-byte fragment piece of all four classes: 8 k = a class's 2x2 taps of two output channels of one input
// channel, and the 16 taps of the two are read once for the four.  A thread per class read them four times and found its place
// with 64-bit divisions: 10 x 512 x 256 channels 24 -> 17 us, 3 models 8.4 -> 6.  Consecutive lanes read consecutive channels and write
// consecutive pieces.  grid.y: the model.
__global__ __launch_bounds__(256) void ig_pack_class_w_kernel(const bf16_raw* __restrict__ Wt, bf16_raw* __restrict__ Wp, int Ci,
                                                              int Co, int tm, int ktiles, uint32_t pieces) {
  const uint32_t i = blockIdx.x * 256u + threadIdx.x;                // piece of one class of one model
  if (i >= pieces) return;
  const int64_t b = blockIdx.y;
  const int lane = (int)(i & 63u), s2 = (int)((i >> 6) & 1u);
  uint32_t r = i >> 7;
  const uint32_t rbs = (uint32_t)tm >> 5;                            // 2 or 4
  const int rb = (int)(r & (rbs - 1u));
  r = rbs == 4 ? r >> 2 : r >> 1;
  const int tile_m = (int)(r / (uint32_t)ktiles), kt = (int)(r - (uint32_t)tile_m * (uint32_t)ktiles);
  const int c = tile_m * tm + rb * 32 + (lane & 31);
  const int o0 = (kt * 32 + s2 * 16 + (lane >> 5) * 8) >> 2;       // two output channels: o0, o0 + 1
  uint32_t w[2][4][2] = {};                                // rows ky = 0 .. 3; two taps per 32-bit word
  if (c < Ci) {
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      if (o0 + q < Co) {
        const uint4* src = reinterpret_cast<const uint4*>(Wt + ((b * Co + o0 + q) * Ci + c) * 16);
        const uint4 lo = src[0], hi = src[1];
        w[q][0][0] = lo.x; w[q][0][1] = lo.y; w[q][1][0] = lo.z; w[q][1][1] = lo.w;
        w[q][2][0] = hi.x; w[q][2][1] = hi.y; w[q][3][0] = hi.z; w[q][3][1] = hi.w;
      }
    }
  }
#pragma unroll
  for (int cls = 0; cls < 4; ++cls) {
    const int ry = ((cls >> 1) + 1) & 1, rx = ((cls & 1) + 1) & 1;
    uint32_t out[4];
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      auto tap = [&](int ky, int kx) { return (w[q][ky][kx >> 1] >> (16 * (kx & 1))) & 0xffffu; };
      out[2 * q] = tap(ry + 2, rx + 2) | (tap(ry + 2, rx) << 16);      // (jy, jx) = (0, 0), (0, 1)
      out[2 * q + 1] = tap(ry, rx + 2) | (tap(ry, rx) << 16);          // (1, 0), (1, 1)
    }
    *reinterpret_cast<uint4*>(Wp + ((b * 4 + cls) * (int64_t)pieces + i) * 8) = make_uint4(out[0], out[1], out[2], out[3]);
  }
}

#include "conv2d_rows.h"

// out[i] = bf16(act(sum of the k splits' partials + bias of i's channel)); 8 consecutive elements per thread
__global__ __launch_bounds__(256) void ig_split_finish_kernel(const float* __restrict__ part, bf16_raw* __restrict__ out,
                                                              const bf16_raw* __restrict__ bias, int64_t count8, int64_t slice,
                                                              int splits, int64_t o_m, int channels, int act, float slope) {
  const int64_t i8 = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i8 >= count8) return;
  const int64_t i = i8 * 8;
  float v[8];
  {
    const float4 a = *reinterpret_cast<const float4*>(part + i), c = *reinterpret_cast<const float4*>(part + i + 4);
    v[0] = a.x; v[1] = a.y; v[2] = a.z; v[3] = a.w; v[4] = c.x; v[5] = c.y; v[6] = c.z; v[7] = c.w;
  }
  for (int s = 1; s < splits; ++s) {
    const float4 a = *reinterpret_cast<const float4*>(part + s * slice + i), c = *reinterpret_cast<const float4*>(part + s * slice + i + 4);
    v[0] += a.x; v[1] += a.y; v[2] += a.z; v[3] += a.w; v[4] += c.x; v[5] += c.y; v[6] += c.z; v[7] += c.w;
  }
  const float bm = bias ? bf16_to_f32(bias[(i / o_m) % channels]) : 0.f;
#pragma unroll
  for (int e = 0; e < 8; ++e) v[e] = cheap_act(v[e] + bm, act, slope);
  *reinterpret_cast<uint4*>(out + i) = make_uint4(pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3]), pack_bf16x2(v[4], v[5]), pack_bf16x2(v[6], v[7]));
}

// Fewer workgroups of 128-row tiles than compute units: a workgroup is then alone on its unit, its k-tile takes as long as its own
// chain of LDS reads and matrix instructions, and half the rows take about half as long.  us with 128 and with 64 rows (data
// gradient with the weights' regrouping), 3 models x 20 images: 64 <-> 128 channels at 16x16, 120 workgroups, forward 20.0 12.8;
// 128 <-> 256 at 8x8, 120, 21.4 17.8, gradient 22.8 16.8; 256 <-> 512 at 4x4, 144 and 60, 21.6 20.4, gradient 35.3 28.4.  At 192
// the gradient 39.3 36.6; at 384 30.8 29.2 and 31.2 34.0, gradients 30.2 29.8 and 52.0 52.2; at 640 74 90 and 69 78.  32 rows gain
// nothing over 64.
bool few_tiles(int64_t blocks) { return blocks < 256; }

// k split of the forward kernel: taken when the tiles alone leave most compute units with a single workgroup and the
// reduction is long.  512 <- 256 channels at 8x8, unsplit and split in us: 36 tiles 53 21, 96 53 30, 192 53 47, 320 67 71 (the
// bound predates the present kernel; it stays, since another split is another order of the sums).  With 640 tiles and more, and
// for the class-pair data gradient, the split measured no gain or a loss.
int ig_pick_ksplit(int64_t blocks, int ktiles) {
  if (blocks >= 384 || ktiles < 64) return 1;
  return ktiles >= 128 ? 4 : 2;
}

__global__ __launch_bounds__(256) void ig_split_reduce_kernel(const float4* __restrict__ partial, float4* __restrict__ out, int64_t count4, int splits) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= count4) return;
  float4 s = partial[i];
#pragma unroll 8                          // a thread walks up to 64 slices: eight loads in flight, summed in order
  for (int k = 1; k < splits; ++k) {
    const float4 v = partial[(int64_t)k * count4 + i];
    s.x += v.x; s.y += v.y; s.z += v.z; s.w += v.w;
  }
  out[i] = s;
}

#include "conv2d_planes.h"

constexpr size_t IG_MAX_LDS = 96 * 1024;

// Kernels here take more dynamic LDS than the default limit allows: the limit of each instantiation
// is raised before its launches (an idempotent attribute of the loaded kernel, not library state).
template <typename K>
void ig_launch(K kernel, dim3 grid, int threads, size_t lds, hipStream_t st, IgArgs a) {
  if (lds > 48 * 1024) (void)hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, (int)IG_MAX_LDS);
  a.grid = IgGrid{(int)grid.x, (int)grid.y, (int)grid.z};
  hipLaunchKernelGGL(kernel, dim3(grid.x * grid.y * grid.z), dim3((unsigned)threads), lds, st, a);
}

}  // namespace

// Forward of the grouped convolution (also the data gradient of the transposed convolution).
// HFTA_EUNSUPPORTED when the shape is outside what the kernel handles (the caller falls back).
// fp32 partial slices the forward wants for its k split (0: no split).  Without that much workspace it runs unsplit.
size_t conv_ig_fwd_split_bytes(int B, int Nb, int Ci, int Co, int H, int W) {
  const int Ho = H / 2, Wo = W / 2, tm = Co <= 64 ? 64 : 128;
  if (Ho <= 0 || Wo <= 0) return 0;
  const int64_t blocks = (int64_t)((Co + tm - 1) / tm) * (((int64_t)Nb * Ho * Wo + 127) / 128) * B;
  const int ks = ig_pick_ksplit(blocks, (Ci * 16 + 31) / 32);
  return ks > 1 ? (size_t)ks * Nb * B * Co * Ho * Wo * sizeof(float) : 0;
}

int conv_ig_forward(int B, int Nb, int Ci, int Co, int H, int W, int kh, int kw, int stride, int pad, const void* X,
                    const void* Wt, const void* bias, void* Y, int act, float slope, void* ws, size_t ws_bytes,
                    hipStream_t st) {
  const int Ho = (H + 2 * pad - kh) / stride + 1, Wo = (W + 2 * pad - kw) / stride + 1;
  if (kh != 4 || kw != 4 || stride != 2 || pad != 1) return HFTA_EUNSUPPORTED;
  if (!pow2(Ho) || !pow2(Wo) || Wo < 4 || Ho * Wo < 16 || W % 8 != 0 || (128 % (Ho * Wo) != 0 && (Ho * Wo) % 128 != 0)) return HFTA_EUNSUPPORTED;
  if ((Ho * Wo >= 128 && 128 % Wo != 0) || (int64_t)Nb * Ho * Wo > 0x7fffffff) return HFTA_EUNSUPPORTED;
  if (act != HFTA_ACT_NONE && act != HFTA_ACT_RELU && act != HFTA_ACT_LEAKY) return HFTA_EUNSUPPORTED;
  if (reinterpret_cast<uintptr_t>(X) % 16 || reinterpret_cast<uintptr_t>(Wt) % 16 || reinterpret_cast<uintptr_t>(Y) % 16) return HFTA_EUNSUPPORTED;
  IgArgs a{};
  a.X = (const bf16_raw*)X; a.A = (const bf16_raw*)Wt; a.Out = (bf16_raw*)Y; a.bias = (const bf16_raw*)bias;
  a.x_img = (int64_t)B * Ci * H * W; a.x_model = (int64_t)Ci * H * W;
  a.a_model = (int64_t)Co * Ci * 16;
  a.o_img = (int64_t)B * Co * Ho * Wo; a.o_model = (int64_t)Co * Ho * Wo; a.o_m = (int64_t)Ho * Wo;
  a.Nb = Nb; a.Cx = Ci; a.H = H; a.W = W;
  a.M = Co; a.K = Ci * 16; a.N = Nb * Ho * Wo;
  if (!ig_extents(a)) return HFTA_EUNSUPPORTED;
  a.OW = Wo; a.oys = 1; a.oxs = 1;
  a.lgWo = ilog2(Wo); a.lgP = ilog2(Ho * Wo); a.Ho = Ho; a.Wo = Wo;
  rows_fwd_geometry(a);
  const int tm = Co <= 64 ? 64 : 128;
  a.tiles_n = (a.N + 127) / 128;
  a.act = act; a.slope = slope;
  const int tiles_m = (Co + tm - 1) / tm;
  if ((int64_t)tiles_m * a.tiles_n > 0x7fffffff || B > 65535) return HFTA_EUNSUPPORTED;
  const size_t need = conv_ig_fwd_split_bytes(B, Nb, Ci, Co, H, W);
  a.ksplit = (need && ws && ws_bytes >= need && reinterpret_cast<uintptr_t>(ws) % 16 == 0)
                 ? ig_pick_ksplit((int64_t)tiles_m * a.tiles_n * B, (a.K + 31) / 32) : 1;
  a.kt_per_split = ((a.K + 63) / 64 + a.ksplit - 1) / a.ksplit;
  a.part = reinterpret_cast<float*>(ws);
  a.part_split = (int64_t)Nb * a.o_img;
  const size_t lds = rows_fwd_lds_bytes(a, tm);
  if (lds > IG_MAX_LDS) return HFTA_EUNSUPPORTED;
  // Too few 128-row tiles for the chip: tiles of 64 rows, whose sums are the same ones (the k split stays that of the 128-row tiles).
  const bool halves = few_tiles((int64_t)tiles_m * a.tiles_n * a.ksplit * B);
  dim3 grid((unsigned)((halves ? (Co + 63) / 64 : tiles_m) * a.tiles_n), (unsigned)a.ksplit, (unsigned)B);
  if (tm == 64 || halves) ig_launch(conv_rows_fwd_kernel<64>, grid, 256, lds, st, a);
  else ig_launch(conv_rows_fwd_kernel<128>, grid, 256, lds, st, a);
  if (a.ksplit > 1) {
    if (launch_status() != HFTA_OK) return HFTA_ELAUNCH;
    const int64_t count8 = a.part_split / 8;
    hipLaunchKernelGGL(ig_split_finish_kernel, dim3((unsigned)((count8 + 255) / 256)), dim3(256), 0, st, (const float*)a.part,
                       a.Out, a.bias, count8, a.part_split, a.ksplit, a.o_m, B * Co, act, slope);
  }
  return launch_status();
}

}  // namespace hfta

namespace hfta {

// Data gradient of the 4x4 / stride 2 / pad 1 grouped convolution (= forward of the transposed one):
// four parity classes (grid.y = py, the two px of a tile side by side), each a stride-1 2x2 correlation
// over dY with its regrouped weights.
// `pack` receives the regrouped weights: conv_ig_dx_pack_bytes(...) bytes, 16-byte aligned.
size_t conv_ig_dx_pack_bytes(int B, int Ci, int Co) {                  // whole row tiles and k-tiles; a multiple of 256 bytes
  const int tm = Ci <= 64 ? 64 : 128, tiles_m = (Ci + tm - 1) / tm, ktiles = (Co * 4 + 31) / 32;
  return (size_t)B * 4 * tiles_m * tm * ktiles * 32 * sizeof(bf16_raw);
}

bool conv_ig_dx_supported(int Nb, int Ci, int Co, int H, int W, int kh, int kw, int stride, int pad) {
  if (kh != 4 || kw != 4 || stride != 2 || pad != 1 || H % 2 || W % 2) return false;
  const int Hq = H / 2, Wq = W / 2;
  if (!pow2(Hq) || !pow2(Wq) || Wq < 4 || Wq > 64 || Hq * Wq < 16) return false;
  if ((int64_t)Nb * Hq * Wq > 0x7fffffff || Ci < 32 || Co % 2 != 0) return false;
  return true;
}

int conv_ig_dx(int B, int Nb, int Ci, int Co, int H, int W, int kh, int kw, int stride, int pad, const void* Wt,
               const void* dY, void* dX, void* pack, hipStream_t st) {
  if (!conv_ig_dx_supported(Nb, Ci, Co, H, W, kh, kw, stride, pad)) return HFTA_EUNSUPPORTED;
  if (reinterpret_cast<uintptr_t>(dY) % 16 || reinterpret_cast<uintptr_t>(Wt) % 16 || reinterpret_cast<uintptr_t>(dX) % 16 ||
      reinterpret_cast<uintptr_t>(pack) % 16 || B > 65535)
    return HFTA_EUNSUPPORTED;
  const int Hq = H / 2, Wq = W / 2;                      // class grid = the gradient's own grid (Ho x Wo)
  IgArgs a{};
  a.X = (const bf16_raw*)dY; a.A = (const bf16_raw*)pack; a.Out = (bf16_raw*)dX; a.bias = nullptr;
  a.x_img = (int64_t)B * Co * Hq * Wq; a.x_model = (int64_t)Co * Hq * Wq;
  a.Nb = Nb; a.Cx = Co; a.H = Hq; a.W = Wq;
  dx_geometry(a, Hq, Wq);
  const bool planes = dxp_geometry(a);
  a.tiles_n = (int)(((int64_t)Nb * Hq * Wq + 63) / 64);
  const int tm = Ci <= 64 || (planes && few_tiles((int64_t)((Ci + 127) / 128) * a.tiles_n * 2 * B)) ? 64 : 128;
  const int tiles_m = (Ci + tm - 1) / tm, ktiles = (Co * 4 + 31) / 32;
  const int64_t cls_el = (int64_t)tiles_m * tm * ktiles * 32;          // one class of one model, fragment order: at most what the query counts
  a.a_model = 4 * cls_el;
  a.o_img = (int64_t)B * Ci * H * W; a.o_model = (int64_t)Ci * H * W; a.o_m = (int64_t)H * W;
  a.M = Ci; a.K = Co * 4; a.N = Nb * Hq * Wq;
  if (!ig_extents(a)) return HFTA_EUNSUPPORTED;
  a.OW = W; a.oys = 2; a.oxs = 2; a.tap_step = 1;
  if (!planes && !gather_geometry(a)) return HFTA_EUNSUPPORTED;
  a.act = HFTA_ACT_NONE; a.slope = 0.f;
  for (int cls = 0; cls < 4; ++cls) {
    const int py = cls >> 1, px = cls & 1;
    a.cls[cls] = IgClass{py - 1, px - 1, py, px, cls * cls_el};          // window rows qy + py - 1, qy + py
  }
  const size_t lds = planes ? dxp_lds_bytes(a) : ig_lds_bytes(a);
  if (lds > IG_MAX_LDS) return HFTA_EUNSUPPORTED;
  if ((int64_t)tiles_m * a.tiles_n > 0x7fffffff) return HFTA_EUNSUPPORTED;
  const int64_t pieces = cls_el / 8;                                   // 16-byte fragment pieces
  if (pieces > 0x7fffffff) return HFTA_EUNSUPPORTED;
  hipLaunchKernelGGL(ig_pack_class_w_kernel, dim3((unsigned)((pieces + 255) / 256), (unsigned)B), dim3(256), 0, st, (const bf16_raw*)Wt,
                     (bf16_raw*)pack, Ci, Co, tm, ktiles, (uint32_t)pieces);
  a.ksplit = 1;
  a.kt_per_split = ktiles;
  dim3 grid((unsigned)(tiles_m * a.tiles_n), 2u, (unsigned)B);
  if (planes) {
    const bool few = few_tiles((int64_t)tiles_m * a.tiles_n * 2 * B);    // (of 128 rows: never)
    if (a.W == 4) {
      if (tm == 64) few ? ig_launch(conv_dx_planes_kernel<64, true, 2>, grid, 256, lds, st, a) : ig_launch(conv_dx_planes_kernel<64, true, 1>, grid, 256, lds, st, a);
      else ig_launch(conv_dx_planes_kernel<128, true, 1>, grid, 256, lds, st, a);
    } else {
      if (tm == 64) few ? ig_launch(conv_dx_planes_kernel<64, false, 2>, grid, 256, lds, st, a) : ig_launch(conv_dx_planes_kernel<64, false, 1>, grid, 256, lds, st, a);
      else ig_launch(conv_dx_planes_kernel<128, false, 1>, grid, 256, lds, st, a);
    }
  } else {
    if (tm == 64) ig_launch(conv_ig_gather_kernel<64>, grid, 256, lds, st, a);
    else ig_launch(conv_ig_gather_kernel<128>, grid, 256, lds, st, a);
  }
  return launch_status();
}

}  // namespace hfta

namespace hfta {

// Weight gradient of the 4x4 / stride 2 / pad 1 grouped convolution.  `partial` holds the k splits'
// fp32 slices when conv_ig_dw_splits(...) > 1 (that many times B * Co * Ci * 16 floats).
bool conv_ig_dw_supported(int Nb, int Ci, int Co, int H, int W, int kh, int kw, int stride, int pad) {
  if (kh != 4 || kw != 4 || stride != 2 || pad != 1 || H % 2 || W % 2) return false;
  const int Ho = H / 2, Wo = W / 2;
  if (!pow2(Ho) || !pow2(Wo) || Wo < 4 || Wo > 32 || Ho * Wo < 16) return false;
  if ((int64_t)Nb * Ho * Wo > 0x7fffffff || Co < 32) return false;   // fewer than 8 input channels: the missing columns are zeros
  return true;                                           // a k-tile's second 4x4 sample past the batch reads as zeros
}

int conv_ig_dw_splits(int B, int Nb, int Ci, int Co, int H, int W) {
  const int64_t kt_total = ((int64_t)Nb * (H / 2) * (W / 2) + 31) / 32;
  const int64_t tiles = (int64_t)((Co + 127) / 128) * ((Ci + 7) / 8) * B;
  if (tiles >= 512 || kt_total < 32) return 1;
  // more splits only add partial-slice traffic (measured 512 .. 1536)
  int64_t want = (512 + tiles - 1) / tiles, cap = kt_total / 16;
  if (want > cap) want = cap;
  if (want > 64) want = 64;
  return want < 1 ? 1 : (int)want;
}

int conv_ig_dw(int B, int Nb, int Ci, int Co, int H, int W, int kh, int kw, int stride, int pad, const void* X,
               const void* dY, float* dW, float* partial, hipStream_t st) {
  if (!conv_ig_dw_supported(Nb, Ci, Co, H, W, kh, kw, stride, pad)) return HFTA_EUNSUPPORTED;
  if (reinterpret_cast<uintptr_t>(X) % 16 || reinterpret_cast<uintptr_t>(dY) % 16 || reinterpret_cast<uintptr_t>(dW) % 16 ||
      reinterpret_cast<uintptr_t>(partial) % 16 || B > 65535)
    return HFTA_EUNSUPPORTED;
  const int Ho = H / 2, Wo = W / 2, P = Ho * Wo;
  IgDwArgs a{};
  a.X = (const bf16_raw*)X; a.dY = (const bf16_raw*)dY;
  a.x_img = (int64_t)B * Ci * H * W; a.x_model = (int64_t)Ci * H * W;
  a.y_img = (int64_t)B * Co * P; a.y_model = (int64_t)Co * P;
  a.o_model = (int64_t)Co * Ci * 16;
  if (W % 8 != 0) return HFTA_EUNSUPPORTED;
  a.Nb = Nb; a.Ci = Ci; a.Co = Co; a.H = H; a.W = W; a.Wo = Wo;
  a.lgWo = ilog2(Wo); a.lgP = ilog2(P);
  a.NI = P >= 32 ? 1 : 32 / P;
  a.PR = 2 * (P >= 32 ? 32 / Wo : Ho) + 2;
  a.nchunk = 8 * a.NI * a.PR * (W / 8);                  // at most 256, one per thread: 16 + NI Wo / 2 a channel, NI Wo <= 32
  // the eight lanes that an LDS clock serves read eight taps of a channel (four planes of two rows, 16 bytes each): these
  // pitches put them on different banks
  a.plane_b = Wo * 2 + (Wo >= 16 ? 16 : 0);
  a.row_b = 4 * a.plane_b;
  const int64_t xb = ((int64_t)(Nb - 1) * a.x_img + (int64_t)Ci * H * W) * 2, yb = ((int64_t)(Nb - 1) * a.y_img + (int64_t)Co * P) * 2;
  if (xb >= ((int64_t)1 << 31) || yb >= ((int64_t)1 << 31)) return HFTA_EUNSUPPORTED;
  a.x_bytes = (uint32_t)xb; a.y_bytes = (uint32_t)yb;
  a.tiles_n = (Ci + 7) / 8;
  a.kt_total = (int)(((int64_t)Nb * P + 31) / 32);
  const int splits = conv_ig_dw_splits(B, Nb, Ci, Co, H, W);
  if (splits > 1 && !partial) return HFTA_EWORKSPACE;
  a.kt_per_split = (a.kt_total + splits - 1) / splits;
  a.o_split = (int64_t)B * a.o_model;
  a.Out = splits > 1 ? partial : dW;
  const size_t k_loop = 2 * ((size_t)GEMM_TILE_BYTES + (size_t)8 * a.NI * a.PR * a.row_b);
  const size_t staging = 64 * (size_t)EPI_PITCH4;
  const size_t lds = k_loop > staging ? k_loop : staging;
  if (lds > IG_MAX_LDS) return HFTA_EUNSUPPORTED;
  const int tiles_m = (Co + 127) / 128;
  a.grid = IgGrid{tiles_m * a.tiles_n, splits, B};
  if ((int64_t)a.grid.gx * splits * B > 0x7fffffff) return HFTA_EUNSUPPORTED;
  auto launch = [&](auto kernel) {
    if (lds > 48 * 1024) (void)hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, (int)IG_MAX_LDS);
    hipLaunchKernelGGL(kernel, dim3((unsigned)(a.grid.gx * splits * B)), dim3(256), lds, st, a);
  };
  if (Wo == 4) launch(conv_rows_dw_kernel<true>);
  else launch(conv_rows_dw_kernel<false>);
  if (launch_status() != HFTA_OK) return HFTA_ELAUNCH;
  if (splits > 1) {
    const int64_t count4 = (int64_t)B * a.o_model / 4;
    hipLaunchKernelGGL(ig_split_reduce_kernel, dim3((unsigned)((count4 + 255) / 256)), dim3(256), 0, st, (const float4*)partial,
                       (float4*)dW, count4, splits);
  }
  return launch_status();
}

}  // namespace hfta
