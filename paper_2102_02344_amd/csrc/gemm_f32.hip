// fp32 form of the batched GEMM core (same descriptor, same operand kinds as gemm.h).
//
// The fp32 matrix instruction reaches 154 TFLOP/s here (a library product of 8192 x 8192 x 8192); the bf16 one does
// sixteen times the work per cycle, and an fp32 value IS the sum of three bf16 ones: h, the value rounded, m, the rest
// rounded, l, what is left (8 + 8 + 8 bits).  Six of the nine products of two such sums are formed (hh, hm, mh, hl, mm,
// lh; the others are below 2^-26 of the product), in fp32 accumulators, for 6/16 of the fp32 instruction's time.
// The corrections have accumulators of their own: the bf16 instruction rounds its sum (to nearest: sums of positive values
// are off by 3.0e-7 at K = 4096 and 1.7e-6 at 80000, their signed mean by 5e-9 and 6e-7, where the fp32 instruction, which
// rounds every two k, leaves 8.5e-7 and 4.7e-6, 5e-9 and 1.7e-6), and in one accumulator six roundings per 16 k of a long weight gradient left a
// larger error (1.5e-6) than the fp32 instruction's (1.3e-6); in two it is 4.4e-7.  Measured for 128 -> 1024 channels on 4 x 32 x 2500 points, in the step: data gradient
// 696 -> 520 us, weight gradient 693 -> 499, forward 815 -> 782 (four k-tiles a tile: bound by a tile's first loads and
// its stores); relative errors against float64 5.7e-7 -> 1.9e-7, 1.3e-6 -> 4.4e-7, 2.0e-7 -> 6.5e-8.  On 2 x 4 x 256
// points the data gradient's 64 workgroups take 27 us instead of 39.
// A value is split once, on its way into LDS, whose tiles are three bf16 planes per operand.
//
// The sum of three needs a finite value that is not tiny: an infinity or a NaN has no remainder, nor has what rounds up
// to infinity, and below 2^-110 the last part falls under bf16's smallest numbers.  Both are noticed while splitting
// (the remainder is NaN; a smallest magnitude is kept), and a workgroup that has seen one takes its tile again from the
// start with fp32 matrix instructions (`exact_loop`): one value between 0 and 2^-100 in every tile of the layer above makes it
// 1287 us forward, 1198 and 1197 backward, where the fp32 instruction alone took 803, 688 and 704.  Operands with fewer than four elements along their contiguous
// dimension (VEC = 0, single-element loads) have that loop only.
//
// Every load is a raw buffer load without control flow (out of range = zeros, see gemm_pf.h), in 16-byte pieces whatever
// the row pitch (a multi-dword access needs 4-byte alignment only, and an fp32 row has that).  VEC = 2: no piece straddles
// a row's end, so the k-loop's body is one straight block.  VEC = 1: one that does is read from where the row's last four
// elements start and moved into place on its way into LDS.
//
// NB: matrix blocks per wavefront and dimension.  NB = 2 (128x128 tile): the throughput form; its two sets of
// accumulators leave two workgroups per compute unit, each with one k-tile in flight in registers and one in LDS (two of
// 16 k each were 0-7 % slower: half a line of a k-contiguous row at a time).  NB = 1 (64x64 tile, two k-tiles each):
// four times the workgroups, for problems that would leave compute units idle.
#include "gemm_pf.h"
#include "f32_split.h"

namespace hfta {

namespace {

// floats of k per tile: of the split a whole 128-byte line of a k-contiguous row; of the fp32 instruction half of one
constexpr int f32_bk(bool split) { return split ? 32 : 16; }
constexpr int F32_SMALL_TILES = 512;                       // fewer 128x128 tiles than this: 64x64 tiles
typedef uint32_t pf_u32x4_a4 __attribute__((ext_vector_type(4), aligned(4)));

// rotates a four-element piece that was read `sh` elements early into place; what lies past the end becomes zero
__device__ __forceinline__ float4 shift_piece(float4 v, int sh) {
  if (sh & 1) v = make_float4(v.y, v.z, v.w, 0.f);
  if (sh & 2) v = make_float4(v.z, v.w, 0.f, 0.f);
  return v;
}

__device__ __forceinline__ float4 ld_f4(__amdgpu_buffer_rsrc_t rs, uint32_t off) {
  const pf_u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(rs, (int)off, 0, 0);
  return make_float4(__uint_as_float(v.x), __uint_as_float(v.y), __uint_as_float(v.z), __uint_as_float(v.w));
}
__device__ __forceinline__ float ld_f1(__amdgpu_buffer_rsrc_t rs, uint32_t off) {
  return __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rs, (int)off, 0, 0));
}

template <bool KC, int NB, int VEC, int BK> struct F32Operand;

// k-contiguous: thread t stages 4-float group t % PR of rows t / PR + h * RPI
template <int NB, int VEC, int BK> struct F32Operand<true, NB, VEC, BK> {
  static constexpr int PR = BK / 4, RPI = GEMM_THREADS / PR, H = 64 * NB / RPI;
  static constexpr int PITCH = BK * 4 + 16;                // fp32 tile: [row][BK k + 4 pad]
  static constexpr int BYTES = 64 * NB * PITCH;
  static constexpr int PLANE = 64 * NB * BK * 2;           // bf16 plane: [row][BK k], 16-byte pieces permuted
  typedef float4 Regs[H];
  uint32_t off[H];
  int kg;
  __device__ __forceinline__ void init(int row0, int rows, int64_t ld, int t) {
    kg = (t % PR) * 4;
#pragma unroll
    for (int h = 0; h < H; ++h) {
      const int r = row0 + t / PR + RPI * h;
      off[h] = r < rows ? (uint32_t)((int64_t)r * ld * 4) : PF_OOB;
    }
  }
  __device__ __forceinline__ void load(Regs& q, __amdgpu_buffer_rsrc_t rs, int k0, int K) const {
    const int k = k0 + kg;
#pragma unroll
    for (int h = 0; h < H; ++h) {
      if (VEC) {
        q[h] = ld_f4(rs, k < K ? off[h] + (uint32_t)(VEC == 2 ? k : min(k, K - 4)) * 4u : PF_OOB);
      } else {
        float e[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) e[i] = ld_f1(rs, k + i < K ? off[h] + (uint32_t)(k + i) * 4u : PF_OOB);
        q[h] = make_float4(e[0], e[1], e[2], e[3]);
      }
    }
  }
  // the k-tile reaches past K (the same for the whole workgroup)
  __device__ __forceinline__ void place(Regs& q, int k0, int K) const {
    if (VEC == 1 && k0 + BK > K) {
      const int k = k0 + kg, sh = k < K ? k - min(k, K - 4) : 0;
#pragma unroll
      for (int h = 0; h < H; ++h) q[h] = shift_piece(q[h], sh);
    }
  }
  __device__ __forceinline__ void store(unsigned char* tile, const Regs& q, int t) const {
#pragma unroll
    for (int h = 0; h < H; ++h) *reinterpret_cast<float4*>(tile + (t / PR + RPI * h) * PITCH + kg * 4) = q[h];
  }
  // the four k of step s for row base + lane%32: k = 8 s + 4 (lane/32) + j
  static __device__ __forceinline__ void frag(float (&f)[4], const unsigned char* tile, int base, int s, int lane) {
    const float4 v = *reinterpret_cast<const float4*>(tile + (base + (lane & 31)) * PITCH + (2 * s + (lane >> 5)) * 16);
    f[0] = v.x; f[1] = v.y; f[2] = v.z; f[3] = v.w;
  }
  // 16-byte piece p of row r sits at p ^ swz(r): sixteen rows' pieces of one k cover the 64 banks once
  static __device__ __forceinline__ int swz(int r) { return (r >> 2) & 3; }
  __device__ __forceinline__ void store_split(unsigned char* tile, const Regs& q, int t, SplitSeen& seen) const {
#pragma unroll
    for (int h = 0; h < H; ++h) {
      uint2 o[3];
      split4(q[h], o, seen);
      const int r = t / PR + RPI * h;
      unsigned char* d = tile + r * (BK * 2) + (((kg >> 3) ^ swz(r)) << 4) + (kg & 4) * 2;
#pragma unroll
      for (int i = 0; i < 3; ++i) *reinterpret_cast<uint2*>(d + i * PLANE) = o[i];
    }
  }
  // bf16 fragment of plane `pl`: lane l holds row base + l%32 and k = 16 s + 8 (l/32) + 0..7
  static __device__ __forceinline__ bf16x8_t frag16(const unsigned char* tile, int pl, int base, int s, int lane) {
    const int r = base + (lane & 31);
    return *reinterpret_cast<const bf16x8_t*>(tile + pl * PLANE + r * (BK * 2) + (((2 * s + (lane >> 5)) ^ swz(r)) << 4));
  }
};

// m/n-contiguous: natural [k][column] layout; thread t stages columns 4 (t % CG) .. of k-rows t / CG + h * RS
template <int NB, int VEC, int BK> struct F32Operand<false, NB, VEC, BK> {
  static constexpr int COLS = 64 * NB;
  static constexpr int PITCH = (COLS + 8) * 4;             // fp32 tile: k-rows four apart are 32 banks apart
  static constexpr int BYTES = BK * PITCH;
  static constexpr int PLANE = BK * COLS * 2;              // bf16 plane: [k][column], 16-byte pieces permuted
  static constexpr int CG = COLS / 4, RS = GEMM_THREADS / CG, H = BK / RS;
  typedef float4 Regs[H];
  uint32_t ldb;
  uint32_t coff;                                           // byte offset of the piece in k-row kr, or PF_OOB
  int kr, sh;
  __device__ __forceinline__ void init(int col0, int cols, int64_t ld, int t) {
    ldb = (uint32_t)(ld * 4);
    kr = t / CG;
    const int c = col0 + (t % CG) * 4;
    if (VEC) {
      const int cc = min(c, cols - 4);
      coff = c < cols ? (uint32_t)kr * ldb + (uint32_t)cc * 4u : PF_OOB;
      sh = c < cols ? c - cc : 0;
    } else {
      coff = (uint32_t)kr * ldb + (uint32_t)c * 4u;
      sh = cols - c;                                       // elements of the piece that exist (may exceed four)
    }
  }
  __device__ __forceinline__ void load(Regs& q, __amdgpu_buffer_rsrc_t rs, int k0, int K) const {
#pragma unroll
    for (int h = 0; h < H; ++h) {
      const bool in = k0 + kr + RS * h < K;
      const uint32_t o = coff + (uint32_t)(k0 + RS * h) * ldb;             // slices are below 2 GiB
      if (VEC) {
        q[h] = ld_f4(rs, in && coff != PF_OOB ? o : PF_OOB);
      } else {
        float e[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) e[i] = ld_f1(rs, in && i < sh ? o + 4u * i : PF_OOB);
        q[h] = make_float4(e[0], e[1], e[2], e[3]);
      }
    }
  }
  __device__ __forceinline__ void place(Regs& q, int, int) const {
    if (VEC == 1 && __any(sh != 0)) {
#pragma unroll
      for (int h = 0; h < H; ++h) q[h] = shift_piece(q[h], sh);
    }
  }
  __device__ __forceinline__ void store(unsigned char* tile, const Regs& q, int t) const {
#pragma unroll
    for (int h = 0; h < H; ++h) *reinterpret_cast<float4*>(tile + (kr + RS * h) * PITCH + (t % CG) * 16) = q[h];
  }
  static __device__ __forceinline__ void frag(float (&f)[4], const unsigned char* tile, int base, int s, int lane) {
    const unsigned char* a = tile + (8 * s + 4 * (lane >> 5)) * PITCH + (base + (lane & 31)) * 4;
#pragma unroll
    for (int j = 0; j < 4; ++j) f[j] = *reinterpret_cast<const float*>(a + j * PITCH);
  }
  // piece p of k-row k sits at p ^ swz(k): the four k-rows of a transpose read cover the 64 banks once
  static __device__ __forceinline__ int swz(int k) { return NB == 2 ? (k & 3) << 2 : ((k >> 1) & 1) << 2; }
  __device__ __forceinline__ void store_split(unsigned char* tile, const Regs& q, int t, SplitSeen& seen) const {
    const int c4 = t % CG;
#pragma unroll
    for (int h = 0; h < H; ++h) {
      uint2 o[3];
      split4(q[h], o, seen);
      const int k = kr + RS * h;
      unsigned char* d = tile + k * (COLS * 2) + (((c4 >> 1) ^ swz(k)) << 4) + (c4 & 1) * 8;
#pragma unroll
      for (int i = 0; i < 3; ++i) *reinterpret_cast<uint2*>(d + i * PLANE) = o[i];
    }
  }
  // through the LDS transpose read (see gemm_pf.h)
  static __device__ __forceinline__ bf16x8_t frag16(const unsigned char* tile, int pl, int base, int s, int lane) {
    const int r16 = lane & 15, k = 8 * (lane >> 5) + (r16 >> 2);           // + 16 s: the same position pattern
    const int piece = (base >> 3) + 2 * ((lane >> 4) & 1) + ((r16 & 3) >> 1);
    const unsigned char* a0 = tile + pl * PLANE + (16 * s + k) * (COLS * 2) + ((piece ^ swz(k)) << 4) + (r16 & 1) * 8;
    typedef __attribute__((address_space(3))) pf_v4s* lds_v4s;
    union { pf_v4s h[2]; bf16x8_t v; } u;
    u.h[0] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4s)(a0));
    u.h[1] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4s)(a0 + 4 * (COLS * 2)));
    return u.v;
  }
};

template <int NB>
constexpr int f32_smem_bytes(int tiles) {
  const int epi = 64 * (64 * NB + 4) * 4; // the epilogue's staging: 64 rows at a time
  return tiles > epi ? tiles : epi;
}

// POOL: the epilogue also leaves what a BatchNorm and a maximum over each row need (GemmDesc::pool_part), from the staged
// rows: four threads a row, one loop for sum and maximum, one for the squares about the mean.
// The output itself is stored only if there is a place for it (p.C).
// HITS: columns of the output that get rows of another matrix added (GemmDesc::hit_key), while they are staged.
template <bool A_KC, bool B_KC, int NB, int VEC, bool SPLIT, bool POOL = false, bool HITS = false>
__global__ __launch_bounds__(GEMM_THREADS, NB == 2 && SPLIT ? 2 : 3) void gemm_f32_kernel(GemmArgs p) {
  constexpr int T = 64 * NB, BK = f32_bk(SPLIT);
  typedef F32Operand<A_KC, NB, VEC, BK> OA;
  typedef F32Operand<B_KC, NB, VEC, BK> OB;
  constexpr int PF = NB == 2 && SPLIT ? 1 : 2;             // k-tiles in flight in registers = LDS buffers
  constexpr int EXACT = PF * (OA::BYTES + OB::BYTES), PLANES = SPLIT ? PF * 3 * (OA::PLANE + OB::PLANE) : 0;
  __shared__ __attribute__((aligned(16))) unsigned char smem[f32_smem_bytes<NB>(PLANES > EXACT ? PLANES : EXACT)];

  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  const int wm = wave >> 1, wn = wave & 1;
  int bx = blockIdx.x, bz = blockIdx.z;
  {  // XCD-aware renumbering, as in gemm_kernel
    const int total = gridDim.x * gridDim.z, per = total >> 3;
    const int lin = blockIdx.x + gridDim.x * blockIdx.z;
    if (lin < (per << 3)) {
      const int l2 = (lin & 7) * per + (lin >> 3);
      bz = l2 / gridDim.x;
      bx = l2 - bz * gridDim.x;
    }
  }
  const int tile_m = bx % p.tiles_m, tile_n = bx / p.tiles_m;
  const int m0 = tile_m * T, n0 = tile_n * T;
  const int split = bz % p.splits, g = bz / p.splits;
  const int g0 = g / p.G1, g1 = g % p.G1;
  const float* Ab = reinterpret_cast<const float*>(p.A) + g0 * p.a_g0 + g1 * p.a_g1;
  const float* Bb = reinterpret_cast<const float*>(p.Bm) + g0 * p.b_g0 + g1 * p.b_g1;
  const int t_begin = (int)((int64_t)p.total_tiles * split / p.splits);
  const int t_end = (int)((int64_t)p.total_tiles * (split + 1) / p.splits);

  f32x16_t acc[NB][NB], low[NB][NB];
  auto clear = [&]() {
#pragma unroll
    for (int i = 0; i < NB; ++i)
#pragma unroll
      for (int j = 0; j < NB; ++j)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[i][j][v] = low[i][j][v] = 0.f;
  };

  OA oa;
  OB ob;
  oa.init(m0, p.M, p.a_ld, t);
  ob.init(n0, p.N, p.b_ld, t);
  typename OA::Regs ra[PF];
  typename OB::Regs rb[PF];
  // the loader's k-tile: segment base and k0, stepped without a division; past the end nothing is requested
  const float *la, *lb;
  int lk, lt;
  auto aim = [&](int tt) {
    const int seg = tt / p.tiles_per_seg;
    la = Ab + seg * p.a_ss;
    lb = Bb + seg * p.b_ss;
    lk = (tt - seg * p.tiles_per_seg) * BK;
    lt = tt;
  };
  auto issue = [&](int set) {
    const int Ke = lt < t_end ? p.K : 0;
    oa.load(ra[set], pf_rsrc(la, p.a_extent), lk, Ke);
    ob.load(rb[set], pf_rsrc(lb, p.b_extent), lk, Ke);
    lk += BK;
    const bool wrap = lk >= p.K;
    la += wrap ? p.a_ss : 0;
    lb += wrap ? p.b_ss : 0;
    lk = wrap ? 0 : lk;
    ++lt;
  };
  // the reduction over [t_begin, t_end): `park` puts a register set into an LDS buffer, `multiply` takes a buffer
  auto reduce = [&](auto park, auto multiply) {
    clear();
    if (t_begin >= t_end) return;
    int sk = (t_begin % p.tiles_per_seg) * BK;             // k0 of the tile about to be parked
    auto stage = [&](int buf, int set) {
      oa.place(ra[set], sk, p.K);
      ob.place(rb[set], sk, p.K);
      sk = sk + BK >= p.K ? 0 : sk + BK;
      park(buf, set);
    };
    aim(t_begin);
#pragma unroll
    for (int d = 0; d < PF; ++d) issue(d);
    if constexpr (PF == 1) {
      for (int cur = t_begin; cur < t_end; ++cur) {
        if (cur != t_begin) __syncthreads();
        stage(0, 0);
        __syncthreads();
        issue(0);
        multiply(0);
      }
    } else {
      stage(0, 0);
      __syncthreads();
      for (int cur = t_begin;; cur += 2) {
        bool done = false;
#pragma unroll
        for (int d = 0; d < 2; ++d) {
          issue(d);
          multiply(d);
          stage(d ^ 1, d ^ 1);                             // past the end: zeros that nobody reads
          __syncthreads();
          if (cur + d + 1 >= t_end) { done = true; break; }
        }
        if (done) break;
      }
    }
    __syncthreads();
  };
  auto exact_loop = [&]() {
    auto at = [&](int buf) { return smem + buf * OA::BYTES; };
    auto bt = [&](int buf) { return smem + PF * OA::BYTES + buf * OB::BYTES; };
    reduce([&](int buf, int set) { oa.store(at(buf), ra[set], t); ob.store(bt(buf), rb[set], t); },
           [&](int buf) {
#pragma unroll
             for (int s = 0; s < BK / 8; ++s) {
               float a[NB][4], b[NB][4];
#pragma unroll
               for (int i = 0; i < NB; ++i) {
                 OA::frag(a[i], at(buf), wm * 32 * NB + i * 32, s, lane);
                 OB::frag(b[i], bt(buf), wn * 32 * NB + i * 32, s, lane);
               }
#pragma unroll
               for (int k = 0; k < 4; ++k)
#pragma unroll
                 for (int i = 0; i < NB; ++i)
#pragma unroll
                   for (int j = 0; j < NB; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(b[j][k], a[i][k], acc[i][j], 0, 0, 0);
             }
           });
  };
  if constexpr (SPLIT) {
    SplitSeen seen;
    auto at = [&](int buf) { return smem + buf * 3 * OA::PLANE; };
    auto bt = [&](int buf) { return smem + PF * 3 * OA::PLANE + buf * 3 * OB::PLANE; };
    reduce([&](int buf, int set) { oa.store_split(at(buf), ra[set], t, seen); ob.store_split(bt(buf), rb[set], t, seen); },
           [&](int buf) {
#pragma unroll
             for (int s = 0; s < BK / 16; ++s) {
               bf16x8_t a[3][NB], b[3][NB];
#pragma unroll
               for (int pl = 2; pl >= 0; --pl)
#pragma unroll
                 for (int i = 0; i < NB; ++i) {
                   a[pl][i] = OA::frag16(at(buf), pl, wm * 32 * NB + i * 32, s, lane);
                   b[2 - pl][i] = OB::frag16(bt(buf), 2 - pl, wn * 32 * NB + i * 32, s, lane);
                 }
               constexpr int PA[6] = {2, 1, 0, 1, 0, 0}, PB[6] = {0, 1, 2, 0, 1, 0};
#pragma unroll
               for (int q = 0; q < 6; ++q)
#pragma unroll
                 for (int i = 0; i < NB; ++i)
#pragma unroll
                   for (int j = 0; j < NB; ++j) {
                     f32x16_t& c = q < 5 ? low[i][j] : acc[i][j];
                     c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(b[PB[q]][j], a[PA[q]][i], c, 0, 0, 0);
                   }
             }
           });
#pragma unroll
    for (int i = 0; i < NB; ++i)
#pragma unroll
      for (int j = 0; j < NB; ++j)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[i][j][v] += low[i][j][v];
    if (__syncthreads_or(seen.bad())) exact_loop();
  } else {
    exact_loop();
  }

  // ---- epilogue: 64 rows at a time through LDS, 16-byte pieces of whole row segments out ----
  const bool part = p.splits > 1;
  float* Cb = part ? p.partial + ((int64_t)split * (gridDim.z / p.splits) + g) * (int64_t)p.M * p.N
                   : reinterpret_cast<float*>(p.C) + g0 * p.c_g0 + g1 * p.c_g1;
  const int64_t c_ld = part ? p.N : p.c_ld;
  const float* bias = p.bias && !part ? reinterpret_cast<const float*>(p.bias) + g0 * p.bias_g0 + g1 * p.bias_g1 : nullptr;
  const int act = part ? HFTA_ACT_NONE : p.act;
  float* st = reinterpret_cast<float*>(smem);
  constexpr int SP = T + 4;                                // staging pitch, floats
  const int ml = lane & 31, nq = (lane >> 5) * 4;
#pragma unroll
  for (int pass = 0; pass < NB; ++pass) {
    if (NB == 1 || wm == pass) {
#pragma unroll
      for (int i = 0; i < NB; ++i) {
        const int rl = NB == 1 ? wm * 32 + ml : i * 32 + ml;
        const int m = m0 + pass * 64 + rl;
        float bm = 0.f;
        if (bias && p.bias_mode == 1 && m < p.M) bm = bias[m];
#pragma unroll
        for (int j = 0; j < NB; ++j)
#pragma unroll
          for (int q = 0; q < 4; ++q)
            *reinterpret_cast<float4*>(st + rl * SP + wn * 32 * NB + j * 32 + 8 * q + nq) =
                make_float4(acc[i][j][4 * q] + bm, acc[i][j][4 * q + 1] + bm, acc[i][j][4 * q + 2] + bm, acc[i][j][4 * q + 3] + bm);
      }
    }
    __syncthreads();
    if constexpr (HITS) {
      // A wavefront takes a quarter of the tile's columns, a lane a row: no two touch one element, and a column's hits are
      // added in their order.
      static_assert(NB == 2, "64 rows, four quarters of 32 columns");
      const int* off = p.hit_off + (int64_t)g * (p.tiles_n + 1) + tile_n;
      const int h1 = off[1], m = m0 + pass * 64 + lane;
      const uint32_t* key = p.hit_key + (int64_t)g * p.hit_co;
      const float* val = p.hit_val + (int64_t)g * p.hit_co;
      const float* W = p.hit_w + (int64_t)g0 * p.hit_co * p.M + min(m, p.M - 1);
      constexpr int U = 8;                                 // rows of W in flight
      for (int h0 = off[0]; h0 < h1; h0 += 64) {
        const uint32_t kl = h0 + lane < h1 ? key[h0 + lane] : 0xffffffffu;
        const float vl = h0 + lane < h1 ? val[h0 + lane] : 0.f;
        unsigned long long todo = __ballot((int)((kl >> 10) - (uint32_t)n0) >> 5 == wave);
        while (todo) {
          uint32_t ku[U];
          float vu[U], wu[U];
          const int cnt = min((int)__builtin_popcountll(todo), U);
#pragma unroll
          for (int u = 0; u < U; ++u) {
            const int i = todo ? __builtin_ctzll(todo) : 0;
            todo &= todo - 1;
            ku[u] = (uint32_t)__builtin_amdgcn_readlane((int)kl, i);
            vu[u] = __uint_as_float((uint32_t)__builtin_amdgcn_readlane((int)__float_as_uint(vl), i));
          }
#pragma unroll
          for (int u = 0; u < U; ++u) wu[u] = u < cnt ? W[(int64_t)(ku[u] & 1023u) * p.M] : 0.f;
#pragma unroll
          for (int u = 0; u < U; ++u)
            if (u < cnt) {
              float* d = st + lane * SP + (int)((ku[u] >> 10) - (uint32_t)n0);
              *d = fmaf(vu[u], wu[u], *d);
            }
        }
      }
      __syncthreads();
    }
    constexpr int PPR = T / 4, RPI = GEMM_THREADS / PPR;   // pieces per row, rows per iteration
    const int c = t % PPR, n = n0 + c * 4;
    float cb[4] = {0.f, 0.f, 0.f, 0.f};
    if (bias && p.bias_mode == 2) {
#pragma unroll
      for (int e = 0; e < 4; ++e) cb[e] = n + e < p.N ? bias[n + e] : 0.f;
    }
#pragma unroll 4
    for (int it = 0; it < (POOL && !p.C ? 0 : 64 / RPI); ++it) {
      const int rl = t / PPR + it * RPI, m = m0 + pass * 64 + rl;
      const float4 v = *reinterpret_cast<const float4*>(st + rl * SP + c * 4);
      float e[4] = {v.x + cb[0], v.y + cb[1], v.z + cb[2], v.w + cb[3]};
      if (act != HFTA_ACT_NONE) {
#pragma unroll
        for (int k = 0; k < 4; ++k) e[k] = apply_act(e[k], act, p.slope);
      }
      if (m >= p.M) continue;
      if (n + 4 <= p.N && (part || p.c_seg <= 0)) {
        *reinterpret_cast<pf_u32x4_a4*>(Cb + (int64_t)m * c_ld + n) =
            pf_u32x4_a4{__float_as_uint(e[0]), __float_as_uint(e[1]), __float_as_uint(e[2]), __float_as_uint(e[3])};
      } else {
#pragma unroll
        for (int k = 0; k < 4; ++k)
          if (n + k < p.N) Cb[(int64_t)m * c_ld + (part ? (int64_t)(n + k) : col_offset(n + k, p.c_seg, p.c_seg_stride))] = e[k];
      }
    }
    if constexpr (POOL) {
      constexpr int CW = T / 4;                            // columns per thread
      const int rl = t >> 2, c0 = (t & 3) * CW, m = m0 + pass * 64 + rl;
      const int cnt = min(max(p.N - n0 - c0, 0), CW), all = min(p.N - n0, T);
      const float sgn = m < p.M && p.pool_gamma[(int64_t)g0 * p.M + m] < 0.f ? -1.f : 1.f;
      const float* row = st + rl * SP + c0;
      float v[CW];                                         // the thread's columns, once
#pragma unroll
      for (int c = 0; c < CW; c += 4) {
        const float4 q = *reinterpret_cast<const float4*>(row + c);
        v[c] = q.x; v[c + 1] = q.y; v[c + 2] = q.z; v[c + 3] = q.w;
      }
      const bool edge = n0 + T > p.N;                      // the row's last tile: columns past the end do not take part
      float s4[4] = {0.f, 0.f, 0.f, 0.f}, best = -INFINITY;
#pragma unroll
      for (int c = 0; c < CW; ++c) s4[c & 3] += !edge || c < cnt ? v[c] : 0.f;
      float sum = (s4[0] + s4[1]) + (s4[2] + s4[3]);
      sum += __shfl_xor(sum, 1, 64);
      sum += __shfl_xor(sum, 2, 64);
      const float mean = sum / (float)all;
#pragma unroll
      for (int k = 0; k < 4; ++k) s4[k] = 0.f;
#pragma unroll
      for (int c = 0; c < CW; ++c) {
        const float d = !edge || c < cnt ? v[c] - mean : 0.f;
        s4[c & 3] = fmaf(d, d, s4[c & 3]);
      }
      float sq = (s4[0] + s4[1]) + (s4[2] + s4[3]);
      sq += __shfl_xor(sq, 1, 64);
      sq += __shfl_xor(sq, 2, 64);
      // the maximum, then the first column that holds it (walked downwards)
#pragma unroll
      for (int c = 0; c < CW; ++c) {
        v[c] = !edge || c < cnt ? v[c] * sgn : -INFINITY;
        best = fmaxf(best, v[c]);
      }
      int at = 0;
#pragma unroll
      for (int c = CW - 1; c >= 0; --c) at = v[c] == best ? c : at;
      at += n0 + c0;
#pragma unroll
      for (int o = 1; o < 4; o <<= 1) {
        const float ob = __shfl_xor(best, o, 64);
        const int oa = __shfl_xor(at, o, 64);
        if (ob > best || (ob == best && oa < at)) { best = ob; at = oa; }
      }
      if ((t & 3) == 0 && m < p.M)
        p.pool_part[((int64_t)g * p.tiles_n + tile_n) * p.M + m] = make_float4(sum, sq, best, __int_as_float(at));
    }
    if (pass + 1 < NB) __syncthreads();
  }
}

template <int NB, int VEC, bool SPLIT>
int f32_layout(const GemmDesc& d, const GemmArgs& a, dim3 grid, hipStream_t st) {
  if constexpr (SPLIT && NB == 2) {
    if (a.pool_part) {
      hipLaunchKernelGGL((gemm_f32_kernel<true, false, NB, VEC, true, true>), grid, dim3(GEMM_THREADS), 0, st, a);
      const int rc = launch_status();
      if (rc == HFTA_OK) *d.pool_cols = 64 * NB;
      return rc;
    }
    if (d.hit_key) {
      hipLaunchKernelGGL((gemm_f32_kernel<true, false, NB, VEC, true, false, true>), grid, dim3(GEMM_THREADS), 0, st, a);
      return launch_status();
    }
  }
  if (d.a_kc && !d.b_kc) hipLaunchKernelGGL((gemm_f32_kernel<true, false, NB, VEC, SPLIT>), grid, dim3(GEMM_THREADS), 0, st, a);
  else if (d.a_kc && d.b_kc) hipLaunchKernelGGL((gemm_f32_kernel<true, true, NB, VEC, SPLIT>), grid, dim3(GEMM_THREADS), 0, st, a);
  else if (!d.a_kc && !d.b_kc) hipLaunchKernelGGL((gemm_f32_kernel<false, false, NB, VEC, SPLIT>), grid, dim3(GEMM_THREADS), 0, st, a);
  else return HFTA_EUNSUPPORTED;
  return launch_status();
}

}  // namespace

// whether M x N outputs of G groups are taken in 128x128 tiles
bool gemm_f32_big_tiles(int M, int N, int64_t G) {
  return (int64_t)((M + 127) / 128) * ((N + 127) / 128) * G >= F32_SMALL_TILES && M > 64 && N > 64;
}

// HFTA_EUNSUPPORTED: an operand slice does not fit a buffer descriptor (nothing has been launched).
int gemm_f32_launch(const GemmDesc& d, const GemmArgs& base, hipStream_t st) {
  GemmArgs a = base;
  const int64_t a_ext = ((d.a_kc ? (int64_t)(d.M - 1) * d.a_ld + d.K : (int64_t)(d.K - 1) * d.a_ld + d.M)) * 4;
  const int64_t b_ext = ((d.b_kc ? (int64_t)(d.N - 1) * d.b_ld + d.K : (int64_t)(d.K - 1) * d.b_ld + d.N)) * 4;
  if (a_ext >= (int64_t)1 << 31 || b_ext >= (int64_t)1 << 31 || d.a_ld <= 0 || d.b_ld <= 0) return HFTA_EUNSUPPORTED;
  a.a_extent = (uint32_t)a_ext;
  a.b_extent = (uint32_t)b_ext;
  const int64_t G = (int64_t)d.G0 * d.G1;
  const bool small = !gemm_f32_big_tiles(d.M, d.N, G * a.splits);
  const int T = small ? 64 : 128;
  a.tiles_m = (d.M + T - 1) / T;
  a.tiles_n = (d.N + T - 1) / T;
  const bool vec = d.K >= 4 && (d.a_kc || d.M >= 4) && (d.b_kc || d.N >= 4);
  const bool whole = vec && (d.a_kc ? d.K : d.M) % 4 == 0 && (d.b_kc ? d.K : d.N) % 4 == 0;   // no piece straddles a row's end
  // (64x64 tiles: a pass over so small an output costs less than the epilogue, 2 x 4 x 256 points 188.5 us a step, 191.8 with)
  if (d.pool_part && d.pool_cols && vec && d.a_kc && !d.b_kc && a.splits == 1 && d.act == HFTA_ACT_NONE && d.c_seg <= 0 && !small) {
    a.pool_part = d.pool_part;
    a.pool_gamma = d.pool_gamma;
  }
  // The fp32 instruction, with its shorter k-tiles, takes
  //   single elements, loaded one by one whether they exist or not: forward of 3 -> 64 channels on 4 x 32 x 2500 points 25 us, 36
  //     with 32-k tiles;
  //   small tiles under at most 64 k a workgroup, which are bound by their tensors and better off with its four workgroups per
  //     compute unit than with the split's three (64 -> 64 on 4 x 32 x 2500: 45 us, split 53), and under up to 136 k where pieces
  //     straddle rows' ends (weight gradient of 64 -> 64 on 1 x 8 x 333 10.4 us, split 11.6, on 1 x 2 x 257 9.4, 10.0; forward of
  //     70 -> 90 on 3 x 13 x 1023 15.9, 17.6);
  //   rows (of a reduction over samples: their parts) that leave half of their last 32-k tile empty, while that tile is the
  //     first, in small tiles also the second (forward of 8 -> 128 and 16 -> 256 on 4 x 32 x 2500 37 us, split 46, and 86, 106;
  //     weight gradient of 64 -> 128 on 2 x 16 x 12, 4 x 64 x 7 and 2 x 64 x 48 points 9.9, 11.6, 10.5, 14.3 and 11.1, 12.0).
  const int64_t k_wg = ((int64_t)d.K * d.S + a.splits - 1) / a.splits;
  const bool exact = !vec || (small && k_wg <= (whole ? 64 : 136)) ||
                     (d.K <= (small ? 48 : 16) && (d.K - 1) % 32 < 16 && !a.pool_part);
  // what only the 128x128 tiles of the split product do
  if (d.pool_part && !d.C && (!a.pool_part || exact)) return HFTA_EUNSUPPORTED;
  if (d.hit_key && (small || exact || a.splits != 1 || !d.a_kc || d.b_kc || d.c_seg > 0)) return HFTA_EUNSUPPORTED;
  const int BK = f32_bk(!exact);
  a.tiles_per_seg = (d.K + BK - 1) / BK;
  a.total_tiles = d.S * a.tiles_per_seg;
  dim3 grid((unsigned)(a.tiles_m * a.tiles_n), 1, (unsigned)(G * a.splits));
  if (exact) {
    if (small) return whole ? f32_layout<1, 2, false>(d, a, grid, st) : vec ? f32_layout<1, 1, false>(d, a, grid, st) : f32_layout<1, 0, false>(d, a, grid, st);
    return whole ? f32_layout<2, 2, false>(d, a, grid, st) : vec ? f32_layout<2, 1, false>(d, a, grid, st) : f32_layout<2, 0, false>(d, a, grid, st);
  }
  if (small) return whole ? f32_layout<1, 2, true>(d, a, grid, st) : f32_layout<1, 1, true>(d, a, grid, st);
  return whole ? f32_layout<2, 2, true>(d, a, grid, st) : f32_layout<2, 1, true>(d, a, grid, st);
}

}  // namespace hfta
