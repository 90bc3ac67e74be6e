// Warm-start network kernels for gfx950.
//
// The network (a 3D convolutional encoder-decoder, see unet_host.hpp) maps the
// solute potential of each solvent site to an initial short-range direct
// correlation; the paper itself starts every solve at t = f.  Activations are
// BF16, channels last ([voxel][channel], channel count a multiple of 8), so 8
// channels of one voxel are one 16-byte load.  The 3x3x3 convolutions are
// implicit GEMMs on the matrix cores:
//   v_mfma_f32_16x16x32_bf16:  D[16x16] += A[16x32] B[32x16], FP32 accumulate,
//   A = packed weights (rows = output channels), B = input voxels (columns),
//   K = (tap, input channel) with 8 consecutive channels per lane.
// Lane l supplies row/column (l & 15) and the K slice 8 (l >> 4) .. +7 of its
// operand; it receives D rows 4 (l >> 4) .. +3 of column (l & 15), i.e. four
// consecutive output channels of one voxel (one 8-byte BF16 store).
// Weight gradients use the same instruction on tiles transposed through LDS.
#pragma once

#include "common.hpp"

namespace rism {
namespace net {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));

constexpr int kConvThreads = 256;   // 4 waves

// FP32 -> BF16 with round-to-nearest-even (NaN stays NaN), one conversion
// instruction for two values; BF16 -> FP32 exact.
__device__ __forceinline__ uint32_t f2bf2(float lo, float hi) {
  typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
  return __builtin_bit_cast(uint32_t, bf16x2{(__bf16)lo, (__bf16)hi});
}
__device__ __forceinline__ uint16_t f2bf(float f) { return __builtin_bit_cast(uint16_t, (__bf16)f); }
__device__ __forceinline__ float bf2f(uint16_t h) { return __uint_as_float((uint32_t)h << 16); }

__device__ __forceinline__ bf16x8 ld8(const uint16_t* p) {   // 16-byte aligned
  return __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4*>(p));
}
__device__ __forceinline__ bf16x8 zero8() {
  const u32x4 z = {0u, 0u, 0u, 0u};
  return __builtin_bit_cast(bf16x8, z);
}

// Input of a convolution: channels [0, ca) from tensor a (on the output grid,
// or on the half grid and read through nearest-neighbour upsampling when
// up_a), channels [ca, ca + cb) from tensor b (the skip branch).
struct ConvIn {
  const uint16_t* a;
  const uint16_t* b;
  int ca, cb, up_a;
};

// 8 channels (group cg) of voxel (z, y, x) of the virtual input; zero outside.
__device__ __forceinline__ bf16x8 load_in(const ConvIn& in, int cg, int z, int y, int x, int nz,
                                          int ny, int nx) {
  if ((unsigned)z >= (unsigned)nz || (unsigned)y >= (unsigned)ny || (unsigned)x >= (unsigned)nx)
    return zero8();
  const int c = cg * 8;
  if (c < in.ca) {
    const size_t v = in.up_a ? ((size_t)(z >> 1) * (ny >> 1) + (y >> 1)) * (nx >> 1) + (x >> 1)
                             : ((size_t)z * ny + y) * nx + x;
    return ld8(in.a + v * in.ca + c);
  }
  return ld8(in.b + (((size_t)z * ny + y) * nx + x) * in.cb + (c - in.ca));
}

enum ConvEpilogue {
  EPI_BF16_LEAKY = 0,   // + bias, leaky, BF16 channels last [N][cout_pad]
  EPI_F32_SITE = 1,     // + bias, FP32 site-major [cout][N] (channels < cout)
  EPI_BF16_DLEAKY = 2,  // times leaky'(.) of the activation act, BF16 channels last [N][cout]
  EPI_F32_SPLIT = 3,    // raw FP32 channels last: [0, split) to yf, the others to yf2
};

struct ConvArgs {
  ConvIn in;
  const uint16_t* w;    // packed for cout_pad x (ca + cb) channels (k_pack_weights)
  const float* bias;    // [cout] (EPI 0, 1)
  uint16_t* yb;         // EPI_BF16_LEAKY / EPI_BF16_DLEAKY output
  float* yf;            // EPI_F32_SITE / EPI_F32_SPLIT output
  float* yf2;           // EPI_F32_SPLIT: the skip channels
  const uint16_t* act;  // EPI_BF16_DLEAKY: the activation, BF16 channels last [N][cout]
  int split;            // EPI_F32_SPLIT: channels of yf (a multiple of 4)
  int cout, cout_pad;
  int nz, ny, nx;
  float slope;
};

// d * leaky'(.) of four channels as BF16, the derivative read from the sign of the
// BF16 activation y.
__device__ __forceinline__ u32x2 leaky_bwd4(u32x2 y, f32x4 d, float slope) {
  float h[4];
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const uint16_t a = (uint16_t)(e & 1 ? y[e >> 1] >> 16 : y[e >> 1] & 0xffffu);
    h[e] = bf2f(a) > 0.0f ? d[e] : slope * d[e];
  }
  return u32x2{f2bf2(h[0], h[1]), f2bf2(h[2], h[3])};
}

// Bias of output channels c0 .. c0 + 3 (zero beyond the real ones).
template <int EPI>
__device__ __forceinline__ f32x4 conv_bias(const ConvArgs& p, int c0) {
  f32x4 b = {0.f, 0.f, 0.f, 0.f};
  if (EPI == EPI_BF16_LEAKY || EPI == EPI_F32_SITE)
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if (c0 + e < p.cout) b[e] = p.bias[c0 + e];
  return b;
}

// Epilogue of one accumulator tile: output channels c0 .. c0 + 3 of voxel v.
template <int EPI>
__device__ __forceinline__ void conv_store(const ConvArgs& p, int N, size_t v, int c0, f32x4 bias,
                                           f32x4 r) {
  if (EPI == EPI_BF16_LEAKY) {
    float h[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const float val = r[e] + bias[e];
      h[e] = val > 0.0f ? val : p.slope * val;
    }
    *reinterpret_cast<u32x2*>(p.yb + v * p.cout_pad + c0) =
        u32x2{f2bf2(h[0], h[1]), f2bf2(h[2], h[3])};
  } else if (EPI == EPI_F32_SITE) {
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if (c0 + e < p.cout) p.yf[(size_t)(c0 + e) * N + v] = r[e] + bias[e];
  } else if (EPI == EPI_BF16_DLEAKY) {
    const u32x2 y = *reinterpret_cast<const u32x2*>(p.act + v * p.cout + c0);
    *reinterpret_cast<u32x2*>(p.yb + v * p.cout + c0) = leaky_bwd4(y, r, p.slope);
  } else {
    float* o = c0 < p.split ? p.yf + v * p.split + c0
                            : p.yf2 + v * (p.cout - p.split) + (c0 - p.split);
    *reinterpret_cast<f32x4*>(o) = r;
  }
}

// Convolutions with 8 * CG input channels on a halo-tiled grid: a workgroup
// computes MT tiles of 16 output channels (from MT blockIdx.y) of a 16 x TY x 4
// voxel tile (TY = 8; 2 on small grids, for more workgroups).  It stages the
// tile's input with a one-voxel halo (18 x (TY + 2) x 6 voxels) in LDS, CGC channel
// groups at a time (CG / CGC chunks), and every tap's operand is read from there
// instead of from the cache hierarchy.  LDS layout [hz][hy][cg][hx] (16-byte
// units): the 16 voxels of one operand are consecutive units, conflict-free.  Wave
// w owns the z-slice z0 + w: its TY rows y0 .. y0 + TY - 1 of 16 voxels are its TY
// accumulator tiles per output tile.  Within a chunk the K steps take (tap, channel
// group) pairs in tap-major order, four per matrix instruction: lane group g
// supplies pair q0 + g (its 8 channels), the weights are the A operand (rows =
// output channels), the voxels the B operand (columns).  The weights are packed in
// this order (k_pack_weights), so a step's A operand is one coalesced load at a
// fixed offset, and the halo offsets of the steps are formed once.
//
// Bound by the LDS reads: an operand of 1 KB feeds MT instructions of 16 cycles
// on each of four SIMDs, so one output tile can reach half of the matrix rate and
// two all of it; below that by staging, whose index arithmetic and latency are
// kept small (one row of the halo per thread group, loads in batches, two or three
// waves a SIMD).  Before and after, each layer repeated alone, at 128^3: 16 -> 16
// channels 78 -> 52 us, 48 -> 16 215 -> 121 us (0.29 of the BF16 peak), and at 64^3
// 96 -> 32 136 -> 45 us (0.39).  A trace of the whole network has a tenth more.
constexpr int kTileX = 16, kTileZ = 4;
constexpr int kHaloX = kTileX + 2, kHaloZ = kTileZ + 2;

// K steps of a chunk of CGC channel groups
__host__ __device__ constexpr int conv_steps(int cgc) { return (27 * cgc + 3) / 4; }
// channel groups a chunk takes out of cg: the largest of 4, 3, 2, 1 that divides it
__host__ __device__ constexpr int conv_chunk(int cg) {
  return cg % 4 == 0 ? 4 : cg % 3 == 0 ? 3 : cg % 2 == 0 ? 2 : 1;
}
// elements of the packed weights of cout (a multiple of 16) x cin (of 8) channels
__host__ __device__ constexpr size_t conv_packed(int cout, int cin) {
  return (size_t)(cout / 16) * (cin / 8 / conv_chunk(cin / 8)) * conv_steps(conv_chunk(cin / 8)) * 512;
}

// staging loads a thread has in flight, out of n: in as few batches of at most 9
__host__ __device__ constexpr int conv_batch(int n) { return (n + (n + 8) / 9 - 1) / ((n + 8) / 9); }

// staged units of a chunk
__host__ __device__ constexpr int conv_halo(int cgc, int ty) {
  return kHaloZ * (ty + 2) * cgc * kHaloX;
}
// waves a SIMD that the kernel asks for: three, but two where the LDS holds no third
// workgroup, and for three groups and two output tiles, whose 21 offsets and 16
// accumulator tiles spill in the registers of three (24 -> 32 channels, 128^3:
// forward of the network 668 us with three, 630 with two)
__host__ __device__ constexpr int conv_waves(int cgc, int ty, int mt) {
  return 3 * conv_halo(cgc, ty) * 16 > 160 * 1024 || (ty == 8 && cgc == 3 && mt == 2) ? 2 : 3;
}

template <int EPI, int CGC, int TY, int MT>
__global__ __launch_bounds__(kConvThreads) __attribute__((amdgpu_waves_per_eu(conv_waves(CGC, TY, MT))))
void k_conv3(ConvArgs p) {
  constexpr int kTileY = TY, kHaloY = TY + 2, NQ = 27 * CGC, NS = conv_steps(CGC);
  __shared__ __align__(16) u32x4 halo[conv_halo(CGC, TY)];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int j = lane & 15, g = lane >> 4;
  const int N = p.nz * p.ny * p.nx;
  const int CG = (p.in.ca + p.in.cb) >> 3;   // a multiple of CGC
  const int tiles_x = (p.nx + kTileX - 1) / kTileX, tiles_y = (p.ny + kTileY - 1) / kTileY;
  int b = (int)blockIdx.x;
  const int x0 = (b % tiles_x) * kTileX;
  b /= tiles_x;
  const int y0 = (b % tiles_y) * kTileY;
  const int z0 = (b / tiles_y) * kTileZ;
  f32x4 acc[MT][kTileY];
#pragma unroll
  for (int m = 0; m < MT; ++m)
#pragma unroll
    for (int t = 0; t < kTileY; ++t) acc[m][t] = f32x4{0.f, 0.f, 0.f, 0.f};
  int off[NS];   // halo unit of row 0 of this lane's pair in each step
#pragma unroll
  for (int s = 0; s < NS; ++s) {
    const int q = 4 * s + g < NQ ? 4 * s + g : 0;
    const int tap = q / CGC, cg = q - tap * CGC;
    off[s] = (((wave + tap / 9) * kHaloY + tap / 3 % 3) * CGC + cg) * kHaloX + j + tap % 3;
  }
  const int chunks = CG / CGC;
  const u32x4* aw = reinterpret_cast<const u32x4*>(p.w) +
                    (size_t)blockIdx.y * MT * chunks * NS * 64 + lane;
  for (int c0 = 0; c0 < CG; c0 += CGC, aw += NS * 64) {
    if (c0 > 0) __syncthreads();   // the previous chunk's operands are read
    // stage: a thread keeps its x and channel group and takes every RP-th row (hz,
    // hy); x is the fastest lane index, so the LDS stores are conflict-free.  A
    // batch's loads are all in flight before its first store.
    constexpr int RT = kHaloX * CGC, RP = kConvThreads / RT, ROWS = kHaloZ * kHaloY;
    constexpr int ALL = (ROWS + RP - 1) / RP, B = conv_batch(ALL);
    const int rr = threadIdx.x / RT, l = threadIdx.x - rr * RT;
    const int cg = l / kHaloX, hx = l - cg * kHaloX, x = x0 + hx - 1;
    const int c = (c0 + cg) * 8;
    const bool skip = c >= p.in.ca;
    const int up = skip ? 0 : p.in.up_a, C = skip ? p.in.cb : p.in.ca;
    const int ny = p.ny >> up, nx = p.nx >> up;
    const uint16_t* src = (skip ? p.in.b + (c - p.in.ca) : p.in.a + c) + (size_t)(x >> up) * C;
    const bool in_x = rr < RP && (unsigned)x < (unsigned)p.nx;
    for (int i0 = 0; i0 < ALL; i0 += B) {
      u32x4 v[B];
#pragma unroll
      for (int i = 0; i < B; ++i) {
        const int row = rr + (i0 + i) * RP, hz = row / kHaloY, hy = row - hz * kHaloY;
        const int z = z0 + hz - 1, y = y0 + hy - 1;
        v[i] = u32x4{0u, 0u, 0u, 0u};
        if (in_x && (unsigned)z < (unsigned)p.nz && (unsigned)y < (unsigned)p.ny)
          v[i] = *reinterpret_cast<const u32x4*>(
              src + (size_t)(unsigned)((z >> up) * ny + (y >> up)) * (unsigned)(nx * C));
      }
#pragma unroll
      for (int i = 0; i < B; ++i) {
        const int row = rr + (i0 + i) * RP;
        if (rr < RP && row < ROWS) halo[(row * CGC + cg) * kHaloX + hx] = v[i];
      }
    }
    __syncthreads();
#pragma unroll
    for (int s = 0; s < NS; ++s) {
      bf16x8 a[MT];
#pragma unroll
      for (int m = 0; m < MT; ++m)
        a[m] = __builtin_bit_cast(bf16x8, aw[(size_t)(m * chunks) * NS * 64 + s * 64]);
#pragma unroll
      for (int t = 0; t < kTileY; ++t) {
        u32x4 v = halo[off[s] + t * CGC * kHaloX];
        if (4 * s + 4 > NQ && 4 * s + g >= NQ) v = u32x4{0u, 0u, 0u, 0u};   // beyond the last pair
        const bf16x8 x = __builtin_bit_cast(bf16x8, v);
#pragma unroll
        for (int m = 0; m < MT; ++m)
          acc[m][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[m], x, acc[m][t], 0, 0, 0);
      }
    }
  }
  const int x = x0 + j, z = z0 + wave;
  if (x >= p.nx || z >= p.nz) return;
#pragma unroll
  for (int m = 0; m < MT; ++m) {
    const int ch = ((int)blockIdx.y * MT + m) * 16 + 4 * g;
    const f32x4 bias = conv_bias<EPI>(p, ch);
#pragma unroll
    for (int t = 0; t < kTileY; ++t)
      if (y0 + t < p.ny)
        conv_store<EPI>(p, N, ((size_t)z * p.ny + y0 + t) * p.nx + x, ch, bias, acc[m][t]);
  }
}

// Weight and bias gradients, dW[o][tap][i] = sum_v dy[v][o] x[v + off(tap)][i] and
// db[o] = sum_v dy[v][o].  A workgroup takes one 16-channel tile of inputs and OT
// tiles of outputs (blockIdx.y) over a run of 16 x 8 x 4 voxel tiles, and does all
// 27 taps on each tile it stages: the tiles go through LDS transposed, eight
// voxels in y to a 16-byte operand.
//   dy: [o][z][x][8 y];  x with its halo: [i][hz][hx][10 y, padded to 12].
// One matrix instruction takes 4 voxels in x (lane group g) x 8 in y.  Its dy
// operand serves the 27 taps; the x row of (dz, dx) holds the operands of the
// three dy, the outer two as they lie and the middle one shifted by one element.
// The 27 accumulator tiles and one of the bias (against a column of ones) stay in
// registers.  OT waves' worth of output tiles share an x tile; the other waves
// split the K steps, and their sums are added in order at the end.  Each
// workgroup stores its sums in its own slab (laid out as the layer's parameters),
// and k_sum_slabs adds the slabs in a fixed order, so the gradient is
// deterministic.
//
// Bound by the LDS reads (196 bytes a lane per 27 instructions) close to the
// matrix cores, and by staging between them.  Training step at 128^3: 5070 us in
// all layers with every tap restaging its own transposed chunk (and 250 us for the
// bias in a kernel of its own), 730 us now, 0.15 of the BF16 peak.
struct WgradArgs {
  ConvIn in;
  const uint16_t* dy;   // BF16 [N][cout_pad]
  float* dw;            // FP32 slabs [gridDim.x][cout * 27 * cin_real + cout]
  int cin_real;         // real input channels (the packed input may carry zero padding)
  int cout, cout_pad;
  int nz, ny, nx;
  int tiles, per;       // voxel tiles, and how many a workgroup takes
};

constexpr int kWgX = 16, kWgY = 8, kWgZ = 4;            // voxel tile
constexpr int kWgRows = (kWgX + 2) * (kWgZ + 2);        // x rows of a channel
// dwords of a channel in LDS: 6 a row and a pad that makes the pitch 4 (mod 8),
// for conflict-free 8-byte reads of 16 channels; of a dy channel, likewise
constexpr int kWgXPitch = kWgRows * 6 + 4, kWgDyPitch = kWgX * kWgZ * 4 + 4;
constexpr int wgrad_dwords(int OT) { return 16 * kWgXPitch + 16 * OT * kWgDyPitch; }

// Stores channels 8 cg .. + 7 of two voxels that follow each other in y as one
// dword a channel at dst + c * pitch.
__device__ __forceinline__ void store_pair(uint32_t* dst, int pitch, bf16x8 va, bf16x8 vb) {
  const u32x4 a = __builtin_bit_cast(u32x4, va), b = __builtin_bit_cast(u32x4, vb);
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    dst[(2 * e) * pitch] = (a[e] & 0xffffu) | (b[e] << 16);
    dst[(2 * e + 1) * pitch] = (a[e] >> 16) | (b[e] & 0xffff0000u);
  }
}

template <int OT>
__global__ __launch_bounds__(kConvThreads) void k_conv3_wgrad(WgradArgs p) {
  __shared__ __align__(16) uint32_t wsm[wgrad_dwords(OT)];
  uint32_t* xs = wsm;                      // [16][kWgXPitch]
  uint32_t* ds = wsm + 16 * kWgXPitch;     // [16 OT][kWgDyPitch]
  constexpr int WK = 4 / OT;               // waves that share an output tile
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int j = lane & 15, g = lane >> 4;
  const int ot = wave % OT, ks = wave / OT;
  const int cin = p.in.ca + p.in.cb;
  const int cit = (cin + 15) >> 4;
  const int ti = (int)blockIdx.y % cit, o0 = (int)blockIdx.y / cit * OT * 16;
  const int cgi = (cin - ti * 16) >= 16 ? 2 : 1;   // 8-channel groups of this input tile
  const int tx = (p.nx + kWgX - 1) / kWgX, ty = (p.ny + kWgY - 1) / kWgY;
  f32x4 acc[27], accb = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int t = 0; t < 27; ++t) acc[t] = f32x4{0.f, 0.f, 0.f, 0.f};
  const u32x4 one4 = {0x3f803f80u, 0x3f803f80u, 0x3f803f80u, 0x3f803f80u};
  const bf16x8 ones = __builtin_bit_cast(bf16x8, one4);
  const int t_end = min(((int)blockIdx.x + 1) * p.per, p.tiles);
  for (int t = (int)blockIdx.x * p.per; t < t_end; ++t) {
    const int x0 = t % tx * kWgX, y0 = t / tx % ty * kWgY, z0 = t / (tx * ty) * kWgZ;
    __syncthreads();   // the previous tile's operands are read
    // every load of the tile in flight before the first LDS store
    constexpr int ND = kWgX * kWgZ * (kWgY / 2) * 2 * OT / kConvThreads;
    constexpr int NX = (kWgRows * (kWgY / 2 + 1) * 2 + kConvThreads - 1) / kConvThreads;
    bf16x8 vd[ND][2], vx[NX][2];
#pragma unroll
    for (int k = 0; k < ND; ++k) {
      const int it = threadIdx.x + k * kConvThreads;
      const int cg = it % (2 * OT), r = it / (2 * OT);
      const int xx = r % kWgX, yp = r / kWgX % (kWgY / 2), zz = r / (kWgX * (kWgY / 2));
      const int x = x0 + xx, y = y0 + 2 * yp, z = z0 + zz, o = o0 + cg * 8;
      vd[k][0] = vd[k][1] = zero8();
      if (x < p.nx && z < p.nz && o < p.cout_pad) {
        const uint16_t* q = p.dy + (((size_t)z * p.ny + y) * p.nx + x) * p.cout_pad + o;
        if (y < p.ny) vd[k][0] = ld8(q);
        if (y + 1 < p.ny) vd[k][1] = ld8(q + (size_t)p.nx * p.cout_pad);
      }
    }
    // (an 8-channel input tile repeats its group in rows that no result reads)
#pragma unroll
    for (int k = 0; k < NX; ++k) {
      const int it = threadIdx.x + k * kConvThreads;
      const int cg = it % 2 < cgi ? it % 2 : 0, r = it / 2;
      const int hx = r % (kWgX + 2), q = r / (kWgX + 2);
      const int yp = q % (kWgY / 2 + 1), hz = q / (kWgY / 2 + 1);
      const int x = x0 + hx - 1, y = y0 + 2 * yp - 1, z = z0 + hz - 1;
      if (hz < kWgZ + 2) {
        vx[k][0] = load_in(p.in, ti * 2 + cg, z, y, x, p.nz, p.ny, p.nx);
        vx[k][1] = load_in(p.in, ti * 2 + cg, z, y + 1, x, p.nz, p.ny, p.nx);
      }
    }
#pragma unroll
    for (int k = 0; k < ND; ++k) {
      const int it = threadIdx.x + k * kConvThreads;
      const int cg = it % (2 * OT), r = it / (2 * OT);
      const int xx = r % kWgX, yp = r / kWgX % (kWgY / 2), zz = r / (kWgX * (kWgY / 2));
      store_pair(ds + cg * 8 * kWgDyPitch + (zz * kWgX + xx) * 4 + yp, kWgDyPitch, vd[k][0], vd[k][1]);
    }
#pragma unroll
    for (int k = 0; k < NX; ++k) {
      const int it = threadIdx.x + k * kConvThreads;
      const int cg = it % 2, r = it / 2;
      const int hx = r % (kWgX + 2), q = r / (kWgX + 2);
      const int yp = q % (kWgY / 2 + 1), hz = q / (kWgY / 2 + 1);
      if (hz < kWgZ + 2)
        store_pair(xs + cg * 8 * kWgXPitch + (hz * (kWgX + 2) + hx) * 6 + yp, kWgXPitch, vx[k][0],
                   vx[k][1]);
    }
    __syncthreads();
#pragma unroll 1
    for (int c = ks; c < kWgZ * (kWgX / 4); c += WK) {
      const int zz = c / (kWgX / 4), xb = c % (kWgX / 4) * 4 + g;
      const bf16x8 a = __builtin_bit_cast(
          bf16x8, *reinterpret_cast<const u32x4*>(ds + (ot * 16 + j) * kWgDyPitch +
                                                  (zz * kWgX + xb) * 4));
      accb = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, ones, accb, 0, 0, 0);
#pragma unroll
      for (int dz = 0; dz < 3; ++dz)
#pragma unroll
        for (int dx = 0; dx < 3; ++dx) {
          const uint32_t* row = xs + j * kWgXPitch + ((zz + dz) * (kWgX + 2) + xb + dx) * 6;
          const u32x2 lo = *reinterpret_cast<const u32x2*>(row);
          const u32x2 mi = *reinterpret_cast<const u32x2*>(row + 2);
          const uint32_t hi = row[4];
          const u32x4 b0 = {lo[0], lo[1], mi[0], mi[1]};
          const u32x4 b1 = {__builtin_amdgcn_alignbit(lo[1], lo[0], 16),
                            __builtin_amdgcn_alignbit(mi[0], lo[1], 16),
                            __builtin_amdgcn_alignbit(mi[1], mi[0], 16),
                            __builtin_amdgcn_alignbit(hi, mi[1], 16)};
          const u32x4 b2 = {lo[1], mi[0], mi[1], hi};
          f32x4* q = acc + dz * 9 + dx;
          q[0] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, __builtin_bit_cast(bf16x8, b0), q[0], 0,
                                                         0, 0);
          q[3] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, __builtin_bit_cast(bf16x8, b1), q[3], 0,
                                                         0, 0);
          q[6] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, __builtin_bit_cast(bf16x8, b2), q[6], 0,
                                                         0, 0);
        }
    }
  }
  // the K splits of an output tile, added in order
  f32x4* part = reinterpret_cast<f32x4*>(wsm);   // [OT][28][64]
  static_assert(wgrad_dwords(OT) >= OT * 28 * 64 * 4, "scratch of the sums");
#pragma unroll 1
  for (int k = 1; k < WK; ++k) {
    __syncthreads();
    if (ks == k) {
#pragma unroll
      for (int t = 0; t < 27; ++t) part[(ot * 28 + t) * 64 + lane] = acc[t];
      part[(ot * 28 + 27) * 64 + lane] = accb;
    }
    __syncthreads();
    if (ks == 0) {
#pragma unroll
      for (int t = 0; t < 27; ++t) acc[t] += part[(ot * 28 + t) * 64 + lane];
      accb += part[(ot * 28 + 27) * 64 + lane];
    }
  }
  if (ks != 0) return;
  const size_t nw = (size_t)p.cout * 27 * p.cin_real;
  float* slab = p.dw + (size_t)blockIdx.x * (nw + p.cout);
  const int i = ti * 16 + j;
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const int o = o0 + ot * 16 + 4 * g + e;
    if (o >= p.cout) continue;
    if (i < p.cin_real) {
#pragma unroll
      for (int t = 0; t < 27; ++t) slab[((size_t)o * 27 + t) * p.cin_real + i] = acc[t][e];
    }
    if (ti == 0 && j == 0) slab[nw + o] = accb[e];
  }
}

// dst[e] = sum_b part[b][e] over the n_slab slabs of n elements.  Thread row r of
// blockDim.y adds slabs r, r + blockDim.y, ... in order, and the rows are added in
// order (a fixed order: the gradients are deterministic).
__global__ __launch_bounds__(1024) void k_sum_slabs(const float* __restrict__ part, int n_slab,
                                                    size_t n, float* __restrict__ dst) {
  __shared__ float red[16][64];
  const size_t e = (size_t)blockIdx.x * 64 + threadIdx.x;
  float t = 0.0f;
  if (e < n) {
    int b = threadIdx.y;
    const int Y = blockDim.y;
    for (; b + 7 * Y < n_slab; b += 8 * Y) {   // 8 loads in flight
      float v[8];
#pragma unroll
      for (int k = 0; k < 8; ++k) v[k] = part[(size_t)(b + k * Y) * n + e];
#pragma unroll
      for (int k = 0; k < 8; ++k) t += v[k];
    }
    for (; b < n_slab; b += Y) t += part[(size_t)b * n + e];
  }
  red[threadIdx.y][threadIdx.x] = t;
  __syncthreads();
  if (threadIdx.y == 0 && e < n) {
    for (int r = 1; r < (int)blockDim.y; ++r) t += red[r][threadIdx.x];
    dst[e] = t;
  }
}

// Average over 2x2x2 blocks (BF16 in and out, FP32 sums); one thread per
// coarse voxel and 8-channel group.
__global__ void k_pool2(const uint16_t* __restrict__ in, uint16_t* __restrict__ out, int nz,
                        int ny, int nx, int C) {
  const int hz = nz >> 1, hy = ny >> 1, hx = nx >> 1;
  const int cg = C >> 3;
  const size_t id = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (id >= (size_t)hz * hy * hx * cg) return;
  const int g = (int)(id % cg);
  const size_t cv = id / cg;
  const int x = (int)(cv % hx), y = (int)((cv / hx) % hy), z = (int)(cv / ((size_t)hx * hy));
  float s[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  for (int d = 0; d < 8; ++d) {
    const size_t v = ((size_t)(2 * z + (d >> 2)) * ny + 2 * y + ((d >> 1) & 1)) * nx + 2 * x + (d & 1);
    const u32x4 w4 = *reinterpret_cast<const u32x4*>(in + v * C + g * 8);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      s[2 * e] += bf2f((uint16_t)(w4[e] & 0xffffu));
      s[2 * e + 1] += bf2f((uint16_t)(w4[e] >> 16));
    }
  }
  u32x4 o;
#pragma unroll
  for (int e = 0; e < 4; ++e)
    o[e] = f2bf2(0.125f * s[2 * e], 0.125f * s[2 * e + 1]);
  *reinterpret_cast<u32x4*>(out + cv * C + g * 8) = o;
}

// The gradient at a pooled encoder output, (skip + coarse[v / 2] / 8) leaky'(y) in
// BF16: the skip branch's FP32 part, the adjoint of the 2x2x2 average, and the
// activation's derivative in one pass.  Four channels a thread.
__global__ void k_pool2_bwd_leaky(const float* __restrict__ coarse, const float* __restrict__ skip,
                                  const uint16_t* __restrict__ y, uint16_t* __restrict__ out,
                                  int nz, int ny, int nx, int C, float slope) {
  const size_t id = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int c4 = C >> 2;
  if (id >= (size_t)nz * ny * nx * c4) return;
  const unsigned v = (unsigned)(id / c4), row = v / nx, z = row / ny;
  const unsigned x = v - row * nx, yy = row - z * ny;
  const size_t cv = ((size_t)(z >> 1) * (ny >> 1) + (yy >> 1)) * (nx >> 1) + (x >> 1);
  const f32x4 s = reinterpret_cast<const f32x4*>(skip)[id];
  const f32x4 c = reinterpret_cast<const f32x4*>(coarse)[cv * c4 + (id - (size_t)v * c4)];
  reinterpret_cast<u32x2*>(out)[id] =
      leaky_bwd4(reinterpret_cast<const u32x2*>(y)[id], s + 0.125f * c, slope);
}

// The gradient at an upsampled tensor, the sum of the eight fine voxels of block u
// of dx (C channels) times leaky'(y), in BF16.  Four channels a thread.
__global__ void k_up2_bwd_leaky(const float* __restrict__ dx, const uint16_t* __restrict__ y,
                                uint16_t* __restrict__ out, int nz, int ny, int nx, int C,
                                float slope) {
  const int hz = nz >> 1, hy = ny >> 1, hx = nx >> 1, c4 = C >> 2;
  const size_t id = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (id >= (size_t)hz * hy * hx * c4) return;
  const unsigned cv = (unsigned)(id / c4), row = cv / hx, z = row / hy;
  const unsigned x = cv - row * hx, yy = row - z * hy;
  const int g = (int)(id - (size_t)cv * c4);
  f32x4 s = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int d = 0; d < 8; ++d) {
    const size_t v = ((size_t)(2 * z + (d >> 2)) * ny + 2 * yy + ((d >> 1) & 1)) * nx + 2 * x + (d & 1);
    s += reinterpret_cast<const f32x4*>(dx)[v * c4 + g];
  }
  reinterpret_cast<u32x2*>(out)[id] = leaky_bwd4(reinterpret_cast<const u32x2*>(y)[id], s, slope);
}

// Site-major FP32 [C][N] -> BF16 channels last [N][cpad] (zero padding), one voxel
// a thread.
__global__ void k_to_channels_last(const float* __restrict__ in, int C, int cpad, size_t N,
                                   uint16_t* __restrict__ out) {
  const size_t v = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (v >= N) return;
  for (int c0 = 0; c0 < cpad; c0 += 8) {
    u32x4 o;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int c = c0 + 2 * e;
      const float a = c < C ? in[(size_t)c * N + v] : 0.0f;
      const float b = c + 1 < C ? in[(size_t)(c + 1) * N + v] : 0.0f;
      o[e] = f2bf2(a, b);
    }
    *reinterpret_cast<u32x4*>(out + v * cpad + c0) = o;
  }
}

// Mean squared error over C x N values: per-block FP64 partial sums and the
// BF16 gradient 2 (o - t) / (C N) channels last [N][cpad] (zero padding), one
// voxel a thread and step.
__global__ __launch_bounds__(256) void k_mse(const float* __restrict__ out,
                                             const float* __restrict__ target, int C, int cpad,
                                             size_t N, uint16_t* __restrict__ grad,
                                             double* __restrict__ partials) {
  __shared__ double red[4];
  const double scale = 2.0 / ((double)C * (double)N);
  double s = 0.0;
  for (size_t v = (size_t)blockIdx.x * blockDim.x + threadIdx.x; v < N;
       v += (size_t)gridDim.x * blockDim.x) {
    for (int c0 = 0; c0 < cpad; c0 += 8) {
      u32x4 o = {0u, 0u, 0u, 0u};
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        if (c0 + e < C) {
          const size_t i = (size_t)(c0 + e) * N + v;
          const double d = (double)out[i] - (double)target[i];
          s += d * d;
          float gv = (float)(scale * d);
          asm("" : "+v"(gv));   // rounded to FP32 first: the compiler would round once, to BF16
          o[e >> 1] |= (uint32_t)f2bf(gv) << (16 * (e & 1));
        }
      }
      *reinterpret_cast<u32x4*>(grad + v * cpad + c0) = o;
    }
  }
  for (int off = 32; off > 0; off >>= 1) s += __shfl_down(s, off, 64);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = s;
  __syncthreads();
  if (threadIdx.x == 0) partials[blockIdx.x] = red[0] + red[1] + red[2] + red[3];
}

// *out = scale * the sum of n partials, by one workgroup in a fixed order.
__global__ __launch_bounds__(256) void k_sum_partials(const double* __restrict__ partials, int n,
                                                      double scale, double* __restrict__ out) {
  __shared__ double red[4];
  double s = 0.0;
  for (int i = threadIdx.x; i < n; i += 256) s += partials[i];
  for (int off = 32; off > 0; off >>= 1) s += __shfl_down(s, off, 64);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = s;
  __syncthreads();
  if (threadIdx.x == 0) *out = scale * (red[0] + red[1] + red[2] + red[3]);
}

// FP32 master weights W[cout][27][cin] -> BF16 A operands of k_conv3, [output tile]
// [chunk][step][lane][8]: the 8 input channels of pair 4 step + g of output
// channel 16 tile + j (zeros beyond the last pair and the real channels).  wp: the
// forward convolution; wf: backward data, which is a convolution with outputs and
// inputs exchanged and tap k -> 26 - k.  Every layer in one launch (blockIdx.y),
// one lane's 16 bytes a thread.
constexpr int kNetMaxLayers = 23;   // six levels: 12 + 10 + 1
struct PackLayer {
  const float* w;
  uint16_t *wp, *wf;   // wf null: forward only
  int cout, cin, cout_pad, cin_pad, cin_pad16;
};
struct PackTable {
  PackLayer l[kNetMaxLayers];
};
__global__ void k_pack_weights(PackTable t) {
  const PackLayer& p = t.l[blockIdx.y];
  const unsigned nf = (unsigned)(conv_packed(p.cout_pad, p.cin_pad) / 8);
  const unsigned nb = p.wf ? (unsigned)(conv_packed(p.cin_pad16, p.cout_pad) / 8) : 0;
  for (unsigned id = blockIdx.x * blockDim.x + threadIdx.x; id < nf + nb;
       id += gridDim.x * blockDim.x) {
    const bool fwd = id < nf;
    const unsigned u = fwd ? id : id - nf;
    const int cg_all = (fwd ? p.cin_pad : p.cout_pad) / 8, cgc = conv_chunk(cg_all);
    const int ns = conv_steps(cgc), chunks = cg_all / cgc;
    const int lane = u & 63, s = u / 64 % ns, chunk = u / 64 / ns % chunks, tile = u / 64 / ns / chunks;
    const int q = 4 * s + (lane >> 4), row = tile * 16 + (lane & 15);
    const int tap = q / cgc, col0 = (chunk * cgc + q - tap * cgc) * 8;
    uint32_t h[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const int o = fwd ? row : col0 + e, i = fwd ? col0 + e : row, k = fwd ? tap : 26 - tap;
      h[e] = q < 27 * cgc && o < p.cout && i < p.cin ? f2bf(p.w[((size_t)o * 27 + k) * p.cin + i]) : 0u;
    }
    reinterpret_cast<u32x4*>(fwd ? p.wp : p.wf)[u] =
        u32x4{h[0] | (h[1] << 16), h[2] | (h[3] << 16), h[4] | (h[5] << 16), h[6] | (h[7] << 16)};
  }
}

// Global gradient norm for clipping: per-block FP64 sums of squares (fixed
// block count and order), then one block forms scale = min(1, clip / |g|).
constexpr int kNormBlocks = 256;

__global__ __launch_bounds__(256) void k_sumsq(const float* __restrict__ g, size_t n,
                                               double* __restrict__ partials) {
  __shared__ double red[4];
  double s = 0.0;
  for (size_t id = (size_t)blockIdx.x * blockDim.x + threadIdx.x; id < n;
       id += (size_t)gridDim.x * blockDim.x)
    s += (double)g[id] * (double)g[id];
  for (int off = 32; off > 0; off >>= 1) s += __shfl_down(s, off, 64);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = s;
  __syncthreads();
  if (threadIdx.x == 0) partials[blockIdx.x] = red[0] + red[1] + red[2] + red[3];
}

__global__ void k_clip_scale(double* __restrict__ partials, int nb, double clip) {
  if (threadIdx.x != 0 || blockIdx.x != 0) return;
  double s = 0.0;
  for (int i = 0; i < nb; ++i) s += partials[i];
  const double norm = sqrt(s);
  partials[nb] = norm;                                   // |g| before clipping
  partials[nb + 1] = norm > clip ? clip / norm : 1.0;    // scale applied to g
}

// Adam with bias correction, FP32 master parameters; the gradient is first
// multiplied by *scale when scale is not null (global-norm clipping).
__global__ void k_adam(float* __restrict__ theta, float* __restrict__ m, float* __restrict__ v,
                       const float* __restrict__ grad, size_t n, float lr, float b1, float b2,
                       float eps, float c1, float c2, const double* __restrict__ scale) {
  const size_t id = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (id >= n) return;
  const float gr = scale ? (float)((double)grad[id] * *scale) : grad[id];
  const float mm = b1 * m[id] + (1.0f - b1) * gr;
  const float vv = b2 * v[id] + (1.0f - b2) * gr * gr;
  m[id] = mm;
  v[id] = vv;
  theta[id] -= lr * (mm / c1) / (sqrtf(vv / c2) + eps);
}

}  // namespace net
}  // namespace rism
