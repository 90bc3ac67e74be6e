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

// FP32 -> BF16 with round-to-nearest-even (NaN stays NaN); BF16 -> FP32 exact.
__device__ __forceinline__ uint16_t f2bf(float f) {
  uint32_t u = __float_as_uint(f);
  if ((u & 0x7fffffffu) > 0x7f800000u) return (uint16_t)0x7fc0;
  u += 0x7fffu + ((u >> 16) & 1u);
  return (uint16_t)(u >> 16);
}
__device__ __forceinline__ float bf2f(uint16_t h) { return __uint_as_float((uint32_t)h << 16); }

__device__ __forceinline__ bf16x8 ld8(const uint16_t* p) {   // 16-byte aligned
  return __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4*>(p));
}
__device__ __forceinline__ bf16x8 zero8() {
  const u32x4 z = {0u, 0u, 0u, 0u};
  return __builtin_bit_cast(bf16x8, z);
}

// Offsets of tap k = (dz * 3 + dy) * 3 + dx are (dz - 1, dy - 1, dx - 1).
__device__ __forceinline__ void tap_offset(int tap, int& dz, int& dy, int& dx) {
  dz = tap / 9 - 1;
  dy = (tap / 3) % 3 - 1;
  dx = tap % 3 - 1;
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
  const uint16_t* w;    // packed [cout_pad][27][cin], cin = ca + cb
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
  uint16_t h[4];
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const uint16_t a = (uint16_t)(e & 1 ? y[e >> 1] >> 16 : y[e >> 1] & 0xffffu);
    h[e] = f2bf(bf2f(a) > 0.0f ? d[e] : slope * d[e]);
  }
  return u32x2{(uint32_t)h[0] | ((uint32_t)h[1] << 16), (uint32_t)h[2] | ((uint32_t)h[3] << 16)};
}

// Epilogue of one accumulator tile: output channels c0 .. c0 + 3 of voxel v.
template <int EPI>
__device__ __forceinline__ void conv_store(const ConvArgs& p, int N, size_t v, int c0,
                                           const f32x4& r) {
  if (EPI == EPI_BF16_LEAKY) {
    uint16_t h[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      float val = r[e] + (c0 + e < p.cout ? p.bias[c0 + e] : 0.0f);
      val = val > 0.0f ? val : p.slope * val;
      h[e] = f2bf(val);
    }
    const u32x2 pk = {(uint32_t)h[0] | ((uint32_t)h[1] << 16),
                      (uint32_t)h[2] | ((uint32_t)h[3] << 16)};
    *reinterpret_cast<u32x2*>(p.yb + v * p.cout_pad + c0) = pk;
  } else if (EPI == EPI_F32_SITE) {
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if (c0 + e < p.cout) p.yf[(size_t)(c0 + e) * N + v] = r[e] + p.bias[c0 + e];
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
// computes 16 output channels (tile blockIdx.y) of a 16 x TY x 4 voxel tile
// (TY = 8; 2 on small grids, for more workgroups).  It stages the tile's input
// with a one-voxel halo (18 x (TY + 2) x 6 voxels) in LDS, CGC channel groups at a
// time (CG / CGC chunks), and every tap's operand is read from there instead
// of from the cache hierarchy.  LDS layout [hz][hy][cg][hx] (16-byte units):
// the 16 voxels of one operand are consecutive units, conflict-free.  Wave w
// owns the z-slice z0 + w: its TY rows y0 .. y0 + TY - 1 of 16 voxels are its
// TY accumulator tiles.  Within a chunk the K steps take (tap, channel group)
// pairs in tap-major order, four per matrix instruction: lane group g
// supplies pair q0 + g (its 8 channels), the weights are the A operand (rows
// = output channels), the voxels the B operand (columns).
constexpr int kTileX = 16, kTileZ = 4;
constexpr int kHaloX = kTileX + 2, kHaloZ = kTileZ + 2;

template <int EPI, int CGC, int TY>
__global__ __launch_bounds__(kConvThreads) void k_conv3(ConvArgs p) {
  constexpr int kTileY = TY, kHaloY = TY + 2;
  __shared__ __align__(16) u32x4 halo[kHaloZ * kHaloY * CGC * kHaloX];
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
  const int cbase = (int)blockIdx.y * 16;
  f32x4 acc[kTileY];
#pragma unroll
  for (int t = 0; t < kTileY; ++t) acc[t] = f32x4{0.f, 0.f, 0.f, 0.f};
  constexpr int nq = 27 * CGC;
  const size_t wrow = (size_t)27 * CG * 8;
  for (int c0 = 0; c0 < CG; c0 += CGC) {
    if (c0 > 0) __syncthreads();   // the previous chunk's operands are read
    // stage: item (h, cg), channel group fastest (consecutive 16-byte reads)
    for (int it = threadIdx.x; it < kHaloZ * kHaloY * kHaloX * CGC; it += kConvThreads) {
      const int h = it / CGC, cg = it - h * CGC;
      const int hx = h % kHaloX, hy = (h / kHaloX) % kHaloY, hz = h / (kHaloX * kHaloY);
      const bf16x8 v =
          load_in(p.in, c0 + cg, z0 + hz - 1, y0 + hy - 1, x0 + hx - 1, p.nz, p.ny, p.nx);
      halo[((hz * kHaloY + hy) * CGC + cg) * kHaloX + hx] = __builtin_bit_cast(u32x4, v);
    }
    __syncthreads();
    for (int q0 = 0; q0 < nq; q0 += 4) {
      const int q = q0 + g;
      bf16x8 aw = zero8(), bx[kTileY];
      if (q < nq) {
        const int tap = q / CGC, cg = q - tap * CGC;
        int dz, dy, dx;
        tap_offset(tap, dz, dy, dx);
        aw = ld8(p.w + (size_t)(cbase + j) * wrow + (size_t)(tap * CG + c0 + cg) * 8);
        const int base = ((wave + dz + 1) * kHaloY + dy + 1) * CGC + cg;
#pragma unroll
        for (int t = 0; t < kTileY; ++t)
          bx[t] = __builtin_bit_cast(bf16x8, halo[(base + t * CGC) * kHaloX + j + dx + 1]);
      } else {
#pragma unroll
        for (int t = 0; t < kTileY; ++t) bx[t] = zero8();
      }
#pragma unroll
      for (int t = 0; t < kTileY; ++t)
        acc[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(aw, bx[t], acc[t], 0, 0, 0);
    }
  }
  const int x = x0 + j, z = z0 + wave;
#pragma unroll
  for (int t = 0; t < kTileY; ++t) {
    const int y = y0 + t;
    if (x < p.nx && y < p.ny && z < p.nz)
      conv_store<EPI>(p, N, ((size_t)z * p.ny + y) * p.nx + x, cbase + 4 * g, acc[t]);
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
// bias in a kernel of its own), 820 us now, 0.14 of the BF16 peak.
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
    for (int it = threadIdx.x; it < kWgX * kWgZ * (kWgY / 2) * 2 * OT; it += kConvThreads) {
      const int cg = it % (2 * OT), r = it / (2 * OT);
      const int xx = r % kWgX, yp = r / kWgX % (kWgY / 2), zz = r / (kWgX * (kWgY / 2));
      const int x = x0 + xx, y = y0 + 2 * yp, z = z0 + zz, o = o0 + cg * 8;
      bf16x8 a = zero8(), b = zero8();
      if (x < p.nx && z < p.nz && o < p.cout_pad) {
        const uint16_t* q = p.dy + (((size_t)z * p.ny + y) * p.nx + x) * p.cout_pad + o;
        if (y < p.ny) a = ld8(q);
        if (y + 1 < p.ny) b = ld8(q + (size_t)p.nx * p.cout_pad);
      }
      store_pair(ds + cg * 8 * kWgDyPitch + (zz * kWgX + xx) * 4 + yp, kWgDyPitch, a, b);
    }
    for (int it = threadIdx.x; it < kWgRows * (kWgY / 2 + 1) * cgi; it += kConvThreads) {
      const int cg = it % cgi, r = it / cgi;
      const int hx = r % (kWgX + 2), q = r / (kWgX + 2);
      const int yp = q % (kWgY / 2 + 1), hz = q / (kWgY / 2 + 1);
      const int x = x0 + hx - 1, y = y0 + 2 * yp - 1, z = z0 + hz - 1;
      const bf16x8 a = load_in(p.in, ti * 2 + cg, z, y, x, p.nz, p.ny, p.nx);
      const bf16x8 b = load_in(p.in, ti * 2 + cg, z, y + 1, x, p.nz, p.ny, p.nx);
      store_pair(xs + cg * 8 * kWgXPitch + (hz * (kWgX + 2) + hx) * 6 + yp, kWgXPitch, a, b);
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
    o[e] = (uint32_t)f2bf(0.125f * s[2 * e]) | ((uint32_t)f2bf(0.125f * s[2 * e + 1]) << 16);
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
      const uint32_t a = c < C ? f2bf(in[(size_t)c * N + v]) : 0u;
      const uint32_t b = c + 1 < C ? f2bf(in[(size_t)(c + 1) * N + v]) : 0u;
      o[e] = a | (b << 16);
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
          o[e >> 1] |= (uint32_t)f2bf((float)(scale * d)) << (16 * (e & 1));
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

// FP32 master weights W[cout][27][cin] -> BF16 packed [cout_pad][27][cin_pad]
// (forward) and flipped [cin_pad16][27][cout_pad] with tap k -> 26 - k
// (backward data: the transposed convolution is a convolution with these), every
// layer in one launch (blockIdx.y).
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
  const unsigned nfwd = (unsigned)p.cout_pad * 27 * p.cin_pad;
  const unsigned nflip = p.wf ? (unsigned)p.cin_pad16 * 27 * p.cout_pad : 0;
  for (unsigned id = blockIdx.x * blockDim.x + threadIdx.x; id < nfwd + nflip;
       id += gridDim.x * blockDim.x) {
    if (id < nfwd) {
      const int i = (int)(id % p.cin_pad);
      const int k = (int)((id / p.cin_pad) % 27);
      const int o = (int)(id / ((unsigned)p.cin_pad * 27));
      p.wp[id] = (o < p.cout && i < p.cin) ? f2bf(p.w[((size_t)o * 27 + k) * p.cin + i]) : (uint16_t)0;
    } else {
      const unsigned f = id - nfwd;
      const int o = (int)(f % p.cout_pad);
      const int k = (int)((f / p.cout_pad) % 27);
      const int i = (int)(f / ((unsigned)p.cout_pad * 27));
      p.wf[f] = (o < p.cout && i < p.cin) ? f2bf(p.w[((size_t)o * 27 + (26 - k)) * p.cin + i])
                                          : (uint16_t)0;
    }
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
