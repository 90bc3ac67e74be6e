// Transforms and fused iteration kernels for any axis length the library takes
// (even, 2..512, prime factors 2, 3 and 5), with the plan in kernel arguments.
// They do what the fixed-size kernels of fft.hpp and fused.hpp do for the
// lengths compiled there: in-place Stockham passes over whole lines in LDS, the
// forward x transform fused with the MDIIS update, and the z transforms fused
// with the k-space contraction.  (The residual stays a kernel of its own,
// k_residual: the order of its Gram sums belongs to the results.)
//
// The plan splits n into radices 8, 4 or 2, 3 and 5, in that order.  A trip
// through LDS does one radix, or two in turn: R1 R2 elements of a line are closed
// under two consecutive Stockham passes, so a thread holds them in registers
// across both, with the operations of the two passes unchanged.  Most lengths up
// to 240 need two trips.  A thread holds at most about kFlexHeld complex values
// across the barrier of a trip, which bounds the tile (FlexPlan::cap).  Index
// divisions are one FP32 multiply (flex_div).
#pragma once

#include "fft.hpp"
#include "iterate.hpp"

namespace rism {

constexpr int kFlexHeld = 16;      // complex values a thread holds in a trip (20 for 4 x 5)
constexpr int kFlexMaxPass = 4;    // trips: 486 = 2.3 3.3 3.3 needs three
constexpr int kFlexMaxLds = 65536; // bytes of dynamic LDS of a workgroup

// A length and its trips: radices ra[p] then rb[p] (1: none) after the product
// ns[p] of the earlier ones; nb[p] = n / (ra rb) groups a line; sa[p], sb[p] =
// 2 n over the product of the radices up to and with ra, rb.
struct FlexPlan {
  int n, pitch, np, cap;   // line pitch in LDS; most elements of a tile
  int ra[kFlexMaxPass], rb[kFlexMaxPass], ns[kFlexMaxPass], nb[kFlexMaxPass], sa[kFlexMaxPass],
      sb[kFlexMaxPass];
  float inv_n, inv_nb[kFlexMaxPass], inv_ns[kFlexMaxPass];
};

// f / d for 0 <= f < 2^21 and d < 2^10 from inv = 1 / d: (f + 1/2) / d is at
// least 1 / (2 d) away from an integer, more than its FP32 rounding.
__device__ __forceinline__ int flex_div(int f, float inv) {
  return (int)(((float)f + 0.5f) * inv);
}

// Groups of R elements a thread holds at once.
__host__ __device__ constexpr int flex_held(int R) { return R > 8 ? 1 : kFlexHeld / R; }

// Radices that one trip can do in turn (the cases of flex_fft).
constexpr bool flex_pair(int a, int b) {
  return (a == 8 && b == 2) || (a <= 4 && (b == 3 || b == 5));
}

// Element i of a line: the skew of fft.hpp (one slot every 8 elements).
__device__ __forceinline__ int flex_at(int i) { return i + (i >> 3); }

// x w (sgn < 0) or x conj(w), the twiddle of element r of a radix-R pass.  Which
// products are fused is fixed here rather than left to the compiler: a solve
// amplifies round-off up to its tolerance, so the rounding of the transforms
// belongs to the results that given inputs have.  Even radices fuse both sums,
// odd ones the imaginary sum for r = R - 1 and the real one for the others.
template <int R>
__device__ __forceinline__ float2 flex_twiddle(float2 x, float2 w, float sgn, int r) {
#pragma clang fp contract(off)
  const float wy = sgn < 0.0f ? w.y : -w.y;
  const float yy = x.y * wy, xy = x.x * wy;
  const bool re = R % 2 == 0 || r < R - 1, im = R % 2 == 0 || r == R - 1;
  return make_float2(re ? __builtin_fmaf(x.x, w.x, -yy) : x.x * w.x - yy,
                     im ? __builtin_fmaf(x.y, w.x, xy) : x.y * w.x + xy);
}
template <int R>
__device__ __forceinline__ double2 flex_twiddle(double2 x, double2 w, double sgn, int) {
  return sgn < 0.0 ? cmul(x, w) : cmulc(x, w);
}

// Trip p: the Stockham passes of radix RA and, if RB > 1, RB.  Group j of a line
// holds the elements j + nb (s + RB r), r < RA, s < RB; with k = j mod ns, the
// first pass takes them over r with twiddles r k, the second over s with
// twiddles s (k + r ns), and element (r, s) goes to (j - k) RA RB + k + ns (r + RA s).
template <int RA, int RB, typename C, typename S>
__device__ inline void flex_pass(C* buf, const FlexPlan& P, int p, int nl, const C* tw2, S sgn) {
  constexpr int R = RA * RB, MAXB = flex_held(R);
  const int nb = P.nb[p], ns = P.ns[p], groups = nl * nb;
  C v[MAXB][RB][RA];
#pragma unroll
  for (int q = 0; q < MAXB; ++q) {
    const int t = threadIdx.x + q * kFftThreads;
    if (t < groups) {
      const int b = flex_div(t, P.inv_nb[p]);
      const int j = t - b * nb;
      const C* e = buf + b * P.pitch;
#pragma unroll
      for (int s = 0; s < RB; ++s)
#pragma unroll
        for (int r = 0; r < RA; ++r) v[q][s][r] = e[flex_at(j + nb * (s + RB * r))];
    }
  }
  __syncthreads();
#pragma unroll
  for (int q = 0; q < MAXB; ++q) {
    const int t = threadIdx.x + q * kFftThreads;
    if (t < groups) {
      const int b = flex_div(t, P.inv_nb[p]);
      const int j = t - b * nb;
      int k = 0;
      if (p > 0) {
        k = j - ns * flex_div(j, P.inv_ns[p]);
#pragma unroll
        for (int s = 0; s < RB; ++s)
#pragma unroll
          for (int r = 1; r < RA; ++r) {
            const C w = tw2[r * k * P.sa[p]];   // < 2 n
            v[q][s][r] = flex_twiddle<RA>(v[q][s][r], w, sgn, r);
          }
      }
#pragma unroll
      for (int s = 0; s < RB; ++s) Dft<RA, C, S>::run(v[q][s], sgn);
      C* e = buf + b * P.pitch;
      const int d0 = (j - k) * R + k;
#pragma unroll
      for (int r = 0; r < RA; ++r) {
        C u[RB];
#pragma unroll
        for (int s = 0; s < RB; ++s) {
          u[s] = v[q][s][r];
          if (s > 0) {
            const C w = tw2[s * (k + r * ns) * P.sb[p]];   // < 2 n
            u[s] = flex_twiddle<RB>(u[s], w, sgn, s);
          }
        }
        if constexpr (RB > 1) Dft<RB, C, S>::run(u, sgn);
#pragma unroll
        for (int s = 0; s < RB; ++s) e[flex_at(d0 + ns * (r + RA * s))] = u[s];
      }
    }
  }
  __syncthreads();
}

// All trips over `nl` lines in buf, in groups of lines that fit the registers.
// The sign is hidden from the compiler (the empty asm), so that the butterflies
// fuse the same products in every kernel.
template <typename C, typename S>
__device__ inline void flex_fft(C* buf, const FlexPlan& P, int nl, const C* tw2, S sgn) {
  asm("" : "+v"(sgn));
  const int group = flex_div(P.cap, P.inv_n);
  for (int l0 = 0; l0 < nl; l0 += group) {
    C* b = buf + l0 * P.pitch;
    const int g = nl - l0 < group ? nl - l0 : group;
    for (int p = 0; p < P.np; ++p) {
      switch (P.ra[p] * 8 + P.rb[p]) {
        case 8 * 8 + 1: flex_pass<8, 1>(b, P, p, g, tw2, sgn); break;
        case 8 * 8 + 2: flex_pass<8, 2>(b, P, p, g, tw2, sgn); break;
        case 4 * 8 + 1: flex_pass<4, 1>(b, P, p, g, tw2, sgn); break;
        case 4 * 8 + 3: flex_pass<4, 3>(b, P, p, g, tw2, sgn); break;
        case 4 * 8 + 5: flex_pass<4, 5>(b, P, p, g, tw2, sgn); break;
        case 2 * 8 + 1: flex_pass<2, 1>(b, P, p, g, tw2, sgn); break;
        case 2 * 8 + 3: flex_pass<2, 3>(b, P, p, g, tw2, sgn); break;
        case 2 * 8 + 5: flex_pass<2, 5>(b, P, p, g, tw2, sgn); break;
        case 3 * 8 + 1: flex_pass<3, 1>(b, P, p, g, tw2, sgn); break;
        case 3 * 8 + 3: flex_pass<3, 3>(b, P, p, g, tw2, sgn); break;
        case 3 * 8 + 5: flex_pass<3, 5>(b, P, p, g, tw2, sgn); break;
        default: flex_pass<5, 1>(b, P, p, g, tw2, sgn); break;
      }
    }
  }
}

// Two neighbouring complex values as one 16-byte access (FP32), or two.
__device__ __forceinline__ void ld2(const float2* p, float2& a, float2& b) {
  const float4 v = *reinterpret_cast<const float4*>(p);
  a = make_float2(v.x, v.y);
  b = make_float2(v.z, v.w);
}
__device__ __forceinline__ void ld2(const double2* p, double2& a, double2& b) {
  a = p[0];
  b = p[1];
}
__device__ __forceinline__ void st2(float2* p, float2 a, float2 b) {
  *reinterpret_cast<float4*>(p) = make_float4(a.x, a.y, b.x, b.y);
}
__device__ __forceinline__ void st2(double2* p, double2 a, double2 b) {
  p[0] = a;
  p[1] = b;
}

template <int W, typename C>
__device__ __forceinline__ void ld_w(const C* p, C* v) {
  if constexpr (W == 2) ld2(p, v[0], v[1]);
  else v[0] = p[0];
}
template <int W, typename C>
__device__ __forceinline__ void st_w(C* p, const C* v) {
  if constexpr (W == 2) st2(p, v[0], v[1]);
  else p[0] = v[0];
}

template <typename C>
__device__ __forceinline__ C* flex_twiddles(C* buf, int elems, int n, const C* __restrict__ tw2_g) {
  C* tw2 = buf + elems;
  for (int i = threadIdx.x; i < 2 * n; i += kFftThreads) tw2[i] = tw2_g[i];
  return tw2;
}

// Axis pass over complex grids data[npair][nz][ny][nx] (as k_fft_fixed).  A tile
// is `lines` rows (axis 0) or `lines` neighbouring columns.  W = 2: nx is even
// and data 16-byte aligned, and two neighbouring columns (or points of a row)
// move as one 16-byte vector in FP32; W = 1: any nx and alignment.
//
// Bound by the phases of a workgroup in turn (load, two trips, store) where they
// do not fill the chip, else by HBM: 160 x 120 x 90, three grids (83 MB a pass):
// 65 us before (one radix a trip, two LDS buffers, run-time divisions), 24 now,
// 17 at the rate of a large copy.
template <typename C, int W>
__global__ __launch_bounds__(kFftThreads) void k_flex_axis(
    C* __restrict__ data, int nx, int ny, int nz, int npair, int axis, FlexPlan P,
    const C* __restrict__ tw2_g, int forward, int lines, const int* __restrict__ done) {
  using S = typename ScalarOf<C>::type;
  if (done && skip_iteration<std::is_same<C, double2>::value>(*done)) return;
  extern __shared__ __align__(16) unsigned char smem[];
  C* buf = reinterpret_cast<C*>(smem);
  const int n = P.n;
  C* tw2 = flex_twiddles(buf, lines * P.pitch, n, tw2_g);
  size_t base, istride;
  int nl;
  if (axis == 0) {
    const size_t rows = (size_t)npair * nz * ny, row0 = (size_t)blockIdx.x * lines;
    nl = (int)((rows - row0) < (size_t)lines ? (rows - row0) : (size_t)lines);
    base = row0 * nx;
    istride = n;
  } else {
    const int tiles_x = (nx + lines - 1) / lines;
    const int outer = blockIdx.x / tiles_x;
    const int x0 = (blockIdx.x - outer * tiles_x) * lines;
    nl = (nx - x0) < lines ? (nx - x0) : lines;
    if (axis == 1) {
      base = (size_t)outer * n * nx + x0;
      istride = nx;
    } else {
      const int p = outer / ny;
      base = ((size_t)p * n * ny + (outer - p * ny)) * nx + x0;
      istride = (size_t)ny * nx;
    }
  }
  // item f = (a, h): elements W h .. of row a (axis 0), or element a of columns W h ..
  const bool row = axis == 0;
  const int part = (row ? n : nl) / W;
  const int total = part * (row ? nl : n);
  const float inv = 1.0f / (float)part;
  __syncthreads();   // twiddles visible
  constexpr int U = sizeof(C) == 8 ? 8 : 4;   // loads in flight per thread
  for (int f0 = threadIdx.x; f0 < total; f0 += U * kFftThreads) {
    C v[U][2];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int f = f0 + u * kFftThreads;
      if (f < total) {
        const int a = flex_div(f, inv), h = f - a * part;
        ld_w<W>(data + base + (size_t)a * istride + W * h, v[u]);
      }
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int f = f0 + u * kFftThreads;
      if (f < total) {
        const int a = flex_div(f, inv), h = f - a * part;
#pragma unroll
        for (int k = 0; k < W; ++k) {
          const int b = row ? a : W * h + k, i = row ? W * h + k : a;
          buf[b * P.pitch + flex_at(i)] = forward ? cmul(v[u][k], tw2[i]) : v[u][k];   // exp(-i pi i / n)
        }
      }
    }
  }
  __syncthreads();
  flex_fft(buf, P, nl, tw2, forward ? S(-1) : S(1));
  for (int f = threadIdx.x; f < total; f += kFftThreads) {
    const int a = flex_div(f, inv), h = f - a * part;
    C v[2];
#pragma unroll
    for (int k = 0; k < W; ++k) {
      const int b = row ? a : W * h + k, i = row ? W * h + k : a;
      v[k] = buf[b * P.pitch + flex_at(i)];
      if (!forward) v[k] = cmulc(v[k], tw2[i]);
    }
    st_w<W>(data + base + (size_t)a * istride + W * h, v);
  }
}

// MDIIS update + closure fused with the forward x transform (k_update_fftx).
// Bound by HBM: 120 x 100 x 90, 3 sites: 32 us for 186 MB (5.8 TB/s); update and
// transform apart took 28 + 33.
// V points a thread and step: 4 where rows are whole 16-byte vectors, else 2.
template <bool ANCHOR, int V, int MM>
__global__ __launch_bounds__(kFftThreads) void k_flex_update(
    const IterState* __restrict__ st, float* __restrict__ tau_hist,
    const float* __restrict__ res_hist, const float* __restrict__ w,
    const float* __restrict__ tau_ref, const float* __restrict__ tau_lo,
    const float* __restrict__ dref, float* __restrict__ dg_out, void* __restrict__ spec_v,
    int ny, int nz, int nv, int npair, int M, int kind, int order, FlexPlan P, int lines,
    const typename std::conditional<ANCHOR, double2, float2>::type* __restrict__ tw2_g) {
  using C = typename std::conditional<ANCHOR, double2, float2>::type;
  using S = typename ScalarOf<C>::type;
  if (skip_iteration<ANCHOR>(st->done)) return;
  extern __shared__ __align__(16) unsigned char smem[];
  C* buf = reinterpret_cast<C*>(smem);
  const int n = P.n, Q = n / V;
  C* tw2 = flex_twiddles(buf, lines * P.pitch, n, tw2_g);
  const size_t plane = (size_t)nz * ny, rows = (size_t)npair * plane;
  const size_t row0 = (size_t)blockIdx.x * lines;
  const int nl = (int)((rows - row0) < (size_t)lines ? (rows - row0) : (size_t)lines);
  const size_t N3 = (size_t)n * plane;
  const UpdateCtl u = load_update_ctl(st, M);
  __syncthreads();
  for (int t = threadIdx.x; t < nl * Q; t += kFftThreads) {
    const int b = flex_div(t, (float)V * P.inv_n);
    const int i0 = (t - b * Q) * V;
    const size_t row = row0 + b;
    const int p = (int)(row / plane);
    const size_t g = (row - (size_t)p * plane) * n + i0;
    double o64[2][V];
    float o32[2][V];
    update_points<ANCHOR, V, MM>(u, tau_hist, res_hist, w, tau_ref, tau_lo, dref, dg_out, N3, nv, p,
                                 g, kind, order, o64, o32);
#pragma unroll
    for (int v = 0; v < V; ++v) {
      const C val = ANCHOR ? make_c((S)o64[0][v], (S)o64[1][v]) : make_c((S)o32[0][v], (S)o32[1][v]);
      buf[b * P.pitch + flex_at(i0 + v)] = cmul(val, tw2[i0 + v]);   // exp(-i pi a / n)
    }
  }
  __syncthreads();
  flex_fft(buf, P, nl, tw2, S(-1));
  C* spec = static_cast<C*>(spec_v) + row0 * n;
  const int half = n / 2;
  for (int f = threadIdx.x; f < nl * half; f += kFftThreads) {
    const int b = flex_div(f, 2.0f * P.inv_n), i = 2 * (f - b * half);
    const C* s = buf + b * P.pitch;
    st2(spec + (size_t)b * n + i, s[flex_at(i)], s[flex_at(i + 1)]);
  }
}

// Forward z transform + contraction + inverse z transform (k_zcz): a workgroup
// owns the columns (x0 .. x0 + B - 1, y) of every pair and their mirror columns;
// B is even, and column pairs move as 16-byte vectors in FP32.  Bound, as the
// fixed kernel is, by a workgroup's phases in turn: 120 x 100 x 90, 3 sites: 20
// us; two z passes and the contraction apart took 33 + 10 + 33.
template <typename C, int NV, bool WITHF>
__global__ __launch_bounds__(kFftThreads) void k_flex_zcz(
    C* __restrict__ spec, int nx, int ny, FlexPlan P, int B, const C* __restrict__ tw2_g,
    double dkx, double dky, double dkz, const C* __restrict__ F,
    const typename ScalarOf<C>::type* __restrict__ chi,
    const typename ScalarOf<C>::type* __restrict__ qtab, double inv_dkt, int m_tab,
    const int* __restrict__ done) {
  using S = typename ScalarOf<C>::type;
  constexpr int NP = (NV + 1) / 2;
  if (done && skip_iteration<std::is_same<C, double2>::value>(*done)) return;
  extern __shared__ __align__(16) unsigned char smem[];
  C* buf = reinterpret_cast<C*>(smem);   // line l = (side * NP + p) * B + b
  const int nz = P.n;
  C* tw2 = flex_twiddles(buf, 2 * NP * B * P.pitch, nz, tw2_g);
  const int tiles_x = (nx + B - 1) / B;
  const int tile = xcd_tile((int)blockIdx.x, (int)gridDim.x);
  const int jy = tile / tiles_x;   // 0 .. ny/2 - 1
  const int x0 = (tile - jy * tiles_x) * B;
  const int nb = (nx - x0) < B ? (nx - x0) : B, H = nb / 2;
  const float inv_h = 1.0f / (float)H;
  const int jy2 = ny - 1 - jy;
  const size_t zs = (size_t)nx * ny, N = zs * nz;
  const int total = 2 * NP * H * nz;
  // item f: element z of columns 2 h and 2 h + 1 of (side, p); side 1 columns run
  // backwards in x, so that pair is stored reversed
  auto item = [&](int f, size_t* g, int* l, int* z, int* side) {
    const int r = flex_div(f, inv_h), h = f - r * H;
    const int sp = flex_div(r, P.inv_n);
    *z = r - sp * nz;
    *side = sp >= NP;
    const int p = sp - (*side ? NP : 0);
    *l = (sp * B + 2 * h) * P.pitch + flex_at(*z);
    const int x = *side ? nx - 2 - x0 - 2 * h : x0 + 2 * h;
    *g = (size_t)p * N + (size_t)*z * zs + (size_t)(*side ? jy2 : jy) * nx + x;
  };
  __syncthreads();   // twiddles visible
  constexpr int U = sizeof(C) == 8 ? 8 : 4;   // loads in flight per thread
  for (int f0 = threadIdx.x; f0 < total; f0 += U * kFftThreads) {
    C a[U], b[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int f = f0 + u * kFftThreads;
      size_t g;
      int l, z, side;
      if (f < total) {
        item(f, &g, &l, &z, &side);
        ld2(spec + g, a[u], b[u]);
      }
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int f = f0 + u * kFftThreads;
      size_t g;
      int l, z, side;
      if (f < total) {
        item(f, &g, &l, &z, &side);
        buf[l] = cmul(side ? b[u] : a[u], tw2[z]);
        buf[l + P.pitch] = cmul(side ? a[u] : b[u], tw2[z]);
      }
    }
  }
  __syncthreads();
  flex_fft(buf, P, 2 * NP * B, tw2, S(-1));   // (unused tail columns carry stale data)

  for (int t = threadIdx.x; t < nb * nz; t += kFftThreads) {
    const int b = flex_div(t, P.inv_n);
    const int jz = t - b * nz;
    const int jx = x0 + b;
    int m;
    S fr;
    table_pos<S>(kappa<S>(jx, nx, dkx), kappa<S>(jy, ny, dky), kappa<S>(jz, nz, dkz), inv_dkt,
                 m_tab, &m, &fr);
    C* pa = buf + b * P.pitch + flex_at(jz);
    C* pb = buf + (NP * B + b) * P.pitch + flex_at(nz - 1 - jz);
    C X[NV];
#pragma unroll
    for (int p = 0; p < NP; ++p) {
      const C z = pa[p * B * P.pitch], zb = pb[p * B * P.pitch];
      X[2 * p] = make_c(S(0.5) * (z.x + zb.x), S(0.5) * (z.y - zb.y));
      if (2 * p + 1 < NV) X[2 * p + 1] = make_c(S(0.5) * (z.y + zb.y), S(-0.5) * (z.x - zb.x));
    }
    C Fk = make_c(S(0), S(0));
    if (WITHF) {
      const size_t L = ((size_t)jz * ny + jy) * nx + jx;
      Fk = L < (N + 1) / 2 ? F[L] : cconj(F[N - 1 - L]);
    }
    C h[NV];
    contract_point<NV, C, WITHF>(X, Fk, m, fr, chi, qtab, h);
#pragma unroll
    for (int p = 0; p < NP; ++p) {
      const C a = h[2 * p];
      const C bb = (2 * p + 1 < NV) ? h[2 * p + 1] : make_c(S(0), S(0));
      pa[p * B * P.pitch] = make_c(a.x - bb.y, a.y + bb.x);
      pb[p * B * P.pitch] = make_c(a.x + bb.y, -a.y + bb.x);
    }
  }
  __syncthreads();
  flex_fft(buf, P, 2 * NP * B, tw2, S(1));
  for (int f = threadIdx.x; f < total; f += kFftThreads) {
    size_t g;
    int l, z, side;
    item(f, &g, &l, &z, &side);
    const C a = cmulc(buf[l], tw2[z]), b = cmulc(buf[l + P.pitch], tw2[z]);
    st2(spec + g, side ? b : a, side ? a : b);
  }
}

}  // namespace rism
