// Per-solute set-up kernels: solute potential (Eq 22), long-range split
// (Eq 29-30), chi interpolation tables and FFT twiddles.  They run once per
// solve, so they work in FP64 and round only their stored results to FP32.
#pragma once

#include "common.hpp"

namespace rism {

constexpr int kPotThreads = 256;
constexpr int kPotChunk = 256;   // atoms staged in LDS at a time

// A coordinate within 2^510, so that squared distances stay finite and 1/d^3 is 0
// (kFarAway: an infinite one); NaN stays NaN.
__device__ __forceinline__ double in_range(double x) {
  const double most = isinf(x) ? kFarAway : 0.5 * kFarAway;
  return fabs(x) > most || isinf(x) ? copysign(most, x) : x;
}

// Solute atoms relative to the grid corner r0 (with the charge in .w), and per
// (atom, site) LJ coefficients beta*4*eps*sigma^12 and beta*4*eps*sigma^6
// (Lorentz-Berthelot mixing).  The pair loops clamp distances with maxima, which
// take the other operand for a NaN, and form 1/d by steps that need d^2 finite:
// so a NaN coordinate is carried by the charge and the coefficients, and far
// coordinates are brought into range here, once an atom.
__global__ void k_prep_atoms(const double* __restrict__ xyz, const double* __restrict__ q,
                             const double* __restrict__ sigma, const double* __restrict__ eps,
                             int n_atoms, double r0x, double r0y, double r0z, double beta,
                             int nv, SiteLJ sites, double4* __restrict__ atoms,
                             double2* __restrict__ lj) {
  const int a = blockIdx.x * blockDim.x + threadIdx.x;
  if (a >= n_atoms) return;
  const double x = in_range(xyz[3 * a] - r0x), y = in_range(xyz[3 * a + 1] - r0y),
               z = in_range(xyz[3 * a + 2] - r0z);
  const double nan = isnan(x) || isnan(y) || isnan(z) ? x + y + z : 0.0;
  atoms[a] = make_double4(x, y, z, q[a] + nan);
  for (int g = 0; g < nv; ++g) {
    const double s = 0.5 * (sigma[a] + sites.sigma[g]);
    const double e = sqrt(eps[a] * sites.eps[g]);
    const double s6 = s * s * s * s * s * s + nan;
    lj[(size_t)a * nv + g] = make_double2(beta * 4.0 * e * s6 * s6, beta * 4.0 * e * s6);
  }
}

// e^{-d} in FP64 for d >= 0, to about 1 ulp: d = -(n ln 2 + r) with |r| <= ln(2)/2,
// the Taylor polynomial of e^r of degree 12 (remainder r^13 / 13! < 2e-16),
// scaled by 2^n.  ln 2 is its double plus the remainder.  The coefficients sit
// in scalar registers (the empty asm hides their values): as literals each
// would be moved into vector registers again for every term.
struct ExpNeg {
  double c[13] = {1.0, 1.0, 1.0 / 2, 1.0 / 6, 1.0 / 24, 1.0 / 120, 1.0 / 720, 1.0 / 5040,
                  1.0 / 40320, 1.0 / 362880, 1.0 / 3628800, 1.0 / 39916800, 1.0 / 479001600};
  double l2e = -1.4426950408889634, hi = -0.69314718055994529, lo = -2.3190468138462996e-17;
  __device__ __forceinline__ ExpNeg() {
#pragma unroll
    for (int i = 2; i < 13; ++i) asm("" : "+s"(c[i]));
    asm("" : "+s"(l2e));
    asm("" : "+s"(hi));
    asm("" : "+s"(lo));
  }
  // K values at a time, term by term: K independent chains
  template <int K>
  __device__ __forceinline__ void run(const double (&d)[K], double (&out)[K]) const {
    double n[K], r[K];
#pragma unroll
    for (int k = 0; k < K; ++k) {
      n[k] = rint(d[k] * l2e);
      r[k] = fma(n[k], lo, fma(n[k], hi, -d[k]));
      out[k] = fma(r[k], c[12], c[11]);
    }
#pragma unroll
    for (int i = 10; i >= 0; --i)
#pragma unroll
      for (int k = 0; k < K; ++k) out[k] = fma(out[k], r[k], c[i]);
#pragma unroll
    for (int k = 0; k < K; ++k) out[k] = ldexp(out[k], (int)n[k]);
  }
};

// w_g = min(beta u_g, cap) - f_g and phi_lr on every grid point.
//   beta u_g = sum_a [beta LJ_ag(dc) + coul_g q_a / dc],  dc = max(d, D_MIN)
//   f_g      = coul_g * phi_lr,  phi_lr = sum_a q_a (1 - e^{-d}) / d
// Two FP64 sums hold the Coulomb part: phi = sum_a q_a / dc and the short-ranged
//   phi_sr = sum_a q_a s(d),  s(d) = e^{-d}/d (d >= D_MIN),
//                             s(d) = 1/D_MIN - (1 - e^{-d})/d (d < D_MIN),
// so that phi_lr = phi - phi_sr, and the uncapped w is accumulated directly as
// beta LJ + coul_g phi_sr.  Pair terms and sums are FP64 (the twelfth power of a
// rounded FP32 distance would cost ~1e-5 relative in w near the solute).
//
// Bound by the FP64 issue rate.  A thread takes K points that follow each other
// in x: they share the atom's data, read at a wave-uniform address (scalar
// loads), and dy^2 + dz^2; and their K independent chains hide the FP64
// latency.  1/dc and dc come from one reciprocal square root, e^{-d} from
// ExpNeg; beyond 38 A it adds below FP64 resolution and is taken as 0 (and not
// evaluated where no point of the wave is nearer).  128^3, 200 atoms, 5 sites: 1439 us
// with a square root, two divisions and the library's exp at one point a thread, 642
// us now (45 FP64 operations a pair, 0.75 of the FP64 issue rate), both repeated back
// to back.  Behind the kernels that write the atoms traces have 1446 and 700 to 760 us:
// the scalar loads then wait for memory.
//
// A small grid has too few waves to hide the scalar loads, whose data, just
// written, is in no nearby cache: it waits for memory atom after atom.  STAGE
// copies the atoms to LDS, a workgroup's loads at once, and one point a thread
// keeps the most waves.  200 atoms, 3 sites: 32^3 59 us staged, 120 with scalar
// loads and two points a thread; 48^3 69 and 121; 64^3 106 and 113, and beyond it
// the LDS reads beside the FP64 operations lose.
template <int NV, int K, bool STAGE>
__global__ __launch_bounds__(kPotThreads) void k_potential(
    const double4* __restrict__ atoms, const double2* __restrict__ lj, int n_atoms, int nx, int ny,
    int nz, double dr, SiteConsts sc, float* __restrict__ w, float* __restrict__ phi_out) {
  const size_t N = (size_t)nx * ny * nz;   // a multiple of K, as nx is
  const unsigned idx = (blockIdx.x * kPotThreads + threadIdx.x) * K;   // N <= 512^3
  if (!STAGE && idx >= N) return;   // (staged: every thread copies)
  __shared__ double4 s_at[STAGE ? kPotChunk : 1];
  __shared__ double2 s_lj[STAGE ? kPotChunk * NV : 1];
  const unsigned row = idx / (unsigned)nx;
  const int ix = (int)(idx - row * nx), iz = (int)(row / (unsigned)ny), iy = (int)(row - iz * ny);
  const double py = iy * dr, pz = iz * dr;
  double px[K], acc[K][NV], phi[K], phi_sr[K];
#pragma unroll
  for (int k = 0; k < K; ++k) {
    px[k] = (ix + k) * dr;
    phi[k] = phi_sr[k] = 0.0;
#pragma unroll
    for (int g = 0; g < NV; ++g) acc[k][g] = 0.0;
  }
  const ExpNeg ex;
  for (int a = 0; a < n_atoms; ++a) {
    if constexpr (STAGE) {
      if (a % kPotChunk == 0) {
        const int cnt = n_atoms - a < kPotChunk ? n_atoms - a : kPotChunk;
        __syncthreads();   // the previous atoms are read
        for (int t = threadIdx.x; t < cnt; t += kPotThreads) s_at[t] = atoms[a + t];
        for (int t = threadIdx.x; t < cnt * NV; t += kPotThreads) s_lj[t] = lj[(size_t)a * NV + t];
        __syncthreads();
      }
    }
    const double4 at = STAGE ? s_at[a % kPotChunk] : atoms[a];
    const double2* la = STAGE ? s_lj + a % kPotChunk * NV : lj + (size_t)a * NV;
    const double dy = py - at.y, dz = pz - at.z;
    const double dyz = dy * dy + dz * dz;
    double d2[K], inv[K], q[K];
    double least = 1.0e300;
#pragma unroll
    for (int k = 0; k < K; ++k) {
      const double dx = px[k] - at.x;
      d2[k] = dx * dx + dyz;
      least = fmin(least, d2[k]);
    }
#pragma unroll
    for (int k = 0; k < K; ++k) {
      inv[k] = rsqrt_nr(fmax(d2[k], kDMin * kDMin));
      q[k] = at.w * inv[k];
      phi[k] += q[k];
    }
    if (least < 38.0 * 38.0) {
      double d[K], e[K];
#pragma unroll
      for (int k = 0; k < K; ++k) d[k] = fmax(d2[k], kDMin * kDMin) * inv[k];
      ex.run<K>(d, e);
      if (least < kDMin * kDMin) {   // a point on an atom: s(d) in its clamped form
#pragma unroll
        for (int k = 0; k < K; ++k)
          if (d2[k] < kDMin * kDMin) {
            const double t = sqrt(d2[k]);
            e[k] = 1.0 - kDMin * ((t > 1.0e-300) ? -expm1(-t) / t : 1.0);
          }
      }
#pragma unroll
      for (int k = 0; k < K; ++k) phi_sr[k] += q[k] * (d[k] < 38.0 ? e[k] : 0.0);
    }
#pragma unroll
    for (int k = 0; k < K; ++k) {
      const double s2 = inv[k] * inv[k];
      const double s6 = s2 * s2 * s2;
#pragma unroll
      for (int g = 0; g < NV; ++g) {
        const double2 c = la[g];
        acc[k][g] += (c.x * s6 - c.y) * s6;
      }
    }
  }
  if (STAGE && idx >= N) return;
#pragma unroll
  for (int k = 0; k < K; ++k) phi[k] -= phi_sr[k];   // phi_lr
#pragma unroll
  for (int g = 0; g < NV; ++g) {
    const double coul = sc.coul64[g];
    float o[K];
#pragma unroll
    for (int k = 0; k < K; ++k) {
      const double u = acc[k][g] + coul * phi_sr[k];
      o[k] = (float)((u + coul * phi[k] > kBetaUCap) ? kBetaUCap - coul * phi[k] : u);
    }
    stv<K>(w + (size_t)g * N + idx, o);
  }
  float o[K];
#pragma unroll
  for (int k = 0; k < K; ++k) o[k] = (float)phi[k];
  stv<K>(phi_out + idx, o);
}

__device__ inline double kappa_of(int j, int n, double dk) {
  return (2 * j < n) ? (j + 0.5) * dk : (j + 0.5 - n) * dk;
}

// Per-atom, per-axis phase tables exp(-i kappa(j) (R_a - r0)) in FP64.
__global__ void k_phase_tables(const double* __restrict__ xyz, int n_atoms, int nx, int ny, int nz,
                               double r0x, double r0y, double r0z, double dkx, double dky,
                               double dkz, double2* __restrict__ ph) {
  const int t = blockIdx.x * blockDim.x + threadIdx.x;
  const int nsum = nx + ny + nz;
  if (t >= n_atoms * nsum) return;
  const int a = t / nsum;
  int j = t - a * nsum;
  double kap, rel;
  if (j < nx) {
    kap = kappa_of(j, nx, dkx);
    rel = xyz[3 * a] - r0x;
  } else if (j < nx + ny) {
    j -= nx;
    kap = kappa_of(j, ny, dky);
    rel = xyz[3 * a + 1] - r0y;
  } else {
    j -= nx + ny;
    kap = kappa_of(j, nz, dkz);
    rel = xyz[3 * a + 2] - r0z;
  }
  double s, c;
  sincos(kap * rel, &s, &c);
  ph[t] = make_double2(c, -s);
}

// Long-range spectrum of Eq 30 for the first ceil(N/2) k-points in linear order,
// divided by dV (the forward FFT is unnormalised):
//   F(k) = (4 pi beta C / l^2) / (|k|^2 (|k|^2 + l^-2)) / dV * sum_a q_a e^{-i k.(R_a - r0)}
// so that f~_g / dV = q_g F (the 1/N of the inverse sits in the Q table).  The
// other half follows from F(-k) = conj F(k).  nz is even, so the first half is
// the planes jz < nz / 2.
//
// A workgroup owns 64 columns jx (one a lane) x 4 rows jy (one a wave) x kFtZ
// planes jz (held by each thread), staging the phases of kFtAtoms atoms at a
// time in LDS: the product of the x and y phases is formed once for its kFtZ
// planes, and the y and z phases and the charge are LDS broadcasts.  The terms
// and their order are those of one k-point at a time.  Bound by the FP64 issue
// rate and the broadcasts together.  128^3, 200 atoms: 325 us with one k-point a
// thread and the phases read through the caches, 79 us now.
constexpr int kFtCols = 64, kFtRows = 4, kFtZ = 8, kFtAtoms = 32;

__global__ __launch_bounds__(256) void k_ftilde(const double2* __restrict__ ph,
                                                const double4* __restrict__ atoms, int n_atoms,
                                                int nx, int ny, int nz, double dkx, double dky,
                                                double dkz, double pref,
                                                double2* __restrict__ F) {
  __shared__ double2 ex[kFtAtoms][kFtCols], ey[kFtAtoms][kFtRows], ez[kFtAtoms][kFtZ];
  __shared__ double q[kFtAtoms];
  const int nsum = nx + ny + nz;
  const int x0 = blockIdx.x * kFtCols, y0 = blockIdx.y * kFtRows, z0 = blockIdx.z * kFtZ;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  double2 s[kFtZ];
#pragma unroll
  for (int i = 0; i < kFtZ; ++i) s[i] = make_double2(0.0, 0.0);
  for (int a0 = 0; a0 < n_atoms; a0 += kFtAtoms) {
    const int cnt = n_atoms - a0 < kFtAtoms ? n_atoms - a0 : kFtAtoms;
    __syncthreads();   // the previous atoms' phases are read
    auto stage = [&](double2* dst, int width, int first, int end, int off) {
      for (int t = threadIdx.x; t < cnt * width; t += 256) {
        const int a = t / width, j = first + t % width;
        dst[t] = j < end ? ph[(size_t)(a0 + a) * nsum + off + j] : make_double2(0.0, 0.0);
      }
    };
    stage(&ex[0][0], kFtCols, x0, nx, 0);
    stage(&ey[0][0], kFtRows, y0, ny, nx);
    stage(&ez[0][0], kFtZ, z0, nz / 2, nx + ny);
    if (threadIdx.x < cnt) q[threadIdx.x] = atoms[a0 + threadIdx.x].w;
    __syncthreads();
    for (int a = 0; a < cnt; ++a) {
      const double2 exy = cmul(ex[a][lane], ey[a][wave]);
      const double qa = q[a];
#pragma unroll
      for (int i = 0; i < kFtZ; ++i) {
        // exy ez, the roundings fixed: a solve amplifies them up to its tolerance
        const double2 z = ez[a][i];
        s[i].x = fma(qa, fma(exy.x, z.x, -__dmul_rn(exy.y, z.y)), s[i].x);
        s[i].y = fma(qa, fma(exy.x, z.y, __dmul_rn(exy.y, z.x)), s[i].y);
      }
    }
  }
  const int jx = x0 + lane, jy = y0 + wave;
  if (jx >= nx || jy >= ny) return;
  const double kx = kappa_of(jx, nx, dkx), ky = kappa_of(jy, ny, dky);
#pragma unroll
  for (int i = 0; i < kFtZ; ++i) {
    const int jz = z0 + i;
    if (jz >= nz / 2) return;
    const double kz = kappa_of(jz, nz, dkz);
    const double k2 = kx * kx + ky * ky + kz * kz;
    const double f = pref / (k2 * (k2 + 1.0 / (kScreen * kScreen)));
    F[((size_t)jz * ny + jy) * nx + jx] = make_double2(f * s[i].x, f * s[i].y);
  }
}

// Interpolation tables with the 1/N of the inverse transform folded in:
//   chi[m][a][b] = chi_ab(m dk) / N,  q[m][b] = sum_a q_a chi_ab(m dk) / N,
// in FP32 (bulk increments) and FP64 (anchor evaluations).
__global__ void k_chi_tables(const double* __restrict__ chi, int nv, int n_k, int m_tab,
                             double inv_n, SiteConsts sc, float* __restrict__ chi32,
                             double* __restrict__ chi64, double* __restrict__ q64) {
  const int t = blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= m_tab * nv) return;
  const int m = t / nv;
  const int b = t - m * nv;
  const int rw32 = chi_row<float>(nv), rw64 = chi_row<double>(nv);
  double qs = 0.0;
  for (int a = 0; a < nv; ++a) {
    const double v = chi[((size_t)a * nv + b) * n_k + m];
    chi32[(size_t)m * rw32 + a * nv + b] = (float)(v * inv_n);
    chi64[(size_t)m * rw64 + a * nv + b] = v * inv_n;
    qs += sc.q64[a] * v;
  }
  if (b == 0) {   // row padding (never read into the arithmetic)
    for (int i = nv * nv; i < rw32; ++i) chi32[(size_t)m * rw32 + i] = 0.0f;
    for (int i = nv * nv; i < rw64; ++i) chi64[(size_t)m * rw64 + i] = 0.0;
  }
  q64[(size_t)m * nv + b] = qs * inv_n;
}

// tw2[m] = exp(-2 pi i m / (2n)), m = 0..2n-1, computed in FP64, of the three
// axes (blockIdx.y) in one launch; a launch each cost 1.4 us and its gap.
struct TwiddleAxes {
  int n[3];
  float2* tw32[3];
  double2* tw64[3];
};

__global__ void k_twiddles(TwiddleAxes ax) {
  const int a = blockIdx.y, n = ax.n[a];
  const int m = blockIdx.x * blockDim.x + threadIdx.x;
  if (m >= 2 * n) return;
  double s, c;
  sincospi((double)m / (double)n, &s, &c);
  if (ax.tw32[a]) ax.tw32[a][m] = make_float2((float)c, (float)(-s));
  if (ax.tw64[a]) ax.tw64[a][m] = make_double2(c, -s);
}

}  // namespace rism
