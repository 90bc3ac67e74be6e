// Gradient of the solvation free energy with respect to the solute atom
// positions: the solvent term of the derivative of the MM/3D-RISM free energy
// (section "Hybrid implementation", the derivative of Eq 23),
//
//   d(dmu)/dR_a = sum_g rho_g \int g_g(r) d u_g(r) / dR_a dr,
//
// with u_g the solute-solvent potential of Eq 22.  On the grid the integral is
// the box sum dV sum_n.  Per pair, with d = |r - R_a| and the beta-scaled
// coefficients of k_prep_atoms (A = beta 4 eps sigma^12, B = beta 4 eps
// sigma^6, coul_g = beta C q_g):
//
//   d(beta u_ag)/dR_a = S (R_a - r),   S = -coul_g q_a / d^3 - 12 A / d^14 + 6 B / d^8.
//
// Below d = D_MIN the potential is the clamped constant, so such pairs add
// nothing.  Pair terms and sums are FP64; g is the float32 field the solve
// returns.
//
// Work split: a workgroup holds 64 A atoms (A per lane, 64 apart; its four waves
// take the same atoms) and walks tiles of 256 grid points.  A tile's per-point data
// (coordinates, rho_g g_g, and the atom-independent Coulomb weight
// sum_g rho_g g_g coul_g) sit in LDS and are read as broadcasts; points where
// every g_g is 0 (inside the solute core) are skipped by whole waves.  Each
// workgroup leaves one FP64 partial per (atom, component); a second kernel adds
// them in a fixed order, so the result does not depend on scheduling.
//
// With one atom a lane the n_v + 5 LDS reads of a point cost the compute unit
// more cycles than the pair's FP64 arithmetic; with two the arithmetic bounds
// (200 atoms, 128^3, 5 sites, repeated back to back: 765 us at A = 1, 690 at 2, 675
// at 4, which wastes more lanes at other atom counts; 1230 us before, with a square
// root and a division for 1/d and one atom a lane).  At most 32 atoms leave lanes over: the
// wave then takes 2 or 4 points at a time, each for `lanes` = 32 or 16 lanes.
#pragma once

#include "common.hpp"

namespace rism {

constexpr int kGradThreads = 256;       // four waves
constexpr int kGradLanes = 64;          // lanes of a wave
constexpr int kGradTile = 256;          // grid points staged per round
constexpr double kGradDMin2 = 1.0e-4;   // D_MIN^2 (D_MIN = 0.01 A)

template <int NV, int A>
__global__ __launch_bounds__(kGradThreads) void k_sfe_grad(
    const double4* __restrict__ atoms, const double2* __restrict__ lj, int n_atoms,
    const float* __restrict__ g, int nx, int ny, size_t N, double dr, SiteConsts sc,
    double* __restrict__ out, double scale, int lanes) {
  __shared__ double s_xyz[3][kGradTile];
  __shared__ double s_rg[NV][kGradTile];
  __shared__ double s_gc[kGradTile];
  __shared__ int s_live[kGradTile];
  __shared__ double s_red[kGradThreads / 64][kGradLanes][3];

  const int lane = threadIdx.x & 63;
  const int wave = threadIdx.x >> 6;
  const int al = lane & (lanes - 1), sub = lane / lanes, subs = kGradLanes / lanes;
  const int atom0 = blockIdx.y * lanes * A + al;   // this lane's atoms: atom0 + lanes i
  double4 at[A];
  double a12[A][NV], b6[A][NV], gr[A][3];
#pragma unroll
  for (int i = 0; i < A; ++i) {
    const int a = atom0 + lanes * i;
    const int a_ld = a < n_atoms ? a : n_atoms - 1;   // idle lanes repeat the last atom
    at[i] = atoms[a_ld];
    gr[i][0] = gr[i][1] = gr[i][2] = 0.0;
#pragma unroll
    for (int s = 0; s < NV; ++s) {
      const double2 c = lj[(size_t)a_ld * NV + s];
      a12[i][s] = 12.0 * c.x;
      b6[i][s] = 6.0 * c.y;
    }
  }

  const size_t tiles = (N + kGradTile - 1) / kGradTile;
  for (size_t tile = blockIdx.x; tile < tiles; tile += gridDim.x) {
    const size_t p0 = tile * kGradTile;
    const int cnt = (int)((N - p0) < (size_t)kGradTile ? (N - p0) : (size_t)kGradTile);
    __syncthreads();   // the previous tile's LDS is no longer read
    for (int t = threadIdx.x; t < cnt; t += kGradThreads) {
      const size_t p = p0 + t;
      const int ix = (int)(p % nx);
      const int iy = (int)((p / nx) % ny);
      const int iz = (int)(p / ((size_t)nx * ny));
      s_xyz[0][t] = ix * dr;
      s_xyz[1][t] = iy * dr;
      s_xyz[2][t] = iz * dr;
      double gc = 0.0;
      int live = 0;
#pragma unroll
      for (int s = 0; s < NV; ++s) {
        const float gv = g[(size_t)s * N + p];
        live |= gv != 0.0f;
        const double rg = sc.rho[s] * (double)gv;
        s_rg[s][t] = rg;
        gc += rg * sc.coul64[s];
      }
      s_gc[t] = gc;
      s_live[t] = live;
    }
    __syncthreads();
    for (int t = wave * subs + sub; t < cnt; t += kGradThreads / lanes) {
      if (!s_live[t]) continue;
      const double x = s_xyz[0][t], y = s_xyz[1][t], z = s_xyz[2][t], gc = s_gc[t];
      double rg[NV];
#pragma unroll
      for (int s = 0; s < NV; ++s) rg[s] = s_rg[s][t];
#pragma unroll
      for (int i = 0; i < A; ++i) {
        const double dx = x - at[i].x, dy = y - at[i].y, dz = z - at[i].z;
        const double d2 = dx * dx + dy * dy + dz * dz;
        const double inv = rsqrt_nr(fmax(d2, kGradDMin2));
        const double inv2 = inv * inv;
        const double inv6 = inv2 * inv2 * inv2;
        double sa = 0.0, sb = 0.0;
#pragma unroll
        for (int s = 0; s < NV; ++s) {
          sa += a12[i][s] * rg[s];
          sb += b6[i][s] * rg[s];
        }
        // S summed over sites with the weights rho_g g_g; the gradient adds S (R - r)
        double S = -at[i].w * gc * inv2 * inv - inv6 * inv2 * (inv6 * sa - sb);
        S = d2 < kGradDMin2 ? 0.0 : S;   // the potential is constant there
        gr[i][0] -= S * dx;
        gr[i][1] -= S * dy;
        gr[i][2] -= S * dz;
      }
    }
  }

#pragma unroll
  for (int i = 0; i < A; ++i) {
    const int atom = atom0 + lanes * i;
    __syncthreads();   // the previous atoms' sums are read
#pragma unroll
    for (int c = 0; c < 3; ++c) s_red[wave][lane][c] = gr[i][c];
    __syncthreads();
    if (wave == 0 && sub == 0 && atom < n_atoms) {
      double* o = out + ((size_t)blockIdx.x * n_atoms + atom) * 3;
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        double v = 0.0;
        for (int w = 0; w < kGradThreads / 64; ++w)
          for (int k = 0; k < subs; ++k) v += s_red[w][k * lanes + al][c];
        o[c] = v * scale;
      }
    }
  }
}

// out[i] = sum over the nb partial rows of part[b][i] (part may be out), and NaN for
// an infinite coordinate, whose pair force is 0 times infinity.  A workgroup takes
// kGradRedCols columns; thread group r of kGradRedRows adds rows r, r + kGradRedRows, ...
// in row order and the groups are added in order (fixed, so deterministic).
// Bound by the latency of a thread's loads in turn: 126 us for 512 rows x 600
// columns with one thread per column, 21 us with 16.
constexpr int kGradRedCols = 16, kGradRedRows = 16;

__global__ __launch_bounds__(kGradRedCols* kGradRedRows) void k_sfe_grad_reduce(
    const double* part, int nb, int n3, const double4* __restrict__ atoms, double* out) {
  __shared__ double red[kGradRedRows][kGradRedCols];
  const int c = threadIdx.x % kGradRedCols, r = threadIdx.x / kGradRedCols;
  const int i = blockIdx.x * kGradRedCols + c;
  double v = 0.0;
  if (i < n3)
    for (int b = r; b < nb; b += kGradRedRows) v += part[(size_t)b * n3 + i];
  const double pos = r == 0 && i < n3 ? reinterpret_cast<const double*>(atoms + i / 3)[i % 3] : 0.0;
  red[r][c] = v;
  __syncthreads();
  if (r == 0 && i < n3) {
    for (int k = 1; k < kGradRedRows; ++k) v += red[k][c];
    out[i] = fabs(pos) < kFarAway ? v : __longlong_as_double(0x7ff8000000000000);
  }
}

}  // namespace rism
