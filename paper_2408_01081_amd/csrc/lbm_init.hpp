// FP64 second-order initialisation (Eq. ic_second) shared by the single-lattice
// and batched entry points.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "lbm.h"
#include "lbm_kernels.hpp"
#include "lbm_plan.hpp"
#include "lbm_step.hpp"

namespace lbmk {

// What the two field arrays of an initialisation hold: (v0, Cauchy stress)
// or (v0, displacement gradient of u0)
constexpr int INIT_FROM_STRESS = 0;
constexpr int INIT_FROM_GRADIENT = 1;

struct InitConst {
  double kK, km, cK, cmu, dx;
  // Cauchy stress -> j (inverse of Eq. sigma_num): 1 / (2 rho c_K),
  // 1 / (2 rho c_mu), 1 / (rho c_mu) (the last two unused for c_mu = 0, which
  // starts from the displacement gradient)
  double js, jd, jxy;
  int bc;
};

inline InitConst init_const(double kK, double km, double cK, double cmu, double rho, double dx,
                            int bc) {
  return InitConst{kK, km, cK, cmu, dx, 0.5 / (rho * cK), 0.5 / (rho * cmu), 1.0 / (rho * cmu), bc};
}

// Phi_x(V)/c and Phi_y(V)/c in double precision
__device__ inline void flux_x(const InitConst& k, const double V[NC], double o[NC]) {
  o[0] = k.kK * V[2] + k.km * V[3];
  o[1] = k.km * V[4];
  o[2] = k.kK * V[0];
  o[3] = k.km * V[0];
  o[4] = k.km * V[1];
}
__device__ inline void flux_y(const InitConst& k, const double V[NC], double o[NC]) {
  o[0] = k.km * V[4];
  o[1] = k.kK * V[2] - k.km * V[3];
  o[2] = k.kK * V[1];
  o[3] = -k.km * V[1];
  o[4] = k.km * V[0];
}

// U = (v, j) from velocity and Cauchy stress at a node (inverse of Eq. sigma_num)
__device__ inline void to_U(const InitConst& k, double vx, double vy, double sxx, double syy,
                            double sxy, double U[NC]) {
  U[0] = vx;
  U[1] = vy;
  U[2] = -k.js * (sxx + syy);
  U[3] = -k.jd * (sxx - syy);
  U[4] = -k.jxy * sxy;
}

// Eq. ic_vector: U from v and the displacement gradient (uxx = du_x/dx,
// uxy = du_x/dy, uyx = du_y/dx, uyy = du_y/dy); linear, so it also maps
// derivatives of these fields to derivatives of U
__device__ inline void from_gradient(const InitConst& k, double vx, double vy, double uxx,
                                     double uxy, double uyx, double uyy, double U[NC]) {
  U[0] = vx;
  U[1] = vy;
  U[2] = -k.cK * (uxx + uyy);
  U[3] = -k.cmu * (uxx - uyy);
  U[4] = -k.cmu * (uyx + uxy);
}

// The initial data of a node: v0 and, with SRC = INIT_FROM_STRESS, the Cauchy
// stress [3][ny][nx], with INIT_FROM_GRADIENT the displacement gradient
// [4][ny][nx] (du_x/dx, du_x/dy, du_y/dx, du_y/dy)
constexpr int NRAW = 6;

template <int SRC, typename T>
__device__ inline void load_raw(const T* __restrict__ v0, const T* __restrict__ s0, int64_t n,
                                int64_t id, double r[NRAW]) {
  r[0] = (double)v0[id];
  r[1] = (double)v0[n + id];
  r[2] = (double)s0[id];
  r[3] = (double)s0[n + id];
  r[4] = (double)s0[2 * n + id];
  r[5] = SRC == INIT_FROM_GRADIENT ? (double)s0[3 * n + id] : 0.0;
}

// U0 from those data.  Linear, so it also maps their derivatives to those of
// U0.  The gradient route (j = -c (derivatives of u0)) divides by no c_mu, so
// c_mu = 0 is allowed there.
template <int SRC>
__device__ inline void raw_U(const InitConst& k, const double r[NRAW], double U[NC]) {
  if (SRC == INIT_FROM_GRADIENT)
    from_gradient(k, r[0], r[1], r[2], r[3], r[4], r[5], U);
  else
    to_U(k, r[0], r[1], r[2], r[3], r[4], U);
}

// Lattice derivative (dx d/dx) at position m of an axis of n nodes as
// wa F[a] + wb F[b] + wm F[m]: central differences, at walls the one-sided
// second-order formula (first order on two nodes, zero on one).  The weights
// are selected, not branched on, so that a node's loads along both axes are
// all in flight together.
struct Diff {
  int a, b;
  double wa, wb, wm;
};

__device__ inline Diff lattice_diff(int bc, int m, int n) {
  Diff d;
  const bool lo = m == 0, hi = m == n - 1;
  const bool wall = bc != LBM_PERIODIC && (lo || hi);
  const double s = lo ? 1.0 : -1.0;  // inward
  const int i = lo ? 1 : -1;
  if (n < 2) return Diff{m, m, 0.0, 0.0, 0.0};
  d.a = wall ? m + i : (hi ? 0 : m + 1);
  d.b = wall ? (n == 2 ? m : m + 2 * i) : (lo ? n - 1 : m - 1);
  d.wa = wall ? (n == 2 ? s : 2.0 * s) : 0.5;
  d.wb = wall ? (n == 2 ? 0.0 : -0.5 * s) : -0.5;
  d.wm = wall ? (n == 2 ? -s : -1.5 * s) : 0.0;
  return d;
}

// B_hat(x, y, t_0) = (dt / rho) b_bar in FP64 from the separable tables (zero
// without a load)
__device__ inline void body_hat0(const Force& F, int x, int y, double& bx, double& by) {
  double a = 0.0, b = 0.0;
  for (int r = 0; r < F.rank; ++r) {
    const double yt = (double)F.Y[(int64_t)r * F.ny + y] * (double)F.Trow[r];
    const float* X = F.X + (int64_t)r * 2 * F.nx;
    a += (double)X[x] * yt;
    b += (double)X[F.nx + x] * yt;
  }
  bx = (double)F.scale * a;
  by = (double)F.scale * b;
}

// Populations f*(0) of one node (x, y): Eq. ic_second in FP64 followed by the
// first omega = 2 collision, rounded once to FP32.  v0 [2][ny][nx] and s0
// (load_raw) are the instance's fields (double or float); grad is nullable
// FP64 physical derivatives d/dx, d/dy of the input fields: [2][5][ny][nx] of
// (v, sigma_bar), or [2][6][ny][nx] of (v, grad u0) with INIT_FROM_GRADIENT;
// F the body load at t_0 (rank 0: none).
//
// Eq. ic_second in lattice units (c dt = dx absorbed into UX, UY) is
//   f_q = 1/4 [U + 2 C_q U]
//     - 1/8 { B + 2 C_q B + i UX + (2i^2-1) X(UX) - 2 C_q X(UX)
//             + j UY + (2j^2-1) Y(UY) - 2 C_q Y(UY) },  B = (B_hat_x, B_hat_y, 0, 0, 0),
// whose sum is U - B/2, so the first collision's U_num is U.  With
// P = X(UX) - Y(UY), S = X(UX) + Y(UY) (X and Y linear, C_q = i X + j Y) the
// collided populations f* = U/2 + C_q U - f pair up by axis:
//   f*_(+-1,0) = U/4 + (B + P)/8 +- [X(U)/2 + (2 X(B) + UX - 2 X(S))/8],
//   f*_(0,+-1) = U/4 + (B - P)/8 +- [Y(U)/2 + (2 Y(B) + UY - 2 Y(S))/8].
// The pass is bound by memory (120 B per node).  Written out per direction,
// with FP64 divisions in the conversion of all five nodes and its loads behind
// the branches of the boundary rule, it took 789 us on 4096 x 4096 and 92 us
// on 2048 x 1024; in this form with plain stores 536 and 38 us, with
// nontemporal ones 515 and 37 us, the pass repeated alone (3.9 and 6.9 TB/s);
// between the steps and outputs of a run 526 and 70.

template <bool NT>
__device__ __forceinline__ void init_store(float v, float* p) {
  if (NT)
    __builtin_nontemporal_store(v, p);
  else
    *p = v;
}

template <int SRC, bool NT, typename T>
__device__ inline void init_node(const T* __restrict__ v0, const T* __restrict__ s0,
                                 const double* __restrict__ grad, float* __restrict__ dst,
                                 const Grid& g, const InitConst& k, int x, int y,
                                 const Force& F = Force{}) {
  const int64_t n = (int64_t)g.nx * g.ny;
  const int64_t id = (int64_t)y * g.nx + x;
  double U[NC], UX[NC], UY[NC], r[NRAW];
  if (grad) {
    // physical derivatives of the input fields -> lattice derivatives of U
    load_raw<SRC>(v0, s0, n, id, r);
    raw_U<SRC>(k, r, U);
    constexpr int nf = SRC == INIT_FROM_GRADIENT ? 6 : 5;
    load_raw<SRC>(grad, grad + 2 * n, n, id, r);
    raw_U<SRC>(k, r, UX);
    load_raw<SRC>(grad + nf * n, grad + (nf + 2) * n, n, id, r);
    raw_U<SRC>(k, r, UY);
    for (int c = 0; c < NC; ++c) {
      UX[c] *= k.dx;
      UY[c] *= k.dx;
    }
  } else {
    const Diff dx = lattice_diff(k.bc, x, g.nx), dy = lattice_diff(k.bc, y, g.ny);
    const int64_t row = (int64_t)y * g.nx;
    double xa[NRAW], xb[NRAW], ya[NRAW], yb[NRAW];
    load_raw<SRC>(v0, s0, n, id, r);
    load_raw<SRC>(v0, s0, n, row + dx.a, xa);
    load_raw<SRC>(v0, s0, n, row + dx.b, xb);
    load_raw<SRC>(v0, s0, n, (int64_t)dy.a * g.nx + x, ya);
    load_raw<SRC>(v0, s0, n, (int64_t)dy.b * g.nx + x, yb);
    for (int c = 0; c < NRAW; ++c) {
      xa[c] = fma(dx.wa, xa[c], fma(dx.wb, xb[c], dx.wm * r[c]));
      ya[c] = fma(dy.wa, ya[c], fma(dy.wb, yb[c], dy.wm * r[c]));
    }
    raw_U<SRC>(k, r, U);
    raw_U<SRC>(k, xa, UX);
    raw_U<SRC>(k, ya, UY);
  }
  double XUX[NC], YUY[NC], P[NC], S[NC], A[NC], B[NC], o[NC];
  flux_x(k, UX, XUX);
  flux_y(k, UY, YUY);
  for (int c = 0; c < NC; ++c) {
    P[c] = XUX[c] - YUY[c];
    S[c] = XUX[c] + YUY[c];
  }
  double Bh[NC] = {0.0, 0.0, 0.0, 0.0, 0.0};
  if (F.rank > 0) body_hat0(F, x, y, Bh[0], Bh[1]);
  // odd parts: X(U)/2 + (2 X(B) + UX - 2 X(S))/8 = X(U/2 + B/4 - S/4) + UX/8
  for (int c = 0; c < NC; ++c) o[c] = fma(0.25, Bh[c] - S[c], 0.5 * U[c]);
  flux_x(k, o, A);
  flux_y(k, o, B);
  for (int c = 0; c < NC; ++c) {
    const double e = fma(0.125, Bh[c], 0.25 * U[c]);
    const double ex = fma(0.125, P[c], e), ey = fma(-0.125, P[c], e);
    const double ox = fma(0.125, UX[c], A[c]), oy = fma(0.125, UY[c], B[c]);
    init_store<NT>((float)(ex + ox), dst + pidx(g, 0 * NC + c, y, x));
    init_store<NT>((float)(ey + oy), dst + pidx(g, 1 * NC + c, y, x));
    init_store<NT>((float)(ex - ox), dst + pidx(g, 2 * NC + c, y, x));
    init_store<NT>((float)(ey - oy), dst + pidx(g, 3 * NC + c, y, x));
  }
}

// A workgroup of 256 threads covers a tile of 64 columns x 4 rows (one wave
// per row): a node's y neighbours are mostly another wave's row of the same
// tile, and finding (x, y) takes no 64-bit division per thread.
constexpr int FT_X = 64, FT_Y = 4;

inline int field_tiles(const Grid& g) {
  return ((g.nx + FT_X - 1) / FT_X) * ((g.ny + FT_Y - 1) / FT_Y);
}

// node (x, y) of this thread; false beyond the grid
__device__ inline bool field_node(const Grid& g, int& x, int& y) {
  const int tx = (g.nx + FT_X - 1) / FT_X, ty = (g.ny + FT_Y - 1) / FT_Y;
  const int tile = xcd_tile(blockIdx.x, tx * ty);
  const int ry = tile / tx;
  x = (tile - ry * tx) * FT_X + (int)(threadIdx.x & 63);
  // (one row per wave: uniform, so row addresses are formed in scalar registers)
  y = ry * FT_Y + __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  return x < g.nx && y < g.ny;
}

// The passes that read no neighbours (moments, displacement, populations) take
// 256 consecutive nodes per workgroup, so every lane has a node whatever nx and
// ny are.  per_xcd: each XCD a contiguous part of the lattice, whose lines two
// XCDs then share nowhere but at its ends; for states whose two buffers the
// last-level cache holds (INIT_NT_BYTES).  Beyond, grid order, in which the
// workgroups in flight read and write one stretch of memory.  Two lattices in
// turn (initialisation, steps, moments), moments in grid order / a part per XCD
// / in tiles with a part per XCD: 1000 x 777 15.7 / 14.4 / 15.0 us, 200000 x 6
// 21.8 / 19.9 / 23.4, 2048 x 1024 33 / 38 / 43, 1000 x 2500 44 / 60 / 63,
// 2500 x 1500 82 / 95 / 100.
inline unsigned flat_blocks(const Grid& g) {
  return (unsigned)(((int64_t)g.nx * g.ny + 255) / 256);
}

// (a lattice of more than 2^32 - 256 nodes exceeds the card's memory)
__device__ inline bool flat_node(const Grid& g, bool per_xcd, int& x, int& y) {
  const unsigned block = per_xcd ? (unsigned)xcd_tile(blockIdx.x, gridDim.x) : blockIdx.x;
  const unsigned id = block * 256u + threadIdx.x;
  y = (int)(id / (unsigned)g.nx);
  x = (int)(id - (unsigned)y * (unsigned)g.nx);
  return y < g.ny;
}

}  // namespace lbmk
