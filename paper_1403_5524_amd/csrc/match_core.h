// Matching, K-matrix, T-matrix and collision strengths: one team of
// wavefronts per energy (team.h).
//
// With channels sorted by threshold the open channels at energy E are the
// prefix P = [0, n_o).  For each open channel j the solution has open parts
// s_i d_ij + c_i K_ij and closed parts e_i X_ij; the R-matrix relation
// u(a) = R a u'(a) becomes the linear system
//     (D1 - R D2) [K; X] = R[:, P] diag(a s'_P) - [diag(s_P); 0]
// with D1 = diag(c_P, e_Q), D2 = diag(a c'_P, a e'_Q) -- no division by any
// channel function.  Then, with K symmetrised,
//     (1 + K^2) Y = K,  Q = K Y,  T = 2(X - 1) + 2iY, X = (1 + K^2)^-1
// so |T_ij|^2 = 4 (Y_ij^2 + Q_ij^2), and
//     Omega(t, u) += (g/2) sum_{i in t, j in u, open} |T_ij|^2.
//
// Work is split into kernels along the steps, each a team per energy of one
// symmetry: assembly, LU, K and T with the collision strengths (or the
// photoionization amplitudes), and the T step's two rarer routes.  A kernel
// that held all of them called its routines out of line and spilled 2-6 KB a
// lane around the calls.  Symmetries run in a fixed order on one stream, and
// an energy's Omega row belongs to one team of a kernel, so the symmetries'
// sums need no atomics and have a fixed order.
//
// One wavefront per energy, looping over the whole chain, left each energy a
// serial walk through memory and a chunk as long as its slowest energies:
// 24.5 ms for 4096 energies at 200 channels, 69 ms for photoionization at
// 1000-channel sizes (15.2 of 87 ms were its pole sum).
#pragma once

#include <algorithm>

#include "chanfn.h"
#include "team.h"

namespace rmx {

// Residual of the matching system in FP64 for iterative refinement.  With R
// (n x n, leading dimension ld) and the current solution Z (n x no, ld),
//   B - M Z = R (D2 Z + E) - [diag(s); 0] - D1 Z,   E_kj = a s'_j [k == j],
// from the channel slots (d1, d2, s, a s'), so neither M nor B is kept.  R W
// runs as 16x16x4 FP64 MFMAs over 32 x 32 output tiles with W formed in the
// fragment loads; the residual goes to `out` (FP32, leading dimension ldo).
// Returns max |r| (team-uniform).
template <int NW>
__device__ __forceinline__ double team_residual(const RM_G double *Rm, int ld, const RM_G double *Z,
                                const RM_G ChanSlot *ch, int n, int no,
                                RM_G float *out, int ldo, RM_L TeamLds<NW> &W) {
  ld = uni(ld); n = uni(n); no = uni(no); ldo = uni(ldo);
  const int lane = lane_id();
  const int col = lane & 15, kq = lane >> 4;
  const int nct = (no + 31) >> 5, ntile = ((n + 31) >> 5) * nct;
  double rmax = 0.0;
  for (int t = team_wave<NW>(); t < ntile; t += NW) {
    const int rb = (t / nct) * 32, cb = (t % nct) * 32;
    d4 acc[2][2];
#pragma unroll
    for (int x = 0; x < 2; ++x)
#pragma unroll
      for (int y = 0; y < 2; ++y) acc[x][y] = d4{0.0, 0.0, 0.0, 0.0};
    for (int k0 = 0; k0 < n; k0 += 16) {
      double a[4][2], b[4][2];
#pragma unroll
      for (int s4 = 0; s4 < 4; ++s4) {
        const int k = k0 + 4 * s4 + kq;
        const bool kv = k < n;
        const double d2 = kv ? ch[k].d2 : 0.0;
        const double asp = kv ? ch[k].asp : 0.0;
#pragma unroll
        for (int x = 0; x < 2; ++x) {
          const int i = rb + 16 * x + col;
          a[s4][x] = (kv && i < n) ? Rm[(int64_t)i * ld + k] : 0.0;
          const int j = cb + 16 * x + col;
          const double z = (kv && j < no) ? Z[(int64_t)k * ld + j] : 0.0;
          b[s4][x] = (kv && j < no) ? fma(d2, z, k == j ? asp : 0.0) : 0.0;
        }
      }
#pragma unroll
      for (int s4 = 0; s4 < 4; ++s4)
#pragma unroll
        for (int x = 0; x < 2; ++x)
#pragma unroll
          for (int y = 0; y < 2; ++y)
            acc[x][y] = __builtin_amdgcn_mfma_f64_16x16x4f64(
                a[s4][x], b[s4][y], acc[x][y], 0, 0, 0);
    }
#pragma unroll
    for (int x = 0; x < 2; ++x)
#pragma unroll
      for (int y = 0; y < 2; ++y)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int i = rb + 16 * x + kq + 4 * r, j = cb + 16 * y + col;
          if (i >= n || j >= no) continue;
          const double z = Z[(int64_t)i * ld + j];
          double v = acc[x][y][r] - ch[i].d1 * z;
          if (i == j) v -= ch[i].s;
          rmax = fmax(rmax, fabs(v));
          out[(int64_t)i * ldo + j] = (float)v;
        }
  }
  rmax = team_max(rmax, W);
  team_sync<NW>();
  return rmax;
}

// Copy a rows x cols block (row-major source ld sl, destination ld dl).
template <int NW>
__device__ __forceinline__ void team_copy(RM_G double *dst, int dl, const RM_G double *src,
                                 int sl, int rows, int cols) {
  dl = uni(dl); sl = uni(sl); rows = uni(rows); cols = uni(cols);
  team_each<NW>(
      rows, cols, [&](int i, int j) { return src[(int64_t)i * sl + j]; },
      [&](int i, int j, double v) { dst[(int64_t)i * dl + j] = v; });
}

// ---------------------------------------------------------------------------
// T step by Cholesky.  T = 2iK (1 - iK)^-1 = 2(1 - iK)^-1 - 2 and
// (1 - iK)^-1 = (1 + iK)(1 + K^2)^-1, so with A = (1 + K^2)^-1 (K, A and
// K A are symmetric and commute)
//     Re T = -2 Q,  Q = K^2 A = 1 - A,     Im T = 2 Y,  Y = K A,
// and |T_ij|^2 = 4 (Y_ij^2 + Q_ij^2).  1 + K^2 is symmetric positive
// definite (eigenvalues 1 + k^2 >= 1): no pivoting, only its lower triangle
// is formed and factored, 1 + K^2 = L L^T.  A = L^-T L^-1 from the lower
// triangular L^-1 (forward substitution on the identity, each block only
// on the columns left of its end) and a product that starts each tile's sum
// at its first row; Y = K A with A read from its lower triangle.  That is
// (1 + 1/3 + 1/3 + 1/3 + 1) no^3 flops with the product 1 + K^2; the route
// Z = L^-1 K, Q = Z^T Z, Y = L^-T Z takes (1 + 1/3 + 1 + 1 + 1) no^3.
// Off the diagonal Q = -A exactly; on it Q_ii = 1 - A_ii, whose absolute
// error (unit roundoff) matters only where Q_ii itself is that small.
// Forming 1 + K^2 squares the condition number of 1 - iK, and the product
// K A multiplies the rounding of A by |K|: this route's error grows as the
// square of K's largest row norm (about 3e-17 |K|_row^2 against the exact
// T, 1e-8 at 1e4, 3e-2 at 2.5e7, which a 1e5-point mesh reaches where an
// eigenphase is within ~1e-8 of pi/2).  Energies where 1 + K^2 has a
// diagonal entry (1 + that row norm squared) above kTInvMax instead solve
// (1 - iK) W = 1 directly, as the real system
//     [ 1  K ] [X]   [1]
//     [-K  1 ] [Y] = [0],    W = X + iY,  X = A,  Y = K A,
// by the team's LU with partial pivoting: its condition number is that
// of 1 - iK, about |K|, so the error stays near u |K| (6e-10 at 7e7 in an
// FP64 emulation).  That takes a slot of 6 n^2 doubles from the launch's
// pool; without one the energy takes the route through Z = L^-1 K
// (Q = Z^T Z, Y = L^-T Z), whose error grows more slowly than the A route's
// but still with |K|^2.  At 200 channels about 0.5 % of a uniform mesh's
// energies are above the threshold.
constexpr double kTInvMax = 1e8;

// Factor the jb x jb (jb <= 32) diagonal block at (j0, j0) of A = L L^T in
// registers: lane i holds row i; per column, a broadcast of the diagonal and
// of the column, no memory round trip.  Rows and columns past jb are the
// identity, so nothing in the loop depends on jb.  Writes L11 back (lower
// triangle with its diagonal) and stages it in T for inversion.  One
// wavefront, no barrier.  Returns 1 if a diagonal was not positive.
__device__ __forceinline__ int wave_chol_diag(RM_G double *A, int ld, int j0,
                                              int jb,
                                              RM_L double (*T)[NB2 + 1]) {
  ld = uni(ld); j0 = uni(j0); jb = uni(jb);
  const int lane = lane_id();
  double x[NB2];  // row `lane` of the block
#pragma unroll
  for (int k = 0; k < NB2; ++k)
    x[k] = (lane < jb && k <= lane) ? A[(int64_t)(j0 + lane) * ld + j0 + k]
           : k == lane              ? 1.0
                                    : 0.0;
  int flag = 0;
  // 8 columns per turn at register indices 0..7, then the registers rotate
#pragma unroll 1
  for (int g = 0; g < 4; ++g) {
#pragma unroll
    for (int jj = 0; jj < 8; ++jj) {
      const int j = 8 * g + jj;
      const double djj = read_lane(x[jj], j);
      if (!(djj > 0.0)) flag = 1;
      const double d = sqrt(djj), rd = 1.0 / d;
      const double lij = lane > j ? x[jj] * rd : lane == j ? d : x[jj];
      x[jj] = lij;
#pragma unroll
      for (int b = 0; b < 4; ++b) {
        if (b > 0 && g + b >= 4) continue;  // uniform: done columns
#pragma unroll
        for (int q = b == 0 ? jj + 1 : 8 * b; q < 8 * b + 8; ++q) {
          const double lkj = read_lane(lij, 8 * g + q);  // L[k][j]
          if (lane >= 8 * g + q) x[q] = fma(-lij, lkj, x[q]);
        }
      }
    }
    double k[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) k[q] = x[q];
#pragma unroll
    for (int q = 0; q < 24; ++q) x[q] = x[q + 8];
#pragma unroll
    for (int q = 0; q < 8; ++q) x[24 + q] = k[q];
  }
#pragma unroll
  for (int k = 0; k < NB2; ++k)
    if (lane < jb && k <= lane) A[(int64_t)(j0 + lane) * ld + j0 + k] = x[k];
  if (lane < NB2) {
#pragma unroll
    for (int k = 0; k < NB2; ++k) T[lane][k] = k <= lane ? x[k] : 0.0;
  }
  return flag;
}

// Rows [r0, r1) of columns [j0, j0 + jb): X <- X Ti^T (the panel of a
// Cholesky factor, L21 = A21 L11^-T), 16 rows at a time as FP64 MFMA
// blocks; each row block is loaded whole before it is stored.
template <int NW>
__device__ __forceinline__ void team_rows_times_tit(RM_G double *A, int ld, int r0, int r1, int j0,
                                    int jb, const RM_L TeamLds<NW> &W) {
  ld = uni(ld); r0 = uni(r0); r1 = uni(r1); j0 = uni(j0); jb = uni(jb);
  const int lane = lane_id();
  const int col = lane & 15, kq = lane >> 4;
  double b[2][8];  // B[k][j] = Ti[j][k], j = 16 cb + col, k = 4 s + kq
#pragma unroll
  for (int cb = 0; cb < 2; ++cb)
#pragma unroll
    for (int s = 0; s < 8; ++s) b[cb][s] = W.Ti[16 * cb + col][4 * s + kq];
  for (int rb = r0 + team_wave<NW>() * 32; rb < r1; rb += NW * 32) {
    double a[2][8];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int r = rb + 16 * h + col;
#pragma unroll
      for (int s = 0; s < 8; ++s) {
        const int k = 4 * s + kq;
        a[h][s] = (r < r1 && k < jb) ? A[(int64_t)r * ld + j0 + k] : 0.0;
      }
    }
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      d4 acc[2];
#pragma unroll
      for (int cb = 0; cb < 2; ++cb) acc[cb] = d4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
      for (int s = 0; s < 8; ++s)
#pragma unroll
        for (int cb = 0; cb < 2; ++cb)
          acc[cb] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[h][s], b[cb][s],
                                                         acc[cb], 0, 0, 0);
#pragma unroll
      for (int cb = 0; cb < 2; ++cb)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int row = rb + 16 * h + kq + 4 * r, j = 16 * cb + col;
          if (row < r1 && j < jb) A[(int64_t)row * ld + j0 + j] = acc[cb][r];
        }
    }
  }
  team_sync<NW>();
}

// One block step of the Cholesky factorisation: the diagonal block factored and
// inverted (W.Ti) by the first wavefront, then the panel below it.
template <int NW>
__device__ __forceinline__ int team_chol_block(RM_G double *A, int ld, int j0,
                                               int jb, int na,
                                               RM_L TeamLds<NW> &W) {
  ld = uni(ld); j0 = uni(j0); jb = uni(jb); na = uni(na);
  int flag = 0;
  if (team_wave<NW>() == 0) {
    flag = wave_chol_diag(A, ld, j0, jb, W.T);
    wave_sync();
    wave_tile_invert<TILE_LOWER>(
        W.T, [&](int i, int j, double v) { W.Ti[i][j] = v; });
  }
  team_sync<NW>();
  if (j0 + jb < na) team_rows_times_tit<NW>(A, ld, j0 + jb, na, j0, jb, W);
  return flag;
}

// Photoionization: one block step of the forward substitution y = L^-1 v
// of the dipole amplitudes v (no entries, global memory), with Ti = L11^-1
// of the block in W: y_b = Ti v_b (first wavefront), then v[r] -= L[r][b] y_b
// below it.  y_b is broadcast through the first row of W.T, free once Ti is
// formed.
template <int NW>
__device__ __forceinline__ void team_photo_forward(const RM_G double *Aug, int ld, int j0, int jb,
                                   int no, RM_L TeamLds<NW> &W, RM_G double *v) {
  ld = uni(ld); j0 = uni(j0); jb = uni(jb); no = uni(no);
  const int lane = lane_id();
  if (team_wave<NW>() == 0) {
    const double vb = lane < jb ? v[j0 + lane] : 0.0;
    double y = 0.0;
#pragma unroll
    for (int k = 0; k < NB2; ++k)
      y = fma(W.Ti[lane & (NB2 - 1)][k], read_lane(vb, k), y);
    y = lane < jb ? y : 0.0;
    if (lane < NB2) W.T[0][lane] = y;
    if (lane < jb) v[j0 + lane] = y;
  }
  team_sync<NW>();
  for (int r = j0 + jb + team_tid<NW>(); r < no; r += WT * NW) {
    const RM_G double *Lr = Aug + (int64_t)r * ld + j0;
    double acc = v[r];
#pragma unroll
    for (int k0 = 0; k0 < NB2; k0 += 8) {
      double lv[8];
#pragma unroll
      for (int k = 0; k < 8; ++k) lv[k] = k0 + k < jb ? Lr[k0 + k] : 0.0;
#pragma unroll
      for (int k = 0; k < 8; ++k) acc = fma(-lv[k], W.T[0][k0 + k], acc);
    }
    v[r] = acc;
  }
  team_sync<NW>();
}

// ---------------------------------------------------------------------------
// Collision strengths.
//
// V_ij = Y_ij^2 + Q_ij^2 over the open block; Omega(t, u) += 2g sum_{i in t,
// j in u} V_ij.  When every target level holds one channel the sum is a
// relabelling of V's upper triangle; otherwise it is G^T V G with the 0/1
// channel-to-level matrix G (two MFMA products).

__device__ inline int64_t omega_index(int t, int u, int n_out) {
  if (t > u) {
    const int x = t;
    t = u;
    u = x;
  }
  return (int64_t)t * n_out - ((int64_t)t * (t - 1)) / 2 + (u - t);
}

// The lower triangles of Y (leading dimension ldy) and of Q, or of A with
// Q = 1 - A (q_is_a), in Qm (ldq) over the open block in; V (ldv, disjoint
// from both) is scratch, and so is Qm once V is formed.  Returns 1 if a
// contribution was not finite.
template <int NW>
__device__ __forceinline__ int team_omega(const SymDev &S, int n_out, const RM_G double *Y, int ldy,
                          RM_G double *Qm, int ldq, bool q_is_a, RM_G double *V, int ldv,
                          int no, RM_G double *om) {
  n_out = uni(n_out); ldy = uni(ldy); ldq = uni(ldq); ldv = uni(ldv); no = uni(no);
  const double g2 = 2.0 * S.g;
  int nonfinite = 0;
  if (uni(S.ntu) == uni(S.n)) {
    // one channel per level: walk the open block's lower triangle, a row of
    // it per wavefront (consecutive lanes read consecutive elements)
    for (int i = team_wave<NW>(); i < no; i += NW) {
      const int ti = S.tgt[i];
      const RM_G double *yr = Y + (int64_t)i * ldy;
      const RM_G double *qr = Qm + (int64_t)i * ldq;
      for (int j0 = lane_id(); j0 <= i; j0 += UNR * WT) {
        double yv[UNR], qv[UNR], ov[UNR];
        int64_t oi[UNR];
#pragma unroll
        for (int u = 0; u < UNR; ++u) {
          const int j = min(j0 + u * WT, i);
          const double qa = qr[j];
          qv[u] = q_is_a ? (i == j ? 1.0 : 0.0) - qa : qa;
          yv[u] = yr[j];
          oi[u] = omega_index(S.tgt[j], ti, n_out);
          ov[u] = om[oi[u]];
        }
#pragma unroll
        for (int u = 0; u < UNR; ++u) {
          if (j0 + u * WT > i) continue;
          const double v = g2 * (yv[u] * yv[u] + qv[u] * qv[u]);
          if (!isfinite(v)) nonfinite = 1;
          om[oi[u]] = ov[u] + v;
        }
      }
    }
    return nonfinite;
  }
  // V, both triangles, from the lower ones
  for (int i = team_wave<NW>(); i < no; i += NW) {
    const RM_G double *yr = Y + (int64_t)i * ldy;
      const RM_G double *qr = Qm + (int64_t)i * ldq;
    for (int j0 = lane_id(); j0 <= i; j0 += UNR * WT) {
      double v[UNR];
#pragma unroll
      for (int u = 0; u < UNR; ++u) {
        const int j = min(j0 + u * WT, i);
        const double qa = qr[j], y = yr[j];
        const double q = q_is_a ? (i == j ? 1.0 : 0.0) - qa : qa;
        v[u] = y * y + q * q;
      }
#pragma unroll
      for (int u = 0; u < UNR; ++u) {
        const int j = j0 + u * WT;
        if (j > i) continue;
        V[(int64_t)i * ldv + j] = v[u];
        V[(int64_t)j * ldv + i] = v[u];
      }
    }
  }
  team_sync<NW>();
  const int nt = uni(S.ntu);
  // W1 = G^T V (nt x no) into Qm's place, then Omega_u = W1 G (nt x nt) into V
  team_gemm<NW, 2>(Qm, ldq, as_g(S.GT), S.n, V, ldv, nt, no, no);
  team_gemm<NW, 2>(V, ldv, Qm, ldq, as_g(S.G), nt, nt, nt, no);
  for (int a = team_wave<NW>(); a < nt; a += NW) {
    const int ta = S.ut[a];
    for (int c = a + lane_id(); c < nt; c += WT) {
      const int64_t oi = omega_index(ta, S.ut[c], n_out);
      const double v = g2 * V[(int64_t)a * ldv + c];
      if (!isfinite(v)) nonfinite = 1;
      om[oi] += v;
    }
  }
  return nonfinite;
}

// Channel functions of symmetry S at energy Ee into ch[0..n), sorted order.
template <int NW>
__device__ __forceinline__ int team_channel_functions(const SymDev &S, double Ee,
                                      RM_G ChanSlot *ch) {
  int bits = 0;
  const int n = uni(S.n);
  const double ra = S.r_match;
  for (int i = team_tid<NW>(); i < n; i += WT * NW) {
    const double diff = Ee - S.e_thr[i];
    ChanSlot c;
    if (diff > 0.0) {
      const OpenVals v = coulomb_open(S.l[i], S.z, sqrt(diff), ra);
      c.d1 = v.c;
      c.d2 = ra * v.cp;
      c.s = v.s;
      c.asp = ra * v.sp;
      if (!v.ok) bits |= RM_E_CF_NOCONV;
    } else if (diff < 0.0) {
      const ClosedVals v = whittaker_closed(S.l[i], S.z, sqrt(-diff), ra);
      c.d1 = v.e;
      c.d2 = v.ep;
      c.s = 0.0;
      c.asp = 0.0;
      if (!v.ok) bits |= RM_E_CF_NOCONV;
    } else {
      c.d1 = 1.0;
      c.d2 = 0.0;
      c.s = 0.0;
      c.asp = 0.0;
      bits |= RM_E_ON_THRESHOLD;
    }
    ch[i].d1 = c.d1;
    ch[i].d2 = c.d2;
    ch[i].s = c.s;
    ch[i].asp = c.asp;
  }
  return bits;
}

__device__ inline int count_open(const SymDev &S, double Ee) {
  int lo = 0, hi = S.n;  // thresholds strictly below E
  while (lo < hi) {
    const int mid = (lo + hi) >> 1;
    if (S.e_thr[mid] < Ee)
      lo = mid + 1;
    else
      hi = mid;
  }
  return uni(lo);
}

// [D1 - R D2 | R[:, P] diag(a s'_P) - diag(s_P)] from R in Aug's left half.
template <int NW>
__device__ __forceinline__ void team_assemble(RM_G double *Aug, int ld, const RM_G ChanSlot *ch,
                                     int n, int no) {
  ld = uni(ld); n = uni(n); no = uni(no);
  team_each<NW>(
      n, n, [&](int i, int j) { return Aug[(int64_t)i * ld + j]; },
      [&](int i, int j, double r) {
        Aug[(int64_t)i * ld + j] = (i == j ? ch[i].d1 : 0.0) - r * ch[j].d2;
        if (j < no)
          Aug[(int64_t)i * ld + n + j] = r * ch[j].asp - (i == j ? ch[i].s : 0.0);
      });
}

// The matching solve with an FP32 factorisation refined in FP64: [M | B]
// rounded to FP32 in K's place (n x 2n floats), factored and solved there;
// the solution Z in FP64 in Aug's right half, then per iteration the FP64
// residual (team_residual, from R kept in Aug's left half) solved with the
// FP32 factors and added to Z.  Converged when a correction is below the
// rounding of Z (max|dZ| <= 2^-50 max|Z|), or when the corrections stop
// contracting (max|dZ| over half the previous one) at a residual that passes
// the backward-error test of LAPACK's mixed-precision dsgesv, max|r| <=
// 4 sqrt(n) u ||M||_inf max|Z| (u = 2^-53): the floor that the system's
// conditioning sets in FP64.  Otherwise, after refine_iters corrections,
// the energy is flagged RM_E_REFINE_NOCONV and left assembled for the FP64
// factorisation.  Returns RM_E_* bits.
template <int NW, int NAMAX>
__device__ __forceinline__ int team_solve_fp32(int refine_iters, int n,
                               RM_G double *Aug, RM_G double *Kb, const RM_G ChanSlot *ch,
                               int no, RM_L TeamLds<NW> &W) {
  refine_iters = uni(refine_iters); n = uni(n); no = uni(no);
  const int tid = team_tid<NW>();
  const int ld = 2 * n, ld32 = 2 * n;
  RM_G float *A32 = (RM_G float *)Kb;
  RM_G int *piv = (RM_G int *)(Aug + (int64_t)3 * n * n + 2 * n);
  int bits = 0;
  team_each<NW>(
      n, n, [&](int i, int j) { return Aug[(int64_t)i * ld + j]; },
      [&](int i, int j, double r) {
        A32[(int64_t)i * ld32 + j] =
            (float)((i == j ? ch[i].d1 : 0.0) - r * ch[j].d2);
        if (j < no)
          A32[(int64_t)i * ld32 + n + j] =
              (float)(r * ch[j].asp - (i == j ? ch[i].s : 0.0));
      });
  // ||M||_inf from the FP64 entries (row sums of |d1 - R d2|)
  double anrm = 0.0;
  for (int i = tid; i < n; i += WT * NW) {
    double rs = 0.0;
    for (int j = 0; j < n; ++j)
      rs += fabs((i == j ? ch[i].d1 : 0.0) - Aug[(int64_t)i * ld + j] * ch[j].d2);
    anrm = fmax(anrm, rs);
  }
  anrm = team_max(anrm, W);
  team_sync<NW>();
  if (team_lu_solve<NW, NAMAX>(A32, n, ld32, no, W, piv)) bits |= RM_E_SINGULAR;
  // Z in FP64
  double zmax = 0.0;
  team_each<NW>(
      n, no, [&](int i, int j) { return (double)A32[(int64_t)i * ld32 + n + j]; },
      [&](int i, int j, double z) {
        Aug[(int64_t)i * ld + n + j] = z;
        zmax = fmax(zmax, fabs(z));
      });
  zmax = team_max(zmax, W);
  team_sync<NW>();
  const double tol = 4.0 * sqrt((double)n) * 0x1p-53 * anrm;
  bool conv = false;
  double dprev = 1e300;
  double rmax = team_residual(Aug, ld, Aug + n, ch, n, no, A32 + n, ld32, W);
  for (int it = 0; it < refine_iters; ++it) {
    if (uni(rmax == 0.0)) {
      conv = true;
      break;
    }
    if (uni(!(rmax < 1e300))) break;  // not finite
    team_lu_resolve(A32, n, ld32, no, piv, W);
    double dmax = 0.0;
    zmax = 0.0;
    team_each<NW>(
        n, no,
        [&](int i, int j) {
          return make_double2((double)A32[(int64_t)i * ld32 + n + j],
                              Aug[(int64_t)i * ld + n + j]);
        },
        [&](int i, int j, double2 v) {
          const double z = v.y + v.x;
          Aug[(int64_t)i * ld + n + j] = z;
          zmax = fmax(zmax, fabs(z));
          dmax = fmax(dmax, fabs(v.x));
        });
    zmax = team_max(zmax, W);
    dmax = team_max(dmax, W);
    team_sync<NW>();
    // the correction is below the rounding of Z itself
    if (uni(dmax <= 0x1p-50 * zmax)) {
      conv = true;
      break;
    }
    rmax = team_residual(Aug, ld, Aug + n, ch, n, no, A32 + n, ld32, W);
    // corrections no longer contract: the FP64 floor of this system, if the
    // residual passes the backward-error test there
    if (uni(dmax > 0.5 * dprev)) {
      conv = uni(rmax <= tol * zmax);
      break;
    }
    dprev = dmax;
  }
  // otherwise the system is assembled again in FP64 from R, still in Aug's
  // left half, for the FP64 factorisation, as LAPACK's dsgesv does: the FP32
  // factors cannot refine it (cond(M) u_32 near 1, e.g. within ~1e-6 Ry of a
  // pole at 200 channels)
  if (!conv) {
    bits |= RM_E_REFINE_NOCONV;
    team_assemble<NW>(Aug, ld, ch, n, no);
  }
  return bits;
}

// Radiation-damped photoionization: the driven system of one energy.  With the
// pole energies E_k - i Gamma_k/2 the pole sums are complex, R_c = R_re +
// i R_im and g_c = g_re + i g_im (the pole-sum kernels' parts 1 and 2), and
// the driven solution of (E - H_eff) psi = D Psi_0 with outgoing waves
// outside satisfies
//     (diag(d1) - R_c diag(d2)) x = -g_c,
// d1 = c + i s, d2 = a (c' + i s') on open channels (u = (c + i s) alpha)
// and the closed function (e, a e') on closed ones; its flux into the open
// channels is sum_f |alpha_f|^2 (c s' - s c' = 1), and sigma +=
// (4 pi alpha a0^2 / 3) omega sum_f |alpha_f|^2.  The complex system is
// solved as the real 2n x 2n system [[A_r, -A_i], [A_i, A_r]] [x_r; x_i] =
// [-g_re; -g_im] by the team's LU.
template <int NW>
__device__ __forceinline__ void team_assemble_damped(RM_G double *Sys,
                                                     const RM_G ChanSlot *ch,
                                                     int n) {
  n = uni(n);
  const int n2 = 2 * n, ld = 2 * n + 2;
  const RM_G double *Rre = Sys + (int64_t)n2 * ld;
  const RM_G double *Rim = Rre + (int64_t)n * n;
  const RM_G double *gre = Rim + (int64_t)n * n;
  const RM_G double *gim = gre + n;
  team_each<NW>(
      n, n,
      [&](int i, int j) {
        return make_double2(Rre[(int64_t)i * n + j], Rim[(int64_t)i * n + j]);
      },
      [&](int i, int j, double2 r) {
        const double d2 = ch[j].d2, asp = ch[j].asp;
        const double ar =
            (i == j ? ch[i].d1 : 0.0) - (r.x * d2 - r.y * asp);
        const double ai = (i == j ? ch[i].s : 0.0) - (r.x * asp + r.y * d2);
        Sys[(int64_t)i * ld + j] = ar;
        Sys[(int64_t)i * ld + n + j] = -ai;
        Sys[(int64_t)(n + i) * ld + j] = ai;
        Sys[(int64_t)(n + i) * ld + n + j] = ar;
      });
  for (int i = team_tid<NW>(); i < n; i += WT * NW) {
    Sys[(int64_t)i * ld + n2] = -gre[i];
    Sys[(int64_t)(n + i) * ld + n2] = -gim[i];
  }
}


// ---------------------------------------------------------------------------
// Kernels.  blockIdx.x is the energy (but for the routes by list), L.sym the
// symmetry.

// Where symmetry S's data of energy e sit.
struct Place {
  RM_G double *work;
  RM_G ChanSlot *ch;
  RM_G int *flag;  // the energy's route
};
__device__ inline Place place_of(const MatchLaunch &L, const SymDev &S, int sym,
                                 int e) {
  Place p;
  p.work = as_g(L.work + (int64_t)e * L.work_estride + L.work_off[sym]);
  p.ch = as_g(L.chan + (int64_t)e * L.chan_estride + L.chan_off[sym]);
  p.flag = as_g(L.route) + (int64_t)sym * L.m + e;
  return p;
}

__device__ inline void put_status(const MatchLaunch &L, int e, int bits) {
  bits = wave_or(bits);
  if (lane_id() == 0 && L.status && bits) atomicOr(&L.status[e], bits);
}

// Channel functions and the matching system of one energy, or the driven
// system of the damped photoionization, in place of R.  (With the asymptotic
// expansion the system at A is already there; the FP32 solve assembles its
// own.)
template <int NW, bool DAMPED>
__global__ __launch_bounds__(WT *NW) void assemble_kernel(MatchLaunch L) {
  const SymDev &S = L.syms[L.sym];
  const int e = blockIdx.x, n = S.n;
  const Place P = place_of(L, S, L.sym, e);
  const double Ee = L.E[e];
  const int no = count_open(S, Ee);
  if (L.n_open_out && threadIdx.x == 0) L.n_open_out[e] = no;
  if (no == 0) {
    put_status(L, e, RM_E_NO_OPEN);
    return;
  }
  if (uni(S.gl_terms) > 0) return;
  const int bits = team_channel_functions<NW>(S, Ee, P.ch);
  team_sync<NW>();
  if constexpr (DAMPED)
    team_assemble_damped<NW>(P.work, P.ch, n);
  else if (!L.solve_fp32)
    team_assemble<NW>(P.work, 2 * n, P.ch, n, no);
  put_status(L, e, bits);
}

// The LU solve of the assembled systems.
template <int NW, int NAMAX>
__global__ __launch_bounds__(WT *NW) __attribute__((amdgpu_waves_per_eu(2, 2)))
void lu_kernel(MatchLaunch L) {
  __shared__ TeamLds<NW> lds;
  RM_L TeamLds<NW> &W = *(RM_L TeamLds<NW> *)&lds;
  const SymDev &S = L.syms[L.sym];
  const int e = blockIdx.x, n = S.n;
  const Place P = place_of(L, S, L.sym, e);
  const int no = count_open(S, L.E[e]);
  if (no == 0) return;
  if (L.solve_fp32 && uni(*P.flag) == 0) return;  // refined from FP32 factors
  const int na = L.damped ? 2 * n : n, ld = L.damped ? 2 * n + 2 : 2 * n;
  const int f = team_lu_solve<NW, NAMAX>(P.work, na, ld, L.damped ? 1 : no, W);
  put_status(L, e, f ? RM_E_SINGULAR : 0);
}

// The FP32 solve refined in FP64; flags the energies it could not refine.
template <int NW, int NAMAX>
__global__ __launch_bounds__(WT *NW) __attribute__((amdgpu_waves_per_eu(2, 2)))
void solve_fp32_kernel(MatchLaunch L) {
  __shared__ TeamLds<NW> lds;
  RM_L TeamLds<NW> &W = *(RM_L TeamLds<NW> *)&lds;
  const SymDev &S = L.syms[L.sym];
  const int e = blockIdx.x, n = S.n;
  const Place P = place_of(L, S, L.sym, e);
  const int no = count_open(S, L.E[e]);
  if (no == 0) return;
  const int bits = team_solve_fp32<NW, NAMAX>(
      L.refine_iters, n, P.work, P.work + (int64_t)2 * n * n, P.ch, no, W);
  if (threadIdx.x == 0) *P.flag = (bits & RM_E_REFINE_NOCONV) ? 1 : 0;
  put_status(L, e, bits);
}

// K = sym(Z[0:no, 0:no]) into its place, or K gathered from the caller's.
// Input order of the open channels: rank[i] is the rank of open channel i
// among the open channels' input indices.
template <int NW>
__device__ __forceinline__ void team_rank(const SymDev &S, int no,
                                          RM_G int *rank) {
  no = uni(no);
  for (int i = team_tid<NW>(); i < no; i += WT * NW) {
    const int pi = S.perm[i];
    int r = 0;
#pragma unroll 8
    for (int j = 0; j < no; ++j) r += (S.perm[j] < pi);
    rank[i] = r;
  }
  team_sync<NW>();
}

template <int NW>
__device__ __forceinline__ void team_k_sym(RM_G double *Kb, int n, int no,
                                           const RM_G double *Z, int ld) {
  n = uni(n); no = uni(no); ld = uni(ld);
  team_each<NW>(
      no, no,
      [&](int i, int j) {
        return make_double2(Z[(int64_t)i * ld + j], Z[(int64_t)j * ld + i]);
      },
      [&](int i, int j, double2 z) {
        Kb[(int64_t)i * n + j] = 0.5 * (z.x + z.y);
      });
}

// K to the caller, zeros outside the open block.
template <int NW>
__global__ __launch_bounds__(WT *NW) void k_out_kernel(MatchLaunch L) {
  const SymDev &S = L.syms[L.sym];
  const int e = blockIdx.x, n = S.n, ld = 2 * n;
  const Place P = place_of(L, S, L.sym, e);
  const int no = count_open(S, L.E[e]);
  RM_G int *rank = (RM_G int *)P.ch;  // the channel slots are consumed
  RM_G double *Ko = as_g(L.K_out + (int64_t)e * n * n);
  team_rank<NW>(S, no, rank);
  const RM_G double *Z = P.work + n;
  int nonfinite = 0;
  team_each<NW>(
      n, n,
      [&](int i, int j) {
        return i < no && j < no
                   ? 0.5 * (Z[(int64_t)i * ld + j] + Z[(int64_t)j * ld + i])
                   : 0.0;
      },
      [&](int i, int j, double v) {
        const bool in = i < no && j < no;
        if (in && !isfinite(v)) nonfinite = 1;
        Ko[(int64_t)(in ? rank[i] : i) * n + (in ? rank[j] : j)] = v;
      });
  put_status(L, e, nonfinite ? RM_E_NONFINITE : 0);
}

// K, the T step's main route and Omega of one energy.  Energies above
// kTInvMax are left to the kernels below, with K in place and their flag set.
template <int NW>
__global__ __launch_bounds__(WT *NW) __attribute__((amdgpu_waves_per_eu(2, 2)))
void t_kernel(MatchLaunch L) {
  __shared__ TeamLds<NW> lds;
  RM_L TeamLds<NW> &W = *(RM_L TeamLds<NW> *)&lds;
  const SymDev &S = L.syms[L.sym];
  const int e = blockIdx.x, n = S.n, ld = 2 * n, tid = team_tid<NW>();
  const Place P = place_of(L, S, L.sym, e);
  const int no = count_open(S, L.E[e]);
  if (no == 0) {
    if (tid == 0) *P.flag = 0;
    return;
  }
  RM_G double *Aug = P.work, *Kb = P.work + (int64_t)2 * n * n;
  if (L.K_in) {
    const RM_G double *Ki = as_g(L.K_in + (int64_t)e * n * n);
    RM_G int *rank = (RM_G int *)P.ch;
    team_rank<NW>(S, no, rank);
    team_each<NW>(
        no, no, [&](int i, int j) { return Ki[(int64_t)rank[i] * n + rank[j]]; },
        [&](int i, int j, double v) { Kb[(int64_t)i * n + j] = v; });
  } else {
    team_k_sym<NW>(Kb, n, no, Aug + n, ld);
  }
  team_sync<NW>();
  // lower triangle of 1 + K^2; the route by its largest diagonal entry
  // 1 + sum_j K_ij^2 (team-uniform)
  team_gemm_wide<NW, 1, G_LOWER, 2, 4>(Aug, ld, Kb, n, Kb, n, no, no, no);
  double gmax = 0.0;
  for (int i = tid; i < no; i += WT * NW)
    gmax = fmax(gmax, Aug[(int64_t)i * ld + i]);
  gmax = team_max(gmax, W);
  const bool inv = uni(gmax <= kTInvMax);
  if (tid == 0) *P.flag = inv ? 0 : 1;
  if (!inv) return;
  // right-looking blocked Cholesky with the forward substitution on the
  // identity, whose rows of block b have nonzeros only left of the block's end
  team_each<NW>(
      no, no, [&](int i, int j) { return i == j ? 1.0 : 0.0; },
      [&](int i, int j, double v) { Aug[(int64_t)i * ld + no + j] = v; });
  team_sync<NW>();
  int bits = 0;
  for (int j0 = 0; j0 < no; j0 += NB2) {
    const int jb = min(NB2, no - j0), r0 = j0 + jb;
    if (team_chol_block<NW>(Aug, ld, j0, jb, no, W)) bits |= RM_E_SINGULAR;
    team_tile_apply<NW>(Aug, ld, j0, jb, no, no + r0, W, false);
    if (r0 < no) {
      team_gemm_wide<NW, 0, G_TB | G_LOWER, 2, 4>(
          Aug + (int64_t)r0 * ld + r0, ld, Aug + (int64_t)r0 * ld + j0, ld,
          Aug + (int64_t)r0 * ld + j0, ld, no - r0, no - r0, jb);
      team_gemm_wide<NW, 0, 0, 2, 4>(Aug + (int64_t)r0 * ld + no, ld,
                                     Aug + (int64_t)r0 * ld + j0, ld,
                                     Aug + (int64_t)j0 * ld + no, ld, no - r0,
                                     r0, jb);
    }
  }
  // A = (L^-1)^T L^-1, lower triangle, over L's place
  team_gemm_wide<NW, 2, G_TA | G_LOWER | G_KTRI, 2, 4>(
      Aug, ld, Aug + no, ld, Aug + no, ld, no, no, no);
  // Y = K A, lower triangle, over L^-1's place
  team_gemm_wide<NW, 2, G_BSYM | G_LOWER, 2, 4>(Aug + no, ld, Kb, n, Aug, ld,
                                                no, no, no);
  if (team_omega<NW>(S, L.n_target_out, Aug + no, ld, Aug, ld, true, Kb, n, no,
                     as_g(L.omega + (int64_t)e * L.omega_stride)))
    bits |= RM_E_NONFINITE;
  put_status(L, e, bits);
}

// The T step's route for large K: (1 - iK) W = 1 as the real system
// [1 K; -K 1] [X; Y] = [1; 0] (2 no x 3 no, leading dimension 3 no) by the
// team's LU, in the pool's slot blockIdx.x, for every symmetry of the launch.
// A team alone on a CU is a serial chain (2.6 ms at 200 open channels, 6.3 at
// 400) and few energies take it, so what counts is that chains run side by
// side: the q-th energy of the chunk with a flag in any symmetry goes to slot
// q mod the slots, each team counting the flags for itself, and its symmetries
// follow each other in that team (one owner of the energy's Omega row).  With
// every slots-th energy to a slot, flagged or not, two of about twenty met at
// 200 channels, 5.2 ms of a 29 ms sweep; with a launch per symmetry a plan of
// eight symmetries up to 400 channels spent 20 ms here, now 12.3.  The flags lie
// together, 64 energies to two cache lines, since every team reads all of them.
template <int NW, int NAMAX>
__global__ __launch_bounds__(WT *NW) __attribute__((amdgpu_waves_per_eu(2, 2)))
void t_complex_kernel(MatchLaunch L) {
  __shared__ TeamLds<NW> lds;
  RM_L TeamLds<NW> &W = *(RM_L TeamLds<NW> *)&lds;
  const int m = L.m;
  RM_G double *ext = as_g(L.ext + (int64_t)blockIdx.x * L.ext_estride);
  constexpr int FB = 8;  // batches of 64 flags in flight
  int skip = blockIdx.x;  // flagged energies before this slot's next one
  unsigned long long flags = 0;
  int eb = -WT, cached = 0;
  unsigned int mine = 0;  // this lane's flags of the next `cached` batches
#pragma unroll 1
  for (;;) {
    // the next energy of this slot: skip flagged ones
    int e = -1;
#pragma unroll 1
    while (e < 0) {
      if (flags == 0) {
        eb += WT;
        if (eb >= m) break;
        if (cached == 0) {
          mine = 0;
#pragma unroll 1
          for (int q = 0; q < L.n_sym; ++q) {
            const RM_G int *route = as_g(L.route) + (int64_t)q * m;
#pragma unroll
            for (int u = 0; u < FB; ++u) {
              const int f = eb + u * WT + lane_id();
              mine |= (f < m && route[min(f, m - 1)] != 0 ? 1u : 0u) << u;
            }
          }
          cached = FB;
        }
        flags = __ballot(mine & 1u);
        mine >>= 1;
        --cached;
        continue;
      }
      const int have = __popcll(flags);
      if (have <= skip) {
        skip -= have;
        flags = 0;
        continue;
      }
      for (; skip > 0; --skip) flags &= flags - 1;
      e = eb + __builtin_ctzll(flags);
      flags &= flags - 1;
      skip = gridDim.x - 1;
    }
    e = uni(e);
    if (e < 0) break;
#pragma unroll 1
    for (int q = 0; q < L.n_sym; ++q) {
      const SymDev &S = L.syms[q];
      const Place P = place_of(L, S, q, e);
      if (uni(*P.flag) == 0) continue;
      const int n = uni(S.n), no = uni(count_open(S, L.E[e]));
      RM_G double *Kb = P.work + (int64_t)2 * n * n;
      const int l3 = 3 * no;
      team_each<NW>(
          no, no, [&](int i, int j) { return Kb[(int64_t)i * n + j]; },
          [&](int i, int j, double k) {
            const double one = i == j ? 1.0 : 0.0;
            RM_G double *r = ext + (int64_t)i * l3 + j;
            RM_G double *s = ext + (int64_t)(no + i) * l3 + j;
            r[0] = one;
            r[no] = k;
            r[2 * no] = one;
            s[0] = -k;
            s[no] = one;
            s[2 * no] = 0.0;
          });
      team_sync<NW>();
      int bits =
          team_lu_solve<NW, NAMAX>(ext, 2 * no, l3, no, W) ? RM_E_SINGULAR : 0;
      // X = A (rows [0, no)), Y (rows [no, 2 no)) of the solution; V in K's
      // place
      if (team_omega<NW>(S, L.n_target_out, ext + (int64_t)no * l3 + 2 * no, l3,
                         ext + 2 * no, l3, true, Kb, n, no,
                         as_g(L.omega + (int64_t)e * L.omega_stride)))
        bits |= RM_E_NONFINITE;
      put_status(L, e, bits);
      team_sync<NW>();
    }
  }
}

// The same energies where the pool has no slot for the symmetry: Cholesky
// 1 + K^2 = L L^T, Z = L^-1 K, Q = Z^T Z (= K^2 A), Y = L^-T Z.
template <int NW>
__global__ __launch_bounds__(WT *NW) __attribute__((amdgpu_waves_per_eu(2, 2)))
void t_z_kernel(MatchLaunch L) {
  __shared__ TeamLds<NW> lds;
  RM_L TeamLds<NW> &W = *(RM_L TeamLds<NW> *)&lds;
  const SymDev &S = L.syms[L.sym];
  const int e = blockIdx.x, n = S.n, ld = 2 * n;
  const Place P = place_of(L, S, L.sym, e);
  if (uni(*P.flag) == 0) return;
  const int no = count_open(S, L.E[e]);
  RM_G double *Aug = P.work, *Kb = P.work + (int64_t)2 * n * n;
  // 1 + K^2 is in Aug; the right-hand side is K
  team_copy<NW>(Aug + no, ld, Kb, n, no, no);
  team_sync<NW>();
  int bits = 0;
  for (int j0 = 0; j0 < no; j0 += NB2) {
    const int jb = min(NB2, no - j0), r0 = j0 + jb;
    if (team_chol_block<NW>(Aug, ld, j0, jb, no, W)) bits |= RM_E_SINGULAR;
    team_tile_apply<NW>(Aug, ld, j0, jb, no, 2 * no, W, false);
    if (r0 < no) {
      team_gemm_wide<NW, 0, G_TB | G_LOWER, 2, 4>(
          Aug + (int64_t)r0 * ld + r0, ld, Aug + (int64_t)r0 * ld + j0, ld,
          Aug + (int64_t)r0 * ld + j0, ld, no - r0, no - r0, jb);
      team_gemm_wide<NW, 0, 0, 2, 4>(Aug + (int64_t)r0 * ld + no, ld,
                                     Aug + (int64_t)r0 * ld + j0, ld,
                                     Aug + (int64_t)j0 * ld + no, ld, no - r0,
                                     no, jb);
    }
  }
  // Q in K's place, lower triangle
  team_gemm_wide<NW, 2, G_TA | G_LOWER, 2, 4>(Kb, n, Aug + no, ld, Aug + no, ld,
                                              no, no, no);
  // Y = L^-T Z, blocks from the bottom, left-looking as the LU's back
  // substitution: Z_b -= L[>b, b]^T Y[>b]
  for (int j0 = ((no - 1) / NB2) * NB2; j0 >= 0; j0 -= NB2) {
    const int jb = min(NB2, no - j0), r1 = j0 + jb;
    if (r1 < no)
      team_gemm_wide<NW, 0, G_TA, 2, 4>(Aug + (int64_t)j0 * ld + no, ld,
                                        Aug + (int64_t)r1 * ld + j0, ld,
                                        Aug + (int64_t)r1 * ld + no, ld, jb, no,
                                        no - r1);
    team_tile_stage<NW, false>(Aug, ld, j0, jb, W.T, TILE_LOWER);
    if (team_wave<NW>() == 0)
      wave_tile_invert<TILE_LOWER>(
          W.T, [&](int i, int j, double v) { W.Ti[i][j] = v; });
    team_sync<NW>();
    team_tile_apply<NW, true>(Aug, ld, j0, jb, no, 2 * no, W, false);
  }
  if (team_omega<NW>(S, L.n_target_out, Aug + no, ld, Kb, n, false, Aug, ld, no,
                     as_g(L.omega + (int64_t)e * L.omega_stride)))
    bits |= RM_E_NONFINITE;
  put_status(L, e, bits);
}

// Cross section in Mb per unit sum of squared amplitudes, (4 pi^2 alpha a0^2
// / 3) / pi.
constexpr double kSigma = 4.0 * 3.14159265358979323846 * 7.2973525693e-3 *
                          28.00285205 / 3.0;

// sigma[e] += kSigma omega s2 (one team per energy and symmetry in turn).
__device__ inline int add_sigma(const MatchLaunch &L, int e, double s2) {
  const double add = kSigma * (L.E[e] - L.e0) * s2;
  if (threadIdx.x == 0) L.sigma[e] += add;
  return isfinite(add) ? 0 : RM_E_NONFINITE;
}

// Photoionization: the dipole amplitudes v of the K-matrix solutions and
// |L^-1 v|^2 with 1 + K^2 = L L^T.  With u_ij'(a) = (a s'_j delta_ij + d2_i
// Z_ij) / a over every channel i (Z = [K; X]), v_j = sum_i u_ij'(a) g_i.
template <int NW>
__global__ __launch_bounds__(WT *NW) __attribute__((amdgpu_waves_per_eu(2, 2)))
void photo_kernel(MatchLaunch L) {
  __shared__ TeamLds<NW> lds;
  RM_L TeamLds<NW> &W = *(RM_L TeamLds<NW> *)&lds;
  const SymDev &S = L.syms[L.sym];
  const int e = blockIdx.x, n = S.n, ld = 2 * n, tid = team_tid<NW>();
  const Place P = place_of(L, S, L.sym, e);
  const int no = count_open(S, L.E[e]);
  if (no == 0) return;
  RM_G double *Aug = P.work, *Kb = P.work + (int64_t)2 * n * n;
  const RM_G double *g = Aug + (int64_t)3 * n * n;
  RM_G double *v = Aug + (int64_t)3 * n * n + n;
  team_k_sym<NW>(Kb, n, no, Aug + n, ld);
  for (int j = tid; j < no; j += WT * NW) {
    double acc = 0.0;
    for (int i0 = 0; i0 < n; i0 += 8) {
      double z[8], h[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const int i = min(i0 + u, n - 1);
        z[u] = Aug[(int64_t)i * ld + n + j];
        h[u] = i0 + u < n ? P.ch[i].d2 * g[i] : 0.0;
      }
#pragma unroll
      for (int u = 0; u < 8; ++u)
        if (i0 + u < n) acc = fma(h[u], z[u], acc);
    }
    v[j] = (P.ch[j].asp * g[j] + acc) / S.a;
  }
  team_sync<NW>();
  team_gemm_wide<NW, 1, G_LOWER, 2, 4>(Aug, ld, Kb, n, Kb, n, no, no, no);
  int bits = 0;
  for (int j0 = 0; j0 < no; j0 += NB2) {
    const int jb = min(NB2, no - j0), r0 = j0 + jb;
    if (team_chol_block<NW>(Aug, ld, j0, jb, no, W)) bits |= RM_E_SINGULAR;
    team_photo_forward(Aug, ld, j0, jb, no, W, v);
    if (r0 < no)
      team_gemm_wide<NW, 0, G_TB | G_LOWER, 2, 4>(
          Aug + (int64_t)r0 * ld + r0, ld, Aug + (int64_t)r0 * ld + j0, ld,
          Aug + (int64_t)r0 * ld + j0, ld, no - r0, no - r0, jb);
  }
  double s2 = 0.0;
  for (int j = tid; j < no; j += WT * NW) s2 = fma(v[j], v[j], s2);
  put_status(L, e, bits | add_sigma(L, e, team_sum(s2, W)));
}

// Damped photoionization: the flux of the solved driven system into the open
// channels.
template <int NW>
__global__ __launch_bounds__(WT *NW) void damped_sigma_kernel(MatchLaunch L) {
  __shared__ TeamLds<NW> lds;
  RM_L TeamLds<NW> &W = *(RM_L TeamLds<NW> *)&lds;
  const SymDev &S = L.syms[L.sym];
  const int e = blockIdx.x, n = S.n, ld = 2 * n + 2;
  const Place P = place_of(L, S, L.sym, e);
  const int no = count_open(S, L.E[e]);
  if (no == 0) return;
  double s2 = 0.0;
  for (int f = team_tid<NW>(); f < no; f += WT * NW) {
    const double xr = P.work[(int64_t)f * ld + 2 * n];
    const double xi = P.work[(int64_t)(n + f) * ld + 2 * n];
    s2 = fma(xr, xr, fma(xi, xi, s2));
  }
  put_status(L, e, add_sigma(L, e, team_sum(s2, W)));
}

// A step of the matching by teams of NW wavefronts (instantiated in a unit per
// team size, so that they compile side by side).
template <int NW, int NAMAX>
hipError_t launch_team(const MatchLaunch &L, MatchStep step, hipStream_t st) {
  const dim3 g(step == STEP_T_COMPLEX ? L.ext_slots : L.m), b(WT * NW);
  switch (step) {
    case STEP_ASSEMBLE:
      hipLaunchKernelGGL((assemble_kernel<NW, false>), g, b, 0, st, L);
      break;
    case STEP_ASSEMBLE_DAMPED:
      hipLaunchKernelGGL((assemble_kernel<NW, true>), g, b, 0, st, L);
      break;
    case STEP_LU:
      hipLaunchKernelGGL((lu_kernel<NW, NAMAX>), g, b, 0, st, L);
      break;
    case STEP_FP32:
      hipLaunchKernelGGL((solve_fp32_kernel<NW, NAMAX>), g, b, 0, st, L);
      break;
    case STEP_K_OUT:
      hipLaunchKernelGGL(k_out_kernel<NW>, g, b, 0, st, L);
      break;
    case STEP_T:
      hipLaunchKernelGGL(t_kernel<NW>, g, b, 0, st, L);
      break;
    case STEP_T_COMPLEX:
      hipLaunchKernelGGL((t_complex_kernel<NW, NAMAX>), g, b, 0, st, L);
      break;
    case STEP_T_Z:
      hipLaunchKernelGGL(t_z_kernel<NW>, g, b, 0, st, L);
      break;
    case STEP_PHOTO:
      hipLaunchKernelGGL(photo_kernel<NW>, g, b, 0, st, L);
      break;
    case STEP_DAMPED_SIGMA:
      hipLaunchKernelGGL(damped_sigma_kernel<NW>, g, b, 0, st, L);
      break;
  }
  return hipGetLastError();
}

}  // namespace rmx
