// FP64 pole sum over groups of 128 consecutive energies.
//
// R(E) = (1/2a) sum_k w_k w_k^T / (E_k - E).  Over a short stretch of energies
// [c - h, c + h] the poles far from it give a smooth function, and the
// interpolant through its values at the 16 Chebyshev points c + h x_i is that
// function to FP64 rounding: for one pole at c + z h the error relative to its
// term is T_16(x) / T_16(z), below 1.3e-17 for |z| >= 6 (damped poles lie off
// the real axis, which only helps).  So a group sums its far poles at 16
// points instead of at 128 energies, and each energy's R is the interpolant
// plus the few poles within 6 h.  At 200 channels, 8000 poles and a mesh step
// of 2e-4 that is 31 + 3 of 250 chunks' work per 16 energies.  The node values
// are sums of the same products in the same order as a direct sum; the squares
// of an energy's 16 weights sum to 1 on average and to less than 2 at the ends
// of the group, their magnitudes to less than 2.73.  So the far part is rounded
// like a direct sum of it, up to 1.4 times that at the ends, while the near part
// is shorter: against 80-bit sums R is off by 2.3e-15 (relative rms) where the
// direct kernel is off by 5.2e-15 (200 channels, 12400 damped poles).
// Groups are cut on the whole mesh, not on the chunk, so results do not depend
// on the chunk length; an energy's last bits do depend on its group, so on the
// energies beside it.
//
// Groups whose energies are not close together (unsorted, coarse, not finite)
// or too few to pay for 16 points are left to the direct kernel, which runs
// after this one and makes the same decision.
//
// A workgroup holds one 16 x 16 tile of the upper triangle: the far phase
// gives each wavefront four nodes, then the node values stay in LDS while 16
// energies at a time, four per wavefront, add the near poles.  Tiles of 16
// keep the node values at 32 KB of LDS, two workgroups per CU, and give a
// group of 200 channels 91 workgroups.  What bounds it is the FP64 matrix
// pipe, 64 cycles per 16x16x4.  Measured against the direct kernel: 200
// channels, 8000 poles, 4096 energies 5.2 ms, was 27.2;
// 400 channels, 512 energies 3.7 ms, was 20.2.
#include <algorithm>

#include "polesum_group.h"

namespace rmx {

typedef double d4 __attribute__((ext_vector_type(4)));

constexpr int PG_B = 16;     // energies per batch of the near phase
constexpr int PG_EW = 4;     // nodes or energies per wavefront

// cos((2 i + 1) pi / 32) and the barycentric weights (-1)^i sin((2 i + 1) pi
// / 32) of the Chebyshev points of the first kind.
__device__ const double kNode[PG_NODE] = {
    0.9951847266721969, 0.9569403357322088, 0.881921264348355,
    0.773010453362737, 0.6343932841636455, 0.47139673682599764,
    0.2902846772544624, 0.0980171403295606, -0.0980171403295606,
    -0.2902846772544624, -0.47139673682599764, -0.6343932841636455,
    -0.773010453362737, -0.881921264348355, -0.9569403357322088,
    -0.9951847266721969};
__device__ const double kBary[PG_NODE] = {
    0.0980171403295606, -0.2902846772544624, 0.47139673682599764,
    -0.6343932841636455, 0.773010453362737, -0.881921264348355,
    0.9569403357322088, -0.9951847266721969, 0.9951847266721969,
    -0.9569403357322088, 0.881921264348355, -0.773010453362737,
    0.6343932841636455, -0.47139673682599764, 0.2902846772544624,
    -0.0980171403295606};

struct PgSmem {
  // two stages: one feeds the MFMAs while the next fills
  double As[2][PG_KC][16];
  double Bs[2][PG_KC][16];
  double Ds[2][16][PG_KC];
  double N[PG_NODE][4][64];    // node values, [node][register][lane]
  double Lw[PG_G][PG_NODE];    // interpolation weights of every energy
  PgDecide dec;
};

// Weight of a pole at distance x = E_k - E with half width h (PsLaunch::part).
template <int PART>
__device__ __forceinline__ double pg_weight(double x, double h) {
  if constexpr (PART == 0)
    return 1.0 / x;
  else
    return (PART == 1 ? x : h) / fma(x, x, h * h);
}

// acc[u] += sum over the chunks chunk(0..count) of A D_u B for this
// wavefront's slots u (a node or an energy each); dist(q, pole energy, x) gives
// the distance E_k - E of slot tid / 32 + 8 q, or false where a slot has no
// energy: it weighs zero.
template <int PART, class Chunk, class Dist>
__device__ __forceinline__ void pg_sum(d4 (&acc)[PG_EW], const SymDev &S, int i0,
                                       int j0, int count, Chunk chunk, Dist dist,
                                       PgSmem &sm) {
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int col = lane & 15, kq = lane >> 4;
  // staging: half the threads take A's columns, half B's, four doubles each
  const int row = (tid & 127) >> 2, c4 = (tid & 3) * 4;
  const double *w = S.Wt + (int64_t)row * S.n_pad + (tid < 128 ? i0 : j0) + c4;
  const int dk = tid & 31, ds = tid >> 5;  // weights: pole, first slot
  double2 r0, r1;
  double ep = 0.0, hw = 0.0;
  auto fetch = [&](int kc) {
    const double *p = w + (int64_t)kc * PG_KC * S.n_pad;
    r0 = *(const double2 *)p;
    r1 = *(const double2 *)(p + 2);
    ep = S.E_pole[kc * PG_KC + dk];
    if constexpr (PART != 0) hw = 0.5 * S.gam[kc * PG_KC + dk];
  };
  auto stage = [&](int buf) {
    double *d = tid < 128 ? &sm.As[buf][row][c4] : &sm.Bs[buf][row][c4];
    *(double2 *)d = r0;
    *(double2 *)(d + 2) = r1;
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      double x;
      const bool on = dist(q, ep, x);
      sm.Ds[buf][ds + 8 * q][dk] = on ? pg_weight<PART>(x, hw) : 0.0;
    }
  };
  if (count <= 0) return;  // uniform
  fetch(chunk(0));
  stage(0);
  if (count > 1) fetch(chunk(1));
  __syncthreads();
#pragma unroll 1
  for (int c = 0; c < count; ++c) {
    const int buf = c & 1;
#pragma unroll
    for (int kk = 0; kk < PG_KC; kk += 4) {
      const double a = sm.As[buf][kk + kq][col];
      const double b = sm.Bs[buf][kk + kq][col];
#pragma unroll
      for (int u = 0; u < PG_EW; ++u)
        acc[u] = __builtin_amdgcn_mfma_f64_16x16x4f64(
            a * sm.Ds[buf][wave * PG_EW + u][kk + kq], b, acc[u], 0, 0, 0);
    }
    if (c + 1 < count) {
      stage(buf ^ 1);
      if (c + 2 < count) fetch(chunk(c + 2));
    }
    __syncthreads();
  }
}

template <int PART>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 2)))
void polesum_group_kernel(PsLaunch L) {
  __shared__ PgSmem sm;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int col = lane & 15, kq = lane >> 4;
  // four blocks an item, the tiles of its 32 x 32 pair; consecutive blocks of
  // an XCD share W columns
  const int per = (4 * L.n_items + 7) / 8;
  const int lin = (blockIdx.x & 7) * per + (blockIdx.x >> 3);
  if (lin >= 4 * L.n_items) return;
  const PsItem item = L.items[lin >> 2];
  const int sub = lin & 3;
  const SymDev &S = L.syms[item.sym];
  const int i0 = item.x * 32 + 16 * (sub >> 1), j0 = item.y * 32 + 16 * (sub & 1);
  if (i0 >= S.n || j0 >= S.n || j0 < i0) return;
  const PgGroup P = pg_decide(L, S, item.grp, sm.dec);
  if (!P.interp) return;  // the direct kernel's
  const int g0 = P.g0, s0 = P.s0, s1 = P.s1, ka = P.ka, kb = P.kb;
  const int nc = S.nh_pad / PG_KC;
  const double *E = L.E;
  const double ev = P.ev, cen = P.cen, h = P.h;
  {
    d4 acc[PG_EW];
#pragma unroll
    for (int u = 0; u < PG_EW; ++u) acc[u] = d4{0.0, 0.0, 0.0, 0.0};
    // nodes as offsets from cen: a node rounded to an energy would be off by
    // an ulp of cen, which is not small against h
    const double xh[2] = {h * kNode[tid >> 5], h * kNode[(tid >> 5) + 8]};
    pg_sum<PART>(
        acc, S, i0, j0, nc - (kb - ka),
        [&](int c) { return c < ka ? c : c + (kb - ka); },
        [&](int q, double ep, double &x) {
          x = (ep - cen) - xh[q];
          return true;
        },
        sm);
#pragma unroll
    for (int u = 0; u < PG_EW; ++u)
#pragma unroll
      for (int r = 0; r < 4; ++r) sm.N[wave * PG_EW + u][r][lane] = acc[u][r];
    if (tid < PG_G) {
      const double x = (ev - cen) / h;
      double t[PG_NODE], s = 0.0;
      int hit = -1;
#pragma unroll
      for (int i = 0; i < PG_NODE; ++i) {
        const double d = x - kNode[i];
        if (d == 0.0) hit = i;
        t[i] = kBary[i] / d;
        s += t[i];
      }
      const double rs = 1.0 / s;
#pragma unroll
      for (int i = 0; i < PG_NODE; ++i)
        sm.Lw[tid][i] = hit < 0 ? t[i] * rs : i == hit ? 1.0 : 0.0;
    }
    __syncthreads();
  }
  const double scale = 1.0 / (2.0 * S.a);
  const int ld = L.out.ld_mult * S.n;
  double *Rbase = L.out.out + L.out.off[item.sym];
#pragma unroll 1
  for (int t = 0; t < PG_G / PG_B; ++t) {
    const int eb = g0 + PG_B * t;  // the batch's first energy
    if (eb >= s1 || eb + PG_B <= s0) continue;
    double es[2];  // energies of this thread's weight slots
    bool on[2];
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      const int e = eb + (tid >> 5) + 8 * q;
      on[q] = e >= s0 && e < s1;
      es[q] = on[q] ? E[e] : 0.0;
    }
    d4 acc[PG_EW];
#pragma unroll
    for (int u = 0; u < PG_EW; ++u) acc[u] = d4{0.0, 0.0, 0.0, 0.0};
#pragma unroll 4
    for (int i = 0; i < PG_NODE; ++i) {
      double nv[4];
#pragma unroll
      for (int r = 0; r < 4; ++r) nv[r] = sm.N[i][r][lane];
#pragma unroll
      for (int u = 0; u < PG_EW; ++u) {
        const double lw = sm.Lw[PG_B * t + PG_EW * wave + u][i];
#pragma unroll
        for (int r = 0; r < 4; ++r) acc[u][r] = fma(lw, nv[r], acc[u][r]);
      }
    }
    pg_sum<PART>(
        acc, S, i0, j0, kb - ka, [&](int c) { return ka + c; },
        [&](int q, double ep, double &x) {
          x = ep - es[q];
          return on[q];
        },
        sm);
    // lane holds D[i][j] with j = lane % 16, i = lane / 16 + 4 r
#pragma unroll
    for (int u = 0; u < PG_EW; ++u) {
      const int e = eb + PG_EW * wave + u;
      if (e < s0 || e >= s1) continue;
      double *Re = Rbase + (int64_t)e * L.out.estride;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int gi = i0 + kq + 4 * r, gj = j0 + col;
        // diagonal tiles: the upper triangle is mirrored so R is exactly
        // symmetric
        if (gi < S.n && gj < S.n && gi <= gj) {
          const double v = acc[u][r] * scale;
          Re[(int64_t)gi * ld + gj] = v;
          Re[(int64_t)gj * ld + gi] = v;
        }
      }
    }
  }
}

__global__ __launch_bounds__(256) void group_work_kernel(PsLaunch L,
                                                         int64_t *work) {
  __shared__ PgDecide dec;
  const PgGroup P = pg_decide(L, L.syms[0], blockIdx.x, dec);
  if (threadIdx.x != 0) return;
  const int nc = L.syms[0].nh_pad / PG_KC;
  const int64_t direct = (int64_t)P.cnt * nc;
  work[2 * blockIdx.x] = P.interp ? pg_work(P, nc) : direct;
  work[2 * blockIdx.x + 1] = direct;
}

hipError_t launch_group_work(const SymDev *sym, const double *E, int64_t m,
                             int ngrp, int64_t *work, hipStream_t st) {
  PsLaunch L{};
  L.syms = sym;
  L.E = E;
  L.m = (int)m;
  L.m_all = m;
  hipLaunchKernelGGL(group_work_kernel, dim3((unsigned)ngrp), dim3(256), 0, st, L,
                     work);
  return hipGetLastError();
}

hipError_t launch_polesum_group(const PsLaunch &L, hipStream_t st) {
  const dim3 grid((unsigned)(8 * ((4 * L.n_items + 7) / 8)));
  if (L.part == 1)
    hipLaunchKernelGGL(polesum_group_kernel<1>, grid, dim3(256), 0, st, L);
  else if (L.part == 2)
    hipLaunchKernelGGL(polesum_group_kernel<2>, grid, dim3(256), 0, st, L);
  else
    hipLaunchKernelGGL(polesum_group_kernel<0>, grid, dim3(256), 0, st, L);
  return hipGetLastError();
}

}  // namespace rmx
