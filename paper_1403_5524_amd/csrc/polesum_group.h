// Groups of consecutive energies whose far poles can be interpolated: the
// decision, shared by the kernel that sums such groups and the one that sums
// the others.
#pragma once

#include "rm_internal.h"

namespace rmx {

constexpr int PG_KC = 32;    // poles per chunk
constexpr int PG_G = 128;    // energies per group
constexpr int PG_NODE = 16;  // interpolation points

struct PgDecide {  // LDS
  double red[4][2];
  int redi[4][3];
};

struct PgGroup {
  int g0, cnt;   // the group's energies are E[g0 + q], q < cnt
  int s0, s1;    // those of this chunk, [s0, s1)
  int ka, kb;    // near chunks of poles
  int interp;    // 1: the other chunks are interpolated
  double ev;     // energy tid % 128 of the group (the last one past cnt)
  double cen, h; // centre and half width
};

// Energies times chunks of poles of an interpolated group, nc chunks in all.
__device__ __forceinline__ int64_t pg_work(const PgGroup &p, int nc) {
  const int nn = p.kb - p.ka;
  return (int64_t)PG_NODE * (nc - nn) + (int64_t)p.cnt * nn;
}

// Group grp of the launch's chunk (groups are cut on the whole mesh, so the
// chunk may begin or end inside one), for a workgroup of 256.  The two kernels
// have to come to the same decision, or a group is summed by both or by neither:
// no product is fused with a sum here, so every step is rounded by itself and
// the result does not depend on what the compiler makes of either kernel.
__device__ __forceinline__ PgGroup pg_decide(const PsLaunch &L, const SymDev &S,
                                             int grp, PgDecide &sm) {
#pragma clang fp contract(off)
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  PgGroup p;
  const int64_t G = L.e_off / PG_G + grp;
  p.g0 = (int)(G * PG_G - L.e_off);
  p.cnt = (int)min((int64_t)PG_G, L.m_all - G * PG_G);
  p.s0 = max(0, p.g0);
  p.s1 = min(L.m, p.g0 + PG_G);
  p.interp = 0;
  p.ka = p.kb = 0;
  p.ev = p.cen = p.h = 0.0;
  if (p.s0 >= p.s1) return p;  // uniform
  p.ev = L.E[p.g0 + min(tid & (PG_G - 1), p.cnt - 1)];
  double mn = p.ev, mx = p.ev;
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    mn = fmin(mn, __shfl_xor(mn, o));
    mx = fmax(mx, __shfl_xor(mx, o));
  }
  const int odd = __ballot(!(fabs(p.ev) < 1e300)) != 0;
  if (lane == 0) {
    sm.red[wave][0] = mn;
    sm.red[wave][1] = mx;
    sm.redi[wave][2] = odd;
  }
  __syncthreads();
  mn = fmin(sm.red[0][0], sm.red[1][0]);
  mx = fmax(sm.red[0][1], sm.red[1][1]);
  p.cen = 0.5 * (mn + mx);
  p.h = fmax(mx - p.cen, p.cen - mn);
  // near chunks [ka, kb): those that reach into [cen - 6 h, cen + 6 h]
  const int nc = S.nh_pad / PG_KC;
  const double lo = p.cen - 6.0 * p.h, hi = p.cen + 6.0 * p.h;
  int ka = 0, kb = 0;
  for (int k = tid; k < nc; k += 256) {
    ka += S.E_pole[k * PG_KC + PG_KC - 1] < lo ? 1 : 0;
    kb += S.E_pole[k * PG_KC] <= hi ? 1 : 0;
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    ka += __shfl_xor(ka, o);
    kb += __shfl_xor(kb, o);
  }
  if (lane == 0) {
    sm.redi[wave][0] = ka;
    sm.redi[wave][1] = kb;
  }
  __syncthreads();
  ka = sm.redi[0][0] + sm.redi[1][0] + sm.redi[2][0] + sm.redi[3][0];
  kb = sm.redi[0][1] + sm.redi[1][1] + sm.redi[2][1] + sm.redi[3][1];
  p.ka = __builtin_amdgcn_readfirstlane(ka);
  p.kb = __builtin_amdgcn_readfirstlane(kb);
  const int fine = __builtin_amdgcn_readfirstlane(
      (sm.redi[0][2] | sm.redi[1][2]) == 0 && p.h > 0.0 ? 1 : 0);
  // The far phase costs 16 energies' worth of the far chunks; required to
  // take a quarter off, since the direct sum has eight times the workgroups.
  p.interp = fine && 4 * pg_work(p, nc) < (int64_t)3 * p.cnt * nc;
  return p;
}

}  // namespace rmx
