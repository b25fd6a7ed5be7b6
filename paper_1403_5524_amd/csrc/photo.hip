// Dipole pole sum of the photoionization path: at every energy of a chunk
//     g_i(E) = (1/sqrt2) sum_k w_ik d_k / (E_k - E),
// the vector that turns the matching solution into bound-free dipole
// amplitudes (the inner-region expansion of the continuum, Bloch b = 0, in
// the convention R_ij = (1/2a) sum_k w_ik w_jk / (E_k - E)).  It is the
// pole sum of Sec. 6, Eq. 1-2, with the second factor W replaced by one
// dipole vector: an (n x N_H) by (N_H x m) product on the FP64 matrix cores
// whose right operand d_k / (E_k - E) each lane forms in its register.
//
// The output is small (n x m) and the poles many, so the chip is filled by
// splitting the poles: a workgroup of eight wavefronts holds 32 channels x 16
// energies and each wavefront takes every eighth group of four poles, without
// LDS or barriers; the eight parts are added in a fixed order.  A step of four
// poles is two matrix instructions (128 cycles) and one division.  With 64 x
// 64 outputs per workgroup, weights staged through LDS 16 poles at a time and
// each workgroup walking all poles, 400 channels and 256 energies made 28
// workgroups: 2.94 ms, now 0.30.
#include "rm_internal.h"

namespace rmx {

typedef double d4 __attribute__((ext_vector_type(4)));

constexpr int DP_N = 32;   // channels per workgroup
constexpr int DP_E = 16;   // energies per workgroup
constexpr int DP_W = 8;    // wavefronts, each an eighth of the poles
constexpr int DP_U = 4;    // steps in flight

// PART 0: weights d_k / (E_k - E); 1, 2: real and imaginary part of
// d_k / (E_k - i Gamma_k/2 - E)
template <int PART>
__global__ __launch_bounds__(64 * DP_W) void dip_polesum_kernel(
    SymDev S, const double *__restrict__ E, int m, double *__restrict__ out,
    int64_t estride, int64_t off) {
  __shared__ double part[DP_W][8][64];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int col = lane & 15, kq = lane >> 4;
  const int i0 = blockIdx.x * DP_N, e0 = blockIdx.y * DP_E;
  // energies past the end repeat the last one and are not stored; channels
  // up to n_pad (a multiple of 32) are there, with zero amplitudes past n
  const double Ee = E[min(e0 + col, m - 1)];
  const double *w = S.Wt + i0 + col;
  d4 acc[2] = {d4{0.0, 0.0, 0.0, 0.0}, d4{0.0, 0.0, 0.0, 0.0}};
  // nh_pad is a multiple of 64: a turn of DP_W wavefronts takes 32 poles
  const int turns = S.nh_pad / (4 * DP_W);
  for (int t0 = 0; t0 < turns; t0 += DP_U) {
    double a[DP_U][2], b[DP_U];
#pragma unroll
    for (int u = 0; u < DP_U; ++u) {
      const int t = min(t0 + u, turns - 1);
      const int k = (t * DP_W + wave) * 4 + kq;
      const double *wk = w + (int64_t)k * S.n_pad;
      a[u][0] = wk[0];
      a[u][1] = wk[16];
      const double x = S.E_pole[k] - Ee;
      double v;
      if constexpr (PART == 0) {
        v = S.dip[k] / x;
      } else {
        const double h = 0.5 * S.gam[k];
        v = S.dip[k] * (PART == 1 ? x : h) / fma(x, x, h * h);
      }
      b[u] = t0 + u < turns ? v : 0.0;
    }
#pragma unroll
    for (int u = 0; u < DP_U; ++u)
#pragma unroll
      for (int c = 0; c < 2; ++c)
        acc[c] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[u][c], b[u], acc[c], 0, 0, 0);
  }
#pragma unroll
  for (int c = 0; c < 2; ++c)
#pragma unroll
    for (int r = 0; r < 4; ++r) part[wave][4 * c + r][lane] = acc[c][r];
  __syncthreads();
  // FP64 16x16x4 result: lane holds row kq + 4 r (channel), column col
  // (energy) of block c; thread tid adds register tid / 64 of lane tid % 64
  double s = 0.0;
#pragma unroll
  for (int q = 0; q < DP_W; ++q) s += part[q][wave][lane];
  const int i = i0 + 16 * (wave >> 2) + kq + 4 * (wave & 3), e = e0 + col;
  if (i < S.n && e < m)
    out[(int64_t)e * estride + off + i] = s * 0.70710678118654752440;
}

hipError_t launch_dip_polesum(const SymDev &S, const double *E, int m,
                              double *out, int64_t estride, int64_t off,
                              hipStream_t st, int part) {
  if (m <= 0) return hipSuccess;
  const dim3 grid((unsigned)((S.n + DP_N - 1) / DP_N), (unsigned)((m + DP_E - 1) / DP_E));
  hipLaunchKernelGGL(part == 1   ? dip_polesum_kernel<1>
                     : part == 2 ? dip_polesum_kernel<2>
                                 : dip_polesum_kernel<0>,
                     grid, dim3(64 * DP_W), 0, st, S, E, m, out, estride, off);
  return hipGetLastError();
}

}  // namespace rmx
