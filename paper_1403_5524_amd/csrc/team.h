// Dense linear algebra of one energy by a team of NW wavefronts.
//
// A team is one workgroup of NW wavefronts.  All matrices are row-major in a
// per-energy global workspace.  The work of a routine is split by output
// tiles, column chunks or rows over the team's wavefronts, so every element
// sees the same operations in the same order whatever NW is; the routines end
// with the team's barrier.
//
// What bounds it: at one wavefront per energy, two per SIMD, 2048 energies
// were in flight and their 0.96 MB workspaces (200 channels) streamed through
// HBM between the block steps: 30.8 MB and 6.6 us per energy with all channels
// open.  A team keeps a quarter or an eighth as many energies in flight, reads
// each panel once per team through the CU's own cache, and spreads the serial
// phases (pivot search, diagonal blocks) over as many SIMDs: 20.1 MB and 5.2 us
// (LU 2.3, T step 2.5, assembly 0.3) at 8192 energies.  The LU and the T step
// then move 3.9 TB/s, where a copy reaches 4.3.
//
// Every pass over memory is written as "issue all loads of a batch, then
// compute, then store": the compiler cannot move a load above a store it
// cannot prove disjoint.
#pragma once

#include <hip/hip_runtime.h>

#include "rm_internal.h"

// Address spaces of device memory and LDS.  With plain pointers a routine
// that is not inlined would load through flat instructions, whose results
// can only be waited for all at once.
#ifndef RM_G
#define RM_G __attribute__((address_space(1)))
#define RM_L __attribute__((address_space(3)))
#endif

namespace rmx {

template <class T>
__device__ inline RM_G T *as_g(T *p) {
  return (RM_G T *)p;
}

constexpr int WT = 64;    // lanes per wavefront
constexpr int NB = 16;    // panel width of the memory panel
constexpr int NB2 = 32;   // block width: panel, update and diagonal blocks
constexpr int UNR = 4;    // independent elements per lane per batch

typedef double d4 __attribute__((ext_vector_type(4)));
typedef float f4 __attribute__((ext_vector_type(4)));

// Element types of the wavefront linear algebra: FP64 (the default path) and
// FP32 (the factorisation of the FP32 solve, refined in FP64).  The 16x16x4
// MFMAs of both read A[i][k] and B[k][j] at i = j = lane % 16, k = lane / 16;
// their 16x16 results differ in layout: FP64 row kq + 4r, FP32 row 4kq + r
// of register r (kq = lane / 16).
template <class T>
struct Mx;
template <>
struct Mx<double> {
  typedef d4 acc;
  __device__ static inline acc mfma(double a, double b, acc c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
  }
  __device__ static inline int row(int kq, int r) { return kq + 4 * r; }
};
template <>
struct Mx<float> {
  typedef f4 acc;
  __device__ static inline acc mfma(float a, float b, acc c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
  }
  __device__ static inline int row(int kq, int r) { return 4 * kq + r; }
};

// LDS of one team: the current diagonal block and the inverses of its
// triangles, the row moves of its interchanges, and the pivot candidates of
// the register panel (double-buffered by column).
template <int NW>
struct TeamLds {
  double T[NB2][NB2 + 1];
  double Ti[NB2][NB2 + 1];  // inverse applied next
  double cand[2][NW][NB2];  // pivot candidate rows of the wavefronts ...
  double cmax[2][NW];       // ... their magnitudes (-1: none)
  int cpos[2][NW];          // ... and positions
  double red[NW];           // team reductions
  int piv[NB2];   // pivot row chosen at each column of the block
  int srcp[NB2];  // after the interchanges, block row q holds old row srcp[q]
  int opos[NB2];  // rows below the block that receive another row ...
  int osrc[NB2];  // ... namely old row osrc[m]
  int nout;
  int bcast;
};

__device__ inline int lane_id() { return threadIdx.x & (WT - 1); }

// A team-uniform value as a scalar.  Everything that decides a branch or a
// loop around a barrier or a block step goes through this, and every routine
// passes its sizes through it: with such a condition in a vector register the
// compiler masks lanes instead of branching, and has been seen to reload
// spilled registers on the way out of such a loop while the mask is empty (a
// spilled LDS address then came back as whatever the register held).
__device__ __forceinline__ int uni(int v) {
  return __builtin_amdgcn_readfirstlane(v);
}

// Thread index and wavefront (scalar) within the team.
template <int NW>
__device__ __forceinline__ int team_tid() {
  return (int)threadIdx.x;
}
template <int NW>
__device__ __forceinline__ int team_wave() {
  return NW == 1 ? 0 : __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
}

// Make this lane's earlier writes visible to the other lanes of the
// wavefront and keep the compiler from moving memory operations across.
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
}

template <int NW>
__device__ __forceinline__ void team_sync() {
  if constexpr (NW == 1)
    wave_sync();
  else
    __syncthreads();
}

__device__ inline double read_lane(double v, int l) {
  const long long b = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_readlane((int)(b & 0xffffffffLL), l);
  const int hi = __builtin_amdgcn_readlane((int)(b >> 32), l);
  return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}

__device__ inline float read_lane(float v, int l) {
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), l));
}

// Largest a of the wavefront (a finite or infinite, not NaN), in every lane.
template <int CTRL>
__device__ inline double dpp_max_step(double a) {
  const long long b = __double_as_longlong(a);
  const int lo = (int)b, hi = (int)(b >> 32);
  const int l2 = __builtin_amdgcn_update_dpp(lo, lo, CTRL, 0xf, 0xf, false);
  const int h2 = __builtin_amdgcn_update_dpp(hi, hi, CTRL, 0xf, 0xf, false);
  const double o = __longlong_as_double(((long long)h2 << 32) | (unsigned int)l2);
  return o > a ? o : a;
}
__device__ __forceinline__ double wave_max(double a) {
  a = dpp_max_step<0x111>(a);  // row_shr:1
  a = dpp_max_step<0x112>(a);  // row_shr:2
  a = dpp_max_step<0x114>(a);  // row_shr:4
  a = dpp_max_step<0x118>(a);  // row_shr:8
  a = dpp_max_step<0x142>(a);  // row_bcast:15
  a = dpp_max_step<0x143>(a);  // row_bcast:31
  return read_lane(a, WT - 1);
}

// Wavefront argmax of a = |v| (ties -> smaller index), carrying v.
template <class T>
__device__ __forceinline__ void wave_argmax(T &a, T &v, int &idx) {
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) {
    const T oa = __shfl_xor(a, off);
    const T ov = __shfl_xor(v, off);
    const int oi = __shfl_xor(idx, off);
    if (oa > a || (oa == a && oi < idx)) {
      a = oa;
      v = ov;
      idx = oi;
    }
  }
}

__device__ __forceinline__ int wave_or(int v) {
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) v |= __shfl_xor(v, off);
  return v;
}

// Sum and maximum over the team, in every thread (NaN in the maximum is
// skipped).  Two barriers.
template <int NW>
__device__ __forceinline__ double team_sum(double v, RM_L TeamLds<NW> &W) {
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off);
  if constexpr (NW == 1) return v;
  const int wv = team_wave<NW>();
  team_sync<NW>();
  if (lane_id() == 0) W.red[wv] = v;
  team_sync<NW>();
  double s = 0.0;
#pragma unroll
  for (int w = 0; w < NW; ++w) s += W.red[w];
  return s;
}
template <int NW>
__device__ __forceinline__ double team_max(double v, RM_L TeamLds<NW> &W) {
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) v = fmax(v, __shfl_xor(v, off));
  if constexpr (NW == 1) return v;
  const int wv = team_wave<NW>();
  team_sync<NW>();
  if (lane_id() == 0) W.red[wv] = v;
  team_sync<NW>();
  double s = W.red[0];
#pragma unroll
  for (int w = 1; w < NW; ++w) s = fmax(s, W.red[w]);
  return s;
}

// Body f(i, j) over a rows x cols block, consecutive lanes along j: whole
// rows per wavefront where a row fills most of one, a flat index otherwise.
// Batches of UNR elements, each batch's loads (ld) before its stores (st).
template <int NW, class LD, class ST>
__device__ __forceinline__ void team_each(int rows, int cols, LD ld, ST st) {
  rows = uni(rows); cols = uni(cols);
  if (cols >= 48) {
    for (int i0 = team_wave<NW>() * UNR; i0 < rows; i0 += NW * UNR)
      for (int j = lane_id(); j < cols; j += WT) {
        decltype(ld(0, 0)) v[UNR];
#pragma unroll
        for (int u = 0; u < UNR; ++u)
          v[u] = ld(i0 + u < rows ? i0 + u : rows - 1, j);
#pragma unroll
        for (int u = 0; u < UNR; ++u)
          if (i0 + u < rows) st(i0 + u, j, v[u]);
      }
  } else {
    const int nq = rows * cols;
    for (int q0 = team_tid<NW>(); q0 < nq; q0 += UNR * WT * NW) {
      decltype(ld(0, 0)) v[UNR];
#pragma unroll
      for (int u = 0; u < UNR; ++u) {
        const int q = min(q0 + u * WT * NW, nq - 1);
        v[u] = ld(q / cols, q % cols);
      }
#pragma unroll
      for (int u = 0; u < UNR; ++u) {
        const int q = q0 + u * WT * NW;
        if (q < nq) st(q / cols, q % cols, v[u]);
      }
    }
  }
}

// ---------------------------------------------------------------------------
// GEMM of a team, operands in global memory: wavefront w takes every NW-th
// output tile from the w-th on.
//   MODE 0: C -= A B  (the rank-16 and rank-32 updates of the LU)
//   MODE 1: C = A B + I
//   MODE 2: C = A B
// A wavefront walks 32 x 32 output tiles (2 x 2 MFMA blocks sharing their
// A and B fragments) in k-steps of 16.
template <class T>
struct Frag {
  T a[4][2], b[4][2];
};

// Operand storage flags of team_gemm.
constexpr int G_TA = 1;     // A[i][k] stored at A[k * lda + i]
constexpr int G_TB = 2;     // B[k][j] stored at B[j * ldb + k]
constexpr int G_LOWER = 4;  // only the tiles of C that meet its lower triangle
constexpr int G_BSYM = 8;   // B symmetric, only its lower triangle stored
constexpr int G_KTRI = 16;  // A^T with A lower triangular (team_gemm_wide,
                            // with G_TA): a tile's sum starts at its first row

template <int FL, class T>
__device__ inline void frag_load(Frag<T> &f, const RM_G T *A, int lda,
                                 const RM_G T *B, int ldb, int rows, int cols,
                                 int kd, int rb, int cb, int k0) {
  const int lane = lane_id();
  const int col = lane & 15, kq = lane >> 4;
  const int ra0 = rb + col, ra1 = ra0 + 16, c0 = cb + col, c1 = c0 + 16;
#pragma unroll
  for (int s = 0; s < 4; ++s) {
    const int k = k0 + 4 * s + kq;
    const bool kv = k < kd;
    if (FL & G_TA) {
      f.a[s][0] = (kv && ra0 < rows) ? A[(int64_t)k * lda + ra0] : T(0);
      f.a[s][1] = (kv && ra1 < rows) ? A[(int64_t)k * lda + ra1] : T(0);
    } else {
      f.a[s][0] = (kv && ra0 < rows) ? A[(int64_t)ra0 * lda + k] : T(0);
      f.a[s][1] = (kv && ra1 < rows) ? A[(int64_t)ra1 * lda + k] : T(0);
    }
    if (FL & G_TB) {
      f.b[s][0] = (kv && c0 < cols) ? B[(int64_t)c0 * ldb + k] : T(0);
      f.b[s][1] = (kv && c1 < cols) ? B[(int64_t)c1 * ldb + k] : T(0);
    } else {
      f.b[s][0] = (kv && c0 < cols) ? B[(int64_t)k * ldb + c0] : T(0);
      f.b[s][1] = (kv && c1 < cols) ? B[(int64_t)k * ldb + c1] : T(0);
    }
  }
}

// C tile in the result layout of the type's 16x16x4 MFMA (Mx<T>::row).
template <class T>
__device__ inline void ctile_load(T (&c)[2][2][4], const RM_G T *C,
                                  int ldc, int rows, int cols, int rb, int cb) {
  const int lane = lane_id();
  const int col = lane & 15, kq = lane >> 4;
#pragma unroll
  for (int x = 0; x < 2; ++x)
#pragma unroll
    for (int y = 0; y < 2; ++y)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int i = rb + 16 * x + Mx<T>::row(kq, r), j = cb + 16 * y + col;
        c[x][y][r] = (i < rows && j < cols) ? C[(int64_t)i * ldc + j] : T(0);
      }
}

// The k-th tile after t (row-major over 32 x 32 tiles), counting only the
// tiles on or below the diagonal when only the lower triangle is wanted.
template <int FL>
__device__ inline int gemm_next_tile(int t, int nct, int ntile, int k) {
  if (!(FL & G_LOWER)) return t + k;
  for (; k > 0; --k) {
    ++t;
    while (t < ntile && (t % nct) > (t / nct)) ++t;
  }
  return t;
}

template <int NW, int MODE, int FL = 0, class T = double>
__device__ __forceinline__ void team_gemm(RM_G T *C, int ldc, const RM_G T *A, int lda,
                          const RM_G T *B, int ldb, int rows, int cols,
                          int kd) {
  ldc = uni(ldc); lda = uni(lda); ldb = uni(ldb); rows = uni(rows); cols = uni(cols); kd = uni(kd);
  typedef typename Mx<T>::acc acc_t;
  const int lane = lane_id();
  const int col = lane & 15, kq = lane >> 4;
  const int nct = (cols + 31) >> 5;
  const int ntile = ((rows + 31) >> 5) * nct;
  const int nk = max(1, (kd + 15) >> 4);
  const int t0 = gemm_next_tile<FL>(0, nct, ntile, team_wave<NW>());
  if (t0 < ntile) {
    Frag<T> cur, nxt;
    T cv[2][2][4], cn[2][2][4];
    frag_load<FL>(cur, A, lda, B, ldb, rows, cols, kd, (t0 / nct) * 32,
                  (t0 % nct) * 32, 0);
    if (MODE == 0)
      ctile_load(cv, C, ldc, rows, cols, (t0 / nct) * 32, (t0 % nct) * 32);
    for (int t = t0; t < ntile;) {
      const int tn = gemm_next_tile<FL>(t, nct, ntile, NW);
      const int rb = (t / nct) * 32, cb = (t % nct) * 32;
      acc_t acc[2][2];
#pragma unroll
      for (int x = 0; x < 2; ++x)
#pragma unroll
        for (int y = 0; y < 2; ++y) acc[x][y] = acc_t{0, 0, 0, 0};
      for (int kc = 0; kc < nk; ++kc) {
        // prefetch: the next k-step of this tile, else the next tile (whose
        // A, B and C do not overlap this tile's C)
        if (kc + 1 < nk) {
          frag_load<FL>(nxt, A, lda, B, ldb, rows, cols, kd, rb, cb, (kc + 1) * 16);
        } else if (tn < ntile) {
          const int rn = (tn / nct) * 32, cnb = (tn % nct) * 32;
          frag_load<FL>(nxt, A, lda, B, ldb, rows, cols, kd, rn, cnb, 0);
          if (MODE == 0) ctile_load(cn, C, ldc, rows, cols, rn, cnb);
        }
#pragma unroll
        for (int s = 0; s < 4; ++s)
#pragma unroll
          for (int x = 0; x < 2; ++x)
#pragma unroll
            for (int y = 0; y < 2; ++y)
              acc[x][y] = Mx<T>::mfma(cur.a[s][x], cur.b[s][y], acc[x][y]);
        cur = nxt;
      }
#pragma unroll
      for (int x = 0; x < 2; ++x)
#pragma unroll
        for (int y = 0; y < 2; ++y)
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const int i = rb + 16 * x + Mx<T>::row(kq, r), j = cb + 16 * y + col;
            if (i >= rows || j >= cols) continue;
            T v = acc[x][y][r];
            if (MODE == 0) v = cv[x][y][r] - v;
            if (MODE == 1 && i == j) v += T(1);
            C[(int64_t)i * ldc + j] = v;
          }
      if (MODE == 0) {
#pragma unroll
        for (int x = 0; x < 2; ++x)
#pragma unroll
          for (int y = 0; y < 2; ++y)
#pragma unroll
            for (int r = 0; r < 4; ++r) cv[x][y][r] = cn[x][y][r];
      }
      t = tn;
    }
  }
  team_sync<NW>();
}

// Wide form: output tiles of (16 BM) x (16 BN), so each A row panel is read
// once per 16 BN columns and each B column panel once per 16 BM rows (the
// 32 x 32 tiles above read both twice as often).  MODE 0 loads C into the
// accumulators and subtracts A B through them (no separate C registers),
// MODE 1 starts from the identity, MODE 2 from zero.  With G_LOWER only tiles
// whose first column is on or left of their last row are formed.  G_BSYM
// reads B[k][j] from B's lower triangle; G_KTRI skips the k-steps below the
// tile's first row (they multiply the zeros above the diagonal of a
// lower-triangular A stored transposed).
//
// Loads are never predicated: rows, columns and k are clamped into the
// operand (what a clamped row or column adds falls outside C and is not
// stored; clamped k-steps are zeroed), and each operand is a scalar base
// that advances with k plus 32-bit lane offsets that stay for the tile.
// Predicated 64-bit addresses took more registers than the accumulators.
template <int NW, int MODE, int FL, int BM, int BN, class T = double>
__device__ __forceinline__ void team_gemm_wide(RM_G T *C, int ldc,
                                               const RM_G T *A, int lda,
                                               const RM_G T *B, int ldb,
                                               int rows, int cols, int kd) {
  ldc = uni(ldc); lda = uni(lda); ldb = uni(ldb); rows = uni(rows); cols = uni(cols); kd = uni(kd);
  typedef typename Mx<T>::acc acc_t;
  constexpr int TH = 16 * BM, TW = 16 * BN;
  constexpr uint32_t SZ = sizeof(T);
  const int lane = lane_id();
  const int col = lane & 15, kq = lane >> 4;
  const int nct = (cols + TW - 1) / TW;
  const int ntile = ((rows + TH - 1) / TH) * nct;
  const int nk = (kd + 15) >> 4;
  auto skip = [&](int t) {
    return (FL & G_LOWER) && (t % nct) * TW > (t / nct) * TH + TH - 1;
  };
  auto next = [&](int t, int k) {
    if (!(FL & G_LOWER)) return t + k;
    for (; k > 0; --k) {
      ++t;
      while (t < ntile && skip(t)) ++t;
    }
    return t;
  };
  // first k-step of tile t
  auto kfirst = [&](int t) {
    return (FL & G_KTRI) ? min((t / nct) * TH, kd) >> 4 : 0;
  };
  auto at = [](const RM_G T *base, uint32_t off) {
    return *(const RM_G T *)((const RM_G char *)base + off);
  };
  // (tile 0 always meets the lower triangle)
  for (int t = next(0, team_wave<NW>()); t < ntile; t = next(t, NW)) {
    const int rb = (t / nct) * TH, cb = (t % nct) * TW;
    const bool inside = rb + TH <= rows && cb + TW <= cols;  // uniform
    uint32_t cofs[BM][4], cj[BN], ra[BM];
#pragma unroll
    for (int y = 0; y < BN; ++y) cj[y] = min(cb + 16 * y + col, cols - 1);
#pragma unroll
    for (int x = 0; x < BM; ++x) {
      ra[x] = min(rb + 16 * x + col, rows - 1);
#pragma unroll
      for (int r = 0; r < 4; ++r)
        cofs[x][r] =
            (uint32_t)min(rb + 16 * x + Mx<T>::row(kq, r), rows - 1) * ldc * SZ;
    }
    acc_t acc[BM][BN];
#pragma unroll
    for (int x = 0; x < BM; ++x)
#pragma unroll
      for (int y = 0; y < BN; ++y)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          T v = T(0);
          if (MODE == 0) v = at(C, cofs[x][r] + cj[y] * SZ);
          if (MODE == 1)
            v = (rb + 16 * x + Mx<T>::row(kq, r) == cb + 16 * y + col) ? T(1) : T(0);
          acc[x][y][r] = v;
        }
    // lane offsets of the operands at k = kq; k advances the scalar base
    // (G_BSYM: the side of the diagonal depends on k, so offsets are formed
    // per load)
    uint32_t ao[BM], bo[BN];
#pragma unroll
    for (int x = 0; x < BM; ++x)
      ao[x] = ((FL & G_TA) ? kq * (uint32_t)lda + ra[x] : ra[x] * lda + kq) * SZ;
#pragma unroll
    for (int y = 0; y < BN; ++y)
      bo[y] = ((FL & G_TB) ? cj[y] * ldb + kq : kq * (uint32_t)ldb + cj[y]) * SZ;
    auto fload = [&](T (&a)[4][BM], T (&b)[4][BN], int k0) {
      if (k0 + 16 <= kd) {
        const RM_G T *Ak = A + ((FL & G_TA) ? (int64_t)k0 * lda : k0);
        const RM_G T *Bk = B + ((FL & G_TB) ? k0 : (int64_t)k0 * ldb);
#pragma unroll
        for (int s4 = 0; s4 < 4; ++s4) {
          const RM_G T *As = Ak + ((FL & G_TA) ? (int64_t)4 * s4 * lda : 4 * s4);
          const RM_G T *Bs = Bk + ((FL & G_TB) ? 4 * s4 : (int64_t)4 * s4 * ldb);
#pragma unroll
          for (int x = 0; x < BM; ++x) a[s4][x] = at(As, ao[x]);
#pragma unroll
          for (int y = 0; y < BN; ++y) {
            if (FL & G_BSYM) {
              const uint32_t k = k0 + 4 * s4 + kq, j = cj[y];
              b[s4][y] = at(B, (max(k, j) * ldb + min(k, j)) * SZ);
            } else {
              b[s4][y] = at(Bs, bo[y]);
            }
          }
        }
      } else {
#pragma unroll
        for (int s4 = 0; s4 < 4; ++s4) {
          const int k = k0 + 4 * s4 + kq;
          const uint32_t kc = min(k, kd - 1);
#pragma unroll
          for (int x = 0; x < BM; ++x) {
            const T v = at(A, ((FL & G_TA) ? kc * lda + ra[x] : ra[x] * lda + kc) * SZ);
            a[s4][x] = k < kd ? v : T(0);
          }
#pragma unroll
          for (int y = 0; y < BN; ++y) {
            const uint32_t j = cj[y];
            const bool tr = (FL & G_TB) || ((FL & G_BSYM) && kc < j);
            const T v = at(B, (tr ? j * ldb + kc : kc * ldb + j) * SZ);
            b[s4][y] = k < kd ? v : T(0);
          }
        }
      }
    };
    T ca[4][BM], cbf[4][BN], na[4][BM], nb[4][BN];
    int kc = kfirst(t);
    if (kc < nk) fload(ca, cbf, 16 * kc);
    for (; kc < nk; ++kc) {
      if (kc + 1 < nk) fload(na, nb, 16 * (kc + 1));
#pragma unroll
      for (int s4 = 0; s4 < 4; ++s4)
#pragma unroll
        for (int x = 0; x < BM; ++x)
#pragma unroll
          for (int y = 0; y < BN; ++y)
            acc[x][y] = Mx<T>::mfma(MODE == 0 ? -ca[s4][x] : ca[s4][x],
                                    cbf[s4][y], acc[x][y]);
#pragma unroll
      for (int s4 = 0; s4 < 4; ++s4) {
#pragma unroll
        for (int x = 0; x < BM; ++x) ca[s4][x] = na[s4][x];
#pragma unroll
        for (int y = 0; y < BN; ++y) cbf[s4][y] = nb[s4][y];
      }
    }
#pragma unroll
    for (int x = 0; x < BM; ++x)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int i = rb + 16 * x + Mx<T>::row(kq, r);
#pragma unroll
        for (int y = 0; y < BN; ++y)
          if (inside || (i < rows && cb + 16 * y + col < cols))
            *(RM_G T *)((RM_G char *)C + (cofs[x][r] + cj[y] * SZ)) = acc[x][y][r];
      }
  }
  team_sync<NW>();
}

// ---------------------------------------------------------------------------
// LU with partial pivoting.

// Factor columns [j0, j0 + jb) (jb <= 16) of rows [j0, na) in place;
// interchanges swap the row segments [sw0, j0 + jb) (the panel and the L
// columns of an earlier panel of the same block); pivots -> W.piv[po + .].
// Returns 1 if a pivot was zero or not a number.
template <int NW, class T>
__device__ __forceinline__ int team_panel_mem(RM_G T *A, int na, int ld, int j0, int jb, int sw0,
                              int po, RM_L TeamLds<NW> &W) {
  na = uni(na); ld = uni(ld); j0 = uni(j0); jb = uni(jb); sw0 = uni(sw0); po = uni(po);
  const int lane = lane_id(), tid = team_tid<NW>(), wv = team_wave<NW>();
  int flag = 0;
#pragma unroll 1
  for (int jj = 0; jj < jb; ++jj) {
    const int col = j0 + jj;
    T ba = T(-1), bv = T(0);
    int bi = na;
    for (int r0 = col + tid; r0 < na; r0 += UNR * WT * NW) {
      T v[UNR];
#pragma unroll
      for (int u = 0; u < UNR; ++u) {
        const int r = r0 + u * WT * NW;
        v[u] = r < na ? A[(int64_t)r * ld + col] : T(0);
      }
#pragma unroll
      for (int u = 0; u < UNR; ++u) {
        const int r = r0 + u * WT * NW;
        if (r < na && fabs(v[u]) > ba) {
          ba = fabs(v[u]);
          bv = v[u];
          bi = r;
        }
      }
    }
    wave_argmax(ba, bv, bi);
    if (lane == 0) {
      W.cmax[jj & 1][wv] = (double)ba;
      W.cand[jj & 1][wv][0] = (double)bv;
      W.cpos[jj & 1][wv] = bi;
    }
    team_sync<NW>();
    double best = -1.0;
    int pr = na;
    T pv = T(0);
#pragma unroll
    for (int w = 0; w < NW; ++w) {
      const double a = W.cmax[jj & 1][w];
      const int r = W.cpos[jj & 1][w];
      if (a > best || (a == best && r < pr)) {
        best = a;
        pr = r;
        pv = (T)W.cand[jj & 1][w][0];
      }
    }
    pr = __builtin_amdgcn_readfirstlane(pr);
    if (pr >= na) {  // every candidate is NaN
      pr = col;
      pv = (T)__builtin_nan("");
    }
    if (tid == 0) W.piv[po + jj] = pr;
    // swap the segments [sw0, j0 + jb) of rows col and pr; lane q keeps the
    // new pivot row's element of panel column j0 + q
    const int sw = lane + sw0 - j0;  // this lane's column, relative to j0
    T xv = T(0), yv = T(0);
    RM_G T *x = A + (int64_t)col * ld + j0 + sw;
    RM_G T *y = A + (int64_t)pr * ld + j0 + sw;
    if (sw < jb) {
      xv = *x;
      yv = *y;
    }
    // the lane that holds panel column j0 + q has its pivot-row value
    const T prow = __shfl(yv, min(lane + j0 - sw0, WT - 1));
    team_sync<NW>();  // every wavefront has read both rows
    if (wv == 0 && sw < jb && pr != col) {
      *x = yv;
      *y = xv;
    }
    team_sync<NW>();
    if (!(fabs(pv) > T(0))) flag = 1;
    const T inv = T(1) / pv;
    T pc[NB];
#pragma unroll
    for (int q = 0; q < NB; ++q) pc[q] = read_lane(prow, q);
    // eliminate below the pivot, two rows per lane per batch
    for (int r0 = col + 1 + tid; r0 < na; r0 += 2 * WT * NW) {
      const int r1 = r0 + WT * NW;
      RM_G T *p0 = A + (int64_t)r0 * ld + j0;
      RM_G T *p1 = A + (int64_t)r1 * ld + j0;
      const bool h1 = r1 < na;
      T x0[NB], x1[NB];
#pragma unroll
      for (int q = 0; q < NB; ++q) {
        const bool in = q >= jj && q < jb;
        x0[q] = in ? p0[q] : T(0);
        x1[q] = (in && h1) ? p1[q] : T(0);
      }
      T l0 = T(0), l1 = T(0);
#pragma unroll
      for (int q = 0; q < NB; ++q)
        if (q == jj) {
          l0 = x0[q] * inv;
          l1 = x1[q] * inv;
        }
#pragma unroll
      for (int q = 0; q < NB; ++q) {
        if (q < jj || q >= jb) continue;
        const T v0 = q == jj ? l0 : fma(-l0, pc[q], x0[q]);
        const T v1 = q == jj ? l1 : fma(-l1, pc[q], x1[q]);
        p0[q] = v0;
        if (h1) p1[q] = v1;
      }
    }
    team_sync<NW>();
  }
  return flag;
}

// Factor the block of columns [j0, j0 + jb) (jb <= 32) of rows [j0, na) in
// registers: thread t of the team holds rows j0 + t + 64 NW s (s < R) of the
// panel, all 32 columns, and no row ever moves: an interchange swaps the two
// rows' positions, and each row is stored at its final one.  Per column one
// barrier: each wavefront's best candidate publishes its magnitude, position
// and remaining row in LDS, every thread picks the team's pivot (largest
// magnitude, then smallest position) and eliminates its own rows.  Leaves
// the block's factors in W.T (L11 below the diagonal, U11 on and above it,
// identity padding), the row moves of its interchanges in W (srcp, opos,
// osrc, nout) and, if asked, the pivots in W.piv.  Returns 1 if a pivot was
// zero or not a number.
template <int NW, int R, class T>
__device__ __forceinline__ int team_panel_regs(RM_G T *A, int na, int ld,
                                               int j0, int jb, bool want_piv,
                                               RM_L TeamLds<NW> &W) {
  na = uni(na); ld = uni(ld); j0 = uni(j0); jb = uni(jb);
  const int lane = lane_id(), tid = team_tid<NW>(), wv = team_wave<NW>();
  constexpr int GW = 8, NG = NB2 / GW;  // columns per group, groups
  T x[R][NB2];
  int pos[R];
#pragma unroll
  for (int s = 0; s < R; ++s) {
    const int r = j0 + tid + WT * NW * s;
    pos[s] = r < na ? r : -1;  // -1: no row
#pragma unroll
    for (int q = 0; q < NB2; ++q)
      x[s][q] = (r < na && q < jb) ? A[(int64_t)r * ld + j0 + q] : T(0);
  }
  if (tid == 0) W.nout = 0;
  int flag = 0;
  // 8 columns per turn, at register indices 0..7; the registers then rotate
  // by one group, so the code is one group's (all 32 columns written out
  // take 45 KB of instructions)
#pragma unroll 1
  for (int g = 0; g < NG; ++g) {
#pragma unroll
    for (int jj = 0; jj < GW; ++jj) {
      if (GW * g + jj >= jb) continue;  // uniform
      const int col = j0 + GW * g + jj, bf = jj & 1;
      // this thread's candidate, then the wavefront's (a row at a position
      // above col is done; NaN never compares larger)
      double ba = -1.0;
      int bp = na;
#pragma unroll
      for (int s = 0; s < R; ++s) {
        const double a = fabs((double)x[s][jj]);
        if (pos[s] >= col && (a > ba || (a == ba && pos[s] < bp))) {
          ba = a;
          bp = pos[s];
        }
      }
      const double wm = wave_max(ba);
      unsigned long long who = __ballot(ba == wm && bp < na);
      int wp = na, wl = -1;
      while (who) {  // almost always one lane
        const int l = __builtin_ctzll(who);
        who &= who - 1;
        const int p = __builtin_amdgcn_readlane(bp, l);
        if (p < wp) {
          wp = p;
          wl = l;
        }
      }
      if (lane == 0) {
        W.cmax[bf][wv] = wl >= 0 ? wm : -1.0;
        W.cpos[bf][wv] = wp;
      }
      if (lane == wl) {
#pragma unroll
        for (int b = 0; b < NG; ++b) {
          if (b > 0 && g + b >= NG) continue;
#pragma unroll
          for (int q = b == 0 ? jj : GW * b; q < GW * b + GW; ++q) {
            T v = x[0][q];
#pragma unroll
            for (int s = 1; s < R; ++s)
              if (pos[s] == wp) v = x[s][q];
            W.cand[bf][wv][q] = (double)v;
          }
        }
      }
      team_sync<NW>();
      double best = -1.0;
      int pr = na, pw = 0;
#pragma unroll
      for (int w = 0; w < NW; ++w) {
        const double a = W.cmax[bf][w];
        const int p = W.cpos[bf][w];
        if (a > best || (a == best && p < pr)) {
          best = a;
          pr = p;
          pw = w;
        }
      }
      pr = __builtin_amdgcn_readfirstlane(pr);
      pw = __builtin_amdgcn_readfirstlane(pw);
      const bool bad = pr >= na;  // every candidate is NaN
      if (bad) pr = col;
      const T pv = bad ? (T)__builtin_nan("") : (T)W.cand[bf][pw][jj];
      if (want_piv && tid == 0) W.piv[GW * g + jj] = pr;
      if (!(fabs(pv) > T(0))) flag = 1;
      const T inv = T(1) / pv;
      T l[R];
#pragma unroll
      for (int s = 0; s < R; ++s) {
        pos[s] = pos[s] == pr ? col : pos[s] == col ? pr : pos[s];
        // rows at or above the pivot keep their values: multiplier 0 below
        const bool el = pos[s] > col;
        l[s] = el ? x[s][jj] * inv : T(0);
        if (el) x[s][jj] = l[s];
      }
#pragma unroll
      for (int b = 0; b < NG; ++b) {
        if (b > 0 && g + b >= NG) continue;  // uniform: done columns
#pragma unroll
        for (int q = b == 0 ? jj + 1 : GW * b; q < GW * b + GW; ++q) {
          const T pc = (T)W.cand[bf][pw][q];
#pragma unroll
          for (int s = 0; s < R; ++s)
            if (pos[s] > col) x[s][q] = fma(-l[s], pc, x[s][q]);
        }
      }
    }
#pragma unroll
    for (int s = 0; s < R; ++s) {
      T k[GW];
#pragma unroll
      for (int q = 0; q < GW; ++q) k[q] = x[s][q];
#pragma unroll
      for (int q = 0; q < NB2 - GW; ++q) x[s][q] = x[s][q + GW];
#pragma unroll
      for (int q = 0; q < GW; ++q) x[s][NB2 - GW + q] = k[q];
    }
  }
  // rows to their positions, the block's own rows to W.T, the moves
#pragma unroll
  for (int s = 0; s < R; ++s) {
    const int r = j0 + tid + WT * NW * s, p = pos[s];
    if (p < 0) continue;
#pragma unroll
    for (int q = 0; q < NB2; ++q)
      if (q < jb) A[(int64_t)p * ld + j0 + q] = x[s][q];
    if (p < j0 + jb) {
      W.srcp[p - j0] = r;
#pragma unroll
      for (int q = 0; q < NB2; ++q)
        W.T[p - j0][q] = q < jb ? (double)x[s][q] : 0.0;
    } else if (p != r) {
      const int m = atomicAdd((int *)&W.nout, 1);
      W.opos[m] = p;
      W.osrc[m] = r;
    }
  }
  for (int q = tid; q < (NB2 - jb) * NB2; q += WT * NW) {
    const int i = jb + q / NB2, j = q % NB2;
    W.T[i][j] = i == j ? 1.0 : 0.0;
  }
  team_sync<NW>();
  return flag;
}

// Invert a triangle of the 32 x 32 block T, one wavefront (lanes 0..31 each
// form one column of the inverse and put(row, column, value) it; no barrier).  Kinds: unit lower
// triangle (L11 of the LU), upper triangle with its diagonal (U11), lower
// triangle with its diagonal (a Cholesky factor).  Padded rows and columns
// must hold the identity; the other triangle is not read.
enum TileKind { TILE_UNIT_LOWER = 0, TILE_UPPER = 1, TILE_LOWER = 2 };
template <int KIND, class PUT>
__device__ __forceinline__ void wave_tile_invert(const RM_L double (*T)[NB2 + 1], PUT put) {
  const int j = lane_id();  // column of the inverse formed by this lane
  double x[NB2];
  if constexpr (KIND != TILE_UPPER) {
#pragma unroll
    for (int q = 0; q < NB2; ++q) {
      double acc = q == j ? 1.0 : 0.0;
#pragma unroll
      for (int p = 0; p < q; ++p) acc = fma(-T[q][p], x[p], acc);
      if constexpr (KIND == TILE_LOWER) acc /= T[q][q];
      x[q] = acc;
    }
  } else {
#pragma unroll
    for (int q = NB2 - 1; q >= 0; --q) {
      double acc = q == j ? 1.0 : 0.0;
#pragma unroll
      for (int p = q + 1; p < NB2; ++p) acc = fma(-T[q][p], x[p], acc);
      x[q] = acc / T[q][q];
    }
  }
  if (j < NB2) {
#pragma unroll
    for (int q = 0; q < NB2; ++q) put(q, j, x[q]);
  }
}

// Stage rows and columns [j0, j0 + jb) of A into dst with identity padding
// to 32 x 32, one triangle (TILE_UPPER, TILE_LOWER: the other is zero) or
// the whole block (ALL).
template <int NW, bool ALL, class T>
__device__ __forceinline__ void team_tile_stage(const RM_G T *A, int ld, int j0, int jb,
                                RM_L double (*dst)[NB2 + 1], int kind) {
  ld = uni(ld); j0 = uni(j0); jb = uni(jb); kind = uni(kind);
  for (int q = team_tid<NW>(); q < NB2 * NB2; q += WT * NW) {
    const int i = q / NB2, j = q % NB2;
    double v = i == j ? 1.0 : 0.0;
    const bool in = ALL || (kind == TILE_UPPER ? j >= i : j <= i);
    if (i < jb && j < jb)
      v = in ? (double)A[(int64_t)(j0 + i) * ld + j0 + j] : 0.0;
    dst[i][j] = v;
  }
  team_sync<NW>();
}

// Row moves of the cnt interchanges W.piv[po + q] at positions j0 + q
// (they act in sequence; a position, once passed, is never moved again):
// W.srcp, W.opos, W.osrc, W.nout.  The first wavefront holds the tables in
// registers, entry q or m in lane q or m.
template <int NW>
__device__ __forceinline__ void team_build_moves(RM_L TeamLds<NW> &W, int j0, int cnt, int po = 0) {
  j0 = uni(j0); cnt = uni(cnt); po = uni(po);
  team_sync<NW>();
  if (team_wave<NW>() == 0) {
    const int lane = lane_id();
    const int pv = lane < cnt ? W.piv[po + lane] : 0;
    int src = j0 + lane, opos = -1, osrc = 0, nout = 0;
    for (int q = 0; q < cnt; ++q) {
      const int p = __builtin_amdgcn_readlane(pv, q);
      if (p == j0 + q) continue;
      const int t = __builtin_amdgcn_readlane(src, q);
      if (p < j0 + cnt) {
        const int o = __builtin_amdgcn_readlane(src, p - j0);
        src = lane == q ? o : lane == p - j0 ? t : src;
      } else {
        const unsigned long long hit = __ballot(lane < nout && opos == p);
        const int m = hit ? __builtin_ctzll(hit) : nout;
        if (!hit) {
          if (lane == m) opos = osrc = p;
          ++nout;
        }
        const int o = __builtin_amdgcn_readlane(osrc, m);
        if (lane == q) src = o;
        if (lane == m) osrc = t;
      }
    }
    if (lane < NB2) {
      W.srcp[lane] = src;
      W.opos[lane] = opos;
      W.osrc[lane] = osrc;
    }
    if (lane == 0) W.nout = nout;
  }
  team_sync<NW>();
}

// Columns [c0, c1) of rows j0 .. j0+31:  X <- Ti X (or Ti^T X), where row q of X is
// taken from row srcp[q] (moves) or row j0 + q, and rows opos[m] receive
// rows osrc[m] (m < nout) in the same pass; only rows q < jb are written.
// 16 x 16 FP64 MFMA blocks over 8 k-steps; every load of a batch is
// issued before any store, so sources and destinations may coincide.
template <int NW, bool TRANS = false, class T = double>
__device__ __forceinline__ void team_tile_apply(RM_G T *A, int ld, int j0, int jb, int c0,
                                int c1, const RM_L TeamLds<NW> &W, bool moves) {
  ld = uni(ld); j0 = uni(j0); jb = uni(jb); c0 = uni(c0); c1 = uni(c1);
  constexpr int NS = NB2 / 4, NRB = NB2 / 16, CB = 2;
  typedef typename Mx<T>::acc acc_t;
  const int lane = lane_id();
  const int col = lane & 15, kq = lane >> 4;
  T ainv[NRB][NS];  // Ti, or its transpose
#pragma unroll
  for (int rb = 0; rb < NRB; ++rb)
#pragma unroll
    for (int s = 0; s < NS; ++s)
      ainv[rb][s] = (T)(TRANS ? W.Ti[4 * s + kq][rb * 16 + col]
                              : W.Ti[rb * 16 + col][4 * s + kq]);
  int srow[NS], orow[NS], drow[NS];
  bool sv[NS], ov[NS];
  const int nout = moves ? W.nout : 0;
#pragma unroll
  for (int s = 0; s < NS; ++s) {
    const int q = 4 * s + kq;
    sv[s] = q < jb;
    srow[s] = moves ? (sv[s] ? W.srcp[q] : 0) : j0 + q;
    ov[s] = q < nout;
    orow[s] = ov[s] ? W.osrc[q] : 0;
    drow[s] = ov[s] ? W.opos[q] : 0;
  }
  for (int cb = c0 + team_wave<NW>() * 16 * CB; cb < c1; cb += NW * 16 * CB) {
    T b[CB][NS], y[CB][NS];
#pragma unroll
    for (int u = 0; u < CB; ++u) {
      const int c = cb + 16 * u + col;
      const bool cv = c < c1;
#pragma unroll
      for (int s = 0; s < NS; ++s) {
        b[u][s] = (cv && sv[s]) ? A[(int64_t)srow[s] * ld + c] : T(0);
        y[u][s] = (cv && ov[s]) ? A[(int64_t)orow[s] * ld + c] : T(0);
      }
    }
#pragma unroll
    for (int u = 0; u < CB; ++u) {
      acc_t acc[NRB];
#pragma unroll
      for (int rb = 0; rb < NRB; ++rb) acc[rb] = acc_t{0, 0, 0, 0};
#pragma unroll
      for (int s = 0; s < NS; ++s)
#pragma unroll
        for (int rb = 0; rb < NRB; ++rb)
          acc[rb] = Mx<T>::mfma(ainv[rb][s], b[u][s], acc[rb]);
      const int c = cb + 16 * u + col;
      if (c < c1) {
#pragma unroll
        for (int s = 0; s < NS; ++s)
          if (ov[s]) A[(int64_t)drow[s] * ld + c] = y[u][s];
#pragma unroll
        for (int rb = 0; rb < NRB; ++rb)
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const int q = rb * 16 + Mx<T>::row(kq, r);  // result row
            if (q < jb) A[(int64_t)(j0 + q) * ld + c] = acc[rb][r];
          }
      }
    }
  }
  team_sync<NW>();
}

// The triangles' inverses of the block in W.T: L11^-1 into W.Ti and U11^-1
// over U11 in A (its strict lower part keeps L11), by two wavefronts at once
// where the team has them.
template <int NW, class T>
__device__ __forceinline__ void team_invert_lu(RM_G T *A, int ld, int j0, int jb, RM_L TeamLds<NW> &W) {
  ld = uni(ld); j0 = uni(j0); jb = uni(jb);
  const int wv = team_wave<NW>();
  if (wv == 0)
    wave_tile_invert<TILE_UNIT_LOWER>(
        W.T, [&](int i, int j, double v) { W.Ti[i][j] = v; });
  if (wv == NW - 1)
    wave_tile_invert<TILE_UPPER>(W.T, [&](int i, int j, double v) {
      if (i <= j && j < jb) A[(int64_t)(j0 + i) * ld + j0 + j] = (T)v;
    });
  team_sync<NW>();
}

// Back substitution U X = B' on the right-hand sides in columns [na, na +
// nrhs), 32 rows at a time, with U11^-1 in place of the diagonal blocks.
// Left-looking: a block's rows take the solved rows below at once
// (X_b -= U[b, >b] X[>b]), so the right-hand sides above are not rewritten
// once per block.
template <int NW, class T>
__device__ __forceinline__ void team_back_subst(RM_G T *A, int na, int ld, int nrhs,
                                RM_L TeamLds<NW> &W) {
  na = uni(na); ld = uni(ld); nrhs = uni(nrhs);
  for (int j0 = ((na - 1) / NB2) * NB2; j0 >= 0; j0 -= NB2) {
    const int jb = min(NB2, na - j0);
    const int r1 = j0 + jb;
    team_tile_stage<NW, false>(A, ld, j0, jb, W.Ti, TILE_UPPER);
    if (r1 < na)
      team_gemm_wide<NW, 0, 0, 2, 4>(A + (int64_t)j0 * ld + na, ld,
                                     A + (int64_t)j0 * ld + r1, ld,
                                     A + (int64_t)r1 * ld + na, ld, jb, nrhs,
                                     na - r1);
    team_tile_apply<NW>(A, ld, j0, jb, na, na + nrhs, W, false);
  }
}

// Solve A X = B in place for the na x na matrix in columns [0, na) of rows
// [0, na) (leading dimension ld), right-hand sides in columns
// [na, na + nrhs); on return those columns hold X.  Blocks of 32 columns: the
// panel, then the block's interchanges and L11^-1 applied to the columns on
// its right and one rank-32 trailing update, so the trailing matrix is read
// and written once per 32 columns.  On return the diagonal blocks hold
// U11^-1.  Returns nonzero if a pivot was zero or not a number.  piv
// (nullable) receives the pivot row of every column, block by block, for
// later solves with the factors (team_lu_resolve).
//
// NAMAX bounds na.  The panel is held in registers up to two rows per thread
// (512 rows for four wavefronts, 1024 for eight: 128 registers a lane; more
// would spill), and in memory, as two 16-column panels, above.
template <int NW, int NAMAX, class T>
__device__ __forceinline__ int team_lu_solve(RM_G T *A, int na, int ld, int nrhs, RM_L TeamLds<NW> &W,
                             RM_G int *piv = nullptr) {
  na = uni(na); ld = uni(ld); nrhs = uni(nrhs);
  const int ntot = na + nrhs, tid = team_tid<NW>();
  int flag = 0;
  for (int j0 = 0; j0 < na; j0 += NB2) {
    const int jb = min(NB2, na - j0);
    bool done = false;
    if (NAMAX <= WT * NW || na - j0 <= WT * NW) {
      flag |= team_panel_regs<NW, 1>(A, na, ld, j0, jb, piv != nullptr, W);
      done = true;
    }
    if constexpr (NAMAX > WT * NW) {
      if (!done && na - j0 <= 2 * WT * NW) {
        flag |= team_panel_regs<NW, 2>(A, na, ld, j0, jb, piv != nullptr, W);
        done = true;
      }
    }
    if constexpr (NAMAX > 2 * WT * NW) {
      if (!done) {
        const int ja = min(NB, jb);
        // two 16-column panels; turn 1: the first one's interchanges and
        // L^-1 on the second one's columns and its update of them, then
        // the second panel
#pragma unroll 1
        for (int h = 0; h < 2 && h * NB < jb; ++h) {
          if (h) {
            team_build_moves(W, j0, ja);
            team_tile_stage<NW, true>(A, ld, j0, ja, W.T, 0);
            if (team_wave<NW>() == 0)
              wave_tile_invert<TILE_UNIT_LOWER>(
                  W.T, [&](int i, int j, double v) { W.Ti[i][j] = v; });
            team_sync<NW>();
            team_tile_apply<NW>(A, ld, j0, ja, j0 + ja, j0 + jb, W, true);
            team_gemm<NW, 0>(A + (int64_t)(j0 + ja) * ld + j0 + ja, ld,
                             A + (int64_t)(j0 + ja) * ld + j0, ld,
                             A + (int64_t)j0 * ld + j0 + ja, ld, na - j0 - ja,
                             jb - ja, ja);
          }
          flag |= team_panel_mem(A, na, ld, j0 + h * NB, h ? jb - ja : ja, j0,
                                 h * NB, W);
        }
        team_build_moves(W, j0, jb);
        team_tile_stage<NW, true>(A, ld, j0, jb, W.T, 0);
      }
    }
    if (piv && tid < jb) piv[j0 + tid] = W.piv[tid];
    team_invert_lu(A, ld, j0, jb, W);
    // the block's interchanges and L11^-1 on every column to its right
    team_tile_apply<NW>(A, ld, j0, jb, j0 + jb, ntot, W, true);
    const int r0 = j0 + jb;
    if (r0 < na)
      team_gemm_wide<NW, 0, 0, 2, 4>(A + (int64_t)r0 * ld + r0, ld,
                                     A + (int64_t)r0 * ld + j0, ld,
                                     A + (int64_t)j0 * ld + r0, ld, na - r0,
                                     ntot - r0, jb);
  }
  team_back_subst(A, na, ld, nrhs, W);
  return flag;
}

// Solve A X = B again with the factors team_lu_solve left in columns
// [0, na) and its pivots `piv`, for new right-hand sides in columns
// [na, na + nrhs); on return those columns hold X.  Same block order as the
// factorisation: per 32-column block its interchanges and L11^-1 on the
// right-hand sides, then the rank-32 update of the rows below (the L
// columns of a block were never permuted by later blocks, so they match the
// right-hand sides at that point), then back substitution with U.
template <int NW, class T>
__device__ __forceinline__ void team_lu_resolve(RM_G T *A, int na, int ld, int nrhs,
                                const RM_G int *piv, RM_L TeamLds<NW> &W) {
  na = uni(na); ld = uni(ld); nrhs = uni(nrhs);
  const int tid = team_tid<NW>();
  for (int j0 = 0; j0 < na; j0 += NB2) {
    const int jb = min(NB2, na - j0);
    if (tid < jb) W.piv[tid] = piv[j0 + tid];
    team_build_moves(W, j0, jb);
    team_tile_stage<NW, true>(A, ld, j0, jb, W.T, 0);
    if (team_wave<NW>() == 0)
      wave_tile_invert<TILE_UNIT_LOWER>(
          W.T, [&](int i, int j, double v) { W.Ti[i][j] = v; });
    team_sync<NW>();
    team_tile_apply<NW>(A, ld, j0, jb, na, na + nrhs, W, true);
    const int r0 = j0 + jb;
    if (r0 < na)
      team_gemm_wide<NW, 0, 0, 2, 4>(A + (int64_t)r0 * ld + na, ld,
                                     A + (int64_t)r0 * ld + j0, ld,
                                     A + (int64_t)j0 * ld + na, ld, na - r0,
                                     nrhs, jb);
  }
  team_back_subst(A, na, ld, nrhs, W);
}

}  // namespace rmx
