// Internal declarations shared by the HIP translation units of librmatrix.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>
#include <algorithm>
#include <utility>
#include <vector>

#include "../../include/rmatrix.h"

namespace rmx {

// Padding granularity of channels and poles in the staged W layouts.
constexpr int kChanPad = 32;
constexpr int kPolePad = 64;
constexpr double kPadPole = 1.0e30;  // padding poles sit far from any energy
// The T step's well-conditioned route (the real 2n x 2n form of
// (1 - iK) W = 1 with its right-hand sides, 6 n^2 doubles) runs at few
// energies, so its buffers form a small pool: the team of slot q takes every
// q-th, (q + slots)-th, ... energy of the chunk that needs the route.  Without
// a pool those energies take the route through Z = L^-1 K instead.
__host__ __device__ inline int64_t t_ext_doubles(int n) {
  return (int64_t)6 * n * n;
}
// Slots of symmetries of up to n channels: `least` of them, more while they take
// no more than `room` bytes together, up to the teams that are resident at once.
// At a tenth of the energies and more the slots are what the chunk waits for
// (20 channels, all of 8192 energies: 13.7 ms with 64 slots, 1.4 with 1024;
// 200 channels, a tenth of 2048: 16.5 ms with 64, 11.3 with 133).
inline int64_t t_ext_slots(int n, int64_t least, double room) {
  const int64_t resident = n <= 32 ? 1024 : n <= 128 ? 512 : 256;
  const int64_t fit = (int64_t)(room / (8.0 * (double)t_ext_doubles(n)));
  return std::min(resident, std::max(least, fit));
}
constexpr int kTExtSlots = 64;       // at least, of an allocating sweep ...
constexpr double kTExtRoom = 256e6;  // ... and more within this
constexpr int kTExtSlotsArena = 16;  // at least, of a sweep that may not allocate

// The asymptotic expansion beyond A works on blocks of kGlCols open
// channels; its per-energy scratch (after the symmetry's workspace) holds a
// doubled ring of 2 Q coefficient slots (Q = max(lmax, 2) + 1), two slots
// of the coupling products, the sums g and g', and two slots for the final
// product with R, each slot n rows of 2 kGlCols doubles (real | imaginary).
// Doubles of one energy's matching workspace of an n-channel symmetry:
// [M | B] n x 2n, K n x n, 2n for photoionization, n pivots.
__host__ __device__ inline int64_t match_work_doubles(int n) {
  return (int64_t)3 * n * n + 3 * n;
}

constexpr int kGlCols = 16;
constexpr int kGlMaxTerms = 200;
__host__ __device__ inline int gl_ring(int lmax) { return (lmax > 2 ? lmax : 2) + 1; }
__host__ __device__ inline int64_t gl_doubles(int n, int lmax) {
  return (int64_t)(2 * gl_ring(lmax) + 6) * n * 2 * kGlCols;
}

// Device-side view of one symmetry (plain data, copied into a descriptor
// table that the grouped kernels index by symmetry number).
struct SymDev {
  int n, nh, n_pad, nh_pad;
  int n_target;
  double a, z, g;
  const double *E_pole;       // [nh_pad] ascending, padding = kPadPole
  const double *Wt;           // [nh_pad][n_pad] FP64, pole-major
  const float *W32c;          // [n_pad][nh_pad] FP32, channel-major
  const uint16_t *Whc, *Wlc;  // [n_pad][nh_pad] BF16 split, channel-major
  const double *e_thr;        // [n] sorted
  const int32_t *l;           // [n] sorted order
  const int32_t *perm;        // [n] sorted position -> input channel
  const int32_t *tgt;         // [n] sorted position -> target level
  int ntu;                    // target levels that hold a channel
  const int32_t *ut;          // [ntu] those levels, ascending
  const double *G;            // [n][ntu] 0/1, channel -> used level
  const double *GT;           // [ntu][n] its transpose
  int np, np_pad;             // pairs i <= j (row-major upper triangle)
  const int32_t *pair_ij;     // [np_pad] (i << 16) | j
  const uint16_t *Ph, *Pl;    // [np_pad][nh_pad] BF16 hi/lo of w_ik w_jk
  const float *P32;           // [np_pad][nh_pad] FP32 w_ik w_jk
  const double *P64;          // [np_pad][nh_pad] FP64 w_ik w_jk
  const double *dip;          // [nh_pad] bound-free dipoles, or null
  const double *gam;          // [nh_pad] radiative widths Gamma_k, or null
  // outer-region propagation from a to A (n_sec = 0: none): sector s
  // rotates the reduced R-matrix by O_s (X <- O_s^T X O_s) and then steps
  // it across width h_sec with eigenvalues eps_s; O_{n_sec} returns to the
  // channel basis.  Sorted channel order, leading dimension n.
  int n_sec;
  double A, h_sec;
  double r_match;             // radius of the matching: A with sectors, else a
  const double *prop_O;       // [n_sec + 1][n][n]
  const double *prop_eps;     // [n_sec][n]
  // asymptotic expansion at A (gl_terms = 0: matching to Coulomb functions):
  // gl_beta [n][lmax n], row i holds beta^lam_im / A^lam for lam = 1..lmax
  int gl_terms, lmax;
  const double *gl_beta;
};

// A symmetry resident on one device.  Channels are stored sorted by
// threshold (stable), so at any energy the open channels are a prefix.
struct Sym {
  int device;
  int n, nh;            // channels, poles
  int n_pad, nh_pad;    // padded to kChanPad / kPolePad
  double a, z, g;
  int n_target;         // max target level + 1
  // device arrays (owned)
  double *E_pole;
  double *Wt;
  float *W32c;
  uint16_t *Whc, *Wlc;  // w = hi + lo + O(2^-16 |w|)
  double *e_thr;
  int32_t *l;
  int32_t *perm;
  int32_t *inv;         // [n] input channel -> sorted position
  int32_t *tgt;
  int ntu;
  int32_t *ut;
  double *G, *GT;
  int np, np_pad;       // channel pairs, padded to the pair-block size
  int32_t *pair_ij;
  uint16_t *Ph, *Pl;    // pair products, formed on first use (owned)
  float *P32;
  double *P64;
  double *dip = nullptr;  // [nh_pad] dipoles with the initial state (owned)
  double *gam = nullptr;  // [nh_pad] radiative widths of the poles (owned)
  int n_sec = 0;          // outer-region sectors (0: match at r = a)
  double A = 0.0, h_sec = 0.0;
  double *prop_O = nullptr, *prop_eps = nullptr;  // owned
  int lmax = 0, gl_terms = 0;   // multipole order; expansion terms (0: off)
  double *gl_beta = nullptr;    // [n][lmax n] beta / A^lam, sorted (owned)
  // host copies
  double *h_e_thr;      // [n] sorted
  int32_t *h_perm;
  SymDev dev() const {
    SymDev d;
    d.n = n; d.nh = nh; d.n_pad = n_pad; d.nh_pad = nh_pad;
    d.n_target = n_target; d.a = a; d.z = z; d.g = g;
    d.E_pole = E_pole; d.Wt = Wt; d.W32c = W32c; d.Whc = Whc; d.Wlc = Wlc;
    d.e_thr = e_thr; d.l = l; d.perm = perm; d.tgt = tgt;
    d.ntu = ntu; d.ut = ut; d.G = G; d.GT = GT;
    d.np = np; d.np_pad = np_pad; d.pair_ij = pair_ij;
    d.Ph = Ph; d.Pl = Pl; d.P32 = P32; d.P64 = P64; d.dip = dip; d.gam = gam;
    d.n_sec = n_sec; d.A = A; d.h_sec = h_sec;
    d.r_match = n_sec > 0 ? A : a;
    d.prop_O = prop_O; d.prop_eps = prop_eps;
    d.gl_terms = n_sec > 0 ? gl_terms : 0;
    d.lmax = lmax;
    d.gl_beta = gl_beta;
    return d;
  }
};

// Per-energy channel data, sorted channel order: (d1, d2, s, a s') with
// d1 = c, d2 = a c' for open channels and (e, a e') of the closed-channel
// function for closed ones.
struct ChanSlot {
  double d1, d2, s, asp;
};

// Work item of the grouped pole-sum kernels: symmetry, two tile
// coordinates (meaning per kernel) and an energy group.
struct PsItem {
  int sym, x, y, grp;
};

// Where the pole sum writes R of symmetry s at chunk energy e:
// out + e*estride + off[s] + i*(ld_mult*n_s) + j.
struct PsOut {
  double *out;
  int64_t estride;
  const int64_t *off;   // device [n_sym]
  int ld_mult;
};

// hipMallocFromPoolAsync from the library's own pool, hipMallocAsync and
// hipMalloc; none of them fails for memory that the pool holds idle.
hipError_t pool_alloc(void **p, size_t bytes, hipStream_t st);
hipError_t stream_malloc(void **p, size_t bytes, hipStream_t st);
hipError_t device_malloc(void **p, size_t bytes);

// Tile variants of the pole-sum kernels (chosen by the autotuner).
enum PsVariant {
  PS_F64_T32_E16 = 0,   // FP64, 32x32 tile pairs, 16 energies per WG
  PS_MX_J16_E8 = 1,     // mixed, 16 column blocks, 8 energies per WG
  PS_MX_J8_E8 = 2,      // mixed, 8 column blocks, 8 energies per WG
  PS_MX_J16_E4 = 3,     // mixed, 16 column blocks, 4 energies per WG
  PS_PD = 4,            // mixed, pair-major GEMM over precomputed w_ik w_jk
  PS_PD64 = 5,          // FP64, pair-major GEMM
  PS_F64_GROUP = 6      // FP64, far poles interpolated over 128 energies
};
constexpr int kPairBlock = 256;   // pairs per pair-major workgroup tile

// ---- launchers (return the hipError_t of the launch) ----

hipError_t launch_chanfn(const Sym &s, const double *E, int64_t m,
                         ChanSlot *chan, int32_t *n_open, int32_t *status,
                         hipStream_t st);

// Grouped pole sum (Sec. 6, Eq. 1-2) over a table of work items that may
// span several symmetries.  FP64 variants use MFMA over every pole; mixed
// variants use FP32 or split-BF16 MFMA over the far poles, |E_k - E| >=
// band, and add the near tier (|E_k - E| < delta, FP64 operands) and the
// band tier (FP32 operands, FP64 products and sum) in their epilogues.
struct PsLaunch {
  const SymDev *syms;
  const PsItem *items;
  int n_items;
  const double *E;
  int m;
  int64_t e_off, m_all; // E[-e_off .. m_all - e_off) is the whole mesh
  int ngrp, units;      // PS_F64_GROUP: groups, and sixteens of energies, a tile
  PsOut out;
  int prec;
  double delta;         // near tier: FP64 operands
  double band;          // band tier (>= delta): FP32 operands, FP64 sum
  // FP64 scaled-W variant only: 0 the weights 1/(E_k - E); 1 and 2 the
  // real and imaginary parts of 1/(E_k - i Gamma_k/2 - E) (damped poles)
  int part;
};
hipError_t launch_polesum(const PsLaunch &L, int variant, hipStream_t st);
hipError_t launch_polesum_pd(const PsLaunch &L, hipStream_t st);
hipError_t launch_polesum_pd64(const PsLaunch &L, hipStream_t st);
hipError_t launch_polesum_group(const PsLaunch &L, hipStream_t st);
// Chunks of poles that PS_F64_GROUP sums for each of the ngrp groups of a mesh
// of m energies, and those of a direct sum: work[g][0], work[g][1] (device).
hipError_t launch_group_work(const SymDev *sym, const double *E, int64_t m,
                             int ngrp, int64_t *work, hipStream_t st);
// The FP64 scaled-W sum of nh poles on a mesh of m energies: in groups from
// 64 energies and 512 poles on.  Far poles then cost 16 energies' work per
// group (200 channels, 8000 poles, mesh step 1e-4: 0.40 ms at 64 energies
// against 1.17); fewer energies than that leave too little to save, and with
// few poles the decision and the interpolation weights are most of the time
// (5 channels, 64 poles: 22 us against 6.8; 33 channels, 1000 poles: 73 us
// against 114).
constexpr int kPsGroupMin = 64, kPsGroupPoles = 512;
inline int ps_f64_variant(int variant, int nh, int64_t m) {
  return variant == PS_F64_T32_E16 && m >= kPsGroupMin && nh >= kPsGroupPoles
             ? PS_F64_GROUP
             : variant;
}
hipError_t launch_pd64_build(const Sym &s, hipStream_t st);
// Form the pair products of s for prec (FP32 or BF16X3) into its planes.
hipError_t launch_pd_build(const Sym &s, int prec, hipStream_t st);
int ps_energy_group(int variant);         // energies per work item
// Energy groups of a chunk of m energies, and (PS_F64_GROUP) how many blocks
// of 16 energies they make.  Groups of that variant are cut on the whole mesh:
// unless chunks begin at multiples of a group (`aligned`) one may begin and
// end inside a group.
int ps_groups(int variant, int64_t m, bool aligned);
int ps_units(int variant, int64_t m, bool aligned);
// Tile items of one symmetry for a variant: (x, y) pairs, in order.
void ps_tiles(const Sym &s, int variant, std::vector<std::pair<int, int>> &out);

// Channel functions, matching, K, T and Omega: one team of wavefronts per
// energy, the symmetries in turn (so an energy's Omega row has one owner).
struct MatchLaunch {
  const SymDev *syms;
  int n_sym;
  const int *h_n;             // host [n_sym]: channels of each symmetry
  const int *h_outer;         // host [n_sym]: 1 sectors, 2 and the expansion
  int sym;                    // the symmetry of a kernel (set per launch)
  const double *E;
  int m;
  // photoionization: the dipole pole sum g of each symmetry sits after its
  // K block in the workspace ([Aug 2n^2 | K n^2 | g n | v n]); sigma[e] is
  // accumulated over the symmetries (nullable)
  double *sigma;
  double e0;
  double *work;               // [M | B] (n x 2n), K (n x n), 2n, n pivots
  int64_t work_estride;
  const int64_t *work_off;    // device [n_sym]
  int *route;                 // device [n_sym][m]: an energy's way (below)
  ChanSlot *chan;
  int64_t chan_estride;
  const int64_t *chan_off;    // device [n_sym]
  int32_t *n_open_out;        // nullable, symmetry 0 only
  double *K_out;              // nullable, symmetry 0 only: [m][n][n]
  const double *K_in;         // nullable, symmetry 0 only (skip matching)
  double *omega;              // nullable
  int64_t omega_stride;
  int n_target_out;
  int32_t *status;            // nullable
  int do_t;
  int solve_fp32;             // FP32 factorisation refined in FP64
  int refine_iters;           // at most this many corrections
  // radiation-damped photoionization: per symmetry the workspace holds the
  // 2n x 2n real form of the complex driven system (leading dimension
  // 2n + 2), then R_re, R_im (n x n each) and g_re, g_im (n each)
  int damped;
  // route: 1 where a step leaves an energy to a later one, which reads it: the
  // FP32 solve to the FP64 factorisation, then the T step to the routes for
  // large K
  // the T step's complex-system pool (nullable): ext_slots slots of
  // ext_estride doubles (at least t_ext_doubles(n) of every symmetry) at
  // ext + slot * ext_estride
  double *ext;
  int64_t ext_estride;
  int ext_slots;
};
enum MatchStep {
  STEP_ASSEMBLE, STEP_ASSEMBLE_DAMPED, STEP_LU, STEP_FP32, STEP_K_OUT, STEP_T,
  STEP_T_COMPLEX, STEP_T_Z, STEP_PHOTO, STEP_DAMPED_SIGMA
};
hipError_t launch_match(const MatchLaunch &L, hipStream_t st);
// R(a) -> R(A) for the symmetries with outer-region sectors (same launch
// description as the matching; run between the pole sum and the matching).
hipError_t launch_propagate(const MatchLaunch &L, hipStream_t st);

// Dipole pole sum g_i(E) = (1/sqrt2) sum_k w_ik d_k / (E_k - E) of one
// symmetry (sorted channel order) at the m energies E, written to
// out + e*estride + off + i.
// part as for PsLaunch: 0 undamped, 1 and 2 the real and imaginary parts
// with damped pole energies E_k - i Gamma_k/2.
hipError_t launch_dip_polesum(const SymDev &S, const double *E, int m,
                              double *out, int64_t estride, int64_t off,
                              hipStream_t st, int part = 0);

hipError_t launch_fill(double *p, int64_t count, double v, hipStream_t st);
hipError_t launch_fill_i32(int32_t *p, int64_t count, int32_t v,
                           hipStream_t st);
// Copy R from sorted to input order into a dense [m][n][n] array.
hipError_t launch_unsort_square(const Sym &s, const double *src,
                                int64_t src_estride, int src_ld, double *dst,
                                int64_t m, hipStream_t st);

// rm_profile stage timing: while rm_profile(1) is in force, the launches a
// scope issues on `st` are bracketed by events recorded under `stage`.
struct ProfileScope {
  ProfileScope(int stage, hipStream_t st);
  ~ProfileScope();
  hipEvent_t end_ = nullptr;
  hipStream_t st_;
};

}  // namespace rmx
