// Learned adaptive mesh: a small MLP trained on the device, and the
// density -> mesh placement.
//
// The network maps per-window features of a scattering system to a
// log-density of mesh points.  Layers are dense, width W, SiLU activations
// (x sigma(x)) between them and a linear output.  Matrix products run on the
// gfx950 matrix cores with BF16 operands (weights and activations rounded to
// BF16 as they enter a product) and FP32 accumulation (v_mfma_f32_16x16x32_bf16);
// a debug precision runs the same kernels with FP32 operands
// (v_mfma_f32_16x16x4f32).  Master weights, gradients and Adam moments are
// FP32.  Parameters are one flat FP32 array: per layer W_l [out][in] then
// b_l [out].
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdint>
#include <cstring>
#include <new>
#include <vector>

#include "rm_internal.h"

namespace rmx {

typedef float f4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf8 __attribute__((ext_vector_type(8)));

const char *set_error(int code, const char *msg);  // defined in rm_api.hip

__device__ inline float sigm(float x) { return 1.f / (1.f + expf(-x)); }

// What a product's result goes through on its way out.
enum { EPI_FORWARD, EPI_BACKWARD, EPI_WEIGHTS };

// One product C = A B of a layer, FP32 in memory.  Operands are stored with
// the summed index k contiguous, X[row * ld + k], or (transposed) with the
// row contiguous, X[k * ld + row].
struct MlpProduct {
  const float *A, *B;
  int lda, ldb;
  int M, N, K;
  const float *bias;  // forward: b_l
  float *Z, *out;     // forward: pre-activations; the result
  const float *Zin;   // backward: pre-activations of the layer below
  float *db;          // weights: the bias gradient, sum over k of A's rows
  int act;            // forward: SiLU, else linear
};

// Eight consecutive k of one operand row for this lane, zero from K on.
// `whole` (uniform): the 32-wide chunk ends at or before K.
// (The compiler joins the contiguous ones into 16-byte loads, which need no
// alignment here.)
template <bool TR>
__device__ __forceinline__ void mlp_load(float (&x)[8], const float *X, int ld,
                                         int row, int k, int K, bool whole) {
  if (whole) {
#pragma unroll
    for (int q = 0; q < 8; ++q)
      x[q] = TR ? X[(int64_t)(k + q) * ld + row] : X[(int64_t)row * ld + k + q];
  } else {
#pragma unroll
    for (int q = 0; q < 8; ++q)
      x[q] = k + q >= K ? 0.f
             : TR       ? X[(int64_t)(k + q) * ld + row]
                        : X[(int64_t)row * ld + k + q];
  }
}

// The layers are small (a 256-wide layer of 1024 samples is 0.13 GFLOP on
// 2 MB that sit in L2), so a product is bound by its chain of loads and by
// launches, not by the matrix cores.  Operands therefore go from L2 to the
// fragment registers without LDS or barriers, G chunks of 32 k at a time and
// the next group in flight during the products; tiles are small enough that
// such a layer fills the chip, and everything elementwise rides on the
// product: bias and activation (forward), the activation's derivative
// (backward), the bias gradient (weights).  Through LDS with a barrier pair
// per 32 k and scalar strided loads a product took 48 us, and the bias
// gradient, one thread per column, 178 us; a step of 16 -> 256 -> 256 -> 256
// -> 1 with 1024 samples took 1280 us and takes 74 us.
//
// A wavefront holds 16 F x 16 F of the result.  Forward and backward: WJ
// wavefronts side by side, 4 / WJ above each other, each summing all of K in
// steps of 32 in ascending order.
// Weights: K is the batch, the longest index, and the result the smallest,
// so the block's KW wavefronts split K and add their parts in LDS in a fixed
// order.  The bias gradient sums A's FP32 values before they are rounded.
template <bool BF16, int EPI, int F, int WJ, int KW>
__global__ __launch_bounds__(EPI == EPI_WEIGHTS ? 64 * KW : 256) void mlp_product_kernel(
    MlpProduct p) {
  constexpr bool TA = EPI == EPI_WEIGHTS, TB = EPI != EPI_FORWARD;
  constexpr int G = F == 1 ? 4 : F == 2 ? 2 : 1;
  constexpr int WI = EPI == EPI_WEIGHTS ? 1 : 4 / WJ;
  constexpr int TW = 16 * F;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int col = lane & 15, kq = lane >> 4;
  const int i0 = (blockIdx.y * WI + (EPI == EPI_WEIGHTS ? 0 : wave / WJ)) * TW;
  const int j0 = (blockIdx.x * WJ + (EPI == EPI_WEIGHTS ? 0 : wave % WJ)) * TW;
  // this wavefront's k: all, or its share in whole chunks
  int kb = 0, ke = p.K;
  if (EPI == EPI_WEIGHTS) {
    const int per = ((p.K + 31) / 32 + KW - 1) / KW * 32;
    kb = min(p.K, wave * per);
    ke = min(p.K, kb + per);
  }
  // rows past the edge read the last one; what they give is not stored
  int ri[F], rj[F];
#pragma unroll
  for (int t = 0; t < F; ++t) {
    ri[t] = min(i0 + 16 * t + col, p.M - 1);
    rj[t] = min(j0 + 16 * t + col, p.N - 1);
  }
  f4 acc[F][F];
  float rs[F];
#pragma unroll
  for (int x = 0; x < F; ++x) {
    rs[x] = 0.f;
#pragma unroll
    for (int y = 0; y < F; ++y) acc[x][y] = f4{0.f, 0.f, 0.f, 0.f};
  }
  float a[G][F][8], b[G][F][8], an[G][F][8], bn[G][F][8];
  auto load = [&](float (&u)[G][F][8], float (&v)[G][F][8], int k0) {
#pragma unroll
    for (int g = 0; g < G; ++g) {
      const int kc = k0 + 32 * g;
      const bool whole = kc + 32 <= ke;
#pragma unroll
      for (int t = 0; t < F; ++t) {
        mlp_load<TA>(u[g][t], p.A, p.lda, ri[t], kc + 8 * kq, ke, whole);
        mlp_load<TB>(v[g][t], p.B, p.ldb, rj[t], kc + 8 * kq, ke, whole);
      }
    }
  };
  if (kb < ke) load(a, b, kb);
  for (int k0 = kb; k0 < ke; k0 += 32 * G) {
    if (k0 + 32 * G < ke) load(an, bn, k0 + 32 * G);
#pragma unroll
    for (int g = 0; g < G; ++g) {
      if (k0 + 32 * g >= ke) break;
      if (EPI == EPI_WEIGHTS) {
#pragma unroll
        for (int t = 0; t < F; ++t)
#pragma unroll
          for (int q = 0; q < 8; ++q) rs[t] += a[g][t][q];
      }
      if (BF16) {
        bf8 af[F], bf[F];
#pragma unroll
        for (int t = 0; t < F; ++t)
#pragma unroll
          for (int q = 0; q < 8; ++q) {
            af[t][q] = (__bf16)a[g][t][q];
            bf[t][q] = (__bf16)b[g][t][q];
          }
#pragma unroll
        for (int x = 0; x < F; ++x)
#pragma unroll
          for (int y = 0; y < F; ++y)
            acc[x][y] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                af[x], bf[y], acc[x][y], 0, 0, 0);
      } else {
        // step q takes k = 8 kq + q of every lane
#pragma unroll
        for (int q = 0; q < 8; ++q)
#pragma unroll
          for (int x = 0; x < F; ++x)
#pragma unroll
            for (int y = 0; y < F; ++y)
              acc[x][y] = __builtin_amdgcn_mfma_f32_16x16x4f32(
                  a[g][x][q], b[g][y][q], acc[x][y], 0, 0, 0);
      }
    }
#pragma unroll
    for (int g = 0; g < G; ++g)
#pragma unroll
      for (int t = 0; t < F; ++t)
#pragma unroll
        for (int q = 0; q < 8; ++q) {
          a[g][t][q] = an[g][t][q];
          b[g][t][q] = bn[g][t][q];
        }
  }
  // D[i][j]: j = lane % 16, i = 4 (lane / 16) + r
  if constexpr (EPI == EPI_WEIGHTS) {
    __shared__ float part[KW][F * F * 4][64];
    __shared__ float rows[KW][F][64];
#pragma unroll
    for (int x = 0; x < F; ++x) {
      rows[wave][x][lane] = rs[x];
#pragma unroll
      for (int y = 0; y < F; ++y)
#pragma unroll
        for (int r = 0; r < 4; ++r) part[wave][(x * F + y) * 4 + r][lane] = acc[x][y][r];
    }
    __syncthreads();
    for (int q = tid; q < F * F * 256; q += 64 * KW) {
      const int f = q >> 6, ln = q & 63, r = f & 3, y = (f >> 2) % F, x = (f >> 2) / F;
      const int gi = i0 + 16 * x + 4 * (ln >> 4) + r, gj = j0 + 16 * y + (ln & 15);
      float s = 0.f;
#pragma unroll
      for (int w = 0; w < KW; ++w) s += part[w][f][ln];
      if (gi < p.M && gj < p.N) p.out[(int64_t)gi * p.N + gj] = s;
    }
    if (blockIdx.x == 0 && tid < TW && i0 + tid < p.M) {
      float s = 0.f;
#pragma unroll
      for (int w = 0; w < KW; ++w)
#pragma unroll
        for (int h = 0; h < 4; ++h) s += rows[w][tid >> 4][16 * h + (tid & 15)];
      p.db[i0 + tid] = s;
    }
  } else {
#pragma unroll
    for (int x = 0; x < F; ++x)
#pragma unroll
      for (int y = 0; y < F; ++y)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int gi = i0 + 16 * x + 4 * kq + r, gj = j0 + 16 * y + col;
          if (gi >= p.M || gj >= p.N) continue;
          const int64_t o = (int64_t)gi * p.N + gj;
          if (EPI == EPI_FORWARD) {
            const float z = acc[x][y][r] + p.bias[gj];
            p.Z[o] = z;
            p.out[o] = p.act ? z * sigm(z) : z;
          } else {
            // dZ = dA silu'(Z)
            const float z = p.Zin[o], s = sigm(z);
            p.out[o] = acc[x][y][r] * s * (1.f + z * (1.f - s));
          }
        }
  }
}

// MSE: loss = mean (y - t)^2, dY = 2 (y - t) / B; one workgroup
__global__ void mse_kernel(const float *Y, const float *T, float *dY,
                           float *loss, int B) {
  __shared__ float red[256];
  float s = 0.f;
  for (int b = threadIdx.x; b < B; b += 256) {
    const float d = Y[b] - T[b];
    dY[b] = 2.f * d / B;
    s += d * d;
  }
  red[threadIdx.x] = s;
  __syncthreads();
  for (int w = 128; w > 0; w >>= 1) {
    if ((int)threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x == 0 && loss) *loss = red[0] / B;
}

__global__ void adam_kernel(float *p, const float *g, float *m, float *v,
                            int64_t n, float lr, float b1, float b2, float eps,
                            float c1, float c2) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const float gi = g[i];
  const float mi = b1 * m[i] + (1.f - b1) * gi;
  const float vi = b2 * v[i] + (1.f - b2) * gi * gi;
  m[i] = mi;
  v[i] = vi;
  p[i] -= lr * (mi / c1) / (sqrtf(vi / c2) + eps);
}

__global__ void copy_f32_kernel(const float *s, float *d, int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) d[i] = s[i];
}

// Mesh placement: cum[w] = exclusive prefix of the floored, normalised
// density; one workgroup, sequential blocks of windows per thread.
__global__ void density_cdf_kernel(const float *dens, int nw, double floor_frac,
                                   double *cum) {
  __shared__ double part[256];
  __shared__ double tot_s;
  const int tid = threadIdx.x;
  const int per = (nw + 255) / 256;
  const int w0 = min(nw, tid * per), w1 = min(nw, w0 + per);
  double s = 0.0;
  for (int w = w0; w < w1; ++w) s += fmax((double)dens[w], 0.0);
  part[tid] = s;
  __syncthreads();
  if (tid == 0) {
    double t = 0.0;
    for (int q = 0; q < 256; ++q) {
      const double v = part[q];
      part[q] = t;
      t += v;
    }
    tot_s = t;
  }
  __syncthreads();
  const double tot = tot_s;
  const double fl = floor_frac / nw;
  const double sc = tot > 0.0 ? (1.0 - floor_frac) / tot : 0.0;
  const double fl2 = tot > 0.0 ? fl : 1.0 / nw;
  double run = part[tid] * sc + w0 * fl2;
  for (int w = w0; w < w1; ++w) {
    cum[w] = run;
    run += fmax((double)dens[w], 0.0) * sc + fl2;
  }
  if (tid == 255) cum[nw] = 1.0;
}

__global__ void mesh_place_kernel(const double *cum, int nw, double lo,
                                  double hi, int64_t M, double *E) {
  const int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (j >= M) return;
  const double u = (j + 0.5) / (double)M;
  int a = 0, b = nw;  // largest w with cum[w] <= u
  while (b - a > 1) {
    const int mid = (a + b) >> 1;
    if (cum[mid] <= u)
      a = mid;
    else
      b = mid;
  }
  const double c0 = cum[a], c1 = cum[a + 1];
  const double f = c1 > c0 ? (u - c0) / (c1 - c0) : 0.5;
  const double h = (hi - lo) / nw;
  E[j] = lo + (a + fmin(fmax(f, 0.0), 1.0)) * h;
}

struct Mlp {
  int d_in, width, layers, prec;
  std::vector<int> din, dout;        // per layer
  std::vector<int64_t> woff, boff;   // offsets into the flat array
  int64_t n_params;
  float *p, *g, *m, *v;              // device [n_params]
  int64_t step;
  int cap_b;                         // activation capacity (batch)
  float *Z, *A, *dA, *dZ, *Y;        // device activations
  int device;
};

static unsigned g1(int64_t n) { return (unsigned)((n + 255) / 256); }

// Launch of a product.  A block's result is 32 x 32 (weights: 16 x 16) while
// that gives up to 1024 blocks, four per CU; beyond, four times as large,
// which halves what each multiply reads.  From 2048 blocks of 64 x 64 on a
// wavefront holds 64 x 64 by itself, which halves it once more and still gives
// every CU two blocks (width 256, forward of 65536 samples 319 us, with 32 x 32
// a wavefront 519; of 16384, 1024 blocks, 141 us); up to 64 columns the
// four wavefronts stand above each other.
template <bool BF16, int EPI, int F, int WJ>
static void launch_product(const MlpProduct &p, hipStream_t st) {
  constexpr int KW = 8, TJ = 16 * F * WJ;
  constexpr int TI = EPI == EPI_WEIGHTS ? 16 * F : 16 * F * (4 / WJ);
  const dim3 grid((p.N + TJ - 1) / TJ, (p.M + TI - 1) / TI);
  hipLaunchKernelGGL((mlp_product_kernel<BF16, EPI, F, WJ, KW>), grid,
                     dim3(EPI == EPI_WEIGHTS ? 64 * KW : 256), 0, st, p);
}

template <bool BF16, int EPI>
static void product_of(const MlpProduct &p, hipStream_t st) {
  constexpr int WJ = EPI == EPI_WEIGHTS ? 1 : 2, T = 16 * WJ;
  auto blocks = [&](int t) {
    return (int64_t)((p.N + t - 1) / t) * ((p.M + t - 1) / t);
  };
  if (blocks(T) <= 1024) return launch_product<BF16, EPI, 1, WJ>(p, st);
  if constexpr (EPI != EPI_WEIGHTS)
    if (blocks(64) >= 2048)
      return p.N <= 64 ? launch_product<BF16, EPI, 4, 1>(p, st)
                       : launch_product<BF16, EPI, 4, 2>(p, st);
  launch_product<BF16, EPI, 2, WJ>(p, st);
}

template <int EPI>
static void product(const Mlp &q, const MlpProduct &p, hipStream_t st) {
  q.prec == 0 ? product_of<true, EPI>(p, st) : product_of<false, EPI>(p, st);
}

static int ensure_cap(Mlp &q, int B) {
  if (B <= q.cap_b) return RM_OK;
  for (float *x : {q.Z, q.A, q.dA, q.dZ, q.Y})
    if (x) (void)hipFree(x);
  q.Z = q.A = q.dA = q.dZ = q.Y = nullptr;
  q.cap_b = 0;  // until they are there again
  const size_t per = (size_t)B * q.width * q.layers * sizeof(float);
  hipError_t e = device_malloc((void **)&q.Z, per);
  if (e == hipSuccess) e = device_malloc((void **)&q.A, per);
  const size_t one = (size_t)B * std::max(q.width, q.d_in) * sizeof(float);
  if (e == hipSuccess) e = device_malloc((void **)&q.dA, one);
  if (e == hipSuccess) e = device_malloc((void **)&q.dZ, one);
  if (e == hipSuccess) e = device_malloc((void **)&q.Y, (size_t)B * sizeof(float));
  if (e != hipSuccess) return RM_ERR_NOMEM;
  q.cap_b = B;
  return RM_OK;
}

// Z_l / A_l of layer l live at offset l*B*width (the last layer uses width 1
// of its slot); the input is X.
static void forward(Mlp &q, const float *X, int B, hipStream_t st) {
  const float *in = X;
  for (int l = 0; l < q.layers; ++l) {
    MlpProduct p{};
    // Z[b][j] = sum_k in[b][k] W[j][k] + b[j]
    p.A = in;
    p.B = q.p + q.woff[l];
    p.lda = p.ldb = p.K = q.din[l];
    p.M = B;
    p.N = q.dout[l];
    p.bias = q.p + q.boff[l];
    p.Z = q.Z + (int64_t)l * B * q.width;
    p.out = q.A + (int64_t)l * B * q.width;
    p.act = (l + 1 < q.layers) ? 1 : 0;
    product<EPI_FORWARD>(q, p, st);
    in = p.out;
  }
}

static void backward(Mlp &q, const float *X, int B, const float *dY,
                     hipStream_t st) {
  // dZ of the last layer is dY (linear output); below, two buffers in turn
  const float *dZ = dY;
  for (int l = q.layers - 1; l >= 0; --l) {
    const int N = q.dout[l], K = q.din[l];
    // dW[j][k] = sum_b dZ[b][j] in[b][k], db[j] = sum_b dZ[b][j]
    MlpProduct w{};
    w.A = dZ;
    w.lda = w.M = N;
    w.B = (l == 0) ? X : q.A + (int64_t)(l - 1) * B * q.width;
    w.ldb = w.N = K;
    w.K = B;
    w.out = q.g + q.woff[l];
    w.db = q.g + q.boff[l];
    product<EPI_WEIGHTS>(q, w, st);
    if (l == 0) break;
    // dZ_{l-1}[b][k] = silu'(Z_{l-1}[b][k]) sum_j dZ[b][j] W[j][k]
    MlpProduct a{};
    a.A = dZ;
    a.lda = a.K = N;
    a.B = q.p + q.woff[l];
    a.ldb = a.N = K;
    a.M = B;
    a.Zin = q.Z + (int64_t)(l - 1) * B * q.width;
    a.out = (l & 1) ? q.dZ : q.dA;
    product<EPI_BACKWARD>(q, a, st);
    dZ = a.out;
  }
}

}  // namespace rmx

using namespace rmx;

struct rm_mlp : public rmx::Mlp {};

static uint64_t splitmix(uint64_t &s) {
  uint64_t z = (s += 0x9e3779b97f4a7c15ull);
  z = (z ^ (z >> 30)) * 0xbf58476d1ce4e5b9ull;
  z = (z ^ (z >> 27)) * 0x94d049bb133111ebull;
  return z ^ (z >> 31);
}

extern "C" {

int rm_mlp_create(int32_t d_in, int32_t width, int32_t n_layers, int32_t prec,
                  uint64_t seed, rm_mlp_t *out) {
  if (!out) return (set_error(RM_ERR_ARG, "null out"), RM_ERR_ARG);
  *out = nullptr;
  if (d_in < 1 || width < 1 || n_layers < 2 || prec < 0 || prec > 1 ||
      d_in > 4096 || width > 4096 || n_layers > 16)
    return (set_error(RM_ERR_ARG, "bad MLP shape or precision"), RM_ERR_ARG);
  rm_mlp *q = new (std::nothrow) rm_mlp();
  if (!q) return (set_error(RM_ERR_NOMEM, "host allocation"), RM_ERR_NOMEM);
  q->d_in = d_in;
  q->width = width;
  q->layers = n_layers;
  q->prec = prec;
  q->step = 0;
  q->cap_b = 0;
  q->Z = q->A = q->dA = q->dZ = q->Y = nullptr;
  q->p = q->g = q->m = q->v = nullptr;
  (void)hipGetDevice(&q->device);
  int64_t off = 0;
  for (int l = 0; l < n_layers; ++l) {
    const int in = (l == 0) ? d_in : width;
    const int o = (l + 1 == n_layers) ? 1 : width;
    q->din.push_back(in);
    q->dout.push_back(o);
    q->woff.push_back(off);
    off += (int64_t)in * o;
    q->boff.push_back(off);
    off += o;
  }
  q->n_params = off;
  // He-style uniform init from a seeded splitmix64 stream
  std::vector<float> h((size_t)off, 0.0f);
  uint64_t s = seed;
  for (int l = 0; l < n_layers; ++l) {
    const double bound = std::sqrt(6.0 / q->din[l]) * (l + 1 == n_layers ? 0.1 : 1.0);
    for (int64_t i = 0; i < (int64_t)q->din[l] * q->dout[l]; ++i) {
      const double u = (splitmix(s) >> 11) * (1.0 / 9007199254740992.0);
      h[q->woff[l] + i] = (float)((2.0 * u - 1.0) * bound);
    }
  }
  hipError_t e = hipSuccess;
  for (float **x : {&q->p, &q->g, &q->m, &q->v})
    if (e == hipSuccess) e = device_malloc((void **)x, (size_t)off * sizeof(float));
  if (e == hipSuccess) e = hipMemcpy(q->p, h.data(), (size_t)off * sizeof(float), hipMemcpyHostToDevice);
  if (e == hipSuccess) e = hipMemset(q->g, 0, (size_t)off * sizeof(float));
  if (e == hipSuccess) e = hipMemset(q->m, 0, (size_t)off * sizeof(float));
  if (e == hipSuccess) e = hipMemset(q->v, 0, (size_t)off * sizeof(float));
  if (e != hipSuccess) {
    for (float *x : {q->p, q->g, q->m, q->v})
      if (x) (void)hipFree(x);
    delete q;
    return (set_error(RM_ERR_NOMEM, "MLP device allocation"), RM_ERR_NOMEM);
  }
  *out = q;
  return RM_OK;
}

int rm_mlp_free(rm_mlp_t q) {
  if (!q) return RM_OK;
  (void)hipDeviceSynchronize();
  for (float *x : {q->p, q->g, q->m, q->v, q->Z, q->A, q->dA, q->dZ, q->Y})
    if (x) (void)hipFree(x);
  delete q;
  return RM_OK;
}

int rm_mlp_n_params(rm_mlp_t q, int64_t *n) {
  if (!q || !n) return (set_error(RM_ERR_ARG, "null argument"), RM_ERR_ARG);
  *n = q->n_params;
  return RM_OK;
}

int rm_mlp_get_params(rm_mlp_t q, float *dst, void *stream) {
  if (!q || !dst) return (set_error(RM_ERR_ARG, "null argument"), RM_ERR_ARG);
  hipLaunchKernelGGL(copy_f32_kernel, dim3(g1(q->n_params)), dim3(256), 0,
                     (hipStream_t)stream, q->p, dst, q->n_params);
  return hipGetLastError() == hipSuccess ? RM_OK : RM_ERR_HIP;
}

int rm_mlp_set_params(rm_mlp_t q, const float *src, void *stream) {
  if (!q || !src) return (set_error(RM_ERR_ARG, "null argument"), RM_ERR_ARG);
  hipLaunchKernelGGL(copy_f32_kernel, dim3(g1(q->n_params)), dim3(256), 0,
                     (hipStream_t)stream, src, q->p, q->n_params);
  return hipGetLastError() == hipSuccess ? RM_OK : RM_ERR_HIP;
}

int rm_mlp_forward(rm_mlp_t q, const float *X, int32_t B, float *Y,
                   void *stream) {
  if (!q || !X || !Y || B < 1)
    return (set_error(RM_ERR_ARG, "bad forward arguments"), RM_ERR_ARG);
  if (ensure_cap(*q, B)) return (set_error(RM_ERR_NOMEM, "activations"), RM_ERR_NOMEM);
  hipStream_t st = (hipStream_t)stream;
  forward(*q, X, B, st);
  const float *out = q->A + (int64_t)(q->layers - 1) * B * q->width;
  hipLaunchKernelGGL(copy_f32_kernel, dim3(g1(B)), dim3(256), 0, st, out, Y,
                     (int64_t)B);
  return hipGetLastError() == hipSuccess ? RM_OK : RM_ERR_HIP;
}

int rm_mlp_grad(rm_mlp_t q, const float *X, const float *target, int32_t B,
                float *loss, float *grad, void *stream) {
  if (!q || !X || !target || B < 1)
    return (set_error(RM_ERR_ARG, "bad grad arguments"), RM_ERR_ARG);
  if (ensure_cap(*q, B)) return (set_error(RM_ERR_NOMEM, "activations"), RM_ERR_NOMEM);
  hipStream_t st = (hipStream_t)stream;
  forward(*q, X, B, st);
  const float *out = q->A + (int64_t)(q->layers - 1) * B * q->width;
  hipLaunchKernelGGL(mse_kernel, dim3(1), dim3(256), 0, st, out, target, q->Y,
                     loss, B);
  backward(*q, X, B, q->Y, st);
  if (grad)
    hipLaunchKernelGGL(copy_f32_kernel, dim3(g1(q->n_params)), dim3(256), 0,
                       st, q->g, grad, q->n_params);
  return hipGetLastError() == hipSuccess ? RM_OK : RM_ERR_HIP;
}

int rm_mlp_adam_step(rm_mlp_t q, float lr, float beta1, float beta2, float eps,
                     void *stream) {
  if (!q || !(lr > 0.f) || !(beta1 >= 0.f && beta1 < 1.f) ||
      !(beta2 >= 0.f && beta2 < 1.f) || !(eps > 0.f))
    return (set_error(RM_ERR_ARG, "bad Adam arguments"), RM_ERR_ARG);
  q->step += 1;
  const float c1 = 1.f - std::pow(beta1, (float)q->step);
  const float c2 = 1.f - std::pow(beta2, (float)q->step);
  hipLaunchKernelGGL(adam_kernel, dim3(g1(q->n_params)), dim3(256), 0,
                     (hipStream_t)stream, q->p, q->g, q->m, q->v, q->n_params,
                     lr, beta1, beta2, eps, c1, c2);
  return hipGetLastError() == hipSuccess ? RM_OK : RM_ERR_HIP;
}

int rm_mesh_from_density(const float *dens, int32_t nw, double lo, double hi,
                         double floor_frac, int64_t M, double *E_out,
                         void *stream) {
  if (!dens || !E_out || nw < 1 || M < 1 || !(hi > lo) ||
      !(floor_frac >= 0.0 && floor_frac <= 1.0))
    return (set_error(RM_ERR_ARG, "bad mesh arguments"), RM_ERR_ARG);
  hipStream_t st = (hipStream_t)stream;
  double *cum = nullptr;
  if (stream_malloc((void **)&cum, (size_t)(nw + 1) * sizeof(double), st) !=
      hipSuccess)
    return (set_error(RM_ERR_NOMEM, "cdf buffer"), RM_ERR_NOMEM);
  hipLaunchKernelGGL(density_cdf_kernel, dim3(1), dim3(256), 0, st, dens, nw,
                     floor_frac, cum);
  hipLaunchKernelGGL(mesh_place_kernel, dim3(g1(M)), dim3(256), 0, st, cum, nw,
                     lo, hi, M, E_out);
  (void)hipFreeAsync(cum, st);
  return hipGetLastError() == hipSuccess ? RM_OK : RM_ERR_HIP;
}

}  // extern "C"
