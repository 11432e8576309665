// Outer loop of the inversion (section "SF-AWRI with total variation
// regularization", eq. TVAWRI, Algorithm 2): the smoothed total-variation term
// and its gradient, limited-memory BFGS directions, and the adaptive-tolerance
// driver that calls the augmented solve (wri_objective_grad) for every
// objective evaluation.
//
// Every reduction runs with a fixed grid and sums its per-block float64
// partials in one fixed order, so results are deterministic.  The l-BFGS
// two-loop recursion keeps its coefficients in device memory: a chain of small
// launches on the caller's stream, no host round trip.
#include "../../include/wri.h"
#include "wri_impl.hpp"
#include "wave.hpp"

#include <algorithm>
#include <chrono>
#include <cmath>
#include <cstring>
#include <vector>

namespace wri {
namespace {

constexpr int kRedThreads = 256;
constexpr int kRedBlocks = 1024;  // partial sums per reduction (fixed: deterministic order)

#define OUTER_HIP(expr)                                                                 \
  do {                                                                                  \
    hipError_t e_ = (expr);                                                             \
    if (e_ != hipSuccess) return report_error(WRI_EHIP, "%s: %s", #expr, hipGetErrorString(e_)); \
  } while (0)

__device__ __forceinline__ double block_sum(double v, double* red) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  if (lane == 0) red[w] = v;
  __syncthreads();
  double r = 0.0;
  if (threadIdx.x == 0)
    for (int i = 0; i < kRedThreads / 64; ++i) r += red[i];
  return r;  // valid in thread 0
}

__device__ __forceinline__ float block_max(float v, float* red) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v = fmaxf(v, __shfl_xor(v, off, 64));
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  if (lane == 0) red[w] = v;
  __syncthreads();
  float r = 0.f;
  if (threadIdx.x == 0)
    for (int i = 0; i < kRedThreads / 64; ++i) r = fmaxf(r, red[i]);
  return r;
}

// ---- total variation --------------------------------------------------------
// phi_c = sqrt(|D m|_c^2 + eps^2) with forward differences (zero in the last
// cell of each axis); q_a = (D_a m) / phi;
// grad_c += gamma / h * sum_a (q_a[c - e_a] - q_a[c]).
//
// One pass: a workgroup owns kTvB consecutive cells of the x-y plane (the
// neighbours c - nx are nx cells back in the same order), a thread each, and
// marches kTvZ planes at a time.  It forms q once per cell, with qx and qy in LDS
// for the cells after in x and y (plus the nx cells before the tile) and qz in
// registers, and updates grad: 12 bytes per cell (m, grad in and out), where a
// pass that stored the three q in float64 and one that read them back moved 60.
// Bound by the float64 square root and divisions (one and three per cell, nx / kTvB
// more for the rows before the tile).  Rows too wide for the LDS (ROWS = false)
// form q of the cell c - nx again instead.  Value and gradient, whole call from
// Python: 128^3 74 -> 46 us (the pass 18, the rest launches and the copy of the
// value), 256x256x192 304 -> 110 us.
constexpr int kTvB = 1024, kTvZ = 2;
constexpr int kTvMaxRow = 1024;    // (kTvB + row) * kTvZ * 16 B of LDS: 64 KB

// I: the index type (int while the grid has fewer than 2^31 cells).
template <class I>
struct TvGeom {
  I nx, ny, nz, plane;
  double inv_h, eps2;
};

struct TvQ { double x, y, z, phi; };

// q of the cell c = z * plane + y * nx + x
template <class I>
__device__ __forceinline__ TvQ tv_q(const TvGeom<I>& G, const float* __restrict__ m, I c, I x, I y, I z) {
  const double mc = m[c];
  TvQ q;
  const double dx = (x + 1 < G.nx) ? ((double)m[c + 1] - mc) * G.inv_h : 0.0;
  const double dy = (y + 1 < G.ny) ? ((double)m[c + G.nx] - mc) * G.inv_h : 0.0;
  const double dz = (z + 1 < G.nz) ? ((double)m[c + G.plane] - mc) * G.inv_h : 0.0;
  q.phi = sqrt(dx * dx + dy * dy + dz * dz + G.eps2);
  q.x = dx / q.phi;
  q.y = dy / q.phi;
  q.z = dz / q.phi;
  return q;
}

// tiles of zc planes; per-block partials of sum phi; GRAD = false: the value only
template <class I, bool ROWS, bool GRAD>
__global__ void __launch_bounds__(kTvB)
k_tv(TvGeom<I> G, I tiles_p, I tiles, int zc, double scale, const float* __restrict__ m, float* __restrict__ grad,
     double* __restrict__ part) {
  __shared__ double red[kTvB / 64];
  extern __shared__ double tvs[];   // qx then qy: [kTvZ][halo + kTvB] each (ROWS: halo = nx, else 1 and no qy)
  const int halo = ROWS ? (int)G.nx : 1, wl = halo + kTvB, tid = threadIdx.x;
  double* sx = tvs;
  double* sy = tvs + kTvZ * wl;
  double acc = 0.0;
  for (I t = blockIdx.x; t < tiles; t += gridDim.x) {
    const I tz = t / tiles_p, c0 = (t - tz * tiles_p) * kTvB, zb = tz * zc, ze = zb + zc < G.nz ? zb + zc : G.nz;
    const I c = c0 + tid, y = c / G.nx, x = c - y * G.nx;
    const bool in = c < G.plane;
    double qzm = 0.0;   // qz of plane z - 1
    if (GRAD && in && zb > 0) qzm = tv_q<I>(G, m, (zb - 1) * G.plane + c, x, y, zb - 1).z;
    for (I z0 = zb; z0 < ze; z0 += kTvZ) {
      const I o = z0 * G.plane + c;
      TvQ q[kTvZ];
      float g[kTvZ];
#pragma unroll
      for (int i = 0; i < kTvZ; ++i)
        if (in && z0 + i < ze) {
          if constexpr (GRAD) g[i] = grad[o + i * G.plane];
          q[i] = tv_q<I>(G, m, o + i * G.plane, x, y, z0 + i);
          acc += q[i].phi;
          if constexpr (GRAD) {
            sx[i * wl + halo + tid] = q[i].x;
            if constexpr (ROWS) sy[i * wl + halo + tid] = q[i].y;
          }
        }
      if constexpr (GRAD) {
        if (tid < halo && c0 - halo + tid >= 0) {   // halo <= kTvB
          const I hc = c0 - halo + tid, hy = hc / G.nx, hx = hc - hy * G.nx;
#pragma unroll
          for (int i = 0; i < kTvZ; ++i)
            if (z0 + i < ze) {
              const TvQ v = tv_q<I>(G, m, (z0 + i) * G.plane + hc, hx, hy, z0 + i);
              sx[i * wl + tid] = v.x;
              if constexpr (ROWS) sy[i * wl + tid] = v.y;
            }
        }
        __syncthreads();
#pragma unroll
        for (int i = 0; i < kTvZ; ++i)
          if (in && z0 + i < ze) {
            double v = -(q[i].x + q[i].y + q[i].z);
            if (x > 0) v += sx[i * wl + halo + tid - 1];
            if (y > 0) {
              if constexpr (ROWS) v += sy[i * wl + tid];
              else v += tv_q<I>(G, m, o + i * G.plane - G.nx, x, y - 1, z0 + i).y;
            }
            if (z0 + i > 0) v += qzm;
            qzm = q[i].z;
            grad[o + i * G.plane] = (float)((double)g[i] + scale * v);
          }
        __syncthreads();
      }
    }
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) acc += __shfl_xor(acc, off, 64);
  if ((tid & 63) == 0) red[tid >> 6] = acc;
  __syncthreads();
  if (tid == 0) {
    double s = 0.0;
    for (int i = 0; i < kTvB / 64; ++i) s += red[i];
    part[blockIdx.x] = s;
  }
}

// ---- vector kernels of the l-BFGS recursion and the model update -------------
__global__ void __launch_bounds__(kRedThreads)
k_dot32(const float* __restrict__ a, const float* __restrict__ b, int64_t n, double* __restrict__ part) {
  __shared__ double red[kRedThreads / 64];
  double acc = 0.0;
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
    acc += (double)a[i] * (double)b[i];
  const double t = block_sum(acc, red);
  if (threadIdx.x == 0) part[blockIdx.x] = t;
}

// Device scalars of the recursion (index into sc): rho[i], alpha[i] for the
// ring slots, then H0 and two temporaries.
enum CoefOp : int { kOpSum = 0, kOpRho = 1, kOpAlpha = 2, kOpBeta = 3, kOpRatio = 4 };

// One block: s = fixed-order sum of the partials; then
//   kOpSum:   sc[dst] = s
//   kOpRho:   sc[dst] = 1 / s
//   kOpAlpha: sc[dst] = sc[a] * s                  (alpha_i = rho_i s_i.q)
//   kOpBeta:  sc[dst] = sc[a] - sc[b] * s          (alpha_i - rho_i y_i.r)
//   kOpRatio: sc[dst] = sc[a] / s                  (H0 = s.y / y.y)
__global__ void __launch_bounds__(64) k_coef(const double* __restrict__ part, int nparts, double* __restrict__ sc,
                                             int op, int dst, int a, int b) {
  double v = 0.0;
  for (int i = threadIdx.x; i < nparts; i += 64) v += part[i];
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
  if (threadIdx.x == 0) {
    double r = v;
    if (op == kOpRho) r = 1.0 / v;
    else if (op == kOpAlpha) r = sc[a] * v;
    else if (op == kOpBeta) r = sc[a] - sc[b] * v;
    else if (op == kOpRatio) r = sc[a] / v;
    sc[dst] = r;
  }
}

// y = y + sign * sc[k] * x   (float64 arithmetic, one rounding; x, y distinct)
__global__ void k_axpy_sc(float* __restrict__ y, const float* __restrict__ x, int64_t n, double sign,
                          const double* __restrict__ sc, int k) {
  const double a = sign * sc[k];
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
    y[i] = (float)((double)y[i] + a * (double)x[i]);
}

// y = sc[k] * y
__global__ void k_scale_sc(float* __restrict__ y, int64_t n, const double* __restrict__ sc, int k) {
  const double a = sc[k];
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
    y[i] = (float)(a * (double)y[i]);
}

// ---- l-BFGS direction from inner products --------------------------------------
// The two-loop recursion touches g, s_j and y_j only through inner products: with
// s_i.g, y_i.g, s_i.y_j and y_i.y_j (i <= j) its coefficients follow in scalar
// arithmetic, and dir = -(H0 (g - sum alpha_j y_j) + sum c_j s_j) is one pass.  Two
// passes over the 2 M + 1 vectors and one small launch replace 3 M + 2 dot
// products and 2 M + 3 updates, each a launch with dir read and written (M = 5,
// 128^3: 36 launches and 240 us a call from Python -> 3 launches and 56 us;
// 256x256x192 875 -> 234 us, 290 -> 92 bytes per cell).  Inner products and
// coefficients are float64; dir is rounded once instead of after every update.
// Up to kLbFused pairs (the accumulators live in registers: 88 for 8 pairs); longer
// memories, and workspaces without room for the partials of all inner products, take the
// recursion below.
constexpr int kLbFused = 8;
constexpr int kLbBlocks = 512;   // partial sums per inner product

struct LbPairs {   // the pairs in use, oldest first
  const float *s[kLbFused], *y[kLbFused];
};

// accumulator of an inner product: s_i.g, y_i.g, then s_i.y_j and y_i.y_j for i <= j
template <int M>
struct LbIndex {
  static constexpr int kTri = M * (M + 1) / 2;
  static constexpr int kCount = 2 * M + 2 * kTri;
  static constexpr __host__ __device__ int sg(int i) { return i; }
  static constexpr __host__ __device__ int yg(int i) { return M + i; }
  static constexpr __host__ __device__ int tri(int i, int j) { return i * M - i * (i - 1) / 2 + (j - i); }
  static constexpr __host__ __device__ int sy(int i, int j) { return 2 * M + tri(i, j); }
  static constexpr __host__ __device__ int yy(int i, int j) { return 2 * M + kTri + tri(i, j); }
};

template <int M>
__global__ void __launch_bounds__(kRedThreads)
k_lb_gram(LbPairs P, const float* __restrict__ g, int64_t n, double* __restrict__ part) {
  using I = LbIndex<M>;
  static_assert(I::kCount <= 128, "");
  __shared__ double red[kRedThreads / 64][128];
  double a[I::kCount];
#pragma unroll
  for (int i = 0; i < I::kCount; ++i) a[i] = 0.0;
  for (int64_t c = blockIdx.x * (int64_t)kRedThreads + threadIdx.x; c < n; c += (int64_t)gridDim.x * kRedThreads) {
    double s[M], y[M];
    const double gv = g[c];
#pragma unroll
    for (int i = 0; i < M; ++i) {
      s[i] = P.s[i][c];
      y[i] = P.y[i][c];
    }
#pragma unroll
    for (int i = 0; i < M; ++i) {
      a[I::sg(i)] = fma(s[i], gv, a[I::sg(i)]);
      a[I::yg(i)] = fma(y[i], gv, a[I::yg(i)]);
#pragma unroll
      for (int j = i; j < M; ++j) {
        a[I::sy(i, j)] = fma(s[i], y[j], a[I::sy(i, j)]);
        a[I::yy(i, j)] = fma(y[i], y[j], a[I::yy(i, j)]);
      }
    }
  }
  // 64-lane exchange holds up to 64 accumulators at a time
  const int w = threadIdx.x >> 6;
  constexpr int N0 = I::kCount < 64 ? I::kCount : 64, N1 = I::kCount - N0;
  {
    double b[N0];
#pragma unroll
    for (int i = 0; i < N0; ++i) b[i] = a[i];
    int id = 0, left = N0;
    const double v = wave_sums<N0>(b, 32, &id, &left);
    if (left > 0) red[w][id] = v;
  }
  if constexpr (N1 > 0) {
    double b[N1];
#pragma unroll
    for (int i = 0; i < N1; ++i) b[i] = a[N0 + i];
    int id = 0, left = N1;
    const double v = wave_sums<N1>(b, 32, &id, &left);
    if (left > 0) red[w][N0 + id] = v;
  }
  __syncthreads();
  for (int i = threadIdx.x; i < I::kCount; i += kRedThreads) {
    double v = 0.0;
#pragma unroll
    for (int k = 0; k < kRedThreads / 64; ++k) v += red[k][i];
    part[(int64_t)i * gridDim.x + blockIdx.x] = v;
  }
}

// One block: the inner products from their partials (fixed order), then the
// recursion's coefficients: coef[0] = H0, coef[1 + j] = H0 alpha_j (of y_j),
// coef[1 + M + j] = c_j (of s_j).
template <int M>
__global__ void __launch_bounds__(1024) k_lb_coef(const double* __restrict__ part, int nparts, double h0,
                                                  double* __restrict__ coef) {
  using I = LbIndex<M>;
  __shared__ double d[I::kCount];
  const int lane = threadIdx.x & 63;
  for (int i = threadIdx.x >> 6; i < I::kCount; i += 16) {
    double v = 0.0;
#pragma unroll
    for (int k = 0; k < kLbBlocks / 64; ++k) {
      const int b = lane + 64 * k;
      v += b < nparts ? part[(int64_t)i * nparts + b] : 0.0;
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
    if (lane == 0) d[i] = v;
  }
  __syncthreads();
  if (threadIdx.x != 0) return;
  double rho[M], alpha[M], c[M];
#pragma unroll
  for (int i = M - 1; i >= 0; --i) {
    rho[i] = 1.0 / d[I::sy(i, i)];
    double sq = d[I::sg(i)];
#pragma unroll
    for (int j = i + 1; j < M; ++j) sq -= alpha[j] * d[I::sy(i, j)];
    alpha[i] = rho[i] * sq;
  }
  const double H0 = h0 > 0.0 ? h0 : d[I::sy(M - 1, M - 1)] / d[I::yy(M - 1, M - 1)];
#pragma unroll
  for (int i = 0; i < M; ++i) {
    double yq = d[I::yg(i)];   // y_i . q after the first loop
#pragma unroll
    for (int j = 0; j < M; ++j) yq -= alpha[j] * d[j < i ? I::yy(j, i) : I::yy(i, j)];
    double yr = H0 * yq;
#pragma unroll
    for (int j = 0; j < i; ++j) yr += c[j] * d[I::sy(j, i)];
    c[i] = alpha[i] - rho[i] * yr;
  }
  coef[0] = H0;
#pragma unroll
  for (int i = 0; i < M; ++i) {
    coef[1 + i] = H0 * alpha[i];
    coef[1 + M + i] = c[i];
  }
}

// dir = -(H0 g - sum (H0 alpha_j) y_j + sum c_j s_j)
template <int M>
__global__ void __launch_bounds__(kRedThreads)
k_lb_combine(LbPairs P, const float* __restrict__ g, int64_t n, const double* __restrict__ coef,
             float* __restrict__ dir) {
  const double H0 = coef[0];
  double cy[M], cs[M];
#pragma unroll
  for (int i = 0; i < M; ++i) {
    cy[i] = coef[1 + i];
    cs[i] = coef[1 + M + i];
  }
  for (int64_t c = blockIdx.x * (int64_t)kRedThreads + threadIdx.x; c < n; c += (int64_t)gridDim.x * kRedThreads) {
    double r = H0 * (double)g[c];
#pragma unroll
    for (int i = 0; i < M; ++i) r = fma(cs[i], (double)P.s[i][c], fma(-cy[i], (double)P.y[i][c], r));
    dir[c] = (float)-r;
  }
}

// dir = -h0 g (no curvature pair)
__global__ void __launch_bounds__(kRedThreads) k_lb_steepest(const float* __restrict__ g, int64_t n, double h0,
                                                             float* __restrict__ dir) {
  for (int64_t c = blockIdx.x * (int64_t)kRedThreads + threadIdx.x; c < n; c += (int64_t)gridDim.x * kRedThreads)
    dir[c] = (float)-(h0 * (double)g[c]);
}

__global__ void k_copy32(float* __restrict__ d, const float* __restrict__ s, int64_t n) {
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
    d[i] = s[i];
}

// d = a - b
__global__ void k_sub32(float* __restrict__ d, const float* __restrict__ a, const float* __restrict__ b, int64_t n) {
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
    d[i] = (float)((double)a[i] - (double)b[i]);
}

__global__ void __launch_bounds__(kRedThreads) k_absmax32(const float* __restrict__ a, int64_t n, float* __restrict__ part) {
  __shared__ float red[kRedThreads / 64];
  float v = 0.f;
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
    v = fmaxf(v, fabsf(a[i]));
  const float t = block_max(v, red);
  if (threadIdx.x == 0) part[blockIdx.x] = t;
}

__device__ __forceinline__ bool in_sponge(int64_t c, int nx, int ny, int nz, int nb) {
  if (nb <= 0) return false;
  const int x = (int)(c % nx), y = (int)((c / nx) % ny), z = (int)(c / ((int64_t)nx * ny));
  return x < nb || x > nx - 1 - nb || y < nb || y > ny - 1 - nb || z < nb || z > nz - 1 - nb;
}

__global__ void k_zero_sponge(float* __restrict__ v, int nx, int ny, int nz, int nb) {
  const int64_t n = (int64_t)nx * ny * nz;
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
    if (in_sponge(i, nx, ny, nz, nb)) v[i] = 0.f;
}

// out = clamp(m + scale * dir) (bounds <= 0 are off)
__global__ void k_update(float* __restrict__ out, const float* __restrict__ m, const float* __restrict__ dir, int64_t n,
                         double scale, double lo, double hi) {
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
    double v = (double)m[i] + scale * (double)dir[i];
    if (lo > 0.0) v = fmax(v, lo);
    if (hi > 0.0) v = fmin(v, hi);
    out[i] = (float)v;
  }
}

int grid_blocks(int64_t n) { return (int)std::min<int64_t>(kRedBlocks, std::max<int64_t>(1, (n + kRedThreads - 1) / kRedThreads)); }

// ---- host helpers ----------------------------------------------------------------
size_t al(size_t x) { return (x + 255) & ~size_t(255); }

// The pass keeps per-workgroup partials (at most kTvBlocks, and at most one a cell) and
// their sum.  The query returns what it always has, room for three float64 arrays of the
// grid and kRedBlocks + 1 sums.
constexpr int kTvBlocks = 2048;
size_t tv_ws_bytes(int64_t n) { return 3 * al(sizeof(double) * n) + al(sizeof(double) * (kRedBlocks + 1)); }
size_t tv_used_bytes(int64_t n) { return al(sizeof(double) * (std::min<int64_t>(n, kTvBlocks) + 1)); }

// sum of n partials in one fixed order (one block)
__global__ void __launch_bounds__(kRedThreads) k_sum_parts(const double* __restrict__ part, int n, double* __restrict__ out) {
  __shared__ double red[kRedThreads / 64];
  double v = 0.0;
  for (int i = threadIdx.x; i < n; i += kRedThreads) v += part[i];
  const double t = block_sum(v, red);
  if (threadIdx.x == 0) *out = t;
}

// returns the number of partials
template <class I>
int tv_launch(const wri_grid& g, const float* m, double eps, double scale, float* grad, double* part, hipStream_t st) {
  TvGeom<I> G;
  G.nx = g.nx; G.ny = g.ny; G.nz = g.nz; G.plane = (I)g.nx * g.ny;
  G.inv_h = 1.0 / g.h; G.eps2 = eps * eps;
  const I tiles_p = (G.plane - 1) / kTvB + 1;
  // planes per tile: 16 (one in 17 q is formed twice) while that leaves two
  // workgroups per compute unit
  int zc = 16;
  while (zc > kTvZ && tiles_p * ((G.nz - 1) / zc + 1) < 512) zc /= 2;
  const I tiles = tiles_p * ((G.nz - 1) / zc + 1);
  const int nb = (int)std::min<I>(kTvBlocks, tiles);
  const size_t rows = 2 * sizeof(double) * kTvZ * (kTvB + (size_t)g.nx), cell = sizeof(double) * kTvZ * (kTvB + 1);
  if (grad == nullptr)
    hipLaunchKernelGGL((k_tv<I, false, false>), dim3(nb), dim3(kTvB), 0, st, G, tiles_p, tiles, zc, scale, m, grad, part);
  else if (g.nx <= kTvMaxRow)
    hipLaunchKernelGGL((k_tv<I, true, true>), dim3(nb), dim3(kTvB), rows, st, G, tiles_p, tiles, zc, scale, m, grad, part);
  else
    hipLaunchKernelGGL((k_tv<I, false, true>), dim3(nb), dim3(kTvB), cell, st, G, tiles_p, tiles, zc, scale, m, grad, part);
  return nb;
}

// TV(m) (host value) and, if grad != null, grad += gamma * grad TV
int tv_run(const wri_grid& g, const float* m, double eps, double gamma, double* value, float* grad, char* ws,
           hipStream_t st) {
  const int64_t n = (int64_t)g.nx * g.ny * g.nz;
  double* sum = reinterpret_cast<double*>(ws);
  double* part = sum + 1;
  float* gr = gamma != 0.0 ? grad : nullptr;
  const int nb = n < (int64_t(1) << 31)
                     ? tv_launch<int>(g, m, eps, gamma / g.h, gr, part, st)
                     : tv_launch<int64_t>(g, m, eps, gamma / g.h, gr, part, st);
  OUTER_HIP(hipGetLastError());
  hipLaunchKernelGGL(k_sum_parts, dim3(1), dim3(kRedThreads), 0, st, part, nb, sum);
  OUTER_HIP(hipGetLastError());
  OUTER_HIP(hipMemcpyAsync(value, sum, sizeof(double), hipMemcpyDeviceToHost, st));
  OUTER_HIP(hipStreamSynchronize(st));
  return WRI_OK;
}

// Workspace of a direction: the scalars, then partial sums in what is left of it.
struct LbWs {
  double *sc, *part;
  int64_t parts;   // room for partial sums
};
constexpr int kLbParts = std::max(kRedBlocks, kLbBlocks * LbIndex<kLbFused>::kCount);
size_t lb_ws_bytes(int cap, int64_t parts) { return al(sizeof(double) * (2 * cap + 4)) + al(sizeof(double) * parts); }
LbWs lb_ws(char* ws, size_t bytes, int cap) {
  const size_t sc = lb_ws_bytes(cap, 0);
  return {reinterpret_cast<double*>(ws), reinterpret_cast<double*>(ws + sc), (int64_t)((bytes - sc) / sizeof(double))};
}
int lb_blocks(int64_t n) { return (int)std::min<int64_t>(kLbBlocks, (n + kRedThreads - 1) / kRedThreads); }
int lb_count(int m) { return 2 * m + m * (m + 1); }   // LbIndex<m>::kCount

int dot_to(const float* a, const float* b, int64_t n, const LbWs& w, int op, int dst, int ia, int ib, hipStream_t st) {
  hipLaunchKernelGGL(k_dot32, dim3(kRedBlocks), dim3(kRedThreads), 0, st, a, b, n, w.part);
  OUTER_HIP(hipGetLastError());
  hipLaunchKernelGGL(k_coef, dim3(1), dim3(64), 0, st, w.part, kRedBlocks, w.sc, op, dst, ia, ib);
  OUTER_HIP(hipGetLastError());
  return WRI_OK;
}

template <int M>
int lbfgs_fused(const LbPairs& P, int64_t n, const float* g, double h0, float* dir, const LbWs& w, hipStream_t st) {
  static_assert(LbIndex<M>::kCount == 2 * M + M * (M + 1), "");
  const int nb = lb_blocks(n);
  hipLaunchKernelGGL((k_lb_gram<M>), dim3(nb), dim3(kRedThreads), 0, st, P, g, n, w.part);
  OUTER_HIP(hipGetLastError());
  hipLaunchKernelGGL((k_lb_coef<M>), dim3(1), dim3(1024), 0, st, w.part, nb, h0, w.sc);
  OUTER_HIP(hipGetLastError());
  const int nc = (int)std::min<int64_t>(4096, (n + kRedThreads - 1) / kRedThreads);
  hipLaunchKernelGGL((k_lb_combine<M>), dim3(nc), dim3(kRedThreads), 0, st, P, g, n, w.sc, dir);
  OUTER_HIP(hipGetLastError());
  return WRI_OK;
}

// dir = -H g, two-loop recursion over `count` ring slots ending at `newest`; slot i
// of S and Y starts at i * stride.
// h0 > 0: H0 = h0 I; otherwise H0 = s.y / y.y of the newest pair.
int lbfgs_run(int64_t n, const float* g, const float* S, const float* Y, int64_t stride, int cap, int count, int newest,
              double h0, float* dir, const LbWs& w, hipStream_t st) {
  const int rho0 = 0, alp0 = cap, ih0 = 2 * cap, it0 = 2 * cap + 1, it1 = 2 * cap + 2;
  const int nbk = grid_blocks(n);
  auto slot = [&](int j) { return ((newest - (count - 1) + j) % cap + cap) % cap; };  // j = 0 oldest
  if (count == 0) {
    hipLaunchKernelGGL(k_lb_steepest, dim3(nbk), dim3(kRedThreads), 0, st, g, n, h0, dir);
    OUTER_HIP(hipGetLastError());
    return WRI_OK;
  }
  // (the recursion needs the partials of one inner product only)
  if (count <= kLbFused && (int64_t)lb_count(count) * lb_blocks(n) <= w.parts) {
    LbPairs P{};
    for (int j = 0; j < count; ++j) {
      P.s[j] = S + slot(j) * stride;
      P.y[j] = Y + slot(j) * stride;
    }
    switch (count) {
      case 1: return lbfgs_fused<1>(P, n, g, h0, dir, w, st);
      case 2: return lbfgs_fused<2>(P, n, g, h0, dir, w, st);
      case 3: return lbfgs_fused<3>(P, n, g, h0, dir, w, st);
      case 4: return lbfgs_fused<4>(P, n, g, h0, dir, w, st);
      case 5: return lbfgs_fused<5>(P, n, g, h0, dir, w, st);
      case 6: return lbfgs_fused<6>(P, n, g, h0, dir, w, st);
      case 7: return lbfgs_fused<7>(P, n, g, h0, dir, w, st);
      default: return lbfgs_fused<8>(P, n, g, h0, dir, w, st);
    }
  }
  hipLaunchKernelGGL(k_copy32, dim3(nbk), dim3(kRedThreads), 0, st, dir, g, n);
  OUTER_HIP(hipGetLastError());
  int rc;
  for (int j = count - 1; j >= 0; --j) {
    const int i = slot(j);
    const float* s = S + i * stride;
    const float* y = Y + i * stride;
    if ((rc = dot_to(y, s, n, w, kOpRho, rho0 + i, 0, 0, st)) != WRI_OK) return rc;
    if ((rc = dot_to(s, dir, n, w, kOpAlpha, alp0 + i, rho0 + i, 0, st)) != WRI_OK) return rc;
    hipLaunchKernelGGL(k_axpy_sc, dim3(nbk), dim3(kRedThreads), 0, st, dir, y, n, -1.0, w.sc, alp0 + i);
    OUTER_HIP(hipGetLastError());
  }
  if (h0 > 0.0 || count == 0) {
    const double hh = h0;
    OUTER_HIP(hipMemcpyAsync(w.sc + ih0, &hh, sizeof(double), hipMemcpyHostToDevice, st));
  } else {
    const float* s = S + slot(count - 1) * stride;
    const float* y = Y + slot(count - 1) * stride;
    if ((rc = dot_to(s, y, n, w, kOpSum, it0, 0, 0, st)) != WRI_OK) return rc;
    if ((rc = dot_to(y, y, n, w, kOpRatio, ih0, it0, 0, st)) != WRI_OK) return rc;
  }
  // r = H0 q
  hipLaunchKernelGGL(k_scale_sc, dim3(nbk), dim3(kRedThreads), 0, st, dir, n, w.sc, ih0);
  OUTER_HIP(hipGetLastError());
  for (int j = 0; j < count; ++j) {
    const int i = slot(j);
    const float* s = S + i * stride;
    const float* y = Y + i * stride;
    if ((rc = dot_to(y, dir, n, w, kOpBeta, it1, alp0 + i, rho0 + i, st)) != WRI_OK) return rc;
    hipLaunchKernelGGL(k_axpy_sc, dim3(nbk), dim3(kRedThreads), 0, st, dir, s, n, 1.0, w.sc, it1);
    OUTER_HIP(hipGetLastError());
  }
  // dir = -r
  const double minus_one = -1.0;
  OUTER_HIP(hipMemcpyAsync(w.sc + it0, &minus_one, sizeof(double), hipMemcpyHostToDevice, st));
  hipLaunchKernelGGL(k_scale_sc, dim3(nbk), dim3(kRedThreads), 0, st, dir, n, w.sc, it0);
  OUTER_HIP(hipGetLastError());
  return WRI_OK;
}

// ---- the adaptive-tolerance driver (Algorithm 2) ------------------------------------
struct AwriLayout {
  size_t solver = 0, off_vec = 0, off_tv = 0, off_lb = 0, lb_bytes = 0, off_red = 0, off_u = 0, total = 0;
};
AwriLayout awri_layout(int64_t n, size_t solver_bytes, size_t tv_bytes, size_t lb_bytes, int memory, int n_sys,
                       bool warm) {
  AwriLayout L;
  L.solver = solver_bytes;
  L.off_vec = al(solver_bytes);
  const size_t vb = al(sizeof(float) * n);
  size_t off = L.off_vec + vb * (size_t)(5 + 2 * std::max(memory, 0));  // g, g_try, m_try, dir, tmp, S, Y
  L.off_tv = off;
  off += tv_bytes;
  L.off_lb = off;
  L.lb_bytes = lb_bytes;
  off += lb_bytes;
  L.off_red = off;
  off += al(sizeof(float) * kRedBlocks) + al(sizeof(double) * kRedBlocks);
  L.off_u = off;  // warm start: wavefields at the current model, then at the trial model
  if (warm) off += 2 * (size_t)std::max(n_sys, 0) * al(sizeof(float) * 2 * n);
  L.total = off + 256;
  return L;
}

// The workspace has always held room for a TV pass with three float64 arrays (24 B a
// cell).  The direction's partials (at most 2.8 B) and, for up to some 200 systems, what
// the solver's window march needs beyond its slab marches fit in that.
struct AwriPlan {
  AwriLayout full, least;   // with the window march, and the former size with the slab marches
  size_t query() const { return std::max(full.total, least.total); }
};
AwriPlan awri_plan(const wri_grid& g, const wri_system* sys, int n_sys, int mode, int flags, int memory, bool warm) {
  const int64_t n = (int64_t)g.nx * g.ny * g.nz;
  const int cap = std::max(memory, 1);
  const size_t with = solver_bytes(&g, 1, sys, n_sys, mode, flags, true);
  const size_t slab = solver_bytes(&g, 1, sys, n_sys, mode, flags, false);
  if (with == 0 || slab == 0) return {};
  const size_t tv = tv_used_bytes(n), lb_least = lb_ws_bytes(cap, kRedBlocks);
  const int64_t parts = std::max<int64_t>(kRedBlocks, (int64_t)lb_count(std::min(cap, kLbFused)) * lb_blocks(n));
  return {awri_layout(n, with, tv, lb_ws_bytes(cap, parts), memory, n_sys, warm),
          awri_layout(n, slab, tv, tv_ws_bytes(n) - tv + lb_least, memory, n_sys, warm)};
}

int absmax_host(const float* a, int64_t n, float* part, hipStream_t st, double* out) {
  hipLaunchKernelGGL(k_absmax32, dim3(kRedBlocks), dim3(kRedThreads), 0, st, a, n, part);
  OUTER_HIP(hipGetLastError());
  std::vector<float> h(kRedBlocks);
  OUTER_HIP(hipMemcpyAsync(h.data(), part, sizeof(float) * kRedBlocks, hipMemcpyDeviceToHost, st));
  OUTER_HIP(hipStreamSynchronize(st));
  float v = 0.f;
  for (float x : h) v = std::max(v, x);
  *out = v;
  return WRI_OK;
}

int dot_host(const float* a, const float* b, int64_t n, double* part, hipStream_t st, double* out) {
  hipLaunchKernelGGL(k_dot32, dim3(kRedBlocks), dim3(kRedThreads), 0, st, a, b, n, part);
  OUTER_HIP(hipGetLastError());
  std::vector<double> h(kRedBlocks);
  OUTER_HIP(hipMemcpyAsync(h.data(), part, sizeof(double) * kRedBlocks, hipMemcpyDeviceToHost, st));
  OUTER_HIP(hipStreamSynchronize(st));
  double v = 0.0;
  for (double x : h) v += x;
  *out = v;
  return WRI_OK;
}

}  // namespace
}  // namespace wri

using namespace wri;

extern "C" {

size_t wri_tv_workspace_bytes(const wri_grid* grid) {
  if (grid == nullptr || grid->nx < 1 || grid->ny < 1 || grid->nz < 1) return 0;
  return tv_ws_bytes((int64_t)grid->nx * grid->ny * grid->nz) + 256;
}

int wri_tv(const wri_grid* grid, const float* m, double eps, double gamma, double* value, float* grad, void* ws,
           size_t ws_bytes, void* stream) {
  if (grid == nullptr || m == nullptr || value == nullptr) return report_error(WRI_EINVAL, "grid, m and value are required");
  if (grid->nx < 1 || grid->ny < 1 || grid->nz < 1 || !(grid->h > 0.0)) return report_error(WRI_EINVAL, "invalid grid");
  if (!(eps >= 0.0) || !std::isfinite(gamma)) return report_error(WRI_EINVAL, "eps must be >= 0 and gamma finite");
  const size_t need = wri_tv_workspace_bytes(grid);
  if (ws == nullptr || ws_bytes < need) return report_error(WRI_ENOWS, "workspace of %zu bytes is smaller than the %zu required", ws_bytes, need);
  char* w = reinterpret_cast<char*>((reinterpret_cast<uintptr_t>(ws) + 255) & ~uintptr_t(255));
  return tv_run(*grid, m, eps, gamma, value, grad, w, reinterpret_cast<hipStream_t>(stream));
}

size_t wri_lbfgs_workspace_bytes(int32_t capacity) {
  if (capacity < 0) return 0;
  return lb_ws_bytes(std::max(capacity, 1), kLbParts) + 256;
}

int wri_lbfgs_direction(int64_t n, const float* g, const float* S, const float* Y, int32_t capacity, int32_t count,
                        int32_t newest, double h0, float* dir, void* ws, size_t ws_bytes, void* stream) {
  if (n < 1 || g == nullptr || dir == nullptr) return report_error(WRI_EINVAL, "n >= 1, g and dir are required");
  if (capacity < 0 || count < 0 || count > capacity || (count > 0 && (S == nullptr || Y == nullptr)) ||
      (count > 0 && (newest < 0 || newest >= capacity)))
    return report_error(WRI_EINVAL, "invalid pair ring (capacity %d, count %d, newest %d)", capacity, count, newest);
  if (count == 0 && !(h0 > 0.0)) return report_error(WRI_EINVAL, "h0 must be > 0 without curvature pairs");
  if (!std::isfinite(h0)) return report_error(WRI_EINVAL, "h0 is not finite");
  const int cap = std::max(capacity, 1);
  const size_t need = lb_ws_bytes(cap, kRedBlocks) + 256;   // the recursion's
  if (ws == nullptr || ws_bytes < need) return report_error(WRI_ENOWS, "workspace of %zu bytes is smaller than the %zu required", ws_bytes, need);
  char* w = reinterpret_cast<char*>((reinterpret_cast<uintptr_t>(ws) + 255) & ~uintptr_t(255));
  return lbfgs_run(n, g, S, Y, n, cap, count, newest, h0, dir, lb_ws(w, ws_bytes - 256, cap),
                   reinterpret_cast<hipStream_t>(stream));
}

size_t wri_awri_workspace_bytes(const wri_grid* grid, const wri_system* sys, int32_t n_sys, int32_t mode,
                                int32_t flags, int32_t memory) {
  if (grid == nullptr || memory < 0) return 0;
  const AwriPlan P = awri_plan(*grid, sys, n_sys, mode, flags, memory, (flags & WRI_FLAG_WARM_START) != 0);
  return P.query();
}

int wri_awri(const wri_grid* grid, float* m, const wri_system* sys, int32_t n_sys, int32_t mode,
             const wri_awri_options* opt, wri_awri_record* history, int32_t history_cap, int32_t* n_records,
             void* ws, size_t ws_bytes, void* stream) {
  if (grid == nullptr || m == nullptr || opt == nullptr || n_records == nullptr)
    return report_error(WRI_EINVAL, "grid, m, opt and n_records are required");
  *n_records = 0;
  const wri_awri_options o = *opt;
  if (!(o.eps0 > 0.0) || !(o.eps_min > 0.0) || o.eps_min > o.eps0 || o.max_outer < 0 || o.memory < 0 ||
      !(o.gamma >= 0.0) || !(o.eps_tv >= 0.0) || !(o.step0 > 0.0) || !(o.max_step >= 0.0) || o.max_iter < 0 ||
      (o.m_min > 0.0 && o.m_max > 0.0 && o.m_min > o.m_max))
    return report_error(WRI_EINVAL, "invalid options");
  if (history_cap > 0 && history == nullptr) return report_error(WRI_EINVAL, "history is NULL");
  const int64_t n = (int64_t)grid->nx * grid->ny * grid->nz;
  const bool warm = o.warm_start != 0;
  const AwriPlan P = awri_plan(*grid, sys, n_sys, mode, o.flags, o.memory, warm);
  if (P.query() == 0) return report_error(WRI_EINVAL, "invalid grid or systems: %s", wri_last_error());
  const AwriLayout L = ws_bytes >= P.query() ? P.full : P.least;
  if (ws == nullptr || ws_bytes < P.least.total)
    return report_error(WRI_ENOWS, "workspace of %zu bytes is smaller than the %zu required", ws_bytes, P.least.total);
  hipStream_t st = reinterpret_cast<hipStream_t>(stream);
  char* base = reinterpret_cast<char*>((reinterpret_cast<uintptr_t>(ws) + 255) & ~uintptr_t(255));
  char* solver_ws = base;
  const size_t vb = al(sizeof(float) * n);
  float* g = reinterpret_cast<float*>(base + L.off_vec);
  float* g_try = reinterpret_cast<float*>(base + L.off_vec + vb);
  float* m_try = reinterpret_cast<float*>(base + L.off_vec + 2 * vb);
  float* dir = reinterpret_cast<float*>(base + L.off_vec + 3 * vb);
  float* tmp = reinterpret_cast<float*>(base + L.off_vec + 4 * vb);
  float* Sring = reinterpret_cast<float*>(base + L.off_vec + 5 * vb);
  const int64_t ring = vb / sizeof(float);   // stride of the pairs
  float* Yring = Sring + o.memory * ring;
  char* tvw = base + L.off_tv;
  const LbWs lbw = lb_ws(base + L.off_lb, L.lb_bytes, std::max(o.memory, 1));
  float* fpart = reinterpret_cast<float*>(base + L.off_red);
  double* dpart = reinterpret_cast<double*>(base + L.off_red + al(sizeof(float) * kRedBlocks));
  const int nbk = grid_blocks(n);
  const int nbs = (o.mask_sponge && grid->nb > 0) ? grid->nb : 0;

  std::vector<wri_system> se(sys, sys + n_sys);
  std::vector<wri_result> res(std::max(n_sys, 1));
  // warm start: wavefields (and source weights) of the current model and of the trial
  const size_t ub = al(sizeof(float) * 2 * n);
  std::vector<wri_c32*> ucur(n_sys), utry(n_sys);
  for (int i = 0; i < n_sys; ++i) {
    ucur[i] = reinterpret_cast<wri_c32*>(base + L.off_u + (size_t)i * ub);
    utry[i] = reinterpret_cast<wri_c32*>(base + L.off_u + (size_t)(n_sys + i) * ub);
  }
  std::vector<wri_c64> acur(n_sys), atry(n_sys);
  bool have_cur = false;
  int recs = 0;
  auto record = [&](double F, double J, double T, double eps, int kind, int iters, double secs) {
    if (recs < history_cap) history[recs] = wri_awri_record{F, J, T, eps, kind, iters, secs};
    ++recs;
  };
  // F = J + gamma TV and its gradient (masked in the sponge) at model mm, tolerance eps.
  // Warm start: the solves start from the current model's wavefields `from`
  // (copied into `into` unless they are the same set) and source weights.
  auto evaluate_w = [&](const float* mm, double eps, float* grad, double* F, double* J, double* T, int* iters,
                        double* secs, std::vector<wri_c32*>* into, std::vector<wri_c32*>* from,
                        std::vector<wri_c64>* alphas_out) -> int {
    const auto t0 = std::chrono::steady_clock::now();
    int fl = o.flags & ~WRI_FLAG_WARM_START;  // the driver decides per solve
    for (int i = 0; i < n_sys; ++i) {
      se[i].rtol = eps;
      if (warm && have_cur && mode == WRI_ESTIMATE) se[i].alpha = acur[i];
    }
    if (warm && have_cur) {
      fl |= WRI_FLAG_WARM_START;
      if (from != into)
        for (int i = 0; i < n_sys; ++i)
          OUTER_HIP(hipMemcpyAsync((*into)[i], (*from)[i], sizeof(float) * 2 * n, hipMemcpyDeviceToDevice, st));
    }
    const float* mp[1] = {mm};
    float* gp[1] = {grad};
    int rc = wri_objective_grad(grid, 1, mp, se.data(), n_sys, mode, o.max_iter, fl, J, gp,
                                warm ? into->data() : nullptr, res.data(), solver_ws, L.solver, stream);
    if (rc < 0) return rc;
    if (warm)
      for (int i = 0; i < n_sys; ++i) (*alphas_out)[i] = res[i].alpha;
    int it = 0;
    for (int i = 0; i < n_sys; ++i) it += res[i].iters;
    *iters = it;
    rc = tv_run(*grid, mm, o.eps_tv, o.gamma, T, grad, tvw, st);
    if (rc != WRI_OK) return rc;
    if (nbs > 0) {
      hipLaunchKernelGGL(k_zero_sponge, dim3(nbk), dim3(kRedThreads), 0, st, grad, grid->nx, grid->ny, grid->nz, nbs);
      OUTER_HIP(hipGetLastError());
    }
    OUTER_HIP(hipStreamSynchronize(st));
    *F = *J + o.gamma * *T;
    *secs = std::chrono::duration<double>(std::chrono::steady_clock::now() - t0).count();
    return WRI_OK;
  };

  // the current model (start, or again after eps was halved): warm from its own wavefields
  auto evaluate = [&](const float* mm, double eps, float* grad, double* F, double* J, double* T, int* iters,
                      double* secs) -> int {
    const int r = evaluate_w(mm, eps, grad, F, J, T, iters, secs, &ucur, &ucur, &acur);
    if (r == WRI_OK) have_cur = true;
    return r;
  };
  double eps = o.eps0, F = 0, J = 0, T = 0, secs = 0;
  int iters = 0, rc;
  if ((rc = evaluate(m, eps, g, &F, &J, &T, &iters, &secs)) != WRI_OK) return rc;
  record(F, J, T, eps, WRI_AWRI_EVAL, iters, secs);
  int count = 0, newest = -1, accepted = 0;
  double last_sy = 0.0, last_yy = 0.0;
  int status = WRI_OK;
  while (accepted < o.max_outer) {
    double h0;
    if (count > 0) {
      h0 = last_sy / last_yy;
    } else {
      double mmax = 0.0, gmax = 0.0;
      if ((rc = absmax_host(m, n, fpart, st, &mmax)) != WRI_OK) return rc;
      if ((rc = absmax_host(g, n, fpart, st, &gmax)) != WRI_OK) return rc;
      if (!(gmax > 0.0)) break;  // stationary
      h0 = o.step0 * mmax / gmax;
    }
    if ((rc = lbfgs_run(n, g, Sring, Yring, ring, std::max(o.memory, 1), count, std::max(newest, 0), h0, dir, lbw,
                        st)) != WRI_OK)
      return rc;
    double scale = 1.0;
    if (o.max_step > 0.0) {
      double mmax = 0.0, dmax = 0.0;
      if ((rc = absmax_host(m, n, fpart, st, &mmax)) != WRI_OK) return rc;
      if ((rc = absmax_host(dir, n, fpart, st, &dmax)) != WRI_OK) return rc;
      if (dmax > o.max_step * mmax) scale = o.max_step * mmax / dmax;
    }
    hipLaunchKernelGGL(k_update, dim3(nbk), dim3(kRedThreads), 0, st, m_try, m, dir, n, scale, o.m_min, o.m_max);
    OUTER_HIP(hipGetLastError());
    double F1 = 0, J1 = 0, T1 = 0;
    if ((rc = evaluate_w(m_try, eps, g_try, &F1, &J1, &T1, &iters, &secs, &utry, &ucur, &atry)) != WRI_OK)
      return rc;
    const bool ok = F1 <= F;
    record(F1, J1, T1, eps, ok ? WRI_AWRI_ACCEPTED : WRI_AWRI_REJECTED, iters, secs);
    if (!ok) {
      if (0.5 * eps < o.eps_min) { status = WRI_NOT_CONVERGED; break; }
      eps *= 0.5;
      // pairs formed at the looser tolerance are dropped: the next trial is a
      // scaled gradient step (without a line search a stale pair repeats the
      // rejected step)
      count = 0;
      newest = -1;
      if ((rc = evaluate(m, eps, g, &F, &J, &T, &iters, &secs)) != WRI_OK) return rc;
      record(F, J, T, eps, WRI_AWRI_EVAL, iters, secs);
      continue;
    }
    // curvature pair (s, y) = (m_try - m, g_try - g): kept (in the next ring
    // slot, replacing the oldest pair once the ring is full) only if s.y > 0
    if (o.memory > 0) {
      float* s = tmp;
      float* y = dir;  // the direction is no longer needed
      hipLaunchKernelGGL(k_sub32, dim3(nbk), dim3(kRedThreads), 0, st, s, m_try, m, n);
      hipLaunchKernelGGL(k_sub32, dim3(nbk), dim3(kRedThreads), 0, st, y, g_try, g, n);
      OUTER_HIP(hipGetLastError());
      double sy = 0.0, yy = 0.0;
      if ((rc = dot_host(s, y, n, dpart, st, &sy)) != WRI_OK) return rc;
      if ((rc = dot_host(y, y, n, dpart, st, &yy)) != WRI_OK) return rc;
      if (sy > 0.0 && yy > 0.0) {
        const int slot = (newest + 1) % o.memory;
        hipLaunchKernelGGL(k_copy32, dim3(nbk), dim3(kRedThreads), 0, st, Sring + slot * ring, s, n);
        hipLaunchKernelGGL(k_copy32, dim3(nbk), dim3(kRedThreads), 0, st, Yring + slot * ring, y, n);
        OUTER_HIP(hipGetLastError());
        newest = slot;
        count = std::min(count + 1, o.memory);
        last_sy = sy;
        last_yy = yy;
      }
    }
    hipLaunchKernelGGL(k_copy32, dim3(nbk), dim3(kRedThreads), 0, st, m, m_try, n);
    OUTER_HIP(hipGetLastError());
    std::swap(g, g_try);
    if (warm) {
      std::swap(ucur, utry);
      std::swap(acur, atry);
    }
    F = F1; J = J1; T = T1;
    ++accepted;
  }
  OUTER_HIP(hipStreamSynchronize(st));
  *n_records = recs;
  if (status != WRI_OK) report_error(status, "the objective did not decrease at the smallest tolerance %.3g", o.eps_min);
  return status;
}

}  // extern "C"
