// Preconditioned CGLS: the batched augmented solve with S preconditioned on the
// right by one multigrid V(1,1) cycle of the complex-shifted Helmholtz operator
//   A_beta = L_h + diag(omega^2 (1 - i beta) m - i omega b),   beta = 1/2,
// i.e. CGLS on min ||S M y - b|| with x = M y.  This goes beyond the paper,
// whose only reducer of the iteration count is the adaptive tolerance of
// Algorithm 2: the minimiser is that of eq. SimpObj, the iterates and their
// number differ.  S is the printed one (source column -e, weight 1), and the
// stopping test is the plain solver's, on the true normal residual
// ||S^H r|| <= rtol ||S^H b||.
//
// Per iteration, over all systems of a grid in lockstep (finished systems skip
// inside the kernels; step scalars live in device memory; the host checks the
// statuses between chunks of iterations):
//   p = z + beta p;  q = M p (V-cycle);  t = S q;  a = gamma / ||t||^2;
//   x += a q;  r -= a t;  s = S^H r (stopping test);  z = M^H s (V-cycle on
//   conj(A_beta), M being complex symmetric);  beta = ||z||^2 / gamma.
// The V-cycle on a level with right-hand side f: y = w D^-1 f (one damped
// Jacobi step from zero), the residual f - A_beta y restricted with P^T / 8 to
// the next level (halved along every axis, h doubled, m and sponge restricted
// as weighted means), the next level's result prolonged (trilinear) and added,
// one more Jacobi step; four Jacobi steps from zero on the coarsest level.
// Every reduction sums fixed per-block partials in one fixed order.
#include "../../include/wri.h"
#include "wri_impl.hpp"
#include "stencil.hpp"
#include "window.hpp"

#include <algorithm>
#include <cfloat>
#include <cmath>
#include <cstring>
#include <vector>

namespace wri {
namespace {

constexpr int kThr = 256;
constexpr int kParts = 256;        // blocks (and partial sums) per system for the level-0 passes
constexpr int kMaxLev = 12;
constexpr int kCheck = 16;         // iterations between host checks of the statuses
constexpr double kBeta = 0.5;      // imaginary shift of the mass term in A_beta
constexpr double kJac = 0.7;       // Jacobi damping
constexpr int kCoarseSweeps = 4;   // Jacobi steps on the coarsest level
constexpr int64_t kCoarsestCells = 512;
constexpr size_t kAl = 256;
size_t al(size_t v) { return (v + kAl - 1) / kAl * kAl; }

#define PC_HIP(expr)                                                                                \
  do {                                                                                              \
    hipError_t e_ = (expr);                                                                         \
    if (e_ != hipSuccess) return report_error(WRI_EHIP, "%s: %s", #expr, hipGetErrorString(e_));   \
  } while (0)

// One level of one system's V-cycle.  m and b are the grid's (shared by its
// systems); f, y, o, res are the system's: right-hand side, the prolonged and
// corrected iterate, the level's result, the restricted residual's source.
struct PcLevel {
  int nx, ny, nz, n;
  double h2inv;
  const float* m;
  const float* b;
  const float2* wdinv;   // w D^-1 of A_beta on this level (per grid and frequency), complex64
  float2 *f, *y, *o, *res;
};

struct PcSys {
  float2 *x, *r[2], *p[2], *q, *t, *s, *z, *r2, *t2;   // r, p: current vector by iteration parity (tiled passes)
  double* part;   // partial sums of a level-0 pass
  const float2* d;
  const int* rec;
  const float* m;
  int nb, nr, est, max_iter, nlev, src;
  int tiled;    // 1: the passes by window tiles; 0: one thread per cell, r and p updated in place
  int nparts;   // partial sums in part
  double lam, rtol2, omega, omega2, sp_scale, inv_nb;
  double2 alpha;  // KNOWN-mode weight
  PcLevel lev[kMaxLev];
};

// Mutable scalars of one system (float64).
struct PcState {
  double gamma, ss0, ss, ssmin, a, beta, J;
  double2 xa, pa, za;
  int status, iters, pad_[2];
};

__device__ __forceinline__ double bsum(double v, double* red) {  // block total, every thread
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
  __syncthreads();
  double r = 0.0;
#pragma unroll
  for (int i = 0; i < kThr / 64; ++i) r += red[i];
  __syncthreads();
  return r;
}

// residual after `iters` iterations, and the direction p that iteration's forward cycle reads
__device__ __forceinline__ float2* pc_r(const PcSys& S, int iters) { return S.r[S.tiled & iters & 1]; }
__device__ __forceinline__ float2* pc_p(const PcSys& S, int iters) { return S.p[S.tiled & (iters + 1) & 1]; }

__device__ __forceinline__ double nrm(float2 v) { return (double)v.x * v.x + (double)v.y * v.y; }
__device__ __forceinline__ float2 fd(double a, double b) { return make_float2((float)a, (float)b); }

// partials of one system's level-0 pass, summed in one fixed order
__device__ double sum_parts(const double* __restrict__ part, int n, double* red) {
  double v = 0.0;
  for (int i = threadIdx.x; i < n; i += kThr) v += part[i];
  return bsum(v, red);
}

// ---------------------------------------------------------------------------
// level-0 CGLS passes (grid (kParts, systems of the group))
// ---------------------------------------------------------------------------

__device__ __forceinline__ bool active(const PcState* stv, int k) { return stv[k].status == kActive; }

// x = 0, r = 0, p = 0
__global__ void __launch_bounds__(kThr) k_pc_zero(const PcSys* __restrict__ sy, int g0) {
  const PcSys& S = sy[g0 + blockIdx.y];
  const float2 z = make_float2(0.f, 0.f);
  for (int c = blockIdx.x * kThr + threadIdx.x; c < S.lev[0].n; c += gridDim.x * kThr) {
    S.x[c] = z;
    S.r[0][c] = z;
    S.p[0][c] = z;
  }
}

// r1[src] = alpha (KNOWN), r2 = lam d, scalars reset (one block per system)
__global__ void __launch_bounds__(kThr) k_pc_init(const PcSys* __restrict__ sy, PcState* __restrict__ stv, int g0) {
  const int k = g0 + blockIdx.x;
  const PcSys& S = sy[k];
  for (int q = threadIdx.x; q < S.nr; q += kThr) {
    const float2 dv = S.d[q];
    S.r2[q] = fd(S.lam * dv.x, S.lam * dv.y);
  }
  if (threadIdx.x == 0) {
    if (!S.est) S.r[0][S.src] = fd(S.alpha.x, S.alpha.y);
    PcState& T = stv[k];
    T = PcState{};
    T.status = kActive;
  }
}

__device__ __forceinline__ float2 pc_pupd(const PcSys& S, double be, int c) {
  const float2 zv = S.z[c], pv = S.p[0][c], p = fd((double)zv.x + be * pv.x, (double)zv.y + be * pv.y);
  S.p[0][c] = p;
  return p;
}
// p = z + beta p (beta of the state; 0 at the start)
__global__ void __launch_bounds__(kThr) k_pc_pupd(const PcSys* __restrict__ sy, const PcState* __restrict__ stv,
                                                  int g0) {
  const int k = g0 + blockIdx.y;
  if (!active(stv, k)) return;
  const PcSys& S = sy[k];
  const double be = stv[k].beta;
  for (int c = blockIdx.x * kThr + threadIdx.x; c < S.lev[0].n; c += gridDim.x * kThr) pc_pupd(S, be, c);
}

__device__ __forceinline__ double sponge_at(const PcSys& S, int x, int y, int z) {
  return S.sp_scale * ((sponge_axis_d(x, S.lev[0].nx, S.nb, S.inv_nb) + sponge_axis_d(y, S.lev[0].ny, S.nb, S.inv_nb)) +
                       sponge_axis_d(z, S.lev[0].nz, S.nb, S.inv_nb));
}

// one cell of A v (adj = 0) or A^H v (adj = 1) in float64 from float32 storage
__device__ __forceinline__ double2 apply_cell(const PcSys& S, const float2* __restrict__ v, int c, bool adj) {
  const int plane = S.lev[0].nx * S.lev[0].ny;
  const int z = c / plane, rem = c - z * plane, y = rem / S.lev[0].nx, x = rem - y * S.lev[0].nx;
  const float2 zero = make_float2(0.f, 0.f);
  const float2 xm = x > 0 ? v[c - 1] : zero, xp = x < S.lev[0].nx - 1 ? v[c + 1] : zero;
  const float2 ym = y > 0 ? v[c - S.lev[0].nx] : zero, yp = y < S.lev[0].ny - 1 ? v[c + S.lev[0].nx] : zero;
  const float2 zm = z > 0 ? v[c - plane] : zero, zp = z < S.lev[0].nz - 1 ? v[c + plane] : zero;
  const double kim = S.omega * sponge_at(S, x, y, z);
  return helm(v[c], xm, xp, ym, yp, zm, zp, S.lev[0].h2inv, S.omega2 * (double)S.m[c], adj ? kim : -kim);
}

// t = A q - p_alpha e_src (ESTIMATE; q_alpha = p_alpha); partials of ||t||^2
__global__ void __launch_bounds__(kThr) k_pc_fwd(const PcSys* __restrict__ sy, const PcState* __restrict__ stv,
                                                 int g0) {
  __shared__ double red[kThr / 64];
  const int k = g0 + blockIdx.y;
  if (!active(stv, k)) return;
  const PcSys& S = sy[k];
  const double2 pa = stv[k].pa;
  double acc = 0.0;
  for (int c = blockIdx.x * kThr + threadIdx.x; c < S.lev[0].n; c += gridDim.x * kThr) {
    double2 tv = apply_cell(S, S.q, c, false);
    if (S.est && c == S.src) { tv.x -= pa.x; tv.y -= pa.y; }
    const float2 t = round2(tv);
    S.t[c] = t;
    acc += nrm(t);
  }
  const double tot = bsum(acc, red);
  if (threadIdx.x == 0) S.part[blockIdx.x] = tot;
}

// receiver rows t2 = lam q[rec]; delta, a; x_alpha += a p_alpha; r2 -= a t2
// (one block per system)
__global__ void __launch_bounds__(kThr) k_pc_step(const PcSys* __restrict__ sy, PcState* __restrict__ stv, int g0) {
  __shared__ double red[kThr / 64];
  const int k = g0 + blockIdx.x;
  if (!active(stv, k)) return;
  const PcSys& S = sy[k];
  PcState& T = stv[k];
  double acc = 0.0;
  for (int q = threadIdx.x; q < S.nr; q += kThr) {
    const float2 qv = S.q[S.rec[q]];
    const float2 t2 = fd(S.lam * qv.x, S.lam * qv.y);
    S.t2[q] = t2;
    acc += nrm(t2);
  }
  const double delta = sum_parts(S.part, S.nparts, red) + bsum(acc, red);
  const bool bad = !(delta > 0.0) || !(delta <= DBL_MAX) || !(T.gamma <= DBL_MAX);
  const double a = bad ? 0.0 : T.gamma / delta;
  for (int q = threadIdx.x; q < S.nr; q += kThr) {
    const float2 r2 = S.r2[q], t2 = S.t2[q];
    S.r2[q] = fd((double)r2.x - a * t2.x, (double)r2.y - a * t2.y);
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    T.a = a;
    if (bad) {
      T.status = kBreakdown;
    } else if (S.est) {
      T.xa = make_double2(T.xa.x + a * T.pa.x, T.xa.y + a * T.pa.y);
    }
  }
}

// r -= a t, x += a q
__global__ void __launch_bounds__(kThr) k_pc_rupd(const PcSys* __restrict__ sy, const PcState* __restrict__ stv,
                                                  int g0) {
  const int k = g0 + blockIdx.y;
  if (!active(stv, k)) return;
  const PcSys& S = sy[k];
  const double a = stv[k].a;
  for (int c = blockIdx.x * kThr + threadIdx.x; c < S.lev[0].n; c += gridDim.x * kThr) {
    const float2 r = S.r[0][c], t = S.t[c], x = S.x[c], q = S.q[c];
    S.r[0][c] = fd((double)r.x - a * t.x, (double)r.y - a * t.y);
    S.x[c] = fd((double)x.x + a * q.x, (double)x.y + a * q.y);
  }
}

// s = A^H r (the receiver and source-row terms are added per system); partials of ||s||^2
__global__ void __launch_bounds__(kThr) k_pc_adj(const PcSys* __restrict__ sy, const PcState* __restrict__ stv,
                                                 int g0) {
  __shared__ double red[kThr / 64];
  const int k = g0 + blockIdx.y;
  if (!active(stv, k)) return;
  const PcSys& S = sy[k];
  double acc = 0.0;
  for (int c = blockIdx.x * kThr + threadIdx.x; c < S.lev[0].n; c += gridDim.x * kThr) {
    const float2 s = round2(apply_cell(S, S.r[0], c, true));
    S.s[c] = s;
    acc += nrm(s);
  }
  const double tot = bsum(acc, red);
  if (threadIdx.x == 0) S.part[blockIdx.x] = tot;
}

// s += lam P^H r2 (distinct receiver cells), s_alpha = -r1[src] (ESTIMATE);
// ||s||^2, the stopping test (one block per system).  setup = 1: ||s_0||^2.
__global__ void __launch_bounds__(kThr) k_pc_check(const PcSys* __restrict__ sy, PcState* __restrict__ stv,
                                                   int g0, int setup) {
  __shared__ double red[kThr / 64];
  const int k = g0 + blockIdx.x;
  if (!active(stv, k)) return;
  const PcSys& S = sy[k];
  PcState& T = stv[k];
  double corr = 0.0;
  for (int q = threadIdx.x; q < S.nr; q += kThr) {
    const int c = S.rec[q];
    const float2 s0 = S.s[c], r2 = S.r2[q];
    const float2 s1 = fd((double)s0.x + S.lam * r2.x, (double)s0.y + S.lam * r2.y);
    S.s[c] = s1;
    corr += nrm(s1) - nrm(s0);
  }
  const double ss_u = sum_parts(S.part, S.nparts, red) + bsum(corr, red);
  if (threadIdx.x == 0) {
    double2 sa = make_double2(0.0, 0.0);
    if (S.est) {
      const float2 r1 = pc_r(S, setup ? 0 : T.iters + 1)[S.src];
      sa = make_double2(-(double)r1.x, -(double)r1.y);
    }
    const double ss = ss_u + sa.x * sa.x + sa.y * sa.y;
    T.za = sa;  // M leaves the source-weight component as it is: z_alpha = s_alpha
    T.ss = ss;
    if (setup) {
      T.ss0 = ss;
      T.ssmin = ss;
      if (ss == 0.0) T.status = kZeroRhs;
      else if (!(ss <= DBL_MAX)) T.status = kBreakdown;
      else if (S.rtol2 >= 1.0) T.status = kConverged;   // ||s_0|| <= rtol ||s_0||
      else if (S.max_iter <= 0) T.status = kMaxIter;
    } else {
      T.iters += 1;
      // below what float32 storage resolves the recurrences iterate on
      // rounding noise: a rise of ||S^H r|| 1e4 times above its running
      // minimum stops the system (as in the plain solver)
      T.ssmin = fmin(T.ssmin, ss);
      if (!(ss <= DBL_MAX)) T.status = kBreakdown;
      else if (ss <= S.rtol2 * T.ss0) T.status = kConverged;
      else if (T.iters >= S.max_iter) T.status = kMaxIter;
      else if (ss > kDivergeRatio * T.ssmin) T.status = kDiverged;
    }
  }
}

// gamma' = ||z||^2, beta = gamma'/gamma, p_alpha = z_alpha + beta p_alpha
// (one block per system).  setup = 1: gamma = ||z_0||^2, beta = 0.
__global__ void __launch_bounds__(kThr) k_pc_beta(const PcSys* __restrict__ sy, PcState* __restrict__ stv,
                                                  int g0, int setup) {
  __shared__ double red[kThr / 64];
  const int k = g0 + blockIdx.x;
  if (!active(stv, k)) return;
  const PcSys& S = sy[k];
  PcState& T = stv[k];
  const double zz = sum_parts(S.part, S.nparts, red) + (T.za.x * T.za.x + T.za.y * T.za.y);
  if (threadIdx.x == 0) {
    const double be = setup ? 0.0 : zz / T.gamma;
    T.beta = be;
    T.gamma = zz;
    T.pa = make_double2(T.za.x + be * T.pa.x, T.za.y + be * T.pa.y);
    if (!(zz > 0.0) || !(zz <= DBL_MAX)) T.status = (T.ss == 0.0) ? T.status : kBreakdown;
  }
}

// ---------------------------------------------------------------------------
// V-cycle passes (grid (blocks, systems of the group)); conj = 1: the cycle on
// conj(A_beta).  A level-0 pass reads its right-hand side from `in0` (p or s)
// and the level-0 result goes to `out0` (q or z).
// ---------------------------------------------------------------------------

// diagonal of A_beta (or its conjugate) at a cell: -6/h^2 + omega^2 (1 - i beta) m - i omega b
__device__ __forceinline__ double2 diag_beta(const PcSys& S, const PcLevel& L, int c, int conj) {
  const double m = L.m[c], b = L.b[c];
  const double im = -kBeta * S.omega2 * m - S.omega * b;
  return make_double2(-6.0 * L.h2inv + S.omega2 * m, conj ? -im : im);
}
// w D^-1 v with the tabulated w D^-1 (conjugated for the cycle on conj(A_beta))
__device__ __forceinline__ double2 jac(const PcLevel& L, int c, int conj, float2 v) {
  const float2 w = L.wdinv[c];
  const double wr = w.x, wi = conj ? -(double)w.y : (double)w.y;
  return make_double2(wr * v.x - wi * v.y, wr * v.y + wi * v.x);
}
__device__ __forceinline__ void coords(const PcLevel& L, int c, int& x, int& y, int& z) {
  const int plane = L.nx * L.ny;
  z = c / plane;
  const int rem = c - z * plane;
  y = rem / L.nx;
  x = rem - y * L.nx;
}

__device__ __forceinline__ const float2* level_in(const PcSys& S, int iters, int l, int which) {
  return l > 0 ? S.lev[l].f : (which ? S.s : pc_p(S, iters));
}

// res = f - A_beta (w D^-1 f) on level l (w D^-1 f recomputed at each neighbour)
__global__ void __launch_bounds__(kThr) k_pc_vdown(const PcSys* __restrict__ sy, const PcState* __restrict__ stv,
                                                   int g0, int l, int which, int conj) {
  const int k = g0 + blockIdx.y;
  if (!active(stv, k)) return;
  const PcSys& S = sy[k];
  if (l >= S.nlev - 1) return;
  const PcLevel& L = S.lev[l];
  const float2* __restrict__ f = level_in(S, stv[k].iters, l, which);
  for (int c = blockIdx.x * kThr + threadIdx.x; c < L.n; c += gridDim.x * kThr) {
    int x, y, z;
    coords(L, c, x, y, z);
    const int plane = L.nx * L.ny;
    double sr = 0.0, si = 0.0;
    const int nb[6] = {x > 0 ? c - 1 : -1, x < L.nx - 1 ? c + 1 : -1, y > 0 ? c - L.nx : -1,
                       y < L.ny - 1 ? c + L.nx : -1, z > 0 ? c - plane : -1, z < L.nz - 1 ? c + plane : -1};
#pragma unroll
    for (int i = 0; i < 6; ++i) {
      if (nb[i] < 0) continue;
      const double2 yn = jac(L, nb[i], conj, f[nb[i]]);
      sr += yn.x;
      si += yn.y;
    }
    const double2 d = diag_beta(S, L, c, conj);
    const float2 fc = f[c];
    const double2 yc = jac(L, c, conj, fc);
    const double ar = sr * L.h2inv + (d.x * yc.x - d.y * yc.y);
    const double ai = si * L.h2inv + (d.x * yc.y + d.y * yc.x);
    L.res[c] = fd((double)fc.x - ar, (double)fc.y - ai);
  }
}

// f_{l+1} = P^T res_l / 8 (27 fine cells around fine (2i+1, 2j+1, 2k+1))
__global__ void __launch_bounds__(kThr) k_pc_vrestrict(const PcSys* __restrict__ sy, const PcState* __restrict__ stv,
                                                       int g0, int l) {
  const int k = g0 + blockIdx.y;
  if (!active(stv, k)) return;
  const PcSys& S = sy[k];
  if (l >= S.nlev - 1) return;
  const PcLevel& F = S.lev[l];
  const PcLevel& C = S.lev[l + 1];
  for (int c = blockIdx.x * kThr + threadIdx.x; c < C.n; c += gridDim.x * kThr) {
    int cx, cy, cz;
    coords(C, c, cx, cy, cz);
    double sr = 0.0, si = 0.0;
    for (int dz = -1; dz <= 1; ++dz) {
      const int fz = 2 * cz + 1 + dz;
      if (fz < 0 || fz >= F.nz) continue;
      for (int dy = -1; dy <= 1; ++dy) {
        const int fy = 2 * cy + 1 + dy;
        if (fy < 0 || fy >= F.ny) continue;
        for (int dx = -1; dx <= 1; ++dx) {
          const int fx = 2 * cx + 1 + dx;
          if (fx < 0 || fx >= F.nx) continue;
          const double w = (dz ? 0.5 : 1.0) * (dy ? 0.5 : 1.0) * (dx ? 0.5 : 1.0);
          const float2 v = F.res[((size_t)fz * F.ny + fy) * F.nx + fx];
          sr += w * v.x;
          si += w * v.y;
        }
      }
    }
    C.f[c] = fd(0.125 * sr, 0.125 * si);
  }
}

// Jacobi step on the coarsest level: sweep 0: o = w D^-1 f; sweep j > 0:
// out = in + w D^-1 (f - A_beta in), in/out alternating o (j odd reads o) and y.
// Where level 0 is the only one (a grid too small or too thin to coarsen), the first
// sweep of the forward cycle also updates p, and the last one writes q or z, with the
// partials of ||z||^2 (kParts blocks).
__global__ void __launch_bounds__(kThr) k_pc_vcoarse(const PcSys* __restrict__ sy, const PcState* __restrict__ stv,
                                                     int g0, int which, int conj, int sweep) {
  __shared__ double red[kThr / 64];
  const int k = g0 + blockIdx.y;
  if (!active(stv, k)) return;
  const PcSys& S = sy[k];
  const int l = S.nlev - 1;
  const PcLevel& L = S.lev[l];
  const float2* __restrict__ f = level_in(S, stv[k].iters, l, which);
  const float2* __restrict__ in = (sweep & 1) ? L.o : L.y;
  const bool final = S.nlev == 1 && sweep == kCoarseSweeps - 1;
  float2* __restrict__ out = final ? (which ? S.z : S.q) : (sweep & 1) ? L.y : L.o;
  double acc = 0.0;
  for (int c = blockIdx.x * kThr + threadIdx.x; c < L.n; c += gridDim.x * kThr) {
    const double2 d = diag_beta(S, L, c, conj);
    if (sweep == 0) {
      const double2 v = jac(L, c, conj, S.nlev == 1 && which == 0 ? pc_pupd(S, stv[k].beta, c) : f[c]);
      out[c] = fd(v.x, v.y);
      continue;
    }
    int x, y, z;
    coords(L, c, x, y, z);
    const int plane = L.nx * L.ny;
    const float2 zero = make_float2(0.f, 0.f);
    const float2 xm = x > 0 ? in[c - 1] : zero, xp = x < L.nx - 1 ? in[c + 1] : zero;
    const float2 ym = y > 0 ? in[c - L.nx] : zero, yp = y < L.ny - 1 ? in[c + L.nx] : zero;
    const float2 zm = z > 0 ? in[c - plane] : zero, zp = z < L.nz - 1 ? in[c + plane] : zero;
    const float2 xc = in[c];
    const double sr = (((double)xm.x + xp.x) + ((double)ym.x + yp.x)) + ((double)zm.x + zp.x);
    const double si = (((double)xm.y + xp.y) + ((double)ym.y + yp.y)) + ((double)zm.y + zp.y);
    const double ar = sr * L.h2inv + (d.x * xc.x - d.y * xc.y);
    const double ai = si * L.h2inv + (d.x * xc.y + d.y * xc.x);
    const float2 fc = f[c];
    const double2 corr = jac(L, c, conj, fd((double)fc.x - ar, (double)fc.y - ai));
    const float2 o = fd((double)xc.x + corr.x, (double)xc.y + corr.y);
    out[c] = o;
    acc += nrm(o);
  }
  if (final && which) {
    const double tot = bsum(acc, red);
    if (threadIdx.x == 0) S.part[blockIdx.x] = tot;
  }
}

// the coarsest level's result: after kCoarseSweeps sweeps it is in o (odd count) or y
__device__ __forceinline__ const float2* coarse_out(const PcSys& S, int l) {
  const PcLevel& L = S.lev[l];
  if (l < S.nlev - 1) return L.o;
  return (kCoarseSweeps & 1) ? L.o : L.y;
}

// y_l = w D^-1 f_l + P e_{l+1} (trilinear)
__global__ void __launch_bounds__(kThr) k_pc_vprolong(const PcSys* __restrict__ sy, const PcState* __restrict__ stv,
                                                      int g0, int l, int which, int conj) {
  const int k = g0 + blockIdx.y;
  if (!active(stv, k)) return;
  const PcSys& S = sy[k];
  if (l >= S.nlev - 1) return;
  const PcLevel& F = S.lev[l];
  const PcLevel& C = S.lev[l + 1];
  const float2* __restrict__ e = coarse_out(S, l + 1);
  const float2* __restrict__ f = level_in(S, stv[k].iters, l, which);
  for (int c = blockIdx.x * kThr + threadIdx.x; c < F.n; c += gridDim.x * kThr) {
    int x, y, z;
    coords(F, c, x, y, z);
    // 1D interpolation: odd fine f <- coarse (f-1)/2 (1); even f <- f/2 - 1 and f/2 (1/2 each)
    int ix[2], iy[2], iz[2];
    double wx[2], wy[2], wz[2];
    auto axis = [](int fi, int nc, int* id, double* w) {
      if (fi & 1) { id[0] = (fi - 1) >> 1; w[0] = 1.0; id[1] = -1; w[1] = 0.0; }
      else {
        id[0] = (fi >> 1) - 1; w[0] = 0.5; id[1] = fi >> 1; w[1] = 0.5;
        if (id[1] >= nc) id[1] = -1;
      }
      if (id[0] >= nc) id[0] = -1;
    };
    axis(x, C.nx, ix, wx);
    axis(y, C.ny, iy, wy);
    axis(z, C.nz, iz, wz);
    double sr = 0.0, si = 0.0;
    for (int a = 0; a < 2; ++a) {
      if (iz[a] < 0) continue;
      for (int b = 0; b < 2; ++b) {
        if (iy[b] < 0) continue;
        for (int cc = 0; cc < 2; ++cc) {
          if (ix[cc] < 0) continue;
          const double w = wz[a] * wy[b] * wx[cc];
          const float2 v = e[((size_t)iz[a] * C.ny + iy[b]) * C.nx + ix[cc]];
          sr += w * v.x;
          si += w * v.y;
        }
      }
    }
    const double2 j = jac(F, c, conj, f[c]);
    F.y[c] = fd(j.x + sr, j.y + si);
  }
}

// o_l = y + w D^-1 (f - A_beta y); level 0 writes `out0` (q: which = 0, z:
// which = 1) and, for z, the partials of ||z||^2
__global__ void __launch_bounds__(kThr) k_pc_vsmooth(const PcSys* __restrict__ sy, const PcState* __restrict__ stv,
                                                     int g0, int l, int which, int conj) {
  __shared__ double red[kThr / 64];
  const int k = g0 + blockIdx.y;
  if (!active(stv, k)) return;
  const PcSys& S = sy[k];
  if (l >= S.nlev - 1) return;
  const PcLevel& L = S.lev[l];
  const float2* __restrict__ f = level_in(S, stv[k].iters, l, which);
  const float2* __restrict__ in = L.y;
  float2* __restrict__ out = l > 0 ? L.o : (which ? S.z : S.q);
  double acc = 0.0;
  for (int c = blockIdx.x * kThr + threadIdx.x; c < L.n; c += gridDim.x * kThr) {
    int x, y, z;
    coords(L, c, x, y, z);
    const int plane = L.nx * L.ny;
    const float2 zero = make_float2(0.f, 0.f);
    const float2 xm = x > 0 ? in[c - 1] : zero, xp = x < L.nx - 1 ? in[c + 1] : zero;
    const float2 ym = y > 0 ? in[c - L.nx] : zero, yp = y < L.ny - 1 ? in[c + L.nx] : zero;
    const float2 zm = z > 0 ? in[c - plane] : zero, zp = z < L.nz - 1 ? in[c + plane] : zero;
    const float2 xc = in[c];
    const double2 d = diag_beta(S, L, c, conj);
    const double sr = (((double)xm.x + xp.x) + ((double)ym.x + yp.x)) + ((double)zm.x + zp.x);
    const double si = (((double)xm.y + xp.y) + ((double)ym.y + yp.y)) + ((double)zm.y + zp.y);
    const double ar = sr * L.h2inv + (d.x * xc.x - d.y * xc.y);
    const double ai = si * L.h2inv + (d.x * xc.y + d.y * xc.x);
    const float2 fc = f[c];
    const double2 corr = jac(L, c, conj, fd((double)fc.x - ar, (double)fc.y - ai));
    const float2 o = fd((double)xc.x + corr.x, (double)xc.y + corr.y);
    out[c] = o;
    acc += nrm(o);
  }
  if (l == 0 && which) {
    const double tot = bsum(acc, red);
    if (threadIdx.x == 0) S.part[blockIdx.x] = tot;
  }
}

// ---------------------------------------------------------------------------
// the same passes by window tiles
//
// One thread per cell with two divisions and up to 27 loads from the caches left
// an iteration of 39 launches of 3 to 10 us on the medium workload.  Here a
// workgroup owns consecutive cells of the x-y plane and kPcZ planes (window.hpp):
// all its loads are issued at once and the neighbours come from LDS.  The p update
// is part of the first pass of the forward cycle, prolongation and the step after
// it are one pass (the prolonged iterate is formed on the tile and its halo and
// never stored), the r and x updates are part of s = A^H r, and the levels of up to
// kPcLdsCells cells are one workgroup per system with every array in LDS: 19
// launches.  Every stored value is rounded where it was, so iterates differ only
// through the order of the float64 sums; r and p are written to their other
// buffer because neighbouring tiles still read the old one.
//
// Per iteration (eager launches): 8 systems of 64^3 401 us before and 194 now,
// 48 of 128^3 11.7 ms and 5.07, 2 of 24x20x18 178 us and 75.
// ---------------------------------------------------------------------------

constexpr int kPcW = 4, kPcZ = 4;
constexpr int kPcMaxRow = 512;         // widest row of the tiled passes (LDS: 96 KB for the residual pass)
constexpr int kPcLdsCells = 4096;      // largest level of the one-workgroup cycle
constexpr int kPcLdsThr = 1024;

// (system, tile) of a block: neighbouring tiles of a system on one XCD.  The same tile
// of 2 or 4 systems on consecutive blocks, so that they share w D^-1, m and b in L2,
// measured 5.19 and 5.24 ms an iteration against 5.14 (48 systems of 128^3).
__device__ __forceinline__ void pc_block(int tiles, int* sys, int* tile) {
  const int logical = xcd_remap(blockIdx.x, gridDim.x, max(16, tiles / 2));
  *sys = logical / tiles;
  *tile = logical - *sys * tiles;
}

// y = w D^-1 f in float64
__device__ __forceinline__ double2 jac_w(float2 w, int conj, float2 v) {
  const double wr = w.x, wi = conj ? -(double)w.y : (double)w.y;
  return make_double2(wr * v.x - wi * v.y, wr * v.y + wi * v.x);
}
__device__ __forceinline__ double2 diag_mb(const PcSys& S, double h2inv, float m_, float b_, int conj) {
  const double m = m_, b = b_;
  const double im = -kBeta * S.omega2 * m - S.omega * b;
  return make_double2(-6.0 * h2inv + S.omega2 * m, conj ? -im : im);
}

// res = f - A_beta (w D^-1 f) on level l; PUPD: level 0 of the forward cycle, with
// f = p = z + beta p formed and stored here
template <int CX, bool PUPD>
__global__ void __launch_bounds__(64 * kPcW)
k_pw_down(const PcSys* __restrict__ sy, const PcState* __restrict__ stv, int g0, int l, int which, int conj,
          int tiles_x, int tiles) {
  using Tile = Win<kPcW, CX, kPcZ>;
  constexpr int NT = Tile::NT;
  extern __shared__ double2 pw_y[];   // [kPcZ][B + 2 nx]: w D^-1 f
  const int tid = threadIdx.x;
  int sys, tile;
  pc_block(tiles, &sys, &tile);
  const int k = g0 + sys;
  const PcState& T = stv[k];
  if (T.status != kActive) return;
  const PcSys& S = sy[k];
  const PcLevel& L = S.lev[l];
  Tile Q;
  Q.setup(L.nx, L.ny, L.nz, tile, tiles_x);
  const int nx = Q.nx, wl = Q.wl;
  const float2* f = PUPD ? S.z : level_in(S, T.iters, l, which);
  const float2* po = S.p[T.iters & 1];
  float2* pn = S.p[(T.iters + 1) & 1];
  float2 fv[CX][kPcZ + 2], wv[CX][kPcZ + 2], pv[CX][kPcZ + 2];
  float mm[CX][kPcZ], bb[CX][kPcZ];
#pragma unroll
  for (int j = 0; j < CX; ++j)
#pragma unroll
    for (int i = 0; i < kPcZ + 2; ++i) {
      fv[j][i] = Q.load2(f, i, Q.own2(j));
      wv[j][i] = Q.load2(L.wdinv, i, Q.own2(j));
      if constexpr (PUPD) pv[j][i] = Q.load2(po, i, Q.own2(j));
    }
#pragma unroll
  for (int j = 0; j < CX; ++j)
#pragma unroll
    for (int i = 0; i < kPcZ; ++i) {
      mm[j][i] = Q.load1(L.m, i + 1, Q.own1(j));
      bb[j][i] = Q.load1(L.b, i + 1, Q.own1(j));
    }
  issue_point();
  const double be = PUPD ? T.beta : 0.0;
  auto dir = [&](float2 z, float2 p) { return fd((double)z.x + be * p.x, (double)z.y + be * p.y); };
  for (int h = tid; h < 2 * nx; h += NT) {
    const unsigned o = Q.halo_off(h);
    const int sl = Q.halo_slot(h);
    float2 hf[kPcZ], hw[kPcZ], hp[kPcZ];
#pragma unroll
    for (int i = 0; i < kPcZ; ++i) {
      hf[i] = Q.load2(f, i + 1, o);
      hw[i] = Q.load2(L.wdinv, i + 1, o);
      if constexpr (PUPD) hp[i] = Q.load2(po, i + 1, o);
    }
#pragma unroll
    for (int i = 0; i < kPcZ; ++i) {
      if constexpr (PUPD) hf[i] = dir(hf[i], hp[i]);
      pw_y[i * wl + sl] = jac_w(hw[i], conj, hf[i]);
    }
  }
  double2 y[CX][kPcZ + 2];
#pragma unroll
  for (int j = 0; j < CX; ++j)
#pragma unroll
    for (int i = 0; i < kPcZ + 2; ++i) {
      if constexpr (PUPD) fv[j][i] = dir(fv[j][i], pv[j][i]);
      y[j][i] = jac_w(wv[j][i], conj, fv[j][i]);
      if (i >= 1 && i <= kPcZ) pw_y[(i - 1) * wl + nx + j * NT + tid] = y[j][i];
    }
  __syncthreads();
#pragma unroll
  for (int j = 0; j < CX; ++j) {
    int cx, cy;
    Q.row_of(Q.cell[j], &cx, &cy);
    const unsigned mxm = row_mask(cx > 0), mxp = row_mask(cx < nx - 1);
#pragma unroll
    for (int i = 0; i < kPcZ; ++i) {
      const double2* row = pw_y + i * wl + nx + j * NT + tid;
      const double2 xm = masked(row[-1], mxm), xp = masked(row[1], mxp), ym = row[-nx], yp = row[nx];
      const double2 yc = y[j][i + 1], zm = y[j][i], zp = y[j][i + 2];
      const double sr = ((((xm.x + xp.x) + ym.x) + yp.x) + zm.x) + zp.x;
      const double si = ((((xm.y + xp.y) + ym.y) + yp.y) + zm.y) + zp.y;
      const double2 d = diag_mb(S, L.h2inv, mm[j][i], bb[j][i], conj);
      const float2 fc = fv[j][i + 1];
      const double ar = sr * L.h2inv + (d.x * yc.x - d.y * yc.y);
      const double ai = si * L.h2inv + (d.x * yc.y + d.y * yc.x);
      Q.store2(L.res, i + 1, Q.own2(j), fd((double)fc.x - ar, (double)fc.y - ai));
      if constexpr (PUPD) Q.store2(pn, i + 1, Q.own2(j), fc);
    }
  }
}

// f_{l+1} = P^T res_l / 8: one coarse cell per thread.  A row of the 27 cells is one
// 16-byte load of the first two (contiguous across lanes) and the next lane's
// first; only the last lane and the end of a row load their third cell.  Weights are
// powers of two and the values float32, so the float64 sums are exact in any order
// unless the magnitudes span more than 2^26.
__global__ void __launch_bounds__(kThr)
k_pw_restrict(const PcSys* __restrict__ sy, const PcState* __restrict__ stv, int g0, int l, int tiles) {
  int sys, tile;
  pc_block(tiles, &sys, &tile);
  const int k = g0 + sys;
  if (!active(stv, k)) return;
  const PcSys& S = sy[k];
  const PcLevel& F = S.lev[l];
  const PcLevel& C = S.lev[l + 1];
  const int c = tile * kThr + threadIdx.x;
  const bool live = c < C.n;
  int cx, cy, cz;
  coords(C, live ? c : C.n - 1, cx, cy, cz);
  const int plane = F.nx * F.ny, o = 2 * cz * plane + 2 * cy * F.nx + 2 * cx;   // fine corner: 2i .. 2i + 2
  const BufRes R = mkbuf(F.res, 0, F.n, 8);
  // the next lane holds the next coarse cell of the row
  const bool from_next = (threadIdx.x & 63) != 63 && cx + 1 < C.nx && c + 1 < C.n;
  const bool third = 2 * cx + 2 < F.nx;
  float4 v[9];
  float2 w[9];
#pragma unroll
  for (int dz = 0; dz < 3; ++dz)
#pragma unroll
    for (int dy = 0; dy < 3; ++dy) {
      const bool in = 2 * cy + dy < F.ny && 2 * cz + dz < F.nz;   // a coarse cell has two fine ones in x
      const unsigned off = (unsigned)((o + dz * plane + dy * F.nx) * 8);
      v[dz * 3 + dy] = bld4(R, in ? off : kOOB);
      w[dz * 3 + dy] = bld2(R, in && third && !from_next ? off + 16 : kOOB);
    }
  double sr = 0.0, si = 0.0;
#pragma unroll
  for (int dz = 0; dz < 3; ++dz)
#pragma unroll
    for (int dy = 0; dy < 3; ++dy) {
      const int i = dz * 3 + dy;
      const float nx_ = __shfl_down(v[i].x, 1, 64), ny_ = __shfl_down(v[i].y, 1, 64);
      const float tx = from_next ? nx_ : w[i].x, ty = from_next ? ny_ : w[i].y;
      const double wt = (dz != 1 ? 0.5 : 1.0) * (dy != 1 ? 0.5 : 1.0);
      sr += wt * ((double)v[i].z + 0.5 * ((double)v[i].x + (double)tx));
      si += wt * ((double)v[i].w + 0.5 * ((double)v[i].y + (double)ty));
    }
  if (live) C.f[c] = fd(0.125 * sr, 0.125 * si);
}

// One column of P e on the coarse planes z0 / 2 - 1 + p, interpolated in x and y
// (exact in float64, see the restriction).  Cells outside the coarse grid read zero.
template <int NP>
__device__ __forceinline__ void coarse_column(BufRes R, const PcLevel& C, bool ok, int x, int y, int z0,
                                              double2 (&out)[NP]) {
  const bool ox = x & 1, oy = y & 1;
  const int x1 = x >> 1, x0 = ox ? x1 : x1 - 1;   // odd: one coarse cell; even: two
  const int y1 = y >> 1, y0 = oy ? y1 : y1 - 1;
  const double w = (ox ? 1.0 : 0.5) * (oy ? 1.0 : 0.5);
  const bool bx0 = ok && x0 >= 0 && x0 < C.nx, bx1 = ok && !ox && x1 < C.nx;
  const bool by0 = y0 >= 0 && y0 < C.ny, by1 = !oy && y1 < C.ny;
  const int plane = C.nx * C.ny;
  auto off = [&](bool in, int yy, int xx) { return in ? (unsigned)((yy * C.nx + xx) * 8) : kOOB; };
  const unsigned o[4] = {off(by0 && bx0, y0, x0), off(by0 && bx1, y0, x1), off(by1 && bx0, y1, x0),
                         off(by1 && bx1, y1, x1)};
  float2 v[NP][4];
#pragma unroll
  for (int p = 0; p < NP; ++p) {
    const int z = z0 / 2 - 1 + p;
    const unsigned zo = z >= 0 && z < C.nz ? (unsigned)(z * plane * 8) : kOOB;
#pragma unroll
    for (int i = 0; i < 4; ++i) v[p][i] = bld2(R, (o[i] & kOOB) ? kOOB : o[i] + zo);
  }
#pragma unroll
  for (int p = 0; p < NP; ++p)
    out[p] = make_double2(w * (((double)v[p][0].x + (double)v[p][1].x) + ((double)v[p][2].x + (double)v[p][3].x)),
                          w * (((double)v[p][0].y + (double)v[p][1].y) + ((double)v[p][2].y + (double)v[p][3].y)));
}
// P e on the fine plane z0 - 1 + i (z0 even) from the coarse planes z0 / 2 - 1 + p
template <int NP>
__device__ __forceinline__ double2 prolong_z(const double2 (&e)[NP], int i) {
  const int p = i >> 1;   // odd planes (i even): one coarse plane; even planes: two
  if ((i & 1) == 0) return e[p];
  return make_double2(0.5 * (e[p].x + e[p + 1].x), 0.5 * (e[p].y + e[p + 1].y));
}

// o_l = y + w D^-1 (f - A_beta y) with y = w D^-1 f + P e_{l+1}; level 0 writes q
// (which = 0) or z (which = 1, with the partials of ||z||^2)
template <int CX>
__global__ void __launch_bounds__(64 * kPcW)
k_pw_up(const PcSys* __restrict__ sy, const PcState* __restrict__ stv, int g0, int l, int which, int conj,
        int tiles_x, int tiles) {
  using Tile = Win<kPcW, CX, kPcZ>;
  constexpr int NT = Tile::NT, NP = kPcZ / 2 + 2;
  __shared__ double red[kPcW];
  extern __shared__ float2 pw_f[];   // [kPcZ][B + 2 nx]: y
  const int tid = threadIdx.x;
  int sys, tile;
  pc_block(tiles, &sys, &tile);
  const int k = g0 + sys;
  const PcState& T = stv[k];
  if (T.status != kActive) return;
  const PcSys& S = sy[k];
  const PcLevel& L = S.lev[l];
  const PcLevel& C = S.lev[l + 1];
  Tile Q;
  Q.setup(L.nx, L.ny, L.nz, tile, tiles_x);
  const int nx = Q.nx, wl = Q.wl;
  const float2* f = level_in(S, T.iters, l, which);
  const BufRes Re = mkbuf(coarse_out(S, l + 1), 0, C.n, 8);   // one resource: per plane ones became a loop per load
  float2* out = l > 0 ? L.o : (which ? S.z : S.q);
  float2 fv[CX][kPcZ + 2], wv[CX][kPcZ + 2];
  float mm[CX][kPcZ], bb[CX][kPcZ];
#pragma unroll
  for (int j = 0; j < CX; ++j)
#pragma unroll
    for (int i = 0; i < kPcZ + 2; ++i) {
      fv[j][i] = Q.load2(f, i, Q.own2(j));
      wv[j][i] = Q.load2(L.wdinv, i, Q.own2(j));
    }
#pragma unroll
  for (int j = 0; j < CX; ++j)
#pragma unroll
    for (int i = 0; i < kPcZ; ++i) {
      mm[j][i] = Q.load1(L.m, i + 1, Q.own1(j));
      bb[j][i] = Q.load1(L.b, i + 1, Q.own1(j));
    }
  issue_point();
  for (int h = tid; h < 2 * nx; h += NT) {
    const unsigned o = Q.halo_off(h);
    const int sl = Q.halo_slot(h);
    const bool ok = (o & kOOB) == 0;
    float2 hf[kPcZ], hw[kPcZ];
#pragma unroll
    for (int i = 0; i < kPcZ; ++i) {
      hf[i] = Q.load2(f, i + 1, o);
      hw[i] = Q.load2(L.wdinv, i + 1, o);
    }
    int x, y;
    Q.row_of((h < nx ? Q.c0 - nx + h : Q.c0 + Tile::B + (h - nx)) + nx, &x, &y);   // the row above: not negative
    double2 ec[NP];
    coarse_column(Re, C, ok, x, y - 1, Q.z0, ec);
#pragma unroll
    for (int i = 0; i < kPcZ; ++i) {
      const double2 jv = jac_w(hw[i], conj, hf[i]), pe = prolong_z(ec, i + 1);
      pw_f[i * wl + sl] = ok && Q.zin(i + 1) ? fd(jv.x + pe.x, jv.y + pe.y) : make_float2(0.f, 0.f);
    }
  }
  float2 yv[CX][kPcZ + 2];
  int cx[CX];
#pragma unroll
  for (int j = 0; j < CX; ++j) {
    int cy;
    Q.row_of(Q.cell[j], &cx[j], &cy);
    double2 ec[NP];
    coarse_column(Re, C, Q.in[j], cx[j], cy, Q.z0, ec);
#pragma unroll
    for (int i = 0; i < kPcZ + 2; ++i) {
      const double2 jv = jac_w(wv[j][i], conj, fv[j][i]), pe = prolong_z(ec, i);
      yv[j][i] = Q.in[j] && Q.zin(i) ? fd(jv.x + pe.x, jv.y + pe.y) : make_float2(0.f, 0.f);
      if (i >= 1 && i <= kPcZ) pw_f[(i - 1) * wl + nx + j * NT + tid] = yv[j][i];
    }
  }
  __syncthreads();
  double acc = 0.0;
#pragma unroll
  for (int j = 0; j < CX; ++j) {
    const unsigned mxm = row_mask(cx[j] > 0), mxp = row_mask(cx[j] < nx - 1);
#pragma unroll
    for (int i = 0; i < kPcZ; ++i) {
      const float2* row = pw_f + i * wl + nx + j * NT + tid;
      const float2 xm = masked(row[-1], mxm), xp = masked(row[1], mxp), ym = row[-nx], yp = row[nx];
      const float2 xc = yv[j][i + 1], zm = yv[j][i], zp = yv[j][i + 2], fc = fv[j][i + 1];
      const double2 d = diag_mb(S, L.h2inv, mm[j][i], bb[j][i], conj);
      const double sr = (((double)xm.x + xp.x) + ((double)ym.x + yp.x)) + ((double)zm.x + zp.x);
      const double si = (((double)xm.y + xp.y) + ((double)ym.y + yp.y)) + ((double)zm.y + zp.y);
      const double ar = sr * L.h2inv + (d.x * xc.x - d.y * xc.y);
      const double ai = si * L.h2inv + (d.x * xc.y + d.y * xc.x);
      const double2 corr = jac_w(wv[j][i + 1], conj, fd((double)fc.x - ar, (double)fc.y - ai));
      const float2 o = fd((double)xc.x + corr.x, (double)xc.y + corr.y);
      Q.store2(out, i + 1, Q.own2(j), o);
      if (Q.live(j, i)) acc += nrm(o);
    }
  }
  if (l == 0 && which) {
    const double tot = bsum(acc, red);
    if (tid == 0) S.part[tile] = tot;
  }
}

// t = A q - p_alpha e_src; partials of ||t||^2 (ADJ = false), or the step on r and x
// and s = A^H r with the partials of ||s||^2 (ADJ = true; setup = 1: s = A^H r_0)
template <int CX, bool ADJ>
__global__ void __launch_bounds__(64 * kPcW)
k_pw_apply(const PcSys* __restrict__ sy, const PcState* __restrict__ stv, int g0, int setup, int tiles_x, int tiles) {
  using Tile = Win<kPcW, CX, kPcZ>;
  constexpr int NT = Tile::NT;
  __shared__ double red[kThr / 64];
  extern __shared__ float2 pw_f[];   // [kPcZ][B + 2 nx]
  const int tid = threadIdx.x;
  int sys, tile;
  pc_block(tiles, &sys, &tile);
  const int k = g0 + sys;
  const PcState& T = stv[k];
  if (T.status != kActive) return;
  const PcSys& S = sy[k];
  Tile Q;
  Q.setup(S.lev[0].nx, S.lev[0].ny, S.lev[0].nz, tile, tiles_x);
  const int nx = Q.nx, wl = Q.wl;
  const float2* in = ADJ ? pc_r(S, setup ? 0 : T.iters) : S.q;
  float2* rn = pc_r(S, T.iters + 1);
  const unsigned tbit = setup ? kOOB : 0u;   // the set-up pass makes no step
  float2 v[CX][kPcZ + 2], tv[CX][kPcZ + 2], xv[CX][kPcZ], qv[CX][kPcZ];
  float mm[CX][kPcZ];
#pragma unroll
  for (int j = 0; j < CX; ++j)
#pragma unroll
    for (int i = 0; i < kPcZ + 2; ++i) {
      v[j][i] = Q.load2(in, i, Q.own2(j));
      if constexpr (ADJ) tv[j][i] = Q.load2(S.t, i, Q.own2(j) | tbit);
    }
#pragma unroll
  for (int j = 0; j < CX; ++j)
#pragma unroll
    for (int i = 0; i < kPcZ; ++i) {
      mm[j][i] = Q.load1(S.m, i + 1, Q.own1(j));
      if constexpr (ADJ) {
        xv[j][i] = Q.load2(S.x, i + 1, Q.own2(j) | tbit);
        qv[j][i] = Q.load2(S.q, i + 1, Q.own2(j) | tbit);
      }
    }
  issue_point();
  const double a = ADJ && !setup ? T.a : 0.0;
  auto step = [&](float2 r, float2 t) { return setup ? r : fd((double)r.x - a * t.x, (double)r.y - a * t.y); };
  for (int h = tid; h < 2 * nx; h += NT) {
    const unsigned o = Q.halo_off(h);
    const int sl = Q.halo_slot(h);
    float2 hv[kPcZ], ht[kPcZ];
#pragma unroll
    for (int i = 0; i < kPcZ; ++i) {
      hv[i] = Q.load2(in, i + 1, o);
      if constexpr (ADJ) ht[i] = Q.load2(S.t, i + 1, o | tbit);
    }
#pragma unroll
    for (int i = 0; i < kPcZ; ++i) {
      if constexpr (ADJ) hv[i] = step(hv[i], ht[i]);
      pw_f[i * wl + sl] = hv[i];
    }
  }
#pragma unroll
  for (int j = 0; j < CX; ++j)
#pragma unroll
    for (int i = 0; i < kPcZ + 2; ++i) {
      if constexpr (ADJ) v[j][i] = step(v[j][i], tv[j][i]);
      if (i >= 1 && i <= kPcZ) pw_f[(i - 1) * wl + nx + j * NT + tid] = v[j][i];
    }
  __syncthreads();
  const bool src_tile = !ADJ && S.est;
  const double2 pa = T.pa;
  double acc = 0.0;
#pragma unroll
  for (int j = 0; j < CX; ++j) {
    int cx, cy;
    Q.row_of(Q.cell[j], &cx, &cy);
    const unsigned mxm = row_mask(cx > 0), mxp = row_mask(cx < nx - 1);
    const double sxy = sponge_axis_d(cx, nx, S.nb, S.inv_nb) + sponge_axis_d(cy, Q.ny, S.nb, S.inv_nb);
#pragma unroll
    for (int i = 0; i < kPcZ; ++i) {
      const float2* row = pw_f + i * wl + nx + j * NT + tid;
      const float2 xm = masked(row[-1], mxm), xp = masked(row[1], mxp), ym = row[-nx], yp = row[nx];
      const double kim = S.omega * (S.sp_scale * (sxy + sponge_axis_d(Q.z0 + i, Q.nz, S.nb, S.inv_nb)));
      double2 y = helm(v[j][i + 1], xm, xp, ym, yp, v[j][i], v[j][i + 2], S.lev[0].h2inv, S.omega2 * (double)mm[j][i],
                       ADJ ? kim : -kim);
      if (src_tile && S.src == (Q.z0 + i) * Q.plane + Q.cell[j] && Q.in[j]) { y.x -= pa.x; y.y -= pa.y; }
      const float2 o = round2(y);
      Q.store2(ADJ ? S.s : S.t, i + 1, Q.own2(j), o);
      if (Q.live(j, i)) acc += nrm(o);
      if constexpr (ADJ) {
        if (!setup) {
          Q.store2(rn, i + 1, Q.own2(j), v[j][i + 1]);
          Q.store2(S.x, i + 1, Q.own2(j), fd((double)xv[j][i].x + a * qv[j][i].x, (double)xv[j][i].y + a * qv[j][i].y));
        }
      }
    }
  }
  const double tot = bsum(acc, red);
  if (tid == 0) S.part[tile] = tot;
}

// The levels from lc on (at most kPcLdsCells cells each, lc >= 1): down, the Jacobi
// steps of the coarsest, up, with f and the iterate of every level in LDS.  One
// workgroup per system; f_{lc} is read from and the result of level lc written to
// memory.  Bound by one compute unit's vector rate on the first level: w D^-1 f is
// formed once per cell (float64, in LDS) and coordinates come without divisions.
struct SmallDiv {   // quotients of integers below 2^16 by d, through the float reciprocal
  int d;
  float r;
  __device__ __forceinline__ explicit SmallDiv(int d_) : d(d_), r(1.0f / (float)d_) {}
  __device__ __forceinline__ int quot(int c) const { return (int)(((float)c + 0.5f) * r); }
};

// SINGLE: the whole cycle of a grid of one level (lc = 0), with the partials of ||z||^2 as
// the per-cell passes form them: a grid this small is bound by its launches, five for a
// cycle otherwise.  300 iterations of two systems of 8x8x8: 17.8 ms with eager passes, 15.4
// replayed from a graph, 11.4 now; of 5x1x7 18.1, 13.6 and 10.6.
template <bool SINGLE>
__global__ void __launch_bounds__(kPcLdsThr)
k_pw_coarse(const PcSys* __restrict__ sy, const PcState* __restrict__ stv, int g0, int lc, int which, int conj) {
  constexpr int KC = kPcLdsCells / kPcLdsThr;   // cells per thread
  extern __shared__ double2 pc_lds[];
  const int k = g0 + blockIdx.x;
  if (!active(stv, k)) return;
  const PcSys& S = sy[k];
  const int last = S.nlev - 1, tid = threadIdx.x;
  const float2 zero = make_float2(0.f, 0.f);
  // w D^-1 f of the level at hand (the coarsest: its second iterate), then per level f and y (or the residual)
  double2* yd = pc_lds;
  float2* pl = reinterpret_cast<float2*>(pc_lds + S.lev[lc].n);
  auto base = [&](int l) {
    int o = 0;
    for (int i = lc; i < l; ++i) o += 2 * S.lev[i].n;
    return pl + o;
  };
  auto coord = [&](const PcLevel& L, const SmallDiv& dx, const SmallDiv& dp, int c, int* x, int* y, int* z) {
    *z = dp.quot(c);
    const int rem = c - *z * dp.d;
    *y = dx.quot(rem);
    *x = rem - *y * L.nx;
  };
  // A_beta v of a float2 array in LDS
  auto apply = [&](const PcLevel& L, const float2* v, int c, int x, int y, int z, const double2& d) {
    const int plane = L.nx * L.ny;
    const float2 xm = x > 0 ? v[c - 1] : zero, xp = x < L.nx - 1 ? v[c + 1] : zero;
    const float2 ym = y > 0 ? v[c - L.nx] : zero, yp = y < L.ny - 1 ? v[c + L.nx] : zero;
    const float2 zm = z > 0 ? v[c - plane] : zero, zp = z < L.nz - 1 ? v[c + plane] : zero;
    const float2 xc = v[c];
    const double sr = (((double)xm.x + xp.x) + ((double)ym.x + yp.x)) + ((double)zm.x + zp.x);
    const double si = (((double)xm.y + xp.y) + ((double)ym.y + yp.y)) + ((double)zm.y + zp.y);
    return make_double2(sr * L.h2inv + (d.x * xc.x - d.y * xc.y), si * L.h2inv + (d.x * xc.y + d.y * xc.x));
  };
  // own cells' w D^-1 and diagonal of a level
  auto own = [&](const PcLevel& L, float2 (&w)[KC], double2 (&d)[KC]) {
    float mv[KC], bv[KC];
#pragma unroll
    for (int i = 0; i < KC; ++i) {
      const int c = min(tid + i * kPcLdsThr, L.n - 1);
      w[i] = L.wdinv[c];
      mv[i] = L.m[c];
      bv[i] = L.b[c];
    }
#pragma unroll
    for (int i = 0; i < KC; ++i) d[i] = diag_mb(S, L.h2inv, mv[i], bv[i], conj);
  };
  for (int c = tid; c < S.lev[lc].n; c += kPcLdsThr) {
    if constexpr (SINGLE) pl[c] = which ? S.s[c] : pc_pupd(S, stv[k].beta, c);
    else pl[c] = S.lev[lc].f[c];
  }
  for (int l = lc; l < last; ++l) {
    const PcLevel& L = S.lev[l];
    const PcLevel& C = S.lev[l + 1];
    const int plane = L.nx * L.ny;
    const SmallDiv dx(L.nx), dp(plane), cdx(C.nx), cdp(C.nx * C.ny);
    float2 *f = base(l), *res = f + L.n, *fc = base(l + 1);
    float2 w[KC];
    double2 d[KC];
    own(L, w, d);
#pragma unroll
    for (int i = 0; i < KC; ++i) {   // f of the own cells was written by this thread, or behind a barrier
      const int c = tid + i * kPcLdsThr;
      if (c < L.n) yd[c] = jac_w(w[i], conj, f[c]);
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < KC; ++i) {
      const int c = tid + i * kPcLdsThr;
      if (c >= L.n) break;
      int x, y, z;
      coord(L, dx, dp, c, &x, &y, &z);
      double sr = 0.0, si = 0.0;
      auto add = [&](bool in, int q) {
        if (!in) return;
        sr += yd[q].x;
        si += yd[q].y;
      };
      add(x > 0, c - 1); add(x < L.nx - 1, c + 1);
      add(y > 0, c - L.nx); add(y < L.ny - 1, c + L.nx);
      add(z > 0, c - plane); add(z < L.nz - 1, c + plane);
      const double2 yc = yd[c];
      const double ar = sr * L.h2inv + (d[i].x * yc.x - d[i].y * yc.y);
      const double ai = si * L.h2inv + (d[i].x * yc.y + d[i].y * yc.x);
      res[c] = fd((double)f[c].x - ar, (double)f[c].y - ai);
    }
    __syncthreads();
    for (int c = tid; c < C.n; c += kPcLdsThr) {
      int cx, cy, cz;
      coord(C, cdx, cdp, c, &cx, &cy, &cz);
      double sr = 0.0, si = 0.0;
#pragma unroll
      for (int dz = 0; dz < 3; ++dz)
#pragma unroll
        for (int dy = 0; dy < 3; ++dy)
#pragma unroll
          for (int dx3 = 0; dx3 < 3; ++dx3) {
            if (2 * cz + dz >= L.nz || 2 * cy + dy >= L.ny || 2 * cx + dx3 >= L.nx) continue;
            const double wt = (dz != 1 ? 0.5 : 1.0) * (dy != 1 ? 0.5 : 1.0) * (dx3 != 1 ? 0.5 : 1.0);
            const float2 v = res[(2 * cz + dz) * plane + (2 * cy + dy) * L.nx + 2 * cx + dx3];
            sr += wt * v.x;
            si += wt * v.y;
          }
      fc[c] = fd(0.125 * sr, 0.125 * si);
    }
  }
  // coarsest level: kCoarseSweeps steps between y and a third array
  {
    const PcLevel& L = S.lev[last];
    const SmallDiv dx(L.nx), dp(L.nx * L.ny);
    float2 *f = base(last), *ya = f + L.n, *yb = reinterpret_cast<float2*>(yd);
    float2 w[KC];
    double2 d[KC];
    own(L, w, d);
    __syncthreads();   // the residual and w D^-1 f of the level before are no longer read
    for (int sweep = 0; sweep < kCoarseSweeps; ++sweep) {
      const float2* in = (sweep & 1) ? yb : ya;   // the last sweep ends in ya
      float2* out = (sweep & 1) ? ya : yb;
#pragma unroll
      for (int i = 0; i < KC; ++i) {
        const int c = tid + i * kPcLdsThr;
        if (c >= L.n) break;
        if (sweep == 0) {
          const double2 v = jac_w(w[i], conj, f[c]);
          out[c] = fd(v.x, v.y);
          continue;
        }
        int x, y, z;
        coord(L, dx, dp, c, &x, &y, &z);
        const double2 av = apply(L, in, c, x, y, z, d[i]);
        const double2 corr = jac_w(w[i], conj, fd((double)f[c].x - av.x, (double)f[c].y - av.y));
        out[c] = fd((double)in[c].x + corr.x, (double)in[c].y + corr.y);
      }
      __syncthreads();
    }
    static_assert(kCoarseSweeps % 2 == 0, "the coarsest result is in y");
    if constexpr (SINGLE) {
      float2* out = which ? S.z : S.q;
      double* red = reinterpret_cast<double*>(ya + L.n);   // a sum per 64 cells, as the waves of the per-cell passes have it
#pragma unroll
      for (int i = 0; i < KC; ++i) {
        const int c = tid + i * kPcLdsThr;
        if (c < L.n) out[c] = ya[c];
        double v = c < L.n ? nrm(ya[c]) : 0.0;
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
        if ((tid & 63) == 0) red[c >> 6] = v;
      }
      __syncthreads();
      static_assert(kPcLdsCells <= kParts * kThr && kParts <= kPcLdsThr, "");
      if (which && tid < kParts) {
        double tot = 0.0;
        if (tid * kThr < L.n)
          for (int i = 0; i < kThr / 64; ++i) tot += red[tid * (kThr / 64) + i];
        S.part[tid] = tot;
      }
      return;
    }
    if (last == lc) {
      for (int c = tid; c < L.n; c += kPcLdsThr) L.y[c] = ya[c];   // coarse_out() of the coarsest level
      return;
    }
  }
  for (int l = last - 1; l >= lc; --l) {
    const PcLevel& L = S.lev[l];
    const PcLevel& C = S.lev[l + 1];
    const SmallDiv dx(L.nx), dp(L.nx * L.ny);
    float2 *f = base(l), *yv = f + L.n;
    const float2* e = l + 1 == last ? base(l + 1) + C.n : base(l + 1);   // the coarsest result, or o over f
    float2 w[KC];
    double2 d[KC];
    own(L, w, d);
#pragma unroll
    for (int i = 0; i < KC; ++i) {
      const int c = tid + i * kPcLdsThr;
      if (c >= L.n) break;
      int x, y, z;
      coord(L, dx, dp, c, &x, &y, &z);
      double sr = 0.0, si = 0.0;
#pragma unroll
      for (int a = 0; a < 2; ++a) {
        const int iz = (z & 1) ? (a ? -1 : z >> 1) : (z >> 1) - 1 + a;
        if (iz < 0 || iz >= C.nz) continue;
#pragma unroll
        for (int b = 0; b < 2; ++b) {
          const int iy = (y & 1) ? (b ? -1 : y >> 1) : (y >> 1) - 1 + b;
          if (iy < 0 || iy >= C.ny) continue;
#pragma unroll
          for (int q = 0; q < 2; ++q) {
            const int ix = (x & 1) ? (q ? -1 : x >> 1) : (x >> 1) - 1 + q;
            if (ix < 0 || ix >= C.nx) continue;
            const float2 v = e[(iz * C.ny + iy) * C.nx + ix];
            sr += v.x;
            si += v.y;
          }
        }
      }
      const double wt = ((z & 1) ? 1.0 : 0.5) * ((y & 1) ? 1.0 : 0.5) * ((x & 1) ? 1.0 : 0.5);
      const double2 j = jac_w(w[i], conj, f[c]);
      yv[c] = fd(j.x + wt * sr, j.y + wt * si);
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < KC; ++i) {
      const int c = tid + i * kPcLdsThr;
      if (c >= L.n) break;
      int x, y, z;
      coord(L, dx, dp, c, &x, &y, &z);
      const double2 av = apply(L, yv, c, x, y, z, d[i]);
      const double2 corr = jac_w(w[i], conj, fd((double)f[c].x - av.x, (double)f[c].y - av.y));
      const float2 o = fd((double)yv[c].x + corr.x, (double)yv[c].y + corr.y);
      if (l == lc) L.o[c] = o;
      else f[c] = o;   // f of this cell is not needed again
    }
    __syncthreads();
  }
}

// ---------------------------------------------------------------------------
// grid set-up and results
// ---------------------------------------------------------------------------

// w D^-1 of A_beta on one level for one frequency: w / (-6/h^2 + omega^2 (1 - i beta) m - i omega b)
__global__ void __launch_bounds__(kThr) k_pc_wdinv(const float* __restrict__ m, const float* __restrict__ b, int n,
                                                   double h2inv, double omega, float2* __restrict__ out) {
  for (int c = blockIdx.x * kThr + threadIdx.x; c < n; c += gridDim.x * kThr) {
    const double mm = m[c], bb = b[c];
    const double dr = -6.0 * h2inv + omega * omega * mm;
    const double di = -kBeta * omega * omega * mm - omega * bb;
    const double den = dr * dr + di * di;
    out[c] = fd(kJac * dr / den, -kJac * di / den);
  }
}

// b_0 = the sponge of the grid (float32)
__global__ void __launch_bounds__(kThr) k_pc_sponge(float* __restrict__ b, int nx, int ny, int nz, int nb,
                                                    double sp_scale, double inv_nb) {
  const int n = nx * ny * nz, plane = nx * ny;
  for (int c = blockIdx.x * kThr + threadIdx.x; c < n; c += gridDim.x * kThr) {
    const int z = c / plane, rem = c - z * plane, y = rem / nx, x = rem - y * nx;
    b[c] = (float)(sp_scale * ((sponge_axis_d(x, nx, nb, inv_nb) + sponge_axis_d(y, ny, nb, inv_nb)) +
                               sponge_axis_d(z, nz, nb, inv_nb)));
  }
}

// coarse = P^T fine / P^T 1 (weighted mean over the 27 fine cells)
__global__ void __launch_bounds__(kThr) k_pc_restrict_mean(const float* __restrict__ fine, float* __restrict__ coarse,
                                                           int fnx, int fny, int fnz, int cnx, int cny, int cnz) {
  const int n = cnx * cny * cnz, plane = cnx * cny;
  for (int c = blockIdx.x * kThr + threadIdx.x; c < n; c += gridDim.x * kThr) {
    const int cz = c / plane, rem = c - cz * plane, cy = rem / cnx, cx = rem - cy * cnx;
    double s = 0.0, wsum = 0.0;
    for (int dz = -1; dz <= 1; ++dz) {
      const int fz = 2 * cz + 1 + dz;
      if (fz < 0 || fz >= fnz) continue;
      for (int dy = -1; dy <= 1; ++dy) {
        const int fy = 2 * cy + 1 + dy;
        if (fy < 0 || fy >= fny) continue;
        for (int dx = -1; dx <= 1; ++dx) {
          const int fx = 2 * cx + 1 + dx;
          if (fx < 0 || fx >= fnx) continue;
          const double w = (dz ? 0.5 : 1.0) * (dy ? 0.5 : 1.0) * (dx ? 0.5 : 1.0);
          s += w * fine[((size_t)fz * fny + fy) * fnx + fx];
          wsum += w;
        }
      }
    }
    coarse[c] = (float)(s / wsum);
  }
}

// partials of ||r1||^2 of the final residual (grid (kParts, systems of the group))
__global__ void __launch_bounds__(kThr) k_pc_rnorm(const PcSys* __restrict__ sy, const PcState* __restrict__ stv,
                                                   double* __restrict__ part, int g0) {
  __shared__ double red[kThr / 64];
  const int k = g0 + blockIdx.y;
  const PcSys& S = sy[k];
  const float2* __restrict__ r = pc_r(S, stv[k].iters);
  double acc = 0.0;
  for (int c = blockIdx.x * kThr + threadIdx.x; c < S.lev[0].n; c += kParts * kThr) acc += nrm(r[c]);
  const double tot = bsum(acc, red);
  if (threadIdx.x == 0) part[(size_t)k * kParts + blockIdx.x] = tot;
}

// J = ||r1||^2 + ||r2||^2 (recurred), alpha_ls = (A u)[src] in float64
// (one block per system; the sum over a whole residual in one block took 287 us
// on 64^3)
__global__ void __launch_bounds__(kThr) k_pc_final(const PcSys* __restrict__ sy, PcState* __restrict__ stv,
                                                   double* __restrict__ part, int g0) {
  __shared__ double red[kThr / 64];
  const int k = g0 + blockIdx.x;
  const PcSys& S = sy[k];
  PcState& T = stv[k];
  double acc = 0.0;
  for (int q = threadIdx.x; q < S.nr; q += kThr) acc += nrm(S.r2[q]);
  const double J = sum_parts(part + (size_t)k * kParts, kParts, red) + bsum(acc, red);
  if (threadIdx.x == 0) {
    T.J = J;
    if (S.est) {
      const double2 au = apply_cell(S, S.x, S.src, false);
      T.za = au;  // alpha_ls
    }
  }
}

// g = -sum over the grid's systems of 2 omega^2 Re(conj(u) r1); systems
// idx[0..cnt) in fixed order, the loads of four in flight
__global__ void __launch_bounds__(kThr) k_pc_grad(const PcSys* __restrict__ sy, const PcState* __restrict__ stv,
                                                  const int* __restrict__ idx, int cnt, int n, float* __restrict__ g) {
  for (int c = blockIdx.x * kThr + threadIdx.x; c < n; c += gridDim.x * kThr) {
    double acc = 0.0;
#pragma unroll 4
    for (int i = 0; i < cnt; ++i) {
      const PcSys& S = sy[idx[i]];
      const float2 u = S.x[c], r = pc_r(S, stv[idx[i]].iters)[c];
      acc -= 2.0 * S.omega2 * ((double)u.x * r.x + (double)u.y * r.y);
    }
    g[c] = (float)acc;
  }
}

// ---------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------

struct LevelDims {
  int nx, ny, nz;
  double h;
};

// levels: halve every axis (n -> n/2) while all axes have >= 4 cells and the
// level holds more than kCoarsestCells cells
std::vector<LevelDims> levels_of(const wri_grid& g) {
  std::vector<LevelDims> v;
  LevelDims d{g.nx, g.ny, g.nz, g.h};
  v.push_back(d);
  while (std::min({d.nx, d.ny, d.nz}) >= 4 && (int64_t)d.nx * d.ny * d.nz > kCoarsestCells &&
         (int)v.size() < kMaxLev) {
    d = LevelDims{d.nx / 2, d.ny / 2, d.nz / 2, 2.0 * d.h};
    v.push_back(d);
  }
  return v;
}

int64_t cells_of(const LevelDims& d) { return (int64_t)d.nx * d.ny * d.nz; }

struct PcLayout {
  size_t sys = 0, state = 0, parts = 0, idx = 0, head_bytes = 0, total = 0;
  std::vector<size_t> grid_arrays;   // per grid: m_l (l >= 1) and b_l (l >= 0)
  std::vector<std::pair<int, double>> pairs;   // distinct (grid, omega) of the systems
  std::vector<int> pair_of;                    // per system
  std::vector<size_t> pair_arrays;             // per pair: w D^-1 on every level
  std::vector<size_t> vec, rvec, rec;
};

// cells per thread of the tiled passes: two once a plane fills 64 tiles of 256 cells
int pc_cx(int64_t plane) { return plane >= 64 * 256 ? 2 : 1; }
struct PcTiles { int cx, x, n; };   // cells per thread, tiles per plane, tiles
PcTiles pc_tiles(const LevelDims& d) {
  const int64_t plane = (int64_t)d.nx * d.ny;
  const int cx = pc_cx(plane), b = 64 * kPcW * cx;
  const int x = (int)((plane + b - 1) / b);
  return {cx, x, x * ((d.nz + kPcZ - 1) / kPcZ)};
}
// the tiled passes: rows whose halo fits the LDS (96 KB), a level to coarsen to, and levels that one buffer
// resource covers
bool pc_tiled(const std::vector<LevelDims>& lv) {
  return lv.size() > 1 && lv[0].nx <= kPcMaxRow && cells_of(lv[0]) < (int64_t(1) << 28);
}

// first level of the one-workgroup cycle (the number of levels: none fits)
int pc_lds_level(const std::vector<LevelDims>& lv) {
  int lc = 1;
  while (lc < (int)lv.size() && cells_of(lv[lc]) > kPcLdsCells) ++lc;
  return lc;
}
// levels with a residual and a prolongation pass in memory
int pc_memory_levels(const std::vector<LevelDims>& lv) { return std::min(pc_lds_level(lv), (int)lv.size() - 1); }

PcLayout pc_layout(const wri_grid* grids, int n_grids, const wri_system* sys, int n_sys) {
  PcLayout L;
  size_t o = 0;
  auto take = [&](size_t b) { size_t r = o; o = al(o + std::max<size_t>(b, 1)); return r; };
  // the tables the host writes, in one piece
  L.rec.resize(n_sys);
  L.sys = take(sizeof(PcSys) * std::max(n_sys, 1));
  L.idx = take(sizeof(int) * std::max(n_sys, 1));
  for (int k = 0; k < n_sys; ++k) L.rec[k] = take(sizeof(int) * (size_t)sys[k].n_rec);
  L.head_bytes = o;
  L.state = take(sizeof(PcState) * std::max(n_sys, 1));
  L.parts = take(sizeof(double) * (size_t)kParts * std::max(n_sys, 1));
  L.grid_arrays.resize(n_grids);
  for (int g = 0; g < n_grids; ++g) {
    size_t b = 0;
    for (const auto& d : levels_of(grids[g])) b += 2 * al(sizeof(float) * (size_t)cells_of(d));
    L.grid_arrays[g] = take(b);
  }
  L.pair_of.assign(n_sys, -1);
  for (int k = 0; k < n_sys; ++k) {
    const std::pair<int, double> key(sys[k].grid, sys[k].omega);
    auto it = std::find(L.pairs.begin(), L.pairs.end(), key);
    L.pair_of[k] = (int)(it - L.pairs.begin());
    if (it == L.pairs.end()) L.pairs.push_back(key);
  }
  for (const auto& pr : L.pairs) {
    size_t b = 0;
    for (const auto& d : levels_of(grids[pr.first])) b += al(sizeof(float2) * (size_t)cells_of(d));
    L.pair_arrays.push_back(take(b));
  }
  L.vec.resize(n_sys);
  L.rvec.resize(n_sys);
  for (int k = 0; k < n_sys; ++k) {
    const wri_grid& g = grids[sys[k].grid];
    const auto lv = levels_of(g);
    size_t b = 9 * al(sizeof(float2) * (size_t)cells_of(lv[0]));   // x r p q t s z, res0 and y0 or the other r and p
    for (size_t l = 1; l < lv.size(); ++l) b += 4 * al(sizeof(float2) * (size_t)cells_of(lv[l]));
    L.vec[k] = take(b);
    L.rvec[k] = take(2 * al(sizeof(float2) * (size_t)sys[k].n_rec));
  }
  L.total = o + kAl;
  return L;
}

int blocks_for(int64_t n) { return (int)std::max<int64_t>(1, std::min<int64_t>((n + kThr - 1) / kThr, 1024)); }

int pc_run(const wri_grid* grids, int n_grids, const float* const* m, const wri_system* sys, int n_sys, int mode,
           int max_iter, int flags, double* J_out, float* const* grad, wri_c32* const* u_out, wri_result* res,
           void* ws, size_t ws_bytes, hipStream_t st) {
  int rc = wri_validate(grids, n_grids, sys, n_sys, mode, max_iter);
  if (rc != WRI_OK) return rc;
  if (n_sys > 0 && res == nullptr) return report_error(WRI_EINVAL, "res is NULL");
  if (flags & ~WRI_FLAG_NO_GRAPH)
    return report_error(WRI_EINVAL, "the preconditioned solver takes only WRI_FLAG_NO_GRAPH");
  if (n_grids > 0 && m == nullptr) return report_error(WRI_EINVAL, "m is NULL");
  for (int g = 0; g < n_grids; ++g)
    if (m[g] == nullptr || (grad != nullptr && grad[g] == nullptr))
      return report_error(WRI_EINVAL, "m[%d] or grad[%d] is NULL", g, g);
  const PcLayout L = pc_layout(grids, n_grids, sys, n_sys);
  if (ws == nullptr || ws_bytes < L.total)
    return report_error(WRI_ENOWS, "workspace of %zu bytes is smaller than the %zu required", ws_bytes, L.total);
  char* base = reinterpret_cast<char*>(al(reinterpret_cast<uintptr_t>(ws)));
  if (J_out) *J_out = 0.0;
  // per-grid level arrays: b_0 from the sponge, m_l and b_l restricted
  std::vector<std::vector<const float*>> gm(n_grids), gb(n_grids);
  for (int g = 0; g < n_grids; ++g) {
    const wri_grid& G = grids[g];
    const auto lv = levels_of(G);
    char* p = base + L.grid_arrays[g];
    std::vector<float*> mm(lv.size()), bb(lv.size());
    for (size_t l = 0; l < lv.size(); ++l) {
      const size_t nb = al(sizeof(float) * (size_t)cells_of(lv[l]));
      mm[l] = reinterpret_cast<float*>(p);
      bb[l] = reinterpret_cast<float*>(p + nb);
      p += 2 * nb;
    }
    double sp = 0.0, inb = 0.0;
    if (G.nb > 0) {
      const double d0 = 3.0 * G.v_ref * std::log(1000.0) / (2.0 * G.nb * G.h);
      sp = 2.0 * d0 / (G.v_ref * G.v_ref);
      inb = 1.0 / G.nb;
    }
    hipLaunchKernelGGL(k_pc_sponge, dim3(blocks_for(cells_of(lv[0]))), dim3(kThr), 0, st, bb[0], G.nx, G.ny, G.nz,
                       G.nb, sp, inb);
    PC_HIP(hipGetLastError());
    gm[g].assign(lv.size(), nullptr);
    gb[g].assign(lv.size(), nullptr);
    gm[g][0] = m[g];
    gb[g][0] = bb[0];
    for (size_t l = 1; l < lv.size(); ++l) {
      const float* fm = (l == 1) ? m[g] : mm[l - 1];
      hipLaunchKernelGGL(k_pc_restrict_mean, dim3(blocks_for(cells_of(lv[l]))), dim3(kThr), 0, st, fm, mm[l],
                         lv[l - 1].nx, lv[l - 1].ny, lv[l - 1].nz, lv[l].nx, lv[l].ny, lv[l].nz);
      hipLaunchKernelGGL(k_pc_restrict_mean, dim3(blocks_for(cells_of(lv[l]))), dim3(kThr), 0, st, bb[l - 1], bb[l],
                         lv[l - 1].nx, lv[l - 1].ny, lv[l - 1].nz, lv[l].nx, lv[l].ny, lv[l].nz);
      PC_HIP(hipGetLastError());
      gm[g][l] = mm[l];
      gb[g][l] = bb[l];
    }
  }
  // w D^-1 per distinct (grid, frequency) and level
  std::vector<std::vector<const float2*>> pw(L.pairs.size());
  for (size_t q = 0; q < L.pairs.size(); ++q) {
    const int g = L.pairs[q].first;
    const double om = L.pairs[q].second;
    const auto lv = levels_of(grids[g]);
    char* p = base + L.pair_arrays[q];
    for (size_t l = 0; l < lv.size(); ++l) {
      float2* w = reinterpret_cast<float2*>(p);
      const int64_t nl = cells_of(lv[l]);
      hipLaunchKernelGGL(k_pc_wdinv, dim3(blocks_for(nl)), dim3(kThr), 0, st, gm[g][l], gb[g][l], (int)nl,
                         1.0 / (lv[l].h * lv[l].h), om, w);
      PC_HIP(hipGetLastError());
      pw[q].push_back(w);
      p += al(sizeof(float2) * (size_t)nl);
    }
  }
  if (n_sys == 0) {
    if (grad != nullptr)
      for (int g = 0; g < n_grids; ++g) PC_HIP(launch_zero_f32(grad[g], (size_t)grids[g].nx * grids[g].ny * grids[g].nz, st));
    PC_HIP(hipStreamSynchronize(st));
    return WRI_OK;
  }
  // systems in grid order; groups of consecutive systems on one grid
  std::vector<int> order(n_sys);
  for (int k = 0; k < n_sys; ++k) order[k] = k;
  std::stable_sort(order.begin(), order.end(), [&](int a, int b) { return sys[a].grid < sys[b].grid; });
  struct Group { int grid, p0, cnt; int64_t n; };
  std::vector<Group> groups;
  std::vector<PcSys> hs(n_sys);
  std::vector<char> head(L.head_bytes, 0);   // image of the tables, one copy
  struct Drain { hipStream_t st; ~Drain() { (void)hipStreamSynchronize(st); } } drain{st};   // before head goes
  for (int p = 0; p < n_sys; ++p) {
    const int k = order[p];
    const wri_system& s = sys[k];
    const wri_grid& g = grids[s.grid];
    const auto lv = levels_of(g);
    const int64_t n = cells_of(lv[0]);
    if (groups.empty() || groups.back().grid != s.grid) groups.push_back({s.grid, p, 0, n});
    groups.back().cnt++;
    PcSys& S = hs[p];
    S = PcSys{};
    const size_t vb = al(sizeof(float2) * (size_t)n);
    char* v = base + L.vec[k];
    auto vec = [&](int i) { return reinterpret_cast<float2*>(v + i * vb); };
    S.x = (u_out != nullptr && u_out[k] != nullptr) ? reinterpret_cast<float2*>(u_out[k]) : vec(0);
    const bool tiled = pc_tiled(lv);
    S.tiled = tiled ? 1 : 0;
    S.nparts = tiled ? pc_tiles(lv[0]).n : kParts;
    // Tiled passes take the two vectors that they use for nothing else (the level-0
    // iterate and, as t is dead during a cycle and shares the residual, the residual)
    // for the other r and p: nine vectors either way.
    S.r[0] = vec(1); S.r[1] = tiled ? vec(7) : vec(1);
    S.p[0] = vec(2); S.p[1] = tiled ? vec(8) : vec(2);
    S.q = vec(3); S.t = vec(4); S.s = vec(5); S.z = vec(6);
    char* cv = v + 9 * vb;
    for (size_t l = 0; l < lv.size(); ++l) {
      PcLevel& Lv = S.lev[l];
      Lv.nx = lv[l].nx; Lv.ny = lv[l].ny; Lv.nz = lv[l].nz; Lv.n = (int)cells_of(lv[l]);
      Lv.h2inv = 1.0 / (lv[l].h * lv[l].h);
      Lv.m = gm[s.grid][l];
      Lv.b = gb[s.grid][l];
      Lv.wdinv = pw[L.pair_of[k]][l];
      if (l == 0) {
        Lv.f = nullptr; Lv.o = nullptr;
        Lv.res = tiled ? vec(4) : vec(7); Lv.y = tiled ? nullptr : vec(8);
      } else {
        const size_t cb = al(sizeof(float2) * (size_t)Lv.n);
        Lv.f = reinterpret_cast<float2*>(cv);
        Lv.y = reinterpret_cast<float2*>(cv + cb);
        Lv.o = reinterpret_cast<float2*>(cv + 2 * cb);
        Lv.res = reinterpret_cast<float2*>(cv + 3 * cb);
        cv += 4 * cb;
      }
    }
    if (lv.size() == 1) S.lev[0].o = vec(7);   // single-level cycle: Jacobi steps ping-pong between y and o
    // The tiles' partial sums are more than kParts on large grids: they lie in an array of
    // level 1 (at most a quarter of it) that no tiled pass touches, the iterate of a level
    // that goes through the residual and prolongation passes in memory, else the residual.
    S.part = !tiled ? reinterpret_cast<double*>(base + L.parts) + (size_t)p * kParts
                    : reinterpret_cast<double*>(pc_memory_levels(lv) > 1 ? S.lev[1].y : S.lev[1].res);
    S.nlev = (int)lv.size();
    const size_t rb = al(sizeof(float2) * (size_t)s.n_rec);
    S.r2 = reinterpret_cast<float2*>(base + L.rvec[k]);
    S.t2 = reinterpret_cast<float2*>(base + L.rvec[k] + rb);
    S.d = reinterpret_cast<const float2*>(s.d);
    int* drec = reinterpret_cast<int*>(base + L.rec[k]);
    if (s.n_rec > 0) std::memcpy(head.data() + L.rec[k], s.rec, sizeof(int) * s.n_rec);
    S.rec = drec;
    S.m = m[s.grid];
    S.nb = g.nb; S.nr = s.n_rec;
    S.est = mode == WRI_ESTIMATE;
    S.max_iter = max_iter;
    S.src = s.src;
    S.lam = s.lambda;
    S.rtol2 = s.rtol * s.rtol;
    S.omega = s.omega;
    S.omega2 = s.omega * s.omega;
    if (g.nb > 0) {
      const double d0 = 3.0 * g.v_ref * std::log(1000.0) / (2.0 * g.nb * g.h);
      S.sp_scale = 2.0 * d0 / (g.v_ref * g.v_ref);
      S.inv_nb = 1.0 / g.nb;
    }
    S.alpha = make_double2(s.alpha.re, s.alpha.im);
  }
  PcSys* dsys = reinterpret_cast<PcSys*>(base + L.sys);
  PcState* dst = reinterpret_cast<PcState*>(base + L.state);
  double* parts = reinterpret_cast<double*>(base + L.parts);
  int* didx = reinterpret_cast<int*>(base + L.idx);
  std::memcpy(head.data() + L.sys, hs.data(), sizeof(PcSys) * n_sys);
  for (int p = 0; p < n_sys; ++p) std::memcpy(head.data() + L.idx + sizeof(int) * p, &p, sizeof(int));
  PC_HIP(hipMemcpyAsync(base, head.data(), L.head_bytes, hipMemcpyHostToDevice, st));

  // tiled pass on level d: launch LAUNCH(template cx, grid, dynamic LDS of one element of `elem` bytes per cell)
  auto lds_of = [](const PcTiles& t, const LevelDims& d, size_t elem) {
    return (unsigned)(elem * kPcZ * (size_t)(64 * kPcW * t.cx + 2 * d.nx));
  };
#define PW_LAUNCH(K1, K2, D, ELEM, ...)                                                                     \
  do {                                                                                                      \
    const PcTiles t_ = pc_tiles(D);                                                                     \
    const dim3 g_((unsigned)(t_.n * G.cnt));                                                                \
    if (t_.cx == 1) hipLaunchKernelGGL(K1, g_, dim3(64 * kPcW), lds_of(t_, D, ELEM), st, dsys, dst, __VA_ARGS__, t_.x, t_.n); \
    else hipLaunchKernelGGL(K2, g_, dim3(64 * kPcW), lds_of(t_, D, ELEM), st, dsys, dst, __VA_ARGS__, t_.x, t_.n);            \
  } while (0)
  // one V-cycle (which = 0: q = M p with the p update, 1: z = M^H s with the partials of ||z||^2)
  auto vcycle = [&](const Group& G, int which) -> int {
    const int conj = which;
    const std::vector<LevelDims> lv = levels_of(grids[G.grid]);
    const int nl = (int)lv.size();
    auto sweeps = [&]() {
      for (int j = 0; j < kCoarseSweeps; ++j) {
        const int nbk = nl == 1 && j == kCoarseSweeps - 1 ? kParts : blocks_for(cells_of(lv[nl - 1]));
        hipLaunchKernelGGL(k_pc_vcoarse, dim3(nbk, G.cnt), dim3(kThr), 0, st, dsys, dst, G.p0, which, conj, j);
      }
    };
    if (pc_tiled(lv)) {
      // levels of one workgroup: from lc on (nl: none fits, the coarsest by separate sweeps)
      const int lc = pc_lds_level(lv), lm = pc_memory_levels(lv);
      for (int l = 0; l < lm; ++l) {
        if (l == 0 && which == 0)
          PW_LAUNCH((k_pw_down<1, true>), (k_pw_down<2, true>), lv[l], sizeof(double2), G.p0, l, which, conj);
        else
          PW_LAUNCH((k_pw_down<1, false>), (k_pw_down<2, false>), lv[l], sizeof(double2), G.p0, l, which, conj);
        const int rt = (int)((cells_of(lv[l + 1]) + kThr - 1) / kThr);
        hipLaunchKernelGGL(k_pw_restrict, dim3((unsigned)(rt * G.cnt)), dim3(kThr), 0, st, dsys, dst, G.p0, l, rt);
      }
      if (lc < nl) {
        size_t lds = sizeof(double2) * (size_t)cells_of(lv[lc]);
        for (int l = lc; l < nl; ++l) lds += 2 * sizeof(float2) * (size_t)cells_of(lv[l]);
        hipLaunchKernelGGL(k_pw_coarse<false>, dim3(G.cnt), dim3(kPcLdsThr), (unsigned)lds, st, dsys, dst, G.p0, lc, which, conj);
      } else {
        sweeps();
      }
      for (int l = lm - 1; l >= 0; --l)
        PW_LAUNCH((k_pw_up<1>), (k_pw_up<2>), lv[l], sizeof(float2), G.p0, l, which, conj);
      PC_HIP(hipGetLastError());
      return WRI_OK;
    }
    if (which == 0 && nl > 1) hipLaunchKernelGGL(k_pc_pupd, dim3(kParts, G.cnt), dim3(kThr), 0, st, dsys, dst, G.p0);
    if (nl == 1 && cells_of(lv[0]) <= kPcLdsCells) {
      // w D^-1 f, f and y of the level, and the sums
      const size_t lds = (sizeof(double2) + 2 * sizeof(float2)) * (size_t)cells_of(lv[0]) + sizeof(double) * kPcLdsCells / 64;
      hipLaunchKernelGGL(k_pw_coarse<true>, dim3(G.cnt), dim3(kPcLdsThr), (unsigned)lds, st, dsys, dst, G.p0, 0, which,
                         conj);
      PC_HIP(hipGetLastError());
      return WRI_OK;
    }
    for (int l = 0; l + 1 < nl; ++l) {
      hipLaunchKernelGGL(k_pc_vdown, dim3(blocks_for(cells_of(lv[l])), G.cnt), dim3(kThr), 0, st, dsys, dst, G.p0,
                         l, which, conj);
      hipLaunchKernelGGL(k_pc_vrestrict, dim3(blocks_for(cells_of(lv[l + 1])), G.cnt), dim3(kThr), 0, st, dsys, dst,
                         G.p0, l);
    }
    sweeps();
    for (int l = nl - 2; l >= 0; --l) {
      const int nbk = (l == 0) ? kParts : blocks_for(cells_of(lv[l]));
      hipLaunchKernelGGL(k_pc_vprolong, dim3(blocks_for(cells_of(lv[l])), G.cnt), dim3(kThr), 0, st, dsys, dst,
                         G.p0, l, which, conj);
      hipLaunchKernelGGL(k_pc_vsmooth, dim3(nbk, G.cnt), dim3(kThr), 0, st, dsys, dst, G.p0, l, which, conj);
    }
    PC_HIP(hipGetLastError());
    return WRI_OK;
  };
  auto iteration = [&]() -> int {
    for (const Group& G : groups) {
      const dim3 pg(kParts, G.cnt);
      const std::vector<LevelDims> lv = levels_of(grids[G.grid]);
      const bool tiled = pc_tiled(lv);
      int e = vcycle(G, 0);
      if (e != WRI_OK) return e;
      if (tiled) PW_LAUNCH((k_pw_apply<1, false>), (k_pw_apply<2, false>), lv[0], sizeof(float2), G.p0, 0);
      else hipLaunchKernelGGL(k_pc_fwd, pg, dim3(kThr), 0, st, dsys, dst, G.p0);
      hipLaunchKernelGGL(k_pc_step, dim3(G.cnt), dim3(kThr), 0, st, dsys, dst, G.p0);
      if (tiled) {
        PW_LAUNCH((k_pw_apply<1, true>), (k_pw_apply<2, true>), lv[0], sizeof(float2), G.p0, 0);
      } else {
        hipLaunchKernelGGL(k_pc_rupd, pg, dim3(kThr), 0, st, dsys, dst, G.p0);
        hipLaunchKernelGGL(k_pc_adj, pg, dim3(kThr), 0, st, dsys, dst, G.p0);
      }
      hipLaunchKernelGGL(k_pc_check, dim3(G.cnt), dim3(kThr), 0, st, dsys, dst, G.p0, 0);
      e = vcycle(G, 1);
      if (e != WRI_OK) return e;
      hipLaunchKernelGGL(k_pc_beta, dim3(G.cnt), dim3(kThr), 0, st, dsys, dst, G.p0, 0);
      PC_HIP(hipGetLastError());
    }
    return WRI_OK;
  };
  // set-up: x = 0, r = b, s_0 = S^H b, z_0 = M^H s_0, p_0 = z_0
  for (const Group& G : groups) {
    const dim3 pg(kParts, G.cnt);
    const std::vector<LevelDims> lv = levels_of(grids[G.grid]);
    hipLaunchKernelGGL(k_pc_zero, pg, dim3(kThr), 0, st, dsys, G.p0);
    hipLaunchKernelGGL(k_pc_init, dim3(G.cnt), dim3(kThr), 0, st, dsys, dst, G.p0);
    if (pc_tiled(lv)) PW_LAUNCH((k_pw_apply<1, true>), (k_pw_apply<2, true>), lv[0], sizeof(float2), G.p0, 1);
    else hipLaunchKernelGGL(k_pc_adj, pg, dim3(kThr), 0, st, dsys, dst, G.p0);
    hipLaunchKernelGGL(k_pc_check, dim3(G.cnt), dim3(kThr), 0, st, dsys, dst, G.p0, 1);
    rc = vcycle(G, 1);
    if (rc != WRI_OK) return rc;
    hipLaunchKernelGGL(k_pc_beta, dim3(G.cnt), dim3(kThr), 0, st, dsys, dst, G.p0, 1);
    PC_HIP(hipGetLastError());
  }
#undef PW_LAUNCH
  std::vector<PcState> hst(n_sys);
  auto read = [&]() -> int {
    PC_HIP(hipMemcpyAsync(hst.data(), dst, sizeof(PcState) * n_sys, hipMemcpyDeviceToHost, st));
    PC_HIP(hipStreamSynchronize(st));
    return WRI_OK;
  };
  // Eager launches: building a graph of a chunk cost more than a solve of a few
  // iterations (1.9 ms for 624 nodes), and on all but the smallest grids a pass takes
  // longer than the host needs to enqueue the next.  Every system has stopped after
  // max_iter iterations, so the statuses are looked at between chunks only.
  for (int64_t done = 0; done < max_iter;) {
    const int chunk = (int)std::min<int64_t>(kCheck, max_iter - done);
    for (int i = 0; i < chunk; ++i)
      if ((rc = iteration()) != WRI_OK) return rc;
    done += chunk;
    if (done >= max_iter) break;
    if ((rc = read()) != WRI_OK) return rc;
    bool any = false;
    for (const auto& T : hst) any = any || (T.status == kActive);
    if (!any) break;
  }
  // results: J, alpha_ls, gradient per grid
  for (const Group& G : groups) {
    hipLaunchKernelGGL(k_pc_rnorm, dim3(kParts, G.cnt), dim3(kThr), 0, st, dsys, dst, parts, G.p0);
    hipLaunchKernelGGL(k_pc_final, dim3(G.cnt), dim3(kThr), 0, st, dsys, dst, parts, G.p0);
  }
  PC_HIP(hipGetLastError());
  if (grad != nullptr) {
    for (int g = 0; g < n_grids; ++g) {
      const Group* G = nullptr;
      for (const auto& gg : groups)
        if (gg.grid == g) G = &gg;
      const int64_t n = (int64_t)grids[g].nx * grids[g].ny * grids[g].nz;
      if (G == nullptr) {
        PC_HIP(launch_zero_f32(grad[g], (size_t)n, st));
        continue;
      }
      hipLaunchKernelGGL(k_pc_grad, dim3(blocks_for(n)), dim3(kThr), 0, st, dsys, dst, didx + G->p0, G->cnt, (int)n,
                         grad[g]);
      PC_HIP(hipGetLastError());
    }
  }
  if ((rc = read()) != WRI_OK) return rc;
  for (const auto& T : hst)
    if (T.status == kActive) return report_error(WRI_EHIP, "internal: systems still active after max_iter iterations");
  int ret = WRI_OK;
  double J = 0.0;
  for (int p = 0; p < n_sys; ++p) {
    const int k = order[p];
    const PcState& T = hst[p];
    wri_result& r = res[k];
    r.iters = T.iters;
    r.status = T.status;
    r.relres = (T.ss0 > 0.0) ? std::sqrt(std::max(T.ss, 0.0) / T.ss0) : 0.0;
    r.J = T.J;
    if (mode == WRI_ESTIMATE) {
      r.alpha.re = T.xa.x; r.alpha.im = T.xa.y;
      r.alpha_ls.re = T.za.x; r.alpha_ls.im = T.za.y;
    } else {
      r.alpha = sys[k].alpha;
      r.alpha_ls = sys[k].alpha;
    }
    J += T.J;
    if (T.status == kBreakdown) ret = WRI_EBREAKDOWN;
    else if ((T.status == kMaxIter || T.status == kDiverged) && ret == WRI_OK) ret = WRI_NOT_CONVERGED;
  }
  if (J_out) *J_out = J;
  if (ret == WRI_EBREAKDOWN) report_error(WRI_EBREAKDOWN, "at least one system broke down");
  return ret;
}

}  // namespace
}  // namespace wri

using namespace wri;

extern "C" {

size_t wri_precond_workspace_bytes(const wri_grid* grids, int32_t n_grids, const wri_system* sys, int32_t n_sys,
                                   int32_t mode) {
  if (wri_validate(grids, n_grids, sys, n_sys, mode, 0) != WRI_OK) return 0;
  return pc_layout(grids, n_grids, sys, n_sys).total;
}

int wri_objective_grad_precond(const wri_grid* grids, int32_t n_grids, const float* const* m, const wri_system* sys,
                               int32_t n_sys, int32_t mode, int32_t max_iter, int32_t flags, double* J_out,
                               float* const* grad, wri_c32* const* u_out, wri_result* res, void* ws, size_t ws_bytes,
                               void* stream) {
  try {
    return pc_run(grids, n_grids, m, sys, n_sys, mode, max_iter, flags, J_out, grad, u_out, res, ws, ws_bytes,
                  reinterpret_cast<hipStream_t>(stream));
  } catch (const std::exception& e) {
    return report_error(WRI_EINVAL, "exception: %s", e.what());
  }
}

}  // extern "C"
