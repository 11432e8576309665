// Sources and receivers off the grid nodes: the source vector e and the
// receiver sampling P of eqs. ObjPen / SimpObj become trilinear interpolation
// weights over up to 8 cells each, and the same CGLS (the reading of
// Algorithm 1 used throughout the library) runs for all systems of a call in
// lockstep, four launches per iteration: a forward pass (p update and
// t = A p at each cell from its neighbours' recomputed p), a one-block-per-
// system pass for the source column, P p and the step a, an adjoint pass
// (r update, s = A^H r, x update) and a one-block-per-system pass for P^H r2,
// the source row and beta.  The stencil arithmetic is the fused kernels'
// (stencil.hpp); step scalars live in device memory and the host checks the
// statuses between chunks of iterations.
//
// P p: one thread per receiver sums its weighted cells (reads only).  P^H r2:
// a gather over the distinct receiver cells of a system (each cell's list of
// (receiver, weight) pairs is built on the host), so cells shared by several
// receivers need no atomics.  Source cells are distinct by construction.
// Every reduction runs in one fixed order.
#include "../../include/wri.h"
#include "wri_impl.hpp"
#include "stencil.hpp"
#include "window.hpp"

#include <algorithm>
#include <cmath>
#include <cstring>
#include <vector>

namespace wri {
namespace {

constexpr int kThreads = 256;
constexpr size_t kAl = 256;
size_t al(size_t v) { return (v + kAl - 1) / kAl * kAl; }

#define OG_HIP(expr)                                                                    \
  do {                                                                                  \
    hipError_t e_ = (expr);                                                             \
    if (e_ != hipSuccess) return report_error(WRI_EHIP, "%s: %s", #expr, hipGetErrorString(e_)); \
  } while (0)

int nblk(int64_t n) { return (int)std::max<int64_t>(1, std::min<int64_t>((n + kThreads - 1) / kThreads, 4096)); }

constexpr int kParts = 128;  // blocks (and partial sums) per system in the column passes and the norms
constexpr int kMaxCells = 8;  // cells of one point
constexpr int kCheck = 32;   // iterations between host checks of the statuses

// One system, resident in the workspace.  r and p are ping-pong pairs (the
// stencil passes read neighbours of the old vector while writing the new one).
struct OgSys {
  float2 *x, *r[2], *p[2], *s, *t, *r2, *t2;
  const float2* d;
  const int* scell; const double* sw;
  const int* rptr; const int* rcell; const double* rw;
  const int* uptr; const int* ucell; const int* uq; const double* uw;
  const float* m;
  int n, ns, nr, nu;
  int est, max_iter, nx, ny, nz, nb;
  int part0, nparts;   // first partial sum of the system, and partial sums of a stencil pass
  double c, lam, rtol2, omega, omega2, h2inv, sp_scale, inv_nb;
  double2 alpha;  // KNOWN-mode weight
};

// Mutable scalars of one system (float64).  iters = k while iteration k runs:
// p_k is in p[k & 1], r_k in r[k & 1].
struct OgState {
  double gamma, gamma0, a, beta, J;
  double2 xa, pa, sa, eau;
  int status, iters, pad_[2];
};

__device__ __forceinline__ double bsum(double v, double* red) {  // all threads get the block total
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
  __syncthreads();
  double r = 0.0;
#pragma unroll
  for (int i = 0; i < kThreads / 64; ++i) r += red[i];
  __syncthreads();
  return r;
}

__device__ __forceinline__ float2 f2d(double a, double b) { return make_float2((float)a, (float)b); }
__device__ __forceinline__ double nrm(float2 v) { return (double)v.x * v.x + (double)v.y * v.y; }
// y + a x in float64, rounded once: the value every neighbour recomputes identically
__device__ __forceinline__ float2 axpyd(float2 y, double a, float2 x) {
  return f2d((double)y.x + a * (double)x.x, (double)y.y + a * (double)x.y);
}

__device__ __forceinline__ double sponge_at(const OgSys& S, int x, int y, int z) {
  return S.sp_scale * ((sponge_axis_d(x, S.nx, S.nb, S.inv_nb) + sponge_axis_d(y, S.ny, S.nb, S.inv_nb)) +
                       sponge_axis_d(z, S.nz, S.nb, S.inv_nb));
}

// x = 0, r_0 = 0, p_{-1} = 0 (grid (blocks, nsys))
__global__ void __launch_bounds__(kThreads) k_og_zero(const OgSys* __restrict__ sy) {
  const OgSys& S = sy[blockIdx.y];
  const float2 z = make_float2(0.f, 0.f);
  for (int c = blockIdx.x * kThreads + threadIdx.x; c < S.n; c += gridDim.x * kThreads) {
    S.x[c] = z;
    S.r[0][c] = z;
    S.p[1][c] = z;
  }
}

// r_0[src] = alpha e (KNOWN), r2 = lam d, state reset (grid nsys)
__global__ void __launch_bounds__(kThreads) k_og_init(const OgSys* __restrict__ sy, OgState* __restrict__ stv) {
  const OgSys& S = sy[blockIdx.x];
  if (!S.est && (int)threadIdx.x < S.ns) {
    const double w = S.sw[threadIdx.x];
    S.r[0][S.scell[threadIdx.x]] = f2d(S.alpha.x * w, S.alpha.y * w);
  }
  for (int q = threadIdx.x; q < S.nr; q += kThreads)
    S.r2[q] = f2d(S.lam * (double)S.d[q].x, S.lam * (double)S.d[q].y);
  if (threadIdx.x == 0) {
    OgState& T = stv[blockIdx.x];
    T = OgState{};
    T.status = kActive;
  }
}

// Work items of the stencil passes: a 64 x 4 tile of (x, y) columns (one
// thread each) and a chunk of planes marched in z (up to 16, and so few that there
// are items for kParts blocks).  Each plane of the
// recomputed vector (p_k or r_{k+1}) is staged with a one-cell halo in LDS for
// the x/y neighbours; the z-neighbours stay in registers.  Every block runs
// the same number of items and planes (the barriers are uniform); threads
// outside the grid hold zeros.
constexpr int kZc = 16;
constexpr int kTy = kThreads / 64;               // tile rows
constexpr int kHalo = 2 * (64 + 2) + 2 * kTy;    // halo cells of one tile plane

struct TileWork {
  int x, y, z0, z1, col;
  bool in;
};

__device__ __forceinline__ int chunk_planes(const OgSys& S) { return max(1, min(kZc, S.n / (kParts * kThreads))); }

__device__ __forceinline__ int tile_items(const OgSys& S) {
  const int zc = chunk_planes(S);
  return ((S.nx + 63) / 64) * ((S.ny + kTy - 1) / kTy) * ((S.nz + zc - 1) / zc);
}

__device__ __forceinline__ TileWork tile_work(const OgSys& S, int w) {
  const int tx_n = (S.nx + 63) / 64, ty_n = (S.ny + kTy - 1) / kTy;
  const int t = w % (tx_n * ty_n), chunk = w / (tx_n * ty_n), planes = chunk_planes(S);
  TileWork W;
  W.x = (t % tx_n) * 64 + (threadIdx.x & 63);
  W.y = (t / tx_n) * kTy + (threadIdx.x >> 6);
  W.z0 = chunk * planes;
  W.z1 = min(W.z0 + planes, S.nz);
  W.in = W.x < S.nx && W.y < S.ny;
  W.col = W.y * S.nx + W.x;
  return W;
}

// halo cell h of the tile containing (x0, y0) (its corner cell): LDS slot and grid cell
__device__ __forceinline__ void halo_cell(int h, int x0, int y0, int* hx, int* hy, int* gx, int* gy) {
  if (h < 66) { *hy = 0; *hx = h; }
  else if (h < 132) { *hy = kTy + 1; *hx = h - 66; }
  else { const int q = h - 132; *hy = 1 + (q >> 1); *hx = (q & 1) ? 65 : 0; }
  *gx = x0 + *hx - 1;
  *gy = y0 + *hy - 1;
}

// Forward pass of iteration k: p_k = s_k + beta p_{k-1} (computed at the cell
// and its neighbours), t = A p_k, per-block partials of ||t||^2 (the
// source-column term is added by k_og_alpha).  grid (kParts, systems from s0 on).
__global__ void __launch_bounds__(kThreads) k_og_fwd(const OgSys* __restrict__ sy, const OgState* __restrict__ stv,
                                                     double* __restrict__ parts, int s0) {
  __shared__ double red[kThreads / 64];
  __shared__ float2 pl[kTy + 2][66];
  const OgSys& S = sy[s0 + blockIdx.y];
  const OgState& T = stv[s0 + blockIdx.y];
  double acc = 0.0;
  if (T.status == kActive) {  // uniform over the block
    const int k = T.iters;
    const float2* __restrict__ sv = S.s;
    const float2* __restrict__ po = S.p[(k + 1) & 1];
    float2* __restrict__ pn = S.p[k & 1];
    const double beta = T.beta;
    const int nx = S.nx, ny = S.ny, nz = S.nz, plane = nx * ny;
    const float2 zero = make_float2(0.f, 0.f);
    const int lx = threadIdx.x & 63, ly = threadIdx.x >> 6;
    auto P = [&](int c) { return axpyd(sv[c], beta, po[c]); };
    const int items = tile_items(S);
    for (int w = blockIdx.x; w < items; w += kParts) {
      const TileWork W = tile_work(S, w);
      int hx = 0, hy = 0, gx = -1, gy = -1;
      if ((int)threadIdx.x < kHalo) halo_cell(threadIdx.x, W.x - lx, W.y - ly, &hx, &hy, &gx, &gy);
      const bool hin = (int)threadIdx.x < kHalo && gx >= 0 && gx < nx && gy >= 0 && gy < ny;
      const double sxy = W.in ? sponge_axis_d(W.x, nx, S.nb, S.inv_nb) + sponge_axis_d(W.y, ny, S.nb, S.inv_nb) : 0.0;
      float2 vm = (W.in && W.z0 > 0) ? P((W.z0 - 1) * plane + W.col) : zero;
      float2 vc = W.in ? P(W.z0 * plane + W.col) : zero;
      for (int z = W.z0; z < W.z1; ++z) {
        pl[ly + 1][lx + 1] = vc;
        if ((int)threadIdx.x < kHalo) pl[hy][hx] = hin ? P(z * plane + gy * nx + gx) : zero;
        __syncthreads();
        const int c = z * plane + W.col;
        const float2 vp = (W.in && z + 1 < nz) ? P(c + plane) : zero;
        if (W.in) {
          pn[c] = vc;
          const double b = S.sp_scale * (sxy + sponge_axis_d(z, nz, S.nb, S.inv_nb));
          const float2 tv = round2(helm(vc, pl[ly + 1][lx], pl[ly + 1][lx + 2], pl[ly][lx + 1], pl[ly + 2][lx + 1], vm,
                                        vp, S.h2inv, S.omega2 * (double)S.m[c], -(S.omega * b)));
          S.t[c] = tv;
          acc += nrm(tv);
        }
        __syncthreads();
        vm = vc;
        vc = vp;
      }
    }
  }
  acc = bsum(acc, red);
  if (threadIdx.x == 0) parts[S.part0 + blockIdx.x] = acc;
}

// delta = ||t||^2 with the source column (t[src] -= c p_a w) + ||t2||^2 with
// t2 = lam P p_k; a = gamma / delta; x_a += a p_a; r2 -= a t2  (grid nsys)
__global__ void __launch_bounds__(kThreads) k_og_alpha(const OgSys* __restrict__ sy, OgState* __restrict__ stv,
                                                       const double* __restrict__ parts) {
  __shared__ double red[kThreads / 64];
  const OgSys& S = sy[blockIdx.x];
  OgState& T = stv[blockIdx.x];
  if (T.status != kActive) return;  // uniform over the block
  const float2* __restrict__ pk = S.p[T.iters & 1];
  double v = 0.0;
  for (int i = threadIdx.x; i < S.nparts; i += kThreads) v += parts[S.part0 + i];
  if (S.est && (int)threadIdx.x < S.ns) {  // distinct source cells, one per thread
    const int c = S.scell[threadIdx.x];
    const double w = S.sw[threadIdx.x];
    const float2 t0 = S.t[c];
    const float2 t1 = f2d((double)t0.x - S.c * T.pa.x * w, (double)t0.y - S.c * T.pa.y * w);
    S.t[c] = t1;
    v += nrm(t1) - nrm(t0);
  }
  for (int q = threadIdx.x; q < S.nr; q += kThreads) {
    double re = 0.0, im = 0.0;
    const int b = S.rptr[q], e = S.rptr[q + 1];   // 1 to kMaxCells cells, all loaded at once
    float2 x[kMaxCells];
    double w[kMaxCells];
#pragma unroll
    for (int j = 0; j < kMaxCells; ++j) {
      x[j] = pk[S.rcell[min(b + j, e - 1)]];
      w[j] = S.rw[min(b + j, e - 1)];
    }
#pragma unroll
    for (int j = 0; j < kMaxCells; ++j)
      if (b + j < e) {
        re += w[j] * (double)x[j].x;
        im += w[j] * (double)x[j].y;
      }
    const float2 t2 = f2d(S.lam * re, S.lam * im);
    S.t2[q] = t2;
    v += nrm(t2);
  }
  const double delta = bsum(v, red);
  const double gamma = T.gamma;
  const bool bad = !(delta > 0.0) || !isfinite(delta) || !isfinite(gamma);
  const double a = bad ? 0.0 : gamma / delta;
  if (!bad)
    for (int q = threadIdx.x; q < S.nr; q += kThreads) S.r2[q] = axpyd(S.r2[q], -a, S.t2[q]);
  __syncthreads();
  if (threadIdx.x == 0) {
    if (bad) {
      T.status = kBreakdown;
    } else {
      T.a = a;
      T.xa = make_double2(T.xa.x + a * T.pa.x, T.xa.y + a * T.pa.y);
    }
  }
}

// Adjoint pass: r_{k+1} = r_k - a t (at the cell and its neighbours),
// s = A^H r_{k+1}, x += a p_k, per-block partials of ||s||^2 (the receiver
// rows are added by k_og_beta).  setup = 1: the pass on r_0 with no update
// (s_0 = A^H r_0, copied r_0 into r_1).  Same tiles as k_og_fwd.
// grid (kParts, systems from s0 on).
__global__ void __launch_bounds__(kThreads) k_og_adj(const OgSys* __restrict__ sy, const OgState* __restrict__ stv,
                                                     double* __restrict__ parts, int s0, int setup) {
  __shared__ double red[kThreads / 64];
  __shared__ float2 pl[kTy + 2][66];
  const OgSys& S = sy[s0 + blockIdx.y];
  const OgState& T = stv[s0 + blockIdx.y];
  double acc = 0.0;
  if (setup || T.status == kActive) {  // uniform over the block
    const int k = setup ? 0 : T.iters;
    const double a = setup ? 0.0 : T.a;
    const float2* __restrict__ ro = S.r[k & 1];
    float2* __restrict__ rn = S.r[(k + 1) & 1];
    const float2* __restrict__ tv = S.t;
    const float2* __restrict__ pk = S.p[k & 1];
    const int nx = S.nx, ny = S.ny, nz = S.nz, plane = nx * ny;
    const float2 zero = make_float2(0.f, 0.f);
    const int lx = threadIdx.x & 63, ly = threadIdx.x >> 6;
    auto R = [&](int c) { return setup ? ro[c] : axpyd(ro[c], -a, tv[c]); };
    const int items = tile_items(S);
    for (int w = blockIdx.x; w < items; w += kParts) {
      const TileWork W = tile_work(S, w);
      int hx = 0, hy = 0, gx = -1, gy = -1;
      if ((int)threadIdx.x < kHalo) halo_cell(threadIdx.x, W.x - lx, W.y - ly, &hx, &hy, &gx, &gy);
      const bool hin = (int)threadIdx.x < kHalo && gx >= 0 && gx < nx && gy >= 0 && gy < ny;
      const double sxy = W.in ? sponge_axis_d(W.x, nx, S.nb, S.inv_nb) + sponge_axis_d(W.y, ny, S.nb, S.inv_nb) : 0.0;
      float2 vm = (W.in && W.z0 > 0) ? R((W.z0 - 1) * plane + W.col) : zero;
      float2 vc = W.in ? R(W.z0 * plane + W.col) : zero;
      for (int z = W.z0; z < W.z1; ++z) {
        pl[ly + 1][lx + 1] = vc;
        if ((int)threadIdx.x < kHalo) pl[hy][hx] = hin ? R(z * plane + gy * nx + gx) : zero;
        __syncthreads();
        const int c = z * plane + W.col;
        const float2 vp = (W.in && z + 1 < nz) ? R(c + plane) : zero;
        if (W.in) {
          rn[c] = vc;
          const double b = S.sp_scale * (sxy + sponge_axis_d(z, nz, S.nb, S.inv_nb));
          const float2 sv = round2(helm(vc, pl[ly + 1][lx], pl[ly + 1][lx + 2], pl[ly][lx + 1], pl[ly + 2][lx + 1], vm,
                                        vp, S.h2inv, S.omega2 * (double)S.m[c], S.omega * b));
          S.s[c] = sv;
          acc += nrm(sv);
          if (!setup) S.x[c] = axpyd(S.x[c], a, pk[c]);
        }
        __syncthreads();
        vm = vc;
        vc = vp;
      }
    }
  }
  acc = bsum(acc, red);
  if (threadIdx.x == 0) parts[S.part0 + blockIdx.x] = acc;
}

// ---------------------------------------------------------------------------
// The stencil passes by window tiles (window.hpp): a workgroup owns consecutive
// cells of the x-y plane and kOwZ planes, all its loads are issued at once and the
// x/y neighbours come from LDS.  The march above gives a workgroup one tile of 64 x 4
// columns and a load latency and two barriers per plane: what bounded it on batches
// that fit the caches.  Every stored value is rounded where it was; only the order of
// the float64 sums differs.  Per iteration (four launches): 8 systems of 64^3 78 us before
// and 45 now, 2 of 24x20x18 35 and 19, 48 of 128^3 2.07 ms and 1.75 (88 bytes a cell at
// 5.1 TB/s: memory).
// ---------------------------------------------------------------------------
constexpr int kOwW = 4, kOwZ = 4;
constexpr int kOwMaxRow = 512;   // wider rows (and planes past one resource) take the march: LDS 48 KB

// The systems of one grid in a launch; the first kOwGroups of them ride in its arguments.
constexpr int kOwGroups = 4;
struct OwGroup {
  int rhs0, ntiles, block0;
};
struct OwGroups {
  int n, xchunk;
  const OwGroup* table;   // when there are more
  OwGroup g[kOwGroups];
};

// (system, tile) of a block: neighbouring tiles of a system on one XCD
__device__ __forceinline__ int ow_block(const OwGroups& G, int* sys) {
  const int logical = xcd_remap(blockIdx.x, gridDim.x, G.xchunk);
  const OwGroup d = group_of(G.g, G.table, G.n, logical);
  const int local = logical - d.block0, q = local / d.ntiles;
  *sys = d.rhs0 + q;
  return local - q * d.ntiles;
}

template <int CX>
__global__ void __launch_bounds__(64 * kOwW)
k_ow_fwd(const OgSys* __restrict__ sy, const OgState* __restrict__ stv, double* __restrict__ parts, OwGroups G) {
  using Tile = Win<kOwW, CX, kOwZ>;
  constexpr int NT = Tile::NT;
  __shared__ double red[kThreads / 64];
  extern __shared__ float2 ow_f[];   // [kOwZ][B + 2 nx]: p
  const int tid = threadIdx.x;
  int sys;
  const int tile = ow_block(G, &sys);
  const OgSys& S = sy[sys];
  const OgState& T = stv[sys];
  if (T.status != kActive) return;
  Tile Q;
  Q.setup(S.nx, S.ny, S.nz, tile, (S.nx * S.ny + Tile::B - 1) / Tile::B);
  const int nx = Q.nx, wl = Q.wl, k = T.iters;
  const float2* po = S.p[(k + 1) & 1];
  float2* pn = S.p[k & 1];
  float2 v[CX][kOwZ + 2], pv[CX][kOwZ + 2];
  float mm[CX][kOwZ];
#pragma unroll
  for (int j = 0; j < CX; ++j)
#pragma unroll
    for (int i = 0; i < kOwZ + 2; ++i) {
      v[j][i] = Q.load2(S.s, i, Q.own2(j));
      pv[j][i] = Q.load2(po, i, Q.own2(j));
    }
#pragma unroll
  for (int j = 0; j < CX; ++j)
#pragma unroll
    for (int i = 0; i < kOwZ; ++i) mm[j][i] = Q.load1(S.m, i + 1, Q.own1(j));
  issue_point();
  const double beta = T.beta;
  for (int h = tid; h < 2 * nx; h += NT) {
    const unsigned o = Q.halo_off(h);
    const int sl = Q.halo_slot(h);
    float2 hs[kOwZ], hp[kOwZ];
#pragma unroll
    for (int i = 0; i < kOwZ; ++i) {
      hs[i] = Q.load2(S.s, i + 1, o);
      hp[i] = Q.load2(po, i + 1, o);
    }
#pragma unroll
    for (int i = 0; i < kOwZ; ++i) ow_f[i * wl + sl] = axpyd(hs[i], beta, hp[i]);
  }
#pragma unroll
  for (int j = 0; j < CX; ++j)
#pragma unroll
    for (int i = 0; i < kOwZ + 2; ++i) {
      v[j][i] = axpyd(v[j][i], beta, pv[j][i]);
      if (i >= 1 && i <= kOwZ) ow_f[(i - 1) * wl + nx + j * NT + tid] = v[j][i];
    }
  __syncthreads();
  double acc = 0.0;
#pragma unroll
  for (int j = 0; j < CX; ++j) {
    int cx, cy;
    Q.row_of(Q.cell[j], &cx, &cy);
    const unsigned mxm = row_mask(cx > 0), mxp = row_mask(cx < nx - 1);
    const double sxy = sponge_axis_d(cx, nx, S.nb, S.inv_nb) + sponge_axis_d(cy, Q.ny, S.nb, S.inv_nb);
#pragma unroll
    for (int i = 0; i < kOwZ; ++i) {
      const float2* row = ow_f + i * wl + nx + j * NT + tid;
      const float2 xm = masked(row[-1], mxm), xp = masked(row[1], mxp), ym = row[-nx], yp = row[nx];
      const double b = S.sp_scale * (sxy + sponge_axis_d(Q.z0 + i, Q.nz, S.nb, S.inv_nb));
      const float2 t = round2(helm(v[j][i + 1], xm, xp, ym, yp, v[j][i], v[j][i + 2], S.h2inv,
                                   S.omega2 * (double)mm[j][i], -(S.omega * b)));
      Q.store2(pn, i + 1, Q.own2(j), v[j][i + 1]);
      Q.store2(S.t, i + 1, Q.own2(j), t);
      if (Q.live(j, i)) acc += nrm(t);
    }
  }
  acc = bsum(acc, red);
  if (tid == 0) parts[S.part0 + tile] = acc;
}

// SETUP: s_0 = A^H r_0, no update
template <int CX, bool SETUP>
__global__ void __launch_bounds__(64 * kOwW)
k_ow_adj(const OgSys* __restrict__ sy, const OgState* __restrict__ stv, double* __restrict__ parts, OwGroups G) {
  using Tile = Win<kOwW, CX, kOwZ>;
  constexpr int NT = Tile::NT;
  __shared__ double red[kThreads / 64];
  extern __shared__ float2 ow_f[];   // [kOwZ][B + 2 nx]: r
  const int tid = threadIdx.x;
  int sys;
  const int tile = ow_block(G, &sys);
  const OgSys& S = sy[sys];
  const OgState& T = stv[sys];
  if (T.status != kActive) return;
  Tile Q;
  Q.setup(S.nx, S.ny, S.nz, tile, (S.nx * S.ny + Tile::B - 1) / Tile::B);
  const int nx = Q.nx, wl = Q.wl, k = T.iters;
  const float2* ro = S.r[k & 1];
  float2* rn = S.r[(k + 1) & 1];
  const float2* pk = S.p[k & 1];
  float2 v[CX][kOwZ + 2], tv[CX][kOwZ + 2], xv[CX][kOwZ], pv[CX][kOwZ];
  float mm[CX][kOwZ];
#pragma unroll
  for (int j = 0; j < CX; ++j)
#pragma unroll
    for (int i = 0; i < kOwZ + 2; ++i) {
      v[j][i] = Q.load2(ro, i, Q.own2(j));
      if constexpr (!SETUP) tv[j][i] = Q.load2(S.t, i, Q.own2(j));
    }
#pragma unroll
  for (int j = 0; j < CX; ++j)
#pragma unroll
    for (int i = 0; i < kOwZ; ++i) {
      mm[j][i] = Q.load1(S.m, i + 1, Q.own1(j));
      if constexpr (!SETUP) {
        xv[j][i] = Q.load2(S.x, i + 1, Q.own2(j));
        pv[j][i] = Q.load2(pk, i + 1, Q.own2(j));
      }
    }
  issue_point();
  const double a = SETUP ? 0.0 : T.a;
  for (int h = tid; h < 2 * nx; h += NT) {
    const unsigned o = Q.halo_off(h);
    const int sl = Q.halo_slot(h);
    float2 hr[kOwZ], ht[kOwZ];
#pragma unroll
    for (int i = 0; i < kOwZ; ++i) {
      hr[i] = Q.load2(ro, i + 1, o);
      if constexpr (!SETUP) ht[i] = Q.load2(S.t, i + 1, o);
    }
#pragma unroll
    for (int i = 0; i < kOwZ; ++i) {
      if constexpr (!SETUP) hr[i] = axpyd(hr[i], -a, ht[i]);
      ow_f[i * wl + sl] = hr[i];
    }
  }
#pragma unroll
  for (int j = 0; j < CX; ++j)
#pragma unroll
    for (int i = 0; i < kOwZ + 2; ++i) {
      if constexpr (!SETUP) v[j][i] = axpyd(v[j][i], -a, tv[j][i]);
      if (i >= 1 && i <= kOwZ) ow_f[(i - 1) * wl + nx + j * NT + tid] = v[j][i];
    }
  __syncthreads();
  double acc = 0.0;
#pragma unroll
  for (int j = 0; j < CX; ++j) {
    int cx, cy;
    Q.row_of(Q.cell[j], &cx, &cy);
    const unsigned mxm = row_mask(cx > 0), mxp = row_mask(cx < nx - 1);
    const double sxy = sponge_axis_d(cx, nx, S.nb, S.inv_nb) + sponge_axis_d(cy, Q.ny, S.nb, S.inv_nb);
#pragma unroll
    for (int i = 0; i < kOwZ; ++i) {
      const float2* row = ow_f + i * wl + nx + j * NT + tid;
      const float2 xm = masked(row[-1], mxm), xp = masked(row[1], mxp), ym = row[-nx], yp = row[nx];
      const double b = S.sp_scale * (sxy + sponge_axis_d(Q.z0 + i, Q.nz, S.nb, S.inv_nb));
      const float2 s = round2(helm(v[j][i + 1], xm, xp, ym, yp, v[j][i], v[j][i + 2], S.h2inv,
                                   S.omega2 * (double)mm[j][i], S.omega * b));
      Q.store2(S.s, i + 1, Q.own2(j), s);
      if (Q.live(j, i)) acc += nrm(s);
      if constexpr (!SETUP) {
        Q.store2(rn, i + 1, Q.own2(j), v[j][i + 1]);
        Q.store2(S.x, i + 1, Q.own2(j), axpyd(xv[j][i], a, pv[j][i]));
      }
    }
  }
  acc = bsum(acc, red);
  if (tid == 0) parts[S.part0 + tile] = acc;
}

// The receiver rows of S^H r (s += lam P^H r2 over the distinct receiver
// cells) and the source row s_a = -c e^H r, with gamma = ||s||^2 + |s_a|^2:
// shared by the set-up (gamma0) and every iteration (beta, statuses).
__device__ void og_finish_s(const OgSys& S, const float2* __restrict__ r, double pv, double* red, double2* src,
                            double* gs, double2* sa) {
  double v = pv;
  if (S.est && (int)threadIdx.x < S.ns) {
    const float2 x = r[S.scell[threadIdx.x]];
    const double w = S.c * S.sw[threadIdx.x];
    src[threadIdx.x] = make_double2(w * (double)x.x, w * (double)x.y);
  }
  for (int u = threadIdx.x; u < S.nu; u += kThreads) {
    double re = 0.0, im = 0.0;
    const int b = S.uptr[u], e = S.uptr[u + 1], c = S.ucell[u];
    const float2 s0 = S.s[c];
    for (int j = b; j < e; j += 4) {   // four pairs' loads at once
      float2 x[4];
      double w[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        x[i] = S.r2[S.uq[min(j + i, e - 1)]];
        w[i] = S.uw[min(j + i, e - 1)];
      }
#pragma unroll
      for (int i = 0; i < 4; ++i)
        if (j + i < e) {
          re += w[i] * (double)x[i].x;
          im += w[i] * (double)x[i].y;
        }
    }
    const float2 s1 = f2d((double)s0.x + S.lam * re, (double)s0.y + S.lam * im);
    S.s[c] = s1;
    v += nrm(s1) - nrm(s0);
  }
  v = bsum(v, red);
  double sr = 0.0, si = 0.0;
  if (S.est)
    for (int i = 0; i < S.ns; ++i) {
      sr -= src[i].x;
      si -= src[i].y;
    }
  *gs = v + sr * sr + si * si;
  *sa = make_double2(sr, si);
}

// gamma0 = ||S^H b||^2 after the set-up pass; p_a = s_a, beta = 0 (p_{-1} = 0)  (grid nsys)
__global__ void __launch_bounds__(kThreads) k_og_start(const OgSys* __restrict__ sy, OgState* __restrict__ stv,
                                                       const double* __restrict__ parts) {
  __shared__ double red[kThreads / 64];
  __shared__ double2 src[kMaxCells];
  const OgSys& S = sy[blockIdx.x];
  OgState& T = stv[blockIdx.x];
  double v = 0.0;
  for (int i = threadIdx.x; i < S.nparts; i += kThreads) v += parts[S.part0 + i];
  double g;
  double2 sa;
  og_finish_s(S, S.r[0], v, red, src, &g, &sa);
  if (threadIdx.x == 0) {
    T.gamma = T.gamma0 = g;
    T.sa = T.pa = sa;
    T.beta = 0.0;
    if (g == 0.0) T.status = kZeroRhs;
    else if (g <= S.rtol2 * g) T.status = kConverged;
    else if (S.max_iter <= 0) T.status = kMaxIter;
  }
}

// s_{k+1} completed, gamma' , beta, statuses, p_a; iteration k done  (grid nsys)
__global__ void __launch_bounds__(kThreads) k_og_beta(const OgSys* __restrict__ sy, OgState* __restrict__ stv,
                                                      const double* __restrict__ parts) {
  __shared__ double red[kThreads / 64];
  __shared__ double2 src[kMaxCells];
  const OgSys& S = sy[blockIdx.x];
  OgState& T = stv[blockIdx.x];
  if (T.status != kActive) return;  // uniform over the block
  double v = 0.0;
  for (int i = threadIdx.x; i < S.nparts; i += kThreads) v += parts[S.part0 + i];
  double gnew;
  double2 sa;
  og_finish_s(S, S.r[(T.iters + 1) & 1], v, red, src, &gnew, &sa);
  if (threadIdx.x == 0) {
    const double beta = gnew / T.gamma;
    T.beta = beta;
    T.gamma = gnew;
    T.sa = sa;
    T.pa = make_double2(sa.x + beta * T.pa.x, sa.y + beta * T.pa.y);
    T.iters += 1;
    if (gnew <= S.rtol2 * T.gamma0) T.status = kConverged;
    else if (!isfinite(gnew)) T.status = kBreakdown;
    else if (T.iters >= S.max_iter) T.status = kMaxIter;
  }
}

// per-system partials of ||r||^2 for the final residual r[iters & 1]  (grid (kParts, nsys))
__global__ void __launch_bounds__(kThreads) k_og_rnorm(const OgSys* __restrict__ sy, const OgState* __restrict__ stv,
                                                       double* __restrict__ parts) {
  __shared__ double red[kThreads / 64];
  const OgSys& S = sy[blockIdx.y];
  const float2* __restrict__ r = S.r[stv[blockIdx.y].iters & 1];
  double acc = 0.0;
  for (int c = blockIdx.x * kThreads + threadIdx.x; c < S.n; c += kParts * kThreads) acc += nrm(r[c]);
  acc = bsum(acc, red);
  if (threadIdx.x == 0) parts[S.part0 + blockIdx.x] = acc;
}

// J = ||r||^2 + ||r2||^2; e^H (A u) from A x at the source cells, each
// rounded to float32 as a stored t = A x would be  (grid nsys)
__global__ void __launch_bounds__(kThreads) k_og_final(const OgSys* __restrict__ sy, OgState* __restrict__ stv,
                                                       const double* __restrict__ parts) {
  __shared__ double red[kThreads / 64];
  __shared__ double2 ax[kMaxCells];
  const OgSys& S = sy[blockIdx.x];
  OgState& T = stv[blockIdx.x];
  double v = 0.0;
  if (S.est && (int)threadIdx.x < S.ns) {
    const int nx = S.nx, ny = S.ny, nz = S.nz, plane = nx * ny, c = S.scell[threadIdx.x];
    const int z = c / plane, rem = c - z * plane, y = rem / nx, x = rem - y * nx;
    const float2 zero = make_float2(0.f, 0.f);
    const float2* __restrict__ in = S.x;
    const float2 xm = x > 0 ? in[c - 1] : zero, xp = x < nx - 1 ? in[c + 1] : zero;
    const float2 ym = y > 0 ? in[c - nx] : zero, yp = y < ny - 1 ? in[c + nx] : zero;
    const float2 zm = z > 0 ? in[c - plane] : zero, zp = z < nz - 1 ? in[c + plane] : zero;
    const float2 t = round2(helm(in[c], xm, xp, ym, yp, zm, zp, S.h2inv, S.omega2 * (double)S.m[c],
                                 -(S.omega * sponge_at(S, x, y, z))));
    const double w = S.sw[threadIdx.x];
    ax[threadIdx.x] = make_double2(w * (double)t.x, w * (double)t.y);
  }
  for (int i = threadIdx.x; i < kParts; i += kThreads) v += parts[S.part0 + i];
  for (int q = threadIdx.x; q < S.nr; q += kThreads) v += nrm(S.r2[q]);
  v = bsum(v, red);
  if (threadIdx.x == 0) {
    T.J = v;
    double er = 0.0, ei = 0.0;
    if (S.est)
      for (int i = 0; i < S.ns; ++i) {
        er += ax[i].x;
        ei += ax[i].y;
      }
    T.eau = make_double2(er, ei);
  }
}

// g = -sum over the grid's systems of 2 omega^2 Re(conj(x) r)  (systems s0 to s0 + k)
__global__ void __launch_bounds__(kThreads) k_og_grad(const OgSys* __restrict__ sy, const OgState* __restrict__ stv,
                                                      int s0, int k, int n, float* __restrict__ g) {
  for (int c = blockIdx.x * kThreads + threadIdx.x; c < n; c += gridDim.x * kThreads) {
    double acc = 0.0;
    for (int i = s0; i < s0 + k; ++i) {
      if (stv[i].status == kBreakdown) continue;
      const OgSys& S = sy[i];
      const float2 a = S.x[c], b = S.r[stv[i].iters & 1][c];
      acc -= 2.0 * S.omega2 * ((double)a.x * b.x + (double)a.y * b.y);
    }
    g[c] = (float)acc;
  }
}

// ---- host-side tables ------------------------------------------------------

struct Point {
  int n = 0;
  int cells[kMaxCells];
  double w[kMaxCells];
};

// trilinear cells (ascending) and weights of point xyz [m] on grid g (zero weights
// dropped, so cells are distinct); the point is clamped into the grid
Point trilinear(const wri_grid& g, const double* xyz) {
  const int n[3] = {g.nx, g.ny, g.nz};
  int i0[3], i1[3];
  double w0[3], w1[3];
  for (int a = 0; a < 3; ++a) {
    if (n[a] == 1) {
      i0[a] = i1[a] = 0;
      w0[a] = 1.0;
      w1[a] = 0.0;
      continue;
    }
    double xi = xyz[a] / g.h;
    xi = xi < 0.0 ? 0.0 : (xi > n[a] - 1.0 ? n[a] - 1.0 : xi);
    int k = (int)std::floor(xi);
    if (k > n[a] - 2) k = n[a] - 2;
    i0[a] = k;
    i1[a] = k + 1;
    w1[a] = xi - k;
    w0[a] = 1.0 - w1[a];
  }
  Point p;
  for (int cz = 0; cz < 2; ++cz)
    for (int cy = 0; cy < 2; ++cy)
      for (int cx = 0; cx < 2; ++cx) {
        const int x = cx ? i1[0] : i0[0], y = cy ? i1[1] : i0[1], z = cz ? i1[2] : i0[2];
        const double w = (cx ? w1[0] : w0[0]) * (cy ? w1[1] : w0[1]) * (cz ? w1[2] : w0[2]);
        if (w == 0.0) continue;
        p.cells[p.n] = (z * g.ny + y) * g.nx + x;
        p.w[p.n++] = w;
      }
  return p;
}

// Receiver tables of one system: cells of receiver q, and the (receiver, weight)
// pairs of distinct cell u
struct RecTables {
  std::vector<int> rptr, rcell;      // receiver q: cells rcell[rptr[q] .. rptr[q+1])
  std::vector<double> rw;
  std::vector<int> uptr, ucell, uq;  // distinct cell u: pairs [uptr[u] .. uptr[u+1])
  std::vector<double> uw;
  size_t bytes() const {
    return al(sizeof(int) * rptr.size()) + al(sizeof(int) * rcell.size()) + al(sizeof(double) * rw.size()) +
           al(sizeof(int) * uptr.size()) + al(sizeof(int) * ucell.size()) + al(sizeof(int) * uq.size()) +
           al(sizeof(double) * uw.size());
  }
};

RecTables build_receivers(const wri_grid& g, const wri_positions& pos, int n_rec) {
  RecTables T;
  T.rptr.reserve(n_rec + 1);
  T.rcell.reserve((size_t)kMaxCells * n_rec);
  T.rw.reserve((size_t)kMaxCells * n_rec);
  std::vector<std::pair<int, int>> by_cell;   // (cell, entry): pairs of one cell in receiver order
  by_cell.reserve((size_t)kMaxCells * n_rec);
  std::vector<int> owner;
  owner.reserve((size_t)kMaxCells * n_rec);
  T.rptr.push_back(0);
  for (int q = 0; q < n_rec; ++q) {
    const Point r = trilinear(g, pos.rec + 3 * (size_t)q);
    for (int j = 0; j < r.n; ++j) {
      by_cell.push_back({r.cells[j], (int)T.rcell.size()});
      owner.push_back(q);
      T.rcell.push_back(r.cells[j]);
      T.rw.push_back(r.w[j]);
    }
    T.rptr.push_back((int)T.rcell.size());
  }
  std::sort(by_cell.begin(), by_cell.end());
  T.uptr.push_back(0);
  T.uq.reserve(by_cell.size());
  T.uw.reserve(by_cell.size());
  for (size_t i = 0; i < by_cell.size(); ++i) {
    if (i == 0 || by_cell[i].first != by_cell[i - 1].first) {
      if (i > 0) T.uptr.push_back((int)i);
      T.ucell.push_back(by_cell[i].first);
    }
    T.uq.push_back(owner[by_cell[i].second]);
    T.uw.push_back(T.rw[by_cell[i].second]);
  }
  if (!by_cell.empty()) T.uptr.push_back((int)by_cell.size());
  return T;
}

// Tables of a call.  Systems with the previous system's receivers share its tables.
struct SysTables {
  std::vector<Point> src;
  std::vector<int> set_of;
  std::vector<RecTables> sets;
  size_t bytes(int k) const {   // of system k's own copy
    return al(sizeof(int) * src[k].n) + al(sizeof(double) * src[k].n) + sets[set_of[k]].bytes();
  }
};

SysTables build_tables(const wri_grid* grids, const wri_system* sys, int n_sys, const wri_positions* pos) {
  SysTables T;
  for (int k = 0; k < n_sys; ++k) {
    const wri_grid& g = grids[sys[k].grid];
    T.src.push_back(trilinear(g, pos[k].src));
    const bool same = k > 0 && sys[k].grid == sys[k - 1].grid && sys[k].n_rec == sys[k - 1].n_rec &&
                      (sys[k].n_rec == 0 ||
                       std::memcmp(pos[k].rec, pos[k - 1].rec, sizeof(double) * 3 * (size_t)sys[k].n_rec) == 0);
    if (!same) T.sets.push_back(build_receivers(g, pos[k], sys[k].n_rec));
    T.set_of.push_back((int)T.sets.size() - 1);
  }
  return T;
}

int64_t ncell(const wri_grid& g) { return (int64_t)g.nx * g.ny * g.nz; }

// Cells per thread of a grid's window passes (two once a plane fills 64 tiles); 0: the
// column march.  By the grid alone: a system gives the same bits in any batch.
int ow_cx(const wri_grid& g) {
  if (g.nx > kOwMaxRow || ncell(g) >= (int64_t(1) << 28)) return 0;
  return g.nx * g.ny >= 64 * 256 ? 2 : 1;
}
int ow_tiles(const wri_grid& g, int cx) {
  const int b = 64 * kOwW * cx;
  return (g.nx * g.ny + b - 1) / b * ((g.nz + kOwZ - 1) / kOwZ);
}

// Systems sorted by passes and grid; the groups (systems of one grid) of each kind of passes.
struct OgPlan {
  std::vector<int> order;              // slot -> system
  std::vector<int> cx;                 // per slot
  std::vector<OwGroup> groups[3];      // by cx (0: rhs0 only)
  int blocks[3] = {0, 0, 0}, nx[3] = {1, 1, 1}, xchunk[3] = {16, 16, 16};
  size_t table_entries() const {       // of the groups that do not ride in the launch arguments
    size_t n = 0;
    for (int c = 1; c <= 2; ++c)
      if (groups[c].size() > (size_t)kOwGroups) n += groups[c].size();
    return n;
  }
};

// window = false: the column march for all, in less memory.
OgPlan og_plan(const wri_grid* grids, const wri_system* sys, int n_sys, bool window) {
  OgPlan P;
  auto cells_a_thread = [&](int k) { return window ? ow_cx(grids[sys[k].grid]) : 0; };
  P.order.resize(n_sys);
  for (int k = 0; k < n_sys; ++k) P.order[k] = k;
  std::stable_sort(P.order.begin(), P.order.end(), [&](int a, int b) {
    const int ga = sys[a].grid, gb = sys[b].grid, ca = cells_a_thread(a), cb = cells_a_thread(b);
    return ca != cb ? ca < cb : ga < gb;
  });
  for (int p = 0; p < n_sys; ++p) {
    const wri_grid& g = grids[sys[P.order[p]].grid];
    const int cx = cells_a_thread(P.order[p]);
    P.cx.push_back(cx);
    auto& v = P.groups[cx];
    if (v.empty() || sys[P.order[p - 1]].grid != sys[P.order[p]].grid)
      v.push_back({p, cx > 0 ? ow_tiles(g, cx) : kParts, P.blocks[cx]});
    P.blocks[cx] += v.back().ntiles;
    P.nx[cx] = std::max(P.nx[cx], (int)g.nx);
    P.xchunk[cx] = std::max(P.xchunk[cx], v.back().ntiles / 2);
  }
  return P;
}

struct OgLayout {
  std::vector<int> part0;         // per slot: first partial sum
  std::vector<size_t> vec, rvec;  // per system: 7 wavefield vectors (x unless u_out), r2 and t2
  size_t sys = 0, state = 0, parts = 0, groups = 0, tables = 0, total = 0;
};

int validate_offgrid(const wri_grid* grids, int n_grids, const wri_system* sys, int n_sys, const wri_positions* pos,
                     int mode, int max_iter) {
  if (n_grids < 0 || n_sys < 0) return report_error(WRI_EINVAL, "negative n_grids or n_sys");
  if (n_grids > 0 && grids == nullptr) return report_error(WRI_EINVAL, "grids is NULL");
  if (n_sys > 0 && (sys == nullptr || pos == nullptr)) return report_error(WRI_EINVAL, "sys or pos is NULL");
  if (mode != WRI_KNOWN && mode != WRI_ESTIMATE) return report_error(WRI_EINVAL, "bad mode %d", mode);
  if (max_iter < 0) return report_error(WRI_EINVAL, "max_iter < 0");
  for (int i = 0; i < n_grids; ++i) {
    const wri_grid& g = grids[i];
    if (g.nx < 1 || g.ny < 1 || g.nz < 1 || ncell(g) >= (int64_t(1) << 31))
      return report_error(WRI_EINVAL, "grid %d: bad size", i);
    if (!(g.h > 0.0) || !std::isfinite(g.h)) return report_error(WRI_EINVAL, "grid %d: h must be > 0", i);
    if (g.nb < 0 || (g.nb > 0 && !(g.v_ref > 0.0))) return report_error(WRI_EINVAL, "grid %d: bad sponge", i);
  }
  for (int k = 0; k < n_sys; ++k) {
    const wri_system& s = sys[k];
    if (s.grid < 0 || s.grid >= n_grids) return report_error(WRI_EINVAL, "system %d: grid index out of range", k);
    if (!(s.omega >= 0.0) || !std::isfinite(s.omega) || !(s.lambda >= 0.0) || !std::isfinite(s.lambda) ||
        !(s.rtol >= 0.0) || !std::isfinite(s.rtol))
      return report_error(WRI_EINVAL, "system %d: omega, lambda and rtol must be finite and >= 0", k);
    if (s.n_rec < 0) return report_error(WRI_EINVAL, "system %d: n_rec < 0", k);
    if (s.n_rec > 0 && (s.d == nullptr || pos[k].rec == nullptr))
      return report_error(WRI_EINVAL, "system %d: d or receiver positions NULL", k);
    if (mode == WRI_KNOWN && (!std::isfinite(s.alpha.re) || !std::isfinite(s.alpha.im)))
      return report_error(WRI_EINVAL, "system %d: alpha not finite", k);
    for (int a = 0; a < 3; ++a)
      if (!std::isfinite(pos[k].src[a])) return report_error(WRI_EINVAL, "system %d: source position not finite", k);
    for (int q = 0; q < 3 * s.n_rec; ++q)
      if (!std::isfinite(pos[k].rec[q])) return report_error(WRI_EINVAL, "system %d: receiver position not finite", k);
  }
  return WRI_OK;
}

int og_layout(const wri_grid* grids, const wri_system* sys, int n_sys, const OgPlan& P, const SysTables& T, OgLayout* L) {
  size_t o = 0;
  auto take = [&](size_t bytes) { size_t r = o; o = al(o + std::max<size_t>(bytes, 1)); return r; };
  int64_t sums = 0;
  L->part0.resize(n_sys);
  for (int p = 0; p < n_sys; ++p) {
    const wri_grid& g = grids[sys[P.order[p]].grid];
    L->part0[p] = (int)sums;
    sums += std::max(kParts, P.cx[p] > 0 ? ow_tiles(g, P.cx[p]) : kParts);
  }
  L->vec.resize(n_sys);
  L->rvec.resize(n_sys);
  for (int k = 0; k < n_sys; ++k) {
    L->vec[k] = take(7 * al(sizeof(float2) * (size_t)ncell(grids[sys[k].grid])));
    L->rvec[k] = take(2 * al(sizeof(float2) * (size_t)sys[k].n_rec));
  }
  L->state = take(sizeof(OgState) * (size_t)std::max(n_sys, 1));
  L->parts = take(sizeof(double) * (size_t)std::max<int64_t>(sums, kParts));
  // the tables the host writes, in one piece
  L->sys = take(sizeof(OgSys) * (size_t)std::max(n_sys, 1));
  L->groups = take(std::max(sizeof(OwGroup) * P.table_entries(), sizeof(int) * (size_t)std::max(n_sys, 1)));
  L->tables = o;
  for (int k = 0; k < n_sys; ++k) o = al(o + T.bytes(k));
  L->total = o + kAl;
  return WRI_OK;
}

int og_run(const wri_grid* grids, int n_grids, const float* const* m, const wri_system* sys, int n_sys,
           const wri_positions* pos, int mode, int max_iter, int flags, double* J_out, float* const* grad,
           wri_c32* const* u_out, wri_result* res, void* ws, size_t ws_bytes, hipStream_t st) {
  int rc = validate_offgrid(grids, n_grids, sys, n_sys, pos, mode, max_iter);
  if (rc != WRI_OK) return rc;
  if (n_sys > 0 && res == nullptr) return report_error(WRI_EINVAL, "res is NULL");
  if (flags & (WRI_FLAG_WARM_START | WRI_FLAG_ADJOINT_SOURCE))
    return report_error(WRI_EINVAL, "off-grid solves take no WRI_FLAG_WARM_START or WRI_FLAG_ADJOINT_SOURCE");
  if (n_grids > 0 && m == nullptr) return report_error(WRI_EINVAL, "m is NULL");
  for (int g = 0; g < n_grids; ++g)
    if (m[g] == nullptr || (grad != nullptr && grad[g] == nullptr))
      return report_error(WRI_EINVAL, "m[%d] or grad[%d] is NULL", g, g);
  const SysTables tabs = build_tables(grids, sys, n_sys, pos);
  OgPlan P = og_plan(grids, sys, n_sys, true);
  OgLayout L;
  og_layout(grids, sys, n_sys, P, tabs, &L);
  if (ws_bytes < L.total) {   // the march's own size is enough for it
    P = og_plan(grids, sys, n_sys, false);
    og_layout(grids, sys, n_sys, P, tabs, &L);
  }
  if (ws == nullptr || ws_bytes < L.total)
    return report_error(WRI_ENOWS, "workspace of %zu bytes is smaller than the %zu required", ws_bytes, L.total);
  char* base = reinterpret_cast<char*>(al(reinterpret_cast<uintptr_t>(ws)));
  if (J_out) *J_out = 0.0;
  if (n_sys == 0) {
    if (grad != nullptr)
      for (int g = 0; g < n_grids; ++g) OG_HIP(launch_zero_f32(grad[g], (size_t)ncell(grids[g]), st));
    OG_HIP(hipStreamSynchronize(st));
    return WRI_OK;
  }
  // device tables: one image of [sys, end of the receiver tables), one copy
  std::vector<OgSys> hs(n_sys);
  std::vector<char> head;
  struct Drain { hipStream_t st; ~Drain() { (void)hipStreamSynchronize(st); } } drain{st};   // before head goes
  head.resize(L.tables - L.sys);
  auto put = [&](const void* v, size_t bytes) {   // appended; its device address
    const size_t at = head.size();
    head.resize(at + al(bytes));
    if (bytes > 0) std::memcpy(head.data() + at, v, bytes);
    return base + L.sys + at;
  };
  auto ints = [&](const std::vector<int>& v) { return reinterpret_cast<const int*>(put(v.data(), sizeof(int) * v.size())); };
  auto dbls = [&](const std::vector<double>& v) {
    return reinterpret_cast<const double*>(put(v.data(), sizeof(double) * v.size()));
  };
  int64_t nmax = 1;
  std::vector<int> first(tabs.sets.size(), -1);   // slot whose tables a set's later systems share
  for (int p = 0; p < n_sys; ++p) {
    const int k = P.order[p];
    const wri_system& s = sys[k];
    const wri_grid& g = grids[s.grid];
    const Point& src = tabs.src[k];
    const RecTables& T = tabs.sets[tabs.set_of[k]];
    const int64_t n = ncell(g);
    const size_t vb = al(sizeof(float2) * (size_t)n);
    const size_t rb = al(sizeof(float2) * (size_t)s.n_rec);
    float2* v = reinterpret_cast<float2*>(base + L.vec[k]);
    OgSys& S = hs[p];
    S = OgSys{};
    S.x = (u_out != nullptr && u_out[k] != nullptr) ? reinterpret_cast<float2*>(u_out[k]) : v;
    S.r[0] = reinterpret_cast<float2*>(base + L.vec[k] + vb);
    S.r[1] = reinterpret_cast<float2*>(base + L.vec[k] + 2 * vb);
    S.p[0] = reinterpret_cast<float2*>(base + L.vec[k] + 3 * vb);
    S.p[1] = reinterpret_cast<float2*>(base + L.vec[k] + 4 * vb);
    S.s = reinterpret_cast<float2*>(base + L.vec[k] + 5 * vb);
    S.t = reinterpret_cast<float2*>(base + L.vec[k] + 6 * vb);
    S.r2 = reinterpret_cast<float2*>(base + L.rvec[k]);
    S.t2 = reinterpret_cast<float2*>(base + L.rvec[k] + rb);
    S.d = reinterpret_cast<const float2*>(s.d);
    S.scell = reinterpret_cast<const int*>(put(src.cells, sizeof(int) * src.n));
    S.sw = reinterpret_cast<const double*>(put(src.w, sizeof(double) * src.n));
    int& f = first[tabs.set_of[k]];
    if (f >= 0) {
      const OgSys& B = hs[f];
      S.rptr = B.rptr; S.rcell = B.rcell; S.rw = B.rw;
      S.uptr = B.uptr; S.ucell = B.ucell; S.uq = B.uq; S.uw = B.uw;
    } else {
      S.rptr = ints(T.rptr); S.rcell = ints(T.rcell); S.rw = dbls(T.rw);
      S.uptr = ints(T.uptr); S.ucell = ints(T.ucell); S.uq = ints(T.uq); S.uw = dbls(T.uw);
      f = p;
    }
    S.n = (int)n;
    S.ns = src.n;
    S.nr = s.n_rec;
    S.nu = (int)T.ucell.size();
    S.est = mode == WRI_ESTIMATE;
    S.max_iter = max_iter;
    S.c = (flags & WRI_FLAG_UNSCALED_ALPHA) ? 1.0 : std::sqrt(42.0) / (g.h * g.h);
    S.lam = s.lambda;
    S.rtol2 = s.rtol * s.rtol;
    S.omega = s.omega;
    S.omega2 = s.omega * s.omega;
    S.alpha = make_double2(s.alpha.re, s.alpha.im);
    S.m = m[s.grid];
    S.nx = g.nx; S.ny = g.ny; S.nz = g.nz; S.nb = g.nb;
    S.part0 = L.part0[p];
    S.nparts = P.cx[p] > 0 ? ow_tiles(g, P.cx[p]) : kParts;
    S.h2inv = 1.0 / (g.h * g.h);
    if (g.nb > 0) {
      const double d0 = 3.0 * g.v_ref * std::log(1000.0) / (2.0 * g.nb * g.h);
      S.sp_scale = 2.0 * d0 / (g.v_ref * g.v_ref);
      S.inv_nb = 1.0 / g.nb;
    }
    nmax = std::max<int64_t>(nmax, n);
  }
  OgSys* dsys = reinterpret_cast<OgSys*>(base + L.sys);
  OgState* dst = reinterpret_cast<OgState*>(base + L.state);
  double* parts = reinterpret_cast<double*>(base + L.parts);
  std::memcpy(head.data(), hs.data(), sizeof(OgSys) * n_sys);
  OwGroups win[3] = {};
  size_t at = L.groups - L.sys;
  for (int c = 1; c <= 2; ++c) {
    const auto& v = P.groups[c];
    win[c].n = (int)v.size();
    win[c].xchunk = P.xchunk[c];
    std::copy_n(v.begin(), std::min(v.size(), (size_t)kOwGroups), win[c].g);
    if (v.size() <= (size_t)kOwGroups) continue;
    win[c].table = reinterpret_cast<const OwGroup*>(base + L.sys + at);
    std::memcpy(head.data() + at, v.data(), sizeof(OwGroup) * v.size());
    at += sizeof(OwGroup) * v.size();
  }
  OG_HIP(hipMemcpyAsync(base + L.sys, head.data(), head.size(), hipMemcpyHostToDevice, st));

  const dim3 vgrid(nblk(nmax), n_sys), pgrid(kParts, n_sys);
  auto lds = [&](int c) { return (unsigned)(sizeof(float2) * kOwZ * (64 * kOwW * c + 2 * P.nx[c])); };
  const int march = P.groups[0].empty() ? 0 : P.blocks[0] / kParts;   // the first systems
  // a stencil pass: a launch for each kind of passes in the call
  auto fwd = [&]() {
    if (march > 0) hipLaunchKernelGGL(k_og_fwd, dim3(kParts, march), dim3(kThreads), 0, st, dsys, dst, parts, 0);
    if (win[1].n > 0) hipLaunchKernelGGL(k_ow_fwd<1>, dim3(P.blocks[1]), dim3(kThreads), lds(1), st, dsys, dst, parts, win[1]);
    if (win[2].n > 0) hipLaunchKernelGGL(k_ow_fwd<2>, dim3(P.blocks[2]), dim3(kThreads), lds(2), st, dsys, dst, parts, win[2]);
  };
  auto adj = [&](bool setup) {
    if (march > 0) hipLaunchKernelGGL(k_og_adj, dim3(kParts, march), dim3(kThreads), 0, st, dsys, dst, parts, 0, setup ? 1 : 0);
    if (win[1].n > 0) {
      if (setup) hipLaunchKernelGGL((k_ow_adj<1, true>), dim3(P.blocks[1]), dim3(kThreads), lds(1), st, dsys, dst, parts, win[1]);
      else hipLaunchKernelGGL((k_ow_adj<1, false>), dim3(P.blocks[1]), dim3(kThreads), lds(1), st, dsys, dst, parts, win[1]);
    }
    if (win[2].n > 0) {
      if (setup) hipLaunchKernelGGL((k_ow_adj<2, true>), dim3(P.blocks[2]), dim3(kThreads), lds(2), st, dsys, dst, parts, win[2]);
      else hipLaunchKernelGGL((k_ow_adj<2, false>), dim3(P.blocks[2]), dim3(kThreads), lds(2), st, dsys, dst, parts, win[2]);
    }
  };
  // `count` iterations of every system (finished systems skip inside the kernels):
  // four launches per iteration.  Eager: a graph of the chunk, which holds this
  // workspace's pointers and so lives for one call only, cost 0.3 ms to build.
  auto enqueue = [&](int count) -> int {
    for (int it = 0; it < count; ++it) {
      fwd();
      hipLaunchKernelGGL(k_og_alpha, dim3(n_sys), dim3(kThreads), 0, st, dsys, dst, parts);
      adj(false);
      hipLaunchKernelGGL(k_og_beta, dim3(n_sys), dim3(kThreads), 0, st, dsys, dst, parts);
      OG_HIP(hipGetLastError());
    }
    return WRI_OK;
  };
  // set-up: x = 0, r_0 = b, s_0 = S^H b, gamma0
  hipLaunchKernelGGL(k_og_zero, vgrid, dim3(kThreads), 0, st, dsys);
  hipLaunchKernelGGL(k_og_init, dim3(n_sys), dim3(kThreads), 0, st, dsys, dst);
  adj(true);
  hipLaunchKernelGGL(k_og_start, dim3(n_sys), dim3(kThreads), 0, st, dsys, dst, parts);
  OG_HIP(hipGetLastError());
  std::vector<OgState> hst(n_sys);
  auto read = [&]() -> int {
    OG_HIP(hipMemcpyAsync(hst.data(), dst, sizeof(OgState) * n_sys, hipMemcpyDeviceToHost, st));
    OG_HIP(hipStreamSynchronize(st));
    return WRI_OK;
  };
  // Every system has stopped after max_iter iterations, so the statuses are looked at
  // between chunks only.
  for (int64_t done = 0, chunk = kCheck / 2; done < max_iter; chunk = kCheck) {
    const int count = (int)std::min<int64_t>(chunk, max_iter - done);
    if ((rc = enqueue(count)) != WRI_OK) return rc;
    done += count;
    if (done >= max_iter) break;
    if ((rc = read()) != WRI_OK) return rc;
    bool active = false;
    for (const auto& T : hst) active |= T.status == kActive;
    if (!active) break;
  }
  // objective, source weights, gradient
  hipLaunchKernelGGL(k_og_rnorm, pgrid, dim3(kThreads), 0, st, dsys, dst, parts);
  OG_HIP(hipGetLastError());
  hipLaunchKernelGGL(k_og_final, dim3(n_sys), dim3(kThreads), 0, st, dsys, dst, parts);
  OG_HIP(hipGetLastError());
  if (grad != nullptr)
    for (int g = 0; g < n_grids; ++g) {
      int s0 = 0, cnt = 0;
      for (const auto& v : P.groups)
        for (const auto& e : v)
          if (sys[P.order[e.rhs0]].grid == g) s0 = e.rhs0;
      while (s0 + cnt < n_sys && sys[P.order[s0 + cnt]].grid == g) ++cnt;
      const int64_t n = ncell(grids[g]);
      hipLaunchKernelGGL(k_og_grad, dim3(nblk(n)), dim3(kThreads), 0, st, dsys, dst, s0, cnt, (int)n, grad[g]);
      OG_HIP(hipGetLastError());
    }
  if ((rc = read()) != WRI_OK) return rc;
  for (const auto& T : hst)
    if (T.status == kActive) return report_error(WRI_EHIP, "internal: systems active past max_iter");
  double Jtot = 0.0;
  int ret = WRI_OK;
  std::vector<int> slot(n_sys);
  for (int p = 0; p < n_sys; ++p) slot[P.order[p]] = p;
  for (int k = 0; k < n_sys; ++k) {
    const OgState& T = hst[slot[k]];
    double ee = 0.0;
    for (int i = 0; i < tabs.src[k].n; ++i) ee += tabs.src[k].w[i] * tabs.src[k].w[i];
    wri_result& r = res[k];
    r.iters = T.iters;
    r.status = T.status;
    r.relres = T.gamma0 > 0.0 ? std::sqrt(std::max(T.gamma, 0.0) / T.gamma0) : 0.0;
    r.J = T.J;
    if (mode == WRI_ESTIMATE) {
      r.alpha = wri_c64{hs[slot[k]].c * T.xa.x, hs[slot[k]].c * T.xa.y};
      r.alpha_ls = ee > 0.0 ? wri_c64{T.eau.x / ee, T.eau.y / ee} : wri_c64{0.0, 0.0};
    } else {
      r.alpha = sys[k].alpha;
      r.alpha_ls = sys[k].alpha;
    }
    Jtot += T.J;
    if (T.status == kBreakdown) ret = WRI_EBREAKDOWN;
    else if (T.status == kMaxIter && ret == WRI_OK) ret = WRI_NOT_CONVERGED;
  }
  if (J_out) *J_out = Jtot;
  if (ret == WRI_EBREAKDOWN) report_error(WRI_EBREAKDOWN, "at least one system broke down");
  return ret;
}

}  // namespace
}  // namespace wri

using namespace wri;

extern "C" {

size_t wri_offgrid_workspace_bytes(const wri_grid* grids, int32_t n_grids, const wri_system* sys, int32_t n_sys,
                                   const wri_positions* pos) {
  try {
    if (validate_offgrid(grids, n_grids, sys, n_sys, pos, WRI_ESTIMATE, 0) != WRI_OK) return 0;
    OgLayout L;
    og_layout(grids, sys, n_sys, og_plan(grids, sys, n_sys, true), build_tables(grids, sys, n_sys, pos), &L);
    return L.total;
  } catch (const std::exception& e) {
    report_error(WRI_EINVAL, "exception: %s", e.what());
    return 0;
  }
}

int wri_objective_grad_offgrid(const wri_grid* grids, int32_t n_grids, const float* const* m, const wri_system* sys,
                               int32_t n_sys, const wri_positions* pos, int32_t mode, int32_t max_iter,
                               int32_t flags, double* J_out, float* const* grad, wri_c32* const* u_out,
                               wri_result* res, void* ws, size_t ws_bytes, void* stream) {
  try {
    return og_run(grids, n_grids, m, sys, n_sys, pos, mode, max_iter, flags, J_out, grad, u_out, res, ws, ws_bytes,
                  reinterpret_cast<hipStream_t>(stream));
  } catch (const std::exception& e) {
    return report_error(WRI_EINVAL, "exception: %s", e.what());
  }
}

}  // extern "C"
