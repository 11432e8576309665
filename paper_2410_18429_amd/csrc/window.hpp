// Geometry, loads and stores of window tiles: 64 W CX consecutive cells of the x-y
// plane and TZ planes per workgroup (see the window march in kernels.hip), with
// the buffer accesses and the block order they share with the slab marches.
// Device-only inline functions.
#pragma once

#include <hip/hip_runtime.h>

#include "wri_impl.hpp"

namespace wri {

__device__ __forceinline__ int xcd_remap(int b, int nb, int q) {
  // Blocks go round-robin to the XCDs (b % 8).  The logical sequence of
  // (group, system, tile) is cut into chunks of q consecutive tiles, dealt to the
  // XCDs round-robin as well: the tiles of a chunk are spatial neighbours on
  // one XCD (halo re-reads hit its L2), and every XCD holds a share of every
  // system, so no XCD idles while others still work when some systems of the
  // batch have converged.  Blocks past the last complete round keep their index.
  const int xcd = b % kXCD, local = b / kXCD;
  const int full = nb / (kXCD * q) * (kXCD * q);
  if (b >= full) return b;
  const int round = local / q, off = local - round * q;
  return (round * kXCD + xcd) * q + off;
}

// The group of a block, from the launch arguments (up to N groups; a load from the
// device table would be one more memory latency in every launch).
template <class Group, int N>
__device__ __forceinline__ Group group_of(const Group (&first)[N], const Group* table, int n, int logical) {
  Group d = first[0];
  if (n <= N) {
#pragma unroll
    for (int i = 1; i < N; ++i)
      if (i < n && logical >= first[i].block0) d = first[i];
  } else {
    int g = 0, end = n;
    while (end - g > 1) {
      const int mid = (g + end) / 2;
      if (logical >= table[mid].block0) g = mid;
      else end = mid;
    }
    d = table[g];
  }
  return d;
}

typedef __amdgpu_buffer_rsrc_t BufRes;
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
constexpr unsigned kOOB = 0x80000000u;   // beyond any resource (records < 2^31)
constexpr int kBufFlags = 0x00020000;    // raw 32-bit buffer, gfx9 family
constexpr int kStoreNT = 2;              // non-temporal store

// Resource over elements [first, first + count) of v (elem bytes each).
__device__ __forceinline__ BufRes mkbuf(const void* v, int64_t first, int64_t count, int elem) {
  const char* b = static_cast<const char*>(v) + first * elem;
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<char*>(b), (short)0, (int)(count * elem), kBufFlags);
}
__device__ __forceinline__ float2 bld2(BufRes r, unsigned off) {
  return __builtin_bit_cast(float2, __builtin_amdgcn_raw_buffer_load_b64(r, off, 0, 0));
}
__device__ __forceinline__ float4 bld4(BufRes r, unsigned off) {
  return __builtin_bit_cast(float4, __builtin_amdgcn_raw_buffer_load_b128(r, off, 0, 0));
}
__device__ __forceinline__ float bld1(BufRes r, unsigned off) {
  return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(r, off, 0, 0));
}
__device__ __forceinline__ void bst2(BufRes r, unsigned off, float2 v) {
  __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2, v), r, off, 0, kStoreNT);
}

// Stores of the window march go through L2 (system scope: sc0 and sc1).  Its
// outputs fit the L2s (4 MB per XCD), where ordinary stores would stay dirty
// until the end of the launch and be written back then, after the last
// workgroup: 8 systems of 64^3 took 42.8 us per iteration with ordinary or
// non-temporal stores and 37.6 us with these.
constexpr int kStoreThrough = 17;

// Loads above this point are issued before anything below it: without it the
// compiler moves them down to their uses (behind the scalars and the stop
// test), one latency after the other.  It waits for nothing.
__device__ __forceinline__ void issue_point() { asm volatile("" ::: "memory"); }

// v where m is all ones, zero where m is zero.  The neighbours in x of a cell at the
// end of a row: selected (x > 0 ? row[-1] : 0) the compiler guards each component's
// LDS read with a branch and waits for it on the spot, four latencies in a row per
// cell; read unconditionally (the window holds a cell on either side) and masked they
// are in flight together.  Preconditioned iteration of 48 systems of 128^3 5.16 -> 5.04
// ms, off-grid gradient of 8 of 64^3 989 -> 942 us, plain gradient of 48 of 32^3 1166 -> 1151.
__device__ __forceinline__ unsigned row_mask(bool inside) { return inside ? ~0u : 0u; }
__device__ __forceinline__ float2 masked(float2 v, unsigned m) {
  return make_float2(__builtin_bit_cast(float, __builtin_bit_cast(unsigned, v.x) & m),
                     __builtin_bit_cast(float, __builtin_bit_cast(unsigned, v.y) & m));
}
__device__ __forceinline__ double2 masked(double2 v, unsigned m) {
  const unsigned long long w = (unsigned long long)m << 32 | m;
  return make_double2(__builtin_bit_cast(double, __builtin_bit_cast(unsigned long long, v.x) & w),
                      __builtin_bit_cast(double, __builtin_bit_cast(unsigned long long, v.y) & w));
}

template <int W, int CX, int TZ>
struct Win {
  static constexpr int NT = 64 * W;
  static constexpr int B = NT * CX;   // own cells per plane
  int nx, ny, nz, plane, c0, z0, wl, zlo, zhi;
  int cell[CX];                       // linear cell in the plane (may lie past its end)
  bool in[CX];
  unsigned obit[CX];                  // out-of-range bit of cells past the end of the plane

  __device__ __forceinline__ void setup(int nx_, int ny_, int nz_, int tile, int tiles_x) {
    nx = nx_; ny = ny_; nz = nz_;
    plane = nx * ny;
    const int tz = tile / tiles_x;
    c0 = (tile - tz * tiles_x) * B;
    z0 = tz * TZ;
    zlo = max(z0 - 1, 0);
    zhi = min(z0 + TZ + 1, nz);
    wl = B + 2 * nx;
#pragma unroll
    for (int j = 0; j < CX; ++j) {
      cell[j] = c0 + j * NT + (int)threadIdx.x;
      in[j] = cell[j] < plane;
      obit[j] = in[j] ? 0u : kOOB;
    }
  }
  // Buffer accesses: plane i (z0 - 1 + i, i = 0 .. TZ + 1) of a stencil input and
  // plane i (z0 + i, i = 0 .. TZ - 1) of a vector of own cells.  The plane is a
  // scalar offset; a plane outside the grid gets a resource without records and
  // a cell outside it the out-of-range bit, so reads there give zero and stores
  // are dropped.
  __device__ __forceinline__ BufRes in_res(const void* v, int i, int elem) const {
    const int z = z0 - 1 + i;
    const bool ok = z >= 0 && z < nz;
    return __builtin_amdgcn_make_buffer_rsrc(
        const_cast<char*>(static_cast<const char*>(v) + (int64_t)zlo * plane * elem), (short)0,
        ok ? (zhi - zlo) * plane * elem : 0, kBufFlags);
  }
  __device__ __forceinline__ unsigned in_off(int i, int elem) const {
    const int z = min(max(z0 - 1 + i, zlo), zhi - 1);
    return (unsigned)((z - zlo) * plane * elem);
  }
  __device__ __forceinline__ float2 load2(const void* v, int i, unsigned voff) const {
    return __builtin_bit_cast(float2, __builtin_amdgcn_raw_buffer_load_b64(in_res(v, i, 8), voff, in_off(i, 8), 0));
  }
  __device__ __forceinline__ float load1(const void* v, int i, unsigned voff) const {
    return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(in_res(v, i, 4), voff, in_off(i, 4), 0));
  }
  __device__ __forceinline__ void store2(void* v, int i, unsigned voff, float2 x) const {
    __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2, x), in_res(v, i, 8), voff, in_off(i, 8), kStoreThrough);
  }
  __device__ __forceinline__ void store2nt(void* v, int i, unsigned voff, float2 x) const {
    __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2, x), in_res(v, i, 8), voff, in_off(i, 8), kStoreNT);
  }
  __device__ __forceinline__ unsigned own2(int j) const { return (unsigned)(cell[j] * 8) | obit[j]; }
  __device__ __forceinline__ unsigned own1(int j) const { return (unsigned)(cell[j] * 4) | obit[j]; }
  __device__ __forceinline__ bool zin(int i) const { return z0 - 1 + i >= 0 && z0 - 1 + i < nz; }
  __device__ __forceinline__ bool live(int j, int i) const { return in[j] && z0 + i < nz; }
  // halo cell h (0 .. 2 nx - 1): byte offset in a plane and window index
  __device__ __forceinline__ unsigned halo_off(int h) const {
    const int c = h < nx ? c0 - nx + h : c0 + B + (h - nx);
    return (unsigned)(c * 8) | ((c >= 0 && c < plane) ? 0u : kOOB);
  }
  __device__ __forceinline__ int halo_slot(int h) const { return h < nx ? h : B + h; }

  // Row of a cell of the tile: the offset from the first cell's row start is
  // below B + nx, where the float quotient (with half a cell's margin) is exact.
  __device__ __forceinline__ void row_of(int c, int* x, int* y) const {
    const int y0 = c0 / nx, d = c - y0 * nx;
    const int r = (int)(((float)d + 0.5f) * (1.0f / (float)nx));
    *y = y0 + r;
    *x = d - r * nx;
  }
};

}  // namespace wri
