// IC(0) in natural and block red-black order, one launch per level, on the
// arrays in voxel order.
//
// The sweeps of fm_natural.hpp read rows packed in step order, of which a column
// of nz voxels takes nz + 15 rounded up to 16, and 8 more: some 30 B a voxel at
// 128x128x64, but 600 to 760 B where the volume is a single slice.  Volumes whose
// rows would take too much (packed_rows_fit in fm_api.hip), or do not fit the
// device, run here, on the arrays that red-black IC(0) has too.
//
// Natural order: the voxels with x + y + z = s need those of smaller s only; a
// thread takes one of the at most min(ny, nz) of an x.  Block red-black: the same
// inside every tile of 8 x 8 columns at once, colour by colour; a thread takes a
// column.  The launches are bound by their number (2401x2399x1: 4799 a sweep), not
// by the work in them.  A preconditioner step of that slice in F64 takes 32 ms (5.3 ms
// with 4.4 GB of packed rows), one of 2741x2743x1 in block red-black order 2.3 ms (4.2).
//
// The arithmetic and its order are those of FwdLane and BwdLane: the same pivots
// and p, to the bit.
#pragma once

#include "fm_natural.hpp"

namespace fm {

constexpr int kLevelNT = 64;  // threads of a workgroup: small ones spread a level over the compute units

template <typename T>
struct LevelArgs {
  Geo geo;
  double beta;
  const uint8_t *code;
  const T *D, *g;
  T *X, *P;
  double *ipiv;
  int32_t *status;
  int32_t per_x;  // threads for each x: natural order min(ny, nz), block red-black ny
};

// The voxel of level s that a thread takes.
struct LevelVoxel {
  int64_t j;
  uint32_t c;
  bool x0, x7, y0, y7;  // on the lower or upper face of its tile
};
// False: the thread has none.
template <bool BLOCK, typename T>
__device__ __forceinline__ bool level_voxel(const LevelArgs<T> &a, int s, int colour, LevelVoxel &v) {
  const Geo &g = a.geo;
  const int64_t t = (int64_t)blockIdx.x * kLevelNT + threadIdx.x;
  const int x = (int)(t / a.per_x), q = (int)(t - (int64_t)x * a.per_x);
  if (x >= g.nx) return false;
  int y, z;
  if constexpr (BLOCK) {
    y = q;
    if (((x / kTile + y / kTile) & 1) != colour) return false;
    z = s - x % kTile - y % kTile;
    if (z < 0 || z >= g.nz) return false;
  } else {
    const int r = s - x;  // = y + z
    y = (r - (g.nz - 1) > 0 ? r - (g.nz - 1) : 0) + q;
    if (y >= g.ny || y > r) return false;
    z = r - y;
  }
  v.j = x * g.sx + y * g.sy + z;
  v.c = a.code[v.j];
  v.x0 = x % kTile == 0;
  v.x7 = x % kTile == kTile - 1;
  v.y0 = y % kTile == 0;
  v.y7 = y % kTile == kTile - 1;
  return true;
}

// Sum over the -z, y and x neighbours that precede a voxel, of val(neighbour).
template <bool BLOCK, typename F>
__device__ __forceinline__ double sum_before(const LevelVoxel &v, const Geo &g, int colour, F val) {
#pragma clang fp contract(off)
  const bool late = !BLOCK || colour == 1;  // every neighbour across a face precedes (natural order: the lower ones)
  const double sz = (v.c & NB_ZM) ? val(v.j - 1) : 0.0;
  double sy = (v.c & NB_YM) && (late || !v.y0) ? val(v.j - g.sy) : 0.0;
  if (BLOCK && late && v.y7 && (v.c & NB_YP)) sy = sy + val(v.j + g.sy);
  double sx = (v.c & NB_XM) && (late || !v.x0) ? val(v.j - g.sx) : 0.0;
  if (BLOCK && late && v.x7 && (v.c & NB_XP)) sx = sx + val(v.j + g.sx);
  return (sz + sy) + sx;
}

// The same over the neighbours that follow it.
template <bool BLOCK, typename F>
__device__ __forceinline__ double sum_after(const LevelVoxel &v, const Geo &g, int colour, F val) {
#pragma clang fp contract(off)
  const bool early = !BLOCK || colour == 0;
  const double sz = (v.c & NB_ZP) ? val(v.j + 1) : 0.0;
  double sy = (v.c & NB_YP) && (early || !v.y7) ? val(v.j + g.sy) : 0.0;
  if (BLOCK && early && v.y0 && (v.c & NB_YM)) sy = sy + val(v.j - g.sy);
  double sx = (v.c & NB_XP) && (early || !v.x7) ? val(v.j + g.sx) : 0.0;
  if (BLOCK && early && v.x0 && (v.c & NB_XM)) sx = sx + val(v.j - g.sx);
  return (sz + sy) + sx;
}

template <typename T, bool BLOCK>
__global__ __launch_bounds__(kLevelNT) void k_ic_level_fwd(LevelArgs<T> a, int s, int colour) {
#pragma clang fp contract(off)
  LevelVoxel v;
  if (!level_voxel<BLOCK>(a, s, colour, v)) return;
  double r = 0.0;
  T x = T(0);
  if (v.c & NB_SELF) {
    const double h = (double)a.D[v.j] + a.beta * nb_deg(v.c), b2 = a.beta * a.beta;
    const double piv = fma(-b2, sum_before<BLOCK>(v, a.geo, colour, [&](int64_t k) { return a.ipiv[k]; }), h);
    const double xs = sum_before<BLOCK>(v, a.geo, colour, [&](int64_t k) { return (double)a.X[k]; });
    if (piv > 0.0)
      r = 1.0 / piv;
    else
      set_status(a.status, 5);
    x = (T)(fma(a.beta, xs, (double)a.g[v.j]) * r);
  }
  a.ipiv[v.j] = r;
  a.X[v.j] = x;
}

template <typename T, bool BLOCK>
__global__ __launch_bounds__(kLevelNT) void k_ic_level_bwd(LevelArgs<T> a, int s, int colour) {
#pragma clang fp contract(off)
  LevelVoxel v;
  if (!level_voxel<BLOCK>(a, s, colour, v)) return;
  T p = T(0);
  if (v.c & NB_SELF) {
    const double ps = sum_after<BLOCK>(v, a.geo, colour, [&](int64_t k) { return (double)a.P[k]; });
    p = (T)fma(a.beta * ps, a.ipiv[v.j], (double)a.X[v.j]);
  }
  a.P[v.j] = p;
}

}  // namespace fm
