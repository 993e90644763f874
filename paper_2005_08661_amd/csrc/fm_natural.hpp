// IC(0) in natural order (Sec. III-B eq. (precon)) as a pipelined wavefront.
//
// The recurrences
//   forward   P_j = h_j - beta^2 sum_{k lower} 1/P_k,  x_j = (g_j + beta sum_{k lower} x_k) / P_j
//   backward  p_j = x_j + (beta / P_j) sum_{k upper} p_k
// (lower = -x, -y, -z neighbours in the mask, upper = +x, +y, +z) have a
// dependency chain of length nx+ny+nz-2.  The (x, y) plane is cut into 8x8
// column tiles, one wavefront each: lane (a, b) owns column (8ti+a, 8tj+b) and
// at step S handles z = S - a - b (backward: the mirror image), so its -x and
// -y inputs come from lanes t-8 and t-1 of the previous step (cross-lane
// moves) and its -z input from its own previous step.
//
// What bounds a sweep is that chain: steps, and hops from one diagonal of
// tiles to the next, not bytes.  Both are kept short:
//
// - A step holds nothing but the recurrence.  k_nat_pack lays h and g out
//   beforehand as [tile][step][lane], so a step's loads and stores are one
//   contiguous run per wavefront at uniform offsets, and gives every lane
//   without a voxel (outside the column, the volume or the mask) h = +inf and
//   g = 0, for which the step selects 1/P = 0 and x = p = 0 (selects, not products
//   with zero: a NaN or an infinity must not cross the mask): no masks, no
//   branches, no address arithmetic.  The forward sweep overwrites h by 1/P and g
//   by x in place; k_nat_unpack brings p back to voxel order and takes the
//   dot products.
// - A hop is one trip through memory.  The lanes on a tile's upper x and y
//   faces also store their values in a face buffer, and the neighbour tile
//   reads those values themselves instead of a progress counter: k_nat_pack
//   fills the buffers with a bit pattern that no stored value has, and a value
//   that differs from it has arrived (each 8-byte half of a record tells for
//   itself, so no order between stores is needed).  One load brings a face's
//   values of a whole group of kNatU steps, issued before the arithmetic of the
//   group before; the records it takes per step (one load, two stores) stay
//   below the 64 memory operations a wave may have in flight.
//
// Measured at 128x128x64 (MIX), per launch: forward 598 -> 105 us, backward
// 550 -> 92 us (89 us without the select of p, which lengthens the chain), k_nat_pack
// 12 and k_nat_unpack 13 us on top; a step takes 0.105 and 0.06 us (0.7 us before), a
// hop about 3 us (21 us before).  Groups of 4 steps shorten a hop and lengthen every
// step (a group's loads take 1.7 us to arrive): 117 against 109 us forward.
//
// Progress is deadlock-free: a wave takes a ticket from an atomic counter and
// processes the tile of that rank in anti-diagonal order, so it only waits on
// tiles held by waves that started earlier.  Every wait is bounded; on
// expiry the wave records FM_ERR_TIMEOUT and finishes its loop without
// further waiting.
#pragma once

#include "fm_stream.hpp"

namespace fm {

constexpr int kTile = 8;         // tile edge (8x8 columns = one wavefront)
constexpr int kNatU = 8;  // steps per group (two register sets of one group each)
constexpr int kFaceSlots = 16;   // values per step of a face buffer: 8 of the x face, 7 more of the y face
constexpr int kUnpackZ = 32;     // planes z of a tile per workgroup of k_nat_unpack
constexpr int kSpinLimit = 1 << 16;  // polls per wait (each ~1 us): about 0.1 s

// A 16-byte record of a sweep: a double in words 0-1 and a value of the working
// type whose upper word is word 3 (FP32: word 2 is 0).
typedef uint32_t Rec __attribute__((ext_vector_type(4)));
__device__ __forceinline__ Rec make_rec(double d, float t) {
  const uint64_t b = __builtin_bit_cast(uint64_t, d);
  return Rec{(uint32_t)b, (uint32_t)(b >> 32), 0u, __builtin_bit_cast(uint32_t, t)};
}
__device__ __forceinline__ Rec make_rec(double d, double t) {
  const uint64_t b = __builtin_bit_cast(uint64_t, d), c = __builtin_bit_cast(uint64_t, t);
  return Rec{(uint32_t)b, (uint32_t)(b >> 32), (uint32_t)c, (uint32_t)(c >> 32)};
}
__device__ __forceinline__ double rec_d(const Rec &r) {
  return __builtin_bit_cast(double, (uint64_t)r[1] << 32 | r[0]);
}
__device__ __forceinline__ float rec_t(const Rec &r, float) {
  const uint32_t b = r[3];  // (a bit cast of the vector element itself takes element 0)
  return __builtin_bit_cast(float, b);
}
__device__ __forceinline__ double rec_t(const Rec &r, double) {
  return __builtin_bit_cast(double, (uint64_t)r[3] << 32 | r[2]);
}

struct Wavefront {
  const int2 *order;     // [ntiles] tile (ti, tj) of each ticket, anti-diagonal order
  int32_t ntx, nty;      // tiles along x and y
  int32_t ntiles;
  const int2 *blk[2];    // block red-black: the tiles of colour (ti + tj) mod 2 = 0 and 1
  int32_t nblk[2];
  // natural-order sweeps
  int32_t nrow;          // rows of a sweep: nz + 14 steps and one, rounded up to two groups
  int32_t trow;          // rows of a tile in the packed arrays: nrow and 8 that hold 0
  int32_t frow;          // rows of a tile's face buffer (nrow, and the rows read past it, which hold 0)
  uint32_t *ticket;      // [2] forward, backward
  Rec *rec;              // [ntiles + 1][trow][64] h and g, then 1/P and x (guard rows on each side); tile ntiles holds 0
  void *p;               // [ntiles + 1][trow][64] p of the working type
  Rec *ff;               // [ntiles + 1][frow][16] 1/P and x on the upper faces; tile ntiles holds 0 (no neighbour)
  void *fp;              // the same of the working type: p on the lower faces
};

// Raw buffer views: loads and stores at 32-bit byte offsets from a uniform base;
// a load at or past the view's end reads 0 and a store there is dropped.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t plane_view(const void *base, uint32_t nbytes) {
  // descriptor word 3 of an untyped buffer on gfx9-family GPUs
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(base), (short)0, (int)nbytes, 0x00020000);
}
__device__ __forceinline__ uint32_t view_u8(__amdgpu_buffer_rsrc_t r, uint32_t e) {
  return __builtin_amdgcn_raw_buffer_load_b8(r, e, 0, 0);
}
__device__ __forceinline__ float view_ld(__amdgpu_buffer_rsrc_t r, uint32_t e, float) {
  return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(r, e * 4u, 0, 0));
}
__device__ __forceinline__ double view_ld(__amdgpu_buffer_rsrc_t r, uint32_t e, double) {
  return __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(r, e * 8u, 0, 0));
}
__device__ __forceinline__ void view_st(__amdgpu_buffer_rsrc_t r, uint32_t e, float v) {
  __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(uint32_t, v), r, e * 4u, 0, 0);
}
__device__ __forceinline__ void view_st(__amdgpu_buffer_rsrc_t r, uint32_t e, double v) {
  using B64 = decltype(__builtin_amdgcn_raw_buffer_load_b64(r, 0u, 0, 0));
  __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(B64, v), r, e * 8u, 0, 0);
}

__device__ __forceinline__ Rec view_ld(__amdgpu_buffer_rsrc_t r, uint32_t e, Rec) {
  return __builtin_amdgcn_raw_buffer_load_b128(r, e * 16u, 0, 0);
}
__device__ __forceinline__ void view_st(__amdgpu_buffer_rsrc_t r, uint32_t e, Rec v) {
  __builtin_amdgcn_raw_buffer_store_b128(v, r, e * 16u, 0, 0);
}

// Cache policy of accesses that other workgroups take part in (agent scope: sc1).
constexpr int kAuxCoh = 0x10;

template <typename T>
struct Bits;
template <>
struct Bits<float> {
  using U = uint32_t;
  static constexpr U empty = 0xffffffffu, nan = 0x7fc00000u;
};
template <>
struct Bits<double> {
  using U = uint64_t;
  static constexpr U empty = ~0ull, nan = 0x7ff8000000000000ull;
};
__device__ __forceinline__ uint32_t top_word(uint32_t v) { return v; }
__device__ __forceinline__ uint32_t top_word(uint64_t v) { return (uint32_t)(v >> 32); }

// Any NaN as the default one: the sweeps then form no NaN with an upper word of
// all ones, which marks a face value that has not been stored.
template <typename T>
__device__ __forceinline__ T plain_nan(T v) {
  return v == v ? v : (T)__builtin_nan("");
}

// View of one group of steps, and coherent accesses to face values.
template <typename E>
__device__ __forceinline__ __amdgpu_buffer_rsrc_t group_view(const E *p) {
  return plane_view(p, 64u * kNatU * (uint32_t)sizeof(E));
}
__device__ __forceinline__ uint32_t face_ld(__amdgpu_buffer_rsrc_t r, uint32_t e, uint32_t) {
  return __builtin_amdgcn_raw_buffer_load_b32(r, e * 4u, 0, kAuxCoh);
}
__device__ __forceinline__ uint64_t face_ld(__amdgpu_buffer_rsrc_t r, uint32_t e, uint64_t) {
  return __builtin_bit_cast(uint64_t, __builtin_amdgcn_raw_buffer_load_b64(r, e * 8u, 0, kAuxCoh));
}
__device__ __forceinline__ Rec face_ld(__amdgpu_buffer_rsrc_t r, uint32_t e, Rec) {
  return __builtin_amdgcn_raw_buffer_load_b128(r, e * 16u, 0, kAuxCoh);
}
__device__ __forceinline__ void face_st(__amdgpu_buffer_rsrc_t r, uint32_t e, uint32_t v) {
  __builtin_amdgcn_raw_buffer_store_b32(v, r, e * 4u, 0, kAuxCoh);
}
__device__ __forceinline__ void face_st(__amdgpu_buffer_rsrc_t r, uint32_t e, uint64_t v) {
  using B64 = decltype(__builtin_amdgcn_raw_buffer_load_b64(r, 0u, 0, 0));
  __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(B64, v), r, e * 8u, 0, kAuxCoh);
}
__device__ __forceinline__ void face_st(__amdgpu_buffer_rsrc_t r, uint32_t e, Rec v) {
  __builtin_amdgcn_raw_buffer_store_b128(v, r, e * 16u, 0, kAuxCoh);
}

// The value of lane t - 8 (or t + 8): src = 4 x that lane.
__device__ __forceinline__ uint32_t from_x(uint32_t v, int src) { return (uint32_t)__builtin_amdgcn_ds_bpermute(src, (int)v); }
__device__ __forceinline__ uint64_t from_x(uint64_t v, int src) {
  return (uint64_t)from_x((uint32_t)(v >> 32), src) << 32 | from_x((uint32_t)v, src);
}
// The value of lane t - 1 (CTRL 0x111, row_shr:1) or t + 1 (0x101, row_shl:1).
template <int CTRL>
__device__ __forceinline__ uint32_t from_y(uint32_t v) {
  return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, 0xf, 0xf, true);
}
template <int CTRL>
__device__ __forceinline__ uint64_t from_y(uint64_t v) {
  return (uint64_t)from_y<CTRL>((uint32_t)(v >> 32)) << 32 | from_y<CTRL>((uint32_t)v);
}

template <typename V>
__device__ __forceinline__ V from_x_t(V v, int src) {
  return __builtin_bit_cast(V, from_x(__builtin_bit_cast(typename Bits<V>::U, v), src));
}
template <int CTRL, typename V>
__device__ __forceinline__ V from_y_t(V v) {
  return __builtin_bit_cast(V, from_y<CTRL>(__builtin_bit_cast(typename Bits<V>::U, v)));
}

__device__ __forceinline__ int take_ticket(uint32_t *counter) {
  int t = 0;
  if ((threadIdx.x & 63) == 0) t = (int)atomicAdd(counter, 1u);
  return __builtin_amdgcn_readfirstlane(t);
}

// Lay h = D + beta deg and g out in sweep order, empty the face buffers and
// reset the tickets (h, g and the faces of a sweep are used up by it).
// g stands one row behind h: the sweep forms x one step after 1/P.
template <typename T>
__global__ __launch_bounds__(kNT) void k_nat_pack(IterArgs<T> a, Wavefront w, const T *__restrict__ gsrc) {
  const Geo g = a.geo;
  const T *__restrict__ gg = gsrc ? gsrc : ((a.par & 1) ? a.G[1] : a.G[0]);
  using U = typename Bits<T>::U;
  if (blockIdx.x == 0) {  // the gradient pass's sums: no other block needs them
    const State st = take_state<kNT, 4>(a.sin, a.pin, a.nparts_in, a.nvals_in, a.beta, a.trace, a.status);
    put_state(st, a.sout, PK_NONE, 0);
    if (w.ff && threadIdx.x < 2) w.ticket[threadIdx.x] = 0u;
  }
  // one wavefront per 8 rows and column a: lane (s, b) writes the record of lane
  // (a, b) in row 8 i + s, so its loads run along z and its stores along b
  const int lane = (int)threadIdx.x & 63, lb = lane & 7;
  const int64_t units = (int64_t)w.ntiles * w.nrow;  // nrow / 8 row groups x 8 columns
  for (int64_t q = (int64_t)blockIdx.x * (kNT / kWave) + threadIdx.x / kWave; q < units;
       q += (int64_t)gridDim.x * (kNT / kWave)) {
    const int tile = (int)(q / w.nrow), i = (int)(q - (int64_t)tile * w.nrow);
    const int nb = w.nrow / 8, la = i / nb, S = (i - la * nb) * 8 + (lane >> 3);
    const int tx = tile / w.nty, ty = tile - tx * w.nty;
    const int x = tx * kTile + la, y = ty * kTile + lb, z = S - la - lb;
    double h = __builtin_inf();
    double gv = 0.0;
    if (x < g.nx && y < g.ny) {
      const int64_t j = ((int64_t)x * g.ny + y) * g.nz + z;
      if (z >= 0 && z < g.nz) {
        const uint32_t c = a.code[j];
        const T d = a.D[j];
        if (c & NB_SELF) h = plain_nan((double)d + a.beta * nb_deg(c));
      }
      if (z >= 1 && z <= g.nz) {
        const uint32_t c = a.code[j - 1];
        const T gj = gg[j - 1];
        if (c & NB_SELF) gv = plain_nan((double)gj);
      }
    }
    w.rec[((int64_t)tile * w.trow + S) * 64 + la * kTile + lb] = make_rec(h, gv);
    if (w.ff && la < kFaceSlots / kTile) {
      const int64_t e = ((int64_t)tile * w.frow + S) * kFaceSlots + la * kTile + lb;
      w.ff[e] = Rec{~0u, ~0u, ~0u, ~0u};
      ((U *)w.fp)[e] = Bits<T>::empty;
    }
  }
}

// p back to voxel order, the pivots where they are asked for, and the dot
// products g^T p and g_prev^T p.
template <typename T>
__global__ __launch_bounds__(kNT) void k_nat_unpack(IterArgs<T> a, Wavefront w, const T *__restrict__ gsrc) {
  static_assert(kNT == 4 * kWave, "four waves take a tile's eight column rows");
  constexpr int V = 2 * kUnpackZ / 8;
  const Geo g = a.geo;
  const T *__restrict__ gg = gsrc ? gsrc : ((a.par & 1) ? a.G[1] : a.G[0]);
  const T *__restrict__ gp = (a.par & 1) ? a.G[0] : a.G[1];
  const T *__restrict__ pv = (const T *)w.p;
  // one workgroup per kUnpackZ planes z of a tile, so a line of the packed rows
  // is read by one workgroup; wave k takes columns a = k and k + 4, lane (b, z)
  // runs of 8 voxels of the voxel-order arrays
  const int lb = ((int)threadIdx.x & 63) >> 3, zl = (int)threadIdx.x & 7, wv = (int)threadIdx.x / kWave;
  const int nzb = (g.nz + kUnpackZ - 1) / kUnpackZ, nunit = w.ntiles * nzb;
  double acc[2] = {0.0, 0.0};
  for (int q = (int)blockIdx.x; q < nunit; q += (int)gridDim.x) {
    const int tile = q / nzb, z0 = (q - tile * nzb) * kUnpackZ + zl;
    const int tx = tile / w.nty, y = (tile - tx * w.nty) * kTile + lb;
    uint32_t c[V];
    int j[V];
    T gv[V], gpv[V], p[V];
    double ip[V];
#pragma unroll
    for (int v = 0; v < V; ++v) {
      const int z = z0 + (v >> 1) * 8, la = wv + 4 * (v & 1), x = tx * kTile + la;
      const bool ok = x < g.nx && y < g.ny && z < g.nz;
      j[v] = ok ? (x * g.ny + y) * g.nz + z : -1;
      const int jj = ok ? j[v] : 0;
      const int64_t e = ((int64_t)tile * w.trow + (ok ? z : 0) + la + lb) * 64 + la * kTile + lb;
      c[v] = a.code[jj];
      gv[v] = gg[jj];
      gpv[v] = gp[jj];
      p[v] = pv[e];
      ip[v] = a.store_piv ? rec_d(w.rec[e]) : 0.0;
    }
#pragma unroll
    for (int v = 0; v < V; ++v) {
      if (j[v] < 0) continue;
      const bool in = c[v] & NB_SELF;
      a.P[j[v]] = in ? p[v] : T(0);
      if (a.store_piv) a.ipiv[j[v]] = in ? ip[v] : 0.0;
      acc[0] += in ? (double)gv[v] * (double)p[v] : 0.0;
      acc[1] += in ? (double)gpv[v] * (double)p[v] : 0.0;
    }
  }
  const State st = *a.sin;
  store_partials<2, kNT>(acc, a.pout);
  put_state(st, a.sout, PK_DOTS, (int)gridDim.x);
}

// ---------------------------------------------------------------------------
// The faces of a tile in its buffer: x at the slot of its column (the lanes of
// the upper or lower x side), y at 8 + a, their common corner once, with x.
__device__ __forceinline__ uint32_t y_slot(uint32_t a, uint32_t corner) { return a == corner ? corner : kTile + a; }
constexpr uint32_t kNoSlot = 1u << 24;  // past every view: nothing is stored

#define FM_STAGE __builtin_amdgcn_sched_barrier(0)  // the order of a step's operations is the one written

// One lane of the forward sweep.  A step forms 1/P of its row and x of the row
// before, two chains that run side by side in the order written.
// BLOCK: face values are 0 where a lane has none, and add to the in-tile ones;
// otherwise they take their place on the lanes fx, fy.
template <typename T, bool BLOCK = false>
struct FwdLane {
  double r = 0.0;  // 1/P of the previous row (this column's -z neighbour)
  T x = T(0);      // x of the row before that
  bool own = false;  // the previous row's h is finite (it has a voxel)
  bool bad = false;
  __device__ __forceinline__ Rec step(bool fx, bool fy, int xsrc, const Rec &fxr, const Rec &fyr, const Rec &in,
                                      double beta, double b2) {
#pragma clang fp contract(off)  // x as it is stored, not the product it is rounded from
    FM_STAGE;
    // cross-lane moves by every lane, then the choice
    const double rxl = from_x_t(r, xsrc);
    const T xxl = from_x_t(x, xsrc);
    const double ryl = from_y_t<0x111>(r);
    const T xyl = from_y_t<0x111>(x);
    FM_STAGE;
    double ry, rx, xy, xx;
    if constexpr (BLOCK) {
      ry = (fy ? 0.0 : ryl) + rec_d(fyr);
      xy = (double)(fy ? T(0) : xyl) + (double)rec_t(fyr, T());
    } else {
      ry = fy ? rec_d(fyr) : ryl;
      xy = (double)(fy ? rec_t(fyr, T()) : xyl);
    }
    const double r1 = r + ry;
    const double x1 = (double)x + xy;
    FM_STAGE;
    if constexpr (BLOCK)
      rx = (fx ? 0.0 : rxl) + rec_d(fxr);
    else
      rx = fx ? rec_d(fxr) : rxl;
    const double h = rec_d(in);
    const double piv = fma(-b2, r1 + rx, h);
    double q = __builtin_amdgcn_rcp(piv);
    FM_STAGE;
    const bool pos = piv > 0.0, fin = h < __builtin_inf();
    bad |= !pos;
    if constexpr (BLOCK)
      xx = (double)(fx ? T(0) : xxl) + (double)rec_t(fxr, T());
    else
      xx = (double)(fx ? rec_t(fxr, T()) : xxl);
    FM_STAGE;
    // 1 / piv by Newton's iteration q <- q + q (1 - piv q) from the hardware's estimate, with
    // the last residual exact (Markstein 1990, as the quotients of fm_ict_tile.hpp): the value
    // of a division for a normal pivot, without its scaling and special cases
    double e = fma(-piv, q, 1.0);
    const double x2 = x1 + xx;
    FM_STAGE;
    q = fma(q, e, q);
    const double x3 = fma(beta, x2, rec_t(in, double()));
    FM_STAGE;
    e = fma(-piv, q, 1.0);
    const double x4 = x3 * r;
    FM_STAGE;
    q = fma(q, e, q);
    x = own ? (T)x4 : T(0);
    FM_STAGE;
    e = fma(-piv, q, 1.0);
    q = fma(q, e, q);
    r = pos && fin ? q : 0.0;
    own = fin;
    return make_rec(r, x);
  }
};

// One lane of the backward sweep.
template <typename T, bool BLOCK = false>
struct BwdLane {
  T p = T(0);       // p of the previous step (this column's +z neighbour)
  T x_next = T(0);  // x of this step's row (it stands in the record of the row after)
  __device__ __forceinline__ T step(bool fx, bool fy, int xsrc, typename Bits<T>::U fxv, typename Bits<T>::U fyv,
                                    const Rec &in, double beta) {
#pragma clang fp contract(off)
    FM_STAGE;
    const T pxl = from_x_t(p, xsrc), pyl = from_y_t<0x101>(p);
    const T fxp = __builtin_bit_cast(T, fxv), fyp = __builtin_bit_cast(T, fyv);
    double px, py;
    if constexpr (BLOCK) {
      py = (double)(fy ? T(0) : pyl) + (double)fyp;
      px = (double)(fx ? T(0) : pxl) + (double)fxp;
    } else {
      py = (double)(fy ? fyp : pyl);
      px = (double)(fx ? fxp : pxl);
    }
    const T pj = (T)fma(beta * (((double)p + py) + px), rec_d(in), (double)x_next);
    p = rec_d(in) != 0.0 ? pj : T(0);
    x_next = rec_t(in, T());
    return p;
  }
};

template <typename T>
__global__ __launch_bounds__(64) void k_ic_fwd_wave(Wavefront w, double beta, int32_t *status) {
  constexpr int N = kNatU;
  static_assert(N * kTile <= 64, "a group's face values come in one access of the wavefront");
  __shared__ Rec lx[64], ly[64];
  const int ticket = take_ticket(&w.ticket[0]);
  if (ticket >= w.ntiles) {  // tickets not reset: refuse rather than index out of range
    set_status(status, 8);
    return;
  }
  const int2 tl = w.order[ticket];
  const int tx = __builtin_amdgcn_readfirstlane(tl.x), ty = __builtin_amdgcn_readfirstlane(tl.y);
  const int tile = tx * w.nty + ty, none = w.ntiles;
  const uint32_t lane = threadIdx.x;
  const int la = (int)lane >> 3, lb = (int)lane & 7;
  const bool fx = la == 0, fy = lb == 0;
  const int xsrc = (int)((lane - kTile) & 63u) * 4;
  const int nrow = w.nrow;
  Rec *rows = w.rec + (int64_t)tile * w.trow * 64;
  const int64_t ftile = (int64_t)w.frow * kFaceSlots;
  // the neighbours' faces, 7 steps ahead of this tile's (their upper lanes run 7 steps behind)
  const Rec *xnb = w.ff + (tx > 0 ? tile - w.nty : none) * ftile, *ynb = w.ff + (ty > 0 ? tile - 1 : none) * ftile;
  Rec *out = w.ff + tile * ftile;
  // lane t loads the face values of step t / 8 of a group (lanes past the group: of its last step), column t % 8
  const uint32_t fu = min(lane >> 3, (uint32_t)(N - 1)) * kFaceSlots;
  const uint32_t xs0 = fu + (lane & 7), ys0 = fu + y_slot(lane & 7, kTile - 1);
  const uint32_t so = la == kTile - 1 ? (uint32_t)lb : (lb == kTile - 1 ? (uint32_t)(kTile + la) : kNoSlot);
  const double b2 = beta * beta;
  bool timed_out = false;
  struct Set {
    Rec r[N];   // h and g
    Rec x, y;   // faces: lane t holds slot t % 8 of step t / 8
  };
  auto faces = [&](Set &s, int S0) {
    s.x = face_ld(group_view(xnb + (int64_t)(S0 + kTile - 1) * kFaceSlots), xs0, Rec());
    s.y = face_ld(group_view(ynb + (int64_t)(S0 + kTile - 1) * kFaceSlots), ys0, Rec());
  };
  auto issue = [&](Set &s, int S0) {
    faces(s, S0);
    const auto v = group_view(rows + (int64_t)S0 * 64);
#pragma unroll
    for (int u = 0; u < N; ++u) s.r[u] = view_ld(v, lane + u * 64, Rec());
  };
  // some face value of the set has not been stored yet
  auto empty = [&](const Rec &x, const Rec &y) {
    return __any(max(max(x[1], x[3]), max(y[1], y[3])) == 0xffffffffu);
  };
  auto wait = [&](Set &s, int S0) {
    int spins = 0;
    if (S0 == 0) {  // while a neighbour has not begun it is far off: poll its first row at a distance
      const auto vx = group_view(xnb), vy = group_view(ynb);
      while (empty(face_ld(vx, lane & 7, Rec()), face_ld(vy, y_slot(lane & 7, kTile - 1), Rec())) && ++spins < kSpinLimit) {
        __builtin_amdgcn_s_sleep(8);
        asm volatile("" ::: "memory");  // load anew
      }
    }
    while (empty(s.x, s.y)) {
      if (timed_out || ++spins >= kSpinLimit) {
        if (!timed_out) set_status(status, 8);
        timed_out = true;
        return;
      }
      asm volatile("" ::: "memory");
      faces(s, S0);
    }
  };
  FwdLane<T> st;
  auto compute = [&](const Set &s, int S0) {
    // the loaded face values, step by step, to every lane of their column
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    lx[lane] = s.x;
    ly[lane] = s.y;
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    Rec fxv[N], fyv[N];
#pragma unroll
    for (int u = 0; u < N; ++u) {
      fxv[u] = lx[u * kTile + lb];
      fyv[u] = ly[u * kTile + la];
    }
    const auto v = group_view(rows + (int64_t)S0 * 64), vo = group_view(out + (int64_t)S0 * kFaceSlots);
#pragma unroll
    for (int u = 0; u < N; ++u) {
      const Rec fxr = fxv[u], fyr = fyv[u];
      const Rec o = st.step(fx, fy, xsrc, fxr, fyr, s.r[u], beta, b2);
      face_st(vo, so + u * kFaceSlots, o);
      view_st(v, lane + u * 64, o);
    }
  };
  Set A, B;
  issue(A, 0);
  for (int S0 = 0; S0 < nrow; S0 += 2 * N) {
    wait(A, S0);
    issue(B, S0 + N);
    compute(A, S0);
    wait(B, S0 + N);
    issue(A, S0 + 2 * N);  // past the end: the guard rows
    compute(B, S0 + N);
  }
  if (st.bad) set_status(status, 5);
}

// The mirrored sweep: step B handles row nrow - 1 - B.
template <typename T>
__global__ __launch_bounds__(64) void k_ic_bwd_wave(Wavefront w, double beta, int32_t *status) {
  using U = typename Bits<T>::U;
  constexpr int N = kNatU;
  __shared__ U lx[64], ly[64];
  const int ticket = take_ticket(&w.ticket[1]);
  if (ticket >= w.ntiles) {
    set_status(status, 8);
    return;
  }
  const int2 tl = w.order[w.ntiles - 1 - ticket];  // reverse anti-diagonal order
  const int tx = __builtin_amdgcn_readfirstlane(tl.x), ty = __builtin_amdgcn_readfirstlane(tl.y);
  const int tile = tx * w.nty + ty, none = w.ntiles;
  const uint32_t lane = threadIdx.x;
  const int la = (int)lane >> 3, lb = (int)lane & 7;
  const bool fx = la == kTile - 1, fy = lb == kTile - 1;
  const int xsrc = (int)((lane + kTile) & 63u) * 4;
  const int nrow = w.nrow;
  // a group of rows, the first step's last
  const Rec *rows = w.rec + ((int64_t)tile * w.trow + nrow - N) * 64;
  T *pout = (T *)w.p + ((int64_t)tile * w.trow + nrow - N) * 64;
  const int64_t ftile = (int64_t)w.frow * kFaceSlots;
  const U *xnb = (const U *)w.fp + (tx + 1 < w.ntx ? tile + w.nty : none) * ftile;
  const U *ynb = (const U *)w.fp + (ty + 1 < w.nty ? tile + 1 : none) * ftile;
  U *out = (U *)w.fp + tile * ftile;
  const uint32_t fu = min(lane >> 3, (uint32_t)(N - 1)) * kFaceSlots;
  const uint32_t xs0 = fu + (lane & 7), ys0 = fu + y_slot(lane & 7, 0);
  const uint32_t so = la == 0 ? (uint32_t)lb : (lb == 0 ? (uint32_t)(kTile + la) : kNoSlot);
  bool timed_out = false;
  struct Set {
    Rec r[N];  // 1/P and x of the row before
    U x, y;
  };
  auto faces = [&](Set &s, int B0) {
    s.x = face_ld(group_view(xnb + (int64_t)(B0 + kTile - 1) * kFaceSlots), xs0, U());
    s.y = face_ld(group_view(ynb + (int64_t)(B0 + kTile - 1) * kFaceSlots), ys0, U());
  };
  auto issue = [&](Set &s, int B0) {
    faces(s, B0);
    const auto v = group_view(rows - (int64_t)B0 * 64);
#pragma unroll
    for (int u = 0; u < N; ++u) s.r[u] = view_ld(v, lane + (N - 1 - u) * 64, Rec());
  };
  auto empty = [&](U x, U y) { return __any(max(top_word(x), top_word(y)) == 0xffffffffu); };
  auto wait = [&](Set &s, int B0) {  // as forward
    int spins = 0;
    if (B0 == 0) {
      const auto vx = group_view(xnb), vy = group_view(ynb);
      while (empty(face_ld(vx, lane & 7, U()), face_ld(vy, y_slot(lane & 7, 0), U())) && ++spins < kSpinLimit) {
        __builtin_amdgcn_s_sleep(8);
        asm volatile("" ::: "memory");
      }
    }
    while (empty(s.x, s.y)) {
      if (timed_out || ++spins >= kSpinLimit) {
        if (!timed_out) set_status(status, 8);
        timed_out = true;
        return;
      }
      asm volatile("" ::: "memory");
      faces(s, B0);
    }
  };
  BwdLane<T> st;
  auto compute = [&](const Set &s, int B0) {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    lx[lane] = s.x;
    ly[lane] = s.y;
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    U fxr[N], fyr[N];
#pragma unroll
    for (int u = 0; u < N; ++u) {
      fxr[u] = lx[u * kTile + lb];
      fyr[u] = ly[u * kTile + la];
    }
    const auto v = group_view(pout - (int64_t)B0 * 64), vo = group_view(out + (int64_t)B0 * kFaceSlots);
#pragma unroll
    for (int u = 0; u < N; ++u) {
      const T p = st.step(fx, fy, xsrc, fxr[u], fyr[u], s.r[u], beta);
      face_st(vo, so + u * kFaceSlots, __builtin_bit_cast(U, p));
      view_st(v, lane + (N - 1 - u) * 64, p);
    }
  };
  Set A, B;
  issue(A, 0);
  for (int B0 = 0; B0 < nrow; B0 += 2 * N) {
    wait(A, B0);
    issue(B, B0 + N);
    compute(A, B0);
    wait(B, B0 + N);
    issue(A, B0 + 2 * N);
    compute(B, B0 + N);
  }
}

// ---------------------------------------------------------------------------
// IC(0) in block red-black order: the tiles of one colour ((ti + tj) mod 2,
// colour 0 first) share no face, and inside a tile the order is natural, so
// one launch sweeps every tile of a colour at once, one wavefront per tile as
// above, with no waits between tiles.  A voxel's earlier neighbours are its
// in-tile -x, -y, -z neighbours and, in a colour-1 tile, every neighbour
// across a tile face (colour 0, factored by the previous launch); its later
// neighbours are the in-tile +x, +y, +z ones and, in a colour-0 tile, every
// neighbour across a face.  Forward: colour 0, then colour 1; backward:
// colour 1, then colour 0.  (128x128x64 MIX, per launch: 11.3 and 16.8 us
// forward, 8.4 and 8.9 us backward; 27.7 and 30.1 us with masks, address
// arithmetic and dot products in the step.)  A lane reads the column across its x face and the
// one across its y face from that tile's packed rows (7 steps ahead for a lower
// face, 7 behind for an upper one); a lane without one reads the tile that holds 0.
struct BlockFaces {
  int64_t x, y;  // element of the lane's column in row 0 of the tile across, at this tile's row 0
};
__device__ __forceinline__ BlockFaces block_faces(const Wavefront &w, int2 t, int la, int lb) {
  const int64_t none = (int64_t)w.ntiles * w.trow * 64 + (int)threadIdx.x;
  auto at = [&](int tx, int ty, int a, int b, int rows) {
    return tx >= 0 && tx < w.ntx && ty >= 0 && ty < w.nty
               ? ((int64_t)(tx * w.nty + ty) * w.trow + rows) * 64 + a * kTile + b
               : none;
  };
  constexpr int K = kTile - 1;
  BlockFaces f{none, none};
  if (la == 0) f.x = at(t.x - 1, t.y, K, lb, K);
  if (la == K) f.x = at(t.x + 1, t.y, 0, lb, -K);
  if (lb == 0) f.y = at(t.x, t.y - 1, la, K, K);
  if (lb == K) f.y = at(t.x, t.y + 1, la, 0, -K);
  return f;
}

template <typename T, bool FACES>
__global__ __launch_bounds__(64) void k_icb_fwd(Wavefront w, double beta, int32_t *status, int colour) {
  constexpr int N = kNatU;
  const int2 tl = w.blk[colour][blockIdx.x];
  const int tx = __builtin_amdgcn_readfirstlane(tl.x), ty = __builtin_amdgcn_readfirstlane(tl.y);
  const uint32_t lane = threadIdx.x;
  const int la = (int)lane >> 3, lb = (int)lane & 7;
  const bool fx = la == 0, fy = lb == 0;
  const int xsrc = (int)((lane - kTile) & 63u) * 4;
  const int nrow = w.nrow;
  Rec *rows = w.rec + (int64_t)(tx * w.nty + ty) * w.trow * 64;
  const BlockFaces f = block_faces(w, tl, la, lb);
  const Rec *xr = w.rec + f.x, *yr = w.rec + f.y;
  const double b2 = beta * beta;
  struct Set {
    Rec r[N], x[FACES ? N : 1], y[FACES ? N : 1];
  };
  auto issue = [&](Set &s, int S0) {
    const auto v = group_view(rows + (int64_t)S0 * 64);
#pragma unroll
    for (int u = 0; u < N; ++u) {
      s.r[u] = view_ld(v, lane + u * 64, Rec());
      if constexpr (FACES) {
        s.x[u] = xr[(int64_t)(S0 + u) * 64];
        s.y[u] = yr[(int64_t)(S0 + u) * 64];
      }
    }
  };
  FwdLane<T, true> st;
  auto compute = [&](const Set &s, int S0) {
    const auto v = group_view(rows + (int64_t)S0 * 64);
#pragma unroll
    for (int u = 0; u < N; ++u) {
      const Rec zero = {0u, 0u, 0u, 0u};
      view_st(v, lane + u * 64, st.step(fx, fy, xsrc, FACES ? s.x[FACES ? u : 0] : zero, FACES ? s.y[FACES ? u : 0] : zero,
                                        s.r[u], beta, b2));
    }
  };
  Set A, B;
  issue(A, 0);
  for (int S0 = 0; S0 < nrow; S0 += 2 * N) {
    issue(B, S0 + N);
    compute(A, S0);
    issue(A, S0 + 2 * N);  // past the end: rows that are read and not used
    compute(B, S0 + N);
  }
  if (st.bad) set_status(status, 5);
}

template <typename T, bool FACES>
__global__ __launch_bounds__(64) void k_icb_bwd(Wavefront w, double beta, int colour) {
  using U = typename Bits<T>::U;
  constexpr int N = kNatU;
  const int2 tl = w.blk[colour][blockIdx.x];
  const int tx = __builtin_amdgcn_readfirstlane(tl.x), ty = __builtin_amdgcn_readfirstlane(tl.y);
  const uint32_t lane = threadIdx.x;
  const int la = (int)lane >> 3, lb = (int)lane & 7;
  const bool fx = la == kTile - 1, fy = lb == kTile - 1;
  const int xsrc = (int)((lane + kTile) & 63u) * 4;
  const int nrow = w.nrow;
  const int64_t last = ((int64_t)(tx * w.nty + ty) * w.trow + nrow - N) * 64;  // the first group's rows
  const Rec *rows = w.rec + last;
  T *pout = (T *)w.p + last;
  const BlockFaces f = block_faces(w, tl, la, lb);
  const U *xp = (const U *)w.p + f.x + (int64_t)(nrow - 1) * 64, *yp = (const U *)w.p + f.y + (int64_t)(nrow - 1) * 64;
  struct Set {
    Rec r[N];
    U x[FACES ? N : 1], y[FACES ? N : 1];
  };
  auto issue = [&](Set &s, int B0) {
    const auto v = group_view(rows - (int64_t)B0 * 64);
#pragma unroll
    for (int u = 0; u < N; ++u) {
      s.r[u] = view_ld(v, lane + (N - 1 - u) * 64, Rec());
      if constexpr (FACES) {
        s.x[u] = xp[-(int64_t)(B0 + u) * 64];
        s.y[u] = yp[-(int64_t)(B0 + u) * 64];
      }
    }
  };
  BwdLane<T, true> st;
  auto compute = [&](const Set &s, int B0) {
    const auto v = group_view(pout - (int64_t)B0 * 64);
#pragma unroll
    for (int u = 0; u < N; ++u)
      view_st(v, lane + (N - 1 - u) * 64,
              st.step(fx, fy, xsrc, FACES ? s.x[FACES ? u : 0] : U(0), FACES ? s.y[FACES ? u : 0] : U(0), s.r[u], beta));
  };
  Set A, B;
  issue(A, 0);
  for (int B0 = 0; B0 < nrow; B0 += 2 * N) {
    issue(B, B0 + N);
    compute(A, B0);
    issue(A, B0 + 2 * N);
    compute(B, B0 + N);
  }
}
#undef FM_STAGE

}  // namespace fm
