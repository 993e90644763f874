// Plane-marching tiles of the red-black passes (even column lengths).
//
// A workgroup owns a strip of ty whole columns (all of z) and walks a run of
// xc planes along x.  Per plane, thread slots hold voxel pairs (z even,
// z odd): one black and one red voxel, the black one first when x + y is odd.
// A voxel's six neighbours all have the other colour; they come from
//   -x, +x  the same slot one plane back / ahead, kept in registers as the
//           strip marches, so each plane is fetched once per strip;
//   -y, +y  an LDS copy of the plane's values of that colour, with one halo
//           column on each side of the strip, loaded by the first nz threads;
//   -z, +z  the pair's partner and the neighbouring pair's voxel (LDS).
// The arithmetic, the neighbour order and the outputs are those of
// k_rb_black_pair and k_rb_red_dir_pair; only the order in which voxels add
// to the partial sums differs.  Planes are fetched kTileDepth ahead into a
// ring of registers, so that loads are in flight across the barrier and the
// arithmetic of the planes before them: the passes are bound by the bytes in
// flight.  The ring holds the loads as they come and is indexed at compile
// time (the march is unrolled over its slots): a select on a value or a move
// of it would wait for the load just issued, and a load under a condition
// makes every later wait a full one.  The LDS copy alternates between two
// buffers, so one barrier per plane suffices.  One pair slot per thread and
// two planes ahead keep FP32 at 4 waves per SIMD, all that the partial sums'
// 1024 workgroups fill.  256x256x128 MIX: black 48.6 -> 40 us, red and
// direction 49.8 -> 39 us (20.8 and 29.1 B a voxel across the L2 by the traffic
// counters, 4.4 and 6.2 TB/s); with waits for the newest load the red pass was at 57 us.
#pragma once

#include "fm_stream.hpp"

namespace fm {

constexpr int kTileDepth = 2;               // planes fetched ahead of the current one
constexpr int kTileRing = 4;                // ring slots (even: the LDS buffer of a plane follows from its slot)
constexpr int kTileSlots = kNT;             // pair slots of a workgroup per plane, one per thread
constexpr int kTileMaxNz = kNT;             // the two halo columns hold nz pairs, one per thread
constexpr int kTileLds = kTileSlots + kTileMaxNz;  // LDS entries per buffer, halo included

// Plane-march shape of a volume: columns per strip, planes per run, strips, grid.
struct TileShape {
  int ty, xc, nyt, grid;
};

// The shape a batched volume's descriptor holds.
__device__ __forceinline__ TileShape tile_of(const VolDesc &d) { return TileShape{d.tty, d.txc, d.tnyt, 0}; }

// A workgroup's strip and run, and this thread's slots in them.
struct TileSlots {
  int x0, x1, nzp; // planes of the run, pairs of a column
  int xl;          // last plane to fetch: one past the run (the +x neighbours) if the volume has it
  int base;        // pair index, in a plane, of column y0 - 1's first pair
  int y, zq;       // column and pair of the thread's slot
  int e;           // its LDS entry, and its pair counted from column y0 - 1
  uint32_t l;      // the pair it loads (a slot without a column: one of column y0)
  bool ok;         // the column is the strip's and in the volume
  int he;          // LDS entry of the halo slot: column 0 (y0 - 1) or ty + 1 (y0 + ty)
  int hy;          // its column
  uint32_t hl;     // the pair it loads
  bool hs;         // this thread holds a halo slot
};

// Workgroups are dealt to the chip's XCDs in turn (workgroup i to XCD i mod
// kXcds), each with its own L2.  The tile index is remapped so that every XCD
// owns a contiguous range of strips and runs: the halo columns and planes a
// workgroup shares with its neighbours are then fetched into the same L2.
constexpr int kXcds = 8;

// Workgroup bl of the nb a volume has (a batched launch may give a volume more
// workgroups than its tiles: the surplus ones own no plane and only take part
// in the partial sums).  The XCD remap applies where the volume's workgroups
// start at a multiple of kXcds and come in multiples of it.
__device__ __forceinline__ TileSlots tile_slots(const Geo &g, const TileShape &ts, int bl, int nb, int b0) {
  TileSlots t;
  t.nzp = g.nz >> 1;
  if (nb % kXcds == 0 && b0 % kXcds == 0) bl = (bl % kXcds) * (nb / kXcds) + bl / kXcds;
  const int y0 = (bl % ts.nyt) * ts.ty;
  t.x0 = (bl / ts.nyt) * ts.xc;
  const bool run = t.x0 < g.nx;
  t.x1 = !run ? t.x0 : (t.x0 + ts.xc < g.nx ? t.x0 + ts.xc : g.nx);
  t.xl = t.x1 < g.nx ? t.x1 : g.nx - 1;
  const int cy = (int)threadIdx.x / t.nzp;
  t.zq = (int)threadIdx.x - cy * t.nzp;
  t.ok = run && cy < ts.ty && y0 + cy < g.ny;
  t.base = (y0 - 1) * t.nzp;
  t.y = t.ok ? y0 + cy : y0;
  t.e = (cy + 1) * t.nzp + t.zq;
  t.l = (uint32_t)(t.ok ? t.e : t.nzp + t.zq);
  t.hs = cy < 2;
  const int hy = cy == 0 ? y0 - 1 : y0 + ts.ty;
  t.hy = hy >= 0 && hy < g.ny ? hy : y0;  // a column outside the volume: no voxel has it as a neighbour
  t.he = (cy == 0 ? 0 : ts.ty + 1) * t.nzp + t.zq;
  t.hl = (uint32_t)(t.hs ? (t.hy - y0 + 1) * t.nzp + t.zq : t.nzp);  // without a halo slot: one line for all
  return t;
}

// Pair i of an array counted from a base that is the same for all lanes: the
// address is that base in scalar registers plus one 32-bit offset per lane, which
// a strip's pairs share between arrays and planes (64-bit addresses per lane and
// array took the kernels from 4 waves per SIMD to 2 or 3).
template <typename E>
__device__ __forceinline__ E ld_pair(const void *base, uint32_t i) {
  return *reinterpret_cast<const E *>(static_cast<const char *>(base) + i * (uint32_t)sizeof(E));
}

// March over the workgroup's planes with the ring slot of a plane known at
// compile time: step(slot, x) for x = x0 .. x1 - 1, slot = (x - x0) mod kTileRing.
template <int S>
struct RingSlot {
  static constexpr int v = S;
};
template <int S, typename F>
__device__ __forceinline__ void tile_march_from(int x, int x1, F &step) {
  if constexpr (S < kTileRing) {
    if (x < x1) {
      step(RingSlot<S>{}, x);
      tile_march_from<S + 1>(x + 1, x1, step);
    }
  }
}
template <typename F>
__device__ __forceinline__ void tile_march(int x0, int x1, F &&step) {
  for (int x = x0; x < x1; x += kTileRing) tile_march_from<0>(x, x1, step);
}

// ---------------------------------------------------------------------------
// Black pass (Sec. III-B, the black half of the red-black IC(0) factor and its
// forward/backward solve): p_b for every black voxel from its six red
// neighbours' g, g_prev and 1/h, plus the partial sums of g^T p and
// g_prev^T p over all voxels.

template <typename T>
struct TileB {  // one slot's pair on one plane, first voxel (z even) first
  uint32_t c2;  // both codes (first voxel in the low byte)
  Duo<T> g, gp;
  T db;         // D of the black voxel
  double hr;    // 1/h of the red voxel
};

template <typename T>
struct TileBH {  // a halo pair's red voxel
  T gr, gpr;
  double hr;
};

// o: the pair index of column y0 - 1 of the plane; fb: the pair's first voxel is black.
template <typename T>
__device__ __forceinline__ void tile_b_load(TileB<T> &t, const VArgs<T> &a, int o, uint32_t l, bool fb) {
  t.c2 = ld_pair<uint16_t>(a.code + 2 * (int64_t)o, l);
  t.g = ld_pair<Duo<T>>(a.Gc + 2 * (int64_t)o, l);
  t.gp = ld_pair<Duo<T>>(a.Gp + 2 * (int64_t)o, l);
  t.db = ld_pair<T>(a.D + 2 * (int64_t)o, 2 * l + (fb ? 0 : 1));
  t.hr = ld_pair<double>(a.hinv + o, l);
}

template <typename T>
__device__ __forceinline__ void tile_b_halo(TileBH<T> &t, const VArgs<T> &a, int o, uint32_t l, bool fb) {
  const uint32_t r = 2 * l + (fb ? 1 : 0);
  t.gr = ld_pair<T>(a.Gc + 2 * (int64_t)o, r);
  t.gpr = ld_pair<T>(a.Gp + 2 * (int64_t)o, r);
  t.hr = ld_pair<double>(a.hinv + o, l);
}

// The pair's voxel that comes first in z (first) or second.
template <typename T>
__device__ __forceinline__ T of_pair(const Duo<T> &d, bool first) {
  return first ? d.v0 : d.v1;
}

template <typename T, bool BATCH>
__global__ __launch_bounds__(kNT) void k_rb_black_tile(IterArgs<T> a0, TileShape ts) {
  __shared__ double lh[2][kTileLds];
  __shared__ T lg[2][kTileLds], lgp[2][kTileLds];
  const VolView vw = vol_view<BATCH>(a0);
  const VArgs<T> a = at_volume<BATCH>(a0, vw);
  const Geo g = a.geo;
  const TileSlots t = tile_slots(g, BATCH ? tile_of(a0.bt.vol[vw.vol]) : ts, vw.bl, vw.nb, BATCH ? vw.pfirst : 0);
  const int nzp = t.nzp, sp2 = (int)(g.sx >> 1);  // pairs of a column, of a plane
  TileB<T> q[kTileRing];
  TileBH<T> hq[kTileRing];
  T prg = T(0), prgp = T(0);  // red g, g_prev, 1/h one plane back
  double prh = 0.0;
  if (t.x0 < t.x1) {  // planes x0 - 1 .. x0 + kTileDepth - 1
    const bool fb = ((t.x0 + t.y) & 1) != 0;
    const int xp = t.x0 > 0 ? t.x0 - 1 : 0;
    TileBH<T> pv;
    tile_b_halo(pv, a, xp * sp2 + t.base, t.l, !fb);
    prg = pv.gr;
    prgp = pv.gpr;
    prh = pv.hr;
#pragma unroll
    for (int d = 0; d < kTileDepth; ++d) {
      const int x = t.x0 + d < t.xl ? t.x0 + d : t.xl;
      tile_b_load(q[d], a, x * sp2 + t.base, t.l, ((x + t.y) & 1) != 0);
      tile_b_halo(hq[d], a, x * sp2 + t.base, t.hl, ((x + t.hy) & 1) != 0);
    }
  }
  const State st = take_state<kNT, 4>(a.sin, a.pin, a.nparts_in, a.nvals_in, a.beta, a.trace, a.status, vw.prow,
                                      vw.leader);
  put_state(st, a.sout, PK_DOTS, vw.nb, vw.leader);
  const double beta = a.beta, b2 = a.beta * a.beta;
  double acc[2] = {0.0, 0.0};
  int bad = 0;
  tile_march(t.x0, t.x1, [&](auto slot, int x) {
    constexpr int S = decltype(slot)::v, SN = (S + 1) % kTileRing, SF = (S + kTileDepth) % kTileRing, b = S & 1;
    const TileB<T> &c = q[S], &n = q[SN];
    const bool fb = ((x + t.y) & 1) != 0;  // the pair's first voxel is black
    const T gr = of_pair(c.g, !fb), gpr = of_pair(c.gp, !fb);
    if (t.ok) {
      lg[b][t.e] = gr;
      lgp[b][t.e] = gpr;
      lh[b][t.e] = c.hr;
    }
    if (t.hs) {
      lg[b][t.he] = hq[S].gr;
      lgp[b][t.he] = hq[S].gpr;
      lh[b][t.he] = hq[S].hr;
    }
    // Plane x + kTileDepth is in flight during the barriers and arithmetic before it.  Every
    // lane loads on every plane (past the run the last plane again): a load that may be
    // skipped leaves the count of loads in flight unknown, and the waits become full ones.
    const int xf = x + kTileDepth < t.xl ? x + kTileDepth : t.xl;
    tile_b_load(q[SF], a, xf * sp2 + t.base, t.l, ((xf + t.y) & 1) != 0);
    tile_b_halo(hq[SF], a, xf * sp2 + t.base, t.hl, ((xf + t.hy) & 1) != 0);
    __syncthreads();
    const uint32_t cv = fb ? (c.c2 & 0xffu) : (c.c2 >> 8), cr = fb ? (c.c2 >> 8) : (c.c2 & 0xffu);
    if (t.ok && (cr & NB_SELF)) {
      const double gh = (double)gr * c.hr;
      acc[0] += (double)gr * gh;
      acc[1] += (double)gpr * gh;
    }
    if (t.ok && (cv & NB_SELF)) {
      const int e = t.e;
      // the red voxel of the plane after has the black one's place in the pair
      // -z / +z: the previous pair's red voxel and the partner (black first),
      // or the partner and the next pair's red voxel (red first)
      const int ez = fb ? (t.zq > 0 ? e - 1 : e) : (t.zq + 1 < nzp ? e + 1 : e);
      const double hz = lh[b][ez], hc = c.hr;
      const T gz = lg[b][ez], gpz = lgp[b][ez];
      const double hn[6] = {prh, n.hr, lh[b][e - nzp], lh[b][e + nzp], fb ? hz : hc, fb ? hc : hz};
      const T gn[6] = {prg, of_pair(n.g, fb), lg[b][e - nzp], lg[b][e + nzp], fb ? gz : gr, fb ? gr : gz};
      const T gpn[6] = {prgp, of_pair(n.gp, fb), lgp[b][e - nzp], lgp[b][e + nzp], fb ? gpz : gpr, fb ? gpr : gpz};
      const double h = (double)c.db + beta * nb_deg(cv);
      double sp = 0.0, sxv = 0.0, syp = 0.0;
#pragma unroll
      for (int k = 0; k < 6; ++k)
        if (has_nb(cv, k)) {
          sp += hn[k];
          sxv += (double)gn[k] * hn[k];
          syp += (double)gpn[k] * hn[k];
        }
      const double piv = h - b2 * sp;
      double ip = 1.0 / piv;
      if (!(piv > 0.0)) {
        bad = 1;
        ip = 0.0;
      }
      const double yb = (double)of_pair(c.g, fb) + beta * sxv;
      const double xv = yb * ip;
      a.P[x * sp2 + t.base + e] = (T)xv;
      acc[0] += yb * xv;
      acc[1] += ((double)of_pair(c.gp, fb) + beta * syp) * xv;
    }
    prg = gr;
    prgp = gpr;
    prh = c.hr;
  });
  if (bad) set_status(a.status, 5);
  store_partials<2, kNT>(acc, a.pout);
}

// ---------------------------------------------------------------------------
// Red pass fused with the direction (Sec. III-B, the red half of the backward
// solve; Sec. III eq. (ncg) for z; the line-search setup sums): p_r from the
// six black neighbours' p, then z = -p + mu z_prev for both voxels of the
// pair, and the partial sums of z^T C^T C f, ||C z||^2 and z^T D z.

template <typename T>
struct TileR {  // one slot's pair on one plane, first voxel (z even) first
  uint32_t c2;  // both codes (first voxel in the low byte)
  Duo<T> z, f, d;  // z_prev, f, D
  T pb, gr;     // p of the black, g of the red voxel
  double hr;    // 1/h of the red voxel
};

template <typename T>
struct TileRH {  // a halo pair's black voxel
  T pb, zb, fb;
};

// What the planes beside it need of a plane, and what only its own step does: the
// latter is fetched one plane ahead (six registers fewer, which keeps FP32 at 4 waves).
template <typename T>
__device__ __forceinline__ void tile_r_near(TileR<T> &t, const VArgs<T> &a, int o, uint32_t l) {
  t.z = ld_pair<Duo<T>>(a.Zp + 2 * (int64_t)o, l);
  t.f = ld_pair<Duo<T>>(a.Fc + 2 * (int64_t)o, l);
  t.pb = ld_pair<T>(a.P + o, l);
}

template <typename T>
__device__ __forceinline__ void tile_r_own(TileR<T> &t, const VArgs<T> &a, int o, uint32_t l, bool fb) {
  t.c2 = ld_pair<uint16_t>(a.code + 2 * (int64_t)o, l);
  t.d = ld_pair<Duo<T>>(a.D + 2 * (int64_t)o, l);
  t.gr = ld_pair<T>(a.Gc + 2 * (int64_t)o, 2 * l + (fb ? 1 : 0));
  t.hr = ld_pair<double>(a.hinv + o, l);
}

template <typename T>
__device__ __forceinline__ void tile_r_halo(TileRH<T> &t, const VArgs<T> &a, int o, uint32_t l, bool fb) {
  const uint32_t k = 2 * l + (fb ? 0 : 1);
  t.zb = ld_pair<T>(a.Zp + 2 * (int64_t)o, k);
  t.fb = ld_pair<T>(a.Fc + 2 * (int64_t)o, k);
  t.pb = ld_pair<T>(a.P + o, l);
}

template <typename T, bool BATCH>
__global__ __launch_bounds__(kNT) void k_rb_red_dir_tile(IterArgs<T> a0, TileShape ts) {
  __shared__ T lp[2][kTileLds], lz[2][kTileLds], lf[2][kTileLds];
  const VolView vw = vol_view<BATCH>(a0);
  const VArgs<T> a = at_volume<BATCH>(a0, vw);
  const Geo g = a.geo;
  const TileSlots t = tile_slots(g, BATCH ? tile_of(a0.bt.vol[vw.vol]) : ts, vw.bl, vw.nb, BATCH ? vw.pfirst : 0);
  const int nzp = t.nzp, sp2 = (int)(g.sx >> 1);  // pairs of a column, of a plane
  TileR<T> q[kTileRing];
  TileRH<T> hq[kTileRing];
  T prp = T(0), prz = T(0), prf = T(0);  // black p, z_prev, f one plane back
  if (t.x0 < t.x1) {  // planes x0 - 1 .. x0 + kTileDepth - 1
    const bool fb = ((t.x0 + t.y) & 1) != 0;
    const int xp = t.x0 > 0 ? t.x0 - 1 : 0;
    TileRH<T> pv;
    tile_r_halo(pv, a, xp * sp2 + t.base, t.l, !fb);
    prp = pv.pb;
    prz = pv.zb;
    prf = pv.fb;
#pragma unroll
    for (int d = 0; d < kTileDepth; ++d) {
      const int x = t.x0 + d < t.xl ? t.x0 + d : t.xl;
      tile_r_near(q[d], a, x * sp2 + t.base, t.l);
      if (d == 0) tile_r_own(q[d], a, x * sp2 + t.base, t.l, ((x + t.y) & 1) != 0);
      tile_r_halo(hq[d], a, x * sp2 + t.base, t.hl, ((x + t.hy) & 1) != 0);
    }
  }
  const State st = take_state<kNT, 2>(a.sin, a.pin, a.nparts_in, a.nvals_in, a.beta, a.trace, a.status, vw.prow,
                                      vw.leader);
  put_state(st, a.sout, PK_DIR, vw.nb, vw.leader);
  const double beta = a.beta;
  const T mu = (T)st.mu;
  double acc[3] = {0.0, 0.0, 0.0};
  int bad = 0;
  tile_march(t.x0, t.x1, [&](auto slot, int x) {
    constexpr int S = decltype(slot)::v, SN = (S + 1) % kTileRing, SF = (S + kTileDepth) % kTileRing, b = S & 1;
    const TileR<T> &c = q[S], &n = q[SN];
    const bool fb = ((x + t.y) & 1) != 0;  // the pair's first voxel is black
    const T zb = of_pair(c.z, fb), fbk = of_pair(c.f, fb);
    if (t.ok) {
      lp[b][t.e] = c.pb;
      lz[b][t.e] = zb;
      lf[b][t.e] = fbk;
    }
    if (t.hs) {
      lp[b][t.he] = hq[S].pb;
      lz[b][t.he] = hq[S].zb;
      lf[b][t.he] = hq[S].fb;
    }
    const int xf = x + kTileDepth < t.xl ? x + kTileDepth : t.xl;
    const int xn = x + 1 < t.xl ? x + 1 : t.xl;
    tile_r_near(q[SF], a, xf * sp2 + t.base, t.l);
    tile_r_own(q[SN], a, xn * sp2 + t.base, t.l, ((xn + t.y) & 1) != 0);
    tile_r_halo(hq[SF], a, xf * sp2 + t.base, t.hl, ((xf + t.hy) & 1) != 0);
    __syncthreads();
    if (t.ok) {
      const uint32_t cb = fb ? (c.c2 & 0xffu) : (c.c2 >> 8), cv = fb ? (c.c2 >> 8) : (c.c2 & 0xffu);
      T zrv = T(0), zbv = T(0);
      if (cv & NB_SELF) {
        const int e = t.e;
        const T fr = of_pair(c.f, !fb);
        // the black voxel of the plane after has the red one's place in the pair
        // -z / +z: the partner and the next pair's black voxel (black first),
        // or the previous pair's black voxel and the partner (red first)
        const int ez = fb ? (t.zq + 1 < nzp ? e + 1 : e) : (t.zq > 0 ? e - 1 : e);
        // (values, not a choice between two addresses: that would put the ring in memory)
        const T pz = lp[b][ez], zz = lz[b][ez], fz = lf[b][ez], pc = c.pb;
        const T pn[6] = {prp, n.pb, lp[b][e - nzp], lp[b][e + nzp], fb ? pc : pz, fb ? pz : pc};
        const T zn[6] = {prz, of_pair(n.z, !fb), lz[b][e - nzp], lz[b][e + nzp], fb ? zb : zz, fb ? zz : zb};
        const T fn[6] = {prf, of_pair(n.f, !fb), lf[b][e - nzp], lf[b][e + nzp], fb ? fbk : fz, fb ? fz : fbk};
        double sp = 0.0;
#pragma unroll
        for (int k = 0; k < 6; ++k)
          if (has_nb(cv, k)) sp += (double)pn[k];
        const double ip = c.hr;
        if (!(ip > 0.0)) bad = 1;
        const T pj = (T)((double)c.gr * ip + beta * sp * ip);
        zrv = -pj + mu * of_pair(c.z, !fb);
        acc[2] += (double)zrv * (double)zrv * (double)of_pair(c.d, !fb);
#pragma unroll
        for (int k = 0; k < 6; ++k)
          if (has_nb(cv, k)) {
            const double dz = (double)(zrv - (-pn[k] + mu * zn[k]));
            acc[0] += dz * (double)(fr - fn[k]);
            acc[1] += dz * dz;
          }
      }
      if (cb & NB_SELF) {
        zbv = -c.pb + mu * zb;
        acc[2] += (double)zbv * (double)zbv * (double)of_pair(c.d, fb);
      }
      Duo<T> out;
      out.v0 = fb ? zbv : zrv;
      out.v1 = fb ? zrv : zbv;
      *reinterpret_cast<Duo<T> *>(a.Zc + 2 * (x * sp2 + t.base + t.e)) = out;
    }
    prp = c.pb;
    prz = zb;
    prf = fbk;
  });
  if (bad) set_status(a.status, 5);
  store_partials<3, kNT>(acc, a.pout);
}

}  // namespace fm
