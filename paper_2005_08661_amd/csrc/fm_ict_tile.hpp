// IC_t in one launch per sweep (fill levels 0 and 1): the factorisation and the
// forward solve, and the backward solve, as pipelined wavefronts of tiles.
//
// A launch per level of the schedule of fm_ict.hpp takes 699 launches a sweep at
// 128x128x64, each a chain of scattered loads that waits for the last one (3.0
// and 2.8 ms).  Here, as in fm_natural.hpp, a wavefront sweeps 64 columns step by
// step, tiles hand their face values on through memory, and a pass before and
// one after lay the arrays out in step order.
//
// Tiles.  The level-1 pattern has the entry (1, -1, 0), so square tiles in (x, y)
// would depend on each other both ways.  In the sheared coordinate y' = y + K x
// (K the fill level) every offset of the pattern has dx >= 0 and dy' >= 0: tile
// (ti, c) holds columns x = 8 ti + a, y = 8 c + b - K a (lane (a, b)), and depends
// on (ti - 1, c + K), (ti, c - 1) and (ti - 1, c + K - 1) only.  Lane (a, b) at
// step S handles z = S - a - (K + 1) b, so offset o of the pattern was w(o) = dx +
// (K + 1) dy' + dz >= 1 steps earlier.  (Level 2 reaches two columns across a face
// and seven steps back; it keeps the launch per level.)
//
// Values of other lanes come from a ring of the last steps in LDS, one column of
// positions wider than the tile on its -x and -y sides, where the faces of the
// neighbour tiles are written as they arrive.  A position without a voxel holds
// what leaves every sum as it is: L_kk = 1, no entries, y = p = 0 and an infinite
// drop threshold, by which a row drops its entry there (a NaN is dropped too).  A
// lane without a voxel selects y and p (not products with zero: a NaN or an infinity
// must not cross the mask); it knows itself by the sign of its -beta, which is +0,
// and backward by 1/L_jj = 0.  No masks, as there.
//
// The arithmetic is that of fm_ict.hpp, each product rounded before it is
// subtracted.  Quotients are formed from the reciprocal of L_kk that its row
// leaves, with the remainder's correction that makes them the correctly rounded
// ones (Markstein, Computation of elementary functions on the IBM RISC System/6000
// processor, IBM J. Res. Dev. 34, 1990), in 3 operations instead of a division.
// An infinite L_kk stands as the largest finite number with the reciprocal 0, by
// which every quotient is 0; y and p take an infinite numerator through v_div_fixup.
//
// Measured at 128x128x64 (MIX, level 1): forward 3.0 ms -> 497 us, backward 2.8 ms
// -> 330 us a sweep, k_ict_pack 19 us and k_ict_unpack 14 us on top.  A step takes
// 0.48 us forward and 0.30 us backward, of which the issue of its nine 16-byte
// stores is a good part: stored while the next step's LDS reads are under way they
// cost 613 -> 500 us, and the face values stored ahead of that instead (a shorter
// hop, a longer step) measured 530 us.
#pragma once

#include "fm_ict.hpp"
#include "fm_natural.hpp"

namespace fm {

constexpr int kIctU = 4;      // steps per group: two register sets of face values, and a ring of 8 steps in LDS
constexpr int kIctRing = 8;
constexpr double kIctInf = 0x1.fffffffffffffp+1023;  // an infinite L_jj (a finite one is below 2^512)
constexpr int kIctPos = 81;   // ring positions of a step: (a + 1) * 9 + b + 1 of the 8x8 columns and their halo

// Offset u of the pattern in the sheared coordinates, and the steps back to it.
template <int LEVEL>
__host__ __device__ constexpr int ict_dy(int u) {
  return IctPattern<LEVEL>::off[u][1] + LEVEL * IctPattern<LEVEL>::off[u][0];
}
template <int LEVEL>
__host__ __device__ constexpr int ict_back(int u) {
  return IctPattern<LEVEL>::off[u][0] + (LEVEL + 1) * ict_dy<LEVEL>(u) + IctPattern<LEVEL>::off[u][2];
}
template <int LEVEL>
__host__ __device__ constexpr bool ict_own(int u) {  // the lane's own column
  return IctPattern<LEVEL>::off[u][0] == 0 && IctPattern<LEVEL>::off[u][1] == 0;
}
template <int LEVEL>
__host__ __device__ constexpr bool ict_stencil(int u) {  // an entry of H itself
  return IctPattern<LEVEL>::off[u][0] + IctPattern<LEVEL>::off[u][1] + IctPattern<LEVEL>::off[u][2] == 1 &&
         IctPattern<LEVEL>::off[u][0] >= 0 && IctPattern<LEVEL>::off[u][1] >= 0 && IctPattern<LEVEL>::off[u][2] >= 0;
}
// Row entries that other lanes' rows multiply by, and their place in a step's
// values after L_kk, 1/L_kk, y and the threshold.
template <int LEVEL>
__host__ __device__ constexpr bool ict_shared(int e) {
  for (int u = 0; u < IctPattern<LEVEL>::n; ++u)
    for (int v = 0; v < u; ++v)
      if (!ict_own<LEVEL>(u) && ict_pair<LEVEL>(u, v) == e) return true;
  return false;
}
template <int LEVEL>
__host__ __device__ constexpr int ict_field(int e) {
  int f = 4;
  for (int k = 0; k < e; ++k) f += ict_shared<LEVEL>(k) ? 1 : 0;
  return f;
}

template <int LEVEL>
struct IctTile {
  static constexpr int K = LEVEL, n = IctPattern<LEVEL>::n;
  static constexpr int skew = 7 + 7 * (K + 1);       // steps between the first and the last lane of a tile
  static constexpr int nf = ict_field<LEVEL>(n);     // values of a step in the forward ring
  static constexpr int fr = (nf + 1) / 2;            // 16-byte records of a face value, forward
  static constexpr int nb = n - 1;                   // products L_ij p_i for other lanes
  static constexpr int br = (nb + 1) / 2;            // records of a face value, backward
  static constexpr int planes = 2 + (n + 1) / 2;     // 16-byte planes of the packed rows
  static_assert(n <= 6 && nf <= 8, "");
};

// Device tables of the tiled sweeps.
struct IctSweep {
  const int2 *order;   // [ntiles] tiles (ti, c), by first step
  int32_t ntx, nty, ntiles;
  int32_t nrow, frow;  // rows of a sweep, and of a tile's face buffers
  uint32_t *ticket;    // [2]
  // packed rows [ntiles][nrow][plane][64], guard rows on each side: plane 0 h and threshold, then L_jj and 1/L_jj;
  // plane 1 g and -beta, then y and p; planes 2.. the row entries in pairs
  Rec *rec;
  Rec *ff, *fb;        // face buffers [ntiles + 1][frow][16][fr or br]; tile ntiles stands for no neighbour
};

__device__ __forceinline__ Rec rec2(double a, double b) { return make_rec(a, b); }
__device__ __forceinline__ double rec_d2(const Rec &r) { return rec_t(r, double()); }

// Face values of a position without a voxel.
template <int LEVEL>
__device__ __forceinline__ Rec ict_face_none(int k) {  // record k of a value: fields 2k, 2k + 1
  if (k == 0) return rec2(1.0, 1.0);
  if (k == 1) return rec2(0.0, __builtin_inf());
  return Rec{0u, 0u, 0u, 0u};
}

// Once per plan: every face value "no voxel" (the rows of a sweep are emptied
// before it, the rows past it and the tile that stands for no neighbour stay).
template <int LEVEL>
__global__ __launch_bounds__(kBlock) void k_ict_faces(IctSweep w) {
  using C = IctTile<LEVEL>;
  const int64_t n = ((int64_t)w.ntiles + 1) * w.frow * kFaceSlots;
  for (int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x; i < n; i += (int64_t)gridDim.x * kBlock) {
    for (int k = 0; k < C::fr; ++k) w.ff[i * C::fr + k] = ict_face_none<LEVEL>(k);
    for (int k = 0; k < C::br; ++k) w.fb[i * C::br + k] = Rec{0u, 0u, 0u, 0u};
  }
}

// Lay h, the drop threshold tol ||H(j:N, j)||_1, g and -beta out in step order,
// empty the face buffers, reset the tickets.
template <typename T, int LEVEL>
__global__ __launch_bounds__(kNT) void k_ict_pack(Geo g, double beta, double factor, const double *__restrict__ hmax,
                                                  const uint8_t *__restrict__ code, const T *__restrict__ D,
                                                  const T *__restrict__ gg, IctSweep w) {
#pragma clang fp contract(off)
  using C = IctTile<LEVEL>;
  if (blockIdx.x == 0 && threadIdx.x < 2) w.ticket[threadIdx.x] = 0u;
  const double tol = factor * *hmax;
  // one wavefront per 8 rows and column a: lane (s, b), as k_nat_pack
  const int lane = (int)threadIdx.x & 63, lb = lane & 7, nb = w.nrow / 8;
  const int64_t units = (int64_t)w.ntiles * w.nrow;
  for (int64_t q = (int64_t)blockIdx.x * (kNT / kWave) + threadIdx.x / kWave; q < units;
       q += (int64_t)gridDim.x * (kNT / kWave)) {
    const int tile = (int)(q / w.nrow), i = (int)(q - (int64_t)tile * w.nrow);
    const int la = i / nb, S = (i - la * nb) * 8 + (lane >> 3);
    const int tx = tile / w.nty, ty = tile - tx * w.nty;
    const int x = tx * kTile + la, y = ty * kTile + lb - C::K * la, z = S - la - (C::K + 1) * lb;
    double h = 1.0, t = __builtin_inf(), gv = 0.0, nbeta = 0.0;  // (a voxel's nbeta is negative, or -0)
    if (x < g.nx && y >= 0 && y < g.ny && z >= 0 && z < g.nz) {
      const int64_t j = ((int64_t)x * g.ny + y) * g.nz + z;
      const uint32_t c = code[j];
      const T d = D[j], gj = gg[j];
      if (c & NB_SELF) {
        h = plain_nan((double)d + beta * nb_deg(c));
        double cn = fabs(h);
        if (c & NB_XP) cn = cn + beta;
        if (c & NB_YP) cn = cn + beta;
        if (c & NB_ZP) cn = cn + beta;
        t = tol * cn;
        t = t == t ? t : 0.0;  // factor 0 and an infinite H_max: every entry is kept
        gv = plain_nan((double)gj);
        nbeta = -beta;
      }
    }
    const int64_t r = ((int64_t)tile * w.nrow + S) * C::planes * 64 + la * kTile + lb;
    w.rec[r] = rec2(h, t);
    w.rec[r + 64] = rec2(gv, nbeta);
    if (la == 0) {  // each lane an eighth of its row's face values
      const int64_t e = ((int64_t)tile * w.frow + S) * kFaceSlots;
      for (int k = lb; k < kFaceSlots * C::fr; k += 8) w.ff[e * C::fr + k] = Rec{~0u, ~0u, ~0u, ~0u};
      for (int k = lb; k < kFaceSlots * C::br; k += 8) w.fb[e * C::br + k] = Rec{~0u, ~0u, ~0u, ~0u};
    }
  }
}

// s / b from y = 1 / b, correctly rounded.
__device__ __forceinline__ double quotient(double s, double b, double y) {
  const double q = s * y;
  return fma(fma(-b, q, s), y, q);
}

// The same where s may be infinite or NaN.
__device__ __forceinline__ double quotient_any(double s, double b, double y) {
  return __builtin_amdgcn_div_fixup(quotient(s, b, y), b, s);
}

// One face's values of a group of kIctU steps: R records each, S slots a step,
// in the wavefront's registers and from there to the ring.
template <int R, int S>
struct FaceLoad {
  static constexpr int N = kIctU * S * R, V = (N + 63) / 64;
  Rec r[V];
  // slot(s): the face slot of the s-th value of a step
  template <typename F>
  __device__ __forceinline__ void load(const Rec *base, uint32_t lane, F slot) {
    const auto v = plane_view(base, kIctU * kFaceSlots * R * (uint32_t)sizeof(Rec));
#pragma unroll
    for (int k = 0; k < V; ++k) {
      const uint32_t q = min(lane + 64u * k, (uint32_t)(N - 1));
      const uint32_t u = q / (S * R), s = q / R % S, p = q % R;
      r[k] = face_ld(v, (u * kFaceSlots + slot(s)) * R + p, Rec());
    }
  }
  __device__ __forceinline__ uint32_t top() const {
    uint32_t m = 0u;
#pragma unroll
    for (int k = 0; k < V; ++k) m = max(m, max(r[k][1], r[k][3]));
    return m;
  }
  // pos(s): ring position of the s-th value of a step; slot0: ring slot of the group's first step
  template <int NF, typename F>
  __device__ __forceinline__ void put(double *ring, int slot0, uint32_t lane, F pos) const {
#pragma unroll
    for (int k = 0; k < V; ++k) {
      const uint32_t q = lane + 64u * k;
      const uint32_t u = q / (S * R), s = q / R % S, p = q % R;
      if (q < (uint32_t)N) {
        double *d = ring + (((slot0 + (int)u) & (kIctRing - 1)) * NF + 2 * (int)p) * kIctPos + pos(s);
        d[0] = rec_d(r[k]);
        if (2 * p + 1 < (uint32_t)NF) d[kIctPos] = rec_d2(r[k]);
      }
    }
  }
};

template <int LEVEL>
__global__ __launch_bounds__(64) void k_ict_fwd_wave(IctSweep w, int32_t *status) {
#pragma clang fp contract(off)
  using C = IctTile<LEVEL>;
  constexpr int NO = C::n, NF = C::nf, U = kIctU, K = C::K;
  __shared__ double ring[kIctRing * NF * kIctPos];
  const int ticket = take_ticket(&w.ticket[0]);
  if (ticket >= w.ntiles) {  // tickets not reset: refuse rather than index out of range
    set_status(status, 8);
    return;
  }
  const int2 tl = w.order[ticket];
  const int tx = __builtin_amdgcn_readfirstlane(tl.x), ty = __builtin_amdgcn_readfirstlane(tl.y);
  const int tile = tx * w.nty + ty, none = w.ntiles;
  const uint32_t lane = threadIdx.x;
  const int la = (int)lane >> 3, lb = (int)lane & 7, pos = (la + 1) * 9 + lb + 1;
  const int nrow = w.nrow;
  // every position of the ring: no voxel
  for (int i = (int)lane; i < kIctRing * NF * kIctPos; i += 64) {
    const int f = i / kIctPos % NF;
    ring[i] = f < 2 ? 1.0 : (f == 3 ? __builtin_inf() : 0.0);
  }
  Rec *rows = w.rec + (int64_t)tile * nrow * C::planes * 64;
  const int64_t ftile = (int64_t)w.frow * kFaceSlots * C::fr;
  auto tile_at = [&](int x, int y) { return x >= 0 && y >= 0 && y < w.nty ? x * w.nty + y : none; };
  // ring slot S of a halo position is the neighbour's row S + 8 (-x), + 8 (K + 1) (-y) or both
  const Rec *xnb = w.ff + tile_at(tx - 1, ty + K) * ftile;
  const Rec *ynb = w.ff + tile_at(tx, ty - 1) * ftile;
  const Rec *cnb = w.ff + tile_at(tx - 1, ty + K - 1) * ftile;
  Rec *out = w.ff + tile * ftile;
  const uint32_t so = la == kTile - 1 ? (uint32_t)lb : (lb == kTile - 1 ? (uint32_t)(kTile + la) : kNoSlot);
  struct Halo {
    FaceLoad<C::fr, 8> x, y;
    FaceLoad<C::fr, 1> c;
  };
  struct Set {
    Rec h[U], g[U];
  };
  bool timed_out = false;
  auto xslot = [](uint32_t s) { return s; };
  auto yslot = [](uint32_t s) { return y_slot(s, kTile - 1); };
  auto cslot = [](uint32_t) { return (uint32_t)(kTile - 1); };
  // the halo of ring slots S0 - 1 .. S0 + U - 2, which the steps from S0 on read
  auto halo = [&](Halo &f, int S0) {
    f.x.load(xnb + (int64_t)(S0 + 7) * kFaceSlots * C::fr, lane, xslot);
    f.y.load(ynb + (int64_t)(S0 + 8 * (K + 1) - 1) * kFaceSlots * C::fr, lane, yslot);
    f.c.load(cnb + (int64_t)(S0 + 8 * (K + 1) + 7) * kFaceSlots * C::fr, lane, cslot);
  };
  auto empty = [&](const Halo &f) { return __any(max(f.x.top(), max(f.y.top(), f.c.top())) == 0xffffffffu); };
  int spins = 0;
  auto wait = [&](Halo &f, int S0) {
    while (empty(f)) {
      if (timed_out || ++spins >= kSpinLimit) {
        if (!timed_out) set_status(status, 8);
        timed_out = true;
        return;
      }
      if (S0 <= 0) __builtin_amdgcn_s_sleep(8);  // a neighbour that has not come near yet
      asm volatile("" ::: "memory");             // load anew
      halo(f, S0);
    }
    spins = 0;
  };
  auto put = [&](const Halo &f, int S0) {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    f.x.template put<NF>(ring, S0 - 1, lane, [](uint32_t s) { return (int)s + 1; });
    f.y.template put<NF>(ring, S0 - 1, lane, [](uint32_t s) { return ((int)s + 1) * 9; });
    f.c.template put<NF>(ring, S0 - 1, lane, [](uint32_t) { return 0; });
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  };
  auto issue = [&](Set &s, int S0) {
    const auto v = plane_view(rows + (int64_t)S0 * C::planes * 64, U * C::planes * 64 * (uint32_t)sizeof(Rec));
#pragma unroll
    for (int u = 0; u < U; ++u) {
      s.h[u] = view_ld(v, lane + u * C::planes * 64, Rec());
      s.g[u] = view_ld(v, lane + (u * C::planes + 1) * 64, Rec());
    }
  };
  // this lane's previous row (its -z neighbour)
  double p_l = 1.0, p_r = 1.0, p_y = 0.0, p_t = __builtin_inf(), p_row[NO];
#pragma unroll
  for (int u = 0; u < NO; ++u) p_row[u] = 0.0;
  bool bad5 = false, bad6 = false;
  // Store the previous row, row k - 1 of the views: to the packed rows and, from
  // the face lanes, to the face buffer.
  auto store = [&](__amdgpu_buffer_rsrc_t v, __amdgpu_buffer_rsrc_t vo, int k) {
    double f[2 * C::fr];
    f[0] = p_l;
    f[1] = p_r;
    f[2] = p_y;
    f[3] = p_t;
#pragma unroll
    for (int u = 4; u < 2 * C::fr; ++u) f[u] = 0.0;
#pragma unroll
    for (int u = 0; u < NO; ++u)
      if (ict_shared<LEVEL>(u)) f[ict_field<LEVEL>(u)] = p_row[u];
#pragma unroll
    for (int u = 0; u < C::fr; ++u) face_st(vo, (so + k * kFaceSlots) * C::fr + u, rec2(f[2 * u], f[2 * u + 1]));
    view_st(v, lane + k * C::planes * 64, rec2(p_l, p_r));
    view_st(v, lane + (k * C::planes + 1) * 64, rec2(p_y, 0.0));
#pragma unroll
    for (int u = 0; u < NO; u += 2)
      view_st(v, lane + (k * C::planes + 2 + u / 2) * 64,
              rec2(p_row[u], u + 1 < NO ? p_row[u + 1 < NO ? u + 1 : 0] : 0.0));
  };
  auto compute = [&](const Set &s, int S0) {
    const auto v = plane_view(rows + (int64_t)(S0 - 1) * C::planes * 64, U * C::planes * 64 * (uint32_t)sizeof(Rec));
    const auto vo = plane_view(out + (int64_t)(S0 - 1) * kFaceSlots * C::fr, U * kFaceSlots * C::fr * (uint32_t)sizeof(Rec));
#pragma unroll
    for (int k = 0; k < U; ++k) {
      const int S = S0 + k;
      auto at = [&](int u, int f) {
        return ring[(((S - ict_back<LEVEL>(u)) & (kIctRing - 1)) * NF + f) * kIctPos + pos -
                    IctPattern<LEVEL>::off[u][0] * 9 - ict_dy<LEVEL>(u)];
      };
      // everything of other lanes' rows is read first, and the previous row
      // stored while the reads are under way
      double lkk[NO], rkk[NO], tk[NO], yk[NO], lkm[NO][NO];
#pragma unroll
      for (int u = 0; u < NO; ++u) {
        lkk[u] = ict_own<LEVEL>(u) ? p_l : at(u, 0);
        rkk[u] = ict_own<LEVEL>(u) ? p_r : at(u, 1);
        yk[u] = ict_own<LEVEL>(u) ? p_y : at(u, 2);
        tk[u] = ict_own<LEVEL>(u) ? p_t : at(u, 3);
#pragma unroll
        for (int e = 0; e < NO; ++e) {
          const int m = e < u ? ict_pair<LEVEL>(u, e) : -1;
          lkm[u][e] = m < 0 ? 0.0 : (ict_own<LEVEL>(u) ? p_row[m < 0 ? 0 : m] : at(u, ict_field<LEVEL>(m < 0 ? 0 : m)));
        }
      }
      __builtin_amdgcn_sched_barrier(0);
      if (S > 0) store(v, vo, k);
      __builtin_amdgcn_sched_barrier(0);
      const double h = rec_d(s.h[k]), t = rec_d2(s.h[k]), gj = rec_d(s.g[k]), nbeta = rec_d2(s.g[k]);
      const bool voxel = (int32_t)s.g[k][3] < 0;
      double row[NO];
#pragma unroll
      for (int u = 0; u < NO; ++u) {
        double sum = ict_stencil<LEVEL>(u) ? nbeta : 0.0;  // H_jk
#pragma unroll
        for (int e = 0; e < u; ++e)
          if (ict_pair<LEVEL>(u, e) >= 0) sum = sum - row[e] * lkm[u][e];
        const double val = quotient(sum, lkk[u], rkk[u]);
        row[u] = fabs(val) >= tk[u] ? val : 0.0;
      }
      double diag = h;
#pragma unroll
      for (int u = 0; u < NO; ++u) diag = diag - row[u] * row[u];
      const bool good = diag > 0.0, fin = fabs(diag) < __builtin_inf();
      bad5 |= !good && fin;
      bad6 |= !good && !fin;
      // L_jj = sqrt(diag) and 1 / L_jj: Goldschmidt's coupled iteration for a square
      // root and half its reciprocal from the hardware's estimate (l ~ sqrt, r ~ 1 / (2 sqrt)),
      // two corrections of l by its exact residual, and two Newton steps for the
      // reciprocal of l; no scaling, which a normal diag does not need
      const double q = __builtin_amdgcn_rsq(diag);
      double l = diag * q, r = 0.5 * q;
      double e = fma(-r, l, 0.5);
      l = fma(l, e, l);
      r = fma(r, e, r);
      l = fma(fma(-l, l, diag), r, l);
      l = fma(fma(-l, l, diag), r, l);
      r = 2.0 * r;
      r = fma(r, fma(-l, r, 1.0), r);
      r = fma(r, fma(-l, r, 1.0), r);
      double yv = gj;
#pragma unroll
      for (int u = 0; u < NO; ++u) yv = yv - row[u] * yk[u];
      p_l = good ? fmin(l, kIctInf) : 0.0;  // (l is NaN for an infinite diag)
      const bool live = voxel && good && fin;
      p_r = live ? r : 0.0;
      p_y = live ? quotient_any(yv, l, r) : 0.0;
      p_t = t;
#pragma unroll
      for (int u = 0; u < NO; ++u) p_row[u] = row[u];
      double *d = ring + (S & (kIctRing - 1)) * NF * kIctPos + pos;
      d[0] = p_l;
      d[kIctPos] = p_r;
      d[2 * kIctPos] = p_y;
      d[3 * kIctPos] = p_t;
#pragma unroll
      for (int u = 0; u < NO; ++u)
        if (ict_shared<LEVEL>(u)) d[ict_field<LEVEL>(u) * kIctPos] = row[u];
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");  // the next step reads other lanes' places
    }
  };
  Halo hn;
  Set A, B;
  issue(A, 0);
  halo(hn, -U);  // slots before the first step: -5 .. -2
  wait(hn, -U);
  put(hn, -U);
  halo(hn, 0);
  for (int S0 = 0; S0 < nrow; S0 += 2 * U) {
    wait(hn, S0);
    put(hn, S0);
    halo(hn, S0 + U);
    issue(B, S0 + U);
    compute(A, S0);
    wait(hn, S0 + U);
    put(hn, S0 + U);
    halo(hn, S0 + 2 * U);
    issue(A, S0 + 2 * U);  // past the end: the guard rows
    compute(B, S0 + U);
  }
  store(plane_view(rows + (int64_t)(nrow - 1) * C::planes * 64, C::planes * 64 * (uint32_t)sizeof(Rec)),
        plane_view(out + (int64_t)(nrow - 1) * kFaceSlots * C::fr, kFaceSlots * C::fr * (uint32_t)sizeof(Rec)), 0);
  if (bad5) set_status(status, 5);
  if (bad6) set_status(status, 6);
}

// Backward solve L^T p = y: p_j = (y_j - sum_i L_ij p_i) / L_jj over the later
// voxels i, ascending.  Every lane leaves its products L_ij p_i for the lanes j
// = i - o_u; step B handles row nrow - 1 - B.
template <int LEVEL>
__global__ __launch_bounds__(64) void k_ict_bwd_wave(IctSweep w, int32_t *status) {
#pragma clang fp contract(off)
  using C = IctTile<LEVEL>;
  constexpr int NO = C::n, NF = C::nb, U = kIctU, K = C::K;
  static_assert(ict_own<LEVEL>(NO - 1), "the lane's own column is the last offset");
  __shared__ double ring[kIctRing * NF * kIctPos];
  const int ticket = take_ticket(&w.ticket[1]);
  if (ticket >= w.ntiles) {
    set_status(status, 8);
    return;
  }
  const int2 tl = w.order[w.ntiles - 1 - ticket];
  const int tx = __builtin_amdgcn_readfirstlane(tl.x), ty = __builtin_amdgcn_readfirstlane(tl.y);
  const int tile = tx * w.nty + ty, none = w.ntiles;
  const uint32_t lane = threadIdx.x;
  const int la = (int)lane >> 3, lb = (int)lane & 7, pos = la * 9 + lb;  // the halo is at a = 8 and b = 8
  const int nrow = w.nrow;
  for (int i = (int)lane; i < kIctRing * NF * kIctPos; i += 64) ring[i] = 0.0;
  Rec *rows = w.rec + ((int64_t)tile * nrow + nrow - U) * C::planes * 64;  // a group's rows, the first step's last
  const int64_t ftile = (int64_t)w.frow * kFaceSlots * C::br;
  auto tile_at = [&](int x, int y) { return x < w.ntx && y >= 0 && y < w.nty ? x * w.nty + y : none; };
  const Rec *xnb = w.fb + tile_at(tx + 1, ty - K) * ftile;
  const Rec *ynb = w.fb + tile_at(tx, ty + 1) * ftile;
  const Rec *cnb = w.fb + tile_at(tx + 1, ty - K + 1) * ftile;
  Rec *out = w.fb + tile * ftile;
  const uint32_t so = la == 0 ? (uint32_t)lb : (lb == 0 ? (uint32_t)(kTile + la) : kNoSlot);
  struct Halo {
    FaceLoad<C::br, 8> x, y;
    FaceLoad<C::br, 1> c;
  };
  struct Set {
    Rec l[U], y[U], e[U][C::planes - 2];
  };
  bool timed_out = false;
  auto xslot = [](uint32_t s) { return s; };
  auto yslot = [](uint32_t s) { return y_slot(s, 0); };
  auto cslot = [](uint32_t) { return 0u; };
  auto halo = [&](Halo &f, int B0) {
    f.x.load(xnb + (int64_t)(B0 + 7) * kFaceSlots * C::br, lane, xslot);
    f.y.load(ynb + (int64_t)(B0 + 8 * (K + 1) - 1) * kFaceSlots * C::br, lane, yslot);
    f.c.load(cnb + (int64_t)(B0 + 8 * (K + 1) + 7) * kFaceSlots * C::br, lane, cslot);
  };
  auto empty = [&](const Halo &f) { return __any(max(f.x.top(), max(f.y.top(), f.c.top())) == 0xffffffffu); };
  int spins = 0;
  auto wait = [&](Halo &f, int B0) {
    while (empty(f)) {
      if (timed_out || ++spins >= kSpinLimit) {
        if (!timed_out) set_status(status, 8);
        timed_out = true;
        return;
      }
      if (B0 <= 0) __builtin_amdgcn_s_sleep(8);
      asm volatile("" ::: "memory");
      halo(f, B0);
    }
    spins = 0;
  };
  auto put = [&](const Halo &f, int B0) {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    f.x.template put<NF>(ring, B0 - 1, lane, [](uint32_t s) { return 72 + (int)s; });
    f.y.template put<NF>(ring, B0 - 1, lane, [](uint32_t s) { return (int)s * 9 + 8; });
    f.c.template put<NF>(ring, B0 - 1, lane, [](uint32_t) { return 80; });
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  };
  auto issue = [&](Set &s, int B0) {
    const auto v = plane_view(rows - (int64_t)B0 * C::planes * 64, U * C::planes * 64 * (uint32_t)sizeof(Rec));
#pragma unroll
    for (int u = 0; u < U; ++u) {
      s.l[u] = view_ld(v, lane + (U - 1 - u) * C::planes * 64, Rec());
      s.y[u] = view_ld(v, lane + ((U - 1 - u) * C::planes + 1) * 64, Rec());
#pragma unroll
      for (int k = 2; k < C::planes; ++k) s.e[u][k - 2] = view_ld(v, lane + ((U - 1 - u) * C::planes + k) * 64, Rec());
    }
  };
  // this lane's previous step: its column's product, those for other lanes, y and p
  double own = 0.0, c[2 * C::br], p_y = 0.0, p = 0.0;
#pragma unroll
  for (int u = 0; u < 2 * C::br; ++u) c[u] = 0.0;
  auto store = [&](__amdgpu_buffer_rsrc_t v, __amdgpu_buffer_rsrc_t vo, int k) {  // step k - 1 of the views
#pragma unroll
    for (int u = 0; u < C::br; ++u) face_st(vo, (so + k * kFaceSlots) * C::br + u, rec2(c[2 * u], c[2 * u + 1]));
    view_st(v, lane + ((U - 1 - k) * C::planes + 1) * 64, rec2(p_y, p));
  };
  auto compute = [&](const Set &s, int B0) {
    // views that begin one step earlier (rows run the other way)
    const auto v = plane_view(rows - (int64_t)(B0 - 1) * C::planes * 64, U * C::planes * 64 * (uint32_t)sizeof(Rec));
    const auto vo = plane_view(out + (int64_t)(B0 - 1) * kFaceSlots * C::br, U * kFaceSlots * C::br * (uint32_t)sizeof(Rec));
#pragma unroll
    for (int k = 0; k < U; ++k) {
      const int S = B0 + k;
      double o[NF];
#pragma unroll
      for (int u = 0; u < NF; ++u)
        o[u] = ring[(((S - ict_back<LEVEL>(u)) & (kIctRing - 1)) * NF + u) * kIctPos + pos +
                    IctPattern<LEVEL>::off[u][0] * 9 + ict_dy<LEVEL>(u)];
      __builtin_amdgcn_sched_barrier(0);
      if (S > 0) store(v, vo, k);
      __builtin_amdgcn_sched_barrier(0);
      p_y = rec_d(s.y[k]);
      double sum = p_y - own;
#pragma unroll
      for (int u = NF - 1; u >= 0; --u) sum = sum - o[u];
      const double pj = quotient_any(sum, rec_d(s.l[k]), rec_d2(s.l[k]));
      p = rec_d2(s.l[k]) != 0.0 ? pj : 0.0;
#pragma unroll
      for (int u = 0; u < NF; ++u) c[u] = (u & 1 ? rec_d2(s.e[k][u / 2]) : rec_d(s.e[k][u / 2])) * p;
      own = (NF & 1 ? rec_d2(s.e[k][NF / 2]) : rec_d(s.e[k][NF / 2])) * p;
      double *d = ring + (S & (kIctRing - 1)) * NF * kIctPos + pos;
#pragma unroll
      for (int u = 0; u < NF; ++u) d[u * kIctPos] = c[u];
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    }
  };
  Halo hn;
  Set A, B;
  issue(A, 0);
  halo(hn, -U);
  wait(hn, -U);
  put(hn, -U);
  halo(hn, 0);
  for (int B0 = 0; B0 < nrow; B0 += 2 * U) {
    wait(hn, B0);
    put(hn, B0);
    halo(hn, B0 + U);
    issue(B, B0 + U);
    compute(A, B0);
    wait(hn, B0 + U);
    put(hn, B0 + U);
    halo(hn, B0 + 2 * U);
    issue(A, B0 + 2 * U);
    compute(B, B0 + U);
  }
  // (k = 0 of a view is the row before it: here the first row, the last step's)
  store(plane_view(rows - (int64_t)(nrow - 1) * C::planes * 64, U * C::planes * 64 * (uint32_t)sizeof(Rec)),
        plane_view(out + (int64_t)(nrow - 1) * kFaceSlots * C::br, kFaceSlots * C::br * (uint32_t)sizeof(Rec)), 0);
}

// The packed place of a voxel.
template <int LEVEL>
__device__ __forceinline__ int64_t ict_place(const IctSweep &w, int x, int y, int z) {
  using C = IctTile<LEVEL>;
  const int ti = x / kTile, a = x - ti * kTile, yy = y + C::K * a, c = yy / kTile, b = yy - c * kTile;
  return (((int64_t)(ti * w.nty + c) * w.nrow + z + a + (C::K + 1) * b) * C::planes) * 64 + a * kTile + b;
}

// p to voxel order and the conjugacy dot products, in the chain of scalar state.
template <typename T, int LEVEL>
__global__ __launch_bounds__(kNT) void k_ict_unpack(IterArgs<T> a, IctSweep w, const T *__restrict__ gsrc) {
  using C = IctTile<LEVEL>;
  const Geo g = a.geo;
  const T *__restrict__ gg = gsrc ? gsrc : ((a.par & 1) ? a.G[1] : a.G[0]);
  const T *__restrict__ gp = (a.par & 1) ? a.G[0] : a.G[1];
  const State st = take_state<kNT, 4>(a.sin, a.pin, a.nparts_in, a.nvals_in, a.beta, a.trace, a.status);
  put_state(st, a.sout, PK_DOTS, (int)gridDim.x);
  // one workgroup per kUnpackZ planes z of a tile: wave k takes columns a = k and k + 4, lane (b, z), as k_nat_unpack
  constexpr int V = 2 * kUnpackZ / 8;
  const int lb = ((int)threadIdx.x & 63) >> 3, zl = (int)threadIdx.x & 7, wv = (int)threadIdx.x / kWave;
  const int nzb = (g.nz + kUnpackZ - 1) / kUnpackZ, nunit = w.ntiles * nzb;
  double acc[2] = {0.0, 0.0};
  for (int q = (int)blockIdx.x; q < nunit; q += (int)gridDim.x) {
    const int tile = q / nzb, z0 = (q - tile * nzb) * kUnpackZ + zl, tx = tile / w.nty, ty = tile - tx * w.nty;
    int j[V];
    uint32_t c[V];
    T gv[V], gpv[V];
    Rec yp[V];
#pragma unroll
    for (int v = 0; v < V; ++v) {
      const int z = z0 + (v >> 1) * 8, la = wv + 4 * (v & 1), x = tx * kTile + la, y = ty * kTile + lb - C::K * la;
      const bool ok = x < g.nx && y >= 0 && y < g.ny && z < g.nz;
      j[v] = ok ? (x * g.ny + y) * g.nz + z : -1;
      const int jj = ok ? j[v] : 0;
      const int64_t e = (((int64_t)tile * w.nrow + (ok ? z : 0) + la + (C::K + 1) * lb) * C::planes + 1) * 64 + la * kTile + lb;
      c[v] = a.code[jj];
      gv[v] = gg[jj];
      gpv[v] = gp[jj];
      yp[v] = w.rec[e];
    }
#pragma unroll
    for (int v = 0; v < V; ++v) {
      if (j[v] < 0) continue;
      const bool in = c[v] & NB_SELF;
      const double p = in ? rec_d2(yp[v]) : 0.0;
      a.P[j[v]] = (T)p;
      acc[0] += in ? (double)gv[v] * p : 0.0;
      acc[1] += in ? (double)gpv[v] * p : 0.0;
    }
  }
  store_partials<2, kNT>(acc, a.pout);
}

// The factor in voxel order: L [1 + n][voxels] (all of it, or the pivots L_jj^2 alone).
template <int LEVEL>
__global__ __launch_bounds__(kBlock) void k_ict_factor(Geo g, const uint8_t *__restrict__ code, IctSweep w, double *L,
                                                       double *piv) {
  using C = IctTile<LEVEL>;
  for (int64_t j = (int64_t)blockIdx.x * kBlock + threadIdx.x; j < g.n; j += (int64_t)gridDim.x * kBlock) {
    const int z = (int)(j % g.nz), y = (int)(j / g.nz % g.ny), x = (int)(j / g.sx);
    const bool in = code[j] & NB_SELF;
    const Rec *r = w.rec + ict_place<LEVEL>(w, x, y, z);
    const double lj = in ? rec_d(r[0]) : 0.0, l = lj == kIctInf ? __builtin_inf() : lj;
    if (piv) piv[j] = l * l;
    if (!L) continue;
    L[j] = l;
    for (int u = 0; u < C::n; ++u) {
      const Rec e = r[(2 + u / 2) * 64];
      L[(int64_t)(1 + u) * g.n + j] = in ? (u & 1 ? rec_d2(e) : rec_d(e)) : 0.0;
    }
  }
}

}  // namespace fm
