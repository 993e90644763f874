// Implicit adjoint of the converged field map.
//
// At a stationary point fhat of the cost of Sec. II eq. (cost), grad Psi = 0,
// so a loss L(fhat) has dL/dtheta = -v^T d(grad Psi)/dtheta with H v = dL/df,
// H = diag(h) + beta C^T C the exact Hessian, h_j = sum_{m<n} w_mn (2 pi dt)^2
// cos(x_mn) (the curvature the Huber bound of Sec. III-B eq. (ls_huber)
// replaces).  H v = dL/df is solved by conjugate gradients preconditioned with
// the IC(0) factor of the Huber model D + beta C^T C (Sec. III-B eq.
// (precon)), reusing the iteration's preconditioner passes.  One CG iteration
// is: preconditioner passes (z = M^{-1} r, leaving r^T z), direction pass
// (d = z + (rho / rho_prev) d_prev, partial d^T H d) and update pass
// (v += alpha d, r -= alpha H d, partial ||r||^2).  The direction buffer
// ping-pongs with the CG iteration parity because the Hessian stencil reads
// the previous direction at neighbours.
//
// The gradients then follow from v:
//   dL/dbeta   = -v^T C^T C fhat,
//   dL/dzhat_l = -v_j d g_j / d zhat_l, with g_j = sum_{m<n} 2 (2 pi dt_mn)
//                Im(Gamma_mn conj(zhat_m) zhat_n e^{i 2 pi dt_mn f_j}),
//   dL/dy_cl   = (s_c / sqrt(sum_c |s_c|^2)) dL/dzhat_l  (zhat is linear in y),
// complex gradients in the d/dRe + i d/dIm convention.
//
// With the second-order regulariser (R2) C^T C is the 13-point operator of
// fm_order2.hpp in the Hessian products and in dL/dbeta, and CG is
// preconditioned by diag(H) (the Huber curvature plus beta diag(C^T C)) or
// not at all: the solution v does not depend on the preconditioner, only the
// iteration count does.
#pragma once

#include "fm_stream.hpp"
#include "fm_order2.hpp"

namespace fm {

template <typename T>
struct AdjArgs {
  Geo geo;
  int32_t L;
  double beta;
  const T2<T> *dat;
  const uint8_t *code;
  const PairC<T> *pairs;
  const T *F;      // fhat
  T *R;            // residual (padded: the preconditioner reads neighbours)
  const T *Zp;     // preconditioned residual (padded)
  T *Dd[2];        // CG directions (padded), slot par written this iteration
  T *V;            // solution v
  T *H;            // exact Hessian diagonal h_j (without beta deg)
  T *Dc;           // Huber curvature (the preconditioner's D)
  double *hinv;    // 1 / (D + beta deg) for the red-black preconditioner (pair passes: of the red voxels at j >> 1)
  T *P;            // pair passes: p of the black voxels at j >> 1
  int32_t par;     // CG iteration parity
  int32_t nparts_in;
  int32_t nvals_in;
  const State *sin;
  State *sout;
  const double *pin;
  double *pout;
  int32_t *status;
};

// Data-term curvatures at f: the Huber bound (as in the iteration) and the
// exact second derivative, with the same turn-based wrap as voxel_terms:
// cos(2 pi xi) = 1 - 2 s^2.
template <typename T, int LMAX>
__device__ __forceinline__ void voxel_curvatures(const T (&rho)[LMAX], const T (&tau)[LMAX], int L,
                                                 const PairC<T> *__restrict__ pc, T f, T &curv, T &hess) {
  T c2 = 0, h2 = 0;
  int q = 0;
#pragma unroll
  for (int m = 0; m < LMAX; ++m) {
#pragma unroll
    for (int n = m + 1; n < LMAX; ++n) {
      if (n < L) {
        const PairC<T> P = pc[q];
        const T w = P.w * rho[m] * rho[n];
        const T xi = P.g + (tau[n] - tau[m]) + f * P.dt;
        const T x = T(3.14159265358979323846) * (xi - rint_t(xi));
        T sx, c;
        sinx_cos(x, sx, c);
        const T s = x * sx;
        const T wdd = w * P.d2pi * P.d2pi;
        c2 += wdd * (sx * c);
        h2 += wdd * (T(1) - T(2) * s * s);
        ++q;
      }
    }
  }
  curv = c2;
  hess = h2;
}

// Set-up at fhat: curvatures, r = dL/df, v = 0, d_prev = 0; partial ||r||^2.
template <typename T, int LMAX>
__global__ __launch_bounds__(kNT) void k_adj_setup(AdjArgs<T> a, const double *__restrict__ dldf, double rtol2,
                                                   int write_hinv) {
  const Geo g = a.geo;
  const int n = (int)g.n;
  double acc[1] = {0.0};
  for (int j = (int)blockIdx.x * kNT + (int)threadIdx.x; j < n; j += (int)gridDim.x * kNT) {
    const uint32_t c = a.code[j];
    T r = T(0), curv = T(0), hess = T(0);
    double hv = 0.0;
    if (c & NB_SELF) {
      T rho[LMAX], tau[LMAX];
      load_echoes<T, LMAX>(a.dat, (int64_t)n, j, a.L, rho, tau);
      voxel_curvatures<T, LMAX>(rho, tau, a.L, a.pairs, a.F[j], curv, hess);
      r = (T)dldf[g.user(j)];
      const double h = (double)curv + a.beta * nb_deg(c);
      hv = h > 0.0 ? 1.0 / h : 0.0;
      acc[0] += (double)r * (double)r;
    }
    a.R[j] = r;
    a.Dc[j] = curv;
    a.H[j] = hess;
    a.V[j] = T(0);
    a.Dd[1][j] = T(0);
    if (write_hinv == 1)
      a.hinv[j] = hv;
    else if (write_hinv == 2 && (c & NB_SELF) && !(c & NB_BLACK))
      a.hinv[j >> 1] = hv;
  }
  store_partials<1, kNT>(acc, a.pout);
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    State s{};
    s.kind = PK_ADJ_INIT;
    s.nparts = (int32_t)gridDim.x;
    s.trace_cap = -1;
    s.cg_rtol2 = rtol2;
    *a.sout = s;
  }
}

// Direction d = z + (rho / rho_prev) d_prev and the partial d^T H d.
template <typename T, bool R2>
__global__ __launch_bounds__(kNT) void k_adj_dir(AdjArgs<T> a) {
  constexpr int V = R2 ? 1 : Vpt<T>::v, K2 = R2 ? 6 : 1;
  const Geo g = a.geo;
  const T *__restrict__ dp = a.Dd[(a.par + 1) & 1];
  T *__restrict__ dn = a.Dd[a.par & 1];
  const Offs of(g);
  const int n = (int)g.n, chunk = kNT * V, stride = (int)gridDim.x * chunk;
  uint32_t c[V], cn[V][K2];
  T z0[V], d0[V], h0[V], zn[V][6], dnb[V][6], zn2[V][K2], dnb2[V][K2];
  auto load = [&](int b) {
#pragma unroll
    for (int v = 0; v < V; ++v) {
      const int j = b + v * kNT + (int)threadIdx.x;
      const int jj = j < n ? j : n - 1;
      c[v] = j < n ? a.code[jj] : 0u;
      z0[v] = a.Zp[jj];
      d0[v] = dp[jj];
      h0[v] = a.H[jj];
#pragma unroll
      for (int k = 0; k < 6; ++k) {
        zn[v][k] = a.Zp[jj + of.o[k]];
        dnb[v][k] = dp[jj + of.o[k]];
      }
      if constexpr (R2) {
#pragma unroll
        for (int k = 0; k < 6; ++k) {
          cn[v][k] = a.code[jj + of.o[k]];
          zn2[v][k] = a.Zp[jj + 2 * of.o[k]];
          dnb2[v][k] = dp[jj + 2 * of.o[k]];
        }
      }
    }
  };
  int base = (int)blockIdx.x * chunk;
  if (base < n) load(base);
  State st = take_state<kNT, 2>(a.sin, a.pin, a.nparts_in, a.nvals_in, a.beta, nullptr, a.status);
  double acc[1] = {0.0};
  if (!st.cg_done) {
    const double rho = st.gtp;  // r^T M^{-1} r from the preconditioner passes
    const T bcg = (T)((st.cg_it > 0 && st.cg_rho_prev != 0.0) ? rho / st.cg_rho_prev : 0.0);
    const T beta = (T)a.beta;
    st.cg_rho = rho;
    for (; base < n; base += stride) {
#pragma unroll
      for (int v = 0; v < V; ++v) {
        const int j = base + v * kNT + (int)threadIdx.x;
        if (j >= n) continue;
        const uint32_t cv = c[v];
        if (!(cv & NB_SELF)) {
          dn[j] = T(0);
          continue;
        }
        const T dj = z0[v] + bcg * d0[v];
        T lap = T(0);
        if constexpr (R2) {
          T v1[6], v2[6];
#pragma unroll
          for (int k = 0; k < 6; ++k) {
            v1[k] = zn[v][k] + bcg * dnb[v][k];
            v2[k] = zn2[v][k] + bcg * dnb2[v][k];
          }
          lap = ctc2(Rows2(cv, cn[v]), dj, v1, v2);
        } else {
#pragma unroll
          for (int k = 0; k < 6; ++k)
            if (has_nb(cv, k)) lap += dj - (zn[v][k] + bcg * dnb[v][k]);
        }
        dn[j] = dj;
        const T qj = h0[v] * dj + beta * lap;
        acc[0] += (double)dj * (double)qj;
      }
      if (base + stride < n) load(base + stride);
    }
  }
  store_partials<1, kNT>(acc, a.pout);
  put_state(st, a.sout, PK_ADJ_CURV, gridDim.x);
}

// Red-black IC(0) with an even column length: a CG iteration in three passes.
// As in the iteration (k_rb_black_pair, k_rb_red_dir_pair), the black pass yields
// r^T M^{-1} r in full from the factored form, so the red pass forms the direction
// of both colours and d^T H d over the edges of C from their red ends, and the
// pass over p in between goes.  128x128x64 MIX, per CG iteration: black 11.7, red
// 8.5 and direction 8.2 us -> black 8.0 and red + direction 8.0 us.
template <typename T>
__global__ __launch_bounds__(kNT) void k_adj_black_pair(AdjArgs<T> a) {
  const Geo g = a.geo;
  const T *__restrict__ r = a.R;
  const double *__restrict__ hv = a.hinv;
  const Offs of(g);
  const int np = (int)(g.n >> 1), stride = (int)gridDim.x * kNT;
  uint32_t cb, cr;
  int jb;
  T d0, r0, rr, rn[6];
  double hr, hn[6];
  auto load = [&](int q) {
    const int j0 = 2 * (q < np ? q : np - 1);
    const uint32_t c2 = *reinterpret_cast<const uint16_t *>(a.code + j0);
    const uint32_t cA = q < np ? (c2 & 0xffu) : 0u, cB = q < np ? (c2 >> 8) : 0u;
    const bool fb = first_is_black(cA, cB);
    jb = fb ? j0 : j0 + 1;
    cb = fb ? cA : cB;
    cr = fb ? cB : cA;
    const Duo<T> r2 = ld_duo(r, j0);
    r0 = fb ? r2.v0 : r2.v1;
    rr = fb ? r2.v1 : r2.v0;
    hr = hv[j0 >> 1];
    d0 = a.Dc[jb];
#pragma unroll
    for (int k = 0; k < 6; ++k) {
      rn[k] = r[jb + of.o[k]];
      hn[k] = hv[(jb + of.o[k]) >> 1];  // a red neighbour: its pair's entry
    }
  };
  int q = (int)blockIdx.x * kNT + (int)threadIdx.x;
  if (q < np) load(q);
  const State st = take_state<kNT, 1>(a.sin, a.pin, a.nparts_in, a.nvals_in, a.beta, nullptr, a.status);
  put_state(st, a.sout, PK_DOTS_A, gridDim.x);
  const double beta = a.beta, b2 = a.beta * a.beta;
  double acc[1] = {0.0};
  int bad = 0;
  if (!st.cg_done) {
    for (; q < np; q += stride) {
      if (cr & NB_SELF) acc[0] += (double)rr * ((double)rr * hr);
      if (cb & NB_SELF) {
        double sp = 0.0, sxv = 0.0;
#pragma unroll
        for (int k = 0; k < 6; ++k)
          if (has_nb(cb, k)) {
            sp += hn[k];
            sxv += (double)rn[k] * hn[k];
          }
        const double piv = ((double)d0 + beta * nb_deg(cb)) - b2 * sp;
        double ip = 1.0 / piv;
        if (!(piv > 0.0)) {
          bad = 1;
          ip = 0.0;
        }
        const double yb = (double)r0 + beta * sxv, x = yb * ip;
        a.P[jb >> 1] = (T)x;
        acc[0] += yb * x;
      }
      if (q + stride < np) load(q + stride);
    }
  }
  if (bad) set_status(a.status, 5);
  store_partials<1, kNT>(acc, a.pout);
}

// d = z + (rho / rho_prev) d_prev of both colours, z on the red ones from the
// black pass's p; partial d^T H d = sum h d^2 + beta ||C d||^2.
template <typename T>
__global__ __launch_bounds__(kNT) void k_adj_red_dir_pair(AdjArgs<T> a) {
  const Geo g = a.geo;
  const T *__restrict__ dp = a.Dd[(a.par + 1) & 1];
  T *__restrict__ dn = a.Dd[a.par & 1];
  const T *__restrict__ p = a.P;
  const Offs of(g);
  const int np = (int)(g.n >> 1), stride = (int)gridDim.x * kNT;
  uint32_t cb, cr;
  bool fbk;
  T rr, dr, db, hb, hh, pb, pn[6], dq[6];
  double hr;
  auto load = [&](int q) {
    const int j0 = 2 * (q < np ? q : np - 1);
    const uint32_t c2 = *reinterpret_cast<const uint16_t *>(a.code + j0);
    const uint32_t cA = q < np ? (c2 & 0xffu) : 0u, cB = q < np ? (c2 >> 8) : 0u;
    const bool fb = first_is_black(cA, cB);
    const int jr = fb ? j0 + 1 : j0;
    fbk = fb;
    cb = fb ? cA : cB;
    cr = fb ? cB : cA;
    const Duo<T> d2 = ld_duo(dp, j0), h2 = ld_duo(a.H, j0);
    dr = fb ? d2.v1 : d2.v0;
    db = fb ? d2.v0 : d2.v1;
    hh = fb ? h2.v1 : h2.v0;
    hb = fb ? h2.v0 : h2.v1;
    pb = p[j0 >> 1];
    rr = a.R[jr];
    hr = a.hinv[j0 >> 1];
#pragma unroll
    for (int k = 0; k < 6; ++k) {
      pn[k] = p[(jr + of.o[k]) >> 1];  // a black neighbour: its pair's entry
      dq[k] = dp[jr + of.o[k]];
    }
  };
  int q = (int)blockIdx.x * kNT + (int)threadIdx.x;
  if (q < np) load(q);
  State st = take_state<kNT, 1>(a.sin, a.pin, a.nparts_in, a.nvals_in, a.beta, nullptr, a.status);
  double acc[1] = {0.0};
  int bad = 0;
  if (!st.cg_done) {
    const double rho = st.acc0, beta = a.beta;  // (left as the first of two sums)
    const T bcg = (T)((st.cg_it > 0 && st.cg_rho_prev != 0.0) ? rho / st.cg_rho_prev : 0.0);
    st.cg_rho = rho;
    for (; q < np; q += stride) {
      T drv = T(0), dbv = T(0);
      if (cr & NB_SELF) {
        double sp = 0.0;
#pragma unroll
        for (int k = 0; k < 6; ++k)
          if (has_nb(cr, k)) sp += (double)pn[k];
        if (!(hr > 0.0)) bad = 1;
        const T z = (T)((double)rr * hr + beta * sp * hr);
        drv = z + bcg * dr;
        acc[0] += (double)drv * (double)drv * (double)hh;
#pragma unroll
        for (int k = 0; k < 6; ++k)
          if (has_nb(cr, k)) {
            const double dd = (double)(drv - (pn[k] + bcg * dq[k]));
            acc[0] += beta * (dd * dd);
          }
      }
      if (cb & NB_SELF) {
        dbv = pb + bcg * db;
        acc[0] += (double)dbv * (double)dbv * (double)hb;
      }
      Duo<T> out;
      out.v0 = fbk ? dbv : drv;
      out.v1 = fbk ? drv : dbv;
      *reinterpret_cast<Duo<T> *>(dn + 2 * q) = out;
      if (q + stride < np) load(q + stride);
    }
  }
  if (bad) set_status(a.status, 5);
  store_partials<1, kNT>(acc, a.pout);
  put_state(st, a.sout, PK_ADJ_CURV, gridDim.x);
}

// v += alpha d, r -= alpha H d; partial ||r||^2.
template <typename T, bool R2>
__global__ __launch_bounds__(kNT) void k_adj_update(AdjArgs<T> a) {
  constexpr int V = R2 ? 1 : Vpt<T>::v, K2 = R2 ? 6 : 1;
  const Geo g = a.geo;
  const T *__restrict__ d = a.Dd[a.par & 1];
  const Offs of(g);
  const int n = (int)g.n, chunk = kNT * V, stride = (int)gridDim.x * chunk;
  uint32_t c[V], cn[V][K2];
  T d0[V], h0[V], v0[V], r0[V], dnb[V][6], dnb2[V][K2];
  auto load = [&](int b) {
#pragma unroll
    for (int v = 0; v < V; ++v) {
      const int j = b + v * kNT + (int)threadIdx.x;
      const int jj = j < n ? j : n - 1;
      c[v] = j < n ? a.code[jj] : 0u;
      d0[v] = d[jj];
      h0[v] = a.H[jj];
      v0[v] = a.V[jj];
      r0[v] = a.R[jj];
#pragma unroll
      for (int k = 0; k < 6; ++k) dnb[v][k] = d[jj + of.o[k]];
      if constexpr (R2) {
#pragma unroll
        for (int k = 0; k < 6; ++k) {
          cn[v][k] = a.code[jj + of.o[k]];
          dnb2[v][k] = d[jj + 2 * of.o[k]];
        }
      }
    }
  };
  int base = (int)blockIdx.x * chunk;
  if (base < n) load(base);
  const State st = take_state<kNT, 1>(a.sin, a.pin, a.nparts_in, a.nvals_in, a.beta, nullptr, a.status);
  put_state(st, a.sout, PK_ADJ_UPD, gridDim.x);
  double acc[1] = {0.0};
  if (!st.cg_done) {
    const T alpha = (T)st.cg_alpha;
    const T beta = (T)a.beta;
    for (; base < n; base += stride) {
#pragma unroll
      for (int v = 0; v < V; ++v) {
        const int j = base + v * kNT + (int)threadIdx.x;
        if (j >= n) continue;
        const uint32_t cv = c[v];
        if (!(cv & NB_SELF)) continue;
        const T dj = d0[v];
        T lap = T(0);
        if constexpr (R2) {
          lap = ctc2(Rows2(cv, cn[v]), dj, dnb[v], dnb2[v]);
        } else {
#pragma unroll
          for (int k = 0; k < 6; ++k)
            if (has_nb(cv, k)) lap += dj - dnb[v][k];
        }
        const T qj = h0[v] * dj + beta * lap;
        const T rj = r0[v] - alpha * qj;
        a.V[j] = v0[v] + alpha * dj;
        a.R[j] = rj;
        acc[0] += (double)rj * (double)rj;
      }
      if (base + stride < n) load(base + stride);
    }
  }
  store_partials<1, kNT>(acc, a.pout);
}

// k_adj_update with four consecutive voxels of a column per thread (FP32, first
// differences, nz a multiple of 4): 16-byte loads and stores, the same values.
__global__ __launch_bounds__(kNT) void k_adj_update_q(AdjArgs<float> a) {
  const Geo g = a.geo;
  const float *__restrict__ d = a.Dd[a.par & 1];
  const int nq = (int)(g.n >> 2), stride = (int)gridDim.x * kNT, sx = (int)g.sx, sy = (int)g.sy;
  uint32_t c4;
  float4 d4, h4, v4, r4, dx[2], dy[2];
  float dzm, dzp;
  auto ld4 = [](const float *p) { return *reinterpret_cast<const float4 *>(p); };
  auto load = [&](int q) {
    const int j = 4 * q;
    c4 = *reinterpret_cast<const uint32_t *>(a.code + j);
    d4 = ld4(d + j);
    h4 = ld4(a.H + j);
    v4 = ld4(a.V + j);
    r4 = ld4(a.R + j);
    dx[0] = ld4(d + j - sx);
    dx[1] = ld4(d + j + sx);
    dy[0] = ld4(d + j - sy);
    dy[1] = ld4(d + j + sy);
    dzm = d[j - 1];
    dzp = d[j + 4];
  };
  int q = (int)blockIdx.x * kNT + (int)threadIdx.x;
  if (q < nq) load(q);
  const State st = take_state<kNT, 1>(a.sin, a.pin, a.nparts_in, a.nvals_in, a.beta, nullptr, a.status);
  put_state(st, a.sout, PK_ADJ_UPD, gridDim.x);
  double acc[1] = {0.0};
  if (!st.cg_done) {
    const float alpha = (float)st.cg_alpha, beta = (float)a.beta;
    for (; q < nq; q += stride) {
      const int j = 4 * q;
      const float dv[4] = {d4.x, d4.y, d4.z, d4.w}, hv[4] = {h4.x, h4.y, h4.z, h4.w};
      const float xm[4] = {dx[0].x, dx[0].y, dx[0].z, dx[0].w}, xp[4] = {dx[1].x, dx[1].y, dx[1].z, dx[1].w};
      const float ym[4] = {dy[0].x, dy[0].y, dy[0].z, dy[0].w}, yp[4] = {dy[1].x, dy[1].y, dy[1].z, dy[1].w};
      float vo[4] = {v4.x, v4.y, v4.z, v4.w}, ro[4] = {r4.x, r4.y, r4.z, r4.w};
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const uint32_t cv = (c4 >> (8 * i)) & 0xffu;
        const float dn[6] = {xm[i], xp[i], ym[i], yp[i], i > 0 ? dv[i > 0 ? i - 1 : 0] : dzm, i < 3 ? dv[i < 3 ? i + 1 : 3] : dzp};
        float lap = 0.f;
#pragma unroll
        for (int k = 0; k < 6; ++k)
          if (has_nb(cv, k)) lap += dv[i] - dn[k];
        const float qj = hv[i] * dv[i] + beta * lap;
        const float rj = ro[i] - alpha * qj;
        if (cv & NB_SELF) {
          vo[i] = vo[i] + alpha * dv[i];
          ro[i] = rj;
          acc[0] += (double)rj * (double)rj;
        }
      }
      *reinterpret_cast<float4 *>(a.V + j) = make_float4(vo[0], vo[1], vo[2], vo[3]);
      *reinterpret_cast<float4 *>(a.R + j) = make_float4(ro[0], ro[1], ro[2], ro[3]);
      if (q + stride < nq) load(q + stride);
    }
  }
  store_partials<1, kNT>(acc, a.pout);
}

// Gradients from v: dL/dy (complex64, layout of y), v as float64, and the
// partial v^T C^T C fhat for dL/dbeta.
template <typename T, int LMAX, bool R2>
__global__ __launch_bounds__(kNT) void k_adj_out(AdjArgs<T> a, const float2 *__restrict__ sens, int ncoil,
                                                 float2 *__restrict__ dldy, double *__restrict__ vout) {
  const Geo g = a.geo;
  const int n = (int)g.n;
  const T kPi = T(3.14159265358979323846);
  double acc[1] = {0.0};
  for (int j = (int)blockIdx.x * kNT + (int)threadIdx.x; j < n; j += (int)gridDim.x * kNT) {
    const uint32_t c = a.code[j];
    const T vj = (c & NB_SELF) ? a.V[j] : T(0);
    const int64_t u = g.user(j), nu = g.user_n();
    if (u < 0) continue;  // never in the mask
    if (vout) vout[u] = (double)vj;
    // zhat-gradients in the frame of each echo's own phase: dL/dzhat_l = a_l e^{i theta_l}
    T are[LMAX], aim[LMAX];
#pragma unroll
    for (int l = 0; l < LMAX; ++l) are[l] = aim[l] = T(0);
    T rho[LMAX], tau[LMAX];
#pragma unroll
    for (int l = 0; l < LMAX; ++l) rho[l] = tau[l] = T(0);
    if (c & NB_SELF) {
      const T fj = a.F[j];
      T lap = T(0);
      const int o[6] = {-(int)g.sx, (int)g.sx, -(int)g.sy, (int)g.sy, -1, 1};
      if constexpr (R2) {
        uint32_t cn[6];
        T v1[6], v2[6];
#pragma unroll
        for (int k = 0; k < 6; ++k) {
          cn[k] = a.code[j + o[k]];
          v1[k] = a.F[j + o[k]];
          v2[k] = a.F[j + 2 * o[k]];
        }
        lap = ctc2(Rows2(c, cn), fj, v1, v2);
      } else {
#pragma unroll
        for (int k = 0; k < 6; ++k)
          if (has_nb(c, k)) lap += fj - a.F[j + o[k]];
      }
      acc[0] += (double)vj * (double)lap;
      load_echoes<T, LMAX>(a.dat, (int64_t)n, j, a.L, rho, tau);
      int q = 0;
#pragma unroll
      for (int m = 0; m < LMAX; ++m) {
#pragma unroll
        for (int nn = m + 1; nn < LMAX; ++nn) {
          if (nn < a.L) {
            const PairC<T> P = a.pairs[q];
            const T xi = P.g + (tau[nn] - tau[m]) + fj * P.dt;
            const T x = kPi * (xi - rint_t(xi));
            T sx, cc;
            sinx_cos(x, sx, cc);
            const T s = x * sx;
            const T S2 = T(2) * s * cc;          // sin(2 pi xi)
            const T C2 = T(1) - T(2) * s * s;    // cos(2 pi xi)
            const T coef = -vj * P.d2pi * P.w;
            // d/dzhat_n: coef rho_m (sin + i cos); d/dzhat_m: coef rho_n (sin - i cos)
            are[nn] += coef * rho[m] * S2;
            aim[nn] += coef * rho[m] * C2;
            are[m] += coef * rho[nn] * S2;
            aim[m] -= coef * rho[nn] * C2;
            ++q;
          }
        }
      }
    }
    // rotate by e^{i theta_l}, theta_l = 2 pi tau_l
    T gre[LMAX], gim[LMAX];
#pragma unroll
    for (int l = 0; l < LMAX; ++l) {
      const T x = kPi * (tau[l] - rint_t(tau[l]));
      T sx, cc;
      sinx_cos(x, sx, cc);
      const T s = x * sx;
      const T sn = T(2) * s * cc, cs = T(1) - T(2) * s * s;
      gre[l] = are[l] * cs - aim[l] * sn;
      gim[l] = are[l] * sn + aim[l] * cs;
    }
    if (dldy) {
      double ss = 1.0;
      if (sens) {
        ss = 0.0;
        for (int cc = 0; cc < ncoil; ++cc) {
          const float2 sv = sens[(int64_t)cc * nu + u];
          ss += (double)sv.x * sv.x + (double)sv.y * sv.y;
        }
      }
      const double scale = ss > 0.0 ? 1.0 / sqrt(ss) : 0.0;
      for (int cc = 0; cc < ncoil; ++cc) {
        double sr = scale, si = 0.0;
        if (sens) {
          const float2 sv = sens[(int64_t)cc * nu + u];
          sr = sv.x * scale;
          si = sv.y * scale;
        }
        for (int l = 0; l < a.L; ++l) {
          T xr = T(0), xim = T(0);
#pragma unroll
          for (int k = 0; k < LMAX; ++k)
            if (k == l) {
              xr = gre[k];
              xim = gim[k];
            }
          float2 o;
          o.x = (float)(sr * (double)xr - si * (double)xim);
          o.y = (float)(sr * (double)xim + si * (double)xr);
          dldy[((int64_t)cc * a.L + l) * nu + u] = o;
        }
      }
    }
  }
  store_partials<1, kNT>(acc, a.pout);
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    State s = *a.sin;
    s.kind = PK_ADJ_FIN;
    s.nparts = (int32_t)gridDim.x;
    *a.sout = s;
  }
}

}  // namespace fm
