// Host side of the C ABI declared in include/fmap.h: parameter validation,
// plan and workspace management, the kernel chain of one NCG iteration and
// the HIP graph that replays the whole iteration loop.
#include <hip/hip_ext.h>
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <complex>
#include <cstdio>
#include <cstring>
#include <map>
#include <string>
#include <utility>
#include <type_traits>
#include <vector>

#include "../../include/fmap.h"
#include "fm_kernels.hpp"
#include "fm_stream.hpp"
#include "fm_natural.hpp"
#include "fm_adjoint.hpp"
#include "fm_resident.hpp"
#include "fm_order2.hpp"
#include "fm_ict.hpp"
#include "fm_ict_tile.hpp"
#include "fm_level.hpp"
#include "fm_tile.hpp"

using fm::kBlock;
using fm::kMaxGrid;
using fm::kMaxK;

namespace {

thread_local std::string g_last_error;

fm_status fail(fm_status st, const std::string &msg) {
  g_last_error = msg;
  return st;
}

#define FM_HIP(call)                                                                      \
  do {                                                                                    \
    hipError_t e_ = (call);                                                               \
    if (e_ != hipSuccess)                                                                 \
      return fail(FM_ERR_HIP, std::string(#call) + ": " + hipGetErrorString(e_));         \
  } while (0)

#define FM_LAUNCH_CHECK()                                                                 \
  do {                                                                                    \
    hipError_t e_ = hipGetLastError();                                                    \
    if (e_ != hipSuccess) return fail(FM_ERR_HIP, std::string("kernel launch: ") + hipGetErrorString(e_)); \
  } while (0)

}  // namespace

struct fm_plan {
  fm_params prm;
  int device = 0;
  int64_t n = 0;
  fm::Geo geo{};
  bool mix = false;
  int lmax = 4;
  int npairs = 0;
  int grid = 1;   // blocks of the kBlock-thread kernels
  int sgrid = 1;  // blocks of the streaming iteration passes (kNT threads)
  bool few = false;  // few enough voxels for a thread each
  size_t tsize = 8;  // bytes of the working type
  // device workspace
  void *dat = nullptr;
  uint8_t *code = nullptr;
  void *F[2] = {nullptr, nullptr};
  void *Z[2] = {nullptr, nullptr};
  void *G[2] = {nullptr, nullptr};
  void *D = nullptr, *X = nullptr, *P = nullptr;
  void *X2 = nullptr;          // three-colour IC(0): y' = L^{-1} g_prev of colour 1
  uint8_t *rdiag = nullptr;    // three-colour IC(0): diag(C^T C) of the second-order operator
  // three-colour IC(0): G, D, P, ipiv, X, X2, rdiag and a copy of the codes (ccode) are kept
  // colour-major, cm_elems elements each (three colour blocks with two padding x-planes)
  bool cm = false;
  uint8_t *ccode = nullptr;
  int64_t cm_elems = 0;
  void *Pv = nullptr, *Dv = nullptr;  // voxel-order copies of p and D for the direction pass
  double *ipiv = nullptr;
  double *hinv = nullptr;
  fm::State *S = nullptr;      // two ping-pong state copies
  double *part = nullptr;      // two ping-pong partial-sum buffers [part_rows][kMaxK]
  size_t part_rows = kMaxGrid;
  fm::Wavefront wf{};          // natural-order sweep: tiles, tickets, packed arrays, face buffers
  int wf_pack_grid = 1, wf_unpack_grid = 1;
  void *wf_bases[4] = {};      // allocations of the packed rows and face buffers
  bool by_levels = false;      // no packed rows: natural and block red-black IC(0) run a launch per level
  double *setup_part = nullptr;
  double *nmask = nullptr;
  int32_t *status = nullptr;
  double *trace = nullptr;
  void *pairs = nullptr;
  void *pairs_d = nullptr;
  double *comp_tab = nullptr;  // eq. (wf): te [L], then B = (gamma^H gamma)^{-1} gamma^H [K][L] complex
  int ncomp = 1;
  double *gabs = nullptr;
  double *rho = nullptr;
  double *f0buf = nullptr;
  double2 *sweep_rot = nullptr;  // water-fat sweep: rotation of each pair between sweep values
  double *wf_tmp = nullptr;  // water-fat init: swept map and 3 CG vectors
  bool setup_done = false;
  bool solved = false;
  // position in the kernel chain: launch q reads S[q&1], writes S[(q+1)&1];
  // iteration index and partial-sum count at the current position
  uint64_t q = 0;
  int64_t iter_host = 0;
  int last_nparts = 0;
  int last_nvals = 0;   // values per partial block at the current position
  // device allocations (freed with the plan); stencil-read arrays are
  // padded by pad elements on both sides
  std::vector<void *> bases;
  int64_t pad = 0;
  // graphs of the iteration loop keyed by (chain parity, iterations)
  hipStream_t cap_stream = nullptr;
  std::map<std::vector<int64_t>, std::pair<hipGraph_t, hipGraphExec_t>> graphs;
  // implicit adjoint workspace (allocated by the first fm_adjoint call)
  bool adj_ready = false;
  bool adj_levels = false;  // block red-black plan without face buffers: its CG runs a launch per level
  void *aR = nullptr, *aZ = nullptr, *aX = nullptr, *aDc = nullptr, *aH = nullptr, *aV = nullptr;
  void *aDd[2] = {nullptr, nullptr};
  double *a_hinv = nullptr, *a_ipiv = nullptr, *a_part = nullptr;
  fm::State *aS = nullptr;
  int32_t *a_status = nullptr;
  fm::State *a_host = nullptr;           // [2] pinned copies of the CG state, and the events that follow them
  hipEvent_t a_copied[2] = {nullptr, nullptr};
  // resident schedule (one launch for many iterations)
  bool reg2 = false;           // second-order regulariser
  int32_t sched = FM_SCHED_AUTO;
  bool res_ok = false;         // the plan qualifies (MIX, red-black IC(0), <= 4 echoes, tiles fit)
  bool res_auto = false;       // and FM_SCHED_AUTO takes it (large enough volume)
  fm::ResTile res_tile{};
  int res_grid = 0;
  double *res_part = nullptr;  // [2][kMaxK][res_grid]
  uint32_t *res_bar = nullptr; // barrier counters
  // IC_t (incomplete Cholesky with a drop tolerance, natural order, bounded fill)
  bool ict = false;
  int ict_noff = 0, ict_nlev = 0, ict_kcol = 0, ict_blocks = 0;
  double *ict_lo = nullptr, *ict_ld = nullptr, *ict_y = nullptr, *ict_pd = nullptr;
  double *ict_hmax = nullptr, *ict_hpart = nullptr;
  bool ict_tiled = false;      // fill levels 0 and 1, where the packed rows fit: one launch per sweep
  fm::IctSweep ict_sweep{};
  int ict_pack_grid = 1, ict_unpack_grid = 1;
};

namespace {

// Gamma = gamma (gamma^H gamma)^{-1} gamma^H (Sec. II eq. (gamma)).
std::vector<std::complex<double>> make_gamma(const fm_params &p) {
  const int L = p.necho;
  std::vector<std::complex<double>> G((size_t)L * L);
  if (p.model == FM_FIELDMAP) {
    for (auto &v : G) v = 1.0 / L;
    return G;
  }
  const double two_pi = 6.283185307179586476925286766559;
  std::vector<std::complex<double>> c(L);
  for (int l = 0; l < L; ++l) {
    std::complex<double> s = 0.0;
    for (int q = 0; q < p.npeak; ++q) s += p.fat_amp[q] * std::polar(1.0, two_pi * p.fat_hz[q] * p.te[l]);
    c[l] = s;
  }
  // normal matrix N = [[L, sum c], [sum conj c, sum |c|^2]] and its inverse
  std::complex<double> sc = 0.0;
  double cc = 0.0;
  for (int l = 0; l < L; ++l) {
    sc += c[l];
    cc += std::norm(c[l]);
  }
  const double det = L * cc - std::norm(sc);
  const std::complex<double> i00 = cc / det, i01 = -sc / det, i10 = -std::conj(sc) / det, i11 = (double)L / det;
  for (int m = 0; m < L; ++m)
    for (int n = 0; n < L; ++n)
      G[(size_t)m * L + n] = i00 + i01 * std::conj(c[n]) + c[m] * i10 + c[m] * i11 * std::conj(c[n]);
  return G;
}

// B = (gamma^H gamma)^{-1} gamma^H (K x L, row-major, interleaved complex):
// gamma = 1 (field map, K = 1) or [1, c] (water-fat, K = 2).
std::vector<double> make_component_matrix(const fm_params &p, int *K) {
  const int L = p.necho;
  const double two_pi = 6.283185307179586476925286766559;
  std::vector<double> out;
  if (p.model == FM_FIELDMAP) {
    *K = 1;
    for (int l = 0; l < L; ++l) {
      out.push_back(1.0 / L);
      out.push_back(0.0);
    }
    return out;
  }
  *K = 2;
  std::vector<std::complex<double>> c(L);
  for (int l = 0; l < L; ++l) {
    std::complex<double> v = 0.0;
    for (int q = 0; q < p.npeak; ++q) v += p.fat_amp[q] * std::polar(1.0, two_pi * p.fat_hz[q] * p.te[l]);
    c[l] = v;
  }
  std::complex<double> sc = 0.0;
  double cc = 0.0;
  for (int l = 0; l < L; ++l) {
    sc += c[l];
    cc += std::norm(c[l]);
  }
  const double det = L * cc - std::norm(sc);
  // N^{-1} = [[cc, -sc], [-conj(sc), L]] / det;  B = N^{-1} [1 ... 1; conj(c)]
  const std::complex<double> i00 = cc / det, i01 = -sc / det, i10 = -std::conj(sc) / det, i11 = (double)L / det;
  for (int k = 0; k < 2; ++k)
    for (int l = 0; l < L; ++l) {
      const std::complex<double> v = (k == 0) ? i00 + i01 * std::conj(c[l]) : i10 + i11 * std::conj(c[l]);
      out.push_back(v.real());
      out.push_back(v.imag());
    }
  return out;
}

// The setup kernel for an echo bucket and model.
template <typename T>
using SetupKernel = void (*)(fm::SetupArgs<T>);
template <typename T>
SetupKernel<T> setup_kernel(int lmax, bool wf, int necho) {
  if (wf) {  // 2-6 echoes: the exact count, by which the sweep's recurrence is unrolled
    switch (necho) {
      case 2: return fm::k_setup<T, 2, true>;
      case 3: return fm::k_setup<T, 3, true>;
      case 4: return fm::k_setup<T, 4, true>;
      case 5: return fm::k_setup<T, 5, true>;
      case 6: return fm::k_setup<T, 6, true>;
      default: return lmax <= 8 ? fm::k_setup<T, 8, true> : fm::k_setup<T, 16, true>;
    }
  }
  // the field-map model with 2-4 echoes: the exact echo count, so no echo slot is loaded or summed for nothing
  if (necho == 2) return fm::k_setup<T, 2, false>;
  if (necho == 3) return fm::k_setup<T, 3, false>;
  return lmax <= 4 ? fm::k_setup<T, 4, false> : (lmax <= 8 ? fm::k_setup<T, 8, false> : fm::k_setup<T, 16, false>);
}

template <typename T>
std::vector<fm::PairC<T>> make_pairs(const fm_params &p, const std::vector<std::complex<double>> &G) {
  std::vector<fm::PairC<T>> out;
  const double two_pi = 6.283185307179586476925286766559;
  for (int m = 0; m < p.necho; ++m)
    for (int n = m + 1; n < p.necho; ++n) {
      fm::PairC<T> q{};
      const auto g = G[(size_t)m * p.necho + n];
      q.w = (T)(2.0 * std::abs(g));
      q.g = (T)(std::arg(g) / two_pi);
      q.dt = (T)(p.te[m] - p.te[n]);
      q.d2pi = (T)(two_pi * (p.te[m] - p.te[n]));
      q.m = m;
      q.n = n;
      out.push_back(q);
    }
  return out;
}

// The water-fat sweep covers [-|df|/2, |df|/2], df the offset of the largest fat peak.
double sweep_half(const fm_params &p) {
  int big = 0;
  for (int q = 1; q < p.npeak; ++q)
    if (p.fat_amp[q] > p.fat_amp[big]) big = q;
  return std::fabs(p.fat_hz[big]) / 2.0;
}

// Arguments of chain launch number q (state and partial-sum slots by parity).
template <typename T>
fm::IterArgs<T> iter_args(fm_plan *p, uint64_t q) {
  fm::IterArgs<T> a{};
  a.geo = p->geo;
  a.L = p->prm.necho;
  a.beta = p->prm.beta;
  a.dat = (const fm::T2<T> *)p->dat;
  a.code = p->code;
  a.pairs = (const fm::PairC<T> *)p->pairs;
  for (int i = 0; i < 2; ++i) {
    a.F[i] = (T *)p->F[i];
    a.Z[i] = (T *)p->Z[i];
    a.G[i] = (T *)p->G[i];
  }
  a.D = (T *)p->D;
  a.X = (T *)p->X;
  a.X2 = (T *)p->X2;
  a.P = (T *)p->P;
  a.rdiag = p->rdiag;
  a.ccode = p->ccode;
  a.cm = p->cm ? 1 : 0;
  a.Pv = (T *)p->Pv;
  a.Dv = (T *)p->Dv;
  a.ipiv = p->ipiv;
  a.hinv = p->hinv;
  // the pair-mapped passes (even column length) keep 1/h of red and p of black voxels at the pair's index
  a.write_hinv = (p->prm.precond == FM_PRECOND_IC0 && p->prm.ordering == FM_ORDER_REDBLACK) ? (p->geo.nz % 2 ? 1 : 2) : 0;
  a.store_piv = 0;
  a.par = (int32_t)(p->iter_host & 1);
  a.nparts_in = p->last_nparts;
  a.nvals_in = p->last_nvals;
  a.sin = p->S + (q & 1);
  a.sout = p->S + ((q + 1) & 1);
  a.pin = p->part + (size_t)(q & 1) * p->part_rows * kMaxK;
  a.pout = p->part + (size_t)((q + 1) & 1) * p->part_rows * kMaxK;
  a.status = p->status;
  a.trace = p->trace;
  a.fout = nullptr;
  a.final_pass = 0;
  a.reg2 = p->reg2 ? 1 : 0;
  return a;
}

// Optional per-launch event recorder (measurement path only): the events are
// attached to the dispatch itself (hipExtLaunchKernelGGL), so they bracket the
// kernel's execution without extra packets in between.
struct Recorder {
  std::vector<hipEvent_t> ev;
  std::vector<int> cls;
  hipError_t err = hipSuccess;
  void pair(int c, hipEvent_t *e0, hipEvent_t *e1) {
    *e0 = *e1 = nullptr;
    if (err == hipSuccess) err = hipEventCreate(e0);
    if (err == hipSuccess) err = hipEventCreate(e1);
    ev.push_back(*e0);
    ev.push_back(*e1);
    cls.push_back(c);
  }
  ~Recorder() {
    for (auto e : ev)
      if (e) (void)hipEventDestroy(e);
  }
};

#define FM_LAUNCH(cls, kernel, grid, block, s, ...)                                   \
  do {                                                                                \
    if (rec) {                                                                        \
      hipEvent_t e0_, e1_;                                                            \
      rec->pair(cls, &e0_, &e1_);                                                     \
      hipExtLaunchKernelGGL(kernel, grid, block, 0, s, e0_, e1_, 0, __VA_ARGS__);     \
    } else {                                                                          \
      hipLaunchKernelGGL(kernel, grid, block, 0, s, __VA_ARGS__);                     \
    }                                                                                 \
  } while (0)

// Preconditioner step p = P^{-1} g (g from gsrc, or G[iter&1] if null),
// leaving the dot products g^T p and g_prev^T p as partial sums.
void set_parts(fm_plan *p, int nparts, int nvals) {
  p->last_nparts = nparts;
  p->last_nvals = nvals;
}

// IC_t: H_max, the factorisation with the forward solve, and the backward solve
// (outside the state chain), then the dot products.
template <typename T>
fm_status enqueue_ict_hmax(fm_plan *p, hipStream_t s, Recorder *rec) {
  FM_LAUNCH(FM_K_PRECOND_A, fm::k_ict_hmax<T>, dim3(p->grid), dim3(kBlock), s, p->geo, (const uint8_t *)p->code,
            (const T *)p->D, p->prm.beta, p->ict_hpart);
  FM_LAUNCH_CHECK();
  FM_LAUNCH(FM_K_PRECOND_A, fm::k_ict_hmax_fin, dim3(1), dim3(kBlock), s, (const double *)p->ict_hpart, p->grid,
            p->ict_hmax);
  FM_LAUNCH_CHECK();
  return FM_OK;
}

// Fill levels 0 and 1: one launch per sweep.
template <typename T, int LEVEL>
fm_status enqueue_ict_tiled(fm_plan *p, const T *g, const fm::IterArgs<T> &a, const T *gsrc, hipStream_t s, Recorder *rec) {
  const fm::IctSweep &w = p->ict_sweep;
  FM_LAUNCH(FM_K_PRECOND_A, (fm::k_ict_pack<T, LEVEL>), dim3(p->ict_pack_grid), dim3(fm::kNT), s, p->geo, p->prm.beta,
            p->prm.ict_factor, (const double *)p->ict_hmax, (const uint8_t *)p->code, (const T *)p->D, g, w);
  FM_LAUNCH_CHECK();
  FM_LAUNCH(FM_K_PRECOND_A, (fm::k_ict_fwd_wave<LEVEL>), dim3(w.ntiles), dim3(64), s, w, p->status);
  FM_LAUNCH_CHECK();
  FM_LAUNCH(FM_K_PRECOND_B, (fm::k_ict_bwd_wave<LEVEL>), dim3(w.ntiles), dim3(64), s, w, p->status);
  FM_LAUNCH_CHECK();
  FM_LAUNCH(FM_K_DOTS, (fm::k_ict_unpack<T, LEVEL>), dim3(p->ict_unpack_grid), dim3(fm::kNT), s, a, w, gsrc);
  FM_LAUNCH_CHECK();
  return FM_OK;
}

// Fill level 2, and volumes whose packed rows do not fit: a launch per level of the schedule.
template <typename T, int LEVEL>
fm_status enqueue_ict_levels(fm_plan *p, const T *g, hipStream_t s, Recorder *rec) {
  fm::IctArgs<T> a{};
  a.geo = p->geo;
  a.beta = p->prm.beta;
  a.factor = p->prm.ict_factor;
  a.hmax = p->ict_hmax;
  a.code = p->code;
  a.D = (const T *)p->D;
  a.kcol = p->ict_kcol;
  a.lo = p->ict_lo;
  a.ld = p->ict_ld;
  a.y = p->ict_y;
  a.pd = p->ict_pd;
  a.P = (T *)p->P;
  a.status = p->status;
  for (int lv = 0; lv < p->ict_nlev; ++lv)
    FM_LAUNCH(FM_K_PRECOND_A, (fm::k_ict_fwd<T, LEVEL>), dim3(p->ict_blocks), dim3(fm::kIctNT), s, a, g, lv);
  FM_LAUNCH_CHECK();
  for (int lv = p->ict_nlev - 1; lv >= 0; --lv)
    FM_LAUNCH(FM_K_PRECOND_B, (fm::k_ict_bwd<T, LEVEL>), dim3(p->ict_blocks), dim3(fm::kIctNT), s, a, lv);
  FM_LAUNCH_CHECK();
  return FM_OK;
}

// Natural-order IC(0): pack, the two sweeps (outside the state chain), unpack
// with the dot products.  ain and aout are the chain arguments of the first
// and the last of the four.
template <typename T>
fm_status enqueue_natural(fm_plan *p, const fm::IterArgs<T> &ain, const fm::IterArgs<T> &aout, const T *gsrc,
                          int32_t *status, hipStream_t s, Recorder *rec) {
  const fm::Wavefront &w = p->wf;
  FM_LAUNCH(FM_K_DOTS, fm::k_nat_pack<T>, dim3(p->wf_pack_grid), dim3(fm::kNT), s, ain, w, gsrc);
  FM_LAUNCH_CHECK();
  FM_LAUNCH(FM_K_PRECOND_A, fm::k_ic_fwd_wave<T>, dim3(w.ntiles), dim3(64), s, w, ain.beta, status);
  FM_LAUNCH_CHECK();
  FM_LAUNCH(FM_K_PRECOND_B, fm::k_ic_bwd_wave<T>, dim3(w.ntiles), dim3(64), s, w, ain.beta, status);
  FM_LAUNCH_CHECK();
  FM_LAUNCH(FM_K_DOTS, fm::k_nat_unpack<T>, dim3(p->wf_unpack_grid), dim3(fm::kNT), s, aout, w, gsrc);
  FM_LAUNCH_CHECK();
  return FM_OK;
}

// Block red-black IC(0): pack, forward colours 0 and 1, backward colours 1 and
// 0 (a volume of one tile has no colour-1 tile), unpack.
template <typename T>
fm_status enqueue_block(fm_plan *p, const fm::IterArgs<T> &ain, const fm::IterArgs<T> &aout, const T *gsrc, hipStream_t s,
                        Recorder *rec) {
  fm::Wavefront w = p->wf;
  w.ff = nullptr;  // no values pass between tiles of one launch
  FM_LAUNCH(FM_K_DOTS, fm::k_nat_pack<T>, dim3(p->wf_pack_grid), dim3(fm::kNT), s, ain, w, gsrc);
  FM_LAUNCH_CHECK();
  FM_LAUNCH(FM_K_PRECOND_A, (fm::k_icb_fwd<T, false>), dim3(w.nblk[0]), dim3(64), s, w, ain.beta, p->status, 0);
  FM_LAUNCH_CHECK();
  if (w.nblk[1] > 0) {
    FM_LAUNCH(FM_K_PRECOND_A, (fm::k_icb_fwd<T, true>), dim3(w.nblk[1]), dim3(64), s, w, ain.beta, p->status, 1);
    FM_LAUNCH_CHECK();
    FM_LAUNCH(FM_K_PRECOND_B, (fm::k_icb_bwd<T, false>), dim3(w.nblk[1]), dim3(64), s, w, ain.beta, 1);
    FM_LAUNCH_CHECK();
  }
  FM_LAUNCH(FM_K_PRECOND_B, (fm::k_icb_bwd<T, true>), dim3(w.nblk[0]), dim3(64), s, w, ain.beta, 0);
  FM_LAUNCH_CHECK();
  FM_LAUNCH(FM_K_DOTS, fm::k_nat_unpack<T>, dim3(p->wf_unpack_grid), dim3(fm::kNT), s, aout, w, gsrc);
  FM_LAUNCH_CHECK();
  return FM_OK;
}

// Either order without packed rows: the levels of both sweeps (outside the state
// chain), then the dot products.
template <typename T, bool BLOCK>
fm_status enqueue_ic_levels(fm_plan *p, const fm::IterArgs<T> &ia, const T *gsrc, hipStream_t s, Recorder *rec) {
  const fm::Geo &g = p->geo;
  if (!ia.X) return fail(FM_ERR_ALLOC, "no memory for the level sweeps (the packed rows were given back)");
  const int per_x = BLOCK ? g.ny : std::min(g.ny, g.nz), nlev = BLOCK ? g.nz + 2 * (fm::kTile - 1) : g.nx + g.ny + g.nz - 2;
  fm::LevelArgs<T> a{g,     ia.beta, ia.code, ia.D, gsrc ? gsrc : ((ia.par & 1) ? ia.G[1] : ia.G[0]),
                     ia.X,  ia.P,    ia.ipiv, ia.status, per_x};
  const dim3 grid((unsigned)(((int64_t)g.nx * per_x + fm::kLevelNT - 1) / fm::kLevelNT));
  for (int c = 0; c < (BLOCK ? 2 : 1); ++c)
    for (int lv = 0; lv < nlev; ++lv)
      FM_LAUNCH(FM_K_PRECOND_A, (fm::k_ic_level_fwd<T, BLOCK>), grid, dim3(fm::kLevelNT), s, a, lv, c);
  FM_LAUNCH_CHECK();
  for (int c = BLOCK ? 1 : 0; c >= 0; --c)
    for (int lv = nlev - 1; lv >= 0; --lv)
      FM_LAUNCH(FM_K_PRECOND_B, (fm::k_ic_level_bwd<T, BLOCK>), grid, dim3(fm::kLevelNT), s, a, lv, c);
  FM_LAUNCH_CHECK();
  FM_LAUNCH(FM_K_DOTS, (fm::k_ict_dots<T, T>), dim3(p->sgrid), dim3(fm::kNT), s, ia, (const T *)ia.P, gsrc);
  FM_LAUNCH_CHECK();
  return FM_OK;
}

template <typename T>
fm_status enqueue_precond(fm_plan *p, const T *gsrc, hipStream_t s, Recorder *rec = nullptr) {
  auto pargs = [&](fm_plan *pp, uint64_t q) {
    fm::IterArgs<T> a = iter_args<T>(pp, q);
    a.store_piv = gsrc ? 1 : 0;  // the standalone call reports the pivots
    return a;
  };
  if (p->prm.precond == FM_PRECOND_ICT) {
    const T *g = gsrc ? gsrc : (const T *)p->G[p->iter_host & 1];
    fm_status st = enqueue_ict_hmax<T>(p, s, rec);
    if (st) return st;
    if (p->ict_tiled) {
      const fm::IterArgs<T> a = pargs(p, p->q++);
      st = p->prm.ict_level == 0 ? enqueue_ict_tiled<T, 0>(p, g, a, gsrc, s, rec)
                                 : enqueue_ict_tiled<T, 1>(p, g, a, gsrc, s, rec);
      if (st) return st;
      set_parts(p, p->ict_unpack_grid, 2);
      return FM_OK;
    }
    st = p->prm.ict_level == 0   ? enqueue_ict_levels<T, 0>(p, g, s, rec)
         : p->prm.ict_level == 1 ? enqueue_ict_levels<T, 1>(p, g, s, rec)
                                 : enqueue_ict_levels<T, 2>(p, g, s, rec);
    if (st) return st;
    FM_LAUNCH(FM_K_DOTS, (fm::k_ict_dots<T, double>), dim3(p->sgrid), dim3(fm::kNT), s, pargs(p, p->q++),
              (const double *)p->ict_pd, gsrc);
    FM_LAUNCH_CHECK();
    set_parts(p, p->sgrid, 2);
  } else if (p->prm.precond == FM_PRECOND_IC0 && p->prm.ordering == FM_ORDER_COLOR3) {
    // second-order C: forward colours 0-1, forward colour 2 (+ its p), backward colours 1, 0
    FM_LAUNCH(FM_K_PRECOND_A, (fm::k_ic3_fwd1<T>), dim3(p->sgrid), dim3(fm::kNT), s, pargs(p, p->q++), gsrc);
    FM_LAUNCH_CHECK();
    set_parts(p, p->sgrid, 2);
    FM_LAUNCH(FM_K_PRECOND_A, (fm::k_ic3_fwd2<T>), dim3(p->sgrid), dim3(fm::kNT), s, pargs(p, p->q++), gsrc);
    FM_LAUNCH_CHECK();
    set_parts(p, p->sgrid, 2);
    FM_LAUNCH(FM_K_PRECOND_B, (fm::k_ic3_bwd1<T>), dim3(p->sgrid), dim3(fm::kNT), s, pargs(p, p->q++));
    FM_LAUNCH_CHECK();
    set_parts(p, 0, 0);
    FM_LAUNCH(FM_K_PRECOND_B, (fm::k_ic3_bwd0<T>), dim3(p->sgrid), dim3(fm::kNT), s, pargs(p, p->q++), gsrc);
    FM_LAUNCH_CHECK();
    set_parts(p, 0, 0);
  } else if (p->by_levels) {
    const fm::IterArgs<T> a = pargs(p, p->q++);
    fm_status st = p->prm.ordering == FM_ORDER_BLOCKRB ? enqueue_ic_levels<T, true>(p, a, gsrc, s, rec)
                                                       : enqueue_ic_levels<T, false>(p, a, gsrc, s, rec);
    if (st) return st;
    set_parts(p, p->sgrid, 2);
  } else if (p->prm.precond == FM_PRECOND_IC0 && p->prm.ordering == FM_ORDER_BLOCKRB) {
    const fm::IterArgs<T> ain = pargs(p, p->q++);
    set_parts(p, 0, 0);
    fm_status st = enqueue_block<T>(p, ain, pargs(p, p->q++), gsrc, s, rec);
    if (st) return st;
    set_parts(p, p->wf_unpack_grid, 2);
  } else if (p->prm.precond == FM_PRECOND_IC0) {
    if (p->prm.ordering == FM_ORDER_NATURAL) {
      const fm::IterArgs<T> ain = pargs(p, p->q++);
      set_parts(p, 0, 0);
      fm_status st = enqueue_natural<T>(p, ain, pargs(p, p->q++), gsrc, p->status, s, rec);
      if (st) return st;
      set_parts(p, p->wf_unpack_grid, 2);
    } else {
      FM_LAUNCH(FM_K_PRECOND_A, (fm::k_rb_black<T, false>), dim3(p->sgrid), dim3(fm::kNT), s, pargs(p, p->q++), gsrc);
      FM_LAUNCH_CHECK();
      set_parts(p, p->sgrid, 2);
      FM_LAUNCH(FM_K_PRECOND_B, (fm::k_rb_red<T, false>), dim3(p->sgrid), dim3(fm::kNT), s, pargs(p, p->q++), gsrc);
      FM_LAUNCH_CHECK();
      set_parts(p, p->sgrid, 2);
    }
  } else if (p->reg2) {
    FM_LAUNCH(FM_K_PRECOND_A, (fm::k_diag2<T>), dim3(p->sgrid), dim3(fm::kNT), s, pargs(p, p->q++), gsrc,
              p->prm.precond == FM_PRECOND_NONE ? 1 : 0);
    FM_LAUNCH_CHECK();
    set_parts(p, p->sgrid, 2);
  } else {
    FM_LAUNCH(FM_K_PRECOND_A, (fm::k_diag<T, false>), dim3(p->sgrid), dim3(fm::kNT), s, pargs(p, p->q++), gsrc,
                       p->prm.precond == FM_PRECOND_NONE ? 1 : 0);
    FM_LAUNCH_CHECK();
    set_parts(p, p->sgrid, 2);
  }
  return FM_OK;
}

// Launches per iteration (must match enqueue_iteration).
uint64_t launches_per_iteration(const fm_plan *p) {
  // preconditioner passes + direction; red-black IC(0) forms the direction in its red pass
  uint64_t precond_dir = 2;
  if (p->prm.precond == FM_PRECOND_IC0 && p->prm.ordering == FM_ORDER_NATURAL) precond_dir = 3;
  if (p->prm.precond == FM_PRECOND_IC0 && p->prm.ordering == FM_ORDER_COLOR3) precond_dir = 5;
  if (p->prm.precond == FM_PRECOND_IC0 && p->prm.ordering == FM_ORDER_BLOCKRB) precond_dir = 3;
  if (p->by_levels) precond_dir = 2;
  return 1 + precond_dir + (uint64_t)(p->prm.nmls - 1);
}

bool fused_red_dir(const fm_plan *p) {
  return p->prm.precond == FM_PRECOND_IC0 && p->prm.ordering == FM_ORDER_REDBLACK;
}

// Values per partial block left by the last pass of an iteration.
int tail_nvals(const fm_plan *p) { return p->prm.nmls > 1 ? 2 : 3; }


// Plane-march shape of the tiled red-black passes: strips of ty columns (all
// pair slots of a workgroup on one plane), runs of 4 planes, of fewer where
// that leaves compute units without a workgroup (a run is a serial chain; with
// 512 workgroups aimed at instead of 256, 91x109x91 F64 took 3.35 ms, not 3.19),
// lengthened until the grid fits the partial-sum rows.  grid 0 where the tile
// does not apply (odd or long columns).
fm::TileShape tile_shape(const fm::Geo &g) {
  fm::TileShape t{};
  if (g.nz % 2 != 0 || g.nz > fm::kTileMaxNz) return t;
  const int nzp = g.nz / 2;
  t.ty = std::min(fm::kTileSlots / nzp, g.ny);
  t.nyt = (g.ny + t.ty - 1) / t.ty;
  if (t.nyt > kMaxGrid) return fm::TileShape{};
  const int64_t planes = (int64_t)t.nyt * g.nx;  // over all strips
  t.xc = std::max<int>((int)std::clamp<int64_t>(planes / 256, 1, 4), (int)((planes + kMaxGrid - 1) / kMaxGrid));
  while ((int64_t)t.nyt * ((g.nx + t.xc - 1) / t.xc) > kMaxGrid) ++t.xc;
  t.grid = t.nyt * ((g.nx + t.xc - 1) / t.xc);
  return t;
}

// Workgroups (hence partial sums) of the last pass of an iteration: a line-search
// pass, or the direction step's last pass (tiled or not) when there is none.
int tail_nparts(const fm_plan *p) {
  if (p->prm.nmls > 1) return p->sgrid;
  const fm::TileShape ts = fused_red_dir(p) ? tile_shape(p->geo) : fm::TileShape{};
  return ts.grid > 0 ? ts.grid : p->sgrid;
}

// The four-voxel passes of a plan (2-6 echoes).  With 2-4 echoes they load early where a thread has
// two fours or more (at five and six the registers are too many; the second-order gradient has no such form).
using QuadKernel = void (*)(fm::IterArgs<float>);
struct QuadKernels {
  QuadKernel grad, mls;
};
template <int NE>
QuadKernels quad_kernels_of(bool order2, bool early) {
  if constexpr (NE <= 4)
    if (early) return {order2 ? fm::k_grad2_q<NE> : fm::k_grad_q<NE, false, true>, fm::k_mls_q<NE, false, true>};
  return {order2 ? fm::k_grad2_q<NE> : fm::k_grad_q<NE, false>, fm::k_mls_q<NE, false>};
}
QuadKernels quad_kernels(const fm_plan *p) {
  const bool early = p->n >= (int64_t)8 * kMaxGrid * fm::kNT;
  switch (p->prm.necho) {
    case 2: return quad_kernels_of<2>(p->reg2, early);
    case 3: return quad_kernels_of<3>(p->reg2, early);
    case 4: return quad_kernels_of<4>(p->reg2, early);
    case 5: return quad_kernels_of<5>(p->reg2, early);
    default: return quad_kernels_of<6>(p->reg2, early);
  }
}

// One NCG iteration: gradient, preconditioner (+ dots), direction, and the
// remaining line-search passes; the last pass is consumed by the next
// iteration's gradient pass (or by the final pass).
template <typename T, int LMAX>
fm_status enqueue_iteration(fm_plan *p, hipStream_t s, Recorder *rec = nullptr) {
  // FP32, 2-6 echoes, columns a multiple of 4, not a thread per voxel: the 16-byte-load passes
  // (gradient passes of either stencil; the line-search passes have none)
  const bool quad = std::is_same<T, float>::value && p->prm.necho <= 6 && p->geo.nz % 4 == 0 && !p->few;
  auto launch_quad = [&](int cls, QuadKernel k) {
    FM_LAUNCH(cls, k, dim3(p->sgrid), dim3(fm::kNT), s, iter_args<float>(p, p->q++));
  };
  if (quad) {
    launch_quad(FM_K_GRAD, quad_kernels(p).grad);
  } else if (p->reg2) {
    FM_LAUNCH(FM_K_GRAD, (fm::k_grad2<T, LMAX>), dim3(p->sgrid), dim3(fm::kNT), s, iter_args<T>(p, p->q++));
  } else if (p->few) {
    FM_LAUNCH(FM_K_GRAD, (fm::k_grad<T, LMAX, false, 1>), dim3(p->sgrid), dim3(fm::kNT), s, iter_args<T>(p, p->q++));
  } else {
    FM_LAUNCH(FM_K_GRAD, (fm::k_grad<T, LMAX, false, fm::kVGrad<T>>), dim3(p->sgrid), dim3(fm::kNT), s,
              iter_args<T>(p, p->q++));
  }
  FM_LAUNCH_CHECK();
  set_parts(p, p->sgrid, 4);
  const fm::TileShape ts = fused_red_dir(p) ? tile_shape(p->geo) : fm::TileShape{};
  int dir_parts = p->sgrid;  // workgroups of the pass that ends the direction step
  if (ts.grid > 0) {
    FM_LAUNCH(FM_K_PRECOND_A, (fm::k_rb_black_tile<T, false>), dim3(ts.grid), dim3(fm::kNT), s, iter_args<T>(p, p->q++), ts);
    FM_LAUNCH_CHECK();
    set_parts(p, ts.grid, 2);
    FM_LAUNCH(FM_K_PRECOND_B, (fm::k_rb_red_dir_tile<T, false>), dim3(ts.grid), dim3(fm::kNT), s, iter_args<T>(p, p->q++),
              ts);
    FM_LAUNCH_CHECK();
    dir_parts = ts.grid;
  } else if (fused_red_dir(p) && p->geo.nz % 2 == 0) {
    FM_LAUNCH(FM_K_PRECOND_A, (fm::k_rb_black_pair<T, false>), dim3(p->sgrid), dim3(fm::kNT), s, iter_args<T>(p, p->q++));
    FM_LAUNCH_CHECK();
    set_parts(p, p->sgrid, 2);
    FM_LAUNCH(FM_K_PRECOND_B, (fm::k_rb_red_dir_pair<T, false>), dim3(p->sgrid), dim3(fm::kNT), s,
              iter_args<T>(p, p->q++));
    FM_LAUNCH_CHECK();
  } else if (fused_red_dir(p)) {
    FM_LAUNCH(FM_K_PRECOND_A, (fm::k_rb_black<T, false, true>), dim3(p->sgrid), dim3(fm::kNT), s,
              iter_args<T>(p, p->q++), (const T *)nullptr);
    FM_LAUNCH_CHECK();
    set_parts(p, p->sgrid, 2);
    FM_LAUNCH(FM_K_PRECOND_B, (fm::k_rb_red_dir<T, false>), dim3(p->sgrid), dim3(fm::kNT), s, iter_args<T>(p, p->q++));
    FM_LAUNCH_CHECK();
  } else {
    fm_status st = enqueue_precond<T>(p, nullptr, s, rec);
    if (st) return st;
    if (p->cm) {  // the direction pass reads the voxel-order copies of p and D
      fm::IterArgs<T> a = iter_args<T>(p, p->q++);
      a.P = (T *)p->Pv;
      a.D = (T *)p->Dv;
      FM_LAUNCH(FM_K_DIR, (fm::k_dir2<T>), dim3(p->sgrid), dim3(fm::kNT), s, a);
    } else if (p->reg2) {
      FM_LAUNCH(FM_K_DIR, (fm::k_dir2<T>), dim3(p->sgrid), dim3(fm::kNT), s, iter_args<T>(p, p->q++));
    } else {
      if (p->few)
        FM_LAUNCH(FM_K_DIR, (fm::k_dir<T, false, 1>), dim3(p->sgrid), dim3(fm::kNT), s, iter_args<T>(p, p->q++));
      else
        FM_LAUNCH(FM_K_DIR, (fm::k_dir<T, false, fm::Vpt<T>::v>), dim3(p->sgrid), dim3(fm::kNT), s, iter_args<T>(p, p->q++));
    }
    FM_LAUNCH_CHECK();
  }
  set_parts(p, dir_parts, 3);
  for (int k = 1; k < p->prm.nmls; ++k) {
    if (quad) {
      launch_quad(FM_K_MLS, quad_kernels(p).mls);
    } else if (p->few) {
      FM_LAUNCH(FM_K_MLS, (fm::k_mls<T, LMAX, false, 1>), dim3(p->sgrid), dim3(fm::kNT), s, iter_args<T>(p, p->q++));
    } else {
      FM_LAUNCH(FM_K_MLS, (fm::k_mls<T, LMAX, false, fm::kVMls<T, LMAX>>), dim3(p->sgrid), dim3(fm::kNT), s,
                iter_args<T>(p, p->q++));
    }
    FM_LAUNCH_CHECK();
    set_parts(p, p->sgrid, 2);
  }
  p->iter_host += 1;
  return FM_OK;
}

// Final pass: apply the last step, write the map, and record its cost.
template <typename T, int LMAX>
fm_status enqueue_final(fm_plan *p, double *f_out, hipStream_t s) {
  fm::IterArgs<T> a = iter_args<T>(p, p->q++);
  a.final_pass = 1;
  a.fout = f_out;
  if (p->reg2)
    hipLaunchKernelGGL((fm::k_grad2<T, LMAX>), dim3(p->sgrid), dim3(fm::kNT), 0, s, a);
  else
    hipLaunchKernelGGL((fm::k_grad<T, LMAX, false, fm::kVGrad<T>>), dim3(p->sgrid), dim3(fm::kNT), 0, s, a);
  FM_LAUNCH_CHECK();
  set_parts(p, p->sgrid, 4);
  const uint64_t q = p->q++;
  hipLaunchKernelGGL(fm::k_finish, dim3(1), dim3(kBlock), 0, s, (const fm::State *)(p->S + (q & 1)),
                     p->S + ((q + 1) & 1), (const double *)(p->part + (size_t)(q & 1) * p->part_rows * kMaxK),
                     p->last_nparts, p->last_nvals, p->prm.beta, p->trace, p->status);
  FM_LAUNCH_CHECK();
  set_parts(p, 0, 0);
  return FM_OK;
}

template <typename T, int LMAX>
fm_status enqueue_eval(fm_plan *p, const double *f, double *phi, double *dphi, double *curv, double *lap,
                       hipStream_t s) {
  fm::IterArgs<T> a = iter_args<T>(p, 0);
  hipLaunchKernelGGL((fm::k_eval<T, LMAX>), dim3(p->grid), dim3(kBlock), 0, s, a, f, phi, dphi, curv, lap);
  FM_LAUNCH_CHECK();
  return FM_OK;
}

// Dispatch on the working type and the echo-count bucket.
template <template <typename, int> class Op, typename... Args>
fm_status dispatch(fm_plan *p, Args... args) {
  if (p->mix) {
    switch (p->lmax) {
      case 4: return Op<float, 4>::run(p, args...);
      case 8: return Op<float, 8>::run(p, args...);
      default: return Op<float, 16>::run(p, args...);
    }
  }
  switch (p->lmax) {
    case 4: return Op<double, 4>::run(p, args...);
    case 8: return Op<double, 8>::run(p, args...);
    default: return Op<double, 16>::run(p, args...);
  }
}

template <typename T, int LMAX>
struct OpLoop {
  static fm_status run(fm_plan *p, int niter, hipStream_t s) {
    for (int i = 0; i < niter; ++i) {
      fm_status st = enqueue_iteration<T, LMAX>(p, s);
      if (st) return st;
    }
    return FM_OK;
  }
};
template <typename T, int LMAX>
struct OpIterationTimed {
  static fm_status run(fm_plan *p, hipStream_t s, Recorder *rec) { return enqueue_iteration<T, LMAX>(p, s, rec); }
};
template <typename T, int LMAX>
struct OpFinal {
  static fm_status run(fm_plan *p, double *f, hipStream_t s) { return enqueue_final<T, LMAX>(p, f, s); }
};
template <typename T, int LMAX>
struct OpEval {
  static fm_status run(fm_plan *p, const double *f, double *a, double *b, double *c, double *d, hipStream_t s) {
    return enqueue_eval<T, LMAX>(p, f, a, b, c, d, s);
  }
};

fm_status validate(const fm_params *p) {
  if (!p) return fail(FM_ERR_ARG, "params is NULL");
  if (p->nx < 1 || p->ny < 1 || p->nz < 1) return fail(FM_ERR_SHAPE, "grid sizes must be >= 1");
  if (p->ncoil < 1) return fail(FM_ERR_SHAPE, "ncoil must be >= 1");
  if (p->necho < 2 || p->necho > FM_MAX_ECHO) return fail(FM_ERR_SHAPE, "necho must be in [2, 16]");
  for (int l = 0; l < p->necho; ++l)
    if (!std::isfinite(p->te[l])) return fail(FM_ERR_ARG, "echo times must be finite");
  if (!(p->beta >= 0.0) || !std::isfinite(p->beta)) return fail(FM_ERR_ARG, "beta must be finite and >= 0");
  if (p->niter < 0) return fail(FM_ERR_ARG, "niter must be >= 0");
  if (p->nmls < 1) return fail(FM_ERR_ARG, "nmls must be >= 1");
  if (p->model != FM_FIELDMAP && p->model != FM_WATERFAT) return fail(FM_ERR_ARG, "bad model");
  if (p->precision != FM_PREC_F64 && p->precision != FM_PREC_MIX) return fail(FM_ERR_ARG, "bad precision");
  if (p->ordering != FM_ORDER_NATURAL && p->ordering != FM_ORDER_REDBLACK && p->ordering != FM_ORDER_COLOR3 &&
      p->ordering != FM_ORDER_BLOCKRB)
    return fail(FM_ERR_ARG, "bad ordering");
  if (p->precond < FM_PRECOND_IC0 || p->precond > FM_PRECOND_ICT) return fail(FM_ERR_ARG, "bad preconditioner");
  if (p->reg_order < 0 || p->reg_order > 2) return fail(FM_ERR_ARG, "reg_order must be 1 or 2");
  if (p->reg_order == 2 && p->precond == FM_PRECOND_IC0 && p->ordering != FM_ORDER_COLOR3)
    return fail(FM_ERR_ARG, "IC(0) with second-order differences is built in three-colour order (FM_ORDER_COLOR3)");
  // (a bound of the entry point, from when the sweeps had 32-bit offsets into a tile's planes)
  if (p->ordering == FM_ORDER_BLOCKRB && (int64_t)p->ny * p->nz * 80 >= ((int64_t)1 << 30))
    return fail(FM_ERR_SHAPE, "block red-black order needs ny * nz * 80 below 2^30");
  if (p->ordering == FM_ORDER_COLOR3 && (p->reg_order != 2 || p->precond != FM_PRECOND_IC0))
    return fail(FM_ERR_ARG, "three-colour order is built for IC(0) with second-order differences only");
  if (p->precond == FM_PRECOND_ICT) {
    if (p->ordering != FM_ORDER_NATURAL) return fail(FM_ERR_ARG, "IC_t is built in natural order");
    if (p->reg_order == 2) return fail(FM_ERR_ARG, "IC_t is built for first-order differences");
    if (p->ict_level < 0 || p->ict_level > 2) return fail(FM_ERR_ARG, "ict_level must be 0, 1 or 2");
    if (!(p->ict_factor >= 0.0) || !std::isfinite(p->ict_factor)) return fail(FM_ERR_ARG, "ict_factor must be finite, >= 0");
  }
  if (p->model == FM_FIELDMAP && p->te[1] == p->te[0])
    return fail(FM_ERR_ARG, "field-map initialisation needs t_2 != t_1");
  if (p->model == FM_WATERFAT) {
    if (p->npeak < 1 || p->npeak > FM_MAX_PEAK) return fail(FM_ERR_ARG, "water-fat needs 1..16 fat peaks");
    if (p->nsweep < 2) return fail(FM_ERR_ARG, "water-fat sweep needs >= 2 values");
    if (p->pwls_iters < 0) return fail(FM_ERR_ARG, "pwls_iters must be >= 0");
  }
  const int64_t n = (int64_t)p->nx * p->ny * p->nz;
  if (n > (int64_t)1 << 34) return fail(FM_ERR_SHAPE, "volume too large");
  return FM_OK;
}

bool plan_alloc(fm_plan *p, void **ptr, size_t bytes) {
  void *b = nullptr;
  if (hipMalloc(&b, bytes ? bytes : 1) != hipSuccess) {
    (void)hipGetLastError();  // (the caller may have another way; a later launch must not see the error)
    return false;
  }
  p->bases.push_back(b);
  *ptr = b;
  return true;
}

// Per-voxel array of elems entries of esize bytes with p->pad guard entries
// on each side (readable neighbour slots outside the volume).
bool plan_alloc_padded(fm_plan *p, void **ptr, size_t elems, size_t esize) {
  void *b = nullptr;
  if (!plan_alloc(p, &b, (elems + 2 * (size_t)p->pad) * esize)) return false;
  *ptr = (char *)b + (size_t)p->pad * esize;
  return true;
}

template <typename T>
fm_status upload_pairs(fm_plan *p, const std::vector<std::complex<double>> &G, void **dst) {
  auto pr = make_pairs<T>(p->prm, G);
  p->npairs = (int)pr.size();
  if (!plan_alloc(p, dst, sizeof(fm::PairC<T>) * pr.size())) return fail(FM_ERR_ALLOC, "hipMalloc of pairs failed");
  FM_HIP(hipMemcpy(*dst, pr.data(), sizeof(fm::PairC<T>) * pr.size(), hipMemcpyHostToDevice));
  return FM_OK;
}

// IC(0) swept tile by tile (natural and block red-black order).
bool sweeps_in_tiles(const fm_plan *p) {
  return p->prm.precond == FM_PRECOND_IC0 && (p->prm.ordering == FM_ORDER_NATURAL || p->prm.ordering == FM_ORDER_BLOCKRB);
}

// Free what the plan has allocated since it had `mark` allocations.
void plan_free_from(fm_plan *p, size_t mark) {
  while (p->bases.size() > mark) {
    (void)hipFree(p->bases.back());
    p->bases.pop_back();
  }
}

// Packed rows hold the steps of a tile's skew too, so short columns make them many times
// the volume.  They are taken up to 4 GiB, beyond that up to `per_voxel` bytes a voxel: a
// plan's memory stays within that of the forms that need none.  (The 4 GiB are reached by
// a single slice of 2400x2400 in F64, or by 30 million voxels in columns of 10.)
bool packed_rows_fit(size_t bytes, size_t n, size_t per_voxel) {
  return bytes <= std::max((size_t)4 << 30, per_voxel * n);
}

size_t face_values(const fm::Wavefront &w) { return ((size_t)w.ntiles + 1) * w.frow * fm::kFaceSlots; }

// Face buffers and tickets of the natural-order sweeps: rows past a sweep and
// the last tile (no neighbour) stay 0.  Cleared on the stream whose sweeps come first.
fm_status alloc_faces(fm_plan *p, hipStream_t s) {
  fm::Wavefront &w = p->wf;
  const size_t faces = face_values(w);
  void *ff = nullptr, *fp = nullptr, *tk = nullptr;
  if (!plan_alloc(p, &ff, sizeof(fm::Rec) * faces) || !plan_alloc(p, &fp, p->tsize * faces) ||
      !plan_alloc(p, &tk, sizeof(uint32_t) * 2))
    return fail(FM_ERR_ALLOC, "hipMalloc of the face buffers failed");
  p->wf_bases[2] = ff;
  p->wf_bases[3] = fp;
  if (hipMemsetAsync(ff, 0, sizeof(fm::Rec) * faces, s) != hipSuccess ||
      hipMemsetAsync(fp, 0, p->tsize * faces, s) != hipSuccess)
    return fail(FM_ERR_HIP, "hipMemset of the face buffers failed");
  w.ff = (fm::Rec *)ff;
  w.fp = fp;
  w.ticket = (uint32_t *)tk;
  return FM_OK;
}

// The face buffers have been freed.
void drop_faces(fm_plan *p) {
  p->wf.ff = nullptr;
  p->wf_bases[2] = p->wf_bases[3] = nullptr;
}

// Packed rows of the natural and block red-black sweeps, or what a launch per level takes
// in their place (the face buffers are the natural order's; a block red-black plan gets
// them with the adjoint's workspace).
fm_status alloc_sweep_rows(fm_plan *p) {
  fm::Wavefront &w = p->wf;
  const int U = fm::kNatU, nz = p->geo.nz;
  w.nrow = (nz + 2 * (fm::kTile - 1) + 1 + 2 * U - 1) / (2 * U) * (2 * U);
  w.trow = w.nrow + fm::kTile;
  w.frow = w.nrow + U + fm::kTile - 1;
  const size_t guard = (size_t)(U + fm::kTile) * 64;  // rows read past either end
  const size_t packed = ((size_t)w.ntiles + 1) * w.trow * 64 + 2 * guard, value = sizeof(fm::Rec) + p->tsize;
  const bool natural = p->prm.ordering == FM_ORDER_NATURAL;
  const size_t mark = p->bases.size();
  void *rec = nullptr, *pv = nullptr;
  if (!packed_rows_fit(value * (packed + (natural ? face_values(w) : 0)), (size_t)p->n, 64) ||
      !plan_alloc(p, &rec, sizeof(fm::Rec) * packed) || !plan_alloc(p, &pv, p->tsize * packed) ||
      (natural && alloc_faces(p, nullptr) != FM_OK)) {
    plan_free_from(p, mark);
    drop_faces(p);
    p->by_levels = true;
    if (!plan_alloc_padded(p, &p->X, (size_t)p->n, p->tsize)) return fail(FM_ERR_ALLOC, "hipMalloc of p->X failed");
    return FM_OK;
  }
  p->wf_bases[0] = rec;
  p->wf_bases[1] = pv;
  if (hipMemset(rec, 0, sizeof(fm::Rec) * packed) != hipSuccess || hipMemset(pv, 0, p->tsize * packed) != hipSuccess)
    return fail(FM_ERR_HIP, "hipMemset of the sweep arrays failed");
  w.rec = (fm::Rec *)rec + guard;
  w.p = (char *)pv + p->tsize * guard;
  const int64_t units = (int64_t)w.ntiles * w.nrow, wpb = fm::kNT / fm::kWave;
  p->wf_pack_grid = (int)std::min<int64_t>(8 * kMaxGrid, (units + wpb - 1) / wpb);
  p->wf_unpack_grid = (int)std::min<int64_t>(kMaxGrid, (int64_t)w.ntiles * ((nz + fm::kUnpackZ - 1) / fm::kUnpackZ));
  return FM_OK;
}

// Tables and arrays of the tiled IC_t sweeps (fm_ict_tile.hpp); leaves ict_tiled unset
// where their packed rows do not fit.
template <int LEVEL>
fm_status alloc_ict_sweep(fm_plan *p) {
  using C = fm::IctTile<LEVEL>;
  fm::IctSweep &w = p->ict_sweep;
  const int U = fm::kIctU, t = fm::kTile;
  w.ntx = (p->geo.nx + t - 1) / t;
  w.nty = (p->geo.ny + 7 * C::K + t - 1) / t;
  w.ntiles = w.ntx * w.nty;
  w.nrow = (p->geo.nz + C::skew + 2 * U - 1) / (2 * U) * (2 * U);
  w.frow = w.nrow + 8 * (C::K + 1) + 8 + U;
  std::vector<int2> order;
  order.reserve((size_t)w.ntiles);
  for (int i = 0; i < w.ntx; ++i)
    for (int c = 0; c < w.nty; ++c) order.push_back(make_int2(i, c));
  auto first = [](int2 v) { return v.x + (int64_t)(C::K + 1) * (C::K * v.x + v.y); };  // its first step / 8
  std::stable_sort(order.begin(), order.end(), [&](int2 a, int2 b) { return first(a) < first(b); });
  const size_t row = (size_t)C::planes * 64, packed = ((size_t)w.ntiles * w.nrow + 2 * U) * row;
  const size_t faces = ((size_t)w.ntiles + 1) * w.frow * fm::kFaceSlots;
  void *ord = nullptr, *tk = nullptr, *rec = nullptr, *ff = nullptr, *fb = nullptr;
  const size_t mark = p->bases.size();
  if (!packed_rows_fit(sizeof(fm::Rec) * (packed + faces * (C::fr + C::br)), (size_t)p->n, 256) ||
      !plan_alloc(p, &ord, sizeof(int2) * order.size()) || !plan_alloc(p, &tk, sizeof(uint32_t) * 2) ||
      !plan_alloc(p, &rec, sizeof(fm::Rec) * packed) || !plan_alloc(p, &ff, sizeof(fm::Rec) * faces * C::fr) ||
      !plan_alloc(p, &fb, sizeof(fm::Rec) * faces * C::br)) {
    plan_free_from(p, mark);
    return FM_OK;
  }
  if (hipMemcpy(ord, order.data(), sizeof(int2) * order.size(), hipMemcpyHostToDevice) != hipSuccess ||
      hipMemset(rec, 0, sizeof(fm::Rec) * packed) != hipSuccess)
    return fail(FM_ERR_HIP, "set-up of the IC_t sweep arrays failed");
  w.order = (const int2 *)ord;
  w.ticket = (uint32_t *)tk;
  w.rec = (fm::Rec *)rec + U * row;
  w.ff = (fm::Rec *)ff;
  w.fb = (fm::Rec *)fb;
  hipLaunchKernelGGL(fm::k_ict_faces<LEVEL>, dim3(kMaxGrid), dim3(kBlock), 0, nullptr, w);
  FM_LAUNCH_CHECK();
  FM_HIP(hipStreamSynchronize(nullptr));
  const int64_t units = (int64_t)w.ntiles * w.nrow, wpb = fm::kNT / fm::kWave;
  p->ict_pack_grid = (int)std::min<int64_t>(8 * kMaxGrid, (units + wpb - 1) / wpb);
  p->ict_unpack_grid = (int)std::min<int64_t>(kMaxGrid, (int64_t)w.ntiles * ((p->geo.nz + fm::kUnpackZ - 1) / fm::kUnpackZ));
  p->ict_tiled = true;
  return FM_OK;
}

fm_status wf_init(fm_plan *p, double *f0, hipStream_t s);  // fm_waterfat.inc

void drop_graphs(fm_plan *p) {
  for (auto &kv : p->graphs) {
    if (kv.second.second) (void)hipGraphExecDestroy(kv.second.second);
    if (kv.second.first) (void)hipGraphDestroy(kv.second.first);
  }
  p->graphs.clear();
}

// Give the packed rows back for memory that is needed otherwise; later calls run a
// launch per level.  False where there are none.
bool give_back_rows(fm_plan *p) {
  if (!sweeps_in_tiles(p) || p->by_levels || hipDeviceSynchronize() != hipSuccess) return false;
  drop_graphs(p);  // they hold launches on the packed rows
  for (void *&b : p->wf_bases) {
    const auto it = std::find(p->bases.begin(), p->bases.end(), b);
    if (b && it != p->bases.end()) {
      (void)hipFree(b);
      p->bases.erase(it);
    }
    b = nullptr;
  }
  drop_faces(p);
  p->by_levels = true;
  return plan_alloc_padded(p, &p->X, (size_t)p->n, p->tsize);
}

void free_plan(fm_plan *p) {
  if (!p) return;
  drop_graphs(p);
  if (p->cap_stream) (void)hipStreamDestroy(p->cap_stream);
  for (hipEvent_t e : p->a_copied)
    if (e) (void)hipEventDestroy(e);
  if (p->a_host) (void)hipHostFree(p->a_host);
  for (void *b : p->bases)
    if (b) (void)hipFree(b);
  delete p;
}

// Run niter iterations as one graph launch.  The graph for the current chain
// parity and niter is captured on first use and replayed afterwards (its
// launches occupy the same chain positions modulo 2).
bool use_resident(const fm_plan *p) {
  return p->res_ok && (p->sched == FM_SCHED_RESIDENT || (p->sched == FM_SCHED_AUTO && p->res_auto));
}

size_t res_bar_bytes(const fm_plan *p) { return sizeof(uint32_t) * (fm::kResBarHead + (size_t)p->res_grid); }

template <int LR>
void *resident_kernel() {
  return (void *)fm::k_resident<LR>;
}

void *resident_kernel_for(int necho) {
  return necho <= 2 ? resident_kernel<2>() : (necho == 3 ? resident_kernel<3>() : resident_kernel<4>());
}

// An ordinary launch: the plan has checked that the whole grid fits on the
// device at once (occupancy x compute units), and every wait inside the
// kernel is bounded, so a grid that is not fully resident (another kernel
// holding compute units) ends with FM_ERR_TIMEOUT instead of hanging.  The
// events, when given, are attached to the dispatch itself.
template <int LR>
hipError_t launch_resident(const fm::ResArgs &a, int grid, hipStream_t s, hipEvent_t e0, hipEvent_t e1) {
  if (e0 && e1)
    hipExtLaunchKernelGGL(fm::k_resident<LR>, dim3(grid), dim3(fm::kResNT), 0, s, e0, e1, 0, a);
  else
    hipLaunchKernelGGL(fm::k_resident<LR>, dim3(grid), dim3(fm::kResNT), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_resident_for(int necho, const fm::ResArgs &a, int grid, hipStream_t s, hipEvent_t e0,
                               hipEvent_t e1) {
  return necho <= 2 ? launch_resident<2>(a, grid, s, e0, e1)
                    : (necho == 3 ? launch_resident<3>(a, grid, s, e0, e1) : launch_resident<4>(a, grid, s, e0, e1));
}

// niter iterations in one launch of the resident schedule.
fm_status run_resident(fm_plan *p, int niter, hipStream_t s, hipEvent_t e0 = nullptr, hipEvent_t e1 = nullptr) {
  fm::ResArgs a{};
  a.geo = p->geo;
  a.tile = p->res_tile;
  a.beta = p->prm.beta;
  a.dat = (const fm::T2<float> *)p->dat;
  a.code = p->code;
  a.pairs = (const fm::PairC<float> *)p->pairs;
  for (int i = 0; i < 2; ++i) {
    a.F[i] = (float *)p->F[i];
    a.Z[i] = (float *)p->Z[i];
    a.G[i] = (float *)p->G[i];
  }
  a.Gr = (float *)p->X;  // n floats: the two parity halves of the red face voxels' g (unused otherwise in red-black order)
  a.P = (float *)p->P;
  a.hinv = p->hinv;
  a.par0 = (int32_t)(p->iter_host & 1);
  a.niter = niter;
  a.nparts_in = p->last_nparts;
  a.nvals_in = p->last_nvals;
  const uint64_t q = p->q;
  a.sin = p->S + (q & 1);
  a.sout = p->S + ((q + 1) & 1);
  a.pin = p->part + (size_t)(q & 1) * p->part_rows * kMaxK;
  a.part = p->res_part;
  a.bar = p->res_bar;
  a.status = p->status;
  a.trace = p->trace;
  FM_HIP(hipMemsetAsync(p->res_bar, 0, res_bar_bytes(p), s));
  hipError_t err = launch_resident_for(p->prm.necho, a, p->res_grid, s, e0, e1);
  if (err != hipSuccess) return fail(FM_ERR_HIP, std::string("resident launch: ") + hipGetErrorString(err));
  p->q += 1;
  p->iter_host += niter;
  set_parts(p, 0, 0);
  return FM_OK;
}

// Tiles of whole columns for the resident schedule: at most kResTile voxels
// each, all resident at once.  Every barrier waits for the most loaded CU, so
// the tiling minimises the voxels of the busiest CU (tiles per CU rounded up
// times voxels per tile), then the number of tiles, then the tile perimeter.  False if the plan does
// not qualify.  res_auto: the volume is large enough for the resident
// schedule to beat streaming (measured: below about 1024 voxels per CU the
// fixed cost of its grid barriers dominates).
bool plan_resident(fm_plan *p) {
  const fm_params &q = p->prm;
  if (!p->mix || q.precond != FM_PRECOND_IC0 || q.ordering != FM_ORDER_REDBLACK || q.necho < 2 || q.necho > 4)
    return false;
  // voxel pairs (z even, z odd) of one column: one red and one black voxel
  if (q.nz > fm::kResTile || q.nz % 2) return false;
  int ncu = 0, per = 0;
  if (hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, p->device) != hipSuccess || ncu < 1)
    return false;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per, resident_kernel_for(q.necho), fm::kResNT, 0) != hipSuccess ||
      per < 1)
    return false;
  const long maxblocks = (long)per * ncu;
  const int C = fm::kResTile / q.nz;  // columns per tile, at most
  long best_cost = -1, best_nt = 0;
  for (int tx = 1; tx <= C && tx <= q.nx; ++tx)
    for (int ty = 1; tx * ty <= C && ty <= q.ny; ++ty) {
      // at most one neighbour across a tile face per axis: tiles at least 2 wide (or the whole axis)
      if ((tx < 2 && q.nx > 1) || (ty < 2 && q.ny > 1)) continue;
      const long nt = (long)((q.nx + tx - 1) / tx) * ((q.ny + ty - 1) / ty);
      if (nt > maxblocks) continue;
      const long cost = ((nt + ncu - 1) / ncu) * (long)tx * ty * q.nz;
      const bool squarer = tx + ty < p->res_tile.tx + p->res_tile.ty;  // shorter perimeter: less halo
      if (best_cost < 0 || cost < best_cost || (cost == best_cost && (nt < best_nt || (nt == best_nt && squarer)))) {
        best_cost = cost;
        best_nt = nt;
        p->res_tile.tx = tx;
        p->res_tile.ty = ty;
        p->res_tile.ntx = (q.nx + tx - 1) / tx;
        p->res_tile.nty = (q.ny + ty - 1) / ty;
      }
    }
  if (best_cost < 0) return false;
  p->res_grid = (int)best_nt;
  p->res_auto = p->n >= 512L * ncu;
  return true;
}

// The plan's arrays with columns of nz >= prm.nz voxels.
void plan_geometry(fm_plan *p, int32_t nz) {
  const fm_params &q = p->prm;
  p->geo.nx = q.nx;
  p->geo.ny = q.ny;
  p->geo.nz = nz;
  p->geo.uz = q.nz;
  p->geo.sy = nz;
  p->geo.sx = (int64_t)q.ny * nz;
  p->geo.n = p->n = (int64_t)q.nx * q.ny * nz;
  // one x-plane of guard entries on each side (two for the second-order stencil's +-2 neighbours)
  p->pad = (((p->reg2 ? 2 : 1) * p->geo.sx + 63) / 64) * 64;
}

// Small volumes give each voxel a thread of its own: a pass of such a volume lasts as long as
// one thread's chain, and two or four voxels in it lengthen the chain while most of the chip
// idles.  The lines, each with both sides' times (voxels in fours or twos -> a thread each):
// - FP32: half the threads of the largest grid.  115 200 voxels, second order 973 -> 894 us, red-
//   black 639 -> 577; 163 840 voxels, red-black 582 and 583 (149x148x11: 1.80 -> 1.89 ms).
//   Second-order volumes that take the four-voxel passes stay with them (49x52x52: 2.18, 2.28 ms).
// - FP64, IC(0) or more than 4 echoes: three quarters of them.  192 512 voxels, red-black 804 ->
//   793 us, six echoes 1197 -> 1153; 221 184 voxels, 787 -> 851 and 1220 -> 1280.
// - FP64 otherwise (the passes of the diagonal with few echoes are short, those of second order
//   keep their own voxels per thread): a workgroup per compute unit.  62 208 voxels, diagonal 575 ->
//   525 us, second order 648 -> 612; 92 400 voxels, 603 -> 621 and 682 -> 727.
// The voxels counted are those of the plan's arrays.
bool few_voxels(const fm_params &q, int64_t n) {
  const bool order2 = q.reg_order == 2;
  int64_t most = 65536;
  if (q.precision == FM_PREC_MIX)
    most = 131072;
  else if (!order2 && (q.precond == FM_PRECOND_IC0 || q.precond == FM_PRECOND_ICT || q.necho > 4))
    most = 196608;
  return n <= most &&
         !(order2 && q.precision == FM_PREC_MIX && q.necho <= 6 && q.nz % 4 == 0);
}

// Workgroups of the streaming iteration passes.
int stream_grid(const fm_plan *p) {
  const int64_t v = p->few ? 1 : p->mix ? fm::Vpt<float>::v : fm::Vpt<double>::v, chunk = fm::kNT * v;
  return (int)std::max<int64_t>(1, std::min<int64_t>((p->n + chunk - 1) / chunk, kMaxGrid));
}

// Column length of the plan's arrays.  The pair and tile passes of red-black IC(0) need an even
// one, the 16-byte-load passes (FP32, up to 6 echoes, more than a voxel per thread) a multiple of
// 4; a column is lengthened to it with voxels outside the mask where that adds at most an eighth
// (beyond, the added bytes cost more than the per-voxel passes: 10 -> 12 would add a fifth), and
// by at most a fifteenth where the gain is smaller: FP64 volumes with a voxel per thread (above
// 65536 voxels), and the diagonal's passes with few echoes, which are bound by bytes, above 2^20.
// Unpadded -> padded, 40 iterations: 91x109x91 F64 3.84 -> 3.39 ms, 75x60x33 MIX 1.41 -> 1.35,
// 256x250x121 MIX 15.2 -> 10.5, 90x85x18 MIX with six echoes 2.00 -> 1.81; 20 iterations, not
// padded for it: 105x105x9 F64 0.71 -> 0.74, 244x245x25 MIX diagonal 1.51 -> 1.66.
// Plans that qualify for the resident schedule need no more than the even length they have, orders
// with arrays of their own (natural, block red-black, three colours, IC_t) keep the caller's, and
// so do volumes beyond 2^26 voxels, where the memory would be missed.
int32_t padded_columns(const fm_plan *p) {
  const fm_params &q = p->prm;
  const bool rb = q.precond == FM_PRECOND_IC0 && q.ordering == FM_ORDER_REDBLACK;
  const bool none = q.precond == FM_PRECOND_DIAG || q.precond == FM_PRECOND_NONE;
  const int64_t n = (int64_t)q.nx * q.ny * q.nz;
  if (p->reg2 || p->res_ok || !(rb || none) || n > ((int64_t)1 << 26)) return q.nz;
  const int32_t up4 = (q.nz + 3) / 4 * 4, up2 = (q.nz + 1) / 2 * 2;
  const int at_most4 = none && q.necho <= 4 && n > ((int64_t)1 << 20) ? 15 : 8;
  const int at_most2 = !p->mix && p->few && n > 65536 ? 15 : 8;
  if (p->mix && q.necho <= 6 && !p->few && at_most4 * (up4 - q.nz) <= q.nz) return up4;
  if (rb && at_most2 * (up2 - q.nz) <= q.nz) return up2;
  return q.nz;
}

// Columns and threads of a plan whose precision, regulariser and resident schedule are set:
// a volume that its padding takes past the line of a thread per voxel is not one of few voxels.
void plan_columns(fm_plan *p) {
  plan_geometry(p, p->prm.nz);
  p->few = few_voxels(p->prm, p->n);
  plan_geometry(p, padded_columns(p));
  if (p->few && !few_voxels(p->prm, p->n)) {
    p->few = false;
    plan_geometry(p, padded_columns(p));
  }
}

fm_status run_graph(fm_plan *p, int niter, hipStream_t s);

fm_status run_iterations(fm_plan *p, int niter, hipStream_t s) {
  if (niter <= 0) return FM_OK;
  if (use_resident(p)) return run_resident(p, niter, s);
  if (!p->by_levels && (!p->ict || p->ict_tiled)) return run_graph(p, niter, s);
  // a launch per level (thousands per iteration): one graph of one iteration, replayed niter times
  for (int i = 0; i < niter; ++i) {
    fm_status st = run_graph(p, 1, s);
    if (st) return st;
  }
  return FM_OK;
}

fm_status run_graph(fm_plan *p, int niter, hipStream_t s) {
  const std::vector<int64_t> key = {(int64_t)(p->q & 1), niter, p->iter_host & 1, p->last_nparts, p->last_nvals};
  auto it = p->graphs.find(key);
  if (it == p->graphs.end()) {
    const uint64_t q0 = p->q;
    const int64_t it0 = p->iter_host;
    const int np0 = p->last_nparts, nv0 = p->last_nvals;
    FM_HIP(hipStreamBeginCapture(p->cap_stream, hipStreamCaptureModeThreadLocal));
    fm_status st = dispatch<OpLoop>(p, niter, p->cap_stream);
    hipGraph_t g = nullptr;
    hipError_t e = hipStreamEndCapture(p->cap_stream, &g);
    if (st) {
      if (g) (void)hipGraphDestroy(g);
      p->q = q0;
      p->iter_host = it0;
      set_parts(p, np0, nv0);
      return st;
    }
    if (e != hipSuccess) return fail(FM_ERR_HIP, std::string("hipStreamEndCapture: ") + hipGetErrorString(e));
    hipGraphExec_t ge = nullptr;
    hipError_t ei = hipGraphInstantiate(&ge, g, nullptr, nullptr, 0);
    if (ei != hipSuccess) {
      (void)hipGraphDestroy(g);
      return fail(FM_ERR_HIP, std::string("hipGraphInstantiate: ") + hipGetErrorString(ei));
    }
    it = p->graphs.emplace(key, std::make_pair(g, ge)).first;
  } else {
    p->q += launches_per_iteration(p) * (uint64_t)niter;
    p->iter_host += niter;
    set_parts(p, tail_nparts(p), tail_nvals(p));
  }
  FM_HIP(hipGraphLaunch(it->second.second, s));
  return FM_OK;
}

template <typename T>
fm_status enqueue_start(fm_plan *p, const double *f0, hipStream_t s) {
  const int user_f0 = f0 != p->f0buf;
  p->iter_host = 0;
  set_parts(p, 0, 0);
  const uint64_t q = p->q++;
  hipLaunchKernelGGL(fm::k_start<T>, dim3(p->grid), dim3(kBlock), 0, s, p->geo, f0, user_f0, (const uint8_t *)p->code,
                     (T *)p->F[1], (T *)p->Z[1], (T *)p->G[1], p->cm ? p->cm_elems : p->n, p->S + ((q + 1) & 1),
                     p->prm.niter, p->prm.nmls, (const double *)p->nmask);
  FM_LAUNCH_CHECK();
  return FM_OK;
}

fm_status check_plan(fm_plan *p) {
  if (!p) return fail(FM_ERR_ARG, "plan is NULL");
  int cur = 0;
  FM_HIP(hipGetDevice(&cur));
  if (cur != p->device) return fail(FM_ERR_STATE, "plan was created on another device");
  return FM_OK;
}

fm_status read_status(fm_plan *p, hipStream_t s, int32_t *status) {
  FM_HIP(hipMemcpyAsync(status, p->status, sizeof(int32_t), hipMemcpyDeviceToHost, s));
  FM_HIP(hipStreamSynchronize(s));
  return FM_OK;
}

// ---------------------------------------------------------------------------
// Implicit adjoint: CG on the exact Hessian at fhat, preconditioned like the
// iteration.  The chain has its own state/partial ping-pong (position aq).  The
// workspace is cleared on the call's stream s, which a memset on the default stream
// need not precede.
fm_status adj_alloc(fm_plan *p, hipStream_t s) {
  if (p->adj_ready) return FM_OK;
  const size_t n = (size_t)p->n, ts = p->tsize;
  auto take = [&]() {
    const size_t mark = p->bases.size();
    const bool ok = plan_alloc_padded(p, &p->aR, n, ts) && plan_alloc_padded(p, &p->aZ, n, ts) &&
                    plan_alloc_padded(p, &p->aX, n, ts) && plan_alloc_padded(p, &p->aDc, n, ts) &&
                    plan_alloc_padded(p, &p->aH, n, ts) && plan_alloc_padded(p, &p->aV, n, ts) &&
                    plan_alloc_padded(p, &p->aDd[0], n, ts) && plan_alloc_padded(p, &p->aDd[1], n, ts) &&
                    plan_alloc_padded(p, (void **)&p->a_hinv, n, sizeof(double)) &&
                    plan_alloc_padded(p, (void **)&p->a_ipiv, n, sizeof(double)) &&
                    plan_alloc(p, (void **)&p->a_part, sizeof(double) * 2 * p->part_rows * kMaxK) &&
                    plan_alloc(p, (void **)&p->aS, sizeof(fm::State) * 2) &&
                    plan_alloc(p, (void **)&p->a_status, sizeof(int32_t));
    if (!ok) plan_free_from(p, mark);
    return ok;
  };
  if (!take() && !(give_back_rows(p) && take())) return fail(FM_ERR_ALLOC, "hipMalloc of the adjoint workspace failed");
  if (hipMemsetAsync(p->a_part, 0, sizeof(double) * 2 * p->part_rows * kMaxK, s) != hipSuccess ||
      hipMemsetAsync(p->aS, 0, sizeof(fm::State) * 2, s) != hipSuccess)
    return fail(FM_ERR_HIP, "hipMemset of the adjoint state failed");
  if (sweeps_in_tiles(p) && !p->by_levels && !p->wf.ff) {
    // a block red-black plan's CG is preconditioned in natural order, where the face buffers fit
    const size_t mark = p->bases.size();
    p->adj_levels = !packed_rows_fit((sizeof(fm::Rec) + ts) * face_values(p->wf), n, 64) || alloc_faces(p, s) != FM_OK;
    if (p->adj_levels) {
      plan_free_from(p, mark);
      drop_faces(p);
    }
  }
  if (!p->a_host && hipHostMalloc((void **)&p->a_host, sizeof(fm::State) * 2, hipHostMallocDefault) != hipSuccess)
    return fail(FM_ERR_ALLOC, "pinned memory for the adjoint state failed");
  for (hipEvent_t &e : p->a_copied)
    if (!e) FM_HIP(hipEventCreateWithFlags(&e, hipEventDisableTiming));
  p->adj_ready = true;
  return FM_OK;
}

template <typename T>
fm::AdjArgs<T> adj_args(fm_plan *p, uint64_t q, int par, int nparts_in, int nvals_in) {
  fm::AdjArgs<T> a{};
  a.geo = p->geo;
  a.L = p->prm.necho;
  a.beta = p->prm.beta;
  a.dat = (const fm::T2<T> *)p->dat;
  a.code = p->code;
  a.pairs = (const fm::PairC<T> *)p->pairs;
  a.F = (const T *)p->F[p->iter_host & 1];  // the final pass wrote fhat there
  a.R = (T *)p->aR;
  a.Zp = (const T *)p->aZ;
  a.Dd[0] = (T *)p->aDd[0];
  a.Dd[1] = (T *)p->aDd[1];
  a.V = (T *)p->aV;
  a.H = (T *)p->aH;
  a.Dc = (T *)p->aDc;
  a.hinv = p->a_hinv;
  a.P = (T *)p->aZ;
  a.par = par;
  a.nparts_in = nparts_in;
  a.nvals_in = nvals_in;
  a.sin = p->aS + (q & 1);
  a.sout = p->aS + ((q + 1) & 1);
  a.pin = p->a_part + (size_t)(q & 1) * p->part_rows * kMaxK;
  a.pout = p->a_part + (size_t)((q + 1) & 1) * p->part_rows * kMaxK;
  a.status = p->a_status;
  return a;
}

// Arguments of the iteration's preconditioner passes pointed at the adjoint
// buffers: right-hand side r, output z, curvature D of the Huber model.
template <typename T>
fm::IterArgs<T> adj_precond_args(fm_plan *p, uint64_t q, int nparts_in, int nvals_in) {
  fm::IterArgs<T> a{};
  a.geo = p->geo;
  a.L = p->prm.necho;
  a.beta = p->prm.beta;
  a.dat = (const fm::T2<T> *)p->dat;
  a.code = p->code;
  a.pairs = (const fm::PairC<T> *)p->pairs;
  for (int i = 0; i < 2; ++i) {
    a.F[i] = (T *)p->aV;
    a.Z[i] = (T *)p->aV;
    a.G[i] = (T *)p->aR;
  }
  a.D = (T *)p->aDc;
  a.X = (T *)p->aX;
  a.P = (T *)p->aZ;
  a.ipiv = p->a_ipiv;
  a.hinv = p->a_hinv;
  a.write_hinv = 0;
  a.store_piv = 0;
  a.par = 0;
  a.nparts_in = nparts_in;
  a.nvals_in = nvals_in;
  a.sin = p->aS + (q & 1);
  a.sout = p->aS + ((q + 1) & 1);
  a.pin = p->a_part + (size_t)(q & 1) * p->part_rows * kMaxK;
  a.pout = p->a_part + (size_t)((q + 1) & 1) * p->part_rows * kMaxK;
  a.status = p->a_status;
  a.trace = nullptr;
  return a;
}

// The adjoint's CG iteration in three passes (red-black IC(0), even columns).
bool adj_pairs(const fm_plan *p) {
  return !p->reg2 && p->prm.precond == FM_PRECOND_IC0 && p->prm.ordering == FM_ORDER_REDBLACK && p->geo.nz % 2 == 0;
}

template <typename T>
fm_status adj_enqueue_iteration(fm_plan *p, uint64_t &q, int &np, int &nv, int k, hipStream_t s) {
  const T *r = (const T *)p->aR;
  Recorder *rec = nullptr;
  if (adj_pairs(p)) {
    auto launch = [&](void (*kern)(fm::AdjArgs<T>)) -> fm_status {
      hipLaunchKernelGGL(kern, dim3(p->sgrid), dim3(fm::kNT), 0, s, adj_args<T>(p, q++, k & 1, np, nv));
      FM_LAUNCH_CHECK();
      np = p->sgrid;
      nv = 1;
      return FM_OK;
    };
    fm_status e = launch(fm::k_adj_black_pair<T>);
    if (!e) e = launch(fm::k_adj_red_dir_pair<T>);
    if (e) return e;
    if constexpr (std::is_same<T, float>::value)
      return launch(p->geo.nz % 4 == 0 ? fm::k_adj_update_q : fm::k_adj_update<T, false>);
    else
      return launch(fm::k_adj_update<T, false>);
  }
  if (p->reg2) {
    // second-order C: diag(H) with diag(C^T C) of the 13-point operator (also for IC(0) plans), or none
    FM_LAUNCH(0, fm::k_diag2<T>, dim3(p->sgrid), dim3(fm::kNT), s, adj_precond_args<T>(p, q++, np, nv), r,
              p->prm.precond == FM_PRECOND_NONE ? 1 : 0);
    FM_LAUNCH_CHECK();
    np = p->sgrid;
    nv = 2;
  } else if (p->prm.precond == FM_PRECOND_IC0) {
    // natural-order IC(0) also for block red-black plans (v does not depend on the preconditioner)
    if (p->by_levels || p->adj_levels) {
      fm_status e = enqueue_ic_levels<T, false>(p, adj_precond_args<T>(p, q++, np, nv), r, s, rec);
      if (e) return e;
      np = p->sgrid;
      nv = 2;
    } else if (p->prm.ordering == FM_ORDER_NATURAL || p->prm.ordering == FM_ORDER_BLOCKRB) {
      const fm::IterArgs<T> ain = adj_precond_args<T>(p, q++, np, nv);
      fm_status e = enqueue_natural<T>(p, ain, adj_precond_args<T>(p, q++, 0, 0), r, p->a_status, s, rec);
      if (e) return e;
      np = p->wf_unpack_grid;
      nv = 2;
    } else {
      FM_LAUNCH(0, (fm::k_rb_black<T, false>), dim3(p->sgrid), dim3(fm::kNT), s, adj_precond_args<T>(p, q++, np, nv), r);
      FM_LAUNCH_CHECK();
      np = p->sgrid;
      nv = 2;
      FM_LAUNCH(0, (fm::k_rb_red<T, false>), dim3(p->sgrid), dim3(fm::kNT), s, adj_precond_args<T>(p, q++, np, nv), r);
      FM_LAUNCH_CHECK();
      np = p->sgrid;
      nv = 2;
    }
  } else {
    FM_LAUNCH(0, (fm::k_diag<T, false>), dim3(p->sgrid), dim3(fm::kNT), s, adj_precond_args<T>(p, q++, np, nv), r,
              p->prm.precond == FM_PRECOND_NONE ? 1 : 0);
    FM_LAUNCH_CHECK();
    np = p->sgrid;
    nv = 2;
  }
  if (p->reg2)
    FM_LAUNCH(0, (fm::k_adj_dir<T, true>), dim3(p->sgrid), dim3(fm::kNT), s, adj_args<T>(p, q++, k & 1, np, nv));
  else
    FM_LAUNCH(0, (fm::k_adj_dir<T, false>), dim3(p->sgrid), dim3(fm::kNT), s, adj_args<T>(p, q++, k & 1, np, nv));
  FM_LAUNCH_CHECK();
  np = p->sgrid;
  nv = 1;
  if (p->reg2)
    FM_LAUNCH(0, (fm::k_adj_update<T, true>), dim3(p->sgrid), dim3(fm::kNT), s, adj_args<T>(p, q++, k & 1, np, nv));
  else
    FM_LAUNCH(0, (fm::k_adj_update<T, false>), dim3(p->sgrid), dim3(fm::kNT), s, adj_args<T>(p, q++, k & 1, np, nv));
  FM_LAUNCH_CHECK();
  np = p->sgrid;
  nv = 1;
  return FM_OK;
}

// Consume the last pass's sums and copy the CG state to host slot `slot`.
fm_status adj_finish(fm_plan *p, uint64_t &q, int &np, int &nv, int slot, hipStream_t s) {
  hipLaunchKernelGGL(fm::k_finish, dim3(1), dim3(kBlock), 0, s, (const fm::State *)(p->aS + (q & 1)),
                     p->aS + ((q + 1) & 1), (const double *)(p->a_part + (size_t)(q & 1) * p->part_rows * kMaxK),
                     np, nv, p->prm.beta, (double *)nullptr, p->a_status);
  FM_LAUNCH_CHECK();
  ++q;
  np = 0;
  nv = 0;
  FM_HIP(hipMemcpyAsync(p->a_host + slot, p->aS + (q & 1), sizeof(fm::State), hipMemcpyDeviceToHost, s));
  FM_HIP(hipEventRecord(p->a_copied[slot], s));
  return FM_OK;
}

constexpr int kAdjCheck = 8;  // CG iterations between convergence checks on the host

template <typename T, int LMAX>
struct OpAdjoint {
  static fm_status run(fm_plan *p, const double *dldf, const void *sens, void *dldy, double *vout, int maxit,
                       double rtol, fm::State *out, hipStream_t s) {
    uint64_t q = 0;
    int np = 0, nv = 0;
    const int write_hinv = adj_pairs(p) ? 2 : (p->prm.precond == FM_PRECOND_IC0 && p->prm.ordering == FM_ORDER_REDBLACK) ? 1 : 0;
    hipLaunchKernelGGL((fm::k_adj_setup<T, LMAX>), dim3(p->sgrid), dim3(fm::kNT), 0, s, adj_args<T>(p, q++, 0, 0, 0),
                       dldf, rtol * rtol, write_hinv);
    FM_LAUNCH_CHECK();
    np = p->sgrid;
    nv = 1;
    // The state after a chunk is looked at once the next chunk is in the stream, so the GPU
    // does not wait for the host: the passes find the state converged and do nothing.  Not so
    // after the first chunk, after which many small volumes have converged (3x3x3: 233 us, 326
    // with a second chunk that does nothing), nor for the natural-order sweeps, which do not look
    // at the state (128x128x64 MIX: 0.2 ms an iteration, 7 us a wait; 158 iterations 39.4 -> 38.5 ms).
    const bool ahead = !sweeps_in_tiles(p);
    int k = 0, slot = 0;
    bool seen = true;  // the state after the chunk before
    while (k < maxit) {
      const bool wait = !ahead || k == 0;
      const int chunk = (maxit - k) < kAdjCheck ? (maxit - k) : kAdjCheck;
      for (int i = 0; i < chunk; ++i, ++k) {
        fm_status e = adj_enqueue_iteration<T>(p, q, np, nv, k, s);
        if (e) return e;
      }
      fm_status e = adj_finish(p, q, np, nv, slot, s);
      if (e) return e;
      if (wait || !seen) {
        const int look = wait ? slot : slot ^ 1;
        FM_HIP(hipEventSynchronize(p->a_copied[look]));
        if (p->a_host[look].cg_done) break;
      }
      seen = wait;
      slot ^= 1;
    }
    if (maxit == 0) {
      fm_status e = adj_finish(p, q, np, nv, 0, s);
      if (e) return e;
    }
    if (p->reg2)
      hipLaunchKernelGGL((fm::k_adj_out<T, LMAX, true>), dim3(p->sgrid), dim3(fm::kNT), 0, s,
                         adj_args<T>(p, q++, 0, np, nv), (const float2 *)sens, p->prm.ncoil, (float2 *)dldy, vout);
    else
      hipLaunchKernelGGL((fm::k_adj_out<T, LMAX, false>), dim3(p->sgrid), dim3(fm::kNT), 0, s,
                         adj_args<T>(p, q++, 0, np, nv), (const float2 *)sens, p->prm.ncoil, (float2 *)dldy, vout);
    FM_LAUNCH_CHECK();
    np = p->sgrid;
    nv = 1;
    fm_status e = adj_finish(p, q, np, nv, 0, s);
    if (e) return e;
    FM_HIP(hipStreamSynchronize(s));
    *out = p->a_host[0];
    return FM_OK;
  }
};

}  // namespace

namespace {
fm_status setup_launch(fm_plan *p, const void *y, const void *sens, const uint8_t *mask, hipStream_t s);
}

// ---------------------------------------------------------------------------
extern "C" {

const char *fm_status_string(fm_status st) {
  switch (st) {
    case FM_OK: return "ok";
    case FM_ERR_ARG: return "invalid argument";
    case FM_ERR_SHAPE: return "invalid shape";
    case FM_ERR_ALLOC: return "device allocation failed";
    case FM_ERR_HIP: return "HIP runtime error";
    case FM_ERR_NOT_PD: return "IC(0) pivot not positive";
    case FM_ERR_NONFINITE: return "non-finite value in the iteration";
    case FM_ERR_STATE: return "call out of order";
    case FM_ERR_TIMEOUT: return "device-side wait exceeded its bound";
  }
  return "unknown status";
}

const char *fm_last_error(void) { return g_last_error.c_str(); }

fm_status fm_plan_create(const fm_params *prm, fm_plan **out) {
  if (!out) return fail(FM_ERR_ARG, "plan output pointer is NULL");
  *out = nullptr;
  fm_status vs = validate(prm);
  if (vs) return vs;
  fm_plan *p = new fm_plan();
  p->prm = *prm;
  p->mix = prm->precision == FM_PREC_MIX;
  p->tsize = p->mix ? sizeof(float) : sizeof(double);
  p->reg2 = prm->reg_order == 2;
  plan_geometry(p, prm->nz);
  p->cm = p->reg2 && prm->precond == FM_PRECOND_IC0;
  if (p->cm) {
    const int64_t m = ((int64_t)prm->nz + 2) / 3;
    p->cm_elems = 3 * ((int64_t)prm->nx + 4) * prm->ny * m;
  }
  if (p->n + 2 * p->pad >= ((int64_t)1 << 31) || p->cm_elems >= ((int64_t)1 << 31)) {
    delete p;
    return fail(FM_ERR_SHAPE, "volume too large for 32-bit voxel indices");
  }
  if (hipGetDevice(&p->device) != hipSuccess) {
    delete p;
    return fail(FM_ERR_HIP, "hipGetDevice failed");
  }
  p->res_ok = plan_resident(p);
  plan_columns(p);  // (at most 9/8 of 2^26 voxels: no index bound to check again)
  p->lmax = prm->necho <= 4 ? 4 : (prm->necho <= 8 ? 8 : 16);
  const int64_t blocks = (p->n + kBlock - 1) / kBlock;
  p->grid = (int)(blocks < kMaxGrid ? blocks : kMaxGrid);
  if (p->grid < 1) p->grid = 1;
  p->sgrid = stream_grid(p);
  auto cleanup = [&](fm_status st) {
    free_plan(p);
    return st;
  };
  const size_t n = (size_t)p->n, ts = p->tsize, L = (size_t)prm->necho;
  const size_t trace_bytes = sizeof(double) * FM_TR_W * ((size_t)prm->niter + 1);
#define FM_ALLOC(ptr, bytes)                                                          \
  if (!plan_alloc(p, (void **)&(ptr), (bytes)))                                       \
    return cleanup(fail(FM_ERR_ALLOC, "hipMalloc of " #ptr " failed"));
#define FM_ALLOC_PAD(ptr, esize)                                                      \
  if (!plan_alloc_padded(p, (void **)&(ptr), n, (esize)))                             \
    return cleanup(fail(FM_ERR_ALLOC, "hipMalloc of " #ptr " failed"));
  FM_ALLOC(p->dat, 2 * ts * L * n);
  FM_ALLOC_PAD(p->code, 1);  // padded like every array a kernel may address at neighbour offsets
  for (int i = 0; i < 2; ++i) {
    FM_ALLOC_PAD(p->F[i], ts);
    FM_ALLOC_PAD(p->Z[i], ts);
  }
  if (p->cm) {
    const size_t e = (size_t)p->cm_elems;
    for (int i = 0; i < 2; ++i) FM_ALLOC(p->G[i], ts * e);
    FM_ALLOC(p->D, ts * e);
    FM_ALLOC(p->X, ts * e);
    FM_ALLOC(p->X2, ts * e);
    FM_ALLOC(p->P, ts * e);
    FM_ALLOC(p->ipiv, sizeof(double) * e);
    FM_ALLOC(p->rdiag, e);
    FM_ALLOC(p->ccode, e);
    FM_ALLOC_PAD(p->Pv, ts);
    FM_ALLOC_PAD(p->Dv, ts);
  } else {
    for (int i = 0; i < 2; ++i) FM_ALLOC_PAD(p->G[i], ts);
    FM_ALLOC_PAD(p->D, ts);
    if (!sweeps_in_tiles(p) && prm->precond != FM_PRECOND_ICT) FM_ALLOC_PAD(p->X, ts);
    FM_ALLOC_PAD(p->P, ts);
    if (prm->precond != FM_PRECOND_ICT) FM_ALLOC_PAD(p->ipiv, sizeof(double));  // (IC_t's pivots are L_jj^2)
  }
  FM_ALLOC_PAD(p->hinv, sizeof(double));
  FM_ALLOC(p->S, sizeof(fm::State) * 2);
  {
    // natural-order wavefront: 8x8 column tiles in anti-diagonal order
    fm::Wavefront &w = p->wf;
    w.ntx = (prm->nx + fm::kTile - 1) / fm::kTile;
    w.nty = (prm->ny + fm::kTile - 1) / fm::kTile;
    w.ntiles = w.ntx * w.nty;
    std::vector<int2> order;
    order.reserve((size_t)w.ntiles);
    for (int d = 0; d <= w.ntx + w.nty - 2; ++d)
      for (int ti = 0; ti < w.ntx; ++ti) {
        const int tj = d - ti;
        if (tj >= 0 && tj < w.nty) order.push_back(make_int2(ti, tj));
      }
    void *ord = nullptr;
    FM_ALLOC(ord, sizeof(int2) * order.size());
    if (hipMemcpy(ord, order.data(), sizeof(int2) * order.size(), hipMemcpyHostToDevice) != hipSuccess)
      return cleanup(fail(FM_ERR_HIP, "wavefront tables upload failed"));
    w.order = (const int2 *)ord;
    // block red-black: the tiles of each colour (ti + tj) mod 2
    std::vector<int2> blk[2];
    for (int ti = 0; ti < w.ntx; ++ti)
      for (int tj = 0; tj < w.nty; ++tj) blk[(ti + tj) & 1].push_back(make_int2(ti, tj));
    for (int c = 0; c < 2; ++c) {
      w.nblk[c] = (int32_t)blk[c].size();
      w.blk[c] = nullptr;
      if (blk[c].empty()) continue;
      void *bp = nullptr;
      FM_ALLOC(bp, sizeof(int2) * blk[c].size());
      if (hipMemcpy(bp, blk[c].data(), sizeof(int2) * blk[c].size(), hipMemcpyHostToDevice) != hipSuccess)
        return cleanup(fail(FM_ERR_HIP, "block tables upload failed"));
      w.blk[c] = (const int2 *)bp;
    }
    p->part_rows = (size_t)(w.ntiles > kMaxGrid ? w.ntiles : kMaxGrid);
  }
  FM_ALLOC(p->part, sizeof(double) * 2 * p->part_rows * kMaxK);
  FM_ALLOC(p->setup_part, sizeof(double) * kMaxGrid * kMaxK);
  FM_ALLOC(p->nmask, sizeof(double));
  FM_ALLOC(p->status, sizeof(int32_t));
  FM_ALLOC(p->trace, trace_bytes);
  FM_ALLOC(p->f0buf, sizeof(double) * n);
  if (p->res_ok) {
    FM_ALLOC(p->res_part, sizeof(double) * fm::kResSlots * kMaxK * (size_t)p->res_grid);
    FM_ALLOC(p->res_bar, res_bar_bytes(p));
  }
  if (prm->model == FM_WATERFAT) {
    FM_ALLOC(p->rho, sizeof(double) * n);
    FM_ALLOC(p->gabs, sizeof(double) * L * L);
    FM_ALLOC(p->wf_tmp, sizeof(double) * n * 4);
    FM_ALLOC(p->sweep_rot, sizeof(double2) * L * L);
  }
  // the packed rows last, so that they take no memory that something else needs
  if (sweeps_in_tiles(p)) {
    fm_status rs = alloc_sweep_rows(p);
    if (rs) return cleanup(rs);
  }
  if (prm->precond == FM_PRECOND_ICT) {
    int noff = 0, wa = 1, wb = 1;
    if (prm->ict_level == 0) {
      noff = fm::IctPattern<0>::n, wa = fm::IctPattern<0>::a, wb = fm::IctPattern<0>::b;
    } else if (prm->ict_level == 1) {
      noff = fm::IctPattern<1>::n, wa = fm::IctPattern<1>::a, wb = fm::IctPattern<1>::b;
    } else {
      noff = fm::IctPattern<2>::n, wa = fm::IctPattern<2>::a, wb = fm::IctPattern<2>::b;
    }
    p->ict = true;
    p->ict_noff = noff;
    FM_ALLOC(p->ict_hmax, sizeof(double));
    FM_ALLOC(p->ict_hpart, sizeof(double) * kMaxGrid);
    if (prm->ict_level < 2) {
      fm_status is = prm->ict_level == 0 ? alloc_ict_sweep<0>(p) : alloc_ict_sweep<1>(p);
      if (is) return cleanup(is);
    }
    if (!p->ict_tiled) {
      p->ict_nlev = wa * (prm->nx - 1) + wb * (prm->ny - 1) + (prm->nz - 1) + 1;
      p->ict_kcol = (prm->nz - 1) / wb + 1;
      p->ict_blocks = (int)(((int64_t)prm->nx * p->ict_kcol + fm::kIctNT - 1) / fm::kIctNT);
      FM_ALLOC(p->ict_lo, sizeof(double) * n * (size_t)noff);
      FM_ALLOC(p->ict_ld, sizeof(double) * n);
      FM_ALLOC(p->ict_y, sizeof(double) * n);
      FM_ALLOC(p->ict_pd, sizeof(double) * n);
      if (hipMemset(p->ict_lo, 0, sizeof(double) * n * (size_t)noff) != hipSuccess ||
          hipMemset(p->ict_ld, 0, sizeof(double) * n) != hipSuccess)
        return cleanup(fail(FM_ERR_HIP, "hipMemset of the IC_t factor failed"));
    }
  }
#undef FM_ALLOC
#undef FM_ALLOC_PAD
  if (hipMemset(p->code - p->pad, 0, (size_t)n + 2 * (size_t)p->pad) != hipSuccess ||
      hipMemset(p->S, 0, sizeof(fm::State) * 2) != hipSuccess || hipMemset(p->status, 0, sizeof(int32_t)) != hipSuccess ||
      hipMemset(p->nmask, 0, sizeof(double)) != hipSuccess || hipMemset(p->trace, 0, trace_bytes) != hipSuccess ||
      hipMemset(p->part, 0, sizeof(double) * 2 * p->part_rows * kMaxK) != hipSuccess)
    return cleanup(fail(FM_ERR_HIP, "hipMemset of the plan state failed"));
  const auto G = make_gamma(*prm);
  fm_status st = p->mix ? upload_pairs<float>(p, G, &p->pairs) : upload_pairs<double>(p, G, &p->pairs);
  if (st) return cleanup(st);
  st = upload_pairs<double>(p, G, &p->pairs_d);
  if (st) return cleanup(st);
  {
    int K = 1;
    std::vector<double> tab(prm->te, prm->te + prm->necho);
    const auto Bm = make_component_matrix(*prm, &K);
    tab.insert(tab.end(), Bm.begin(), Bm.end());
    p->ncomp = K;
    if (!plan_alloc(p, (void **)&p->comp_tab, sizeof(double) * tab.size()) ||
        hipMemcpy(p->comp_tab, tab.data(), sizeof(double) * tab.size(), hipMemcpyHostToDevice) != hipSuccess)
      return cleanup(fail(FM_ERR_ALLOC, "upload of the component matrix failed"));
  }
  if (p->gabs) {
    std::vector<double> ga((size_t)L * L);
    for (size_t i = 0; i < ga.size(); ++i) ga[i] = std::abs(G[i]);
    if (hipMemcpy(p->gabs, ga.data(), sizeof(double) * ga.size(), hipMemcpyHostToDevice) != hipSuccess)
      return cleanup(fail(FM_ERR_HIP, "upload of |Gamma| failed"));
    std::vector<double2> rot;
    const double step = 2.0 * sweep_half(*prm) / (prm->nsweep - 1);
    for (int m = 0; m < prm->necho; ++m)
      for (int q = m + 1; q < prm->necho; ++q) {
        const double d = 6.283185307179586476925286766559 * (prm->te[m] - prm->te[q]) * step;
        rot.push_back(make_double2(std::cos(d), std::sin(d)));
      }
    if (hipMemcpy(p->sweep_rot, rot.data(), sizeof(double2) * rot.size(), hipMemcpyHostToDevice) != hipSuccess)
      return cleanup(fail(FM_ERR_HIP, "upload of the sweep rotations failed"));
  }
  if (hipStreamCreateWithFlags(&p->cap_stream, hipStreamNonBlocking) != hipSuccess)
    return cleanup(fail(FM_ERR_HIP, "hipStreamCreate failed"));
  // the plan's arrays are cleared on the default stream, which other streams need not wait for
  if (hipStreamSynchronize(nullptr) != hipSuccess)
    return cleanup(fail(FM_ERR_HIP, "clearing the plan's arrays failed"));
  *out = p;
  return FM_OK;
}

fm_status fm_plan_destroy(fm_plan *p) {
  if (!p) return FM_OK;
  free_plan(p);
  return FM_OK;
}

fm_status fm_ict_offsets(int32_t level, int32_t *offsets, int32_t *count) {
  if (!offsets || !count) return fail(FM_ERR_ARG, "offsets and count must not be NULL");
  auto put = [&](auto pat) {
    using P = decltype(pat);
    for (int u = 0; u < P::n; ++u)
      for (int d = 0; d < 3; ++d) offsets[3 * u + d] = P::off[u][d];
    *count = P::n;
  };
  if (level == 0)
    put(fm::IctPattern<0>{});
  else if (level == 1)
    put(fm::IctPattern<1>{});
  else if (level == 2)
    put(fm::IctPattern<2>{});
  else
    return fail(FM_ERR_ARG, "IC_t level must be 0, 1 or 2");
  return FM_OK;
}

fm_status fm_get_factor(fm_plan *p, double *L, hipStream_t s) {
  fm_status cs = check_plan(p);
  if (cs) return cs;
  if (!L) return fail(FM_ERR_ARG, "L must not be NULL");
  if (!p->ict) return fail(FM_ERR_ARG, "the plan's preconditioner is not IC_t");
  const size_t n = (size_t)p->n;
  if (p->ict_tiled) {
    if (p->prm.ict_level == 0)
      hipLaunchKernelGGL(fm::k_ict_factor<0>, dim3(p->grid), dim3(kBlock), 0, s, p->geo, (const uint8_t *)p->code,
                         p->ict_sweep, L, (double *)nullptr);
    else
      hipLaunchKernelGGL(fm::k_ict_factor<1>, dim3(p->grid), dim3(kBlock), 0, s, p->geo, (const uint8_t *)p->code,
                         p->ict_sweep, L, (double *)nullptr);
    FM_LAUNCH_CHECK();
    return FM_OK;
  }
  FM_HIP(hipMemcpyAsync(L, p->ict_ld, sizeof(double) * n, hipMemcpyDeviceToDevice, s));
  FM_HIP(hipMemcpyAsync(L + n, p->ict_lo, sizeof(double) * n * (size_t)p->ict_noff, hipMemcpyDeviceToDevice, s));
  return FM_OK;
}

fm_status fm_setup(fm_plan *p, const void *y, const void *sens, const uint8_t *mask, hipStream_t s) {
  fm_status cs = check_plan(p);
  if (cs) return cs;
  if (!y || !mask) return fail(FM_ERR_ARG, "y and mask must not be NULL");
  if (!sens && p->prm.ncoil != 1) return fail(FM_ERR_ARG, "sens may be NULL only when ncoil == 1");
  fm_status st = setup_launch(p, y, sens, mask, s);
  if (st) return st;
  p->setup_done = true;
  return FM_OK;
}

}  // extern "C"

namespace {
// The setup kernels of fm_setup (coil combination, codes, initial map, in-mask
// count), on the plan's arrays.
fm_status setup_launch(fm_plan *p, const void *y, const void *sens, const uint8_t *mask, hipStream_t s) {
  const double two_pi = 6.283185307179586476925286766559;
  auto launch = [&](auto tag) -> fm_status {
    using T = decltype(tag);
    fm::SetupArgs<T> a{};
    a.geo = p->geo;
    a.ncoil = p->prm.ncoil;
    a.L = p->prm.necho;
    a.y = (const float2 *)y;
    a.sens = (const float2 *)sens;
    a.mask = mask;
    a.dat = (fm::T2<T> *)p->dat;
    a.estride = p->n;
    a.code = p->code;
    a.f0 = p->f0buf;
    a.inv_2pi_dt = 1.0 / (two_pi * (p->prm.te[1] - p->prm.te[0]));
    a.rho = p->rho;
    a.gabs = p->gabs;
    a.pairs_d = (const fm::PairC<double> *)p->pairs_d;
    a.npairs = p->npairs;
    if (p->prm.model == FM_WATERFAT) {
      a.nsweep = p->prm.nsweep;
      a.sweep_half = sweep_half(p->prm);
      a.sweep_rot = p->sweep_rot;
      a.ftilde = p->wf_tmp;
    }
    a.partials = p->setup_part;
    hipLaunchKernelGGL(setup_kernel<T>(p->lmax, p->prm.model == FM_WATERFAT, p->prm.necho), dim3(p->grid),
                       dim3(kBlock), 0, s, a);
    FM_LAUNCH_CHECK();
    hipLaunchKernelGGL(fm::k_count, dim3(1), dim3(kBlock), 0, s, (const double *)p->setup_part, p->grid, p->nmask);
    FM_LAUNCH_CHECK();
    if (p->cm) {
      const int64_t blocks = (p->cm_elems + kBlock - 1) / kBlock;
      const dim3 grid((unsigned)(blocks < kMaxGrid ? blocks : kMaxGrid));
      hipLaunchKernelGGL(fm::k_colour_major2, grid, dim3(kBlock), 0, s, p->geo, (const uint8_t *)p->code, p->ccode,
                         p->rdiag);
      FM_LAUNCH_CHECK();
    }
    return FM_OK;
  };
  return p->mix ? launch(float{}) : launch(double{});
}
}  // namespace

extern "C" {

fm_status fm_init(fm_plan *p, double *f0, hipStream_t s) {
  fm_status cs = check_plan(p);
  if (cs) return cs;
  if (!f0) return fail(FM_ERR_ARG, "f0 must not be NULL");
  if (!p->setup_done) return fail(FM_ERR_STATE, "fm_init needs fm_setup first");
  const bool padded = p->geo.uz != p->geo.nz;
  if (p->prm.model == FM_WATERFAT) {
    fm_status st = wf_init(p, padded ? p->f0buf : f0, s);
    if (st || !padded) return st;
  }
  if (padded) {
    hipLaunchKernelGGL(fm::k_from_work<double>, dim3(p->grid), dim3(kBlock), 0, s, p->geo, (const double *)p->f0buf, f0);
    FM_LAUNCH_CHECK();
    return FM_OK;
  }
  FM_HIP(hipMemcpyAsync(f0, p->f0buf, sizeof(double) * p->n, hipMemcpyDeviceToDevice, s));
  return FM_OK;
}

fm_status fm_eval(fm_plan *p, const double *f, double *phi, double *dphi, double *curv, double *lap,
                  hipStream_t s) {
  fm_status cs = check_plan(p);
  if (cs) return cs;
  if (!f) return fail(FM_ERR_ARG, "f must not be NULL");
  if (!p->setup_done) return fail(FM_ERR_STATE, "fm_eval needs fm_setup first");
  return dispatch<OpEval>(p, f, phi, dphi, curv, lap, s);
}

fm_status fm_precondition(fm_plan *p, const double *curv, const double *g, double *piv, double *pout,
                          hipStream_t s) {
  fm_status cs = check_plan(p);
  if (cs) return cs;
  if (!curv || !g || !pout) return fail(FM_ERR_ARG, "curv, g and p must not be NULL");
  if (!p->setup_done) return fail(FM_ERR_STATE, "fm_precondition needs fm_setup first");
  auto run = [&](auto tag) -> fm_status {
    using T = decltype(tag);
    if (p->cm) {
      hipLaunchKernelGGL(fm::k_to_cm<T>, dim3(p->grid), dim3(kBlock), 0, s, p->geo, curv, (T *)p->D);
      FM_LAUNCH_CHECK();
      hipLaunchKernelGGL(fm::k_to_cm<T>, dim3(p->grid), dim3(kBlock), 0, s, p->geo, g, (T *)p->G[0]);
      FM_LAUNCH_CHECK();
    } else {
      hipLaunchKernelGGL(fm::k_to_work<T>, dim3(p->grid), dim3(kBlock), 0, s, p->geo, curv, (T *)p->D);
      FM_LAUNCH_CHECK();
      hipLaunchKernelGGL(fm::k_to_work<T>, dim3(p->grid), dim3(kBlock), 0, s, p->geo, g, (T *)p->G[0]);
      FM_LAUNCH_CHECK();
    }
    FM_HIP(hipMemsetAsync(p->status, 0, sizeof(int32_t), s));
    const uint64_t q = p->q++;
    hipLaunchKernelGGL(fm::k_state_init, dim3(1), dim3(1), 0, s, p->S + ((q + 1) & 1), p->prm.niter, p->prm.nmls);
    FM_LAUNCH_CHECK();
    p->iter_host = 0;
    set_parts(p, 0, 0);
    if (p->prm.precond == FM_PRECOND_IC0 && p->prm.ordering == FM_ORDER_REDBLACK) {
      hipLaunchKernelGGL(fm::k_hinv<T>, dim3(p->grid), dim3(kBlock), 0, s, p->geo, p->prm.beta,
                         (const uint8_t *)p->code, (const T *)p->D, p->hinv, p->status);
      FM_LAUNCH_CHECK();
    }
    fm_status st = enqueue_precond<T>(p, (const T *)p->G[0], s);
    if (st) return st;
    if (p->cm) {
      hipLaunchKernelGGL(fm::k_from_cm<T>, dim3(p->grid), dim3(kBlock), 0, s, p->geo, (const T *)p->P, pout);
      FM_LAUNCH_CHECK();
      if (piv) {
        hipLaunchKernelGGL(fm::k_pivots_cm, dim3(p->grid), dim3(kBlock), 0, s, p->geo, (const double *)p->ipiv, piv);
        FM_LAUNCH_CHECK();
      }
    } else {
      hipLaunchKernelGGL(fm::k_from_work<T>, dim3(p->grid), dim3(kBlock), 0, s, p->geo, (const T *)p->P, pout);
      FM_LAUNCH_CHECK();
      if (piv && p->ict_tiled) {
        if (p->prm.ict_level == 0)
          hipLaunchKernelGGL(fm::k_ict_factor<0>, dim3(p->grid), dim3(kBlock), 0, s, p->geo, (const uint8_t *)p->code,
                             p->ict_sweep, (double *)nullptr, piv);
        else
          hipLaunchKernelGGL(fm::k_ict_factor<1>, dim3(p->grid), dim3(kBlock), 0, s, p->geo, (const uint8_t *)p->code,
                             p->ict_sweep, (double *)nullptr, piv);
        FM_LAUNCH_CHECK();
      } else if (piv && p->ict) {
        hipLaunchKernelGGL(fm::k_ict_piv, dim3(p->grid), dim3(kBlock), 0, s, p->n, (const uint8_t *)p->code,
                           (const double *)p->ict_ld, piv);
        FM_LAUNCH_CHECK();
      } else if (piv) {
        hipLaunchKernelGGL(fm::k_pivots, dim3(p->grid), dim3(kBlock), 0, s, p->geo, (const double *)p->ipiv, piv);
        FM_LAUNCH_CHECK();
      }
    }
    int32_t status = 0;
    fm_status rs = read_status(p, s, &status);
    if (rs) return rs;
    if (status) return fail((fm_status)status, "preconditioner: non-positive pivot");
    return FM_OK;
  };
  p->solved = false;  // the iteration state was overwritten
  return p->mix ? run(float{}) : run(double{});
}

fm_status fm_solve(fm_plan *p, const void *y, const void *sens, const uint8_t *mask, const double *f0,
                   double *f_out, hipStream_t s) {
  fm_status cs = check_plan(p);
  if (cs) return cs;
  if (!f_out) return fail(FM_ERR_ARG, "f_out must not be NULL");
  fm_status st = fm_setup(p, y, sens, mask, s);
  if (st) return st;
  const double *start = f0;
  if (!start) {
    if (p->prm.model == FM_WATERFAT) {
      st = wf_init(p, p->f0buf, s);
      if (st) return st;
    }
    start = p->f0buf;
  }
  FM_HIP(hipMemsetAsync(p->status, 0, sizeof(int32_t), s));
  p->q = 0;
  st = p->mix ? enqueue_start<float>(p, start, s) : enqueue_start<double>(p, start, s);
  if (st) return st;
  st = run_iterations(p, p->prm.niter, s);
  if (st) return st;
  st = dispatch<OpFinal>(p, f_out, s);
  if (st) return st;
  p->solved = true;
  return FM_OK;
}

fm_status fm_iterate(fm_plan *p, int32_t niter, double *f_out, hipStream_t s) {
  fm_status cs = check_plan(p);
  if (cs) return cs;
  if (!p->solved) return fail(FM_ERR_STATE, "fm_iterate needs a previous fm_solve");
  if (niter < 0 || !f_out) return fail(FM_ERR_ARG, "niter must be >= 0 and f_out not NULL");
  fm_status st = run_iterations(p, niter, s);
  if (st) return st;
  return dispatch<OpFinal>(p, f_out, s);
}

fm_status fm_time_kernels(fm_plan *p, int32_t niter, double *ms, int32_t *launches, hipStream_t s) {
  fm_status cs = check_plan(p);
  if (cs) return cs;
  if (!ms || !launches || niter < 0) return fail(FM_ERR_ARG, "bad arguments to fm_time_kernels");
  if (!p->solved) return fail(FM_ERR_STATE, "fm_time_kernels needs a previous fm_solve");
  for (int k = 0; k < FM_NK; ++k) {
    ms[k] = 0.0;
    launches[k] = 0;
  }
  Recorder rec;
  if (use_resident(p) && niter > 0) {
    hipEvent_t e0, e1;
    rec.pair(FM_K_RESIDENT, &e0, &e1);
    if (rec.err != hipSuccess) return fail(FM_ERR_HIP, std::string("event create: ") + hipGetErrorString(rec.err));
    fm_status st = run_resident(p, niter, s, e0, e1);
    if (st) return st;
  }
  for (int i = 0; i < niter && !use_resident(p); ++i) {
    fm_status st = dispatch<OpIterationTimed>(p, s, &rec);
    if (st) return st;
    if (rec.err != hipSuccess) return fail(FM_ERR_HIP, std::string("event record: ") + hipGetErrorString(rec.err));
  }
  FM_HIP(hipStreamSynchronize(s));
  for (size_t k = 0; k < rec.cls.size(); ++k) {
    float t = 0.f;
    FM_HIP(hipEventElapsedTime(&t, rec.ev[2 * k], rec.ev[2 * k + 1]));
    ms[rec.cls[k]] += t;
    launches[rec.cls[k]] += 1;
  }
  return FM_OK;
}

fm_status fm_adjoint(fm_plan *p, const double *dldf, const void *sens, void *dldy, double *v_out,
                     double *dldbeta, int32_t maxit, double rtol, int32_t *iters, hipStream_t s) {
  fm_status cs = check_plan(p);
  if (cs) return cs;
  if (!dldf) return fail(FM_ERR_ARG, "dL/df must not be NULL");
  if (!sens && p->prm.ncoil != 1 && dldy) return fail(FM_ERR_ARG, "sens may be NULL only when ncoil == 1");
  if (maxit < 0 || !(rtol >= 0.0) || !std::isfinite(rtol)) return fail(FM_ERR_ARG, "maxit must be >= 0 and rtol finite, >= 0");
  if (!p->solved) return fail(FM_ERR_STATE, "fm_adjoint needs a converged map from fm_solve or fm_iterate");
  if (p->ict) return fail(FM_ERR_ARG, "fm_adjoint preconditions with IC(0), the diagonal or nothing, not IC_t");
  fm_status st = adj_alloc(p, s);
  if (st) return st;
  FM_HIP(hipMemsetAsync(p->a_status, 0, sizeof(int32_t), s));
  fm::State out{};
  st = dispatch<OpAdjoint>(p, dldf, sens, dldy, v_out, (int)maxit, rtol, &out, s);
  if (st) return st;
  int32_t status = 0;
  FM_HIP(hipMemcpyAsync(&status, p->a_status, sizeof(int32_t), hipMemcpyDeviceToHost, s));
  FM_HIP(hipStreamSynchronize(s));
  if (iters) *iters = out.cg_it;
  if (dldbeta) *dldbeta = out.cg_dbeta;
  if (status == FM_ERR_NOT_PD) return fail(FM_ERR_NOT_PD, "adjoint CG: the Hessian is not positive definite at the map");
  if (status) return fail((fm_status)status, "adjoint CG reported a device-side error");
  return FM_OK;
}

fm_status fm_set_beta(fm_plan *p, double beta) {
  fm_status cs = check_plan(p);
  if (cs) return cs;
  if (!(beta >= 0.0) || !std::isfinite(beta)) return fail(FM_ERR_ARG, "beta must be finite and >= 0");
  drop_graphs(p);
  p->prm.beta = beta;
  p->solved = false;
  return FM_OK;
}

fm_status fm_components(fm_plan *p, const void *y, const void *sens, const double *f, void *m_out,
                        hipStream_t s) {
  fm_status cs = check_plan(p);
  if (cs) return cs;
  if (!y || !m_out) return fail(FM_ERR_ARG, "y and m_out must not be NULL");
  if (!sens && p->prm.ncoil != 1) return fail(FM_ERR_ARG, "sens may be NULL only when ncoil == 1");
  if (!p->setup_done) return fail(FM_ERR_STATE, "fm_components needs fm_setup or fm_solve first");
  if (!f && !p->solved) return fail(FM_ERR_STATE, "f is NULL and there is no solved map");
  const double *te = p->comp_tab;
  const double2 *B = (const double2 *)(p->comp_tab + p->prm.necho);
  if (p->mix) {
    hipLaunchKernelGGL(fm::k_components<float>, dim3(p->grid), dim3(kBlock), 0, s, p->geo, p->prm.ncoil,
                       p->prm.necho, p->ncomp, (const float2 *)y, (const float2 *)sens, (const uint8_t *)p->code, f,
                       (const float *)p->F[p->iter_host & 1], te, B, (float2 *)m_out);
  } else {
    hipLaunchKernelGGL(fm::k_components<double>, dim3(p->grid), dim3(kBlock), 0, s, p->geo, p->prm.ncoil,
                       p->prm.necho, p->ncomp, (const float2 *)y, (const float2 *)sens, (const uint8_t *)p->code, f,
                       (const double *)p->F[p->iter_host & 1], te, B, (float2 *)m_out);
  }
  FM_LAUNCH_CHECK();
  return FM_OK;
}

fm_status fm_plan_status(fm_plan *p, hipStream_t s) {
  fm_status cs = check_plan(p);
  if (cs) return cs;
  int32_t status = 0;
  fm_status rs = read_status(p, s, &status);
  if (rs) return rs;
  if (status) return fail((fm_status)status, "the last solve reported a device-side error");
  return FM_OK;
}

fm_status fm_set_schedule(fm_plan *p, int32_t sched) {
  fm_status cs = check_plan(p);
  if (cs) return cs;
  if (sched != FM_SCHED_AUTO && sched != FM_SCHED_STREAM && sched != FM_SCHED_RESIDENT)
    return fail(FM_ERR_ARG, "unknown schedule");
  if (sched == FM_SCHED_RESIDENT && !p->res_ok)
    return fail(FM_ERR_ARG, "the plan does not qualify for the resident schedule");
  p->sched = sched;
  return FM_OK;
}

fm_status fm_get_schedule(fm_plan *p, int32_t *sched) {
  fm_status cs = check_plan(p);
  if (cs) return cs;
  if (!sched) return fail(FM_ERR_ARG, "sched must not be NULL");
  *sched = use_resident(p) ? FM_SCHED_RESIDENT : FM_SCHED_STREAM;
  return FM_OK;
}

fm_status fm_get_trace(fm_plan *p, double *trace, hipStream_t s) {
  fm_status cs = check_plan(p);
  if (cs) return cs;
  if (!trace) return fail(FM_ERR_ARG, "trace must not be NULL");
  FM_HIP(hipMemcpyAsync(trace, p->trace, sizeof(double) * FM_TR_W * ((size_t)p->prm.niter + 1),
                        hipMemcpyDeviceToHost, s));
  int32_t status = 0;
  fm_status rs = read_status(p, s, &status);
  if (rs) return rs;
  if (status) return fail((fm_status)status, "the solve reported a device-side error");
  return FM_OK;
}

fm_status fm_mask_count(fm_plan *p, int64_t *count, hipStream_t s) {
  fm_status cs = check_plan(p);
  if (cs) return cs;
  if (!count) return fail(FM_ERR_ARG, "count must not be NULL");
  if (!p->setup_done) return fail(FM_ERR_STATE, "fm_mask_count needs fm_setup first");
  double v = 0.0;
  FM_HIP(hipMemcpyAsync(&v, p->nmask, sizeof(double), hipMemcpyDeviceToHost, s));
  FM_HIP(hipStreamSynchronize(s));
  *count = (int64_t)v;
  return FM_OK;
}

}  // extern "C"

// Water-fat initialisation lives with the rest of the plan internals.
#include "fm_waterfat.inc"

// Batched solves of many volumes.
#include "fm_batch.inc"

// The allocation-free solve.
#include "fm_noalloc.inc"
