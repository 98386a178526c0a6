// Host side of the stage solver, and its kernels outside the solver launches.
// The solver is a device-resident state machine advanced by launches of one
// kernel (tick.h).  The host captures a fixed number of launches in a graph,
// replays it, and polls a pinned flag written by a small report kernel at the
// end of each replay.
#include <algorithm>
#include <chrono>
#include <cmath>
#include <cstdlib>
#include <cstring>
#include <mutex>
#include <string>
#include <vector>

#include "device.h"
#include "host.h"
#include "solver.h"

namespace pfc {

#ifdef PFC_TICK_TIMING
int tick_trace_set_f64(unsigned long long*, unsigned long long);
int tick_trace_set_f32(unsigned long long*, unsigned long long);
unsigned long long tick_trace_count_f64();
unsigned long long tick_trace_count_f32();
// the two precisions share the buffer: a traced run uses one of them
extern "C" int pfc_debug_trace(unsigned long long* dev_buf, unsigned long long cap) {
  const int rc = tick_trace_set_f64(dev_buf, cap);
  return rc ? rc : tick_trace_set_f32(dev_buf, cap);
}
extern "C" unsigned long long pfc_debug_trace_count(void) {
  return std::max(tick_trace_count_f64(), tick_trace_count_f32());
}
#endif

__global__ void k_report(const InstDev* __restrict__ insts, int count, int* __restrict__ flags) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < count) {
    flags[i] = insts[i].st[0].phase;
    flags[count + i] = insts[i].st[0].launches;
  }
}

// Per-tau operator values: C_d = M + delta K, C_sd = M + sqrt(delta) K (stored
// unless shared_ops) and their Jacobi diagonals, in the inner precision.
template <typename T>
__global__ void k_prep_ops(InstDev I) {
  const int sl = blockIdx.x * PFC_WAVES + (threadIdx.x >> 6);
  if (sl >= I.m.n_slices) return;
  const int lane = threadIdx.x & 63;
  const int i = sl * 64 + lane;
  const int base = I.m.slice_ptr[sl];
  const int w = (I.m.slice_ptr[sl + 1] - base) >> 6;
  double dd = 0.0, ds = 0.0;
  for (int k = 0; k < w; ++k) {
    const long long e = (long long)base + k * 64 + lane;
    const double cd = I.m.M[e] + I.delta * I.m.K[e];
    const double cs = I.m.M[e] + I.sdelta * I.m.K[e];
    if (!I.shared_ops) {
      ((T*)I.Cd)[e] = T(cd);
      ((T*)I.Csd)[e] = T(cs);
    }
    if (I.m.col[e] == i) { dd += cd; ds += cs; }
  }
  if (i < I.n) {
    ((T*)I.dinvCd)[i] = T(1.0 / dd);
    ((T*)I.dinvCsd)[i] = T(1.0 / ds);
  }
}

// S_D = M - 2 delta K + delta K M_D^{-1} K on the second-ring pattern (Section 4.1)
// and its Jacobi diagonal, in the inner precision.
template <typename T>
__global__ void k_prep_sd(InstDev I) {
  const int sl = blockIdx.x * PFC_WAVES + (threadIdx.x >> 6);
  if (sl >= I.m.n_slices) return;
  const int lane = threadIdx.x & 63;
  const int i = sl * 64 + lane;
  const int base = I.m.w_slice_ptr[sl];
  const int w = (I.m.w_slice_ptr[sl + 1] - base) >> 6;
  double dg = 0.0;
  for (int k = 0; k < w; ++k) {
    const long long e = (long long)base + k * 64 + lane;
    const long long p = I.m.w_p1pos[e];
    double v = p >= 0 ? I.m.M[p] - 2.0 * I.delta * I.m.K[p] : 0.0;
    double acc = 0.0;
    for (int t = I.m.w_tri_ptr[e]; t < I.m.w_tri_ptr[e + 1]; ++t) {
      const int e1 = I.m.w_tri[2 * t], e2 = I.m.w_tri[2 * t + 1];
      acc += I.m.K[e1] * I.m.dinvM[I.m.col[e1]] * I.m.K[e2];
    }
    v += I.delta * acc;
    ((T*)I.SDv)[e] = T(v);
    if (I.m.w_col[e] == i) dg += v;
  }
  if (i < I.n) ((T*)I.dinvSD)[i] = T(1.0 / dg);
}

// K_+(psi) and F(mu) of the PFC1 model on the P1 pattern, in place (LDS: 8 per thread)
#define PFC_MOB_CAP 8
__global__ void k_assemble_mob(InstDev I, const double* __restrict__ psi, const double* __restrict__ mu) {
  __shared__ double acc[PFC_MOB_CAP * 256];
  const int sl = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (sl >= I.m.n_slices) return;
  const int lane = threadIdx.x & 63;
  const int base = I.m.slice_ptr[sl];
  const int w = (I.m.slice_ptr[sl + 1] - base) >> 6;
  const long long e0 = (long long)base + lane;
  row_mob<true>(I.m, sl, lane, acc + threadIdx.x, 256, PFC_MOB_CAP, w, [&](int j) { return psi[j]; },
                [&](int j) { return mu[j]; }, I.psi_min, I.Kp + e0, I.Fm + e0);
}

// per slice: sum of (M psi)_i and of (M 1)_i over its rows (the mobility mean
// M0 = 1^T M psi / 1^T M 1 - psi_min is formed on the host in slice order)
__global__ void k_mass_moments(InstDev I, const double* __restrict__ psi) {
  const int sl = blockIdx.x * PFC_WAVES + (threadIdx.x >> 6);
  if (sl >= I.m.n_slices) return;
  const int lane = threadIdx.x & 63;
  const int base = I.m.slice_ptr[sl];
  const int w = (I.m.slice_ptr[sl + 1] - base) >> 6;
  double a = 0.0, b = 0.0;
  for (int k = 0; k < w; ++k) {
    const long long e = (long long)base + k * 64 + lane;
    a += I.m.M[e] * psi[I.m.col[e]];
    b += I.m.M[e];
  }
  a = wave_sum(a);
  b = wave_sum(b);
  if (lane == 0) { I.errpart[sl] = a; I.errpart[I.m.n_slices + sl] = b; }
}

__global__ void k_apply_AR(InstDev I, const double* __restrict__ y, double* __restrict__ out) {
  const int sl = __builtin_amdgcn_readfirstlane((int)(blockIdx.x * PFC_WAVES + (threadIdx.x >> 6)));
  if (sl >= I.m.n_slices) return;
  const int lane = threadIdx.x & 63;
  const int i = sl * 64 + lane;
  const int n = I.n;
  double w0, w1, w2;
  const PatView<PFC_COL_MEM> pv{I.m.slice_ptr, I.m.col, I.m.uw, 0, I.n, 0, 0.0f, nullptr};
  const BlockVec<double> yv{y, y + 2LL * n};
  if (I.model == PFC_MODEL_PFC1) block_row<PFC_COL_MEM, true>(I, pv, sl, lane, I.tau, I.m11, yv, w0, w1, w2);
  else block_row<PFC_COL_MEM, false>(I, pv, sl, lane, I.tau, I.m11, yv, w0, w1, w2);
  if (i < n) { out[i] = w0; out[n + i] = w1; out[2 * n + i] = w2; }
}

// Embedded error of the step just taken (psi block): per slice the sum of
// ((psi_{k+1} - psi_hat) / (atol + rtol max(|psi_k|, |psi_{k+1}|)))^2 with
// psi_hat = psi_k + sum_j mhat_j y_j^psi (Table rosenbrock_scheme).
__global__ void k_embedded_err(InstDev I, const double* __restrict__ xold, const double* __restrict__ xnew, double rtol,
                               double atol) {
  const int sl = blockIdx.x;
  const int lane = threadIdx.x;
  const int n = I.n;
  const long long n3 = 3LL * n;
  const int i = sl * 64 + lane;
  double e2 = 0.0;
  if (i < n) {
    const double po = xold[n + i], pn = xnew[n + i];
    const double ph = po + ROS_MH1 * I.ys[n + i] + ROS_MH2 * I.ys[n3 + n + i] + ROS_MH3 * I.ys[2 * n3 + n + i];
    const double sc = atol + rtol * fmax(fabs(po), fabs(pn));
    const double e = (pn - ph) / sc;
    e2 = e * e;
  }
  e2 = wave_sum(e2);
  if (lane == 0) I.errpart[sl] = e2;
}

// Stage right-hand side with the stage state at the row's neighbours formed once:
// the row products read it, and so do, from LDS, the element sums of the cubic
// load (and of K_+ mu: MOB).
template <int Q, bool MOB>
__global__ __launch_bounds__(PFC_ROW_T) void k_row_rhs(InstDev I, int stage, double* __restrict__ b, int cap) {
  const int T = blockDim.x, tid = threadIdx.x, st = T + 1, n = I.n;
  const int sl = xcd_rank(blockIdx.x, gridDim.x) * (T >> 6) + (tid >> 6), lane = tid & 63, i = sl * 64 + lane;
  if (sl >= I.m.n_slices) return;
  double* sp = pfc_row_lds + tid;
  double* sm = sp + cap * st;
  const int base = I.m.slice_ptr[sl], w = (I.m.slice_ptr[sl + 1] - base) >> 6;
  const long long e0 = (long long)base + lane;
  const WaveCols wc = wave_cols(I.m, sl, lane, e0);
  double b0, b1, b2;
  const StageSums q = stage_rhs_products(I, w, stage, [&](int k) { return e0 + 64LL * k; },
                                         [&](int k) { return wc.at(k); }, [&](int k, double mu, double ps) {
                                           sp[k * st] = ps;
                                           if constexpr (MOB) sm[k * st] = mu;
                                         });
  double g = 0.0, kpm = 0.0;
  for_visits<Q, VisitU<Q>::lds, false, false>(I.m, sl, lane, [=](const Visit<Q>& v, int c) { return sp[v.slot(c) * st]; },
                                       [&](const Visit<Q>& v) {
    g += visit_psi3<Q>(I.m, v);
    if constexpr (MOB)
      kpm += visit_Kplus_mu<Q>(I.m, v, [=](const Visit<Q>& u, int c) { return sm[u.slot(c) * st]; }, I.psi_min);
  });
  stage_rhs_finish(I, q, stage, g, kpm, b0, b1, b2);
  if (i < n) { b[i] = b0; b[n + i] = b1; b[2 * n + i] = b2; }
}

__global__ void k_stage_rhs(InstDev I, int stage, double* __restrict__ b) {
  const int sl = blockIdx.x * PFC_WAVES + (threadIdx.x >> 6);
  if (sl >= I.m.n_slices) return;
  const int lane = threadIdx.x & 63;
  const int i = sl * 64 + lane;
  double b0, b1, b2;
  const PatView<PFC_COL_MEM> pv{I.m.slice_ptr, I.m.col, I.m.uw, 0, I.n, 0, 0.0f, nullptr};
  stage_rhs_row<PFC_COL_MEM>(I, pv, sl, lane, stage, b0, b1, b2);
  if (i < I.n) { b[i] = b0; b[I.n + i] = b1; b[2 * I.n + i] = b2; }
}

static int launch_stage_rhs(const pfc_mesh* m, const InstDev& h, int stage, double* b, hipStream_t s) {
  const bool mob = h.model == PFC_MODEL_PFC1;
  const RowPlan p = row_plan(m, mob ? 2 : 1);
  const size_t lds = p.lds(mob ? 2 : 1);
  if (!p.stage) {
    hipLaunchKernelGGL(k_stage_rhs, dim3(slice_blocks(m->n_slices)), dim3(PFC_WG), 0, s, h, stage, b);
  } else if (mob) {  // P1 meshes
    if (m->dim == 2) hipLaunchKernelGGL((k_row_rhs<3, true>), row_grid(m, p.T), dim3(p.T), lds, s, h, stage, b, p.cap);
    else hipLaunchKernelGGL((k_row_rhs<4, true>), row_grid(m, p.T), dim3(p.T), lds, s, h, stage, b, p.cap);
  } else {
#define PFC_X(Q) hipLaunchKernelGGL((k_row_rhs<Q, false>), row_grid(m, p.T), dim3(p.T), lds, s, h, stage, b, p.cap)
    PFC_FOR_NLOC(m, PFC_X)
#undef PFC_X
  }
  PFC_HIP(hipGetLastError());
  return PFC_OK;
}

// ---- host side ------------------------------------------------------------------

static size_t align_up(size_t x) { return (x + 255) & ~(size_t)255; }

// Halo of the two-iterations-per-launch PCG (N + 1 rows), or 0 where it does not
// apply: float64 single-reduction instances on 2D periodic grids (7 entries per
// row) with computed columns, at most PFC_WAVES slices per workgroup, every
// neighbour within N + 1 rows of its row (mod n), the three LDS arrays within
// PFC_SS_LDS and the halo ranges within the kernel's unrolled passes.
static int sstep_halo(const pfc_mesh* m, const pfc_opts& o, int team_size) {
  const MeshDev& d = m->dev;
  if (o.pcg_steps_per_launch != 2 || o.precision != PFC_FP64 || o.single_reduction != 1 || o.grid_columns != 1) return 0;
  if (d.dim != 2 || d.gN < 3 || d.uw != 7 || team_size < 1) return 0;
  const int spw = (d.n_slices + team_size - 1) / team_size;
  if (spw > PFC_WAVES) return 0;
  const int n = d.n, H = d.gN + 1;
  if (2 * H >= n) return 0;
  for (int c = 0; c < 9; ++c)  // the row classes of a 2D grid
    for (int k = 0; k < d.uw; ++k) {
      int s = d.glin[c * PFC_GRID_W + k];
      s = s > n / 2 ? s - n : (s < -(n / 2) ? s + n : s);
      if (s > H || s < -H) return 0;
    }
  const int rmax = std::min(spw * 64, n);
  if (3 * rmax + 8 * H > PFC_SS_LDS || rmax + 4 * H > PFC_SS_NA * PFC_WG || rmax + 2 * H > PFC_SS_NB * PFC_WG) return 0;
  return H;
}

// Two PCG iterations per launch on blocks of a 3D grid (ph_scg3): float
// (mixed-precision) single-reduction instances on periodic grids of side 64 with
// computed columns and entry directions, one row per thread (a team of 256
// workgroups of 4 x 4 x-lines).
static bool sstep_block3(const pfc_mesh* m, const pfc_opts& o, int team_size) {
  const MeshDev& d = m->dev;
  return o.pcg_steps_per_launch == 2 && o.precision == PFC_MIXED && o.single_reduction == 1 && o.grid_columns == 1 &&
         d.dim == 3 && d.gN == PFC_S3_N && d.uw == 15 && d.gdir_ok && team_size == 256 && d.n_slices == 4096;
}

// Two PCG iterations per launch on blocks of a 2D grid (ph_scg2b): single-
// reduction instances (either precision) on periodic grids whose side is a
// multiple of 64, with computed columns and entry directions, one row per
// thread (a team of N^2 / 1024 workgroups of 64 x 16 rows).
static bool sstep_block2(const pfc_mesh* m, const pfc_opts& o, int team_size) {
  const MeshDev& d = m->dev;
  return o.pcg_steps_per_launch == 2 && o.single_reduction == 1 && o.grid_columns == 1 && d.dim == 2 &&
         d.gN >= 64 && d.gN % 64 == 0 && d.uw == 7 && d.gdir_ok && d.n_slices % PFC_WAVES == 0 &&
         team_size == d.n_slices / PFC_WAVES;
}

bool block_form_applies(const pfc_mesh* m, const pfc_opts& o) {
  pfc_opts o2 = o;
  o2.pcg_steps_per_launch = 2;
  return sstep_block2(m, o2, team_size_for(m->n_slices, o.rows_per_thread));
}

// Workgroups of launches that serve the instance alone: its team, or, on meshes of
// at most PFC_SPREAD slices, as few slices a workgroup as the chip's 256 CUs allow.
// Measured with 16 (the team), 4 and 1 slices at most a workgroup: P_CH apply 2D 50^2
// mixed 954, 851, 818 us; stage solve 2D P2 50^2 48.1, 30.6, 26.8 ms.  Near the limit
// the gain runs out: team and spread, 3D 50^3 float64 1701, 1382 us, mixed 1123, 1057,
// 2D 350^2 mixed 980, 943.  A limit of 3840
// slices (four sums a thread in the prologue instead of two) measured slower above
// 2048 (P_CH apply 3D 56^3 float64 1698 -> 1737 us) and below (3D 20^3 967 -> 1100).
// Not for several rows per thread (a wave's sums have to be one slice's), the block
// forms (their workgroups are blocks) and launches that stage columns (those of the
// team's slices).
int solo_workgroups(const pfc_mesh* m, const pfc_opts& o, int team_size) {
  const MeshDev& d = m->dev;
  const bool grid = d.gN > 0 && o.grid_columns;
  const bool staged = !grid && d.uw >= 1 && d.uw <= PFC_LCOL_W && !(o.precision == PFC_FP64 && d.uw < 8);
  if (o.rows_per_thread > 1 || d.n_slices > PFC_SPREAD || staged || sstep_block2(m, o, team_size) ||
      sstep_block3(m, o, team_size))
    return team_size;
  const int spw = (d.n_slices + 255) / 256, H = sstep_halo(m, o, team_size);
  if (H > 0 && spw * 64 + 4 * H > PFC_SS_NA_SPREAD * PFC_WG) return team_size;
  return (d.n_slices + spw - 1) / spw;
}

// Carve the instance arena.  With base == nullptr only the size is computed.
size_t carve(InstDev& h, char* base, const pfc_mesh* m, const pfc_opts& o, int team_size) {
  size_t off = 0;
  auto take = [&](size_t bytes) -> char* {
    char* p = base ? base + off : nullptr;
    off += align_up(bytes);
    return p;
  };
  const size_t n = (size_t)m->n, n3 = 3 * n, ns = (size_t)m->nnz_sell;
  const size_t w = o.precision == PFC_MIXED ? 4 : 8;
  const int mr = o.restart;
  if (o.schur_variant == 1) {
    h.SDv = take((size_t)m->dev.w_nnz_sell * w);
    h.dinvSD = take(n * w);
  } else {
    h.SDv = nullptr;
    h.dinvSD = nullptr;
  }
  h.Cd = o.shared_ops ? nullptr : (void*)take(ns * w);
  h.Csd = o.shared_ops ? nullptr : (void*)take(ns * w);
  h.dinvCd = take(n * w);
  h.dinvCsd = take(n * w);
  h.N = (double*)take(ns * 8);
  if (o.model == PFC_MODEL_PFC1) {
    h.Kp = (double*)take(ns * 8);
    h.Fm = (double*)take(ns * 8);
  } else {
    h.Kp = nullptr;
    h.Fm = nullptr;
  }
  h.b = (double*)take(n3 * 8);
  h.xk = (double*)take(n3 * 8);
  h.ys = (double*)take(3 * n3 * 8);
  h.V = (double*)take((size_t)(mr + 1) * n3 * 8);
  h.Z = (double*)take((size_t)mr * n3 * 8);
  h.W = (double*)take(n3 * 8);
  h.r_ = take(n * 8); h.pA = take(n * 8); h.pB = take(n * 8); h.q = take(n * 8);
  h.y0 = take(n * 8); h.y1 = take(n * 8); h.zt = take(n * 8); h.x1 = take(n * 8); h.x2 = take(n * 8);
  h.rB = take(n * 8); h.wB = take(n * 8); h.sA = take(n * 8); h.sB = take(n * 8);
  h.xbak = (double*)take(n3 * 8);
  h.errpart = (double*)take((size_t)m->n_slices * 2 * 8);
  h.solo_wgs = solo_workgroups(m, o, team_size);
  h.part = (double*)take(2 * (size_t)team_size * 4 * sizeof(double));
  h.gpart = (double*)take(2 * (size_t)team_size * PFC_GS_NV * sizeof(double));
  h.sH = sstep_halo(m, o, team_size);
  h.sstep = sstep_block2(m, o, team_size) ? 3 : (h.sH > 0 ? 1 : (sstep_block3(m, o, team_size) ? 2 : 0));
  h.sbas = h.sstep ? (double*)take(10 * n * 8) : nullptr;
  // (of launches on more workgroups than the team's, at most one a slice: in sA and sB,
  // 16 n bytes that only the one-iteration form uses, in solves of its own)
  h.spart = !h.sstep ? nullptr
            : h.solo_wgs != team_size ? (double*)h.sA
                                      : (double*)take(2 * (size_t)team_size * 32 * sizeof(double));
  h.st = (State*)take(2 * sizeof(State));
  h.hist = (Hist*)take(sizeof(Hist));
  h.rec_inner = (int*)take((size_t)o.max_steps * 5 * sizeof(int));
  h.info = (InfoDev*)take((size_t)3 * o.max_run_steps * sizeof(InfoDev));
  h.max_infos = 3 * o.max_run_steps;
  return off;
}

int team_size_for(int n_slices, int rows_per_thread) {
  int rpt = rows_per_thread;
  if (rpt <= 0) rpt = 1;
  return (n_slices + PFC_WAVES * rpt - 1) / (PFC_WAVES * rpt);
}

static int validate_opts(const pfc_opts* o) {
  if (!o || o->struct_size != (int)sizeof(pfc_opts)) { set_error("pfc_opts: struct_size mismatch"); return PFC_ERR_ARG; }
  if (o->precision != PFC_FP64 && o->precision != PFC_MIXED) { set_error("pfc_opts: bad precision"); return PFC_ERR_ARG; }
  if (o->restart < 1 || o->restart > PFC_MAXM) { set_error("pfc_opts: restart must be in 1..32"); return PFC_ERR_ARG; }
  if (o->max_steps < 1 || o->inner_maxit < 1 || o->max_run_steps < 1) { set_error("pfc_opts: counts must be positive"); return PFC_ERR_ARG; }
  if (!(o->outer_tol > 0.0) || !(o->inner_tol > 0.0) || !(o->inner_tol < 1.0)) { set_error("pfc_opts: tolerances must be in (0,1)"); return PFC_ERR_ARG; }
  if (o->rows_per_thread < 0 || o->rows_per_thread > 8) { set_error("pfc_opts: rows_per_thread must be 0..8"); return PFC_ERR_ARG; }
  if (o->ticks_per_graph < 0 || o->ticks_per_graph > 4096) { set_error("pfc_opts: ticks_per_graph must be 0..4096"); return PFC_ERR_ARG; }
  if (o->single_reduction != 0 && o->single_reduction != 1) { set_error("pfc_opts: single_reduction must be 0 or 1"); return PFC_ERR_ARG; }
  if (o->schur_variant != 0 && o->schur_variant != 1) { set_error("pfc_opts: schur_variant must be 0 (S_CH) or 1 (S_D)"); return PFC_ERR_ARG; }
  if (o->sd_iters < 1 || o->sd_iters > 10000) { set_error("pfc_opts: sd_iters must be in 1..10000"); return PFC_ERR_ARG; }
  if (o->model != PFC_MODEL_PFC2 && o->model != PFC_MODEL_PFC1) { set_error("pfc_opts: bad model"); return PFC_ERR_ARG; }
  if (!std::isfinite(o->psi_min)) { set_error("pfc_opts: psi_min must be finite"); return PFC_ERR_ARG; }
  if (o->grid_columns != 0 && o->grid_columns != 1) { set_error("pfc_opts: grid_columns must be 0 or 1"); return PFC_ERR_ARG; }
  if (o->pcg_steps_per_launch != 1 && o->pcg_steps_per_launch != 2) {
    set_error("pfc_opts: pcg_steps_per_launch must be 1 or 2");
    return PFC_ERR_ARG;
  }
  if (o->gamma_mode != PFC_GAMMA_SCALE_ROW && o->gamma_mode != PFC_GAMMA_LITERAL) {
    set_error("pfc_opts: bad gamma_mode");
    return PFC_ERR_ARG;
  }
  for (int k = 0; k < 5; ++k)
    if (o->inner_fixed[k] < 0 || o->inner_fixed[k] > 100000) {
      set_error("pfc_opts: inner_fixed counts must be in 0..100000");
      return PFC_ERR_ARG;
    }
  return PFC_OK;
}

void fill_info(pfc_solve_info* dst, const InfoDev& s) {
  dst->status = s.status;
  dst->outer_iters = s.outer_iters;
  dst->cycles = s.cycles;
  dst->inner_applies = s.inner_applies;
  dst->inner_total = s.inner_total;
  for (int k = 0; k < 5; ++k) dst->inner_max[k] = s.inner_max[k];
  dst->reserved = 0;
  dst->est_rel_res = s.est_rel_res;
  dst->true_rel_res = s.true_rel_res;
  dst->t_solve = s.t_solve;
}

// The descriptors (h_descs) must be filled before build(): a one-instance
// group bakes that instance's state and partial-sum buffers into the launches.
int Group::build(hipStream_t capture, int precision, int ticks) {
  for (int i = 0; i < count; ++i)
    if (!h_descs[i].st || !h_descs[i].part || h_descs[i].team_size <= 0) {
      set_error("internal: launch group built before its descriptors were set");
      return PFC_ERR_STATE;
    }
  if (count == 1 && h_descs[0].team_size != n_wg && h_descs[0].solo_wgs != n_wg) {
    set_error("internal: team size mismatch");
    return PFC_ERR_STATE;
  }
  // the mesh pattern of every team entry, and whether the launches stage the
  // columns.  They can when every mesh has a uniform slice width <= PFC_LCOL_W
  // and a workgroup owns at most PFC_WAVES slices (the staging buffer holds
  // exactly that).  Staging moves the column stream into the prologue's round
  // trip; it pays where that stream is a large share of a launch's bytes
  // (measured: 3D 64^3 mixed +5.7%, the mixed 2D/3D served mix +6%, 2D 512^2
  // float64 -2%, where the 7 columns are 16% of an iteration's bytes), so
  // float64 runs stage only from 8 columns per row on (3D: 22%).  When every
  // mesh of the launch is a periodic grid (MeshDev::gN), the columns are
  // computed from the row instead and no column stream is read at all
  // (measured against the stored forms: 2D 512^2 float64 +8.7%, 3D 64^3 mixed
  // +17%, the served mix +11%, the batched 128^2 mixed run with 4 rows per
  // thread +5.5%).
  bool lds = true, grid = true;
  for (TeamEntry& t : h_teams) {
    const MeshDev& m = h_descs[t.inst].m;
    t.uw = m.uw;
    t.col = m.col;
    t.n_slices = m.n_slices;
    if (!(m.uw >= 1 && m.uw <= PFC_LCOL_W && (m.n_slices + t.size - 1) / t.size <= PFC_WAVES)) lds = false;
    if (precision == PFC_FP64 && m.uw < 8) lds = false;
    if (!(m.gN > 0 && m.uw >= 1) || !h_descs[t.inst].grid_cols) grid = false;
  }
#ifdef PFC_NO_COLUMN_STAGING
  lds = false;
#endif
  cols = grid ? PFC_COL_GRID : (lds ? PFC_COL_LDS : PFC_COL_MEM);
  PFC_HIP(hipMemcpy(d_teams, h_teams.data(), sizeof(TeamEntry) * h_teams.size(), hipMemcpyHostToDevice));
  const int* pcol = count == 1 ? h_descs[0].m.col : nullptr;
  const int puw = count == 1 ? h_descs[0].m.uw : 0;
  const int pnsl = count == 1 ? h_descs[0].m.n_slices : 0;
  PFC_HIP(hipStreamBeginCapture(capture, hipStreamCaptureModeThreadLocal));
  for (int t = 0; t < ticks; ++t) {
    const int par = t & 1;
    State* sin = nullptr;
    State* sout = nullptr;
    double* pin = nullptr;
    double* pout = nullptr;
    const double* gin = nullptr;
    if (count == 1) {
      // launches on more workgroups than the team's leave a sum per slice, in the buffer of
      // the orthogonalisation's sums: 64 numbers a workgroup of the team are 4 for each of
      // its 16 slices, and no launch leaves both kinds
      const bool spread = n_wg != h_descs[0].team_size;
      double* part = spread ? h_descs[0].gpart : h_descs[0].part;
      const size_t np = spread ? (size_t)h_descs[0].team_size * (PFC_GS_NV / 4) : n_wg;
      sin = h_descs[0].st + par;
      sout = h_descs[0].st + (1 - par);
      pin = part + (size_t)par * np * 4;
      pout = part + (size_t)(1 - par) * np * 4;
      if (h_descs[0].spart) gin = h_descs[0].spart + (size_t)par * n_wg * 32;
    }
    // the launches have the 2D block form (ph_scg2b) when some instance takes it;
    // the other instances run one PCG iteration per launch in them
    bool b2 = false;
    for (int i = 0; i < count; ++i) b2 = b2 || h_descs[i].sstep == 3;
    const int team = count == 1 ? h_descs[0].team_size : 0;
    const TickLaunch q{d_teams, d_descs, sin, sout, pin, pout, gin, par, pcol, puw, pnsl, team, n_wg, cols, count == 1, b2};
    if (precision == PFC_MIXED) launch_tick_f32(q, capture);
    else launch_tick_f64(q, capture);
  }
  hipLaunchKernelGGL(k_report, dim3((count + 255) / 256), dim3(256), 0, capture, d_descs, count, d_flags);
  hipGraph_t g = nullptr;
  hipError_t e = hipStreamEndCapture(capture, &g);
  if (e != hipSuccess) return hip_fail(e, "hipStreamEndCapture");
  e = hipGraphInstantiate(&exec, g, nullptr, nullptr, 0);
  (void)hipGraphDestroy(g);
  if (e != hipSuccess) return hip_fail(e, "hipGraphInstantiate");
  return PFC_OK;
}

int Group::alloc(const std::vector<int>& team_sizes) {
  count = (int)team_sizes.size();
  h_teams.clear();
  for (int i = 0; i < count; ++i)
    for (int r = 0; r < team_sizes[i]; ++r) h_teams.push_back(TeamEntry{i, r, team_sizes[i], 0, nullptr, 0, 0});
  n_wg = (int)h_teams.size();
  PFC_HIP(hipMalloc((void**)&d_teams, sizeof(TeamEntry) * h_teams.size()));
  PFC_HIP(hipMalloc((void**)&d_descs, sizeof(InstDev) * count));
  PFC_HIP(hipHostMalloc((void**)&h_descs, sizeof(InstDev) * count, hipHostMallocDefault));
  PFC_HIP(hipHostMalloc((void**)&h_states, sizeof(State) * count, hipHostMallocDefault));
  PFC_HIP(hipHostMalloc((void**)&h_flags, sizeof(int) * 2 * count, hipHostMallocMapped));
  PFC_HIP(hipHostGetDevicePointer((void**)&d_flags, h_flags, 0));
  for (int i = 0; i < count; ++i) h_flags[i] = -1;
  PFC_HIP(hipEventCreateWithFlags(&ev[0], hipEventDisableTiming));
  PFC_HIP(hipEventCreateWithFlags(&ev[1], hipEventDisableTiming));
  return PFC_OK;
}

void Group::release() {
  if (exec) (void)hipGraphExecDestroy(exec);
  if (d_teams) (void)hipFree(d_teams);
  if (d_descs) (void)hipFree(d_descs);
  if (h_descs) (void)hipHostFree(h_descs);
  if (h_states) (void)hipHostFree(h_states);
  if (h_flags) (void)hipHostFree(h_flags);
  if (ev[0]) (void)hipEventDestroy(ev[0]);
  if (ev[1]) (void)hipEventDestroy(ev[1]);
  *this = Group();
}

// Upload descriptors and initial states (stream ordered), then replay the
// graph until every instance reports PH_DONE.
int Group::run(hipStream_t s, const std::vector<State*>& dev_states, double timeout_s) {
  PFC_HIP(hipMemcpyAsync(d_descs, h_descs, sizeof(InstDev) * count, hipMemcpyHostToDevice, s));
  for (int i = 0; i < count; ++i)
    PFC_HIP(hipMemcpyAsync(dev_states[i], h_states + i, sizeof(State), hipMemcpyHostToDevice, s));
  const auto t0 = std::chrono::steady_clock::now();
  PFC_HIP(hipGraphLaunch(exec, s));
  PFC_HIP(hipEventRecord(ev[0], s));
  PFC_HIP(hipGraphLaunch(exec, s));
  PFC_HIP(hipEventRecord(ev[1], s));
  long long k = 0;
  for (;;) {
    PFC_HIP(hipEventSynchronize(ev[k & 1]));
    bool all = true;
    for (int i = 0; i < count; ++i)
      if (((volatile int*)h_flags)[i] != PH_DONE) { all = false; break; }
    if (all) break;
    const double el = std::chrono::duration<double>(std::chrono::steady_clock::now() - t0).count();
    if (el > timeout_s) {
      (void)hipStreamSynchronize(s);
      set_error("solver did not finish within the time limit");
      return PFC_ERR_STATE;
    }
    PFC_HIP(hipGraphLaunch(exec, s));
    PFC_HIP(hipEventRecord(ev[k & 1], s));
    ++k;
  }
  graphs_run = k + 2;
  PFC_HIP(hipStreamSynchronize(s));
  launches = 0;
  for (int i = 0; i < count; ++i) launches = std::max(launches, (long long)((volatile int*)h_flags)[count + i]);
  return PFC_OK;
}

static int ensure_group(pfc_instance* I) {
  if (I->grp.exec) return PFC_OK;
  int rc = I->grp.alloc(std::vector<int>{I->solo_wgs});
  if (rc) return rc;
  I->grp.h_descs[0] = I->h;
  return I->grp.build(I->capture, I->opts.precision, I->ticks);
}

static int prep_ops(pfc_instance* I, hipStream_t s) {
  const InstDev& h = I->h;
  if (I->ops_tau_s == h.tau_p) return PFC_OK;
  const int nb = slice_blocks(I->mesh->n_slices);
  if (I->opts.precision == PFC_MIXED)
    hipLaunchKernelGGL(k_prep_ops<float>, dim3(nb), dim3(PFC_WG), 0, s, h);
  else
    hipLaunchKernelGGL(k_prep_ops<double>, dim3(nb), dim3(PFC_WG), 0, s, h);
  if (h.schur_d) {
    if (I->opts.precision == PFC_MIXED)
      hipLaunchKernelGGL(k_prep_sd<float>, dim3(nb), dim3(PFC_WG), 0, s, h);
    else
      hipLaunchKernelGGL(k_prep_sd<double>, dim3(nb), dim3(PFC_WG), 0, s, h);
  }
  PFC_HIP(hipGetLastError());
  I->ops_tau_s = h.tau_p;
  return PFC_OK;
}

int prep_ops_public(pfc_instance* I, hipStream_t s) { return prep_ops(I, s); }

// h.m0 (mobility mean, 1 for PFC2) and h.gamma_mode must be current: FGMRES
// sees block row 1 multiplied by rs, and the preconditioner is built for the
// time step tau_p = m0 rs tau
void set_params(InstDev& h, double r, double tau, double m11) {
  h.r = r; h.tau = tau; h.m11 = m11;
  // (row scaling keeps the arithmetic tau / m11 and an exact unit m11_s)
  const bool lit = (h.gamma_mode == PFC_GAMMA_LITERAL);
  h.rs = lit ? 1.0 : 1.0 / m11;
  h.m11_s = lit ? m11 : 1.0;
  h.tau_s = lit ? tau : tau / m11;
  h.tau_p = h.m0 * h.tau_s;
  h.delta = std::sqrt(h.tau_p);
  h.sdelta = std::sqrt(h.delta);
}

// Mobility mean M0 = (1^T M psi)/(1^T M 1) - psi_min of a PFC1 instance from
// psi (device [n]); PFC2 instances keep M0 = 1.
int set_mobility_mean(pfc_instance* I, const double* psi, hipStream_t s) {
  InstDev& h = I->h;
  if (h.model != PFC_MODEL_PFC1) { h.m0 = 1.0; return PFC_OK; }
  const int ns = I->mesh->n_slices;
  hipLaunchKernelGGL(k_mass_moments, dim3(slice_blocks(ns)), dim3(PFC_WG), 0, s, h, psi);
  PFC_HIP(hipGetLastError());
  std::vector<double> part((size_t)2 * ns);
  PFC_HIP(hipMemcpyAsync(part.data(), h.errpart, sizeof(double) * part.size(), hipMemcpyDeviceToHost, s));
  PFC_HIP(hipStreamSynchronize(s));
  double a = 0.0, b = 0.0;
  for (int k = 0; k < ns; ++k) { a += part[k]; b += part[ns + k]; }
  h.m0 = a / b - h.psi_min;
  if (!(h.m0 > 0.0) || !std::isfinite(h.m0)) {
    set_error("PFC1: the mean mobility of the state is not positive (psi below psi_min on average)");
    return PFC_ERR_ARG;
  }
  return PFC_OK;
}

static State initial_state(int job) {
  State s;
  std::memset(&s, 0, sizeof(s));
  s.phase = PH_START;
  s.job = job;
  return s;
}

// Replay schedules: uploaded into a growable device buffer of the instance.
static int upload_schedules(pfc_instance* I, const pfc_schedule* sch, int count, hipStream_t s) {
  std::vector<int> meta(4 * (size_t)count), cyc, inn;
  for (int k = 0; k < count; ++k) {
    const pfc_schedule& q = sch[k];
    if (q.n_cycles < 0 || q.n_applies < 0 || (q.n_cycles && !q.cycle_len) || (q.n_applies && !q.inner_counts)) {
      set_error("pfc_schedule: invalid schedule");
      return PFC_ERR_ARG;
    }
    int steps = 0;
    for (int c = 0; c < q.n_cycles; ++c) {
      if (q.cycle_len[c] < 1 || q.cycle_len[c] > I->opts.restart) {
        set_error("pfc_schedule: cycle length out of range");
        return PFC_ERR_ARG;
      }
      steps += q.cycle_len[c];
    }
    if (steps != q.n_applies || steps > I->opts.max_steps) {
      set_error("pfc_schedule: applications must equal the sum of cycle lengths and fit max_steps");
      return PFC_ERR_ARG;
    }
    meta[4 * k + 0] = (int)cyc.size();
    meta[4 * k + 1] = q.n_cycles;
    meta[4 * k + 2] = (int)(inn.size() / 5);
    meta[4 * k + 3] = q.n_applies;
    cyc.insert(cyc.end(), q.cycle_len, q.cycle_len + q.n_cycles);
    for (int a = 0; a < 5 * q.n_applies; ++a) {
      if (q.inner_counts[a] < 0 || q.inner_counts[a] > 100000) { set_error("pfc_schedule: bad inner count"); return PFC_ERR_ARG; }
      inn.push_back(q.inner_counts[a]);
    }
  }
  if (cyc.empty()) cyc.push_back(0);
  if (inn.empty()) inn.push_back(0);
  const size_t need = sizeof(int) * (meta.size() + cyc.size() + inn.size()) + 1024;
  if (need > I->sched_bytes) {
    if (I->d_sched) (void)hipFree(I->d_sched);
    I->d_sched = nullptr;
    PFC_HIP(hipMalloc((void**)&I->d_sched, need));
    I->sched_bytes = need;
  }
  PFC_HIP(hipStreamSynchronize(s));
  int* p = I->d_sched;
  PFC_HIP(hipMemcpy(p, meta.data(), sizeof(int) * meta.size(), hipMemcpyHostToDevice));
  PFC_HIP(hipMemcpy(p + meta.size(), cyc.data(), sizeof(int) * cyc.size(), hipMemcpyHostToDevice));
  PFC_HIP(hipMemcpy(p + meta.size() + cyc.size(), inn.data(), sizeof(int) * inn.size(), hipMemcpyHostToDevice));
  I->h.sched_meta = p;
  I->h.sched_cycles = p + meta.size();
  I->h.sched_inner = p + meta.size() + cyc.size();
  I->h.replay = 1;
  return PFC_OK;
}

// Scratch of the allocation-free operator apply (pfc_apply_AR_noalloc): the
// values of N(psi_k) on the mesh's stored pattern (PFC_NOALLOC_MAX_ENTRIES,
// include/pfc.h).  Every GPU the library runs
// on holds its own copy of this array, at its own address, until the process
// ends; host code reaches it only through the address resolved per device
// below (the array's name is a host-side stand-in, not a device address).
#define PFC_NOALLOC_MAX_DEVICES 64
static __device__ __align__(256) double scratch[PFC_NOALLOC_MAX_ENTRIES];
static std::mutex g_scratch_mu;
static double* g_scratch_dev[PFC_NOALLOC_MAX_DEVICES] = {};

// Device address of the current device's scratch array, resolved once per
// device (with that device current) and kept.
static int scratch_address(double** out) {
  int d = 0;
  PFC_HIP(hipGetDevice(&d));
  if (d < 0 || d >= PFC_NOALLOC_MAX_DEVICES) {
    set_error("pfc_apply_AR_noalloc: device ordinal beyond the supported " + std::to_string(PFC_NOALLOC_MAX_DEVICES));
    return PFC_ERR_ARG;
  }
  std::lock_guard<std::mutex> lk(g_scratch_mu);
  if (!g_scratch_dev[d]) {
    void* p = nullptr;
    PFC_HIP(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
    if (!p) { set_error("pfc_apply_AR_noalloc: no device address for the scratch array"); return PFC_ERR_HIP; }
    g_scratch_dev[d] = (double*)p;
  }
  *out = g_scratch_dev[d];
  return PFC_OK;
}

int run_single(pfc_instance* I, hipStream_t s, int job) {
  int rc = ensure_group(I);
  if (rc) return rc;
  I->h.job = job;
  I->grp.h_descs[0] = I->h;
  I->grp.h_states[0] = initial_state(job);
  return I->grp.run(s, std::vector<State*>{I->h.st}, I->timeout_s);
}

}  // namespace pfc

using namespace pfc;

extern "C" {

const char* pfc_status_str(int st) {
  switch (st) {
    case PFC_OK: return "ok";
    case PFC_NOT_CONVERGED: return "not converged";
    case PFC_WARN_TAU_CRITICAL: return "converged; tau at or above the critical time step";
    case PFC_ERR_ARG: return "invalid argument";
    case PFC_ERR_OOM: return "out of memory";
    case PFC_ERR_HIP: return "HIP runtime error";
    case PFC_ERR_BREAKDOWN: return "breakdown: non-finite residual or input";
    case PFC_ERR_ADMISSION: return "request exceeds the memory budget";
    case PFC_ERR_STATE: return "invalid state";
    default: return "unknown status";
  }
}

void pfc_opts_default(pfc_opts* o) {
  if (!o) return;
  std::memset(o, 0, sizeof(*o));
  o->struct_size = (int)sizeof(pfc_opts);
  o->precision = PFC_FP64;
  o->restart = 30;
  o->max_steps = 1000;
  o->outer_tol = 1e-8;
  o->inner_tol = 1e-3;
  o->inner_maxit = 500;
  o->shared_ops = 0;
  o->rows_per_thread = 0;
  o->max_run_steps = 256;
  o->ticks_per_graph = 0;
  o->single_reduction = 1;
  o->schur_variant = 0;
  o->sd_iters = 20;
  o->model = PFC_MODEL_PFC2;
  o->psi_min = -1.5;
  o->grid_columns = 1;
  o->pcg_steps_per_launch = 2;
}

double pfc_tau_critical(double r, double psibar) {
  const double a = 1.0 - 3.0 * r - 9.0 * psibar * psibar;
  if (!(a > 1.0)) return INFINITY;
  const double s = std::sqrt(a);
  return 27.0 / (2.0 * (s - 1.0) * (s + 2.0) * (s + 2.0));
}

size_t pfc_instance_footprint(const pfc_mesh* m, const pfc_opts* o) {
  if (!m || validate_opts(o)) return 0;
  // the S_D layout is part of the mesh; build it (once) to know its size
  if (o->schur_variant == 1 && build_second_ring(const_cast<pfc_mesh*>(m))) return 0;
  InstDev h{};
  const int ts = team_size_for(m->n_slices, o->rows_per_thread);
  return carve(h, nullptr, m, *o, ts);
}

int pfc_instance_create(pfc_mesh* m, const pfc_opts* o, pfc_instance** out) {
  if (!m || !out) { set_error("pfc_instance_create: null argument"); return PFC_ERR_ARG; }
  int rc = validate_opts(o);
  if (rc) return rc;
  *out = nullptr;
  if (o->schur_variant == 1 && (rc = build_second_ring(m))) return rc;
  if (o->model == PFC_MODEL_PFC1 && (!m->dev.elem_K || m->degree != 1)) {
    set_error("pfc_instance_create: the PFC1 model needs a P1 mesh with element geometry (pfc_mesh_create_p1)");
    return PFC_ERR_ARG;
  }
  pfc_instance* I = new pfc_instance();
  I->mesh = m;
  I->opts = *o;
  I->team_size = team_size_for(m->n_slices, o->rows_per_thread);
  I->ticks = o->ticks_per_graph > 0 ? o->ticks_per_graph : 64;
  if (const char* t = std::getenv("PFC_TIMEOUT_S")) I->timeout_s = std::atof(t) > 0 ? std::atof(t) : I->timeout_s;
  if (I->ticks & 1) I->ticks += 1;
  InstDev& h = I->h;
  std::memset(&h, 0, sizeof(h));
  const size_t bytes = carve(h, nullptr, m, *o, I->team_size);
  if (hipMalloc((void**)&I->arena, bytes) != hipSuccess) {
    (void)hipGetLastError();
    delete I;
    set_error("pfc_instance_create: device allocation of " + std::to_string(bytes) + " bytes failed");
    return PFC_ERR_OOM;
  }
  I->bytes = bytes;
  carve(h, I->arena, m, *o, I->team_size);
  h.m = m->dev;  // includes the second-ring layout when it was built
  h.n = m->n;
  h.precision = o->precision;
  h.restart = o->restart;
  h.max_steps = o->max_steps;
  h.inner_maxit = o->inner_maxit;
  h.shared_ops = o->shared_ops;
  h.single_reduction = o->single_reduction;
  h.schur_d = o->schur_variant;
  h.sd_iters = o->sd_iters;
  h.model = o->model;
  h.psi_min = o->psi_min;
  h.grid_cols = o->grid_columns;
  h.gamma_mode = o->gamma_mode;
  for (int k = 0; k < 5; ++k) h.inner_fixed[k] = o->inner_fixed[k];
  h.m0 = 1.0;
  h.team_size = I->team_size;
  I->solo_wgs = h.solo_wgs;
  h.outer_tol = o->outer_tol;
  h.inner_tol = o->inner_tol;
  h.ci_tol = 1e-13;
  if (hipMemset(I->arena, 0, bytes) != hipSuccess || hipStreamCreate(&I->capture) != hipSuccess ||
      hipDeviceSynchronize() != hipSuccess) {
    pfc_instance_destroy(I);
    set_error("pfc_instance_create: HIP setup failed");
    return PFC_ERR_HIP;
  }
  *out = I;
  return PFC_OK;
}

void pfc_instance_destroy(pfc_instance* I) {
  if (!I) return;
  I->grp.release();
  if (I->capture) (void)hipStreamDestroy(I->capture);
  if (I->d_sched) (void)hipFree(I->d_sched);
  if (I->arena) (void)hipFree(I->arena);
  delete I;
}

// One stage solve at psi_k (and mu_k for the PFC1 mobility matrices).
static int solve_impl(pfc_instance* I, const double* psi_k, const double* mu_k, double r, double psibar, double tau,
                      double m11, const double* rhs, double* x, const pfc_schedule* replay, pfc_solve_info* info,
                      void* stream) {
  if (!I || !psi_k || !rhs || !x || !std::isfinite(r) || !std::isfinite(psibar) || !(tau > 0.0) ||
      !std::isfinite(tau) || !(m11 > 0.0) || !std::isfinite(m11)) {
    set_error("pfc_solve: invalid arguments");
    return PFC_ERR_ARG;
  }
  hipStream_t s = (hipStream_t)stream;
  InstDev& h = I->h;
  int rc0 = set_mobility_mean(I, psi_k, s);
  if (rc0) return rc0;
  set_params(h, r, tau, m11);
  h.b_user = rhs;
  h.x_user = x;
  h.replay = 0;
  h.n_steps = 0;
  h.init_mode = PFC_INIT_GIVEN;
  if (replay) {
    int rc = upload_schedules(I, replay, 1, s);
    if (rc) return rc;
  }
  int rc = prep_ops(I, s);
  if (rc) return rc;
  rc = launch_row_N(I->mesh, psi_k, h.N, false, s);
  if (rc) return rc;
  if (h.model == PFC_MODEL_PFC1) hipLaunchKernelGGL(k_assemble_mob, row_grid(I->mesh, 256), dim3(256), 0, s, h, psi_k, mu_k);
  PFC_HIP(hipGetLastError());
  rc = run_single(I, s, JOB_SOLVE);
  h.replay = 0;
  if (rc) return rc;
  InfoDev f;
  PFC_HIP(hipMemcpy(&f, h.info, sizeof(InfoDev), hipMemcpyDeviceToHost));
  I->last_applies = f.inner_applies;
  if (info) fill_info(info, f);
  int st = f.status;
  if (st == PFC_OK && tau >= pfc_tau_critical(r, psibar)) st = PFC_WARN_TAU_CRITICAL;
  return st;
}

int pfc_solve(pfc_instance* I, const double* psi_k, double r, double psibar, double tau, double m11,
              const double* rhs, double* x, const pfc_schedule* replay, pfc_solve_info* info, void* stream) {
  if (I && I->h.model == PFC_MODEL_PFC1) {
    set_error("pfc_solve: a PFC1 instance needs mu_k as well; use pfc_solve_x");
    return PFC_ERR_ARG;
  }
  return solve_impl(I, psi_k, nullptr, r, psibar, tau, m11, rhs, x, replay, info, stream);
}

int pfc_solve_x(pfc_instance* I, const double* x_k, double r, double psibar, double tau, double m11, const double* rhs,
                double* x, const pfc_schedule* replay, pfc_solve_info* info, void* stream) {
  if (!I || !x_k) { set_error("pfc_solve_x: invalid arguments"); return PFC_ERR_ARG; }
  return solve_impl(I, x_k + I->mesh->n, x_k, r, psibar, tau, m11, rhs, x, replay, info, stream);
}

int pfc_instance_launch_stats(const pfc_instance* I, long long* launches, long long* graphs) {
  if (!I) { set_error("pfc_instance_launch_stats: null instance"); return PFC_ERR_ARG; }
  if (graphs) *graphs = I->grp.graphs_run;
  if (launches) *launches = I->grp.launches;
  return PFC_OK;
}

int pfc_instance_config(const pfc_instance* I, int* team_size, int* rows_per_thread, int* pcg_steps_per_launch,
                        int* grid_columns) {
  if (!I) { set_error("pfc_instance_config: null instance"); return PFC_ERR_ARG; }
  if (team_size) *team_size = I->team_size;
  if (rows_per_thread) *rows_per_thread = I->opts.rows_per_thread > 0 ? I->opts.rows_per_thread : 1;
  if (pcg_steps_per_launch) *pcg_steps_per_launch = I->h.sstep ? 2 : 1;
  if (grid_columns) *grid_columns = (I->h.grid_cols && I->mesh->dev.gN > 0 && I->mesh->dev.uw >= 1) ? 1 : 0;
  return PFC_OK;
}

int pfc_last_inner_counts(const pfc_instance* I, int* counts, int cap, int* n_applies) {
  if (!I || !counts || cap < 0 || !n_applies) { set_error("pfc_last_inner_counts: invalid arguments"); return PFC_ERR_ARG; }
  const int na = std::min(I->last_applies, I->opts.max_steps);
  *n_applies = na;
  const int k = std::min(na, cap);
  if (k > 0) PFC_HIP(hipMemcpy(counts, I->h.rec_inner, sizeof(int) * 5 * k, hipMemcpyDeviceToHost));
  return PFC_OK;
}

int pfc_rosenbrock_run(pfc_instance* I, double* state, double r, double psibar, double tau, int n_steps, int init,
                       const pfc_schedule* replays, pfc_solve_info* per_stage, void* stream) {
  if (!I || !state || !std::isfinite(r) || !std::isfinite(psibar) || !(tau > 0.0) || !std::isfinite(tau) ||
      n_steps < 0 || n_steps > I->opts.max_run_steps || (init != PFC_INIT_GIVEN && init != PFC_INIT_CONSISTENT)) {
    set_error("pfc_rosenbrock_run: invalid arguments (n_steps must be <= max_run_steps)");
    return PFC_ERR_ARG;
  }
  hipStream_t s = (hipStream_t)stream;
  InstDev& h = I->h;
  // PFC1: the mobility mean of the initial state (conserved by the scheme)
  int rc = set_mobility_mean(I, state + I->mesh->n, s);
  if (rc) return rc;
  set_params(h, r, tau, 1.0 / ROS_GAMMA);
  double* own_xk = h.xk;
  h.xk = state;
  h.replay = 0;
  if (replays) rc = upload_schedules(I, replays, 3 * n_steps, s);
  if (!rc) rc = prep_ops(I, s);
  if (!rc) {
    h.n_steps = n_steps;
    h.init_mode = init;
    rc = run_single(I, s, JOB_RB);
  }
  h.xk = own_xk;
  h.replay = 0;
  if (rc) return rc;
  std::vector<InfoDev> f((size_t)3 * n_steps);
  if (n_steps > 0) PFC_HIP(hipMemcpy(f.data(), h.info, sizeof(InfoDev) * f.size(), hipMemcpyDeviceToHost));
  State fin;
  PFC_HIP(hipMemcpy(&fin, h.st, sizeof(State), hipMemcpyDeviceToHost));
  int worst = PFC_OK;
  for (size_t k = 0; k < f.size(); ++k) {
    if (per_stage) fill_info(per_stage + k, f[k]);
    if (f[k].status < 0) worst = f[k].status;
    else if (worst >= 0 && f[k].status > worst) worst = f[k].status;
  }
  if (fin.status < 0) worst = fin.status;
  if (worst == PFC_OK && tau >= pfc_tau_critical(r, psibar)) worst = PFC_WARN_TAU_CRITICAL;
  return worst;
}

int pfc_rosenbrock_adaptive(pfc_instance* I, double* state, double r, double psibar, double tau0, double t_end,
                            double rtol, double atol, int max_attempts, int init, double* taus, int* n_accepted,
                            int* n_rejected, pfc_solve_info* infos, void* stream) {
  if (!I || !state || !taus || !n_accepted || !n_rejected || !std::isfinite(r) || !std::isfinite(psibar) ||
      !(tau0 > 0.0) || !(t_end > 0.0) || !std::isfinite(t_end) || !(rtol > 0.0) || !(atol > 0.0) || max_attempts < 1 ||
      (init != PFC_INIT_GIVEN && init != PFC_INIT_CONSISTENT)) {
    set_error("pfc_rosenbrock_adaptive: invalid arguments");
    return PFC_ERR_ARG;
  }
  hipStream_t s = (hipStream_t)stream;
  InstDev& h = I->h;
  const int n = I->mesh->n;
  const int ns = I->mesh->n_slices;
  double* own_xk = h.xk;
  h.xk = state;
  h.replay = 0;
  *n_accepted = 0;
  *n_rejected = 0;
  int rc = set_mobility_mean(I, state + n, s), worst = PFC_OK;
  std::vector<double> part(ns);
  long long graphs = 0, launches = 0;  // launch statistics of the whole call (one run per attempted step)
  if (!rc && init == PFC_INIT_CONSISTENT) {
    set_params(h, r, tau0, 1.0 / ROS_GAMMA);
    h.n_steps = 0;
    h.init_mode = PFC_INIT_CONSISTENT;
    rc = prep_ops(I, s);
    if (!rc) rc = run_single(I, s, JOB_RB);
    graphs += I->grp.graphs_run;
    launches += I->grp.launches;
  }
  double t = 0.0, tau = tau0;
  bool after_reject = false;  // the step after a rejection may not grow
  for (int a = 0; !rc && a < max_attempts && t < t_end * (1.0 - 1e-14); ++a) {
    const double step = std::min(tau, t_end - t);
    if (hipMemcpyAsync(h.xbak, state, sizeof(double) * 3 * (size_t)n, hipMemcpyDeviceToDevice, s) != hipSuccess) { rc = PFC_ERR_HIP; break; }
    set_params(h, r, step, 1.0 / ROS_GAMMA);
    h.n_steps = 1;
    h.init_mode = PFC_INIT_GIVEN;
    rc = prep_ops(I, s);
    if (!rc) rc = run_single(I, s, JOB_RB);
    if (rc) break;
    graphs += I->grp.graphs_run;
    launches += I->grp.launches;
    State fin;
    if (hipMemcpy(&fin, h.st, sizeof(State), hipMemcpyDeviceToHost) != hipSuccess) { rc = PFC_ERR_HIP; break; }
    if (infos) {  // the three stage solves of this attempt, accepted or not
      InfoDev f[3];
      if (hipMemcpy(f, h.info, sizeof(f), hipMemcpyDeviceToHost) != hipSuccess) { rc = PFC_ERR_HIP; break; }
      for (int k = 0; k < 3; ++k) fill_info(infos + 3 * (size_t)a + k, f[k]);
    }
    if (fin.status < 0) { worst = fin.status; break; }
    if (fin.status == PFC_NOT_CONVERGED) {  // a stage solve missed its tolerance: reject, retry with facmin * step
      *n_rejected += 1;
      if (hipMemcpyAsync(state, h.xbak, sizeof(double) * 3 * (size_t)n, hipMemcpyDeviceToDevice, s) != hipSuccess) { rc = PFC_ERR_HIP; break; }
      tau = step * 0.2;
      after_reject = true;
      continue;
    }
    if (fin.status > worst) worst = fin.status;
    hipLaunchKernelGGL(k_embedded_err, dim3(ns), dim3(64), 0, s, h, h.xbak, state, rtol, atol);
    if (hipGetLastError() != hipSuccess || hipMemcpyAsync(part.data(), h.errpart, sizeof(double) * ns, hipMemcpyDeviceToHost, s) != hipSuccess ||
        hipStreamSynchronize(s) != hipSuccess) { rc = PFC_ERR_HIP; break; }
    double sum = 0.0;
    for (int k = 0; k < ns; ++k) sum += part[k];
    const double err = std::sqrt(sum / n);
    if (!std::isfinite(err)) { worst = PFC_ERR_BREAKDOWN; break; }
    const double facmax = (err <= 1.0 && after_reject) ? 1.0 : 5.0;
    if (err <= 1.0) {
      t += step;
      taus[*n_accepted] = step;
      *n_accepted += 1;
      after_reject = false;
      if (*n_accepted >= max_attempts) break;
    } else {
      *n_rejected += 1;
      after_reject = true;
      if (hipMemcpyAsync(state, h.xbak, sizeof(double) * 3 * (size_t)n, hipMemcpyDeviceToDevice, s) != hipSuccess) { rc = PFC_ERR_HIP; break; }
    }
    const double fac = err == 0.0 ? facmax : std::min(facmax, std::max(0.2, 0.9 * std::pow(err, -1.0 / 3.0)));
    tau = step * fac;
  }
  if (!rc && hipStreamSynchronize(s) != hipSuccess) rc = PFC_ERR_HIP;
  I->grp.graphs_run = graphs;
  I->grp.launches = launches;
  h.xk = own_xk;
  if (rc) return rc;
  if (worst < 0) return worst;
  if (t < t_end * (1.0 - 1e-14)) return PFC_NOT_CONVERGED;
  return worst;
}

static int apply_AR_impl(pfc_instance* I, const double* psi_k, const double* mu_k, double r, double tau, double m11,
                         const double* y, double* out, void* stream) {
  if (!I || !psi_k || !y || !out || !std::isfinite(r) || !std::isfinite(tau) || !std::isfinite(m11)) {
    set_error("pfc_apply_AR: invalid arguments");
    return PFC_ERR_ARG;
  }
  hipStream_t s = (hipStream_t)stream;
  InstDev h = I->h;
  h.r = r; h.tau = tau; h.m11 = m11;
  int rc;
  if (h.model == PFC_MODEL_PFC2 && row_AR_applies(I->mesh, psi_k, out)) {
    rc = launch_row_AR(I->mesh, psi_k, r, tau, m11, y, out, s);
  } else {
    rc = launch_row_N(I->mesh, psi_k, h.N, false, s);
    if (!rc && h.model == PFC_MODEL_PFC1)
      hipLaunchKernelGGL(k_assemble_mob, row_grid(I->mesh, 256), dim3(256), 0, s, h, psi_k, mu_k);
    if (!rc) hipLaunchKernelGGL(k_apply_AR, dim3(slice_blocks(I->mesh->n_slices)), dim3(PFC_WG), 0, s, h, y, out);
  }
  if (rc) return rc;
  PFC_HIP(hipGetLastError());
  PFC_HIP(hipStreamSynchronize(s));
  return PFC_OK;
}

int pfc_apply_AR(pfc_instance* I, const double* psi_k, double r, double tau, double m11, const double* y, double* out,
                 void* stream) {
  if (I && I->h.model == PFC_MODEL_PFC1) {
    set_error("pfc_apply_AR: a PFC1 instance needs mu_k as well; use pfc_apply_AR_x");
    return PFC_ERR_ARG;
  }
  return apply_AR_impl(I, psi_k, nullptr, r, tau, m11, y, out, stream);
}

int pfc_apply_AR_x(pfc_instance* I, const double* x_k, double r, double tau, double m11, const double* y, double* out,
                   void* stream) {
  if (!I || !x_k) { set_error("pfc_apply_AR_x: invalid arguments"); return PFC_ERR_ARG; }
  return apply_AR_impl(I, x_k + I->mesh->n, x_k, r, tau, m11, y, out, stream);
}

int pfc_apply_AR_noalloc(const pfc_mesh* m, const double* psi_k, double r, double tau, double m11, const double* y,
                         double* out, void* stream) {
  if (!m || !psi_k || !y || !out || !std::isfinite(r) || !std::isfinite(tau) || !std::isfinite(m11)) {
    set_error("pfc_apply_AR_noalloc: invalid arguments");
    return PFC_ERR_ARG;
  }
  if (m->nnz_sell > PFC_NOALLOC_MAX_ENTRIES) {
    set_error("pfc_apply_AR_noalloc: the mesh stores " + std::to_string(m->nnz_sell) +
              " matrix entries, more than the scratch buffer's " + std::to_string(PFC_NOALLOC_MAX_ENTRIES));
    return PFC_ERR_ARG;
  }
  double* N = nullptr;
  int rc = scratch_address(&N);  // (by whichever call is a device's first: a later one may be captured)
  if (rc) return rc;
  if (row_AR_applies(m, psi_k, out)) return launch_row_AR(m, psi_k, r, tau, m11, y, out, (hipStream_t)stream);
  hipStream_t s = (hipStream_t)stream;
  InstDev h;
  std::memset(&h, 0, sizeof(h));
  h.m = m->dev;
  h.n = m->n;
  h.model = PFC_MODEL_PFC2;
  h.r = r; h.tau = tau; h.m11 = m11;
  h.N = N;
  const int nb = slice_blocks(m->n_slices);
  rc = launch_row_N(m, psi_k, N, false, s);
  if (rc) return rc;
  hipLaunchKernelGGL(k_apply_AR, dim3(nb), dim3(PFC_WG), 0, s, h, y, out);
  PFC_HIP(hipGetLastError());
  return PFC_OK;
}

int pfc_apply_pch(pfc_instance* I, double tau_s, const double* v, double* z, const int* fixed_counts, int* counts_out,
                  void* stream) {
  if (!I || !v || !z || !(tau_s > 0.0) || !std::isfinite(tau_s)) {
    set_error("pfc_apply_pch: invalid arguments");
    return PFC_ERR_ARG;
  }
  hipStream_t s = (hipStream_t)stream;
  InstDev& h = I->h;
  h.m0 = 1.0;  // tau_s is the preconditioner's own time step
  set_params(h, 0.0, tau_s, 1.0);
  h.pch_out = z;
  h.replay = 0;
  int rc = PFC_OK;
  if (fixed_counts) {
    int one = 1;
    pfc_schedule q{1, &one, 1, fixed_counts};
    rc = upload_schedules(I, &q, 1, s);
    if (rc) return rc;
  }
  rc = prep_ops(I, s);
  if (rc) return rc;
  PFC_HIP(hipMemcpyAsync(h.W, v, sizeof(double) * 3 * (size_t)h.n, hipMemcpyDeviceToDevice, s));
  rc = run_single(I, s, JOB_PCH);
  h.replay = 0;
  if (rc) return rc;
  if (counts_out) PFC_HIP(hipMemcpy(counts_out, h.rec_inner, sizeof(int) * 5, hipMemcpyDeviceToHost));
  return PFC_OK;
}

int pfc_stage_rhs(pfc_instance* I, const double* x_k, const double* ys, int stage, double r, double tau, double* b,
                  void* stream) {
  if (!I || !x_k || !ys || !b || stage < 1 || stage > 3 || !std::isfinite(r) || !std::isfinite(tau)) {
    set_error("pfc_stage_rhs: invalid arguments");
    return PFC_ERR_ARG;
  }
  hipStream_t s = (hipStream_t)stream;
  InstDev h = I->h;
  h.r = r; h.tau = tau;
  h.xk = const_cast<double*>(x_k);
  h.ys = const_cast<double*>(ys);
  const int rc = launch_stage_rhs(I->mesh, h, stage, b, s);
  if (rc) return rc;
  PFC_HIP(hipStreamSynchronize(s));
  return PFC_OK;
}

int pfc_batch_run(pfc_instance* const* insts, int count, double* const* states, const double* r, const double* psibar,
                  const double* tau, int n_steps, int init, pfc_solve_info* infos, void* stream) {
  if (!insts || count <= 0 || !states || !r || !psibar || !tau || n_steps < 0 ||
      (init != PFC_INIT_GIVEN && init != PFC_INIT_CONSISTENT)) {
    set_error("pfc_batch_run: invalid arguments");
    return PFC_ERR_ARG;
  }
  const int prec = insts[0] ? insts[0]->opts.precision : -1;
  for (int i = 0; i < count; ++i) {
    if (!insts[i] || !states[i] || insts[i]->opts.precision != prec || n_steps > insts[i]->opts.max_run_steps ||
        !(tau[i] > 0.0) || !std::isfinite(tau[i]) || !std::isfinite(r[i])) {
      set_error("pfc_batch_run: instance " + std::to_string(i) + " invalid (null, mixed precision, or bad parameters)");
      return PFC_ERR_ARG;
    }
  }
  {
    std::vector<const pfc_instance*> sorted(insts, insts + count);
    std::sort(sorted.begin(), sorted.end());
    if (std::adjacent_find(sorted.begin(), sorted.end()) != sorted.end()) {
      set_error("pfc_batch_run: instances must be distinct");
      return PFC_ERR_ARG;
    }
  }
  hipStream_t s = (hipStream_t)stream;
  std::vector<int> ts(count);
  std::vector<State*> sts(count);
  for (int i = 0; i < count; ++i) {
    InstDev& h = insts[i]->h;
    int rcm = set_mobility_mean(insts[i], states[i] + insts[i]->mesh->n, s);
    if (rcm) return rcm;
    set_params(h, r[i], tau[i], 1.0 / ROS_GAMMA);
    h.replay = 0;
    ts[i] = count == 1 ? insts[i]->solo_wgs : insts[i]->team_size;
    sts[i] = h.st;
    int rc = prep_ops(insts[i], s);
    if (rc) return rc;
  }
  int ticks = insts[0]->ticks;
  if (insts[0]->opts.ticks_per_graph == 0) {  // auto: the autotuning table's value for this batch, if any
    const int tt = tuned_ticks(insts[0]->mesh, prec, count);
    if (tt > 0) ticks = tt + (tt & 1);
  }
  int rc = PFC_OK;
  auto one_pass = [&](int precision, int steps, int initm) -> int {
    Group g;
    int e = g.alloc(ts);
    if (!e) {
      for (int i = 0; i < count; ++i) {
        InstDev h = insts[i]->h;
        h.xk = states[i];
        h.job = JOB_RB;
        h.n_steps = steps;
        h.init_mode = initm;
        g.h_descs[i] = h;
        g.h_states[i] = initial_state(JOB_RB);
      }
      e = g.build(insts[0]->capture, precision, ticks);
    }
    if (!e) e = g.run(s, sts, insts[0]->timeout_s * count);
    g.release();
    return e;
  };
  rc = one_pass(prec, n_steps, init);
  if (rc) return rc;
  int worst = PFC_OK;
  std::vector<InfoDev> f((size_t)3 * n_steps);
  for (int i = 0; i < count; ++i) {
    if (n_steps > 0)
      PFC_HIP(hipMemcpy(f.data(), insts[i]->h.info, sizeof(InfoDev) * f.size(), hipMemcpyDeviceToHost));
    for (size_t k = 0; k < f.size(); ++k) {
      if (infos) fill_info(infos + (size_t)i * f.size() + k, f[k]);
      if (f[k].status < 0) worst = f[k].status;
      else if (worst >= 0 && f[k].status > worst) worst = f[k].status;
    }
  }
  return worst;
}

}  // extern "C"
