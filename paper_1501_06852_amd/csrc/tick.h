// The solver kernel: one launch of k_tick advances every active instance by one
// phase (see pfc_internal.h).  A launch first sums the partial reductions that the
// previous launch left behind (every workgroup of a team does this
// redundantly, in fixed order, so all of them take identical decisions), then
// thread 0 of each workgroup applies the transition to a copy of the state in
// LDS, the workgroup executes the work of the new phase, stores its partial
// sums and workgroup 0 of the team writes the new state.  Kernel boundaries
// are the only synchronisation between workgroups: no grid barriers, no
// atomics.  Included by one source per inner precision (tick_f64.hip,
// tick_f32.hip), which compile side by side.
#pragma once
#include <cmath>
#include <cstddef>
#include <type_traits>

#include "device.h"
#include "host.h"
#include "solver.h"

namespace pfc {

__device__ __forceinline__ bool phase_partials(int ph) {
  switch (ph) {
    case PH_SOLVE_INIT: case PH_RB_RHS: case PH_PCG_SETUP: case PH_PCG_A: case PH_PCG_B:
    case PH_GS_UPDATE: case PH_TRUE_RES: case PH_CG_INIT: case PH_CG_ITER:
      return true;
    default:
      return false;
  }
}

__device__ __forceinline__ int solve_index(const State& S) { return S.job == JOB_RB ? S.step * 3 + S.stage - 1 : 0; }

// count slot of an inner solve kind in the per-application record (5 slots)
__device__ __forceinline__ int count_slot(int kind) { return kind == KIND_SD ? KIND_Z : kind; }

__device__ __forceinline__ int inner_limit(const InstDev& I, const State& S, bool& fixed, double& tol) {
  if (is_ci(S.kind)) { fixed = false; tol = I.ci_tol; return 2000; }
  tol = I.inner_tol;
  if (I.replay) {
    fixed = true;
    const int idx = solve_index(S);
    const int* meta = I.sched_meta + 4 * idx;
    if (S.apply >= meta[3]) return 0;
    return I.sched_inner[(long long)(meta[2] + S.apply) * 5 + count_slot(S.kind)];
  }
  if (I.inner_fixed[count_slot(S.kind)] > 0) { fixed = true; return I.inner_fixed[count_slot(S.kind)]; }
  if (S.kind == KIND_SD) { fixed = true; return I.sd_iters; }  // Table inner_solvers: fixed count for S_D
  fixed = false;
  return I.inner_maxit;
}

__device__ void finish_solve(State& S, const InstDev& I, bool wr, int status) {
  if (wr) {
    const int idx = solve_index(S);
    if (idx < I.max_infos) {
      InfoDev& f = I.info[idx];
      f.status = status;
      f.outer_iters = S.total;
      f.cycles = S.cycle;
      f.inner_applies = I.hist->applies;
      f.inner_total = I.hist->inner_total;
      for (int k = 0; k < 5; ++k) f.inner_max[k] = I.hist->inner_max[k];
      f.est_rel_res = S.est;
      f.true_rel_res = S.rel;
      f.t_solve = (double)((long long)wall_clock64() - S.t0) * 1e-8;
    }
  }
  if (status < 0) S.status = status;
  else if (status > S.status && S.status >= 0) S.status = status;
  if (S.job == JOB_RB && status >= 0) {
    if (S.stage < 3) { S.stage += 1; S.phase = PH_RB_RHS; }
    else S.phase = PH_RB_UPDATE;
  } else {
    S.phase = PH_DONE;
  }
}

__device__ void begin_solve(State& S, const InstDev& I, bool wr, Red3 red) {
  S.bnorm = sqrt(red.a);
  S.bnorm_s = sqrt(red.b);
  S.total = 0; S.cycle = 0; S.j = 0; S.apply = 0; S.est = 0.0; S.rel = 0.0;
  if (wr) {
    I.hist->applies = 0;
    I.hist->inner_total = 0;
    for (int k = 0; k < 5; ++k) I.hist->inner_max[k] = 0;
  }
  if (!isfinite(S.bnorm)) { finish_solve(S, I, wr, PFC_ERR_BREAKDOWN); return; }
  if (S.bnorm == 0.0) { finish_solve(S, I, wr, PFC_OK); return; }
  if (I.replay && I.sched_meta[4 * solve_index(S) + 1] == 0) { finish_solve(S, I, wr, PFC_OK); return; }
  S.est_thresh = I.gamma_mode == PFC_GAMMA_LITERAL ? I.outer_tol * S.bnorm : I.outer_tol * S.bnorm / fmax(1.0, I.m11);
  if (wr) I.hist->gpre[0] = S.bnorm_s;
  S.vscale = 1.0 / S.bnorm_s;
  S.kind = KIND_Y0;
  S.phase = PH_PCG_SETUP;
}

__device__ void pcg_done(State& S, const InstDev& I, bool wr) {
  if (!is_ci(S.kind) && wr) {
    const int slot = count_slot(S.kind);
    if (S.apply < I.max_steps) {
      I.rec_inner[S.apply * 5 + slot] = S.it;
      if (S.kind == KIND_SD) I.rec_inner[S.apply * 5 + KIND_X1] = 0;
    }
    I.hist->inner_total += S.it;
    if (S.it > I.hist->inner_max[slot]) I.hist->inner_max[slot] = S.it;
  }
  switch (S.kind) {
    case KIND_Y1:
      S.kind = I.schur_d ? KIND_SD : KIND_Z;
      S.phase = PH_PCG_SETUP;
      break;
    case KIND_SD:
      S.kind = KIND_X2;
      S.phase = PH_PCG_SETUP;
      break;
    case KIND_Y0: case KIND_Z: case KIND_X1:
      S.kind += 1;
      S.phase = PH_PCG_SETUP;
      break;
    case KIND_X2:
      if (wr) I.hist->applies += 1;
      S.apply += 1;
      S.phase = (S.job == JOB_PCH) ? PH_PCH_OUT : PH_ASPMV;
      break;
    case KIND_CI_OMEGA:
      S.kind = KIND_CI_MU;
      S.phase = PH_PCG_SETUP;
      break;
    default:  // KIND_CI_MU: consistent initial values done
      S.step = 0;
      S.phase = (I.n_steps > 0) ? PH_RB_BEGIN : PH_DONE;
      break;
  }
}

__device__ void restart_cycle(State& S, const InstDev& I, bool wr, double beta) {
  if (!(beta > 0.0)) { finish_solve(S, I, wr, PFC_OK); return; }
  if (wr) I.hist->gpre[0] = beta;
  S.j = 0;
  S.vscale = 1.0 / beta;
  S.kind = KIND_Y0;
  S.phase = PH_PCG_SETUP;
}

// Givens rotation of column j, cycle control, back substitution.
__device__ void givens(State& S, const InstDev& I, bool wr, double hn2, double* ybuf, double* col) {
  Hist* H = I.hist;
  const int j = S.j;
  const double hn = sqrt(hn2);
  for (int l = 0; l <= j; ++l) col[l] = H->hcol[l];
  col[j + 1] = hn;
  for (int l = 0; l < j; ++l) {
    const double c = H->cs[l], s = H->sn[l];
    const double t = c * col[l] + s * col[l + 1];
    col[l + 1] = -s * col[l] + c * col[l + 1];
    col[l] = t;
  }
  const double d = hypot(col[j], col[j + 1]);
  double cj = 1.0, sj = 0.0;
  if (d != 0.0) { cj = col[j] / d; sj = col[j + 1] / d; }
  col[j] = d;
  const double gj = H->gpre[j];
  const double gfin = cj * gj;
  const double gnext = -sj * gj;
  if (wr) {
    H->cs[j] = cj; H->sn[j] = sj; H->gfin[j] = gfin; H->gpre[j + 1] = gnext;
    for (int l = 0; l <= j; ++l) H->R[l][j] = col[l];
  }
  S.total += 1;
  S.est = fabs(gnext) / S.bnorm_s;
  const bool breakdown = hn <= 1e-14 * S.w0;
  bool done;
  if (I.replay) {
    const int* meta = I.sched_meta + 4 * solve_index(S);
    done = (j + 1 >= I.sched_cycles[meta[0] + S.cycle]);
  } else {
    done = fabs(gnext) <= S.est_thresh || breakdown || S.total >= I.max_steps || j + 1 == I.restart;
  }
  if (!done) {
    S.vscale = 1.0 / hn;
    S.j = j + 1;
    S.kind = KIND_Y0;
    S.phase = PH_PCG_SETUP;
    return;
  }
  const int k = j + 1;
  for (int l = k - 1; l >= 0; --l) {
    double s = (l == j) ? gfin : H->gfin[l];
    for (int c = l + 1; c < k; ++c) s -= ((c == j) ? col[l] : H->R[l][c]) * ybuf[c];
    ybuf[l] = s / ((l == j) ? col[l] : H->R[l][l]);
  }
  S.kcols = k;
  S.phase = PH_UPDATE_X;
}

// The most frequent transition, a single-reduction PCG iteration that is not
// the last of its solve, kept inline next to the launch prologue (the general
// transition below is out of line and its code is fetched only when needed).
// Same decisions and arithmetic as the PH_CG_ITER case of transition().
__device__ __forceinline__ bool cg_iter_continues(State& S, const InstDev& I, Red3 red) {
  if (S.phase != PH_CG_ITER || I.replay || S.kind == KIND_SD || is_ci(S.kind) || I.inner_fixed[count_slot(S.kind)] > 0)
    return false;
  const int it = S.it + 1;
  const double g = red.a, dl = red.b, rr = red.c;
  const double tol = I.inner_tol;
  if (it >= I.inner_maxit || rr <= tol * tol * S.bb || g == 0.0 || !isfinite(rr)) return false;
  S.it = it;
  S.cur ^= 1;
  const double beta = g / S.rho;
  S.alpha = g / (dl - beta * g / S.alpha);
  S.beta_cg = beta;
  S.rho = g;
  return true;
}

// inner solves that may run two iterations per launch: the five P_CH solves on
// the P1 pattern (not S_D, not the consistent-initial-value mass solves)
__device__ __forceinline__ bool scg_kind(int kind) { return kind >= KIND_Y0 && kind <= KIND_X2; }

// s-step PCG: the next two iterations from the Gram sums g of the basis B = [p,
// Tp, T^2 p, u, Tu] (g[0..14]: B^T D B, g[15..24]: D^2-weighted Gram of B[1..4]),
// with the stopping test of the standard iteration after each of them.  coef
// receives the increment of x and the new p and u as combinations of B;
// S.pcur = 1 marks a launch that only adds the increment (the solve ends there).
__device__ __forceinline__ void scg_transition(State& S, const InstDev& I, bool wr, const double* g, double* coef) {
  if (S.phase == PH_SCG_ITER && S.pcur) { pcg_done(S, I, wr); return; }
  const bool first = (S.phase == PH_PCG_SETUP);  // that launch formed the solve's first basis
  S.phase = PH_SCG_ITER;
  // entries (i <= j) of G = B^T D B and of H = B'^T D^2 B' (basis indices 1..4)
  auto G = [&](int i, int j) { return g[ss_tri(i, j, 5)]; };
  auto Hq = [&](int i, int j) { return g[15 + ss_tri(i - 1, j - 1, 4)]; };
  for (int m = 0; m < 15; ++m) coef[m] = 0.0;
  bool fixed; double tol;
  const int lim = inner_limit(I, S, fixed, tol);
  if (first) {
    S.bb = g[25];
    S.it = 0;
    S.pcur = 0;
    if (S.bb == 0.0 || lim == 0) { pcg_done(S, I, wr); return; }  // x_0 = 0 stands
  }
  // first iteration: alpha_0 = <u,u> / <p,Tp>, u_1 = u - alpha_0 Tp
  const double rho0 = G(3, 3);
  const double a0 = rho0 / G(0, 1);
  const double rho1 = G(3, 3) - 2.0 * a0 * G(1, 3) + a0 * a0 * G(1, 1);
  const double rr1 = Hq(3, 3) - 2.0 * a0 * Hq(1, 3) + a0 * a0 * Hq(1, 1);
  coef[0] = a0;
  S.it += 1;
  S.pcur = 1;
  if (S.it >= lim || (!fixed && rr1 <= tol * tol * S.bb) || rho1 == 0.0 || !isfinite(rr1)) return;
  // second: p_1 = u_1 + beta_0 p = b0 e0 - a0 e1 + e3, T p_1 = b0 e1 - a0 e2 + e4
  const double b0 = rho1 / rho0;
  const double ptp = b0 * (b0 * G(0, 1) - a0 * G(0, 2) + G(0, 4)) - a0 * (b0 * G(1, 1) - a0 * G(1, 2) + G(1, 4)) +
                     (b0 * G(1, 3) - a0 * G(2, 3) + G(3, 4));
  const double a1 = rho1 / ptp;
  // u_2 = u_1 - alpha_1 T p_1 = c1 e1 + c2 e2 + e3 + c4 e4
  const double c1 = -a0 - a1 * b0, c2 = a1 * a0, c4 = -a1;
  auto quad = [&](auto M) {
    return c1 * c1 * M(1, 1) + c2 * c2 * M(2, 2) + M(3, 3) + c4 * c4 * M(4, 4) +
           2.0 * (c1 * c2 * M(1, 2) + c1 * M(1, 3) + c1 * c4 * M(1, 4) + c2 * M(2, 3) + c2 * c4 * M(2, 4) + c4 * M(3, 4));
  };
  const double rho2 = quad(G), rr2 = quad(Hq);
  // x += alpha_0 p + alpha_1 p_1
  coef[0] = a0 + a1 * b0;
  coef[1] = -a1 * a0;
  coef[3] = a1;
  S.it += 1;
  if (S.it >= lim || (!fixed && rr2 <= tol * tol * S.bb) || rho2 == 0.0 || !isfinite(rr2)) return;
  // p_2 = u_2 + beta_1 p_1, u_2
  const double b1 = rho2 / rho1;
  coef[5] = b1 * b0; coef[6] = c1 - b1 * a0; coef[7] = c2; coef[8] = 1.0 + b1; coef[9] = c4;
  coef[11] = c1; coef[12] = c2; coef[13] = 1.0; coef[14] = c4;
  S.pcur = 0;
}

// 2D block form: a solve whose last increment this launch adds (S.pcur) ends
// here if the next P_CH step's set-up reads its x as v (steps (1)-(4) to the
// next one, not into S_D): this launch then also forms that set-up from x plus
// the increment on a three-step frame (S.fuse, the kind ending S.fkind), and
// the next launch stores that x (the increment's coefficients kept in S.xc*).
__device__ __forceinline__ void b2_fuse_end(State& S, const InstDev& I, bool wr, const double* coef) {
  S.fuse = 0;
  if (S.phase != PH_SCG_ITER || !S.pcur) return;
  const int k = S.kind;
  if (!(k == KIND_Y0 || k == KIND_Z || k == KIND_X1 || (k == KIND_Y1 && !I.schur_d))) return;
  pcg_done(S, I, wr);
  S.fuse = 1;
  S.fkind = k;
  S.xc0 = coef[0];
  S.xc1 = coef[1];
  S.xc3 = coef[3];
}

// After w = A_s z_j and its Gram sums g (slots as in ph_aspmv; Ls: the rows of
// L stored by earlier steps of the cycle): h solves (I + L) h = c by forward
// substitution, which is modified Gram-Schmidt's sequence of coefficients.
__device__ void gs_coefficients(State& S, const InstDev& I, bool wr, const double* g, const double* Ls, double* h) {
  const int j = S.j;
  for (int i = 0; i <= j; ++i) {
    double s = g[i];
    for (int k = 0; k < i; ++k) s -= (i == j ? g[32 + k] : Ls[i * PFC_MAXM + k]) * h[k];
    h[i] = s;
  }
  if (wr) {
    for (int k = 0; k < j; ++k) I.hist->L[j][k] = g[32 + k];
    for (int i = 0; i <= j; ++i) I.hist->hcol[i] = h[i];
  }
  S.w0 = sqrt(g[32 + j]);
  S.phase = PH_GS_UPDATE;
}

__device__ void transition(State& S, const InstDev& I, bool wr, Red3 red, double* ybuf, double* col, bool ss) {
  switch (S.phase) {
    case PH_START:
      if (S.job == JOB_SOLVE) S.phase = PH_SOLVE_INIT;
      else if (S.job == JOB_PCH) {
        S.j = 0; S.vscale = 1.0; S.kind = KIND_Y0; S.apply = 0; S.phase = PH_PCG_SETUP;
        if (wr) { I.hist->applies = 0; I.hist->inner_total = 0; for (int k = 0; k < 5; ++k) I.hist->inner_max[k] = 0; }
      } else {  // JOB_RB
        S.step = 0;
        if (I.init_mode == PFC_INIT_CONSISTENT) { S.kind = KIND_CI_OMEGA; S.phase = PH_PCG_SETUP; }
        else S.phase = (I.n_steps > 0) ? PH_RB_BEGIN : PH_DONE;
      }
      break;
    case PH_SOLVE_INIT:
    case PH_RB_RHS:
      begin_solve(S, I, wr, red);
      break;
    case PH_RB_BEGIN:
      S.stage = 1;
      S.phase = PH_RB_RHS;
      break;
    case PH_RB_UPDATE:
      S.step += 1;
      S.phase = (S.step < I.n_steps) ? PH_RB_BEGIN : PH_DONE;
      break;
    case PH_PCG_SETUP: {
      S.rho = red.a; S.bb = red.b; S.it = 0; S.pcur = 0; S.cur = 0; S.beta_cg = 0.0;
      bool fixed; double tol;
      const int lim = inner_limit(I, S, fixed, tol);
      if (S.bb == 0.0 || lim == 0) pcg_done(S, I, wr);
      else if (!I.single_reduction) S.phase = PH_PCG_A;
      else S.phase = PH_CG_INIT;
    } break;
    case PH_CG_INIT:
      S.rho = red.a;             // gamma_0 = (r_0, D^{-1} r_0)
      S.alpha = red.a / red.b;   // gamma_0 / (w_0, u_0)
      S.beta_cg = 0.0;
      S.it = 0;
      S.cur = 0;
      S.phase = PH_CG_ITER;
      break;
    case PH_CG_ITER: {
      S.it += 1;
      S.cur ^= 1;
      bool fixed; double tol;
      const int lim = inner_limit(I, S, fixed, tol);
      const double g = red.a, dl = red.b, rr = red.c;
      const bool done = S.it >= lim || (!fixed && rr <= tol * tol * S.bb) || g == 0.0 || !isfinite(rr);
      if (done) pcg_done(S, I, wr);
      else {
        const double beta = g / S.rho;
        S.alpha = g / (dl - beta * g / S.alpha);
        S.beta_cg = beta;
        S.rho = g;
      }
    } break;
    case PH_PCG_A:
      S.alpha = S.rho / red.a;
      S.pcur ^= 1;
      S.phase = PH_PCG_B;
      break;
    case PH_PCG_B: {
      S.it += 1;
      bool fixed; double tol;
      const int lim = inner_limit(I, S, fixed, tol);
      const double rr = red.a, rzn = red.b;
      const bool done = S.it >= lim || (!fixed && rr <= tol * tol * S.bb) || rzn == 0.0 || !isfinite(rr);
      if (done) pcg_done(S, I, wr);
      else { S.beta_cg = rzn / S.rho; S.rho = rzn; S.phase = PH_PCG_A; }
    } break;
    case PH_GS_UPDATE:
      givens(S, I, wr, red.a, ybuf, col);
      break;
    case PH_UPDATE_X:
      S.phase = PH_TRUE_RES;
      break;
    case PH_TRUE_RES: {
      const double rel = sqrt(red.a) / S.bnorm;
      S.rel = rel;
      S.cycle += 1;
      if (!isfinite(rel)) { finish_solve(S, I, wr, PFC_ERR_BREAKDOWN); break; }
      if (I.replay) {
        const int* meta = I.sched_meta + 4 * solve_index(S);
        if (S.cycle < meta[1]) restart_cycle(S, I, wr, sqrt(red.b));
        else finish_solve(S, I, wr, rel <= I.outer_tol ? PFC_OK : PFC_NOT_CONVERGED);
      } else if (rel <= I.outer_tol) {
        finish_solve(S, I, wr, PFC_OK);
      } else if (S.total >= I.max_steps) {
        finish_solve(S, I, wr, PFC_NOT_CONVERGED);
      } else {
        restart_cycle(S, I, wr, sqrt(red.b));
      }
    } break;
    case PH_PCH_OUT:
      S.phase = PH_DONE;
      break;
    case PH_SCG_ITER:  // a two-iteration solve in a launch without that form: refuse, loudly
      finish_solve(S, I, wr, PFC_ERR_STATE);
      break;
    default:
      S.phase = PH_DONE;
      break;
  }
}

#ifdef PFC_TICK_TIMING
// optional instrumentation (separate build only): wall-clock stamps of one workgroup per launch
static __device__ unsigned long long* g_trace = nullptr;
static __device__ unsigned long long g_trace_n = 0;
static __device__ unsigned long long g_trace_cap = 0;
#define PFC_STAMP(v) unsigned long long v = wall_clock64()
#else
#define PFC_STAMP(v)
#endif

// Inner PCG phase PH of the current solve kind, with one call site per
// distinct instantiation: the float64 solves of the consistent initial values
// (every precision), the S_D solve on its unstaged second-ring pattern, and the
// main path.  (Several call sites of one instantiation make the compiler keep
// it out of line, and the out-of-line call costs a scratch spill of the team
// record on every launch.)
template <typename TT, int L, int PH>
__device__ __forceinline__ Red3 pcg_phase_one(const InstDev& I, const State& S, const Team& tm) {
  if constexpr (PH == PH_PCG_SETUP) return ph_pcg_setup<TT, L>(I, S, tm);
  else if constexpr (PH == PH_PCG_A) return ph_pcg_a<TT, L>(I, S, tm);
  else if constexpr (PH == PH_PCG_B) return ph_pcg_b<TT>(I, S, tm);
  else if constexpr (PH == PH_CG_INIT) return ph_cg_init<TT, L>(I, S, tm);
  else return ph_cg_iter<TT, L>(I, S, tm);
}

template <typename T, int COLS, int PH>
__device__ __forceinline__ Red3 pcg_phase(const InstDev& I, const State& S, const Team& tm, bool sd) {
  constexpr bool uses_pattern = (PH != PH_PCG_SETUP && PH != PH_PCG_B);  // the operator's own SpMV
  if constexpr (!std::is_same<T, double>::value) {
    if (is_ci(__builtin_amdgcn_readfirstlane(S.kind))) return pcg_phase_one<double, COLS, PH>(I, S, tm);
  }
  if constexpr (COLS != PFC_COL_MEM && uses_pattern) {
    if (sd) return pcg_phase_one<T, PFC_COL_MEM, PH>(I, S, tm);
  }
  return pcg_phase_one<T, COLS, PH>(I, S, tm);
}

// One solver launch.  SINGLE: the launch serves one instance and receives its
// state and partial-sum buffers and its mesh pattern as kernel arguments
// (preloaded into scalar registers), so the first memory round trip already
// fetches the state.  Otherwise each workgroup looks up its team entry and
// instance descriptor.  COLS: where the P1 columns come from (PFC_COL_*).
// PFC_COL_LDS stages the workgroup's columns in LDS in the same round trip
// (uniform slice width, at most PFC_WAVES slices per workgroup); PFC_COL_GRID
// computes them from the row (periodic grid meshes).  The host picks the
// variant that the launch's meshes allow.
// SPREAD: a launch that serves one instance and deals its slices to more workgroups
// (wgs) than the instance's team has, fewer to each: a team of 16 slices a
// workgroup leaves most of the chip idle on a small mesh, and the gathers of its 16
// waves queue up in one CU (3D 40^3 float64, 63 workgroups: 15.1 us a launch, the first
// wave's work 4.8).  Phases that leave partial sums then leave one per slice, and the
// next launch adds them up in the team's order (the slices of each of its workgroups,
// then the workgroups): the same bits as the team's own launches.  The sums of the
// orthogonalisation stay the team's.  Measured, P_CH apply 3D 40^3 float64: 1645 ->
// 1110 us; a variant of its own, for in the others the choice at run time cost 2.5%
// (2D 512^2 float64) and 4% (3D 64^3 mixed).
template <typename T, bool SINGLE, int COLS, bool B2, bool SPREAD>
__global__ __launch_bounds__(PFC_WG) void k_tick(const TeamEntry* __restrict__ teams, const InstDev* __restrict__ insts,
                                                 const State* st_in_arg, State* st_out_arg, const double* part_in_arg,
                                                 double* part_out_arg, int parity, const int* __restrict__ col_arg,
                                                 int uw_arg, int nsl_arg, const double* gram_in_arg, int team_arg) {
  __shared__ State S;
  __shared__ State S0;  // entry state of launches that serve many instances (path choice)
  __shared__ InstDev sI;
  __shared__ Red3 lds4[PFC_WAVES];
  __shared__ double ybuf[PFC_MAXM];
  __shared__ double gcol[PFC_MAXM + 1];
  __shared__ double hbuf[PFC_MAXM];          // Gram-Schmidt coefficients of the current Arnoldi step
  __shared__ double gs_g[PFC_GS_NV];         // Gram sums of the step (after PH_ASPMV)
  __shared__ double gs_L[PFC_MAXM * PFC_MAXM];
  // two PCG iterations per launch on periodic grids: blocks of 2D grids (B2,
  // either precision, launches that serve one or many instances), and in
  // launches that serve one instance row ranges of 2D grids in float64 and
  // blocks of 3D grids of side 64 in float
  constexpr bool SB2 = B2 && COLS == PFC_COL_GRID;
  constexpr bool SS = SINGLE && COLS == PFC_COL_GRID && std::is_same<T, double>::value && !B2;
  constexpr bool SS3 = SINGLE && COLS == PFC_COL_GRID && std::is_same<T, float>::value && !B2 && !SPREAD;
  constexpr bool SSX = SS || SS3 || SB2;
  constexpr int NA = SPREAD ? PFC_SS_NA_SPREAD : PFC_SS_NA;
  __shared__ double ss_g[SSX ? 32 : 1];
  __shared__ double ss_coef[SSX ? 16 : 1];
  PFC_STAMP(t_entry);
  const int tid = threadIdx.x;
  TeamEntry te;
  const InstDev* gI;
  const State* st_in;
  State* st_out;
  const double* part_in;
  double* part_out;
  if (SINGLE) {
    te.inst = 0; te.rank = xcd_rank(blockIdx.x, gridDim.x); te.size = SPREAD ? team_arg : (int)gridDim.x;
    te.uw = uw_arg; te.col = col_arg; te.n_slices = nsl_arg; te.pad = 0;
    gI = insts;
    st_in = st_in_arg; st_out = st_out_arg; part_in = part_in_arg; part_out = part_out_arg;
  } else {
    te = teams[xcd_rank(blockIdx.x, gridDim.x)];
    gI = insts + te.inst;
    st_in = gI->st + parity; st_out = gI->st + (1 - parity);
    part_in = gI->part + (long long)parity * te.size * 4;
    part_out = gI->part + (long long)(1 - parity) * te.size * 4;
  }
  static_assert(!SPREAD || (SINGLE && !B2 && COLS != PFC_COL_LDS), "spread launches serve one instance, no blocks");
  const int wgs = SPREAD ? (int)gridDim.x : te.size;
  const int ssz = SS ? wgs : te.size;  // workgroups of the two-iteration form
  // one round trip: the state record and the instance descriptor (a word per
  // thread, every thread loading at a clamped position), the partial sums of
  // the previous launch and, in single-instance launches of two-iteration
  // solves, the previous launch's Gram partials (gram_in_arg; a launch that
  // runs another phase leaves them unused).  Every load is issued before the
  // first of them is waited for.
  constexpr int NS = (int)(sizeof(State) / 4), ND = (int)(sizeof(InstDev) / 4);
  static_assert(NS <= 64 && ND <= PFC_WG - 64, "state / descriptor too large for the staging threads");
  const int word = tid < 64 ? ((const int*)st_in)[min(tid, NS - 1)] : ((const int*)gI)[min(tid - 64, ND - 1)];
  // the fields that choose a workgroup's path before the transition: thread 0
  // rewrites S in the transition while the other waves may still be reading
  // them, so they come from the state record itself (one instance per launch),
  // or from S0, an LDS copy of the entry state that nothing rewrites
  int ph_in = 0, kind_in = 0, pcur_in = 0, fuse_in = 0;
  if constexpr (SINGLE) {
    ph_in = st_in->phase;
    kind_in = st_in->kind;
    pcur_in = st_in->pcur;
    if constexpr (SB2) fuse_in = st_in->fuse;
  }
  double gpl[SSX ? PFC_SS_GL : 1];
  if constexpr (SSX && SINGLE) {
    if (!SPREAD || gram_in_arg) ss_gram_prefetch(gram_in_arg, part_in, ssz, gpl);
  }
  // columns of this workgroup's slices: positions [lo, lo + len) of the SELL
  // pattern, issued first and written to LDS once everything has arrived
  int lo = 0, len = 0;
  int cv[PFC_LCOL_W];
  if (COLS == PFC_COL_LDS) {
    const int spw = (te.n_slices + te.size - 1) / te.size;
    const int sbeg = te.rank * spw;
    const int send = min(sbeg + spw, te.n_slices);
    lo = sbeg * 64 * te.uw;
    len = max(send - sbeg, 0) * 64 * te.uw;
#pragma unroll
    for (int q = 0; q < PFC_LCOL_W; ++q) {
      const int idx = tid + q * PFC_WG;
      if (idx < len) cv[q] = te.col[lo + idx];
    }
  }
  Red3 pre = red3(0.0, 0.0, 0.0), pre2 = red3(0.0, 0.0, 0.0);
  if constexpr (SPREAD) {
    if (tid < te.n_slices) { pre.a = part_in[4 * tid]; pre.b = part_in[4 * tid + 1]; pre.c = part_in[4 * tid + 2]; }
    if (tid + PFC_WG < te.n_slices) {
      const double* q = part_in + 4 * (tid + PFC_WG);
      pre2.a = q[0]; pre2.b = q[1]; pre2.c = q[2];
    }
  } else {
    if (tid < te.size) { pre.a = part_in[4 * tid]; pre.b = part_in[4 * tid + 1]; pre.c = part_in[4 * tid + 2]; }
    for (int k = tid + PFC_WG; k < te.size; k += PFC_WG) {  // teams of more than PFC_WG workgroups
      pre2.a += part_in[4 * k]; pre2.b += part_in[4 * k + 1]; pre2.c += part_in[4 * k + 2];
    }
  }
  if (tid < NS) {
    ((int*)&S)[tid] = word;
    if constexpr (!SINGLE) ((int*)&S0)[tid] = word;
  } else if (tid >= 64 && tid < 64 + ND) {
    ((int*)&sI)[tid - 64] = word;
  }
  if (COLS == PFC_COL_LDS) {
#pragma unroll
    for (int q = 0; q < PFC_LCOL_W; ++q) {
      const int idx = tid + q * PFC_WG;
      if (idx < len) pfc_lcol[idx] = cv[q];
    }
  }
  // their sums over the waves, where the previous launch left any: two-iteration
  // launches leave Gram partials instead.  Launches that serve many instances and
  // have that form know their phase only after the barrier below, and sum there.
  constexpr bool LATE = !SINGLE && SB2;
  auto sum_partials = [&]() {
    pre.a = wave_sum(pre.a + pre2.a);
    pre.b = wave_sum(pre.b + pre2.b);
    pre.c = wave_sum(pre.c + pre2.c);
    if ((tid & 63) == 0) lds4[tid >> 6] = pre;
  };
  if constexpr (!LATE) {
    if (!SINGLE || phase_partials(ph_in)) {
      if constexpr (SPREAD) {
        constexpr int PL = PFC_SPREAD + PFC_SPREAD / 16;
        static_assert(3 * PL <= PFC_SS_LDS && PFC_SPREAD == 2 * PFC_WG, "slice sums in the s-step LDS, two per thread");
        double *sa = pfc_ss, *sb = sa + PL, *sc = sb + PL;  // by slice
        // (a place left free after every 16: the sums read at a stride of 16, all from two
        // banks without it; prologue of 3D 40^3 4.0 -> 2.3 us)
        auto at = [](int sl) { return sl + (sl >> 4); };
        sa[at(tid)] = pre.a; sb[at(tid)] = pre.b; sc[at(tid)] = pre.c;
        sa[at(PFC_WG + tid)] = pre2.a; sb[at(PFC_WG + tid)] = pre2.b; sc[at(PFC_WG + tid)] = pre2.c;
        __syncthreads();
        pre = pre2 = red3(0.0, 0.0, 0.0);
        if (tid < te.size) {  // workgroup tid of the team: its slices (PFC_SLICES), one per wave
          const bool rr = te.uw == 0;
          const int spw = (te.n_slices + te.size - 1) / te.size, first = rr ? tid : tid * spw;
          const int step = rr ? te.size : 1, end = rr ? te.n_slices : min(first + spw, te.n_slices);
#pragma unroll
          for (int w = 0; w < PFC_WAVES; ++w) {
            const int sl = first + w * step;
            if (sl < end) { pre.a += sa[at(sl)]; pre.b += sb[at(sl)]; pre.c += sc[at(sl)]; }
          }
        }
      }
      sum_partials();
    }
  }
  __syncthreads();
#ifdef PFC_TICK_TIMING
  const unsigned long long t_ld = wall_clock64();
  unsigned long long t_red = 0;
#endif
  if constexpr (!SINGLE) {
    ph_in = __builtin_amdgcn_readfirstlane(S0.phase);
    kind_in = __builtin_amdgcn_readfirstlane(S0.kind);
    pcur_in = __builtin_amdgcn_readfirstlane(S0.pcur);
    if constexpr (SB2) fuse_in = __builtin_amdgcn_readfirstlane(S0.fuse);
    if constexpr (LATE) {
      if (phase_partials(ph_in)) {
        sum_partials();
        __syncthreads();
      }
    }
  }
  const InstDev& I = sI;
  const bool writer = (te.rank == 0);
  if (__builtin_expect(ph_in == PH_DONE, 0)) {
    if (writer && tid < NS) ((int*)st_out)[tid] = ((const int*)&S)[tid];
    return;
  }
  // Gram partials of an orthogonalisation (the previous launch formed w = A_s z_j)
  if (__builtin_expect(ph_in == PH_ASPMV, 0))
    gs_gather(I.gpart + (long long)parity * te.size * PFC_GS_NV, te.size, &I.hist->L[0][0], gs_g, gs_L);
  bool scg = false, form = false;
  SsPre<NA> ssp;
  S3Pre<float> s3p;
  B2Pre<T> b2p;
  if constexpr (SSX) {
    // launches after a two-iteration launch, or after the set-up that formed the first basis,
    // of an instance whose two-iteration form is this launch's (a launch that serves many
    // instances may hold instances of either form: the others run one iteration per launch)
    form = __builtin_amdgcn_readfirstlane(I.sstep) == (SB2 ? 3 : (SS ? 1 : 2));
    scg = form && (ph_in == PH_SCG_ITER || (ph_in == PH_PCG_SETUP && scg_kind(kind_in)));
  }
  // (one branch from the loads to the end of the transition: values loaded here would
  // otherwise have to survive the call of the general transition)
  if (SSX && __builtin_expect(scg, 1)) {
    if constexpr (SSX) {
      if (!(ph_in == PH_SCG_ITER && pcur_in)) {
        // the previous launch's Gram partials: loaded in the prologue where the
        // launch serves one instance, else here from the instance's buffer
        const double* gin = SINGLE ? gram_in_arg : I.spart + (long long)parity * te.size * 32;
        if constexpr (!SINGLE) ss_gram_prefetch(gin, gin, te.size, gpl);
        // in flight during the reduction and the transition
        if constexpr (SB2) b2_load<T>(I, te.rank, b2p, parity);
        else if constexpr (SS) ss_load(I, S, ss_rows(I, te.rank, ssz), ssp, parity);
        else s3_load<float>(I, S, te.rank, s3p, parity);
        ss_gram(gin, ssz, gpl, ss_g);
#ifdef PFC_TICK_TIMING
        if (tid == 0) pfc_sst[4] = wall_clock64();
#endif
      }
      if (tid == 0) {
        scg_transition(S, I, writer, ss_g, ss_coef);
        if constexpr (SB2) b2_fuse_end(S, I, writer, ss_coef);
#ifdef PFC_TICK_TIMING
        pfc_sst[5] = wall_clock64();
#endif
      }
      lds_barrier();  // the basis loads stay in flight
    }
  } else {
    if (tid == 0) {
      S.fuse = 0;
      Red3 red = red3(0.0, 0.0, 0.0);
      if (phase_partials(S.phase)) {
#pragma unroll
        for (int w = 0; w < PFC_WAVES; ++w) { red.a += lds4[w].a; red.b += lds4[w].b; red.c += lds4[w].c; }
      }
      if (S.phase == PH_ASPMV) gs_coefficients(S, I, writer, gs_g, gs_L, hbuf);
      else if (!cg_iter_continues(S, I, red)) transition(S, I, writer, red, ybuf, gcol, SS && I.sstep);
      if (S.phase == PH_SOLVE_INIT || S.phase == PH_RB_RHS) S.t0 = (long long)wall_clock64();  // a solve starts
    }
    __syncthreads();
  }
  PFC_STAMP(t_trans);
  // the new state is final: workgroup 0 stores it while the phase runs (and counts the
  // launch there, off the transition's scalar chain)
  if (writer && tid < NS)
    ((int*)st_out)[tid] = ((const int*)&S)[tid] + (tid == (int)(offsetof(State, launches) / 4) ? 1 : 0);
  Team tm{te.rank, wgs, tid >> 6, tid & 63, lo};
  if constexpr (SB2) {
    // the previous launch ended a solve in its set-up: that solve's x on the own rows
    if (__builtin_expect(fuse_in != 0, 0)) {
      const State& Se = SINGLE ? *st_in : S0;
      b2_end_store<T>(I, te.rank, Se.fkind, Se.xc0, Se.xc1, Se.xc3, parity);
    }
  }
  // (scalars: the compiler then branches by phase instead of running through the
  // phases under masks, with what a later phase needs held in registers)
  const int phase = __builtin_amdgcn_readfirstlane(S.phase), kind = __builtin_amdgcn_readfirstlane(S.kind);
  const bool sd = (kind == KIND_SD);  // second-ring pattern, never staged
  const bool mob = __builtin_amdgcn_readfirstlane(I.model) == PFC_MODEL_PFC1;
  Red3 acc = red3(0.0, 0.0, 0.0);
  bool fused = false;  // a set-up launch that formed a two-iteration solve's first basis (Gram partials only)
  bool scg_done = false;
  if constexpr (SSX) {
    if (__builtin_expect(phase == PH_SCG_ITER, 1)) {  // the common launch, laid out first
      double* gout = I.spart + (long long)(1 - parity) * ssz * 32;
      if constexpr (SB2) ph_scg2b<T>(I, S, tm, ss_coef, false, gout, b2p, parity);
      else if constexpr (SS) ph_scg<COLS, NA>(I, S, tm, ss_coef, false, gout, ss_rows(I, te.rank, ssz), ssp, parity);
      else ph_scg3<float>(I, S, tm, ss_coef, false, gout, s3p, parity);
      scg_done = true;
    }
  }
  if (!scg_done) switch (phase) {
    case PH_SOLVE_INIT:
    case PH_RB_RHS: acc = ph_solve_init<COLS>(I, S, tm); break;
    case PH_RB_BEGIN: acc = ph_rb_begin<COLS>(I, tm); break;
    case PH_RB_UPDATE: acc = ph_rb_update(I, tm); break;
    // the mass solves of the consistent initial values run in float64 in every precision
    case PH_PCG_SETUP:
      if constexpr (SSX) {
        if (form && scg_kind(kind)) {  // set-up and first basis of a two-iteration solve
          fused = true;
          double* gout = I.spart + (long long)(1 - parity) * ssz * 32;
          if constexpr (SB2) ph_scg2b<T>(I, S, tm, ss_coef, true, gout, b2p, parity);
          else if constexpr (SS) ph_scg<COLS, NA>(I, S, tm, ss_coef, true, gout, ss_rows(I, te.rank, ssz), ssp, parity);
          else ph_scg3<float>(I, S, tm, ss_coef, true, gout, s3p, parity);
          break;
        }
      }
      acc = pcg_phase<T, COLS, PH_PCG_SETUP>(I, S, tm, sd);
      break;
    case PH_PCG_A: acc = pcg_phase<T, COLS, PH_PCG_A>(I, S, tm, sd); break;
    case PH_PCG_B: acc = pcg_phase<T, COLS, PH_PCG_B>(I, S, tm, sd); break;
    case PH_ASPMV: {
      if constexpr (SPREAD) {  // the team's sums: its workgroups, its slices
        if (te.rank >= te.size) break;
        tm.size = te.size;
      }
      double* gout = I.gpart + (long long)(1 - parity) * te.size * PFC_GS_NV;
      if (mob) ph_aspmv<T, COLS, true>(I, S, tm, gout);
      else ph_aspmv<T, COLS, false>(I, S, tm, gout);
    } break;
    case PH_GS_UPDATE: acc = ph_gs_update(I, S, tm, hbuf); break;
    case PH_UPDATE_X: acc = ph_update_x(I, S, tm, ybuf); break;
    case PH_TRUE_RES:
      acc = mob ? ph_true_res<COLS, true>(I, S, tm) : ph_true_res<COLS, false>(I, S, tm);
      break;
    case PH_PCH_OUT: acc = ph_pch_out<T>(I, tm); break;
    case PH_CG_INIT: acc = pcg_phase<T, COLS, PH_CG_INIT>(I, S, tm, sd); break;
    case PH_CG_ITER: acc = pcg_phase<T, COLS, PH_CG_ITER>(I, S, tm, sd); break;
    default: break;  // PH_SCG_ITER above
  }
  PFC_STAMP(t_work);
  if (phase_partials(phase) && !fused) {
    acc.a = wave_sum(acc.a);
    acc.b = wave_sum(acc.b);
    acc.c = wave_sum(acc.c);
    if constexpr (SPREAD) {  // the slice's own sums (a wave has one slice at most)
      const int wave = tid >> 6, spw = (te.n_slices + wgs - 1) / wgs;
      const int sl = te.uw == 0 ? te.rank + wgs * wave : (wave < spw ? te.rank * spw + wave : te.n_slices);
      if ((tid & 63) == 0 && sl < te.n_slices) {
        double* dst = part_out + 4LL * sl;
        vst(dst, acc.a); vst(dst + 1, acc.b); vst(dst + 2, acc.c);
      }
    } else {
      if ((tid & 63) == 0) lds4[tid >> 6] = acc;
      __syncthreads();
#ifdef PFC_TICK_TIMING
      t_red = wall_clock64();
#endif
      if (tid == 0) {
        Red3 r = red3(0.0, 0.0, 0.0);
#pragma unroll
        for (int w = 0; w < PFC_WAVES; ++w) { r.a += lds4[w].a; r.b += lds4[w].b; r.c += lds4[w].c; }
        double* dst = part_out + (long long)te.rank * 4;
        dst[0] = r.a; dst[1] = r.b; dst[2] = r.c;
      }
    }
  }
#ifdef PFC_TICK_TIMING
  __syncthreads();
  PFC_STAMP(t_exit);
  if (tid == 0 && (te.rank == 0 || te.rank == wgs - 1) && g_trace) {
    const unsigned long long k = atomicAdd(&g_trace_n, 1ULL);
    if (k < g_trace_cap) {
      unsigned long long* r = g_trace + 14 * k;
      r[0] = (unsigned long long)S.phase | ((unsigned long long)te.rank << 8) | ((unsigned long long)S.kind << 40) |
             ((unsigned long long)(S.it & 0xffff) << 48);
      r[1] = t_entry; r[2] = t_ld; r[3] = t_trans; r[4] = t_work; r[5] = t_exit; r[6] = blockIdx.x; r[7] = t_red;
      for (int q = 0; q < 6; ++q) r[8 + q] = (SSX && (fused || S.phase == PH_SCG_ITER)) ? pfc_sst[q] : 0;
    }
  }
#endif
}

// Enqueues one launch on `stream`: the instantiation that the launch allows.
template <typename T>
static void launch_tick_T(const TickLaunch& q, hipStream_t stream) {
#define PFC_TICK(SG, LD, BB, SP)                                                                                       \
  hipLaunchKernelGGL((k_tick<T, SG, LD, BB, SP>), dim3(q.n_wg), dim3(PFC_WG), 0, stream, q.teams, q.insts, q.st_in,     \
                     q.st_out, q.part_in, q.part_out, q.parity, q.col, q.uw, q.n_slices, q.gram_in, q.team)
#define PFC_TICK_COLS(SG)                                                      \
  switch (q.cols) {                                                            \
    case PFC_COL_GRID:                                                         \
      if (q.b2) { PFC_TICK(SG, PFC_COL_GRID, true, false); }                   \
      else { PFC_TICK(SG, PFC_COL_GRID, false, false); }                       \
      break;                                                                   \
    case PFC_COL_LDS: PFC_TICK(SG, PFC_COL_LDS, false, false); break;          \
    default: PFC_TICK(SG, PFC_COL_MEM, false, false); break;                   \
  }
  if (q.single && q.n_wg != q.team) {
    if (q.cols == PFC_COL_GRID) { PFC_TICK(true, PFC_COL_GRID, false, true); }
    else { PFC_TICK(true, PFC_COL_MEM, false, true); }
  } else if (q.single) { PFC_TICK_COLS(true); } else { PFC_TICK_COLS(false); }
#undef PFC_TICK_COLS
#undef PFC_TICK
}

#ifdef PFC_TICK_TIMING
static int tick_trace_set(unsigned long long* dev_buf, unsigned long long cap) {
  unsigned long long z = 0;
  if (hipMemcpyToSymbol(HIP_SYMBOL(g_trace), &dev_buf, sizeof(dev_buf)) != hipSuccess) return -3;
  if (hipMemcpyToSymbol(HIP_SYMBOL(g_trace_cap), &cap, sizeof(cap)) != hipSuccess) return -3;
  if (hipMemcpyToSymbol(HIP_SYMBOL(g_trace_n), &z, sizeof(z)) != hipSuccess) return -3;
  return 0;
}
static unsigned long long tick_trace_count() {
  unsigned long long n = 0;
  (void)hipMemcpyFromSymbol(&n, HIP_SYMBOL(g_trace_n), sizeof(n));
  return n;
}
#define PFC_TICK_TRACE(SUF)                                                                                             \
  int tick_trace_set_##SUF(unsigned long long* b, unsigned long long cap) { return tick_trace_set(b, cap); }            \
  unsigned long long tick_trace_count_##SUF() { return tick_trace_count(); }
#else
#define PFC_TICK_TRACE(SUF)
#endif

}  // namespace pfc
