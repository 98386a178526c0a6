// Device functions of the PFC stage solver: the work of every solver phase,
// executed by one team of workgroups over its block of SELL-64 slices.
//
// Each thread owns row i = slice*64 + lane of the node numbering and, in the
// 3x3 block phases, the three entries i, n+i, 2n+i of a block vector.  Dot
// products are accumulated per thread in float64, reduced per wavefront by a
// fixed butterfly (lane 0's result is used), then per workgroup in fixed
// order, and stored as one partial per workgroup; the next launch sums the
// partials in fixed order.  Results are therefore bitwise reproducible and
// independent of what else runs in the same launch.
#pragma once
#include <type_traits>

#include "pfc_internal.h"

namespace pfc {

struct Team {
  int rank, size;   // workgroup rank within the team, team size
  int wave, lane;   // wave within the workgroup, lane
  int lo;           // SELL position of the first staged column (pfc_lcol[0])
};

// Column indices of the P1 pattern for the workgroup's own slices, staged in
// LDS by the launch prologue when every slice of the mesh has the same width
// (at most PFC_LCOL_W) and a workgroup owns at most PFC_WAVES slices.  They are
// loaded in the same memory round trip as the solver state, which takes the
// index load off the critical path of every SpMV in the launch.
#define PFC_LCOL_W 16
#define PFC_LCOL (PFC_WAVES * 64 * PFC_LCOL_W)
__shared__ int pfc_lcol[PFC_LCOL];

// Frames of the two-iterations-per-launch phases, and the row sums of the
// reassembly of N (8 per thread).
#define PFC_SS_LDS 8192
__shared__ double pfc_ss[PFC_SS_LDS];

// Where a launch takes the columns of the P1 pattern from: memory, the LDS
// staging buffer, or computed from the row (periodic grid meshes, grid_col).
#define PFC_COL_MEM 0
#define PFC_COL_LDS 1
#define PFC_COL_GRID 2

// Slice geometry and columns of a SELL pattern.  L: one of PFC_COL_*; the
// staged and computed forms need a uniform slice width uw.
template <int L>
struct PatView {
  const int* sp;    // slice offsets [n_slices + 1]
  const int* col;   // columns [nnz_sell]
  int uw;           // uniform slice width, or 0
  int lo;           // SELL position of pfc_lcol[0] (L == PFC_COL_LDS)
  int n, gN;        // grid columns (L == PFC_COL_GRID): grid_col with
  float gInv;       //   1/N and the offset table gd
  const int* gd;
  __device__ __forceinline__ int base(int sl) const {
    if constexpr (L != PFC_COL_MEM) return sl * 64 * uw;
    else return uw ? sl * 64 * uw : sp[sl];
  }
  __device__ __forceinline__ int width(int sl) const {
    if constexpr (L != PFC_COL_MEM) return uw;
    else return uw ? uw : ((sp[sl + 1] - sp[sl]) >> 6);
  }
  // column of stored entry e, which belongs to row i (entry e - base(sl) of
  // slice sl = i / 64 sits at position k = (e >> 6) - sl uw of its row)
  __device__ __forceinline__ int at(long long e, int i) const {
    if constexpr (L == PFC_COL_GRID) return grid_col(i, (int)(e >> 6) - (i >> 6) * uw, n, gN, gInv, gd);
    else if constexpr (L == PFC_COL_LDS) return pfc_lcol[(int)(e - lo)];
    else return col[e];
  }
};

template <int L>
__device__ __forceinline__ PatView<L> p1_pat(const InstDev& I, const Team& tm) {
  return PatView<L>{I.m.slice_ptr, I.m.col, I.m.uw, tm.lo, I.n, I.m.gN, I.m.gInv,
                    L == PFC_COL_GRID ? I.m.glin : nullptr};
}

// Cross-lane moves of a double through DPP (register to register, no LDS).
template <int CTRL, int ROWS>
__device__ __forceinline__ double dpp_f64(double v) {
  const long long b = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_update_dpp(0, (int)b, CTRL, ROWS, 0xf, false);
  const int hi = __builtin_amdgcn_update_dpp(0, (int)(b >> 32), CTRL, ROWS, 0xf, false);
  return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}
// Halving exchange between the lanes of a pair: the lane that keeps the lower
// half gets a + (partner's a), the other b + (partner's b).  Partners: lanes
// l and l ^ 32 (permlane32 swap), rows 2k and 2k + 1 (permlane16 swap), or the
// DPP pairs of CTRL within a row.  A swap of (a, b) leaves the lower lanes with
// their a and the partner's a, the upper lanes with the partner's b and their b:
// the sum of its two results is the wanted one in every lane.
__device__ __forceinline__ double ss_pair(unsigned hi, unsigned lo) {
  return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}
template <bool ROWS16>
__device__ __forceinline__ double ss_swap(double a, double b) {
  const unsigned long long ia = (unsigned long long)__double_as_longlong(a), ib = (unsigned long long)__double_as_longlong(b);
  if constexpr (ROWS16) {
    const auto l = __builtin_amdgcn_permlane16_swap((unsigned)ia, (unsigned)ib, false, false);
    const auto h = __builtin_amdgcn_permlane16_swap((unsigned)(ia >> 32), (unsigned)(ib >> 32), false, false);
    return ss_pair(h[0], l[0]) + ss_pair(h[1], l[1]);
  } else {
    const auto l = __builtin_amdgcn_permlane32_swap((unsigned)ia, (unsigned)ib, false, false);
    const auto h = __builtin_amdgcn_permlane32_swap((unsigned)(ia >> 32), (unsigned)(ib >> 32), false, false);
    return ss_pair(h[0], l[0]) + ss_pair(h[1], l[1]);
  }
}
// Sum over the wave, in every lane: the butterfly over lane distances 32, 16, 8,
// 4, 2, 1 without LDS (within a row of 16 a rotation by 8 or 4 meets the lane at
// that distance, or one that holds the same partial sum).
__device__ __forceinline__ double wave_sum(double v) {
  v = ss_swap<false>(v, v);
  v = ss_swap<true>(v, v);
  v += dpp_f64<0x128, 0xf>(v);  // row_ror:8
  v += dpp_f64<0x124, 0xf>(v);  // row_ror:4
  v += dpp_f64<0x4e, 0xf>(v);   // quad_perm [2,3,0,1]
  return v + dpp_f64<0xb1, 0xf>(v);  // quad_perm [1,0,3,2]
}

struct Red3 {
  double a, b, c;
};
__device__ __forceinline__ Red3 red3(double a, double b, double c = 0.0) { return Red3{a, b, c}; }

// Sum (a, b, c) over the workgroup; result valid in thread 0.
__device__ __forceinline__ Red3 wg_sum3(Red3 v, Red3* lds4) {
  v.a = wave_sum(v.a);
  v.b = wave_sum(v.b);
  v.c = wave_sum(v.c);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  if (lane == 0) lds4[wave] = v;
  __syncthreads();
  Red3 r = red3(0.0, 0.0, 0.0);
  if (threadIdx.x == 0) {
#pragma unroll
    for (int w = 0; w < PFC_WAVES; ++w) { r.a += lds4[w].a; r.b += lds4[w].b; r.c += lds4[w].c; }
  }
  __syncthreads();
  return r;
}

// Slices handled by this workgroup, cycled over its waves: a contiguous block
// where every slice of the mesh has the same width; where widths differ (P2
// meshes: vertex rows have 19 entries, edge rows 9, numbered in that order) the
// team's slices are dealt round robin (slice rank + size j), so that every
// workgroup, and every SIMD of it, gets its share of the wide slices.
#define PFC_SLICES(I, tm)                                                          \
  const bool _rr = (I).m.uw == 0;                                                  \
  const int _spw = ((I).m.n_slices + (tm).size - 1) / (tm).size;                   \
  const int _sbeg = _rr ? (tm).rank : (tm).rank * _spw;                            \
  const int _send = _rr ? (I).m.n_slices : min(_sbeg + _spw, (I).m.n_slices);      \
  const int _sstep = _rr ? (tm).size * PFC_WAVES : PFC_WAVES;                      \
  for (int sl = __builtin_amdgcn_readfirstlane(_sbeg + (_rr ? (tm).size * (tm).wave : (tm).wave)); sl < _send; sl += _sstep)

// Row loops over the entries of a slice: the P1 meshes of this solver have 7
// (2D) or 15 (3D) entries per row, 2D P2 meshes 19 (vertex rows) or 9 (edge
// rows); for those widths the loop is unrolled (fully for 7, in chunks of 5 for
// 15 and of 3 for the P2 widths, to stay within the register budget) so that a
// wave issues the index, value and gather loads of many entries at once.
template <typename F>
__device__ __forceinline__ void for_width(int w, F f) {
  if (w == 7) {
#pragma unroll
    for (int k = 0; k < 7; ++k) f(k);
  } else if (w == 15) {
#pragma unroll 5
    for (int k = 0; k < 15; ++k) f(k);
  } else if (w == 9) {  // P2 edge rows (2D)
#pragma unroll 3
    for (int k = 0; k < 9; ++k) f(k);
  } else if (w == 19) {  // P2 vertex rows (2D)
#pragma unroll 3
    for (int k = 0; k < 19; ++k) f(k);
  } else {
    for (int k = 0; k < w; ++k) f(k);
  }
}

// Stores of phase outputs.  PFC_STORE_POLICY selects the cache policy:
// 0 plain (write-back L2), 1 agent-coherent write-through (sc1), 2 streaming (nt).
// Write-through is the default: every phase output is read by other XCDs in
// the next launch, and writing it through during the kernel shortens the
// cache write-back at the kernel boundary.
#ifndef PFC_STORE_POLICY
#define PFC_STORE_POLICY 1
#endif

// Every phase output and every operand lives in device memory (never LDS).  The
// solver's pointers come from the instance record in LDS, so the compiler cannot
// see that and issues flat accesses, which count against the LDS wait counter as
// well and complete in no guaranteed order: every wait for an LDS access then
// also waits for all memory accesses in flight.  Stores, and the loads of the
// phases that issue loads ahead of their use, therefore name the global address
// space explicitly.
template <typename T>
__device__ __forceinline__ __attribute__((address_space(1))) T* gp(T* p) {
  return (__attribute__((address_space(1))) T*)p;
}
template <typename T>
__device__ __forceinline__ T gld(const T* p) {
  return *(const __attribute__((address_space(1))) T*)p;
}

// A pointer that is the same in all lanes, in scalar registers, and accesses at a
// byte offset of 32 bits from it: the address needs no 64-bit arithmetic per lane,
// and constant steps of up to 4 KB from the offset are free.
template <typename T>
__device__ __forceinline__ T* uni(T* p) {
  const unsigned long long a = (unsigned long long)p;
  const unsigned lo = __builtin_amdgcn_readfirstlane((unsigned)a), hi = __builtin_amdgcn_readfirstlane((unsigned)(a >> 32));
  return (T*)(((unsigned long long)hi << 32) | lo);
}
template <typename T>
__device__ __forceinline__ T gldo(const T* base, unsigned off, unsigned step = 0) {
  typedef const __attribute__((address_space(1))) char* P;
  return *(const __attribute__((address_space(1))) T*)((P)base + off + step);
}

template <typename T>
__device__ __forceinline__ void vst(T* p, T v) {
#if PFC_STORE_POLICY == 1
  __hip_atomic_store(gp(p), v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#elif PFC_STORE_POLICY == 2
  __builtin_nontemporal_store(v, gp(p));
#else
  *gp(p) = v;
#endif
}

template <typename T>
__device__ __forceinline__ void vsto(T* base, unsigned off, T v) {
  typedef __attribute__((address_space(1))) char* P;
  vst((T*)((P)base + off), v);
}

// Rows of the solver phases.  A slice belongs to one wave, so its place in the
// value arrays is a scalar; f(W) is called with the slice's width as a constant
// (0: some other width) for the widths named at for_width.
template <bool P2, typename F>
__device__ __forceinline__ void with_width(int w, F f) {
  if (w == 7) { f(std::integral_constant<int, 7>()); return; }
  if (w == 15) { f(std::integral_constant<int, 15>()); return; }
  if constexpr (P2) {
    if (w == 9) { f(std::integral_constant<int, 9>()); return; }
    if (w == 19) { f(std::integral_constant<int, 19>()); return; }
  }
  f(std::integral_constant<int, 0>());
}
// the columns of the row of (slice, lane), all loaded (or computed) at once
template <int W, int L>
__device__ __forceinline__ void row_cols(const PatView<L>& pv, int sl, int lane, int* j) {
  const int i = sl * 64 + lane;
  if constexpr (L == PFC_COL_GRID) {
    const int r = i < pv.n ? i : pv.n - 1;
    const int* gl = pv.gd + grid_class(r, pv.gN, pv.gInv) * PFC_GRID_W;
#pragma unroll
    for (int k = 0; k < W; ++k) j[k] = r + gl[k];
  } else if constexpr (L == PFC_COL_LDS) {
    const int* c = pfc_lcol + (pv.base(sl) + lane - pv.lo);
#pragma unroll
    for (int k = 0; k < W; ++k) j[k] = c[64 * k];
  } else {
    const int* c = uni(pv.col + pv.base(sl));
#pragma unroll
    for (int k = 0; k < W; ++k) j[k] = gldo(c, (unsigned)lane * 4u, k * 256u);
  }
}
#define PFC_LOOP32 (1 << 22)  // entries of a row whose byte offsets fit 32 bits
// sum over the entries of the row of (slice, lane), in order: load(k, j) gives what
// entry k needs of memory (column j), use(v) adds it.  The columns are loaded at
// once and the entries in chunks of CH, whose loads are issued together: a chunk is
// one round trip (the columns' and the entries' loads one entry after the other
// are two each).  Chunks: C::of(W, L) entries.
template <typename C, int L, typename LoadF, typename UseF>
__device__ __forceinline__ void row_entries(const PatView<L>& pv, int sl, int lane, LoadF load, UseF use) {
  with_width<L == PFC_COL_MEM>(pv.width(sl), [&](auto wc) {  // (rows of 9 and 19 entries have no common width)
    constexpr int W = decltype(wc)::value;
    if constexpr (W > 0) {
      constexpr int CH = C::of(W, L);
      int j[W];
      row_cols<W>(pv, sl, lane, j);
#pragma unroll
      for (int c = 0; c < W; c += CH) {
        decltype(load(0, 0)) v[CH];
#pragma unroll
        for (int u = 0; u < CH; ++u)
          if (c + u < W) v[u] = load(c + u, j[c + u]);
#pragma unroll
        for (int u = 0; u < CH; ++u)
          if (c + u < W) use(v[u]);
        __builtin_amdgcn_sched_barrier(0);  // (the next chunk's loads would not fit beside this one's)
        asm volatile("" ::: "memory");
      }
    } else {
      const int w = pv.width(sl), e0 = pv.base(sl) + lane;
      if (L == PFC_COL_MEM && w > PFC_LOOP32) {
        for (long long k = 0; k < w; ++k) use(load(k, pv.at(e0 + 64 * k, sl * 64 + lane)));
      } else {
        for (int k = 0; k < w; ++k) use(load(k, pv.at((long long)e0 + 64LL * k, sl * 64 + lane)));
      }
    }
  });
}

// Workgroup placement.  The dispatcher deals the workgroups of a launch to the
// 8 XCDs in turn (workgroup b lands on XCD b mod 8), and each XCD has its own
// L2.  Rows a workgroup gathers from its neighbours' blocks are only reused
// from L2 when those neighbours sit on the same XCD, so the rank (row block)
// of a workgroup is renumbered to give every XCD one contiguous run of ranks:
// XCD x owns ranks [x*q + min(x, r), ...) with q = g / 8, r = g mod 8.  The
// map is a bijection of [0, g) for every g.
#ifndef PFC_XCD_MAP
#define PFC_XCD_MAP 1
#endif
#define PFC_XCDS 8
__device__ __forceinline__ int xcd_rank(int b, int g) {
#if PFC_XCD_MAP
  const int q = g / PFC_XCDS, r = g % PFC_XCDS, x = b % PFC_XCDS;
  return x * q + (x < r ? x : r) + b / PFC_XCDS;
#else
  (void)g;
  return b;
#endif
}

// ---- typed views ----------------------------------------------------------
template <typename T> struct TV;
template <> struct TV<double> {
  __device__ static const double* M(const InstDev& I) { return I.m.M; }
  __device__ static const double* K(const InstDev& I) { return I.m.K; }
  __device__ static const double* dM(const InstDev& I) { return I.m.dinvM; }
};
template <> struct TV<float> {
  __device__ static const float* M(const InstDev& I) { return I.m.Mf; }
  __device__ static const float* K(const InstDev& I) { return I.m.Kf; }
  __device__ static const float* dM(const InstDev& I) { return I.m.dinvMf; }
};

// ---- element integrals (exact for P1, Section 3) ----------------------------
// int_T psi_h^2 lambda_a lambda_b = |T| c_m (1 + [a==b]) [S1^2 + S2 + 2 S1 (pa + pb) + 2 (pa^2 + pb^2 + pa pb)]
// int_T psi_h^3 lambda_a         = |T| c_m [S1^3 + 3 S1 S2 + 2 S3 + 3 pa (S1^2 + S2) + 6 pa^2 S1 + 6 pa^3]
// with S_k = sum over the vertices of psi^k and c_m = m!/(m+4)!.
__device__ __forceinline__ double cm_of(int dim) { return dim == 2 ? (1.0 / 360.0) : (1.0 / 840.0); }

// P2 (Section 3, p = 2; integrands of degree 8, exact through reference tables
// of the basis' fourfold products over |T|, packed by their symmetry in c, d
// and in b, c, d):
//   Mpsi2^T_ab          = |T| sum_{c <= d} psi_c psi_d C2[a][b][c, d]
//   int_T psi_h^3 phi_a = |T| sum_{b <= c <= d} psi_b psi_c psi_d C3[a][b, c, d]
//
// Element sums are formed row by row: a thread walks the simplices around its
// node once and adds each simplex's terms to the entries of its row, whose
// positions the mesh stores with the visit.  Against walking the simplices of
// every stored entry (dim + 1 times as many visits, each with its own gathers
// of the element's nodes and of psi there) the visit lists are coalesced
// streams and psi is gathered once per neighbour or once per visit.  Bound by
// those gathers' latency, so the loads of several visits are issued together;
// the terms of an entry are added in element order, one at a time.
// Measured per call, launch and wait (17 us) included: pfc_assemble_N on 3D 64^3
// 429 -> 63 us, pfc_apply_AR on 2D 512^2 65 -> 28 us, pfc_stage_rhs on 3D 48^3
// 128 -> 46 us, pfc_load_psi3 on P2 200^2 68 -> 31 us; inside the solver's
// launches (psi through the element's nodes, row_matrix) a 3D 64^3 step 25.8 -> 25.3 ms.

// one visit: the simplex, its volume, the node's local index a, psi at the
// simplex's Q nodes; slot(c): position of its local node c in the row
template <int Q>
struct Visit {
  static constexpr int W = (Q + 3) / 4;
  int el, a;
  double vol, p[Q];
  unsigned word[W];        // narrow rows: the positions, a byte each
  const unsigned* wide;    // long rows: the lane's first position, and the visit; or null
  int t;
  __device__ __forceinline__ int slot(int c) const {
    if (wide) return (int)wide[64LL * ((long long)Q * t + c)];
    unsigned w = word[0];
#pragma unroll
    for (int q = 1; q < W; ++q) w = c >= 4 * q ? word[q] : w;
    return (int)((w >> (8 * (c & 3))) & 255u);
  }
};

// visit(v) for every simplex around the row of (slice, lane), in element order;
// psi(v, c): the value at local node c of the visit's simplex.  Q: nodes per
// simplex (3, 4: P1; 6, 10: P2).  U visits' list entries and volumes are loaded
// together; AHEAD: their psi as well (gathers from memory), else each visit's psi
// (read from LDS) just before the visit.  WIDE: the mesh may have long rows.
template <int Q, int U, bool AHEAD, bool WIDE, typename PsiF, typename F>
__device__ __forceinline__ void for_visits(const MeshDev& m, int sl, int lane, PsiF psi, F visit) {
  constexpr int BITS = Q <= 4 ? 2 : 4, W = Visit<Q>::W;
  const long long vb = m.nv_ptr[sl];
  const int vw = (int)((m.nv_ptr[sl + 1] - vb) >> 6);
  const int* el_l = m.nv_el + vb + lane;
  const unsigned* slot_l = m.nv_slot + vb * m.nv_words + lane;
  const bool wide = WIDE && m.nv_wide != 0;
  for (int t = 0; t < vw; t += U) {
    Visit<Q> v[U];
    int pk[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int tu = min(t + u, vw - 1);
      pk[u] = el_l[64LL * tu];
      v[u].wide = wide ? slot_l : nullptr;
      v[u].t = tu;
#pragma unroll
      for (int q = 0; q < W; ++q) v[u].word[q] = wide ? 0u : slot_l[64LL * ((long long)W * tu + q)];
      if (t + u >= vw) pk[u] = -1;
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      v[u].el = max(pk[u], 0) >> BITS;
      v[u].a = pk[u] & ((1 << BITS) - 1);
      v[u].vol = m.elem_vol[v[u].el];
      if constexpr (AHEAD) {
#pragma unroll
        for (int c = 0; c < Q; ++c) v[u].p[c] = psi(v[u], c);
      }
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (pk[u] < 0) continue;
      if constexpr (!AHEAD) {
#pragma unroll
        for (int c = 0; c < Q; ++c) v[u].p[c] = psi(v[u], c);
      }
      visit(v[u]);
    }
  }
}
// visits per group: with psi gathered from memory, and with psi in LDS
template <int Q> struct VisitU { static constexpr int mem = Q <= 4 ? 2 : 1, lds = Q <= 4 ? (Q == 3 ? 6 : 8) : 2; };

// psi read from a vector over the nodes through the element's node list
template <int Q, typename NodeF>
struct NodePsi {
  const int* en;
  NodeF f;
  __device__ __forceinline__ double operator()(const Visit<Q>& v, int c) const { return f(en[(long long)v.el * Q + c]); }
};
template <int Q, typename NodeF>
__device__ __forceinline__ NodePsi<Q, NodeF> node_psi(const MeshDev& m, NodeF f) {
  return NodePsi<Q, NodeF>{m.elem_nodes, f};
}

// f(table) once per local index a present among the lanes, on the lanes that
// have it, with the table of that index at a wave-uniform address (the tables
// are then read through the scalar cache; on the meshes met in practice the rows
// of a slice have the same local index at the same visit)
template <typename F>
__device__ __forceinline__ void per_local_index(const double* tab, int stride, int a, F f) {
  unsigned long long todo = __ballot(1);
  while (todo) {
    const int au = __builtin_amdgcn_readlane(a, __ffsll((long long)todo) - 1);
    const bool mine = a == au;
    const unsigned long long base = (unsigned long long)(tab + au * stride);
    const unsigned lo = __builtin_amdgcn_readfirstlane((unsigned)base);
    const unsigned hi = __builtin_amdgcn_readfirstlane((unsigned)(base >> 32));
    if (mine) f((const __attribute__((address_space(4))) double*)(((unsigned long long)hi << 32) | lo));
    todo &= ~__ballot(mine);
  }
}

// Sums of a row's entries in LDS: entry k of entries [s0, s0 + c) at acc[(k - s0) st]
// (ALL: of all entries, s0 = 0); add: entry of local node b += x[b] y[b].  The positions of a simplex's nodes differ, so
// its Q sums are read together before any is written.
template <bool ALL>
struct RowAcc {
  double* acc;
  int st, s0, c;
  template <int Q>
  __device__ __forceinline__ void add(const Visit<Q>& v, const double* x, const double* y) const {
    if constexpr (ALL) {
      double t[Q];
      int s[Q];
#pragma unroll
      for (int b = 0; b < Q; ++b) { s[b] = v.slot(b) * st; t[b] = acc[s[b]]; }
#pragma unroll
      for (int b = 0; b < Q; ++b) acc[s[b]] = fma(x[b], y[b], t[b]);
    } else {
#pragma unroll
      for (int b = 0; b < Q; ++b) add1(v.slot(b), x[b], y[b]);
    }
  }
  __device__ __forceinline__ void add1(int pos, double x, double y) const {
    const int k = pos - s0;
    if (ALL || (unsigned)k < (unsigned)c) acc[k * st] = fma(x, y, acc[k * st]);
  }
};

// ... in the row's stored entries themselves: entry k at out[64 k] (device memory)
struct RowMem {
  double* out;
  template <int Q>
  __device__ __forceinline__ void add(const Visit<Q>& v, const double* x, const double* y) const {
    double t[Q];
    int s[Q];
#pragma unroll
    for (int b = 0; b < Q; ++b) { s[b] = 64 * v.slot(b); t[b] = gld(out + s[b]); }
#pragma unroll
    for (int b = 0; b < Q; ++b) *gp(out + s[b]) = fma(x[b], y[b], t[b]);
  }
  __device__ __forceinline__ void add1(int pos, double x, double y) const {
    double* p = out + 64 * pos;
    *gp(p) = fma(x, y, gld(p));
  }
};

// the bracket of int_T psi_h^2 lambda_a lambda_b (one rounding sequence, whatever the
// compiler could contract: with float32 inner solves a last place here can move a
// result by far more)
__device__ __forceinline__ double psi2_product(double S1, double S2, double pa, double pb) {
  return fma(2.0, fma(pa, pb, fma(pa, pa, pb * pb)), fma(pa + pb, S1 + S1, fma(S1, S1, S2)));
}

// the simplex's contributions to Mpsi2 between the node and each of its nodes
template <int Q, typename Acc>
__device__ __forceinline__ void visit_Mpsi2(const MeshDev& m, const Visit<Q>& v, const Acc& acc) {
  if constexpr (Q <= 4) {
    const double cm = cm_of(Q - 1);
    double S1 = 0.0, S2 = 0.0;
#pragma unroll
    for (int c = 0; c < Q; ++c) { S1 += v.p[c]; S2 = fma(v.p[c], v.p[c], S2); }
    double pa = v.p[0];
#pragma unroll
    for (int c = 1; c < Q; ++c) pa = v.a == c ? v.p[c] : pa;
    double x[Q], y[Q];
#pragma unroll
    for (int b = 0; b < Q; ++b) {
      x[b] = v.vol * cm * (v.a == b ? 2.0 : 1.0);
      y[b] = psi2_product(S1, S2, pa, v.p[b]);
    }
    acc.add(v, x, y);
  } else {
    constexpr int NP = Q * (Q + 1) / 2, W = Visit<Q>::W;
    per_local_index(m.p2_C2, Q * NP, v.a, [&](auto C) {
      unsigned pos[W];  // the positions, shifted by a byte per node (an index that varies would put them in memory)
#pragma unroll
      for (int w = 0; w < W; ++w) pos[w] = v.word[w];
#pragma unroll 1
      for (int b = 0; b < Q; ++b) {
        double s = 0.0;
        int q = b * NP;
#pragma unroll
        for (int c = 0; c < Q; ++c) {
          double r = 0.0;
#pragma unroll
          for (int d = c; d < Q; ++d) r += C[q++] * v.p[d];
          s += v.p[c] * r;
        }
        const int k = v.wide ? v.slot(b) : (int)(pos[0] & 255u);
#pragma unroll
        for (int w = 0; w < W; ++w) pos[w] = (pos[w] >> 8) | (w + 1 < W ? pos[w + 1] << 24 : 0u);
        acc.add1(k, v.vol, s);
      }
    });
  }
}

// the simplex's contribution to the cubic load of the node
template <int Q>
__device__ __forceinline__ double visit_psi3(const MeshDev& m, const Visit<Q>& v) {
  if constexpr (Q <= 4) {
    const double cm = cm_of(Q - 1);
    double S1 = 0.0, S2 = 0.0, S3 = 0.0;
#pragma unroll
    for (int c = 0; c < Q; ++c) { S1 += v.p[c]; S2 = fma(v.p[c], v.p[c], S2); S3 = fma(v.p[c], v.p[c] * v.p[c], S3); }
    double pa = v.p[0];
#pragma unroll
    for (int c = 1; c < Q; ++c) pa = v.a == c ? v.p[c] : pa;
    const double s = S1 * S1 * S1 + 3.0 * S1 * S2 + 2.0 * S3 + 3.0 * pa * (S1 * S1 + S2) + 6.0 * pa * pa * S1 + 6.0 * pa * pa * pa;
    return v.vol * cm * s;
  } else {
    constexpr int NT = Q * (Q + 1) * (Q + 2) / 6;
    double s = 0.0;
    per_local_index(m.p2_C3, NT, v.a, [&](auto C) {
      int q = 0;
#pragma unroll
      for (int b = 0; b < Q; ++b) {
        double r2 = 0.0;
#pragma unroll
        for (int c = b; c < Q; ++c) {
          double r = 0.0;
#pragma unroll
          for (int d = c; d < Q; ++d) r += C[q++] * v.p[d];
          r2 += v.p[c] * r;
        }
        s += v.p[b] * r2;
      }
    });
    return v.vol * s;
  }
}

// Row of a matrix of element sums: term(sums) visits the simplices of the row and
// adds to its entries; the sums are held in LDS (acc[k * st], k < cap), in as many
// rounds as the row needs (ALL: in one), and written by put(position, value).
template <bool ALL, typename TermF, typename PutF>
__device__ __forceinline__ void row_sums(double* acc, int st, int cap, int w, TermF term, PutF put) {
  for (int s0 = 0; s0 < w; s0 += cap) {
    const int c = min(cap, w - s0);
    for (int k = 0; k < c; ++k) acc[k * st] = 0.0;
    term(RowAcc<ALL>{acc, st, s0, c});
    for (int k = 0; k < c; ++k) put(s0 + k, acc[k * st]);
    if (ALL) break;
  }
}

// Row of a matrix of element sums in the mesh's layout (entry k at out[64 k]), times
// scale, with room for cap sums per thread in LDS.  A round of row_sums walks all
// simplices of the row again, so its time grows with the square of a long row: rows of
// more than two rounds are summed in place in one walk (ANY: the mesh may have them),
// at the price of a read of the stored sums per visit; P2 rows always, whose visits are
// the dearer part (all Q terms of a visit are formed in every round).  A step with one
// Arnoldi step and one inner iteration a solve, rounds -> in place: hub of 1000
// triangles 86.1 -> 14.5 ms, unstructured tetrahedra with 10^5 nodes (rows of 16, at
// most 54) 4.09 -> 3.77, P2 tetrahedra 20^3 3.92 -> 3.47, unstructured P2 tetrahedra
// with 173665 nodes 25.5 -> 13.7; grids of rows up to 16 keep the rounds (1.06, 1.06).
template <bool ANY, int Q, typename TermF>
__device__ __forceinline__ void row_matrix(double* acc, int st, int cap, int w, double* out, double scale, TermF term) {
  if (Q > 4 || (ANY && w > 2 * cap)) {
    for (int k = 0; k < w; ++k) *gp(out + 64LL * k) = 0.0;
    term(RowMem{out});
    for (int k = 0; k < w; ++k) *gp(out + 64LL * k) = scale * gld(out + 64LL * k);
  } else {
    row_sums<false>(acc, st, cap, w, term, [&](int k, double x) { out[64LL * k] = scale * x; });
  }
}

// ---- mobility matrices of the PFC1 model (Section 3) ---------------------------
// P1: grad lambda is constant on a simplex and int_T lambda_c = |T| / (m+1), so
//   K_+(psi)^T_ab = (sum_c psi^+_c / (m+1)) |T| grad l_a . grad l_b
//   F(mu)^T_ab    = (1 / (m+1)) sum_c mu_c |T| grad l_c . grad l_a   (a: test, b: trial)
// with |T| grad l_a . grad l_b read from the element stiffness (upper triangle).
__device__ __forceinline__ double elem_k(const MeshDev& m, int el, int a, int b) {
  const int k = m.dim + 1;
  if (a > b) { const int t = a; a = b; b = t; }
  return m.elem_K[(long long)el * (k * (k + 1) / 2) + a * k - a * (a - 1) / 2 + (b - a)];
}

template <int Q, typename Acc>
__device__ __forceinline__ void visit_Kplus(const MeshDev& m, const Visit<Q>& v, double psi_min, const Acc& acc) {
  const double ik = 1.0 / Q;
  double s = 0.0;
#pragma unroll
  for (int c = 0; c < Q; ++c) s += v.p[c] - psi_min;
  double x[Q], y[Q];
#pragma unroll
  for (int b = 0; b < Q; ++b) { x[b] = s * ik; y[b] = elem_k(m, v.el, v.a, b); }
  acc.add(v, x, y);
}

// v.p: mu at the simplex's nodes
template <int Q, typename Acc>
__device__ __forceinline__ void visit_F(const MeshDev& m, const Visit<Q>& v, const Acc& acc) {
  const double ik = 1.0 / Q;
  double s = 0.0;
#pragma unroll
  for (int c = 0; c < Q; ++c) s += v.p[c] * elem_k(m, v.el, c, v.a);
  double x[Q], y[Q];
#pragma unroll
  for (int b = 0; b < Q; ++b) { x[b] = s; y[b] = ik; }
  acc.add(v, x, y);
}

// contribution to (K_+(psi) mu)_i of a simplex around node i (the stage
// right-hand side needs it at the stage state, where no assembled K_+ exists);
// mu(v, c): mu at its local node c
template <int Q, typename MuF>
__device__ __forceinline__ double visit_Kplus_mu(const MeshDev& m, const Visit<Q>& v, MuF mu, double psi_min) {
  const double ik = 1.0 / Q;
  double sp = 0.0, km = 0.0;
#pragma unroll
  for (int c = 0; c < Q; ++c) {
    sp += v.p[c] - psi_min;
    km += elem_k(m, v.el, v.a, c) * mu(v, c);
  }
  return sp * ik * km;
}

// Columns of the rows of one slice for the mesh-level kernels: where every row
// of the slice lies inside a periodic grid (no edge row), entry k's column is the
// row plus one offset for the whole wave, so its index is not read and x at the
// neighbours is a coalesced load; elsewhere the stored columns are read.
// (pfc_spmv, 2D 1000^2: 35.1 -> 29.8 us per call)
struct WaveCols {
  const int* col;  // stored columns from the lane's first entry, or null
  const int* off;  // offsets of the interior row class
  int i;
  __device__ __forceinline__ int at(int k) const { return col ? col[64LL * k] : i + off[k]; }
};
__device__ __forceinline__ WaveCols wave_cols(const MeshDev& m, int sl, int lane, long long e0) {
  const int i = sl * 64 + lane, inner = m.dim == 2 ? 4 : 13;
  const bool in = m.gN > 0 && i < m.n && grid_class(i, m.gN, m.gInv) == inner;
  return WaveCols{__all(in) ? nullptr : m.col + e0, m.glin + inner * PFC_GRID_W, i};
}

// LDS of the mesh-level kernels with element sums (RowPlan)
extern __shared__ double pfc_row_lds[];

// f(integral_constant<Q>) for the mesh's nodes per simplex (ANY: the mesh may be P2, and have
// long rows; else it is a P1 grid)
template <bool ANY, typename F>
__device__ __forceinline__ void with_nloc(const MeshDev& m, F f) {
  if constexpr (ANY) {
    if (m.nloc == 6) { f(std::integral_constant<int, 6>()); return; }
    if (m.nloc == 10) { f(std::integral_constant<int, 10>()); return; }
  }
  if (m.dim == 2) f(std::integral_constant<int, 3>());
  else f(std::integral_constant<int, 4>());
}

// int psi_h^3 phi_i at the row of (slice, lane), psi(node) from a functor
template <bool ANY, typename PsiF>
__device__ __forceinline__ double node_psi3(const MeshDev& m, int sl, int lane, PsiF psi) {
  double g = 0.0;
  with_nloc<ANY>(m, [&](auto q) {
    constexpr int Q = decltype(q)::value;
    for_visits<Q, VisitU<Q>::mem, true, ANY>(m, sl, lane, node_psi<Q>(m, psi),
                                        [&](const Visit<Q>& v) { g += visit_psi3<Q>(m, v); });
  });
  return g;
}

// N(psi) = -3 Mpsi2 on the row of (slice, lane), stored at out[64 k]
template <bool ANY, typename PsiF>
__device__ __forceinline__ void row_N(const MeshDev& m, int sl, int lane, double* acc, int st, int cap, int w,
                                      PsiF psi, double* out) {
  with_nloc<ANY>(m, [&](auto q) {
    constexpr int Q = decltype(q)::value;
    row_matrix<ANY, Q>(acc, st, cap, w, out, -3.0, [&](auto sums) {
      for_visits<Q, VisitU<Q>::mem, true, ANY>(m, sl, lane, node_psi<Q>(m, psi),
                                          [&](const Visit<Q>& v) { visit_Mpsi2<Q>(m, v, sums); });
    });
  });
}

// K_+(psi) and F(mu) on the row of (slice, lane) (PFC1: P1 meshes), stored at kp[64 k], fm[64 k]
template <bool ANY, typename PsiF, typename MuF>
__device__ __forceinline__ void row_mob(const MeshDev& m, int sl, int lane, double* acc, int st, int cap, int w,
                                        PsiF psi, MuF mu, double psi_min, double* kp, double* fm) {
  with_nloc<false>(m, [&](auto q) {
    constexpr int Q = decltype(q)::value;
    row_matrix<ANY, Q>(acc, st, cap, w, kp, 1.0, [&](auto sums) {
      for_visits<Q, VisitU<Q>::mem, true, ANY>(m, sl, lane, node_psi<Q>(m, psi),
                                          [&](const Visit<Q>& v) { visit_Kplus<Q>(m, v, psi_min, sums); });
    });
    row_matrix<ANY, Q>(acc, st, cap, w, fm, 1.0, [&](auto sums) {
      for_visits<Q, VisitU<Q>::mem, true, ANY>(m, sl, lane, node_psi<Q>(m, mu),
                                          [&](const Visit<Q>& v) { visit_F<Q>(m, v, sums); });
    });
  });
}

// (K_+(psi) mu)_i at the row of (slice, lane) (PFC1: P1 meshes)
template <bool ANY, typename PsiF, typename MuF>
__device__ __forceinline__ double node_Kplus_mu(const MeshDev& m, int sl, int lane, PsiF psi, MuF mu, double psi_min) {
  double acc = 0.0;
  with_nloc<false>(m, [&](auto q) {
    constexpr int Q = decltype(q)::value;
    for_visits<Q, VisitU<Q>::mem, true, ANY>(m, sl, lane, node_psi<Q>(m, psi), [&](const Visit<Q>& v) {
      acc += visit_Kplus_mu<Q>(m, v, node_psi<Q>(m, mu), psi_min);
    });
  });
  return acc;
}

// ---- phases ---------------------------------------------------------------
// Every phase returns this thread's contribution to the two partial sums.

// N(psi_k) = -3 Mpsi2 reassembled in place (one value per stored entry).
template <int L>
__device__ __forceinline__ Red3 ph_rb_begin(const InstDev& I, const Team& tm) {
  const int n = I.n;
  const double* xk = I.xk;
  auto psi = [&](int j) { return xk[n + j]; };
  const PatView<L> pv = p1_pat<L>(I, tm);
  PFC_SLICES(I, tm) {
    const int lane = tm.lane, w = pv.width(sl);
    const long long e0 = (long long)pv.base(sl) + lane;
    double* acc = pfc_ss + threadIdx.x;
    constexpr int cap = PFC_SS_LDS / PFC_WG;
    row_N<L != PFC_COL_GRID>(I.m, sl, lane, acc, PFC_WG, cap, w, psi, I.N + e0);
    if (I.model == PFC_MODEL_PFC1)
      row_mob<L != PFC_COL_GRID>(I.m, sl, lane, acc, PFC_WG, cap, w, psi, [&](int j) { return xk[j]; }, I.psi_min,
                                 I.Kp + e0, I.Fm + e0);
  }
  return red3(0.0, 0.0);
}

__device__ __forceinline__ double stage_comb(const InstDev& I, int stage, int blk, int j) {
  const long long n3 = 3LL * I.n;
  const long long o = (long long)blk * I.n + j;
  double v = I.xk[o];
  if (stage == 2) v += ROS_A21 * I.ys[o];
  if (stage == 3) v += ROS_A31 * I.ys[o] + ROS_A32 * I.ys[n3 + o];
  return v;
}

// Stage right-hand side at a row (Section 3.1): F(x_i) with block 1 multiplied by
// tau, plus sum_j c_ij M y_j^psi on block 1, with the stage state
// x_i = x_k + sum_j a_ij y_j formed on the fly.  The products with M and K over
// the row's w entries (entry k at position pos(k) of the values, column col(k));
// seen(k, mu, psi) is told the stage state there.
struct StageSums {
  double b0, b2, Kmu, My1, My2;
};
template <typename PosF, typename ColF, typename SeenF>
__device__ __forceinline__ StageSums stage_rhs_products(const InstDev& I, int w, int stage, PosF pos, ColF col, SeenF seen) {
  const int n = I.n;
  double sMmu = 0, sMps = 0, sMom = 0, sKmu = 0, sKps = 0, sKom = 0, sMy1 = 0, sMy2 = 0;
  const long long n3 = 3LL * n;
  for (int k = 0; k < w; ++k) {
    const long long e = pos(k);
    const int j = col(k);
    const double Mv = I.m.M[e], Kv = I.m.K[e];
    const double mu = stage_comb(I, stage, 0, j);
    const double ps = stage_comb(I, stage, 1, j);
    const double om = stage_comb(I, stage, 2, j);
    seen(k, mu, ps);
    sMmu += Mv * mu; sMps += Mv * ps; sMom += Mv * om;
    sKmu += Kv * mu; sKps += Kv * ps; sKom += Kv * om;
    if (stage >= 2) sMy1 += Mv * I.ys[n + j];
    if (stage >= 3) sMy2 += Mv * I.ys[n3 + n + j];
  }
  return StageSums{-sMmu + (1.0 + I.r) * sMps - 2.0 * sKps - sKom, -sMom - sKps, sKmu, sMy1, sMy2};
}

// ... and the element sums: the cubic load g and, for PFC1, (K_+(psi_i) mu_i) = kpm
__device__ __forceinline__ void stage_rhs_finish(const InstDev& I, const StageSums& q, int stage, double g, double kpm,
                                                 double& b0, double& b1, double& b2) {
  b0 = q.b0 + g;
  // (roundings spelled out: the same in a solver launch and on its own)
  const double k = -(I.model == PFC_MODEL_PFC1 ? kpm : q.Kmu);
  b1 = I.tau * k;
  if (stage == 2) b1 = fma(ROS_C21, q.My1, b1);
  if (stage == 3) b1 = fma(I.tau, k, fma(ROS_C31, q.My1, ROS_C32 * q.My2));
  b2 = q.b2;
}

template <int L>
__device__ __forceinline__ void stage_rhs_row(const InstDev& I, const PatView<L>& pv, int sl, int lane, int stage,
                                              double& b0, double& b1, double& b2) {
  const long long e0 = (long long)pv.base(sl) + lane;
  const int i = sl * 64 + lane;
  const StageSums q = stage_rhs_products(I, pv.width(sl), stage, [&](int k) { return e0 + 64LL * k; },
                                         [&](int k) { return pv.at(e0 + 64LL * k, i); }, [](int, double, double) {});
  auto psi = [&](int j) { return stage_comb(I, stage, 1, j); };
  const double g = node_psi3<L != PFC_COL_GRID>(I.m, sl, lane, psi);
  double kpm = 0.0;
  if (I.model == PFC_MODEL_PFC1)
    kpm = node_Kplus_mu<L != PFC_COL_GRID>(I.m, sl, lane, psi, [&](int j) { return stage_comb(I, stage, 0, j); }, I.psi_min);
  stage_rhs_finish(I, q, stage, g, kpm, b0, b1, b2);
}

// Right-hand side of the solve: stage rhs b_i^R for job RB, the caller's rhs
// for job SOLVE.  Writes W = b with block 1 multiplied by rs, X = 0.
template <int L>
__device__ __forceinline__ Red3 ph_solve_init(const InstDev& I, const State& S, const Team& tm) {
  const int n = I.n;
  const bool rb = __builtin_amdgcn_readfirstlane(S.job) == JOB_RB;
  const PatView<L> pv = p1_pat<L>(I, tm);
  double* X = rb ? (I.ys + (long long)(S.stage - 1) * 3 * n) : I.x_user;
  const double im = I.rs;
  double a0 = 0.0, a1 = 0.0;
  PFC_SLICES(I, tm) {
    const int i = sl * 64 + tm.lane;
    double b0 = 0.0, b1 = 0.0, b2 = 0.0;
    if (rb) stage_rhs_row<L>(I, pv, sl, tm.lane, S.stage, b0, b1, b2);
    if (i < n) {
      if (rb) {
        vst(I.b + i, b0); vst(I.b + n + i, b1); vst(I.b + 2 * n + i, b2);
      } else {
        b0 = I.b_user[i]; b1 = I.b_user[n + i]; b2 = I.b_user[2 * n + i];
      }
      const double bs1 = b1 * im;
      vst(I.W + i, b0); vst(I.W + n + i, bs1); vst(I.W + 2 * n + i, b2);
      vst(X + i, 0.0); vst(X + n + i, 0.0); vst(X + 2 * n + i, 0.0);
      a0 += b0 * b0 + b1 * b1 + b2 * b2;
      a1 += b0 * b0 + bs1 * bs1 + b2 * b2;
    }
  }
  return red3(a0, a1);
}

__device__ __forceinline__ Red3 ph_rb_update(const InstDev& I, const Team& tm) {
  const int n = I.n;
  const long long n3 = 3LL * n;
  PFC_SLICES(I, tm) {
    const int i = sl * 64 + tm.lane;
    if (i < n) {
      for (int blk = 0; blk < 3; ++blk) {
        const long long o = (long long)blk * n + i;
        I.xk[o] = I.xk[o] + ROS_M1 * I.ys[o] + ROS_M2 * I.ys[n3 + o] + ROS_M3 * I.ys[2 * n3 + o];
      }
    }
  }
  return red3(0.0, 0.0);
}

// ---- inner PCG --------------------------------------------------------------
template <typename T>
struct PcgOps {
  const T* C;      // stored operator values, or nullptr for M + cK on the fly
  const T* Mv;
  const T* Kv;
  T cK;
  const T* dinv;
  T* x;
  const int* sp;   // slice offsets and columns of the operator's pattern
  const int* colp;
};

__device__ __forceinline__ bool is_ci(int kind) { return kind == KIND_CI_OMEGA || kind == KIND_CI_MU; }

template <typename T>
__device__ __forceinline__ PcgOps<T> pcg_ops(const InstDev& I, int kind) {
  PcgOps<T> o;
  kind = __builtin_amdgcn_readfirstlane(kind);
  o.Mv = TV<T>::M(I);
  o.Kv = TV<T>::K(I);
  o.cK = T(0);
  o.C = o.Mv;
  o.dinv = TV<T>::dM(I);
  o.x = nullptr;
  o.sp = I.m.slice_ptr;
  o.colp = I.m.col;
  const int n = I.n;
  switch (kind) {
    case KIND_Y0: o.x = (T*)I.y0; break;
    case KIND_Y1:
      o.x = (T*)I.y1;
      o.dinv = (const T*)I.dinvCd;
      if (I.shared_ops) { o.C = nullptr; o.cK = T(I.delta); } else o.C = (const T*)I.Cd;
      break;
    case KIND_Z:
    case KIND_X1:
      o.x = (T*)(kind == KIND_Z ? I.zt : I.x1);
      o.dinv = (const T*)I.dinvCsd;
      if (I.shared_ops) { o.C = nullptr; o.cK = T(I.sdelta); } else o.C = (const T*)I.Csd;
      break;
    case KIND_X2: o.x = (T*)I.x2; break;
    case KIND_SD:
      o.x = (T*)I.x1;
      o.C = (const T*)I.SDv;
      o.dinv = (const T*)I.dinvSD;
      o.sp = I.m.w_slice_ptr;
      o.colp = I.m.w_col;
      break;
    case KIND_CI_OMEGA: o.x = (T*)(I.xk + 2LL * n); break;
    case KIND_CI_MU: o.x = (T*)(I.xk); break;
  }
  o.C = uni(o.C);
  o.Mv = uni(o.Mv);
  o.Kv = uni(o.Kv);
  o.dinv = uni(o.dinv);
  o.x = uni(o.x);
  o.sp = uni(o.sp);
  o.colp = uni(o.colp);
  return o;
}

// Pattern of the operator of a PCG solve: the P1 pattern (staged columns when
// L) or, for S_D, the second-ring pattern (never staged).
template <int L, typename T>
__device__ __forceinline__ PatView<L> op_pat(const InstDev& I, const PcgOps<T>& o, const Team& tm) {
  // (the S_D pattern is only ever read with L == PFC_COL_MEM)
  return PatView<L>{o.sp, o.colp, o.sp == I.m.slice_ptr ? I.m.uw : 0, tm.lo, I.n, I.m.gN, I.m.gInv,
                    L == PFC_COL_GRID ? I.m.glin : nullptr};
}

template <typename T>
__device__ __forceinline__ T opval(const PcgOps<T>& o, long long e) {
  return o.C ? o.C[e] : (o.Mv[e] + o.cK * o.Kv[e]);
}
template <typename T>
__device__ __forceinline__ T opval_g(const PcgOps<T>& o, long long e) {
  return o.C ? gld(o.C + e) : (gld(o.Mv + e) + o.cK * gld(o.Kv + e));
}

// values of a slice's entries: entry k of the lane's row.  A step known at compile time
// goes with the scalar base (no lane's register: nothing spills beside the in-place sums
// of long rows); in a loop over k it is a 32-bit offset, which a row of at most
// PFC_LOOP32 entries fits (as a 64-bit scalar step it took 3D P2 10^3 float64 steps from
// 134.6 to 151.0 ms).  S: steps with the scalar base, where registers are short (double,
// or columns from memory); the float grid kernels lose a little by it (3D 64^3 mixed step
// 17.00 -> 17.07 ms)
template <bool S, typename T>
struct SliceVals {
  const T* a;
  unsigned off;
  __device__ __forceinline__ T operator()(int k) const {
    if (S && __builtin_constant_p(k)) return gldo(a + 64LL * k, off);
    return gldo(a, off + (unsigned)k * 64u * (unsigned)sizeof(T));
  }
  __device__ __forceinline__ T operator()(long long k) const { return gldo(a + 64 * k, off); }
};
template <bool S, typename T>
__device__ __forceinline__ SliceVals<S, T> slice_vals(const T* a, int base, int lane) {
  return SliceVals<S, T>{uni(a + base), (unsigned)lane * (unsigned)sizeof(T)};
}
template <typename T, int L>
constexpr bool scalar_steps() { return sizeof(T) == 8 || L == PFC_COL_MEM; }
// row_entries over a row of an operator, stored or M + cK (one choice for the row:
// a branch per entry would keep its loads apart); load(a, j) with the value a
template <typename C, typename T, int L, typename LoadF, typename UseF>
__device__ __forceinline__ void op_entries(const PcgOps<T>& o, const PatView<L>& pv, int sl, int lane, LoadF load, UseF use) {
  const int base = pv.base(sl);
  if (o.C) {
    const auto c = slice_vals<scalar_steps<T, L>()>(o.C, base, lane);
    row_entries<C>(pv, sl, lane, [&](auto k, int j) { return load(c(k), j); }, use);
  } else {
    const auto m = slice_vals<scalar_steps<T, L>()>(o.Mv, base, lane), q = slice_vals<scalar_steps<T, L>()>(o.Kv, base, lane);
    row_entries<C>(pv, sl, lane, [&](auto k, int j) { return load(m(k) + o.cK * q(k), j); }, use);
  }
}
// Chunks of the row loops: as many entries as the kernel's 128 registers hold beside
// the rest of the phase without spilling (the grid kernels also hold the block forms).
template <typename T>
struct ChunkIter {  // five values an entry
  static constexpr int of(int W, int L) {
    if (sizeof(T) == 8) return L == PFC_COL_MEM ? (W == 9 ? 5 : 4) : (W == 7 ? 3 : 4);
    return L == PFC_COL_MEM ? (W == 9 ? 9 : 7) : (W == 7 ? 4 : 7);
  }
};
struct ChunkInit {  // three
  static constexpr int of(int, int L) { return L == PFC_COL_GRID ? 4 : 6; }
};
struct ChunkBlock {  // six (eight with the mobility)
  static constexpr int of(int, int) { return 2; }
};
struct ChunkDot {  // two
  static constexpr int of(int, int L) { return L == PFC_COL_GRID ? 4 : 8; }
};

// an entry of a vector of T
template <typename T>
__device__ __forceinline__ T vat(const T* v, int j) { return gldo(v, (unsigned)j * (unsigned)sizeof(T)); }

// y_i = (A v)_i for a stored operator A (typed) over the row of thread lane
template <typename T>
struct DotTerm {
  T a, v;
};
template <typename T, int L>
__device__ __forceinline__ T row_dot(const PatView<L>& pv, int sl, int lane, const T* A, const T* v) {
  const auto a = slice_vals<scalar_steps<T, L>()>(A, pv.base(sl), lane);
  const T* u = uni(v);
  T acc = T(0);
  row_entries<ChunkDot>(pv, sl, lane, [&](auto k, int j) { return DotTerm<T>{a(k), vat(u, j)}; },
                 [&](const DotTerm<T>& t) { acc += t.a * t.v; });
  return acc;
}

template <typename T, int L>
__device__ __forceinline__ Red3 ph_pcg_setup(const InstDev& I, const State& S, const Team& tm) {
  const int n = I.n;
  const int kind = __builtin_amdgcn_readfirstlane(S.kind);
  PcgOps<T> o = pcg_ops<T>(I, kind);
  const PatView<L> pv = p1_pat<L>(I, tm);   // every right-hand side is a P1 product
  T* r = (T*)I.r_;
  const long long n3 = 3LL * n;
  double* Vj = I.V + (long long)S.j * n3;
  double* Zj = I.Z + (long long)S.j * n3;
  const T* Mv = o.Mv;
  const T* Kv = o.Kv;
  double a0 = 0.0, a1 = 0.0;
  PFC_SLICES(I, tm) {
    const int i = sl * 64 + tm.lane;
    const int lane = tm.lane;
    double rhs = 0.0;
    switch (kind) {
      case KIND_Y0: {
        if (i < n) {
          const double vs = S.vscale;
          const double v0 = I.W[i] * vs, v1 = I.W[n + i] * vs, v2 = I.W[2 * n + i] * vs;
          vst(Vj + i, v0); vst(Vj + n + i, v1); vst(Vj + 2 * n + i, v2);
          rhs = v0;
        }
      } break;
      case KIND_Y1: {  // (2): b1 - tau K y0
        const T* y0 = (const T*)I.y0;
        const T ky = row_dot<T>(pv, sl, lane, Kv, y0);
        if (i < n) rhs = Vj[n + i] - I.tau_p * (double)ky;
      } break;
      case KIND_SD:   // (3) with S_D: M y1
      case KIND_Z: {  // (3.1): M y1
        const T* y1 = (const T*)I.y1;
        const T my = row_dot<T>(pv, sl, lane, Mv, y1);
        rhs = (double)my;
      } break;
      case KIND_X1: {  // (3.2): M z
        const T* zt = (const T*)I.zt;
        const T mz = row_dot<T>(pv, sl, lane, Mv, zt);
        rhs = (double)mz;
      } break;
      case KIND_X2: {  // (5): b2 - K x1, and (4): x0 = y0 + (y1 - x1)/delta
        const T* x1 = (const T*)I.x1;
        const T kx = row_dot<T>(pv, sl, lane, Kv, x1);
        if (i < n) {
          rhs = Vj[2 * n + i] - (double)kx;
          const double y0i = (double)((const T*)I.y0)[i], y1i = (double)((const T*)I.y1)[i];
          const double x1i = (double)x1[i];
          vst(Zj + i, y0i + (y1i - x1i) / I.delta);
          vst(Zj + n + i, x1i);
        }
      } break;
      case KIND_CI_OMEGA: {  // M omega_0 = -K psi_0
        const double kp = row_dot<double>(pv, sl, lane, I.m.K, I.xk + n);
        rhs = -kp;
      } break;
      case KIND_CI_MU: {  // M mu_0 = (1+r) M psi_0 - 2 K psi_0 - K omega_0 + g(psi_0)
        const int base = pv.base(sl);
        const int w = pv.width(sl);
        double sMp = 0, sKp = 0, sKo = 0;
        for (int k = 0; k < w; ++k) {
          const long long e = (long long)base + k * 64 + lane;
          const int j = pv.at(e, i);
          sMp += I.m.M[e] * I.xk[n + j];
          sKp += I.m.K[e] * I.xk[n + j];
          sKo += I.m.K[e] * I.xk[2 * n + j];
        }
        rhs = (1.0 + I.r) * sMp - 2.0 * sKp - sKo +
              node_psi3<L != PFC_COL_GRID>(I.m, sl, lane, [&](int j) { return I.xk[n + j]; });
      } break;
    }
    if (i < n) {
      const T rT = T(rhs);
      vst(r + i, rT);
      vst(o.x + i, T(0));
      const double rd = (double)rT;
      a0 += rd * ((double)o.dinv[i] * rd);
      a1 += rd * rd;
    }
  }
  return red3(a0, a1);
}

// p_j = D^{-1}_j r_j + beta p_old_j, evaluated identically wherever needed
template <typename T>
__device__ __forceinline__ T pval(const T* dinv, const T* r, const T* pold, T beta, bool first, int j) {
  const T z = dinv[j] * r[j];
  return first ? z : (z + beta * pold[j]);
}

template <typename T, int L>
__device__ __forceinline__ Red3 ph_pcg_a(const InstDev& I, const State& S, const Team& tm) {
  const int n = I.n;
  PcgOps<T> o = pcg_ops<T>(I, S.kind);
  const PatView<L> pv = op_pat<L>(I, o, tm);
  const T* r = (const T*)I.r_;
  const T* pold = (const T*)(S.pcur ? I.pB : I.pA);
  T* pnew = (T*)(S.pcur ? I.pA : I.pB);
  T* q = (T*)I.q;
  const bool first = (S.it == 0);
  const T beta = T(S.beta_cg);
  double a0 = 0.0;
  PFC_SLICES(I, tm) {
    const int i = sl * 64 + tm.lane;
    const int base = pv.base(sl);
    const int w = pv.width(sl);
    T acc = T(0);
    for_width(w, [&](int k) {
      const long long e = (long long)base + k * 64 + tm.lane;
      const int j = pv.at(e, i);
      acc += opval(o, e) * pval(o.dinv, r, pold, beta, first, j);
    });
    if (i < n) {
      const T pi = pval(o.dinv, r, pold, beta, first, i);
      vst(pnew + i, pi);
      vst(q + i, acc);
      a0 += (double)pi * (double)acc;
    }
  }
  return red3(a0, 0.0);
}

template <typename T>
__device__ __forceinline__ Red3 ph_pcg_b(const InstDev& I, const State& S, const Team& tm) {
  const int n = I.n;
  PcgOps<T> o = pcg_ops<T>(I, S.kind);
  T* r = (T*)I.r_;
  const T* p = (const T*)(S.pcur ? I.pB : I.pA);
  const T* q = (const T*)I.q;
  const T alpha = T(S.alpha);
  double a0 = 0.0, a1 = 0.0;
  PFC_SLICES(I, tm) {
    const int i = sl * 64 + tm.lane;
    if (i < n) {
      const T xi = o.x[i] + alpha * p[i];
      const T ri = r[i] - alpha * q[i];
      vst(o.x + i, xi);
      vst(r + i, ri);
      const double rd = (double)ri;
      a0 += rd * rd;
      a1 += rd * ((double)o.dinv[i] * rd);
    }
  }
  return red3(a0, a1);
}

// ---- outer block operator ------------------------------------------------------
// (A y)_i for the three block rows at node i:
//   w0 = M mu + (-(1+r) M + 2K + N) psi + K omega
//   w1 = t K mu + s M psi
//   w2 = K psi + M omega
//   PFC1 (MOB): w1 = t K_+ mu + s M psi + t F psi
template <typename X2>
struct BlockVec {  // mu and psi in one vector, omega in another (of X2)
  const double* v;
  const X2* om;
};
template <int L, bool MOB, typename X2>
__device__ __forceinline__ void block_row(const InstDev& I, const PatView<L>& pv, int sl, int lane, double t, double s,
                                          BlockVec<X2> y, double& w0, double& w1, double& w2) {
  const double c1 = -(1.0 + I.r);
  const int base = pv.base(sl);
  constexpr bool S = scalar_steps<X2, L>();
  const auto M = slice_vals<S>(I.m.M, base, lane), K = slice_vals<S>(I.m.K, base, lane), N = slice_vals<S>((const double*)I.N, base, lane);
  const auto Kp = slice_vals<S>((const double*)I.Kp, MOB ? base : 0, lane), Fm = slice_vals<S>((const double*)I.Fm, MOB ? base : 0, lane);
  const double* mu = uni(y.v);
  const double* ps = uni(y.v + I.n);
  const X2* om = uni(y.om);
  struct Term {
    double M, K, N, Kp, Fm, mu, ps;
    X2 om;
  };
  w0 = w1 = w2 = 0.0;
  row_entries<ChunkBlock>(pv, sl, lane, [&](auto k, int j) {
    return Term{M(k), K(k), N(k), MOB ? Kp(k) : 0.0, MOB ? Fm(k) : 0.0, vat(mu, j), vat(ps, j), vat(om, j)};
  }, [&](const Term& q) {
    const double qo = (double)q.om;
    w0 += q.M * q.mu + (c1 * q.M + 2.0 * q.K + q.N) * q.ps + q.K * qo;
    if constexpr (MOB) w1 += t * q.Kp * q.mu + s * q.M * q.ps + t * q.Fm * q.ps;
    else w1 += t * q.K * q.mu + s * q.M * q.ps;
    w2 += q.K * q.ps + q.M * qo;
  });
}

__device__ __forceinline__ Red3 ph_update_x(const InstDev& I, const State& S, const Team& tm, const double* y) {
  const int n = I.n;
  const long long n3 = 3LL * n;
  double* X = (S.job == JOB_RB) ? (I.ys + (long long)(S.stage - 1) * n3) : I.x_user;
  const int kc = S.kcols;
  PFC_SLICES(I, tm) {
    const int i = sl * 64 + tm.lane;
    if (i < n) {
      for (int blk = 0; blk < 3; ++blk) {
        const long long o = (long long)blk * n + i;
        double x = X[o];
        for (int l = 0; l < kc; ++l) x += y[l] * I.Z[(long long)l * n3 + o];
        vst(X + o, x);
      }
    }
  }
  return red3(0.0, 0.0);
}

template <int L, bool MOB>
__device__ __forceinline__ Red3 ph_true_res(const InstDev& I, const State& S, const Team& tm) {
  const int n = I.n;
  const PatView<L> pv = p1_pat<L>(I, tm);
  const long long n3 = 3LL * n;
  const bool rb = __builtin_amdgcn_readfirstlane(S.job) == JOB_RB;
  const double* X = rb ? (I.ys + (long long)(S.stage - 1) * n3) : I.x_user;
  const double* bsrc = rb ? I.b : I.b_user;
  const double im = I.rs;
  double a0 = 0.0, a1 = 0.0;
  PFC_SLICES(I, tm) {
    const int i = sl * 64 + tm.lane;
    double w0, w1, w2;
    block_row<L, MOB, double>(I, pv, sl, tm.lane, I.tau, I.m11, {X, X + 2LL * n}, w0, w1, w2);
    if (i < n) {
      const double r0 = bsrc[i] - w0, r1 = bsrc[n + i] - w1, r2 = bsrc[2 * n + i] - w2;
      const double rs1 = r1 * im;
      vst(I.W + i, r0); vst(I.W + n + i, rs1); vst(I.W + 2 * n + i, r2);
      a0 += r0 * r0 + r1 * r1 + r2 * r2;
      a1 += r0 * r0 + rs1 * rs1 + r2 * r2;
    }
  }
  return red3(a0, a1);
}

template <typename T>
__device__ __forceinline__ Red3 ph_pch_out(const InstDev& I, const Team& tm) {
  const int n = I.n;
  const T* x2 = (const T*)I.x2;
  PFC_SLICES(I, tm) {
    const int i = sl * 64 + tm.lane;
    if (i < n) {
      I.pch_out[i] = I.Z[i];
      I.pch_out[n + i] = I.Z[n + i];
      I.pch_out[2 * n + i] = (double)x2[i];
    }
  }
  return red3(0.0, 0.0);
}

// ---- single-reduction Jacobi PCG (Chronopoulos-Gear form) ----------------------
// Same iterates as the standard PCG in exact arithmetic, with the two inner
// products of an iteration taken in one reduction:
//   s_i = w_i + beta_i s_{i-1},  p_i = u_i + beta_i p_{i-1},
//   x_{i+1} = x_i + alpha_i p_i, r_{i+1} = r_i - alpha_i s_i, u = D^{-1} r, w = C u,
//   gamma = (r, u), delta = (w, u), beta_{i+1} = gamma_{i+1}/gamma_i,
//   alpha_{i+1} = gamma_{i+1} / (delta_{i+1} - beta_{i+1} gamma_{i+1} / alpha_i).
// u_{i+1} at gathered neighbours is recomputed from r_i, w_i, s_{i-1}; r, w, s
// are double-buffered, p and x are updated in place by their owners.
// What an iteration gathers of a row j: r, w, s and d = D^{-1}.  In float they stand side
// by side, 16 bytes a row in two buffers of two vectors each (RA: rB, wB; RB: sA, sB): one
// load an entry instead of four, the address units being what bounds the gathers of
// the long rows (P2 256^2 mixed stage solve 42.6 -> 36.2 ms, 3D 48^3 mixed step 22.0 ->
// 20.4).  In float64 each is a vector of its own: side by side the rows would be 24 or 32
// bytes apart, and measured slower (P2 256^2: 55.0 ms, at 24 bytes 60.3, at 32 59.3; both
// on the grid with its nodes in place, where a solve takes fewer iterations than on
// the moved nodes of the figures below).
typedef float Float4 __attribute__((ext_vector_type(4)));
typedef unsigned UInt4 __attribute__((ext_vector_type(4)));
template <typename T>
struct CgRow {
  T d, r, w, s;
};
template <typename T>
struct CgBufs {  // float64
  const T *r, *w, *s, *dinv;
  __device__ __forceinline__ CgRow<T> operator()(int j) const { return CgRow<T>{vat(dinv, j), vat(r, j), vat(w, j), vat(s, j)}; }
};
template <>
struct CgBufs<float> {
  const Float4* q;
  __device__ __forceinline__ CgRow<float> operator()(int j) const {
    const Float4 v = gld(q + j);
    return CgRow<float>{v.w, v.x, v.y, v.z};
  }
};
// row sl * 64 + lane of such a buffer (write-through, as vst)
__device__ __forceinline__ void cg_row_store(void* q, int sl, int lane, float r, float w, float s, float d) {
  const __amdgpu_buffer_rsrc_t b = __builtin_amdgcn_make_buffer_rsrc((char*)q + (long long)sl * 1024, 0, 1024, 0x00027000);
  const UInt4 v = {__float_as_uint(r), __float_as_uint(w), __float_as_uint(s), __float_as_uint(d)};
  __builtin_amdgcn_raw_buffer_store_b128(v, b, lane * 16, 0, 16);  // sc1
}

template <typename T, int L>
__device__ __forceinline__ Red3 ph_cg_init(const InstDev& I, const State& S, const Team& tm) {
  const int n = I.n;
  PcgOps<T> o = pcg_ops<T>(I, S.kind);
  const PatView<L> pv = op_pat<L>(I, o, tm);
  const T* r = uni((const T*)I.r_);
  T* w = uni((T*)I.q);
  double a0 = 0.0, a1 = 0.0, a2 = 0.0;
  struct Term {
    T a, d, r;
  };
  PFC_SLICES(I, tm) {
    const int i = sl * 64 + tm.lane;
    T acc = T(0);
    op_entries<ChunkInit>(o, pv, sl, tm.lane, [&](T a, int j) { return Term{a, vat(o.dinv, j), vat(r, j)}; },
                  [&](const Term& t) { acc += t.a * (t.d * t.r); });
    if (i < n) {
      const unsigned oi = (unsigned)i * (unsigned)sizeof(T);
      const T ri = gldo(r, oi), di = gldo(o.dinv, oi), u = di * ri;
      if constexpr (sizeof(T) == 4) cg_row_store(uni(I.rB), sl, tm.lane, ri, acc, acc, di);  // (s: read times beta = 0)
      else vsto(w, oi, acc);
      a0 += (double)ri * (double)u;
      a1 += (double)acc * (double)u;
      a2 += (double)ri * (double)ri;
    }
  }
  return red3(a0, a1, a2);
}

// One iteration.  Bound by the round trips of the gathers (four vectors at every
// neighbour), so the columns of a row are loaded at once and its entries in chunks
// that the registers hold (ChunkIter; in float64 4 of the 19 entries of a P2 vertex row:
// 5 + 1 round trips instead of 14; 5 of the 9 of an edge row: 2 + 1): P2 256^2 float64
// solve, nodes moved by up to 0.2 cells, 80.6 -> 65.4 ms.
template <typename T, int L>
__device__ __forceinline__ Red3 ph_cg_iter(const InstDev& I, const State& S, const Team& tm) {
  const int n = I.n;
  PcgOps<T> o = pcg_ops<T>(I, S.kind);
  const PatView<L> pv = op_pat<L>(I, o, tm);
  const int c = __builtin_amdgcn_readfirstlane(S.cur);
  constexpr bool AOS = sizeof(T) == 4;
  const T *rc, *wc;
  T *rn, *wn, *sn;
  if constexpr (!AOS) {
    rc = uni((const T*)(c ? I.rB : I.r_));
    rn = uni((T*)(c ? I.r_ : I.rB));
    wc = uni((const T*)(c ? I.wB : I.q));
    wn = uni((T*)(c ? I.q : I.wB));
    sn = uni((T*)(c ? I.sA : I.sB));
  }
  T* p = uni((T*)I.pA);
  // the first iteration has no previous s (s = w + 0 w) and no previous p
  const bool first = __builtin_amdgcn_readfirstlane(S.it) == 0;
  CgBufs<T> in;
  if constexpr (AOS) in.q = uni((const Float4*)(c ? I.sA : I.rB));
  else in = CgBufs<T>{rc, wc, first ? wc : uni((const T*)(c ? I.sB : I.sA)), o.dinv};
  const T alpha = T(S.alpha), beta = first ? T(0) : T(S.beta_cg);
  double a0 = 0.0, a1 = 0.0, a2 = 0.0;
  struct Term {
    T a;
    CgRow<T> v;
  };
  auto s_of = [&](T w, T s) { return w + beta * s; };
  PFC_SLICES(I, tm) {
    const int i = sl * 64 + tm.lane;
    const unsigned oi = (unsigned)(i < n ? i : n - 1) * (unsigned)sizeof(T);
    const CgRow<T> own = in(i < n ? i : n - 1);
    const T di = own.d, ro = own.r, po = gldo((const T*)p, oi), xo = gldo((const T*)o.x, oi);
    T acc = T(0);
    op_entries<ChunkIter<T>>(
        o, pv, sl, tm.lane, [&](T a, int j) { return Term{a, in(j)}; },
        [&](const Term& t) { acc += t.a * (t.v.d * (t.v.r - alpha * s_of(t.v.w, t.v.s))); });
    if (i < n) {
      const T si = s_of(own.w, own.s);
      const T uo = di * ro;
      const T pi = first ? uo : (uo + beta * po);
      vsto(o.x, oi, T(xo + alpha * pi));
      const T ri = ro - alpha * si;
      const T ui = di * (ro - alpha * si);
      if constexpr (!AOS) vsto(sn, oi, si);
      vsto(p, oi, pi);
      if constexpr (AOS) {
        cg_row_store(uni(c ? I.rB : I.sA), sl, tm.lane, ri, acc, si, di);
      } else {
        vsto(rn, oi, ri);
        vsto(wn, oi, acc);
      }
      a0 += (double)ri * (double)ui;
      a1 += (double)acc * (double)ui;
      a2 += (double)ri * (double)ri;
    }
  }
  return red3(a0, a1, a2);
}

// ---- two Jacobi-PCG iterations per launch (s-step form, s = 2) ---------------
// With T = D^{-1} C (D = diag C) the Jacobi PCG is CG for T in the D-weighted
// inner product <a, b> = a^T D b: u = D^{-1} r, (r, u) = <u, u>, (p, C p) =
// <p, T p>, ||r||^2 = u^T D^2 u.  From the basis B = [p, Tp, T^2 p, u, Tu] of a
// launch, the next two iterates are combinations of B whose coefficients follow
// from the Gram matrices G = B^T D B and H = B'^T D^2 B' (B' = [Tp, T^2 p, u,
// Tu]), so one reduction serves two iterations.  A launch forms the new p, u as
// such combinations on its own rows and on the rows two (p) or one (u) stencil
// steps around them, keeps them in LDS, and applies T there: Tp on the rows one
// step around, T^2 p and Tu on its own rows.  The halo is a contiguous range of
// rows (mod n) on 2D periodic grids, whose neighbours lie within N + 1 rows.
#define PFC_SS_NG 26  // 15 entries of G, 10 of H, and ||b||^2 in the first launch of a solve
#define PFC_SS_NA 4   // passes of a workgroup over the two-step halo (R + 4H <= 4096 rows)
// passes of launches on more workgroups than the team's (at most 512 own rows; grids of
// side 362 at most): half the basis registers of four, and waves without rows in a
// pass skip it.  2D 100^2 float64, one slice a workgroup: 11.9 -> 8.7 us a launch
// (sums over the prefetched Gram partials 3.1 -> 1.4, new p and u 2.8 -> 1.5)
#define PFC_SS_NA_SPREAD 2
#define PFC_SS_NB 3   // passes over the one-step halo (R + 2H <= 3072 rows); 7 entries per row
__shared__ double pfc_ssred[64 * 32];
#ifdef PFC_TICK_TIMING
__shared__ unsigned long long pfc_sst[6];  // optional instrumentation (separate build only)
#define PFC_SS_STAMP(k) \
  if (threadIdx.x == 0) pfc_sst[k] = wall_clock64()
#else
#define PFC_SS_STAMP(k)
#endif

// Workgroup barrier that orders LDS only: the global loads and stores of the
// two-iterations-per-launch phase are never read back within the launch, so
// loads issued ahead stay in flight across it (a full __syncthreads would wait
// for every outstanding memory operation).
__device__ __forceinline__ void lds_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

template <int CTRL>
__device__ __forceinline__ double ss_dppx(double a, double b, bool upper) {
  return (upper ? b : a) + dpp_f64<CTRL, 0xf>(upper ? a : b);
}
// Sums of 32 values over the 64 lanes of a wave by recursive halving (32 value
// exchanges in all instead of 6 per value): the total of value idx ends in lanes
// 2m and 2m + 1 with idx = 16 [l >= 32] + 8 [row odd] + 4 [l mod 16 >= 8] +
// 2 [l mod 8 >= 4] + [l & 2].  Returns the total of the lane's idx.
__device__ __forceinline__ double ss_wave_sums32(const double* v, int lane) {
  double w16[16], w8[8], w4[4], w2[2];
#pragma unroll
  for (int k = 0; k < 16; ++k) w16[k] = ss_swap<false>(v[k], v[k + 16]);
#pragma unroll
  for (int k = 0; k < 8; ++k) w8[k] = ss_swap<true>(w16[k], w16[k + 8]);
#pragma unroll
  for (int k = 0; k < 4; ++k) w4[k] = ss_dppx<0x140>(w8[k], w8[k + 4], (lane & 15) >= 8);  // row_mirror
#pragma unroll
  for (int k = 0; k < 2; ++k) w2[k] = ss_dppx<0x141>(w4[k], w4[k + 2], (lane & 7) >= 4);   // row_half_mirror
  const double w1 = ss_dppx<0x4e>(w2[0], w2[1], (lane & 2) != 0);                          // quad_perm [2,3,0,1]
  return w1 + dpp_f64<0xb1, 0xf>(w1);                                                      // quad_perm [1,0,3,2]
}
__device__ __forceinline__ int ss_wave_sums32_index(int lane) {
  return (lane >= 32 ? 16 : 0) + (((lane >> 4) & 1) ? 8 : 0) + ((lane & 15) >= 8 ? 4 : 0) + ((lane & 7) >= 4 ? 2 : 0) +
         ((lane & 2) ? 1 : 0);
}

__device__ __forceinline__ int ss_wrap(int g, int n) { return g < 0 ? g + n : (g >= n ? g - n : g); }
// offset j - g of a neighbour as a step within the grid (|step| <= N + 1 < n / 2)
__device__ __forceinline__ int ss_step(int d, int n) { return d > (n >> 1) ? d - n : (d < -(n >> 1) ? d + n : d); }

// upper-triangle index of (i, j), i <= j, in a k x k symmetric matrix
__host__ __device__ __forceinline__ int ss_tri(int i, int j, int k) { return i * k - i * (i - 1) / 2 + (j - i); }

// Rows of a workgroup in the two-iterations-per-launch form: own rows [lo, lo + R)
// (at most PFC_WG), halo H; thread tid's passes over the two-step halo are
// q = tid + c PFC_WG, and its own row (if any) is pass position qo.
struct SsRows {
  int lo, R, H, L1, L2, qo, go;
  bool own;
};
__device__ __forceinline__ SsRows ss_rows(const InstDev& I, int rank, int size) {
  SsRows w;
  const int n = I.n;
  const int spw = (I.m.n_slices + size - 1) / size;
  w.lo = min(rank * spw * 64, n);
  w.R = min(w.lo + spw * 64, n) - w.lo;
  w.H = I.sH;
  w.L1 = w.R + 2 * w.H;
  w.L2 = w.R + 4 * w.H;
  const int tid = threadIdx.x;
  w.qo = 2 * w.H + (((tid - 2 * w.H) % PFC_WG) + PFC_WG) % PFC_WG;
  w.own = w.qo < 2 * w.H + w.R;
  w.go = w.lo + (w.qo - 2 * w.H);
  return w;
}

// Loads of the current basis on the two-step halo (and x on the own row), issued
// before the launch's reductions so that their latency overlaps them.
template <int NA>
struct SsPre {
  double bv[NA][5];
  double xo;
};
template <int NA>
__device__ __forceinline__ void ss_load(const InstDev& I, const State& S, const SsRows& w, SsPre<NA>& P, int par) {
  const int n = I.n;
  const long long nn = n;
  const int tid = threadIdx.x;
  const double* bin = I.sbas + (long long)par * 5 * nn;  // the basis of the previous launch
  // (a wave skips the passes in which it has no rows)
  const int first = __builtin_amdgcn_readfirstlane(tid & ~63);
#pragma unroll
  for (int c = 0; c < NA; ++c) {
    if (NA > 2 || first + c * PFC_WG < w.L2) {
      const int g = ss_wrap(w.lo - 2 * w.H + min(tid + c * PFC_WG, w.L2 - 1), n);
#pragma unroll
      for (int k = 0; k < 5; ++k) P.bv[c][k] = gld(bin + k * nn + g);
    }
  }
  P.xo = gld(pcg_ops<double>(I, S.kind).x + min(w.go, n - 1));  // used on the own row only
}

// coef: x increment [0..4], new p [5..9], new u [10..14] over B; S.pcur: x only.
// par: the launch's parity (reads basis [par], writes basis [1 - par]).
template <int L, int NA>
__device__ __forceinline__ void ph_scg(const InstDev& I, const State& S, const Team& tm, const double* coef, bool init,
                                       double* spart_out, const SsRows& w, SsPre<NA>& P, int par) {
  const int n = I.n, H = w.H, R = w.R, L1 = w.L1, L2 = w.L2, lo = w.lo;
  PcgOps<double> o = pcg_ops<double>(I, S.kind);
  const PatView<L> pv = op_pat<L>(I, o, tm);
  const int tid = threadIdx.x, first = __builtin_amdgcn_readfirstlane(tid & ~63);
  const long long nn = n;
  double* bout = I.sbas + (long long)(1 - par) * 5 * nn;
  double bbo = 0.0;  // ||b||^2 over the own rows (first launch of a solve)
  if (init) {
    // the solve's right-hand side b (the set-up of the inner solve, on the own
    // rows and the two-step halo) and u_0 = p_0 = D^{-1} b; x_0 = 0
    const long long n3 = 3 * nn;
    const double* Vj = I.V + (long long)S.j * n3;
    // b = t - s (A v) with, per solve: (1) t = w / ||w||; (2) t = (v_j)_psi, s = tau_p,
    // A v = K y0; (3.1) A v = M y1; (3.2) A v = M z; (5) t = (v_j)_omega, s = 1, A v = K x1
    const int kind = S.kind;
    const double* A = (kind == KIND_Y1 || kind == KIND_X2) ? o.Kv : (kind == KIND_Y0 ? nullptr : o.Mv);
    const double* v = kind == KIND_Y1 ? (const double*)I.y0
                      : kind == KIND_Z ? (const double*)I.y1
                      : kind == KIND_X1 ? (const double*)I.zt
                                        : (const double*)I.x1;
    const double* t = kind == KIND_Y0 ? I.W : (kind == KIND_Y1 ? Vj + nn : (kind == KIND_X2 ? Vj + 2 * nn : nullptr));
    const double ts = kind == KIND_Y0 ? S.vscale : 1.0, sa = kind == KIND_Y1 ? I.tau_p : 1.0;
    double bo = 0.0;
#pragma unroll
    for (int c = 0; c < NA; ++c) {
      if (NA <= 2 && first + c * PFC_WG >= L2) break;
      const int g = ss_wrap(lo - 2 * H + min(tid + c * PFC_WG, L2 - 1), n);
      const int base = (g >> 6) * 64 * 7 + (g & 63);
      double d = 0.0;
      if (A) {
#pragma unroll
        for (int k = 0; k < 7; ++k) {
          const long long e = (long long)base + k * 64;
          d += gld(A + e) * gld(v + pv.at(e, g));
        }
      }
      const double tt = t ? gld(t + g) * ts : 0.0;
      const double b = !A ? tt : (t ? tt - sa * d : d);
      P.bv[c][0] = gld(o.dinv + g);
      P.bv[c][1] = b;
      if (tid + c * PFC_WG == w.qo) bo = b;
    }
    if (w.own) {
      const int g = w.go;
      bbo = bo * bo;
      vst(o.x + g, 0.0);
      if (S.kind == KIND_Y0) {  // the Arnoldi vector v_j = w / ||w||
        double* Vw = (double*)Vj;
        vst(Vw + g, bo);
        vst(Vw + nn + g, gld(I.W + nn + g) * S.vscale);
        vst(Vw + 2 * nn + g, gld(I.W + 2 * nn + g) * S.vscale);
      } else if (S.kind == KIND_X2) {  // (4): z_j = (y0 + (y1 - x1) / delta, x1, x2)
        double* Zj = I.Z + (long long)S.j * n3;
        const double y0i = gld((const double*)I.y0 + g), y1i = gld((const double*)I.y1 + g);
        const double x1i = gld((const double*)I.x1 + g);
        vst(Zj + g, y0i + (y1i - x1i) / I.delta);
        vst(Zj + nn + g, x1i);
      }
    }
  }
  if (!init && __builtin_amdgcn_readfirstlane(S.pcur)) {  // the solve ends within these two iterations: x only
    if (w.own) {
#pragma unroll
      for (int c = 0; c < NA; ++c)
        if (tid + c * PFC_WG == w.qo)
          vst(o.x + w.go, P.xo + (coef[0] * P.bv[c][0] + coef[1] * P.bv[c][1] + coef[3] * P.bv[c][3]));
    }
    return;
  }
  double* sp = pfc_ss;     // new p on [lo - 2H, lo + R + 2H)
  double* su = sp + L2;    // new u on [lo - H, lo + R + H)
  double* stp = su + L1;   // T p on [lo - H, lo + R + H)
#pragma unroll
  for (int c = 0; c < NA; ++c) {
    const int q = tid + c * PFC_WG;
    if (q < L2) {
      const double* b = P.bv[c];
      double pn, un;
      if (init) {
        pn = b[0] * b[1];
        un = pn;
      } else {
        pn = coef[5] * b[0] + coef[6] * b[1] + coef[7] * b[2] + coef[8] * b[3] + coef[9] * b[4];
        un = coef[10] * b[0] + coef[11] * b[1] + coef[12] * b[2] + coef[13] * b[3] + coef[14] * b[4];
      }
      sp[q] = pn;
      if (q >= H && q < H + L1) su[q - H] = un;
      if (q == w.qo && w.own) {
        if (!init) vst(o.x + w.go, P.xo + (coef[0] * b[0] + coef[1] * b[1] + coef[3] * b[3]));
        vst(bout + w.go, pn);
        vst(bout + 3 * nn + w.go, un);
      }
    }
  }
  // operator rows of the one-step halo (at most three passes; the third, if any,
  // holds a few rows of the first wave), in flight across the barrier
  double av[3][7], dv[3];
#pragma unroll
  for (int c = 0; c < 2; ++c) {
    if (NA > 2 || first + c * PFC_WG < L1) {
      const int g = ss_wrap(lo - H + min(tid + c * PFC_WG, L1 - 1), n);
      const int base = (g >> 6) * 64 * 7 + (g & 63);
#pragma unroll
      for (int k = 0; k < 7; ++k) av[c][k] = opval_g(o, (long long)base + k * 64);
      dv[c] = gld(o.dinv + g);
    }
  }
  if (NA > 2 && L1 > 2 * PFC_WG && tid < 64) {
    const int g = ss_wrap(lo - H + min(tid + 2 * PFC_WG, L1 - 1), n);
    const int base = (g >> 6) * 64 * 7 + (g & 63);
#pragma unroll
    for (int k = 0; k < 7; ++k) av[2][k] = opval_g(o, (long long)base + k * 64);
    dv[2] = gld(o.dinv + g);
  }
  lds_barrier();
  PFC_SS_STAMP(0);
  // T p on the one-step halo; T u on the own rows (at most one own row per thread)
  int q1o = -1;
  double tpo = 0.0, tuo = 0.0, dgo = 0.0, dvo = 0.0;
  double ao[7];
  int so[7];  // its entries' steps
#pragma unroll
  for (int k = 0; k < 7; ++k) { ao[k] = 0.0; so[k] = 0; }
  auto trow = [&](int q1, const double* a, double di) {
    const int g = ss_wrap(lo - H + q1, n);
    const bool own = q1 >= H && q1 < H + R;
    const int base = (g >> 6) * 64 * 7 + (g & 63);
    double acc = 0.0, acc2 = 0.0, dg = 0.0;
    int d[7];
#pragma unroll
    for (int k = 0; k < 7; ++k) {
      d[k] = ss_step(pv.at((long long)base + k * 64, g) - g, n);
      acc += a[k] * sp[q1 + H + d[k]];
      dg += d[k] == 0 ? a[k] : 0.0;
    }
    if (own) {
#pragma unroll
      for (int k = 0; k < 7; ++k) acc2 += a[k] * su[q1 + d[k]];
    }
    const double tp = di * acc;
    stp[q1] = tp;
    if (own) {
      q1o = q1; tpo = tp; tuo = di * acc2; dgo = dg; dvo = di;
#pragma unroll
      for (int k = 0; k < 7; ++k) { ao[k] = a[k]; so[k] = d[k]; }
      vst(bout + nn + g, tpo);
      vst(bout + 4 * nn + g, tuo);
    }
  };
#pragma unroll
  for (int c = 0; c < 2; ++c)
    if (tid + c * PFC_WG < L1) trow(tid + c * PFC_WG, av[c], dv[c]);
  if (NA > 2 && tid + 2 * PFC_WG < L1) {  // third pass (at most PFC_SS_NB)
    if (tid < 64) {
      trow(tid + 2 * PFC_WG, av[2], dv[2]);
    } else {
      const int q1 = tid + 2 * PFC_WG;
      const int g = ss_wrap(lo - H + q1, n);
      const int base = (g >> 6) * 64 * 7 + (g & 63);
      double a3[7];
#pragma unroll
      for (int k = 0; k < 7; ++k) a3[k] = opval_g(o, (long long)base + k * 64);
      trow(q1, a3, gld(o.dinv + g));
    }
  }
  lds_barrier();
  PFC_SS_STAMP(1);
  double gp[PFC_SS_NG];
#pragma unroll
  for (int m = 0; m < PFC_SS_NG; ++m) gp[m] = 0.0;
  if (q1o >= 0) {
    const int g = lo + (q1o - H);
    double acc = 0.0;
#pragma unroll
    for (int k = 0; k < 7; ++k) acc += ao[k] * stp[q1o + so[k]];
    const double ttp = dvo * acc;
    vst(bout + 2 * nn + g, ttp);
    const double v[5] = {sp[q1o + H], tpo, ttp, su[q1o], tuo};
#pragma unroll
    for (int i = 0; i < 5; ++i) {
      const double di = dgo * v[i];
#pragma unroll
      for (int j = i; j < 5; ++j) gp[ss_tri(i, j, 5)] = di * v[j];
    }
#pragma unroll
    for (int i = 1; i < 5; ++i) {
      const double di = dgo * dgo * v[i];
#pragma unroll
      for (int j = i; j < 5; ++j) gp[15 + ss_tri(i - 1, j - 1, 4)] = di * v[j];
    }
  }
  gp[25] = bbo;
  PFC_SS_STAMP(2);
  // workgroup sums, fixed order: over each wave by recursive halving, then over
  // the waves
  const int lane = tid & 63, wave = tid >> 6;
  {
    double v32[32];
#pragma unroll
    for (int m = 0; m < 32; ++m) v32[m] = m < PFC_SS_NG ? gp[m] : 0.0;
    const double tot = ss_wave_sums32(v32, lane);
    const int idx = ss_wave_sums32_index(lane);
    if ((lane & 1) == 0) pfc_ssred[wave * 32 + idx] = tot;
  }
  lds_barrier();
  if (tid < PFC_SS_NG) {
    double t = 0.0;
#pragma unroll
    for (int w = 0; w < PFC_WAVES; ++w) t += pfc_ssred[w * 32 + tid];
    vst(spart_out + (long long)tm.rank * 32 + tid, t);
  }
  PFC_SS_STAMP(3);
}

// Sum of the Gram partials of a team ([size][32], fixed order) into g[0..25]:
// the first 8 x 32 partials come from loads issued in the launch's prologue,
// before its phase is known, with the state loads (unconditional loads at
// clamped positions, masked in the sum; from fallback[0] where part is null,
// values then unused); teams of more than 256 add the rest here.
#define PFC_SS_GL 8
__device__ __forceinline__ void ss_gram_prefetch(const double* part, const double* fallback, int size, double* pl) {
  const int tid = threadIdx.x, v = tid & 31, grp = tid >> 5;
#pragma unroll
  for (int c = 0; c < PFC_SS_GL; ++c) {
    const int k = min(grp + 32 * c, size - 1);
    pl[c] = gld(part ? part + (long long)k * 32 + min(v, PFC_SS_NG - 1) : fallback);
  }
}
__device__ __forceinline__ void ss_gram(const double* part, int size, const double* pl, double* g) {
  const int tid = threadIdx.x, v = tid & 31, grp = tid >> 5;
  double s = 0.0;
#pragma unroll
  for (int c = 0; c < PFC_SS_GL; ++c) s += (v < PFC_SS_NG && grp + 32 * c < size) ? pl[c] : 0.0;
  if (v < PFC_SS_NG)
    for (int k = grp + 32 * PFC_SS_GL; k < size; k += 32) s += gld(part + (long long)k * 32 + v);
  pfc_ssred[grp * 32 + v] = s;
  lds_barrier();
  // only thread 0 (the transition) reads the totals: the first wave forms them,
  // lane v over groups 0-15 and lane v + 32 over groups 16-31, added across the
  // halves by a permlane32 swap.  Writers and the reader are lanes of that one
  // wave, so a wave barrier between LDS-only fences orders the writes before
  // thread 0's reads (no workgroup barrier needed)
  if (tid < 64) {
    const int half = tid >> 5;
    double t = 0.0;
#pragma unroll
    for (int q = 0; q < 16; ++q) t += pfc_ssred[(half * 16 + q) * 32 + v];
    t = ss_swap<false>(t, t);
    if (tid < PFC_SS_NG) g[tid] = t;
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
  }
}


// Row of a stored operator (or of M + cK), W entries from byte offset off.
template <int W, typename T>
__device__ __forceinline__ void op_row(const PcgOps<T>& o, unsigned off, T* a) {
  if (o.C) {
#pragma unroll
    for (int k = 0; k < W; ++k) a[k] = gldo(o.C, off, k * 64 * (unsigned)sizeof(T));
  } else {
#pragma unroll
    for (int k = 0; k < W; ++k)
      a[k] = gldo(o.Mv, off, k * 64 * (unsigned)sizeof(T)) + o.cK * gldo(o.Kv, off, k * 64 * (unsigned)sizeof(T));
  }
}
// the diagonal entry of such a row, at position k
template <typename T>
__device__ __forceinline__ T op_at(const PcgOps<T>& o, unsigned off, int k) {
  const unsigned e = off + (unsigned)k * 64u * (unsigned)sizeof(T);
  return o.C ? gldo(o.C, e) : gldo(o.Mv, e) + o.cK * gldo(o.Kv, e);
}
// frame steps of the entries of a row of class c: 2D (MeshDev::goff2), 3D (goff3)
struct Steps2 {
  unsigned long long w;
  __device__ __forceinline__ int operator[](int k) const { return (int)(signed char)(w >> (8 * k)); }
};
__device__ __forceinline__ Steps2 steps2(const MeshDev& m, int c, int f) { return Steps2{m.goff2[c][f]}; }
typedef int Int4 __attribute__((ext_vector_type(4)));
struct Steps3 {
  Int4 a, b;
  __device__ __forceinline__ int operator[](int k) const {
    const int q = k >> 1;
    const int w = q == 0 ? a.x : q == 1 ? a.y : q == 2 ? a.z : q == 3 ? a.w : q == 4 ? b.x : q == 5 ? b.y : q == 6 ? b.z : b.w;
    return (k & 1) ? w >> 16 : (int)(short)w;
  }
};
__device__ __forceinline__ Steps3 steps3(const short* goff3, int c, int f) {
  const unsigned o = (unsigned)(c * 2 + f) * 32u;
  return Steps3{gldo((const Int4*)goff3, o), gldo((const Int4*)goff3, o, 16)};
}

// Gram products of a row's basis values with the diagonal entry dg, their sums over
// the workgroup in fixed order (each wave by recursive halving, then over the waves)
// and the workgroup's partial sums.  Every thread calls this.
template <typename T>
__device__ __forceinline__ void ss_gram_out(T dg, T p, T tp, T ttp, T u, T tu, double bb, double* out) {
  double gp[32];
  const double dgo = (double)dg;
  const double v[5] = {(double)p, (double)tp, (double)ttp, (double)u, (double)tu};
#pragma unroll
  for (int i = 0; i < 5; ++i) {
    const double di = dgo * v[i];
#pragma unroll
    for (int j = i; j < 5; ++j) gp[ss_tri(i, j, 5)] = di * v[j];
  }
#pragma unroll
  for (int i = 1; i < 5; ++i) {
    const double di = dgo * dgo * v[i];
#pragma unroll
    for (int j = i; j < 5; ++j) gp[15 + ss_tri(i - 1, j - 1, 4)] = di * v[j];
  }
  gp[25] = bb;
#pragma unroll
  for (int m = PFC_SS_NG; m < 32; ++m) gp[m] = 0.0;
  PFC_SS_STAMP(2);
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const double tot = ss_wave_sums32(gp, lane);
  if ((lane & 1) == 0) pfc_ssred[wave * 32 + ss_wave_sums32_index(lane)] = tot;
  lds_barrier();
  if (tid < PFC_SS_NG) {
    double t = 0.0;
#pragma unroll
    for (int w = 0; w < PFC_WAVES; ++w) t += pfc_ssred[w * 32 + tid];
    vst(out + tid, t);
  }
  PFC_SS_STAMP(3);
}

// ---- two Jacobi-PCG iterations per launch on 3D periodic grids of side 64 -------
// The s-step iteration of ph_scg with a workgroup's rows a block of the grid
// instead of a range of rows: whole x-lines (64 rows, one SELL slice each) at
// y0..y0+3, z0..z0+3, 1024 rows; rank r has y0 = 4 (r mod 16), z0 = 4 (r / 16).
// The two-step frame is the 8 x 8 lines y0-2..y0+5, z0-2..z0+5, the one-step
// frame the 6 x 6 lines y0-1..y0+4, z0-1..z0+4 (periodic in every direction).  A
// line takes 66 places in LDS, with the row before its first and the one after its
// last (periodic), so a neighbour's place is the row's plus the entry's step, the
// same for every row of a class (MeshDev::goff3).  A wave owns one line, whose basis values
// and operator rows stay in registers; of the 48 lines around the block in the
// two-step frame it takes three, of the 20 in the one-step frame one (waves 0-3
// two), each a whole line: a line's place and addresses are scalars.  New p and u
// are formed on the frames, T p on the one-step frame, T u and T^2 p, the stores
// and the Gram products on the own row.  T is the inner precision (float in
// PFC_MIXED); the Gram sums and the coefficients stay float64.  Bound by the
// instructions issued and the chain of round trips (as ph_scg2b): against passes
// over the frames in thread order, wrapped neighbour places from a direction
// table and a second read of the own rows, 1019 -> 793 vector instructions a wave
// (3D 64^3 mixed step 20.7 -> 17.0 ms).
#define PFC_S3_N 64
#define PFC_S3_L 66  // places of a line
__device__ __forceinline__ int s3_wrap(int v) { return v & (PFC_S3_N - 1); }
struct S3Geo {
  int y0, z0, wave, x;
};
__device__ __forceinline__ S3Geo s3_geo(int rank) {
  return S3Geo{(rank & 15) * 4, (rank >> 4) * 4, __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)),
               (int)(threadIdx.x & 63)};
}
// a line at block coordinates (yl, zl); lb: its first row
struct S3Line {
  int yl, zl, lb;
};
__device__ __forceinline__ S3Line s3_line(const S3Geo& G, int yl, int zl) {
  return S3Line{yl, zl, PFC_S3_N * (s3_wrap(G.y0 + yl) + PFC_S3_N * s3_wrap(G.z0 + zl))};
}
__device__ __forceinline__ S3Line s3_own(const S3Geo& G) { return s3_line(G, G.wave & 3, G.wave >> 2); }
// line c (0..2) of the wave in the ring of the two-step frame
__device__ __forceinline__ S3Line s3_ring2(const S3Geo& G, int c) {
  const int w = G.wave;
  if (c < 2) return s3_line(G, (w & 7) - 2, (w >> 3) + (c ? 4 : -2));
  return s3_line(G, (w & 3) < 2 ? (w & 3) - 2 : (w & 3) + 2, w >> 2);
}
// line q (0..19) of the ring of the one-step frame
__device__ __forceinline__ S3Line s3_ring1(const S3Geo& G, int q) {
  if (q < 12) return s3_line(G, (q < 6 ? q : q - 6) - 1, q < 6 ? -1 : 4);
  return s3_line(G, (q & 1) ? 4 : -1, (q - 12) >> 1);
}
// class (grid_class) of the lane's row of a line
__device__ __forceinline__ int s3_class(const S3Geo& G, const S3Line& l) {
  return grid_edge(G.x, PFC_S3_N) + 3 * grid_edge(s3_wrap(G.y0 + l.yl), PFC_S3_N) +
         9 * grid_edge(s3_wrap(G.z0 + l.zl), PFC_S3_N);
}
// place of the lane's row of a line in the two-step and the one-step frame
__device__ __forceinline__ int s3_p2(const S3Geo& G, const S3Line& l) { return G.x + 1 + PFC_S3_L * (l.yl + 2 + 8 * (l.zl + 2)); }
__device__ __forceinline__ int s3_p1(const S3Geo& G, const S3Line& l) { return G.x + 1 + PFC_S3_L * (l.yl + 1 + 6 * (l.zl + 1)); }
// store at place p and, from the line's ends, at the place beyond its other end
template <typename T>
__device__ __forceinline__ void s3_put(const S3Geo& G, T* f, int p, T v) {
  f[p] = v;
  if (G.x == 0 || G.x == PFC_S3_N - 1) f[G.x == 0 ? p + PFC_S3_N : p - PFC_S3_N] = v;
}

template <typename T>
struct S3Pre {
  T own[5], ring[3][5];
};
// the current basis on the two-step frame, issued before the reductions
template <typename T>
__device__ __forceinline__ void s3_load(const InstDev& I, const State& S, int rank, S3Pre<T>& P, int par) {
  const long long nn = I.n;
  const S3Geo G = s3_geo(rank);
  const T* bin = uni((const T*)I.sbas + (long long)par * 5 * nn);
  const unsigned xo = (unsigned)G.x * (unsigned)sizeof(T);
  const int lo = s3_own(G).lb;
#pragma unroll
  for (int k = 0; k < 5; ++k) P.own[k] = gldo(uni(bin + k * nn + lo), xo);
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    const int lb = s3_ring2(G, c).lb;
#pragma unroll
    for (int k = 0; k < 5; ++k) P.ring[c][k] = gldo(uni(bin + k * nn + lb), xo);
  }
}

template <typename T>
__device__ __forceinline__ void ph_scg3(const InstDev& I, const State& S, const Team& tm, const double* coef, bool init,
                                        double* spart_out, S3Pre<T>& P, int par) {
  constexpr int W15 = 15;
  constexpr unsigned TS = sizeof(T);
  const int n = I.n, tid = threadIdx.x;
  const long long nn = n;
  const S3Geo G = s3_geo(tm.rank);
  const PcgOps<T> o = pcg_ops<T>(I, S.kind);
  T* bout = uni((T*)I.sbas + (long long)(1 - par) * 5 * nn);
  T* sp = (T*)pfc_ss;                  // new p on the two-step frame
  T* su = sp + 64 * PFC_S3_L;          // new u on the one-step frame
  T* stp = su + 36 * PFC_S3_L;         // T p on the one-step frame
  static_assert(136 * PFC_S3_L * sizeof(T) <= sizeof(pfc_ss), "the frames of ph_scg3 exceed the s-step LDS");
  const S3Line lo = s3_own(G);
  const unsigned xo = (unsigned)G.x * TS, xd = (unsigned)G.x * 8u;
  T bo = T(0), dio = T(0), br[3], dir[3];
  if (init) {
    // the solve's right-hand side b on the two-step frame and u_0 = p_0 = D^{-1} b;
    // as ph_scg: b = t - s (A v) by solve kind
    const long long n3 = 3 * nn;
    const double* Vj = uni(I.V + (long long)S.j * n3);
    const int kind = __builtin_amdgcn_readfirstlane(S.kind);
    const T* A = (kind == KIND_Y1 || kind == KIND_X2) ? o.Kv : (kind == KIND_Y0 ? nullptr : o.Mv);
    const T* v = uni(kind == KIND_Y1 ? (const T*)I.y0 : kind == KIND_Z ? (const T*)I.y1 : kind == KIND_X1 ? (const T*)I.zt
                                                                                                          : (const T*)I.x1);
    const double* t = uni(kind == KIND_Y0 ? (const double*)I.W
                                          : (kind == KIND_Y1 ? Vj + nn : (kind == KIND_X2 ? Vj + 2 * nn : nullptr)));
    const double ts = kind == KIND_Y0 ? S.vscale : 1.0, sa = kind == KIND_Y1 ? I.tau_p : 1.0;
    auto rhs = [&](const S3Line& l, T& b, T& di) {
      T d = T(0);
      if (A) {
        const T* Al = A + (long long)l.lb * W15;
        const int* gl = I.m.glin + s3_class(G, l) * PFC_GRID_W;
        const int g = l.lb + G.x;
#pragma unroll 5
        for (int k = 0; k < W15; ++k) d += gldo(Al, xo, k * 64 * TS) * gldo(v, (unsigned)(g + gl[k]) * TS);
      }
      const double tt = t ? gldo(t + l.lb, xd) * ts : 0.0;
      b = T(!A ? tt : (t ? tt - sa * (double)d : (double)d));
      di = gldo(o.dinv + l.lb, xo);
    };
    rhs(lo, bo, dio);
#pragma unroll
    for (int c = 0; c < 3; ++c) rhs(s3_ring2(G, c), br[c], dir[c]);
  } else if (__builtin_amdgcn_readfirstlane(S.pcur)) {  // the solve ends within these two iterations: x only, on the own row
    const double p = P.own[0], tp = P.own[1], u = P.own[3];
    T* x = o.x + lo.lb;
    vsto(x, xo, T((double)gldo((const T*)x, xo) + (coef[0] * p + coef[1] * tp + coef[3] * u)));
    return;
  }
  // the own line's operator row, issued before the new p and u are formed (whose basis
  // loads they wait for); the row of the wave's line of the one-step ring follows when
  // the basis values are used up (both at once would not fit the registers) and is in
  // flight across the barrier and the own line's T p
  T ao[W15], ar[W15], odi, rdi;
  const S3Line l1 = s3_ring1(G, G.wave);
  const short* goff3 = uni(I.m.goff3);
  const unsigned eo = (unsigned)lo.lb * W15 * TS + xo;
  const Steps3 off2 = steps3(goff3, s3_class(G, lo), 1);
  op_row<W15>(o, eo, ao);
  odi = init ? dio : gldo(o.dinv + lo.lb, xo);
  // new p on the two-step frame, new u on the one-step frame
  auto pu = [&](const T* b, T& pn, T& un) {
    pn = T(coef[5] * b[0] + coef[6] * b[1] + coef[7] * b[2] + coef[8] * b[3] + coef[9] * b[4]);
    un = T(coef[10] * b[0] + coef[11] * b[1] + coef[12] * b[2] + coef[13] * b[3] + coef[14] * b[4]);
  };
  T pn, un;
  double dx = 0.0;  // increment of x
  if (init) {
    pn = un = dio * bo;
  } else {
    pu(P.own, pn, un);
    dx = coef[0] * (double)P.own[0] + coef[1] * (double)P.own[1] + coef[3] * (double)P.own[3];
  }
  const int o2 = s3_p2(G, lo), o1 = s3_p1(G, lo);
  s3_put(G, sp, o2, pn);
  s3_put(G, su, o1, un);
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    const S3Line l = s3_ring2(G, c);
    T pr, ur;
    if (init) pr = ur = dir[c] * br[c];
    else pu(P.ring[c], pr, ur);
    s3_put(G, sp, s3_p2(G, l), pr);
    if (l.yl >= -1 && l.yl <= 4 && l.zl >= -1 && l.zl <= 4) s3_put(G, su, s3_p1(G, l), ur);
  }
  __builtin_amdgcn_sched_barrier(0);
  Steps3 offr = steps3(goff3, s3_class(G, l1), 1);
  op_row<W15>(o, (unsigned)l1.lb * W15 * TS + xo, ar);
  rdi = gldo(o.dinv + l1.lb, xo);
  const T dg = op_at(o, eo, off2[15]);
  const T xv = init ? T(0) : gldo((const T*)o.x + lo.lb, xo);
  lds_barrier();
  PFC_SS_STAMP(0);
  const Steps3 off1 = steps3(goff3, s3_class(G, lo), 0);  // (used after the next barrier)
  // T p on the one-step frame
  auto tp_of = [&](const T* a, T di, int p2, const Steps3& off) {
    T acc = T(0);
#pragma unroll
    for (int k = 0; k < W15; ++k) acc += a[k] * sp[p2 + off[k]];
    return T(di * acc);
  };
  const T tpo = tp_of(ao, odi, o2, off2);
  s3_put(G, stp, o1, tpo);
  s3_put(G, stp, s3_p1(G, l1), tp_of(ar, rdi, s3_p2(G, l1), offr));
  if (G.wave < 4) {  // the ring's last four lines
    const S3Line l = s3_ring1(G, 16 + G.wave);
    op_row<W15>(o, (unsigned)l.lb * W15 * TS + xo, ar);
    offr = steps3(goff3, s3_class(G, l), 1);
    s3_put(G, stp, s3_p1(G, l), tp_of(ar, gldo(o.dinv + l.lb, xo), s3_p2(G, l), offr));
  }
  lds_barrier();
  PFC_SS_STAMP(1);
  // own row: T u, T^2 p, the stores and the Gram products
  T au = T(0), att = T(0);
#pragma unroll
  for (int k = 0; k < W15; ++k) {
    const int i1 = o1 + off1[k];
    au += ao[k] * su[i1];
    att += ao[k] * stp[i1];
  }
  const T tuo = odi * au, ttp = odi * att;
  double bbo = 0.0;
  if (init) {
    bbo = (double)bo * (double)bo;
    vsto(o.x + lo.lb, xo, T(0));
    const long long n3 = 3 * nn;
    if (S.kind == KIND_Y0) {  // the Arnoldi vector v_j = w / ||w||
      double* Vw = uni(I.V + (long long)S.j * n3 + lo.lb);
      const double* W = uni(I.W + lo.lb);
#pragma unroll
      for (int blk = 0; blk < 3; ++blk) vsto(Vw + blk * nn, xd, gldo(W + blk * nn, xd) * S.vscale);
    } else if (S.kind == KIND_X2) {  // (4): z_j = (y0 + (y1 - x1) / delta, x1, x2)
      double* Zj = uni(I.Z + (long long)S.j * n3 + lo.lb);
      const double y0i = (double)gldo(uni((const T*)I.y0 + lo.lb), xo), y1i = (double)gldo(uni((const T*)I.y1 + lo.lb), xo);
      const double x1i = (double)gldo(uni((const T*)I.x1 + lo.lb), xo);
      vsto(Zj, xd, y0i + (y1i - x1i) / I.delta);
      vsto(Zj + nn, xd, x1i);
    }
  } else {
    vsto(o.x + lo.lb, xo, T((double)xv + dx));
  }
  vsto(bout + lo.lb, xo, pn);
  vsto(bout + nn + lo.lb, xo, tpo);
  vsto(bout + 2 * nn + lo.lb, xo, ttp);
  vsto(bout + 3 * nn + lo.lb, xo, un);
  vsto(bout + 4 * nn + lo.lb, xo, tuo);
  ss_gram_out(dg, pn, tpo, ttp, un, tuo, bbo, spart_out + (long long)tm.rank * 32);
}

// ---- two Jacobi-PCG iterations per launch on blocks of 2D periodic grids -------
// The iteration of ph_scg3 on a 2D grid of side N, a multiple of 64: rank r
// owns the block of 64 x 16 rows x0 .. x0 + 63, y0 .. y0 + 15 with
// x0 = 64 (r mod N/64), y0 = 16 (r div N/64).  The two-step frame is the
// 68 x 20 rows x0 - 2 .. x0 + 65, y0 - 2 .. y0 + 17, the one-step frame the
// 66 x 18 rows x0 - 1 .. x0 + 64, y0 - 1 .. y0 + 16 (periodic), so a row's
// neighbour in a frame is the row's frame position plus the entry's step, the
// same for every row of a class (MeshDev::goff2).  Against a range of whole grid lines per
// workgroup (ph_scg) the frames hold 1360 and 1188 rows instead of 3076 and 2050
// at N = 512: the basis is read, and p and T p are formed, on fewer rows.
// Thread t owns row x0 + t mod 64, y0 + t / 64 (a wave's own rows are one SELL
// slice), whose basis values and operator row stay in its registers through the
// launch; the rings around the block (336 rows of the two-step frame, 164 of the
// one-step frame, 180 of the three-step frame of a set-up) are second rows of
// waves 0-5, 6-8 and 9-11.  The launch is bound by the instructions its waves
// issue (four waves a SIMD) and by its chain of round trips, not by bytes: frame
// passes over all rows in thread order, with the own row's operator and basis read
// again, division-built coordinates, a direction table in LDS and 64-bit address
// arithmetic per load took 1097 vector instructions a wave, this form 648 (2D
// 512^2 float64: stage solve 13.2 -> 10.0 ms, 128^2 mixed x 64 90.7 -> 71.0 ms a step).
#define PFC_B2_W2 68
#define PFC_B2_N2 (PFC_B2_W2 * 20)  // two-step frame
#define PFC_B2_W1 66
#define PFC_B2_N1 (PFC_B2_W1 * 18)  // one-step frame
#define PFC_B2_W3 70
#define PFC_B2_N3 (PFC_B2_W3 * 22)  // three-step frame (a set-up that also ends the previous solve)
#define PFC_B2_R2 336               // two-step frame rows outside the block: waves 0-5
#define PFC_B2_R1 164               // one-step frame rows outside the block: waves 6-8
#define PFC_B2_R3 180               // three-step frame rows outside the two-step frame: waves 9-11
#define PFC_B2_T2 384
#define PFC_B2_T1 576
#define PFC_B2_T3 768
static_assert(PFC_B2_R2 <= PFC_B2_T2 && PFC_B2_R1 <= PFC_B2_T1 - PFC_B2_T2 && PFC_B2_R3 <= PFC_B2_T3 - PFC_B2_T1 &&
              PFC_B2_T3 <= PFC_WG, "the rings of a 2D block exceed their waves");
struct B2Geo {
  int x0, y0, N;
};
__device__ __forceinline__ B2Geo b2_geo(int rank, int N) {
  const int bx = N >> 6;
  return B2Geo{(rank % bx) * 64, (rank / bx) * 16, N};
}
__device__ __forceinline__ int b2_wrap(int v, int N) { return v < 0 ? v + N : (v >= N ? v - N : v); }
// row at block coordinates (fx, fy), -3 <= fx < 67, -3 <= fy < 19
__device__ __forceinline__ int b2_row(const B2Geo& G, int fx, int fy) {
  return b2_wrap(G.x0 + fx, G.N) + G.N * b2_wrap(G.y0 + fy, G.N);
}
// class (grid_class) of such a row
__device__ __forceinline__ int b2_class(const B2Geo& G, int fx, int fy) {
  return grid_edge(b2_wrap(G.x0 + fx, G.N), G.N) + 3 * grid_edge(b2_wrap(G.y0 + fy, G.N), G.N);
}
// block coordinates of row r of the ring of width d (rows 64 + 2 k wide) around
// the frame k - d steps out: d full lines below, d above, then the sides
template <int K, int D>
__device__ __forceinline__ void b2_ring(int r, int& fx, int& fy) {
  constexpr int W = 64 + 2 * K, L = 2 * D * W;
  if (r < L) {
    const int q = r / W;
    fx = r - W * q - K;
    fy = q < D ? q - K : q - D + 16 + K - D;
  } else {
    const int s = r - L, c = s % (2 * D);
    fy = s / (2 * D) - (K - D);
    fx = c < D ? c - K : 64 + K - 2 * D + c;
  }
}

template <typename T>
struct B2Pre {
  T own[5], ring[5];
};
// the current basis on the own row and on the ring of the two-step frame, issued
// before the reductions
template <typename T>
__device__ __forceinline__ void b2_load(const InstDev& I, int rank, B2Pre<T>& P, int par) {
  const long long nn = I.n;
  const int tid = threadIdx.x;
  const B2Geo G = b2_geo(rank, I.m.gN);
  const T* bin = uni((const T*)I.sbas + (long long)par * 5 * nn);
  const unsigned og = (unsigned)(G.x0 + (tid & 63) + G.N * (G.y0 + (tid >> 6))) * (unsigned)sizeof(T);
#pragma unroll
  for (int k = 0; k < 5; ++k) P.own[k] = gldo(uni(bin + k * nn), og);
  if (tid < PFC_B2_T2) {
    int fx, fy;
    b2_ring<2, 2>(min(tid, PFC_B2_R2 - 1), fx, fy);
    const unsigned g = (unsigned)b2_row(G, fx, fy) * (unsigned)sizeof(T);
#pragma unroll
    for (int k = 0; k < 5; ++k) P.ring[k] = gldo(uni(bin + k * nn), g);
  }
}

// The launch after one that ended a solve in its set-up (State::fuse) stores
// that solve's final x on the own rows: x plus the last increment over the
// basis, which is still the other parity's (this launch writes its own rows'
// basis there only afterwards), as the launch that only adds the increment
// would.
template <typename T>
__device__ __forceinline__ void b2_end_store(const InstDev& I, int rank, int kind, double c0, double c1, double c3,
                                             int par) {
  const long long nn = I.n;
  const int tid = threadIdx.x;
  const B2Geo G = b2_geo(rank, I.m.gN);
  const unsigned og = (unsigned)(G.x0 + (tid & 63) + G.N * (G.y0 + (tid >> 6))) * (unsigned)sizeof(T);
  T* x = pcg_ops<T>(I, kind).x;
  const T* bas = uni((const T*)I.sbas + (long long)(1 - par) * 5 * nn);
  const T xo = gldo(x, og);
  const double p = gldo(bas, og), tp = gldo(uni(bas + nn), og), u = gldo(uni(bas + 3 * nn), og);
  vsto(x, og, T((double)xo + (c0 * p + c1 * tp + c3 * u)));
}

template <typename T>
__device__ __forceinline__ void ph_scg2b(const InstDev& I, const State& S, const Team& tm, const double* coef, bool init,
                                         double* spart_out, B2Pre<T>& P, int par) {
  constexpr int W7 = 7;
  constexpr unsigned TS = sizeof(T);
  const int n = I.n, tid = threadIdx.x;
  const long long nn = n;
  const B2Geo G = b2_geo(tm.rank, I.m.gN);
  const PcgOps<T> o = pcg_ops<T>(I, S.kind);
  T* bout = uni((T*)I.sbas + (long long)(1 - par) * 5 * nn);
  T* sp = (T*)pfc_ss;          // new p on the two-step frame
  T* su = sp + PFC_B2_N2;      // new u on the one-step frame
  T* stp = su + PFC_B2_N1;     // T p on the one-step frame
  T* sv = stp + PFC_B2_N1;     // v on the three-step frame (a set-up that also ends the previous solve)
  static_assert((PFC_B2_N2 + 2 * PFC_B2_N1 + PFC_B2_N3) * sizeof(double) <= sizeof(pfc_ss),
                "the frames of ph_scg2b exceed the s-step LDS");
  // own row: its index, its byte offsets in a vector and in the values, its frame positions
  const int ox = tid & 63, oy = tid >> 6;
  const int gi = G.x0 + ox + G.N * (G.y0 + oy);
  const unsigned og = (unsigned)gi * TS, oe = (unsigned)((gi >> 6) * 64 * W7 + (gi & 63)) * TS;
  const int o1 = (ox + 1) + PFC_B2_W1 * (oy + 1), o2 = (ox + 2) + PFC_B2_W2 * (oy + 2);
  const int o3 = (ox + 3) + PFC_B2_W3 * (oy + 3);
  // the rings' rows
  const bool w2 = tid < PFC_B2_T2, in2 = tid < PFC_B2_R2;
  const bool w1 = tid >= PFC_B2_T2 && tid < PFC_B2_T1, in1 = w1 && tid < PFC_B2_T2 + PFC_B2_R1;
  int rx = 0, ry = 0, rg = 0;
  if (w2) {
    b2_ring<2, 2>(min(tid, PFC_B2_R2 - 1), rx, ry);
    rg = b2_row(G, rx, ry);
  } else if (w1) {
    b2_ring<1, 1>(min(tid - PFC_B2_T2, PFC_B2_R1 - 1), rx, ry);
    rg = b2_row(G, rx, ry);
  }
  const int co = b2_class(G, ox, oy), cr = b2_class(G, rx, ry);  // row classes
  const unsigned rge = (unsigned)((rg >> 6) * 64 * W7 + (rg & 63)) * TS;
  const int r1 = (rx + 1) + PFC_B2_W1 * (ry + 1), r2 = (rx + 2) + PFC_B2_W2 * (ry + 2);
  T x1f = T(0);  // x1 on the own row where this launch ends its solve
  T bo = T(0), dio = T(0), br = T(0), dir = T(0);
  if (init) {
    // the solve's right-hand side b on the two-step frame and u_0 = p_0 = D^{-1} b;
    // as ph_scg: b = t - s (A v) by solve kind
    const long long n3 = 3 * nn;
    const double* Vj = uni(I.V + (long long)S.j * n3);
    const int kind = __builtin_amdgcn_readfirstlane(S.kind);
    const T* A = (kind == KIND_Y1 || kind == KIND_X2) ? o.Kv : (kind == KIND_Y0 ? nullptr : o.Mv);
    const T* v = uni(kind == KIND_Y1 ? (const T*)I.y0 : kind == KIND_Z ? (const T*)I.y1 : kind == KIND_X1 ? (const T*)I.zt
                                                                                                          : (const T*)I.x1);
    const double* t = uni(kind == KIND_Y0 ? (const double*)I.W
                                          : (kind == KIND_Y1 ? Vj + nn : (kind == KIND_X2 ? Vj + 2 * nn : nullptr)));
    const double ts = kind == KIND_Y0 ? S.vscale : 1.0, sa = kind == KIND_Y1 ? I.tau_p : 1.0;
    const bool fz = __builtin_amdgcn_readfirstlane(S.fuse) != 0;
    if (fz) {
      // the previous solve (the P_CH step before, whose x is this solve's v) ends
      // in this launch: its x plus the last increment, formed on the three-step
      // frame; x itself stays unchanged here (other workgroups read it on their
      // halos) and is stored by the next launch (b2_end_store)
      const T* xp = pcg_ops<T>(I, S.fkind).x;
      const double c0 = coef[0], c1 = coef[1], c3 = coef[3];
      // (the basis loads issued ahead are not used here: held for this path they would
      // be live through every other phase's code)
      const T* bold = uni((const T*)I.sbas + (long long)par * 5 * nn);
      const T *b1 = uni(bold + nn), *b3 = uni(bold + 3 * nn);
      auto fin = [&](unsigned q) {
        const double p = gldo(bold, q), tp = gldo(b1, q), u = gldo(b3, q);
        return T((double)gldo(xp, q) + (c0 * p + c1 * tp + c3 * u));
      };
      x1f = fin(og);
      sv[o3] = x1f;
      if (w2) {
        const T xr = fin((unsigned)rg * TS);
        if (in2) sv[(rx + 3) + PFC_B2_W3 * (ry + 3)] = xr;
      } else if (tid >= PFC_B2_T1 && tid < PFC_B2_T3) {
        int qx, qy;
        b2_ring<3, 1>(min(tid - PFC_B2_T1, PFC_B2_R3 - 1), qx, qy);
        const T xr = fin((unsigned)b2_row(G, qx, qy) * TS);
        if (tid < PFC_B2_T1 + PFC_B2_R3) sv[(qx + 3) + PFC_B2_W3 * (qy + 3)] = xr;
      }
      lds_barrier();
    }
    auto rhs = [&](int g, unsigned e, int c, int q3, T& b, T& di) {
      T d = T(0);
      if (A) {
        T a[W7];
#pragma unroll
        for (int k = 0; k < W7; ++k) a[k] = gldo(A, e, k * 64 * TS);
        if (fz) {
          const Steps2 off3 = steps2(I.m, c, 2);
#pragma unroll
          for (int k = 0; k < W7; ++k) d += a[k] * sv[q3 + off3[k]];
        } else {
          const int* gl = I.m.glin + c * PFC_GRID_W;
#pragma unroll
          for (int k = 0; k < W7; ++k) d += a[k] * gldo(v, (unsigned)(g + gl[k]) * TS);
        }
      }
      const double tt = t ? gldo(t, (unsigned)g * 8u) * ts : 0.0;
      b = T(!A ? tt : (t ? tt - sa * (double)d : (double)d));
      di = gldo(o.dinv, (unsigned)g * TS);
    };
    rhs(gi, oe, co, o3, bo, dio);
    if (w2) rhs(rg, rge, cr, (rx + 3) + PFC_B2_W3 * (ry + 3), br, dir);
  } else if (__builtin_amdgcn_readfirstlane(S.pcur)) {  // the solve ends within these two iterations: x only, on the own row
    const double p = P.own[0], tp = P.own[1], u = P.own[3];
    vsto(o.x, og, T((double)gldo(o.x, og) + (coef[0] * p + coef[1] * tp + coef[3] * u)));
    return;
  }
  // operator rows of the own row and of the one-step ring, issued before the new p
  // and u are formed (whose basis loads they wait for) and in flight across the barrier
  T ao[W7], ar[W7], odi, rdi = T(0);
  op_row<W7>(o, oe, ao);
  odi = init ? dio : gldo(o.dinv, og);
  if (w1) {
    op_row<W7>(o, rge, ar);
    rdi = gldo(o.dinv, (unsigned)rg * TS);
  }
  // new p on the two-step frame, new u on the one-step frame
  auto pu = [&](const T* b, T& pn, T& un) {
    pn = T(coef[5] * b[0] + coef[6] * b[1] + coef[7] * b[2] + coef[8] * b[3] + coef[9] * b[4]);
    un = T(coef[10] * b[0] + coef[11] * b[1] + coef[12] * b[2] + coef[13] * b[3] + coef[14] * b[4]);
  };
  T pn, un;
  double dx = 0.0;  // increment of x
  if (init) {
    pn = un = dio * bo;
  } else {
    pu(P.own, pn, un);
    dx = coef[0] * (double)P.own[0] + coef[1] * (double)P.own[1] + coef[3] * (double)P.own[3];
  }
  sp[o2] = pn;
  su[o1] = un;
  if (w2) {
    T pr, ur;
    if (init) pr = ur = dir * br;
    else pu(P.ring, pr, ur);
    if (in2) {
      sp[r2] = pr;
      if (rx >= -1 && rx < 65 && ry >= -1 && ry < 17) su[r1] = ur;
    }
  }
  const Steps2 off1 = steps2(I.m, co, 0);
  const T dg = op_at(o, oe, off1[7]);
  const T xo = init ? T(0) : gldo(o.x, og);
  lds_barrier();
  PFC_SS_STAMP(0);
  // T p on the one-step frame
  auto tp_of = [&](const T* a, T di, int c, int q2) {
    const Steps2 off2 = steps2(I.m, c, 1);
    T acc = T(0);
#pragma unroll
    for (int k = 0; k < W7; ++k) acc += a[k] * sp[q2 + off2[k]];
    return T(di * acc);
  };
  const T tpo = tp_of(ao, odi, co, o2);
  stp[o1] = tpo;
  if (w1) {
    const T tpr = tp_of(ar, rdi, cr, r2);
    if (in1) stp[r1] = tpr;
  }
  lds_barrier();
  PFC_SS_STAMP(1);
  // own row: T u, T^2 p, the stores and the Gram products
  T au = T(0), att = T(0);
#pragma unroll
  for (int k = 0; k < W7; ++k) {
    const int i1 = o1 + off1[k];
    au += ao[k] * su[i1];
    att += ao[k] * stp[i1];
  }
  const T tuo = odi * au, ttp = odi * att;
  double bbo = 0.0;
  if (init) {
    bbo = (double)bo * (double)bo;
    vsto(o.x, og, T(0));
    const long long n3 = 3 * nn;
    const unsigned od = (unsigned)gi * 8u;
    if (S.kind == KIND_Y0) {  // the Arnoldi vector v_j = w / ||w||
      double* Vw = uni(I.V + (long long)S.j * n3);
      const double* W = uni(I.W);
#pragma unroll
      for (int blk = 0; blk < 3; ++blk) vsto(uni(Vw + blk * nn), od, gldo(uni(W + blk * nn), od) * S.vscale);
    } else if (S.kind == KIND_X2) {  // (4): z_j = (y0 + (y1 - x1) / delta, x1, x2)
      double* Zj = uni(I.Z + (long long)S.j * n3);
      const double y0i = (double)gldo(uni((const T*)I.y0), og), y1i = (double)gldo(uni((const T*)I.y1), og);
      // x1: formed above where its solve ends in this launch
      const double x1i = S.fuse ? (double)x1f : (double)gldo(uni((const T*)I.x1), og);
      vsto(Zj, od, y0i + (y1i - x1i) / I.delta);
      vsto(uni(Zj + nn), od, x1i);
    }
  } else {
    vsto(o.x, og, T((double)xo + dx));
  }
  vsto(bout, og, pn);
  vsto(uni(bout + nn), og, tpo);
  vsto(uni(bout + 2 * nn), og, ttp);
  vsto(uni(bout + 3 * nn), og, un);
  vsto(uni(bout + 4 * nn), og, tuo);
  ss_gram_out(dg, pn, tpo, ttp, un, tuo, bbo, spart_out + (long long)tm.rank * 32);
}

// ---- orthogonalisation of an Arnoldi step (one reduction) ----------------------
// Modified Gram-Schmidt against v_0..v_j computes h_i = (w - sum_{k<i} h_k v_k,
// v_i) one after the other, which needs j + 1 reductions.  Expanding the inner
// product gives h_i = c_i - sum_{k<i} (v_i, v_k) h_k with c_i = (w, v_i): h
// solves (I + L) h = c, L the strictly lower part of the basis' Gram matrix.
// This equals modified Gram-Schmidt in exact arithmetic for any basis
// (Swirydowicz, Langou, Ananthan, Yang, Thomas, "Low synchronization
// Gram-Schmidt and GMRES algorithms", 2020).  The launch that forms w = A z_j
// therefore also sums c_0..c_j, row j of L ((v_j, v_k), k < j) and (w, w); the
// transition solves for h; the next launch applies w -= sum_i h_i v_i in the
// order of modified Gram-Schmidt and sums (w, w) for h_{j+1,j}.
// Slots of the 64 sums: c_k -> k, (v_j, v_k) -> 32 + k, (w, w) -> 32 + j.
#define PFC_GS_NV 64
__shared__ double pfc_gsred[PFC_WAVES * PFC_GS_NV];

// Sums of 16 values over the 64 lanes of a wave by recursive halving (as
// ss_wave_sums32 for 32): the total of value idx ends in the four lanes of a
// quad, idx = 8 [l >= 32] + 4 [row odd] + 2 [l mod 16 >= 8] + [l mod 8 >= 4].
__device__ __forceinline__ double gs_wave_sums16(const double* v, int lane) {
  double w8[8], w4[4], w2[2];
#pragma unroll
  for (int k = 0; k < 8; ++k) w8[k] = ss_swap<false>(v[k], v[k + 8]);
#pragma unroll
  for (int k = 0; k < 4; ++k) w4[k] = ss_swap<true>(w8[k], w8[k + 4]);
#pragma unroll
  for (int k = 0; k < 2; ++k) w2[k] = ss_dppx<0x140>(w4[k], w4[k + 2], (lane & 15) >= 8);  // row_mirror
  double w1 = ss_dppx<0x141>(w2[0], w2[1], (lane & 7) >= 4);                                // row_half_mirror
  w1 += dpp_f64<0x4e, 0xf>(w1);                                                             // quad_perm [2,3,0,1]
  return w1 + dpp_f64<0xb1, 0xf>(w1);                                                       // quad_perm [1,0,3,2]
}
__device__ __forceinline__ int gs_wave_sums16_index(int lane) {
  return (lane >= 32 ? 8 : 0) + (((lane >> 4) & 1) ? 4 : 0) + ((lane & 15) >= 8 ? 2 : 0) + ((lane & 7) >= 4 ? 1 : 0);
}

// w = A_s z_j (the block SpMV of A^R on the scaled system) and the Gram sums
// of the orthogonalisation; the workgroup's 64 sums go to gout[rank * 64 + s].
template <typename T, int L, bool MOB>
__device__ __forceinline__ void ph_aspmv(const InstDev& I, const State& S, const Team& tm, double* gout) {
  const int n = I.n;
  const PatView<L> pv = p1_pat<L>(I, tm);
  const long long n3 = 3LL * n;
  double* Zj = I.Z + (long long)S.j * n3;
  const T* x2 = (const T*)I.x2;
  PFC_SLICES(I, tm) {
    const int i = sl * 64 + tm.lane;
    double w0, w1, w2;
    block_row<L, MOB, T>(I, pv, sl, tm.lane, I.tau_s, I.m11_s, {Zj, x2}, w0, w1, w2);
    if (i < n) {
      vst(I.W + i, w0); vst(I.W + n + i, w1); vst(I.W + 2 * n + i, w2);
      vst(Zj + 2 * n + i, (double)x2[i]);
    }
  }
  // the sums, eight basis vectors at a time; a thread reads back only the rows of
  // w it stored itself
  const int j = S.j;
  const double* Vj = I.V + (long long)j * n3;
  const int lane = tm.lane, wave = tm.wave;
  for (int b = 0; b * 8 <= j; ++b) {
    double v16[16];
#pragma unroll
    for (int q = 0; q < 16; ++q) v16[q] = 0.0;
    PFC_SLICES(I, tm) {
      const int i = sl * 64 + lane;
      if (i < n) {
        double w[3], vj[3];
#pragma unroll
        for (int blk = 0; blk < 3; ++blk) { w[blk] = I.W[blk * n + i]; vj[blk] = gld(Vj + blk * n + i); }
#pragma unroll
        for (int q = 0; q < 8; ++q) {
          const int k = 8 * b + q;
          if (k < j) {
            const double* Vk = I.V + (long long)k * n3;
            double c = 0.0, l = 0.0;
#pragma unroll
            for (int blk = 0; blk < 3; ++blk) {
              const double vk = gld(Vk + blk * n + i);
              c += w[blk] * vk;
              l += vj[blk] * vk;
            }
            v16[q] += c;
            v16[8 + q] += l;
          } else if (k == j) {
            v16[q] += w[0] * vj[0] + w[1] * vj[1] + w[2] * vj[2];
            v16[8 + q] += w[0] * w[0] + w[1] * w[1] + w[2] * w[2];
          }
        }
      }
    }
    const double tot = gs_wave_sums16(v16, lane);
    const int idx = gs_wave_sums16_index(lane);
    if ((lane & 3) == 0) pfc_gsred[wave * PFC_GS_NV + (idx < 8 ? 8 * b + idx : 32 + 8 * b + idx - 8)] = tot;
  }
  __syncthreads();
  const int tid = threadIdx.x;
  if (tid < PFC_GS_NV) {
    const int k = tid & 31;
    double t = 0.0;
    if (k <= j) {
#pragma unroll
      for (int w = 0; w < PFC_WAVES; ++w) t += pfc_gsred[w * PFC_GS_NV + tid];
    }
    vst(gout + (long long)tm.rank * PFC_GS_NV + tid, t);
  }
}

// Sum of the orthogonalisation's Gram partials of a team ([size][64], fixed
// order) into g[0..63] (LDS): thread t sums value t mod 64 over the ranks
// t / 64, t / 64 + 16, ...; the first 64 threads add the 16 group sums.  The
// basis' stored Gram rows L (the Hist record) come to Ls[32 * 32] in the same
// round trip.  Every thread of the workgroup calls this.
static_assert(PFC_WG == PFC_MAXM * PFC_MAXM, "gs_gather loads the stored Gram rows one entry per thread");
#define PFC_GS_U 8  // partials per thread whose loads are issued together
__device__ __forceinline__ void gs_gather(const double* part, int size, const double* Lg, double* g, double* Ls) {
  const int tid = threadIdx.x, v = tid & 63, grp = tid >> 6;
  const double lv = Lg[tid];  // PFC_WG = PFC_MAXM * PFC_MAXM entries, one per thread
  double s = 0.0;
  for (int k0 = grp; k0 < size; k0 += PFC_GS_U * PFC_WAVES) {
    double t[PFC_GS_U];
#pragma unroll
    for (int u = 0; u < PFC_GS_U; ++u) t[u] = part[(long long)min(k0 + u * PFC_WAVES, size - 1) * PFC_GS_NV + v];
#pragma unroll
    for (int u = 0; u < PFC_GS_U; ++u)
      if (k0 + u * PFC_WAVES < size) s += t[u];
  }
  pfc_gsred[grp * PFC_GS_NV + v] = s;
  Ls[tid] = lv;
  __syncthreads();
  if (tid < PFC_GS_NV) {
    double t = 0.0;
#pragma unroll
    for (int w = 0; w < PFC_WAVES; ++w) t += pfc_gsred[w * PFC_GS_NV + tid];
    g[tid] = t;
  }
  __syncthreads();
}

// w -= sum_{i <= j} h_i v_i in the order of modified Gram-Schmidt; partial (w, w)
__device__ __forceinline__ Red3 ph_gs_update(const InstDev& I, const State& S, const Team& tm, const double* h) {
  const int n = I.n;
  const long long n3 = 3LL * n;
  const int j = S.j;
  double a0 = 0.0;
  PFC_SLICES(I, tm) {
    const int i = sl * 64 + tm.lane;
    if (i < n) {
#pragma unroll
      for (int blk = 0; blk < 3; ++blk) {
        const long long o = (long long)blk * n + i;
        double w = I.W[o];
        for (int k = 0; k <= j; ++k) w -= h[k] * I.V[(long long)k * n3 + o];
        vst(I.W + o, w);
        a0 += w * w;
      }
    }
  }
  return red3(a0, 0.0);
}

}  // namespace pfc
