// Host-side objects behind the C ABI handles.
#pragma once
#include <hip/hip_runtime.h>

#include <string>
#include <vector>

#include "../../include/pfc.h"
#include "pfc_internal.h"

namespace pfc {

void set_error(const std::string& msg);
int hip_fail(hipError_t e, const char* what);

#define PFC_HIP(call)                                   \
  do {                                                  \
    hipError_t _e = (call);                             \
    if (_e != hipSuccess) return pfc::hip_fail(_e, #call); \
  } while (0)

}  // namespace pfc

struct pfc_mesh {
  int dim = 0, n = 0, nnz = 0, n_elem = 0, n_slices = 0;
  int uniform_width = 0;               // common slice width (1..16), 0 if slices differ
  int degree = 1, nloc = 0;            // Lagrange degree and nodes per element
  double* d_p2tab = nullptr;           // P2 reference tables (M2, D, C2, C3, C2 transposed)
  const double* d_p2C2t = nullptr;
  long long nnz_sell = 0;
  std::vector<int> row_ptr, col_idx;   // CSR pattern (host)
  std::vector<long long> csr2sell;     // CSR slot -> SELL position
  // device arrays
  int* d_slice_ptr = nullptr;
  int* d_col = nullptr;
  double* d_M = nullptr;
  double* d_K = nullptr;
  float* d_Mf = nullptr;
  float* d_Kf = nullptr;
  double* d_dinvM = nullptr;
  float* d_dinvMf = nullptr;
  long long* d_nv_ptr = nullptr;       // simplices containing each node (MeshDev::nv_*)
  int* d_nv_el = nullptr;
  unsigned* d_nv_slot = nullptr;
  int* d_row_ptr = nullptr;            // CSR row offsets
  short* d_goff3 = nullptr;            // MeshDev::goff3
  int* d_elem_nodes = nullptr;
  double* d_vol = nullptr;
  double* d_elemK = nullptr;           // element stiffness (P1 meshes), for the PFC1 mobility
  // second-ring pattern for the S_D preconditioner (built on first use)
  int* d_w_slice_ptr = nullptr;
  int* d_w_col = nullptr;
  long long* d_w_p1pos = nullptr;
  int* d_w_tri_ptr = nullptr;
  int* d_w_tri = nullptr;
  MeshDev dev{};
};

namespace pfc {
int build_second_ring(pfc_mesh* m);
// N(psi) on the mesh's stored pattern (csr: in CSR order); A^R y with N(psi_k)
// formed on the way, where the mesh's rows are short enough for that and psi does
// not overlap out
int launch_row_N(const pfc_mesh* m, const double* psi, double* out, bool csr, hipStream_t s);
bool row_AR_applies(const pfc_mesh* m, const double* psi, const double* out);
int launch_row_AR(const pfc_mesh* m, const double* psi, double r, double tau, double m11, const double* y, double* out,
                  hipStream_t s);
}

namespace pfc {
// Launch shape of the mesh-level kernels with element sums with `arrays` values per row entry in LDS:
// as many threads as keep four workgroups on a CU, down to one wave; rows too
// long for that are not staged.
// The mesh's byte-wide positions (rows of at most PFC_ROW_MAX entries) go with staging.
#define PFC_ROW_T 256  // threads of a workgroup at most, a row each
struct RowPlan {
  int T, cap;
  bool stage;
  size_t lds(int arrays) const { return (size_t)arrays * cap * (T + 1) * sizeof(double); }
};
inline RowPlan row_plan(const pfc_mesh* m, int arrays) {
  if (m->dev.nv_wide) return RowPlan{64, 0, false};
  RowPlan p{PFC_ROW_T, m->dev.zmax, true};
  while (p.T > 64 && p.lds(arrays) > 40 * 1024) p.T /= 2;
  return p;
}
inline dim3 row_grid(const pfc_mesh* m, int T) { return dim3((m->n_slices + T / 64 - 1) / (T / 64)); }

#define PFC_FOR_NLOC(m, X)                                                      \
  switch ((m)->nloc) {                                                          \
    case 3: X(3); break;                                                        \
    case 4: X(4); break;                                                        \
    case 6: X(6); break;                                                        \
    default: X(10); break;                                                      \
  }

// grid of standalone kernels over the slices of a mesh (one wave per slice)
inline int slice_blocks(int n_slices) { return (n_slices + PFC_WAVES - 1) / PFC_WAVES; }
}  // namespace pfc
