// Interface between the host library and the adjoint kernels (internal).
#pragma once
#include "kernels.hpp"

namespace edg {

// ---- discrete adjoint (one run)
constexpr int KIND_ADJ_PREDICT = 3;  // transposed predictions only (start of a segment)
constexpr int KIND_ADJ_UPDATE = 4;   // transposed surface updates only (end of a segment)
constexpr int KIND_ADJ_FUSED = 5;    // transposed predictions, then transposed updates, of the same elements
// adjoint face rows: 9 elastic + 6 omega-weighted memory-variable sums (anelastic only)
constexpr int adj_rows(int M) { return M > 0 ? 15 : 9; }
// Per-element gradient words (internal order, FP64): derivatives of the
// adjoint pairing in the parameters the kernels read.
//   [7f+0..6]        (1/rho, lam, mu, Zp, Zs, Zp+, Zs+) of the own flux of face f
//   [NG_NBR+7f+0..6] the same of the flux of the element across face f (its
//                    neighbour-data part)
//   [NG_AB+2l], [NG_AB+2l+1]  a_l, b_l of the products (time and volume kernel)
//   [NG_RHO]         rho times the products' derivative in rho at fixed vp, vs
//                    (through 1/rho and all moduli, the anelastic ones too)
//   [NG_RHO+1, +2]   lam, mu of the products
constexpr int NG_NBR = 28, NG_AB = 56, NG_RHO = 62;
constexpr int NG = 65;

struct APtrs {
  void* Le;          // adjoint of the elastic rows (Qe layout)
  void* La;          // adjoint of the memory variables (Qa layout)
  const void* Se;    // forward state at the start of the step (Qe layout)
  const void* Sa;    // (Qa layout)
  void* S0;          // [2][Kp][4][adj_rows][FP] face adjoints of each element's last steps (step parity)
  void* S3;          // [4][N3][4][adj_rows][FP] the same of the elements with a coarser neighbour (step mod 4)
  void* De;          // scratch: adjoint_scratch_words() words per element group
  double* gacc;      // [Kp][NG]
  void* recDb;       // [slots][O][9][B] adjoint of the receiver derivatives
};

// d/d(rho, vp, vs) [Kp][3] from the gradient words (mat [Kp][3 + 2m]: rho,
// vp, vs, Yp_l, Ys_l in internal order; rho = 0 for padding)
int launch_material_gradient(const double* gacc, const int* FI, const double* mat, int M, long long Kp, double* out,
                             hipStream_t st);

template <class R, int O, int M>
int launch_adjoint(const KPtrs& p, const APtrs& ad, const LevelArgs& a, hipStream_t st);
// words of De per element group of this variant
template <class R, int O, int M>
size_t adjoint_scratch_words();
// chain [n]: 2 (next receiver in the same element + 1) + (1 for the element's first)
template <class R, int O, int M>
int launch_receivers_adj(const KPtrs& p, const APtrs& ad, const LevelArgs& a, const RecArgs& r, const int* chain,
                         const double* seis_b, hipStream_t st);

}  // namespace edg
