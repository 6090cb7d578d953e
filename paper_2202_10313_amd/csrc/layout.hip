// Conversion between the caller's DOF arrays (FP64, [element][quantity][mode],
// caller's element and vertex order) and the tiled device state Qe / Qa, on
// the device: edg_set_initial, edg_read_dofs and the DOF arguments of
// edg_adjoint.
//
// One workgroup per element: its Nq x B words pass through LDS, thread t forms
// words t, t + 256, ... each as the row's product with the B x B matrix of the
// element's vertex order.  The work is bound by the host link and, on the
// device, by FP64 multiply-adds (2 B per word); the matrices (24 of them,
// 9.8 KB each at O = 5) stay in L2, and are read with the mode that runs
// along the threads contiguous.  The tiled side is accessed in single words
// (an element's words of one mode are 9 apart from its group's neighbours'),
// which the host link hides.  Measured at 3,888 elements, O = 5, 27
// quantities, FP32, for state in + one cycle + state out: 61.9 ms when one host
// thread converted both ways, 3.3 ms with these kernels (of which 0.18 ms is
// the cycle and the rest the two 29 MB copies over the host link).
//
// Sums run over the modes in ascending order without contraction, as the
// host conversions of edg_set_dofs_subset do, so both give the same bits.
#include <hip/hip_runtime.h>

#include "kernels.hpp"
#include "device_common.hpp"

namespace edg {

namespace {

// word of quantity q, mode b of internal element ki: index in Qe (q < 9) or Qa
__device__ __forceinline__ size_t state_index(const DofTables& t, long long ki, int q, int b) {
  const size_t g = (size_t)(ki / EPW);
  const int e = (int)(ki % EPW);
  if (q < LPE) return (g * t.B + b) * NSLOT + e * LPE + q;
  const int jbn = (t.B + LPE - 1) / LPE, jb = b / LPE, r = b % LPE, l = (q - LPE) / 6, c = (q - LPE) % 6;
  return (((g * jbn + jb) * t.M + l) * 6 + c) * NSLOT + e * LPE + r;
}

constexpr int MAX_WORDS = (9 + 6 * MAX_MECH) * (MAX_ORDER * (MAX_ORDER + 1) * (MAX_ORDER + 2) / 6);

// dofs: [n][Nq][B] of caller elements k0 .. k0 + n - 1
template <class R>
__global__ __launch_bounds__(256) void k_set_dofs(DofTables t, long long k0, const double* __restrict__ dofs, R* Qe,
                                                  R* Qa) {
#pragma clang fp contract(off)
  __shared__ double row[MAX_WORDS];
  const long long k = k0 + blockIdx.x, ki = t.u2i[k];
  const int B = t.B, words = (LPE + 6 * t.M) * B;
  const double* src = dofs + (size_t)blockIdx.x * words;
  for (int i = threadIdx.x; i < words; i += 256) row[i] = src[i];
  __syncthreads();
  // row b of the matrix, transposed: [bb][b]
  const double* C = t.mats + (size_t)t.code[k] * 2 * B * B + B * B;
  for (int i = threadIdx.x; i < words; i += 256) {
    const int q = i / B, b = i % B;
    double s = 0.0;
    for (int bb = 0; bb < B; ++bb) s += C[bb * B + b] * row[q * B + bb];
    (q < LPE ? Qe : Qa)[state_index(t, ki, q, b)] = R(s);
  }
}

template <class R>
__global__ __launch_bounds__(256) void k_get_dofs(DofTables t, long long k0, double* __restrict__ dofs, const R* Qe,
                                                  const R* Qa) {
#pragma clang fp contract(off)
  __shared__ double row[MAX_WORDS];
  const long long k = k0 + blockIdx.x, ki = t.u2i[k];
  const int B = t.B, words = (LPE + 6 * t.M) * B;
  double* dst = dofs + (size_t)blockIdx.x * words;
  for (int i = threadIdx.x; i < words; i += 256) {
    const int q = i / B, b = i % B;
    row[i] = (double)(q < LPE ? Qe : Qa)[state_index(t, ki, q, b)];
  }
  __syncthreads();
  const double* C = t.mats + (size_t)t.code[k] * 2 * B * B;
  for (int i = threadIdx.x; i < words; i += 256) {
    const int q = i / B, bb = i % B;
    double s = 0.0;
    for (int b = 0; b < B; ++b) s += C[b * B + bb] * row[q * B + b];
    dst[i] = s;
  }
}

}  // namespace

template <class R>
int launch_set_dofs(const DofTables& t, long long k0, long long n, const double* dofs, R* Qe, R* Qa, hipStream_t st) {
  if (n <= 0) return 0;
  if (n > DOF_LAUNCH) return (int)hipErrorInvalidValue;
  hipLaunchKernelGGL((k_set_dofs<R>), dim3((unsigned)n), dim3(256), 0, st, t, k0, dofs, Qe, Qa);
  return (int)hipGetLastError();
}

template <class R>
int launch_get_dofs(const DofTables& t, long long k0, long long n, double* dofs, const R* Qe, const R* Qa,
                    hipStream_t st) {
  if (n <= 0) return 0;
  if (n > DOF_LAUNCH) return (int)hipErrorInvalidValue;
  hipLaunchKernelGGL((k_get_dofs<R>), dim3((unsigned)n), dim3(256), 0, st, t, k0, dofs, Qe, Qa);
  return (int)hipGetLastError();
}

#define EDG_DOF_INST(R)                                                                                   \
  template int launch_set_dofs<R>(const DofTables&, long long, long long, const double*, R*, R*, hipStream_t); \
  template int launch_get_dofs<R>(const DofTables&, long long, long long, double*, const R*, const R*, hipStream_t);
EDG_DOF_INST(float)
EDG_DOF_INST(double)

}  // namespace edg
