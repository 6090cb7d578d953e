// HIP kernels (gfx950) of the discrete adjoint of the clustered rate-2 LTS
// ADER-DG update: the exact transpose of the forward kernels' arithmetic, for
// gradients of receiver misfits with respect to the materials.  The paper
// names inversion as a use (Sec. II (Related Work)) but gives no adjoint; the
// forward scheme it transposes is that of Sec. III-A (Discrete Formulation)
// and Sec. V-B (Buffers and Algorithm).
//
// The forward advance is a sequence of per-level launches: at finest level j
// the clusters whose step ends there finish it (surface update from the own
// B1 face trace and the neighbour data), then the clusters whose step starts
// there predict (time kernel, B1/B2/B3 traces, volume update).  The adjoint
// runs the levels backwards, one launch per level: of each element the
// transposed prediction of the step that starts there, then the transposed
// update of the step that ends there.
//
//  * transposed update (element k, step n): the adjoint Qbar of k does not
//    change (the update is Q += ...); what flows out are the face adjoints
//    u = trace(Qbar) (9 elastic rows and the 6 omega-weighted sums of the
//    memory-variable rows, 15 x F per face).  They stay in k's own slots (two
//    step parities; elements with a coarser neighbour also keep the last four
//    steps in S3), and whoever needs them gathers them: k itself (its own
//    flux) and the neighbour across each face, whose buffer that flux read.
//  * transposed prediction (element j, step n): recomputes the time
//    derivatives from the stored start-of-step state, then forms the adjoint
//    of the time integrals: the transposed volume kernel and own surface part
//    (from Qbar and its own u), plus its neighbours' u pulled through the
//    transpose of the neighbour's flux (Godunov with the neighbour's
//    parameters): same cluster -> its B1; coarser -> its B3; finer -> its B2
//    from the difference of the neighbour's two steps, B1 from the second.
//    Then the Cauchy-Kowalevski recursion runs backwards and the adjoint of
//    the start-of-step state is added to Qbar.
// Slots are written before they are read in every sweep, and the slot a launch
// writes is none that the same launch reads: the other parity, or for the
// four-step slots another step (mod 4) than the two a coarser neighbour reads.
//
// Material derivatives: every product that involves a material parameter
// (lam, mu, 1/rho, a_l, b_l, the impedances of the flux solver) adds its
// adjoint-weighted partial derivative to per-element FP64 words (NG);
// k_material_gradient applies the chain rule to rho, vp, vs.
//
// dJ/drho of the products (at fixed vp, vs) is not formed from their derivatives
// in 1/rho and in the moduli: those cancel, to 1e-12 of either where the recorded
// stresses depend on rho through lam/rho and mu/rho only (two steps from rest),
// and FP32 sums left rounding there (1e5 times the exact value, FP64 1e-3 of it).
// Every product is linear in a state (stresses s, the rest z = velocities and
// memory variables); rho multiplies its part s <- z and divides its part z <- s,
// so with P the projection on z and L the product, rho dL/drho = L P - P L.
// Summed over the Cauchy-Kowalevski recursion and the volume kernel, <adjoint of
// the output, (L P - P L) input> telescopes to
//   <D_0 adjoint, P D_0> - <receivers' part of the D_d adjoint, P D_d>, all d,
//   - <flux part of the time integral's adjoint, P T> (T and the half step's)
//   - <Qbar, P V>, V the volume term,
// whose terms have the size of the result: 6e-8 .. 1.4e-7 of the exact value in
// FP32 there, 9e-16 in FP64, at the same time (97k tets, a reverse cycle,
// O = 5 m=3 and O = 4 m=0: within 1%).  Of V's memory rows, -omega (eps + T^theta),
// the T^theta part is paired through Lambda_d (T^theta is linear in the strain
// rates of the recursion and in the start-of-step memory variables).
//
// Work mapping: as the forward k_level, W waves per 7 elements, lane 9e + q of
// wave w holds row q of element e for the wave's modes and at most one
// memory-variable mode.  Reference-matrix products are the generated
// straight-line code and its transposes; row-mixing products go through LDS.
//
// What bounds it: vector issue (52-64% of the SIMDs' cycles) and LDS / barrier
// latency at three waves per SIMD; 2.1-3.8 TB/s of memory traffic.
// Measured per reverse cycle of two clusters, 97k tets, FP32 (before: two
// launches per level with neighbour slots updated in place, two waves at O = 4
// and 5 that kept every step's sums, coupling adjoints and Qbar in 0.24 MB of
// scratch per group, one wave otherwise): O = 5 m=3 3,490 -> 2,220 us, O = 4
// m=3 2,290 -> 1,550, m=0 1,330 -> 908, O = 3 m=3 1,540 -> 766; FP64 O = 5 m=3
// 12k tets 7,220 -> 718 (3.8 KB of spills a lane before).  Combining the rows
// of the transposed products with G' before the exchange and forming the lane's
// parameters twice (37k tets): O = 5 m=3 820 -> 761, O = 4 m=3 555 -> 458, m=0
// 330 -> 306, O = 3 m=3 276 -> 245; FP64 O = 5 m=3 10k 624 -> 590.  With dJ/drho
// free of cancelling parts, sums in a fixed order and, up to O = 3, in FP64 (97k
// tets): O = 5 m=3 2,076 -> 2,124, O = 4 m=3 1,247 -> 1,291, m=0 832 -> 854, O = 3
// m=3 671 -> 695; FP64 O = 5 m=3 12k 657 -> 659.
#include <hip/hip_runtime.h>

#include <cstdint>
#include <type_traits>

#include "generated/refmats.h"
#include "adjoint.hpp"
#include "device_common.hpp"

namespace edg {

namespace {

// Reverse mode of godunov(): for the adjoint u of its 15 outputs, adds
// (d out / d qm)^T u to qm_b, (d out / d qp)^T u to qp_b (interior faces) and
// the derivatives of <u, out> in (rho_inv, lam, mu, zpm, zsm, zpp, zsp) to
// pb[0..6].  out is linear in (qm, qp), so the parameter derivatives are
// bilinear: they use the states passed in (zeros for a side that another
// element accounts for).
template <class R>
__host__ __device__ __forceinline__ void godunov_adj(const R* u, const R* qm, const R* qp, R nx, R ny, R nz, R zpm,
                                                     R zsm, R zpp, R zsp, R lam, R mu, R rho_inv, R s, int bc,
                                                     R* qm_b, R* qp_b, R* pb) {
  const R n[3] = {nx, ny, nz};
  // forward intermediates
  R tm[3], vm[3], tp[3], vp[3];
  tm[0] = qm[0] * nx + qm[3] * ny + qm[5] * nz;
  tm[1] = qm[3] * nx + qm[1] * ny + qm[4] * nz;
  tm[2] = qm[5] * nx + qm[4] * ny + qm[2] * nz;
  vm[0] = qm[6]; vm[1] = qm[7]; vm[2] = qm[8];
  if (bc == 0) {
    tp[0] = qp[0] * nx + qp[3] * ny + qp[5] * nz;
    tp[1] = qp[3] * nx + qp[1] * ny + qp[4] * nz;
    tp[2] = qp[5] * nx + qp[4] * ny + qp[2] * nz;
    vp[0] = qp[6]; vp[1] = qp[7]; vp[2] = qp[8];
  } else if (bc == 1) {
    for (int c = 0; c < 3; ++c) { tp[c] = -tm[c]; vp[c] = vm[c]; }
  } else {
    for (int c = 0; c < 3; ++c) { tp[c] = R(0); vp[c] = R(0); }
  }
  const R tnm = tm[0] * nx + tm[1] * ny + tm[2] * nz, vnm = vm[0] * nx + vm[1] * ny + vm[2] * nz;
  const R tnp = tp[0] * nx + tp[1] * ny + tp[2] * nz, vnp = vp[0] * nx + vp[1] * ny + vp[2] * nz;
  const R ip = R(1) / (zpm + zpp), is = R(1) / (zsm + zsp);
  const R Y = zpm * vnm + zpp * vnp + tnp - tnm;
  const R Z = zpp * tnm + zpm * tnp + zpm * zpp * (vnp - vnm);
  const R vn = Y * ip, tn = Z * ip;
  const R zz = zsm * zsp;
  R tTm[3], vTm[3], tTp[3], vTp[3], W[3], X[3], v[3], t[3];
  for (int c = 0; c < 3; ++c) {
    tTm[c] = tm[c] - tnm * n[c];
    vTm[c] = vm[c] - vnm * n[c];
    tTp[c] = tp[c] - tnp * n[c];
    vTp[c] = vp[c] - vnp * n[c];
    W[c] = zsm * vTm[c] + zsp * vTp[c] + tTp[c] - tTm[c];
    X[c] = zsp * tTm[c] + zsm * tTp[c] + zz * (vTp[c] - vTm[c]);
    v[c] = vn * n[c] + W[c] * is;
    t[c] = tn * n[c] + X[c] * is;
  }
  // outputs -> v, t, material parameters
  R vb[3] = {R(0), R(0), R(0)}, tb[3] = {R(0), R(0), R(0)};
  R vnb = R(0), lamb = R(0), mub = R(0), rib = R(0);
  const R hs = R(0.5) * s;
  for (int c = 0; c < 3; ++c) {
    vnb += s * lam * u[c];
    lamb += s * vn * u[c];
    vb[c] += R(2) * mu * s * n[c] * u[c];
    mub += R(2) * s * n[c] * v[c] * u[c];
    tb[c] += s * rho_inv * u[6 + c];
    rib += s * t[c] * u[6 + c];
    vb[c] += s * n[c] * u[9 + c];
  }
  const int pa[3] = {0, 1, 0}, pc[3] = {1, 2, 2};   // (x,y), (y,z), (x,z)
  for (int k = 0; k < 3; ++k) {
    const int a = pa[k], b = pc[k];
    const R ue = u[3 + k], ua = u[12 + k];
    vb[b] += mu * s * n[a] * ue + hs * n[a] * ua;
    vb[a] += mu * s * n[b] * ue + hs * n[b] * ua;
    mub += s * (n[a] * v[b] + n[b] * v[a]) * ue;
  }
  // v = vn n + W is, t = tn n + X is
  R Wb[3], Xb[3];
  R isb = R(0), tnb = R(0);
  for (int c = 0; c < 3; ++c) {
    vnb += vb[c] * n[c];
    tnb += tb[c] * n[c];
    Wb[c] = vb[c] * is;
    Xb[c] = tb[c] * is;
    isb += vb[c] * W[c] + tb[c] * X[c];
  }
  R vTmb[3], vTpb[3], tTmb[3], tTpb[3];
  R zsmb = R(0), zspb = R(0), zzb = R(0);
  for (int c = 0; c < 3; ++c) {
    vTmb[c] = zsm * Wb[c] - zz * Xb[c];
    vTpb[c] = zsp * Wb[c] + zz * Xb[c];
    tTpb[c] = Wb[c] + zsm * Xb[c];
    tTmb[c] = -Wb[c] + zsp * Xb[c];
    zsmb += Wb[c] * vTm[c] + Xb[c] * tTp[c];
    zspb += Wb[c] * vTp[c] + Xb[c] * tTm[c];
    zzb += Xb[c] * (vTp[c] - vTm[c]);
  }
  zsmb += zsp * zzb;
  zspb += zsm * zzb;
  // tangential parts
  R tmb[3], vmb[3], tpb[3], vpb[3];
  R tnmb = R(0), vnmb = R(0), tnpb = R(0), vnpb = R(0);
  for (int c = 0; c < 3; ++c) {
    tmb[c] = tTmb[c];
    vmb[c] = vTmb[c];
    tpb[c] = tTpb[c];
    vpb[c] = vTpb[c];
    tnmb -= tTmb[c] * n[c];
    vnmb -= vTmb[c] * n[c];
    tnpb -= tTpb[c] * n[c];
    vnpb -= vTpb[c] * n[c];
  }
  // normal parts
  const R Yb = vnb * ip, Zb = tnb * ip;
  const R ipb = vnb * Y + tnb * Z;
  vnmb += zpm * Yb - zpm * zpp * Zb;
  vnpb += zpp * Yb + zpm * zpp * Zb;
  tnpb += Yb + zpm * Zb;
  tnmb += -Yb + zpp * Zb;
  R zpmb = Yb * vnm + Zb * (tnp + zpp * (vnp - vnm));
  R zppb = Yb * vnp + Zb * (tnm + zpm * (vnp - vnm));
  zpmb -= ipb * ip * ip;
  zppb -= ipb * ip * ip;
  zsmb -= isb * is * is;
  zspb -= isb * is * is;
  for (int c = 0; c < 3; ++c) {
    tmb[c] += tnmb * n[c];
    vmb[c] += vnmb * n[c];
    tpb[c] += tnpb * n[c];
    vpb[c] += vnpb * n[c];
  }
  // outside state
  if (bc == 0) {
    qp_b[0] += tpb[0] * nx;
    qp_b[1] += tpb[1] * ny;
    qp_b[2] += tpb[2] * nz;
    qp_b[3] += tpb[0] * ny + tpb[1] * nx;
    qp_b[4] += tpb[1] * nz + tpb[2] * ny;
    qp_b[5] += tpb[0] * nz + tpb[2] * nx;
    qp_b[6] += vpb[0];
    qp_b[7] += vpb[1];
    qp_b[8] += vpb[2];
  } else if (bc == 1) {
    for (int c = 0; c < 3; ++c) {
      tmb[c] -= tpb[c];
      vmb[c] += vpb[c];
    }
  }
  qm_b[0] += tmb[0] * nx;
  qm_b[1] += tmb[1] * ny;
  qm_b[2] += tmb[2] * nz;
  qm_b[3] += tmb[0] * ny + tmb[1] * nx;
  qm_b[4] += tmb[1] * nz + tmb[2] * ny;
  qm_b[5] += tmb[0] * nz + tmb[2] * nx;
  qm_b[6] += vmb[0];
  qm_b[7] += vmb[1];
  qm_b[8] += vmb[2];
  pb[0] += rib;
  pb[1] += lamb;
  pb[2] += mub;
  pb[3] += zpmb;
  pb[4] += zsmb;
  pb[5] += zppb;
  pb[6] += zspb;
}

// the element at 32-bit element offset i from a per-workgroup (uniform) base:
// the address is a scalar base plus a zero-extended 32-bit lane byte offset,
// so no 64-bit per-lane address stays live (or spills) across the long loops
template <class T>
__device__ __forceinline__ T& at(T* base, uint32_t i) {
  return *reinterpret_cast<T*>(reinterpret_cast<char*>(base) + (size_t)(i * (uint32_t)sizeof(T)));
}
template <class T>
__device__ __forceinline__ const T& at(const T* base, uint32_t i) {
  return *reinterpret_cast<const T*>(reinterpret_cast<const char*>(base) + (size_t)(i * (uint32_t)sizeof(T)));
}

// adds v to the element's gradient word w (LDS, FP64).  The elements' word
// arrays are an odd number of doubles apart: with a stride of 48 the same word of
// every other element fell into one bank, so an atomic of a wave serialised over
// four elements' lanes
constexpr int NGS = NG | 1;
__device__ __forceinline__ void gadd(double* gs, int w, double v) { atomicAdd(gs + w, v); }

// v of the lane that DPP control CTRL names (a permutation within 16-lane rows)
template <int CTRL>
__device__ __forceinline__ float dpp(float v) {
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, 0xf, 0xf, true));
}
template <int CTRL>
__device__ __forceinline__ double dpp(double v) {
  const unsigned long long u = __builtin_bit_cast(unsigned long long, v);
  const unsigned lo = (unsigned)__builtin_amdgcn_update_dpp(0, (int)(unsigned)u, CTRL, 0xf, 0xf, true);
  const unsigned hi = (unsigned)__builtin_amdgcn_update_dpp(0, (int)(unsigned)(u >> 32), CTRL, 0xf, 0xf, true);
  return __builtin_bit_cast(double, (unsigned long long)hi << 32 | lo);
}
// the sum of v over aligned segments of SEG = 4, 8 or 16 lanes, in all of them
template <int SEG, class R>
__device__ __forceinline__ R seg_sum(R v) {
  v += dpp<0xb1>(v);                       // quad_perm 1 0 3 2
  v += dpp<0x4e>(v);                       // quad_perm 2 3 0 1
  if (SEG > 4) v += dpp<0x141>(v);         // row_half_mirror
  if (SEG > 8) v += dpp<0x140>(v);         // row_mirror
  return v;
}

// This lane's number, formed anew where it is used: kept in a register over the
// face phases it is spilled and reloaded at every use (FP64 O = 4: 50 -> 59 us a
// level of 5k tets).
__device__ __forceinline__ int lane_id() {
  int v;
  asm volatile("v_mbcnt_lo_u32_b32 %0, -1, 0\n\tv_mbcnt_hi_u32_b32 %0, -1, %0" : "=v"(v));
  return v;
}

// Waves per 7 elements: the modes of a wave must number at most nine, so that
// each lane owns at most one memory-variable mode (18 words at three
// mechanisms stay in registers).
template <int O>
constexpr int ADJ_W = O >= 4 ? 4 : 2;

template <class R, int O, int M>
struct AdjLds {
  using RF = edg_gen::Ref<O>;
  static constexpr int B = RF::B, FP = RF::FP;
  static constexpr int up(int v, int m, int r) { return v + ((r - v % m) % m + m) % m; }
  static constexpr int BS = B % 2 ? B : B + 1;       // odd row stride
  static constexpr int FS = FP + 1;
  static constexpr int NSL = 27;                     // forward products: 18 read pairs and an unread dummy; transposed: [row][reference direction]
  static constexpr int GRAD = NSL * BS;
  static constexpr int COUP = 6 * BS;
  static constexpr int RX = LPE * BS;
  static constexpr int PMW = 4 * LPE * FS;           // face traces / their adjoints [face][row][f], over grad and coup
  static constexpr int ROFF = GRAD + COUP > PMW ? GRAD + COUP : PMW;
  static constexpr int REGION = up(ROFF + RX, 32, (9 * BS) % 32);
  static constexpr int TOTAL = EPW * REGION;
};

// Per-wave scratch in device memory, in 16-byte lane pieces side by side (one
// coalesced transfer of up to 1 KB per instruction): what the reverse loop
// needs of each forward derivative D_d and cannot hold on chip.
//   VX [O - 1]: the velocity rows' gradient sums d_d sigma_id, in groups with a
//               receiver (own modes; 21 lanes, padded to 24)
//   EP [O - 1]: the strain rate of the lane's owned mode (6 words)
//   LM [O]:     Lambda_d of the owned mode (6 words, M > 0)
template <class R, int O, int M>
struct AdjScratch {
  using RF = edg_gen::Ref<O>;
  static constexpr int W = ADJ_W<O>;
  static constexpr int NBX = RF::template nbx<W>;
  static constexpr int VL = 24, VXW = NBX * VL;
  static constexpr int OL = (EPW * NBX + 3) / 4 * 4, EPW6 = 6 * OL;   // lanes that own a mode
  static constexpr int VX = 0;
  static constexpr int EP = VX + (O - 1) * VXW;
  static constexpr int LM = EP + (O - 1) * EPW6;
  static constexpr int WAVE = LM + (M > 0 ? O * EPW6 : 0);
};
// N words of one of L lanes: whole 16-byte pieces [piece][lane], then single words [word][lane]
template <int N, int L, class R>
__device__ __forceinline__ void st_words(R* base, int l, const R* v) {
  constexpr int V = 16 / sizeof(R);
  typedef R vec __attribute__((ext_vector_type(V)));
#pragma unroll
  for (int k = 0; k < N / V; ++k) {
    vec x;
#pragma unroll
    for (int i = 0; i < V; ++i) x[i] = v[V * k + i];
    *reinterpret_cast<vec*>(base + k * L * V + l * V) = x;
  }
#pragma unroll
  for (int k = N / V * V; k < N; ++k) base[k * L + l] = v[k];
}
template <int N, int L, class R>
__device__ __forceinline__ void ld_words(const R* base, int l, R* v) {
  constexpr int V = 16 / sizeof(R);
  typedef R vec __attribute__((ext_vector_type(V)));
#pragma unroll
  for (int k = 0; k < N / V; ++k) {
    const vec x = *reinterpret_cast<const vec*>(base + k * L * V + l * V);
#pragma unroll
    for (int i = 0; i < V; ++i) v[V * k + i] = x[i];
  }
#pragma unroll
  for (int k = N / V * V; k < N; ++k) v[k] = base[k * L + l];
}

// (row, direction) -> gradient slot: velocity rows all directions, stress row
// (i, j) directions i and j; 18 = not read
__device__ __forceinline__ int aslot(int row, int dir) {
  constexpr int T[9][3] = {{9, 18, 18}, {18, 10, 18}, {18, 18, 11}, {12, 13, 18}, {18, 14, 15},
                           {16, 18, 17}, {0, 1, 2}, {3, 4, 5}, {6, 7, 8}};
  constexpr unsigned long long W0 = pack_rows5(T, 0), W1 = pack_rows5(T, 1), W2 = pack_rows5(T, 2);
  const unsigned long long w = dir == 0 ? W0 : (dir == 1 ? W1 : W2);   // selects, no table in memory
  return (int)((w >> (5 * row)) & 31);
}

// Waves per SIMD the registers are budgeted for (us per reverse cycle of two
// clusters).  FP32: three; 144-156 registers without a spill but at O = 5 m=3,
// where 112 B a lane spill and still pay (37k tets 761 against 800 at two, 4.6k
// tets 147 against 160); four at O = 4 m=0 spill 116 B: 305 -> 363.  FP64: one
// (up to 512 registers), two at O = 4, whose 60 KB of LDS leave room for a second
// workgroup (10k tets m=0 249 -> 184, m=3 363 -> 314, at 576 tets 80 -> 83; at
// O = 3, 140 B of spills, 161 -> 189; at O = 5 the LDS holds one workgroup).
template <class R, int O, int M>
constexpr int adj_occ() {
  return sizeof(R) == 4 ? 3 : O == 4 ? 2 : 1;
}

// One reverse level: the transposed prediction of the steps that start here
// and, with KIND_ADJ_FUSED, the transposed update of the steps that end here
// (the element's own Qbar, just completed, traced into its face slots); only
// the update at the end of a segment (KIND_ADJ_UPDATE), only the prediction at
// its start (KIND_ADJ_PREDICT).
template <class R, int O, int M, int KIND>
__global__ __launch_bounds__(64 * ADJ_W<O>) __attribute__((amdgpu_waves_per_eu(adj_occ<R, O, M>(), 8)))
void k_adjoint(KPtrs p, APtrs ad, LevelArgs a) {
  using RF = edg_gen::Ref<O>;
  using L = AdjLds<R, O, M>;
  using SC = AdjScratch<R, O, M>;
  constexpr int W = ADJ_W<O>;
  constexpr int B = RF::B, F = RF::F, FP = RF::FP;
  constexpr int MM = M > 0 ? M : 1;
  constexpr int NBX = RF::template nbx<W>, NBN = RF::template nbn<W>;
  constexpr int NTC = RF::template ntc<W>, NCH = FP / 4;
  constexpr int JB = (B + LPE - 1) / LPE;        // memory-variable layout
  constexpr int BS = L::BS, FS = L::FS;
  constexpr int AR = adj_rows(M);
  static_assert(NBX <= LPE, "at most one owned memory mode per lane");
  __shared__ R lds[L::TOTAL];
  __shared__ double gsh[KIND == KIND_ADJ_UPDATE ? 1 : EPW * NGS];
  __shared__ double grsh[KIND == KIND_ADJ_UPDATE ? 1 : W * NSLOT];
  constexpr int FSTW = 17;
  __shared__ R fst[KIND == KIND_ADJ_UPDATE ? 1 : EPW * 4 * FSTW];
  __shared__ int fnb[EPW * 4], fcd[EPW * 4], fax[EPW * 4];
  __shared__ R emat[EPW * 5];
  __shared__ int evalid[EPW];

  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  const int e = lane / LPE, r = lane % LPE;
  const bool act = e < EPW;                 // lane 63 computes a copy of lane 54 and never writes
  const int ec = act ? e : EPW - 1;
  const int q = act ? r : 0;
  const int g = blockIdx.x;
  const int elem = g * EPW + ec;
  const int cl = cluster_of(a, g * EPW);
  const bool valid = act && (elem < a.cl_vend[cl]);
  // lane slot of the element-group layouts; re-declared opaque at the top of
  // the long loops, so the compiler recomputes addresses there instead of
  // hoisting (and spilling) one per access
  int slot = ec * LPE + q;
  int base = RF::mb(W, w);                         // opaque at the loop tops (see slot)
  const int nb = RF::mb(W, w + 1) - base;
  auto has = [&](int lb) { return lb < NBN || lb < nb; };
  const bool own = LPE <= NBN || q < nb;           // this lane owns memory mode base + q
  const int mq = base + q;
  const int mword = (mq / LPE) * MM * 6 * NSLOT + ec * LPE + mq % LPE;   // its word (0, 0) in a group's La / Sa
  R* const reg = lds + ec * L::REGION;
  R* const grad = reg;
  R* const coup = reg + L::GRAD;
  R* const rx = reg + L::ROFF;
  double* const gs = gsh + (KIND == KIND_ADJ_UPDATE ? 0 : ec * NGS);
  const R* P = reinterpret_cast<const R*>(p.P) + (size_t)elem * NPARAM;
  const int* FI = p.FI + (size_t)elem * FI_WORDS;
  R* const Le = reinterpret_cast<R*>(ad.Le) + (size_t)g * B * NSLOT;
  R* const La = reinterpret_cast<R*>(ad.La) + (size_t)g * JB * MM * 6 * NSLOT;
  R* const S0 = reinterpret_cast<R*>(ad.S0);
  R* const S3 = reinterpret_cast<R*>(ad.S3);
  constexpr size_t SS = (size_t)4 * AR * FP;       // words of an element's face slot

  const bool is_stress = q < 6;
  R om[MM];
#pragma unroll
  for (int l = 0; l < MM; ++l) om[l] = M > 0 ? R(a.omega[l]) : R(0);

  // ------------------------------------------------ transposed update of the step that ends here
  // What leaves element k is u = trace(Qbar): 9 elastic rows and the 6
  // omega-weighted sums of the memory-variable rows, one slot per step parity;
  // the transposed predictions of k and of its face neighbours read it.  An
  // element with a coarser neighbour also keeps its last four steps in S3: the
  // coarser one reads two of them in the launch that writes a third.
  auto export_faces = [&](const R (&le)[NBX], const R (&lv)[6 * MM]) {
    const int n = step_fin_of(a, cl);
    if (act) {
#pragma unroll
      for (int lb = 0; lb < NBX; ++lb)
        if (has(lb)) rx[q * BS + base + lb] = le[lb];
      if (M > 0 && own)
#pragma unroll
        for (int c = 0; c < 6; ++c) {
          R v = R(0);
#pragma unroll
          for (int l = 0; l < MM; ++l) v += om[l] * lv[l * 6 + c];
          coup[c * BS + base + q] = v;
        }
    }
    __syncthreads();
    const int slot3 = FI[14];
    const bool coarser = (FI[12] & EF_HAS_COARSER) != 0;
    R* const d0 = S0 + ((size_t)(n & 1) * p.Kp + elem) * SS;
    R* const d3 = S3 + ((size_t)(n & 3) * p.N3 + slot3) * SS;
    auto row = [&](const R* src, int k) {
      R full[B], pt[4 * NTC];
#pragma unroll
      for (int b = 0; b < B; ++b) full[b] = src[b];
      RF::template trace_w<W>(w, full, pt);
#pragma unroll
      for (int ii = 0; ii < NTC; ++ii) {
        const int c = RF::template tchunk<W>(w, ii);
        if (ii < RF::template ntn<W> || c >= 0) {
          const int o = ((c / NCH) * AR + k) * FP + 4 * (c % NCH);
#pragma unroll
          for (int j = 0; j < 4; ++j) d0[o + j] = pt[4 * ii + j];
          if (coarser)
#pragma unroll
            for (int j = 0; j < 4; ++j) d3[o + j] = pt[4 * ii + j];
        }
      }
    };
    if (valid) {
      row(rx + q * BS, q);
      if (M > 0 && is_stress) row(coup + q * BS, 9 + q);
    }
  };
  R le[NBX];
  if constexpr (KIND == KIND_ADJ_UPDATE) {
    R lv[6 * MM];
#pragma unroll
    for (int lb = 0; lb < NBX; ++lb) le[lb] = has(lb) ? at(Le, (base + lb) * NSLOT + slot) : R(0);
#pragma unroll
    for (int k = 0; k < 6 * MM; ++k) lv[k] = M > 0 && own ? at(La, k * NSLOT + mword) : R(0);
    export_faces(le, lv);
    return;
  }

  // ------------------------------------------------ transposed prediction of the step that starts here
  // the wave's scratch block and this lane's place in it
  R* const SW = reinterpret_cast<R*>(ad.De) + ((size_t)g * W + w) * SC::WAVE;
  // (opaque at the loop tops, see slot; l1: lanes that own a mode, lvx: velocity lanes)
  int l1 = ec * NBX + q, lvx = ec * 3 + (q - 6);
  auto stV = [&](int d, const R* v) { st_words<NBX, SC::VL>(SW + SC::VX + d * SC::VXW, lvx, v); };
  auto ldV = [&](int d, R* v) { ld_words<NBX, SC::VL>(SW + SC::VX + d * SC::VXW, lvx, v); };
  auto st6 = [&](int at6, int d, const R* v) { st_words<6, SC::OL>(SW + at6 + d * SC::EPW6, l1, v); };
  auto ld6 = [&](int at6, int d, R* v) { ld_words<6, SC::OL>(SW + at6 + d * SC::EPW6, l1, v); };

  // This lane's parameters and LDS offsets.  Formed twice, before and after the
  // face phases (from opaque copies of the lane's row and address), so that they
  // hold no registers there, where the reverse flux needs the most.
  struct LanePar {
    R G[9], rho_inv, lam, mu, al[MM], bl[MM], wabc, wde, wc;
    int qi, qj, sa, sb, sc, sd, se;
  };
  auto lane_par = [&](const R* Pl, int ql, LanePar& x) {
    const bool st = ql < 6;
    x.qi = x.qj = 0;
    if (ql < 3) { x.qi = ql; x.qj = ql; }
    else if (ql == 3) { x.qi = 0; x.qj = 1; }
    else if (ql == 4) { x.qi = 1; x.qj = 2; }
    else if (ql == 5) { x.qi = 0; x.qj = 2; }
#pragma unroll
    for (int c = 0; c < 9; ++c) x.G[c] = Pl[c];
    x.rho_inv = Pl[9];
    x.lam = Pl[10];
    x.mu = Pl[11];
#pragma unroll
    for (int l = 0; l < MM; ++l) {
      x.al[l] = M > 0 ? Pl[14 + 2 * l] : R(0);
      x.bl[l] = M > 0 ? Pl[15 + 2 * l] : R(0);
    }
    // the star products: stress row ij: lam delta div v + mu (d_j v_i + d_i v_j)
    // + coupling; velocity row i: rho_inv sum_d d_d sigma_id
    if (st) {
      x.sa = aslot(6, 0) * BS; x.sb = aslot(7, 1) * BS; x.sc = aslot(8, 2) * BS;
      x.sd = aslot(6 + x.qi, x.qj) * BS; x.se = aslot(6 + x.qj, x.qi) * BS;
      x.wabc = ql < 3 ? x.lam : R(0); x.wde = x.mu; x.wc = R(1);
    } else {
      const int i = ql - 6;
      x.sa = aslot(sym_index(i, 0), 0) * BS; x.sb = aslot(sym_index(i, 1), 1) * BS;
      x.sc = aslot(sym_index(i, 2), 2) * BS;
      x.sd = x.sa; x.se = x.sb;
      x.wabc = x.rho_inv; x.wde = R(0); x.wc = R(0);
    }
  };
  const int cs = (is_stress ? q : 0) * BS;
  // the row's combined gradient adjoints, one row per reference direction
  R* const yr = grad + q * 3 * BS;

  for (int i = threadIdx.x; i < EPW * NGS; i += 64 * W) gsh[i] = 0.0;

  const int nn = step_new_of(a, cl);
  const bool has_b2 = (FI[12] & EF_HAS_FINER) != 0;
  const bool any_b2 = __syncthreads_or(has_b2);
  const int rec_slot = FI[15];
  // the parameters of each (element, face) pair the transposed surface reads,
  // staged in LDS once (the face items then read no global parameter): the
  // own face words (normal, area weight, outer impedances), the neighbour's
  // 1/rho, lam, mu, Zp, Zs and its words of the shared face
  {
    const int u = w * LPE + q;
#pragma unroll
    for (int k = 0; k < (4 * FSTW + W * LPE - 1) / (W * LPE); ++k) {
      const int idx = u + W * LPE * k;
      if (act && idx < 4 * FSTW) {
        const int i = idx / FSTW, wd = idx % FSTW;
        const int nbr = FI[3 * i], code = FI[3 * i + 1];
        R v = R(0);
        if (wd < 6) {
          v = P[20 + 6 * i + wd];
        } else if (nbr >= 0) {
          const R* Pn = reinterpret_cast<const R*>(p.P) + (size_t)nbr * NPARAM;
          v = wd < 11 ? Pn[9 + (wd - 6)] : Pn[20 + 6 * (code & 15) + (wd - 11)];
        }
        fst[(ec * 4 + i) * FSTW + wd] = v;
        if (wd == 0) {
          fnb[ec * 4 + i] = nbr;
          fcd[ec * 4 + i] = code;
          fax[ec * 4 + i] = FI[3 * i + 2];
        }
      }
    }
  }
  // the element words the face items of other lanes read
  if (w == 0 && act && q == 0) {
#pragma unroll
    for (int k = 0; k < 5; ++k) emat[ec * 5 + k] = P[9 + k];
    evalid[ec] = valid ? 1 : 0;
  }

  // rho dJ/drho of the products (see the head of the file), this lane's part: in
  // LDS during the face phases, the register peak, then in a register
  double* const grl = grsh + w * NSLOT + slot;    // (lane 63 as lane 54)
  *grl = 0.0;
  // - <x, velocity rows of the row exchange>, own modes
  auto pair_exchange = [&](const R (&x)[NBX]) {
    double s = 0.0;
    if (!is_stress)
#pragma unroll
      for (int lb = 0; lb < NBX; ++lb)
        if (has(lb)) s += (double)(x[lb] * rx[q * BS + base + lb]);
    *grl -= s;
  };

  // ---------------------------------------------- forward recompute: D_d, T, T2
  R te[NBX], t2[NBX];
  {
    LanePar x;
    lane_par(P, q, x);
    const int sa = x.sa, sb = x.sb, sc = x.sc, sd = x.sd, se = x.se;
    // gradient slots this lane writes
    R* const gw0 = grad + aslot(q, 0) * BS;
    R* const gw1 = grad + aslot(q, 1) * BS;
    R* const gw2 = grad + aslot(q, 2) * BS;
    const R* Se = reinterpret_cast<const R*>(ad.Se) + (size_t)g * B * NSLOT;
    const R* Sa = reinterpret_cast<const R*>(ad.Sa) + (size_t)g * JB * MM * 6 * NSLOT;
    R dm[MM][6];
#pragma unroll
    for (int lb = 0; lb < NBX; ++lb) {
      te[lb] = R(0);
      t2[lb] = R(0);
      if (has(lb) && act) rx[q * BS + base + lb] = at(Se, (base + lb) * NSLOT + slot);
    }
#pragma unroll
    for (int l = 0; l < MM; ++l)
#pragma unroll
      for (int c = 0; c < 6; ++c) dm[l][c] = (M > 0 && own) ? at(Sa, (l * 6 + c) * NSLOT + mword) : R(0);
#pragma unroll 1
    for (int d = 0; d < O; ++d) {
      asm volatile("" : "+v"(slot), "+s"(base), "+v"(l1), "+v"(lvx));
      const R c_d = R(a.tc[cl][d]), h_d = R(a.th[cl][d]);
      const bool more = d + 1 < O;
      __syncthreads();
      {
        R dv[NBX];
#pragma unroll
        for (int lb = 0; lb < NBX; ++lb) dv[lb] = has(lb) ? rx[q * BS + base + lb] : R(0);
#pragma unroll
        for (int lb = 0; lb < NBX; ++lb) { te[lb] += c_d * dv[lb]; t2[lb] += h_d * dv[lb]; }
      }
      if (!more) break;
      {
        R full[B];
#pragma unroll
        for (int b = 0; b < B; ++b) full[b] = rx[q * BS + b];
        RF::template ck_grad_w<W>(w, full, x.G, gw0, gw1, gw2);
      }
      __syncthreads();
      if (own) {
        const int b = base + q;
        R eps[6];
        eps[0] = grad[aslot(6, 0) * BS + b];
        eps[1] = grad[aslot(7, 1) * BS + b];
        eps[2] = grad[aslot(8, 2) * BS + b];
        eps[3] = R(0.5) * (grad[aslot(6, 1) * BS + b] + grad[aslot(7, 0) * BS + b]);
        eps[4] = R(0.5) * (grad[aslot(7, 2) * BS + b] + grad[aslot(8, 1) * BS + b]);
        eps[5] = R(0.5) * (grad[aslot(6, 2) * BS + b] + grad[aslot(8, 0) * BS + b]);
        st6(SC::EP, d, eps);
        if (M > 0) {
          R cp[6] = {R(0), R(0), R(0), R(0), R(0), R(0)};
#pragma unroll
          for (int l = 0; l < MM; ++l) {
            const R tr = dm[l][0] + dm[l][1] + dm[l][2];
#pragma unroll
            for (int c = 0; c < 6; ++c) cp[c] -= x.bl[l] * dm[l][c] + (c < 3 ? x.al[l] * tr : R(0));
#pragma unroll
            for (int c = 0; c < 6; ++c) dm[l][c] = om[l] * (eps[c] - dm[l][c]);
          }
          if (act)
#pragma unroll
            for (int c = 0; c < 6; ++c) coup[c * BS + b] = cp[c];
        }
      }
      // the coupling rows of a mode are read by the stress rows of the wave
      // that owns the mode
      if (M > 0) wave_lds_sync();
      // next derivative, own modes, into the row exchange (every lane's
      // full-row reads ended before the barrier after the products)
      {
        R nx[NBX], sab[NBX];
#pragma unroll
        for (int lb = 0; lb < NBX; ++lb) {
          const int b = base + lb;
          sab[lb] = R(0);
          nx[lb] = R(0);
          if (has(lb)) {
            sab[lb] = grad[sa + b] + grad[sb + b] + grad[sc + b];
            const R cq = M > 0 ? x.wc * coup[cs + b] : R(0);
            nx[lb] = x.wabc * sab[lb] + x.wde * (grad[sd + b] + grad[se + b]) + cq;
          }
        }
        if (!is_stress && rec_slot >= 0 && act) stV(d, sab);
        if (act)
#pragma unroll
          for (int lb = 0; lb < NBX; ++lb)
            if (has(lb)) rx[q * BS + base + lb] = nx[lb];
      }
    }
  }
  __syncthreads();

  // ---------------------------------------------- face phases
  // The element's traces (full rows through the row exchange, each wave its
  // trace chunks), then per (face, face mode) the Godunov reverse mode, then
  // the lift of the trace adjoints to the wave's modes.
  R lte[NBX], lt2[NBX];
#pragma unroll
  for (int lb = 0; lb < NBX; ++lb) { lte[lb] = R(0); lt2[lb] = R(0); }
  R* const pm = reg;                               // face area (over grad and coup)
  auto face_phase = [&](const bool b2phase, const R (&tint)[NBX], R (&acc)[NBX]) {
    if (act)
#pragma unroll
      for (int lb = 0; lb < NBX; ++lb)
        if (has(lb)) rx[q * BS + base + lb] = tint[lb];
    __syncthreads();
    {
      R full[B], pt[4 * NTC];
#pragma unroll
      for (int b = 0; b < B; ++b) full[b] = rx[q * BS + b];
      RF::template trace_w<W>(w, full, pt);
      if (act)
#pragma unroll
        for (int ii = 0; ii < NTC; ++ii) {
          const int c = RF::template tchunk<W>(w, ii);
          if (ii < RF::template ntn<W> || c >= 0)
#pragma unroll
            for (int k = 0; k < 4; ++k) pm[((c / NCH) * LPE + q) * FS + 4 * (c % NCH) + k] = pt[4 * ii + k];
        }
    }
    __syncthreads();
    // items (face i, mode f) of the whole group, one segment of SEG lanes per
    // (element, face) pair (SEG > F: 4, 8, 16 at O = 2, 3, 4..5): segment
    // SPW (W rr + w) + lane / SEG takes element s % 7 and face s / 7 (s < 28),
    // lane f = lane % SEG its mode f (f < F).  A segment's modes are
    // contiguous in the slots and in the trace area, and its gradient words
    // are summed over it with DPP and written once by its last lane, to words of
    // the pair's own: the faces of an element are in different waves, whose sums
    // into one set of words came in a timing-dependent order (that took, per reverse
    // cycle, O = 5 m=3 35k tets 864 us against 872, O = 4 m=0 353 against 356, FP64
    // O = 4 5k 141 against 150).
    constexpr int SEG = F < 4 ? 4 : F < 8 ? 8 : 16, SPW = 64 / SEG;
    // (the sums are FP64 up to O = 3, where each costs two or three additions; at
    // O = 4, 5 FP32 over sixteen lanes, FP64 from there on)
    typedef typename std::conditional<sizeof(R) == 8 || O <= 3, double, float>::type WS;
#pragma unroll 1
    for (int rr = 0; rr < (4 * EPW + SPW * W - 1) / (SPW * W); ++rr) {
      const int ln = lane_id(), f = ln % SEG;
      const int r8 = SPW * (W * rr + w) + ln / SEG;
      const bool pair = r8 < 4 * EPW;
      const int pe = pair ? r8 % EPW : 0, i = pair ? r8 / EPW : 0;
      const bool pvalid = pair && evalid[pe] != 0;
      const int nbr = fnb[pe * 4 + i], code = fcd[pe * 4 + i];
      const int bc = (code >> 4) & 15, j = code & 15, rel = ((code >> 8) & 15) - 1;
      // the flux across face i that read this element's buffer: B1 or B3 (its
      // whole-step trace), in the second phase B2 (a finer neighbour's)
      const bool nflux = pvalid && nbr >= 0 && (!b2phase || rel < 0);
      R pbo[7], pbn[7];
#pragma unroll
      for (int k = 0; k < 7; ++k) { pbo[k] = R(0); pbn[k] = R(0); }
      if (pair && f < F) {
        // every global operand of the item first, into registers zeroed
        // beforehand, and no use inside the branches that load them: one
        // memory latency per item
        R u0[15], ua[15], ub[15];
#pragma unroll
        for (int k = 0; k < 15; ++k) { u0[k] = R(0); ua[k] = R(0); ub[k] = R(0); }
        if (!b2phase && pvalid) {
          const R* x = S0 + ((size_t)(nn & 1) * p.Kp + (size_t)g * EPW + pe) * SS + (size_t)i * AR * FP + f;
#pragma unroll
          for (int k = 0; k < AR; ++k) u0[k] = x[k * FP];
        }
        if (nflux) {
          // same cluster: its step nn; coarser: the step nn / 2 it is in;
          // finer: its steps 2 nn and 2 nn + 1, whose fluxes read B2 and
          // B1 - B2: B1 gets the second, B2 the difference
          const size_t o = (size_t)j * AR * FP + f;
          const size_t aux = (size_t)fax[pe * 4 + i];
          const R* const x = rel < 0 ? S3 + ((size_t)((2 * nn + 1) & 3) * p.N3 + aux) * SS + o
                                     : S0 + ((size_t)((rel == 0 ? nn : nn >> 1) & 1) * p.Kp + (size_t)nbr) * SS + o;
#pragma unroll
          for (int k = 0; k < AR; ++k) ua[k] = x[k * FP];
          if (b2phase) {
            const R* const y = S3 + ((size_t)((2 * nn) & 3) * p.N3 + aux) * SS + o;
#pragma unroll
            for (int k = 0; k < AR; ++k) ub[k] = y[k * FP];
          }
        }
        const R* const fs = fst + (pe * 4 + i) * FSTW;
        const R* const em = emat + pe * 5;
        R fpv[6], pnv[5], fnv[6], ev[5];
#pragma unroll
        for (int k = 0; k < 6; ++k) fpv[k] = fs[k];
#pragma unroll
        for (int k = 0; k < 5; ++k) pnv[k] = fs[6 + k];
#pragma unroll
        for (int k = 0; k < 6; ++k) fnv[k] = fs[11 + k];
#pragma unroll
        for (int k = 0; k < 5; ++k) ev[k] = em[k];
        R u1[15];
#pragma unroll
        for (int k = 0; k < 15; ++k) u1[k] = b2phase ? ub[k] - ua[k] : ua[k];
        R* const pmp = lds + pe * L::REGION;             // the trace area of element pe
        R tr[9], zero9[9], tb[9], ob[9];
#pragma unroll
        for (int k = 0; k < 9; ++k) { tr[k] = pmp[(i * LPE + k) * FS + f]; zero9[k] = R(0); tb[k] = R(0); ob[k] = R(0); }
        if (!b2phase) {
          // own flux: the element's trace is the inside state; its
          // (rho_inv, lam, mu, Zp, Zs) are ev
          const R zpp = bc == 0 ? fpv[4] : ev[3], zsp = bc == 0 ? fpv[5] : ev[4];
          godunov_adj<R>(u0, tr, zero9, fpv[0], fpv[1], fpv[2], ev[3], ev[4], zpp, zsp, ev[1], ev[2], ev[0], fpv[3], bc,
                         tb, ob, pbo);
        }
        if (nflux) {
          // the neighbour's flux, seen from its side: (rho_inv, lam, mu, Zp, Zs)
          // of the neighbour are its words 9..13
          godunov_adj<R>(u1, zero9, tr, fnv[0], fnv[1], fnv[2], pnv[3], pnv[4], fnv[4], fnv[5], pnv[1], pnv[2], pnv[0],
                         fnv[3], 0, ob, tb, pbn);
        }
#pragma unroll
        for (int k = 0; k < 9; ++k) pmp[(i * LPE + k) * FS + f] = tb[k];
      }
      // the segment sums, every lane taking part (uniform control flow)
      WS so[7], sn[7];
#pragma unroll
      for (int k = 0; k < 7; ++k) { so[k] = seg_sum<SEG>(WS(pbo[k])); sn[k] = seg_sum<SEG>(WS(pbn[k])); }
      if (f == SEG - 1 && pvalid) {
        double* const gp = gsh + pe * NGS + 7 * i;
        if (!b2phase)
#pragma unroll
          for (int k = 0; k < 7; ++k) gp[k] = so[k];
        if (nflux)
#pragma unroll
          for (int k = 0; k < 7; ++k) gadd(gp, NG_NBR + k, sn[k]);
      }
    }
    __syncthreads();
    {
      R pf[4 * FP], lr[NBX];
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int f2 = 0; f2 < FP; ++f2) pf[i * FP + f2] = pm[(i * LPE + q) * FS + f2];
      RF::template lift_w<W>(w, pf, lr);
#pragma unroll
      for (int lb = 0; lb < NBX; ++lb) acc[lb] += lr[lb];
    }
    __syncthreads();
  };
  // (the row exchange holds the integrals of the phase until the next writes it)
  if (any_b2) {
    face_phase(true, t2, lt2);
    pair_exchange(lt2);
  }
  face_phase(false, te, lte);
  pair_exchange(lte);

  // ---------------------------------------------- volume kernel
  // V = -(lam delta div v + mu (d_j v_i + d_i v_j)) (stress), -rho_inv div sigma (velocity), -omega_l eps (memory)
  LanePar x;
  {
    const R* Pl = P;
    int ql = q;
    asm volatile("" : "+v"(Pl), "+v"(ql));
    lane_par(Pl, ql, x);
  }
  const R rho_inv = x.rho_inv, lam = x.lam, mu = x.mu;
  const int qi = x.qi, qj = x.qj, sa = x.sa, sb = x.sb, sc = x.sc;
  R al[MM], bl[MM];
#pragma unroll
  for (int l = 0; l < MM; ++l) { al[l] = x.al[l]; bl[l] = x.bl[l]; }
#pragma unroll
  for (int lb = 0; lb < NBX; ++lb) le[lb] = has(lb) ? at(Le, (base + lb) * NSLOT + slot) : R(0);
  // the directions of this row's gradient-entry adjoints (write_y) and their
  // columns of G', re-read by lane-dependent index (selecting from the register
  // copy would put that into scratch memory)
  const int vi = is_stress ? 0 : q - 6;
  const int k0 = is_stress ? qj : vi, k1 = is_stress ? qi : (vi + 1) % 3, k2 = is_stress ? 0 : (vi + 2) % 3;
  R g0[3], g1[3], g2[3];
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    g0[c] = P[3 * c + k0];
    g1[c] = P[3 * c + k1];
    g2[c] = P[3 * c + k2];
  }
  {
    // (the row exchange still holds the time integrals of the last face phase)
    R full[B];
#pragma unroll
    for (int b = 0; b < B; ++b) full[b] = rx[q * BS + b];
    RF::template vol_grad_w<W>(w, full, x.G, grad + aslot(q, 0) * BS, grad + aslot(q, 1) * BS, grad + aslot(q, 2) * BS);
  }
  __syncthreads();
  // Material words, summed in registers over the whole kernel: a product's
  // adjoint rows x paired with the strain rates give dJ/dlam (tr x tr eps, row by
  // row: the rows' FP32 sum would round before FP64) and dJ/dmu (2 x : eps), mode
  // by mode in the lane that owns the mode.
  double gl = 0.0, gm = 0.0, gr = *grl;
  auto strain_words = [&](const R* eps, const R* x, const double sign) {
    double s = 0.0;
#pragma unroll
    for (int c = 0; c < 6; ++c) s += (double)(x[c] * (R(2) * eps[c]));
    gm += sign * s;
    const R div = eps[0] + eps[1] + eps[2];
    gl += sign * ((double)(x[0] * div) + (double)(x[1] * div) + (double)(x[2] * div));
  };
  if (!is_stress) {
    double s = 0.0;
#pragma unroll
    for (int lb = 0; lb < NBX; ++lb) {
      const int b = base + lb;
      if (has(lb)) s += (double)(le[lb] * (grad[sa + b] + grad[sb + b] + grad[sc + b]));
    }
    gr += (double)rho_inv * s;
  }
  // exchange: elastic adjoint rows, omega-weighted memory-variable adjoints
  // (own modes: the rows and coupling rows that write_y reads)
  if (act)
#pragma unroll
    for (int lb = 0; lb < NBX; ++lb)
      if (has(lb)) rx[q * BS + base + lb] = le[lb];
  wave_lds_sync();
  if (own) {
    const int b = base + q;
    R eps[6], xr[6];
    eps[0] = grad[aslot(6, 0) * BS + b];
    eps[1] = grad[aslot(7, 1) * BS + b];
    eps[2] = grad[aslot(8, 2) * BS + b];
    eps[3] = R(0.5) * (grad[aslot(6, 1) * BS + b] + grad[aslot(7, 0) * BS + b]);
    eps[4] = R(0.5) * (grad[aslot(7, 2) * BS + b] + grad[aslot(8, 1) * BS + b]);
    eps[5] = R(0.5) * (grad[aslot(6, 2) * BS + b] + grad[aslot(8, 0) * BS + b]);
#pragma unroll
    for (int c = 0; c < 6; ++c) xr[c] = rx[c * BS + b];
    strain_words(eps, xr, -1.0);
    if (M > 0) {
      R lv[6 * MM];
#pragma unroll
      for (int k = 0; k < 6 * MM; ++k) lv[k] = at(La, k * NSLOT + mword);
      // Lambda_d = sum_l omega_l^2 C_l(d) Qbar^a_l, C_l(d) = sum_{k >= d}
      // (-omega_l)^(k - d) c_k: the Qbar^a part of the omega-weighted
      // memory-variable adjoints of step d (see the reverse loop)
      R Cl[MM];
#pragma unroll
      for (int l = 0; l < MM; ++l) Cl[l] = R(0);
#pragma unroll
      for (int d = O - 1; d >= 0; --d) {
        const R c_d = R(a.tc[cl][d]);
        R lm[6];
#pragma unroll
        for (int l = 0; l < MM; ++l) Cl[l] = c_d - om[l] * Cl[l];
#pragma unroll
        for (int c = 0; c < 6; ++c) {
          lm[c] = R(0);
#pragma unroll
          for (int l = 0; l < MM; ++l) lm[c] += om[l] * om[l] * Cl[l] * lv[l * 6 + c];
        }
        st6(SC::LM, d, lm);
      }
      if (act)
#pragma unroll
        for (int c = 0; c < 6; ++c) {
          R v = R(0);
#pragma unroll
          for (int l = 0; l < MM; ++l) v += om[l] * lv[l * 6 + c];
          coup[c * BS + b] = v;
          gr += (double)(v * eps[c]);
        }
    }
  }
  wave_lds_sync();
  // Gradient-entry adjoints of this row, own modes, combined with G' to the
  // reference directions (sign s: -1 for the volume kernel, +1 for the time
  // kernel's next derivative).  Combined here, mode by mode, they cost nine
  // multiply-adds per own mode instead of nine per mode in every wave's
  // product.  Branch-free, every lane up to three (row, direction) entries:
  //   velocity row i, directions i, i + 1, i + 2 (mod 3): (1 + delta) mu on
  //     exchange row sym(i, k), 1 or 1/2 on coupling row sym(i, k) (anelastic
  //     only), in the first lam on the sum of the normal-stress rows;
  //   stress row (qi, qj), directions qj and, off the diagonal, qi: rho_inv on
  //     the velocity row of the other index; the rest zero
  const int r0 = (is_stress ? 6 + qi : vi) * BS, r1 = (is_stress ? 6 + qj : sym_index(vi, k1)) * BS,
            r2 = (is_stress ? 0 : sym_index(vi, k2)) * BS;
  const int c0 = is_stress ? 0 : vi * BS;          // (coupling rows: as r1, r2 in velocity lanes, unused else)
  auto write_y = [&](const R sgn) {
    const R A0 = sgn * (is_stress ? rho_inv : R(2) * mu), Lw = is_stress ? R(0) : sgn * lam;
    const R A1 = sgn * (is_stress ? (qi == qj ? R(0) : rho_inv) : mu), A2 = is_stress ? R(0) : sgn * mu;
    const R C0 = is_stress ? R(0) : sgn, C1 = R(0.5) * C0;
    const int x1 = is_stress ? 0 : r1, x2 = is_stress ? 0 : r2;   // coupling rows
    // reads of three modes, then their stores (a store may alias the next
    // mode's reads for the compiler, which would wait for each)
    constexpr int CH = 3;
#pragma unroll
    for (int l0 = 0; l0 < NBX; l0 += CH) {
      R y[CH][3];
#pragma unroll
      for (int k = 0; k < CH; ++k) {
        const int lb = l0 + k, b = base + lb;
        if (lb < NBX && has(lb)) {
          R v0 = A0 * rx[r0 + b] + Lw * (rx[b] + rx[BS + b] + rx[2 * BS + b]);
          R v1 = A1 * rx[r1 + b], v2 = A2 * rx[r2 + b];
          if (M > 0) {
            v0 += C0 * coup[c0 + b];
            v1 += C1 * coup[x1 + b];
            v2 += C1 * coup[x2 + b];
          }
#pragma unroll
          for (int c = 0; c < 3; ++c) y[k][c] = g0[c] * v0 + g1[c] * v1 + g2[c] * v2;
        }
      }
      if (act)
#pragma unroll
        for (int k = 0; k < CH; ++k)
          if (l0 + k < NBX && has(l0 + k))
#pragma unroll
            for (int c = 0; c < 3; ++c) yr[c * BS + base + l0 + k] = y[k][c];
    }
  };
  // adds a transposed product of the combined adjoints to v
  auto add_product = [&](const bool vol, R (&v)[NBX]) {
    R out[NBX];
    if (vol) RF::template vol_grad_T_w<W>(w, yr, yr + BS, yr + 2 * BS, out);
    else RF::template ck_grad_T_w<W>(w, yr, yr + BS, yr + 2 * BS, out);
#pragma unroll
    for (int lb = 0; lb < NBX; ++lb) v[lb] += out[lb];
  };
  // (no barrier: the wave's modes of these rows were read in the wave alone)
  write_y(R(-1));
  __syncthreads();
  add_product(true, lte);
  // (no barrier: the reverse loop's first LDS writes are the wave's own
  // modes of the exchange rows, which the transposed product does not read)

  // ---------------------------------------------- time kernel backwards
  // nbe: adjoint of the next elastic derivative.  The adjoint of D_d^a in
  // closed form: with P_l(d) = sum_{k >= d} (-omega_l)^(k - d) cq_k (cq_k: the
  // coupling adjoint of step k),
  //   abar_{l,d} = -omega_l C_l(d) Qbar^a_l - b_l P_l(d) - a_l tr(P_l(d)) I,
  // so the six words P_l per mechanism are carried in registers.  Its
  // omega-weighted sum over l is what the next (lower) derivative needs.  The
  // anelastic-weight words -sum_d cq_d : D_d^a_l follow from the same P_l:
  // D_d^a is the state's D_0^a and the strain rates eps_k of the steps k < d
  // in the forward recursion, so the words are -omega_l eps_k : P_l(k + 1)
  // step by step and -D_0^a_l : P_l(0) at the end.
  R nbe[NBX], Pl[MM][6];
  double gab[2 * MM];
#pragma unroll
  for (int lb = 0; lb < NBX; ++lb) nbe[lb] = R(0);
#pragma unroll
  for (int l = 0; l < MM; ++l) {
    gab[2 * l] = gab[2 * l + 1] = 0.0;
#pragma unroll
    for (int c = 0; c < 6; ++c) Pl[l][c] = R(0);
  }
  auto anelastic_words = [&](int l, const R* x, const R f) {
    gab[2 * l] -= (double)(f * (Pl[l][0] + Pl[l][1] + Pl[l][2]) * (x[0] + x[1] + x[2]));
#pragma unroll
    for (int c = 0; c < 6; ++c) gab[2 * l + 1] -= (double)(f * Pl[l][c] * x[c]);
  };
  R* const recDb = reinterpret_cast<R*>(ad.recDb);
  const R* const Seg = reinterpret_cast<const R*>(ad.Se) + (size_t)g * B * NSLOT;
#pragma unroll 1
  for (int d = O - 1; d >= 0; --d) {
    asm volatile("" : "+v"(slot), "+s"(base), "+v"(l1), "+v"(lvx));
    const R c_d = R(a.tc[cl][d]), h_d = R(a.th[cl][d]);
    const bool more = d + 1 < O;
    R cur[NBX];
    // the step's scratch operands in one batch
    R eps[6], lm[6], l1m[6];
#pragma unroll
    for (int c = 0; c < 6; ++c) { eps[c] = R(0); lm[c] = R(0); l1m[c] = R(0); }
    if (M > 0 && own) ld6(SC::LM, d, lm);
    if (more && own) {
      ld6(SC::EP, d, eps);
      if (M > 0) ld6(SC::LM, d + 1, l1m);
    }
#pragma unroll
    for (int lb = 0; lb < NBX; ++lb) cur[lb] = c_d * lte[lb] + h_d * lt2[lb];
    if (rec_slot >= 0 && valid) {
      R vx[NBX];                                  // D_d (d > 0: times rho), velocity rows
#pragma unroll
      for (int lb = 0; lb < NBX; ++lb) vx[lb] = R(0);
      if (!is_stress) {
        if (d > 0) ldV(d - 1, vx);
        else
#pragma unroll
          for (int lb = 0; lb < NBX; ++lb)
            if (has(lb)) vx[lb] = at(Seg, (base + lb) * NSLOT + slot);
      }
      R* rd = recDb + (((size_t)rec_slot * O + d) * LPE + q) * B + base;
#pragma unroll
      for (int lb = 0; lb < NBX; ++lb)
        if (has(lb)) {
          const R v = rd[lb];
          cur[lb] += v;
          rd[lb] = R(0);
          if (!is_stress) gr -= (double)(v * (d > 0 ? rho_inv * vx[lb] : vx[lb]));
        }
    }
    if (more) {
      if (act)
#pragma unroll
        for (int lb = 0; lb < NBX; ++lb)
          if (has(lb)) rx[q * BS + base + lb] = nbe[lb];
      // (coup holds the omega-weighted sums of the next memory-variable
      // adjoint, written by the coupling block of the step before)
      __syncthreads();
      if (own) {
        R x[6];
#pragma unroll
        for (int c = 0; c < 6; ++c) x[c] = rx[c * BS + base + q];
        strain_words(eps, x, 1.0);
        if (M > 0)
#pragma unroll
          for (int c = 0; c < 6; ++c) gr += (double)(l1m[c] * eps[c]);
      }
      write_y(R(1));
      __syncthreads();
      add_product(false, cur);
      // (no barrier: the coupling block below writes the wave's own modes of
      // the exchange and coupling rows, which the transposed product does
      // not read; the next iteration's products follow its first barrier)
    }
    if (M > 0) {
      // the coupling E: cq_d enters the volume term c_d cq_d and the next
      // derivative
      if (is_stress && act)
#pragma unroll
        for (int lb = 0; lb < NBX; ++lb)
          if (has(lb)) rx[q * BS + base + lb] = c_d * le[lb] + (more ? nbe[lb] : R(0));
      // the stress rows of a mode are read by its owner, in the same wave
      wave_lds_sync();
      if (own) {
        const int b = base + q;
        R cqb[6], ws[6];
#pragma unroll
        for (int c = 0; c < 6; ++c) cqb[c] = rx[c * BS + b];
#pragma unroll
        for (int c = 0; c < 6; ++c) ws[c] = -lm[c];
#pragma unroll
        for (int l = 0; l < MM; ++l) {
          anelastic_words(l, eps, om[l]);
#pragma unroll
          for (int c = 0; c < 6; ++c) Pl[l][c] = cqb[c] - om[l] * Pl[l][c];
          const R pt = om[l] * al[l] * (Pl[l][0] + Pl[l][1] + Pl[l][2]);
#pragma unroll
          for (int c = 0; c < 6; ++c) ws[c] -= om[l] * bl[l] * Pl[l][c] + (c < 3 ? pt : R(0));
        }
        // the coupling term of the next (lower) derivative's adjoint: coup
        // is not touched again before the next step reads it
        if (act)
#pragma unroll
          for (int c = 0; c < 6; ++c) coup[c * BS + b] = ws[c];
      }
      wave_lds_sync();
    }
#pragma unroll
    for (int lb = 0; lb < NBX; ++lb) nbe[lb] = cur[lb];
  }
  // Qbar += the adjoint of D_0: every load first, then every store (a
  // read-modify-write per word would wait one memory latency per word: the
  // compiler must assume each store may alias the next load)
  R lv[6 * MM];
#pragma unroll
  for (int k = 0; k < 6 * MM; ++k) lv[k] = R(0);
  if (M > 0 && own) {
    const R* Sa = reinterpret_cast<const R*>(ad.Sa) + (size_t)g * JB * MM * 6 * NSLOT;
    R dm[MM][6];
#pragma unroll
    for (int l = 0; l < MM; ++l)
#pragma unroll
      for (int c = 0; c < 6; ++c) {
        lv[l * 6 + c] = at(La, (l * 6 + c) * NSLOT + mword);
        dm[l][c] = at(Sa, (l * 6 + c) * NSLOT + mword);
      }
#pragma unroll
    for (int l = 0; l < MM; ++l) {
      anelastic_words(l, dm[l], R(1));
      R C0 = R(0);
#pragma unroll
      for (int d = O - 1; d >= 0; --d) C0 = R(a.tc[cl][d]) - om[l] * C0;
      const R pt = al[l] * (Pl[l][0] + Pl[l][1] + Pl[l][2]);
#pragma unroll
      for (int c = 0; c < 6; ++c) {
        const R sp = bl[l] * Pl[l][c] + (c < 3 ? pt : R(0));
        lv[l * 6 + c] -= om[l] * C0 * lv[l * 6 + c] + sp;
        gr -= (double)(sp * dm[l][c]);
      }
    }
    if (valid)
#pragma unroll
      for (int k = 0; k < 6 * MM; ++k) at(La, k * NSLOT + mword) = lv[k];
  }
  if (!is_stress)
#pragma unroll
    for (int lb = 0; lb < NBX; ++lb)
      if (has(lb)) gr += (double)(nbe[lb] * at(Seg, (base + lb) * NSLOT + slot));
#pragma unroll
  for (int lb = 0; lb < NBX; ++lb) {
    le[lb] += nbe[lb];
    if (has(lb) && valid) at(Le, (base + lb) * NSLOT + slot) = le[lb];
  }
  // the waves add their words one after the other (LDS atomics of all at once
  // would sum in a timing-dependent order; the face words are pair by pair, so a
  // sweep repeats bit for bit)
#pragma unroll
  for (int ww = 0; ww < W; ++ww) {
    if (w == ww && valid) {
      gadd(gs, NG_RHO, gr);
      if (own) {
        gadd(gs, NG_RHO + 1, gl);
        gadd(gs, NG_RHO + 2, gm);
        if (M > 0)
#pragma unroll
          for (int k = 0; k < 2 * MM; ++k) gadd(gs, NG_AB + k, gab[k]);
      }
    }
    __syncthreads();
  }
  // the element's gradient words, split between the waves, loads first
  if (valid) {
    constexpr int NI = (NG + W * LPE - 1) / (W * LPE);
    double* const gg = ad.gacc + (size_t)elem * NG;
    double x[NI];
#pragma unroll
    for (int k = 0; k < NI; ++k) {
      const int i = q + LPE * (w + W * k);
      x[k] = i < NG ? gg[i] : 0.0;
    }
#pragma unroll
    for (int k = 0; k < NI; ++k) {
      const int i = q + LPE * (w + W * k);
      if (i < NG) gg[i] = x[k] + gsh[ec * NGS + i];
    }
  }
  if constexpr (KIND == KIND_ADJ_FUSED) export_faces(le, lv);
}

// Chain rule from the per-element gradient words to d/d(rho, vp, vs), one
// thread per element (internal order), gathering what the face neighbours
// accumulated about this element.  mat [Kp][3 + 2m]: rho, vp, vs, Yp_l, Ys_l
// (rho = 0 marks padding).  out [Kp][3].
__device__ __forceinline__ void add_param(double* g, int which, double v, double rho, double vp, double vs) {
  switch (which) {
    case 0: g[0] -= v / (rho * rho); break;                                              // 1/rho
    case 1: g[0] += v * (vp * vp - 2 * vs * vs); g[1] += v * 2 * rho * vp; g[2] -= v * 4 * rho * vs; break;  // lam
    case 2: g[0] += v * vs * vs; g[2] += v * 2 * rho * vs; break;                        // mu
    case 3: g[0] += v * vp; g[1] += v * rho; break;                                       // Zp
    default: g[0] += v * vs; g[2] += v * rho; break;                                      // Zs
  }
}

__global__ void k_material_gradient(const double* gacc, const int* FI, const double* mat, int M, long long Kp,
                                    double* out) {
  const long long k = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= Kp) return;
  const int mw = 3 + 2 * M;
  const double rho = mat[k * mw], vp = mat[k * mw + 1], vs = mat[k * mw + 2];
  double g[3] = {0.0, 0.0, 0.0};
  if (rho > 0.0) {
    const double* x = gacc + k * NG;
    // the products: rho at fixed vp, vs, then the moduli's vp, vs
    g[0] += x[NG_RHO] / rho;
    g[1] += x[NG_RHO + 1] * 2 * rho * vp;
    g[2] += (x[NG_RHO + 2] - 2 * x[NG_RHO + 1]) * 2 * rho * vs;
    for (int l = 0; l < M; ++l) {   // a_l = rho vp^2 Yp - 2 rho vs^2 Ys, b_l = 2 rho vs^2 Ys
      const double yp = mat[k * mw + 3 + 2 * l], ys = mat[k * mw + 4 + 2 * l];
      const double ga = x[NG_AB + 2 * l], gb = x[NG_AB + 1 + 2 * l];
      g[1] += ga * 2 * rho * vp * yp;
      g[2] += -ga * 4 * rho * vs * ys + gb * 4 * rho * vs * ys;
    }
    const int* fi = FI + k * FI_WORDS;
    for (int i = 0; i < 4; ++i) {
      for (int t = 0; t < 5; ++t) add_param(g, t, x[7 * i + t], rho, vp, vs);
      const int n = fi[3 * i];
      if (n < 0) {   // the outside impedances are the element's own
        add_param(g, 3, x[7 * i + 5], rho, vp, vs);
        add_param(g, 4, x[7 * i + 6], rho, vp, vs);
        continue;
      }
      const int j = fi[3 * i + 1] & 15;          // the neighbour's face towards this element
      const double* y = x + NG_NBR + 7 * i;      // this element's Zp, Zs in the neighbour's flux
      add_param(g, 3, y[5], rho, vp, vs);
      add_param(g, 4, y[6], rho, vp, vs);
      const double* xn = gacc + (long long)n * NG;
      add_param(g, 3, xn[7 * j + 5], rho, vp, vs);    // this element's impedances in the neighbour's own flux
      add_param(g, 4, xn[7 * j + 6], rho, vp, vs);
      const double* yn = xn + NG_NBR + 7 * j;         // this element's own flux, accumulated by the neighbour
      for (int t = 0; t < 5; ++t) add_param(g, t, yn[t], rho, vp, vs);
    }
  }
  out[k * 3] = g[0];
  out[k * 3 + 1] = g[1];
  out[k * 3 + 2] = g[2];
}

// adjoint of the receiver samples: the derivatives of a receiver element get
// sum_s (t_s - t^n)^d / d! * seisbar_s phi(x_r) for the samples of its receivers
// in the step that starts at this level.  One workgroup per element (that of its
// first receiver; chain[r] = 2 (next receiver in the element + 1) + (first)), one
// thread per (quantity, mode), receivers and their few samples in order: no
// atomics, so the sum is the same every time.  (One thread per quantity, with all
// modes one after the other, took 45 us a level at O = 5 and 32 receivers.)
template <class R, int O, int M>
__global__ void k_receivers_adj(KPtrs p, APtrs ad, LevelArgs a, RecArgs r, const int* chain, const double* seis_b) {
  constexpr int B = edg_gen::Ref<O>::B;
  int rec = blockIdx.x;
  const int q = threadIdx.x / B, b = threadIdx.x % B;
  const int elem = r.elem[rec];
  if (!(chain[rec] & 1) || elem >= a.end || q >= LPE) return;
  R* D = reinterpret_cast<R*>(ad.recDb) + (size_t)r.slot[rec] * O * LPE * B;
  const int cl = cluster_of(a, elem);
  const double dt = a.dt[cl];
  const int n = step_new_of(a, cl);
  const double t0 = (double)n * dt, t1 = (double)(n + 1) * dt;
  // the samples of step n: [t0 - eps, t1 - eps), eps = 1e-9 dt (as sampled)
  const double eps = 1e-9 * dt, lo = t0 - eps, hi = t1 - eps;
  long long s0 = (long long)floor(lo / r.dt_sample) - 1;
  if (s0 < 0) s0 = 0;
  while (s0 < r.ns && (double)s0 * r.dt_sample < lo) ++s0;
  if (!(s0 < r.ns && (double)s0 * r.dt_sample < hi)) return;
  double x[O];
#pragma unroll
  for (int d = 0; d < O; ++d) x[d] = 0.0;
  for (; rec >= 0; rec = (chain[rec] >> 1) - 1) {
    double vb[O];
#pragma unroll
    for (int d = 0; d < O; ++d) vb[d] = 0.0;
    for (long long s = s0; s < r.ns && (double)s * r.dt_sample < hi; ++s) {
      const double t = (double)s * r.dt_sample - t0, sb = seis_b[((size_t)rec * r.ns + s) * LPE + q];
      double pw = 1.0, fact = 1.0;
#pragma unroll
      for (int d = 0; d < O; ++d) {
        vb[d] += pw / fact * sb;
        pw *= t;
        fact *= (double)(d + 1);
      }
    }
    const double phi = r.phi[(size_t)rec * B + b];
#pragma unroll
    for (int d = 0; d < O; ++d) x[d] += vb[d] * phi;
  }
#pragma unroll
  for (int d = 0; d < O; ++d) D[((size_t)d * LPE + q) * B + b] = R(x[d]);   // (zeros before: cleared by its reader)
}

}  // namespace

template <class R, int O, int M>
int launch_adjoint(const KPtrs& p, const APtrs& ad, const LevelArgs& a, hipStream_t st) {
  const int groups = (a.end + EPW - 1) / EPW;
  if (groups <= 0) return 0;
  const dim3 block(64 * ADJ_W<O>);
  if (a.kind == KIND_ADJ_FUSED)
    hipLaunchKernelGGL((k_adjoint<R, O, M, KIND_ADJ_FUSED>), dim3(groups), block, 0, st, p, ad, a);
  else if (a.kind == KIND_ADJ_PREDICT)
    hipLaunchKernelGGL((k_adjoint<R, O, M, KIND_ADJ_PREDICT>), dim3(groups), block, 0, st, p, ad, a);
  else
    hipLaunchKernelGGL((k_adjoint<R, O, M, KIND_ADJ_UPDATE>), dim3(groups), block, 0, st, p, ad, a);
  return (int)hipGetLastError();
}

template <class R, int O, int M>
size_t adjoint_scratch_words() {
  return (size_t)ADJ_W<O> * AdjScratch<R, O, M>::WAVE;
}

template <class R, int O, int M>
int launch_receivers_adj(const KPtrs& p, const APtrs& ad, const LevelArgs& a, const RecArgs& r, const int* chain,
                         const double* seis_b, hipStream_t st) {
  if (r.n <= 0) return 0;
  constexpr int threads = (LPE * edg_gen::Ref<O>::B + 63) / 64 * 64;
  hipLaunchKernelGGL((k_receivers_adj<R, O, M>), dim3((unsigned)r.n), dim3(threads), 0, st, p, ad, a, r, chain,
                     seis_b);
  return (int)hipGetLastError();
}

int launch_material_gradient(const double* gacc, const int* FI, const double* mat, int M, long long Kp, double* out,
                             hipStream_t st) {
  if (Kp <= 0) return 0;
  hipLaunchKernelGGL(k_material_gradient, dim3((unsigned)((Kp + 255) / 256)), dim3(256), 0, st, gacc, FI, mat, M, Kp,
                     out);
  return (int)hipGetLastError();
}

#define EDG_ADJ_INST(R, O, M)                                                                    \
  template int launch_adjoint<R, O, M>(const KPtrs&, const APtrs&, const LevelArgs&, hipStream_t); \
  template size_t adjoint_scratch_words<R, O, M>();                                               \
  template int launch_receivers_adj<R, O, M>(const KPtrs&, const APtrs&, const LevelArgs&, const RecArgs&, \
                                             const int*, const double*, hipStream_t);

EDG_FOR_EACH_VARIANT(EDG_ADJ_INST)

}  // namespace edg

// Host evaluation of the face flux and its reverse mode (FP64), for CPU
// checks of the adjoint's flux transpose.  prm = (nx, ny, nz, zpm, zsm, zpp,
// zsp, lam, mu, rho_inv, s); out [15]; qm_b, qp_b [9] and pb [7] are
// overwritten with the adjoint of the outputs u [15].
extern "C" int edg_godunov_host(int32_t bc, const double* qm, const double* qp, const double* prm, const double* u,
                                double* out, double* qm_b, double* qp_b, double* pb) {
  if (!qm || !qp || !prm || !u || !out || !qm_b || !qp_b || !pb || bc < 0 || bc > 2) return -1;
  edg::godunov<double>(qm, qp, prm[0], prm[1], prm[2], prm[3], prm[4], prm[5], prm[6], prm[7], prm[8], prm[9],
                       prm[10], bc, out);
  for (int k = 0; k < 9; ++k) qm_b[k] = qp_b[k] = 0.0;
  for (int k = 0; k < 7; ++k) pb[k] = 0.0;
  edg::godunov_adj<double>(u, qm, qp, prm[0], prm[1], prm[2], prm[3], prm[4], prm[5], prm[6], prm[7], prm[8], prm[9],
                           prm[10], bc, qm_b, qp_b, pb);
  return 0;
}
