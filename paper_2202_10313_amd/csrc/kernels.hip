// HIP kernels (gfx950) of the ADER-DG element update with clustered rate-2
// LTS: time kernel (Cauchy-Kowalevski), volume kernel, surface kernel with the
// Godunov flux, anelastic relaxation, B1/B2/B3 buffer output, point sources,
// receivers.  Sec. III-A (Discrete Formulation; eqs. ader_taylor, ader_derivative_elastic,
// ader_derivative_anelastic, volume, local/neigh surface kernels, update) and
// Sec. V-B (Buffers and Algorithm; eq. lts_buffers and the buffer consumption rules).
//
// Work mapping.  A workgroup of W waves (2 or 4) owns 7 elements; in each wave
// lane = 9*e + q holds part of the modal row q (0..5 stresses
// xx,yy,zz,xy,yz,xz; 6..8 velocities u,v,w) of element e: the modes are split
// between the waves, and the memory variables of a mode belong to one lane of
// the wave that owns it (the anelastic terms act mode by mode, so this spreads
// them evenly over the 9 lanes and keeps each mechanism's trace inside one
// lane).  Reference-matrix products (K_c, F~_i, F^_i) act inside a row, so
// every lane applies the same sparse matrix: they are straight-line FMAs with
// compile-time constants (generated/refmats.h).  Products that mix rows
// (Jacobians, star matrices, flux solvers, anelastic coupling) go through LDS.
// Lane 63 repeats lane 54's work and never writes global memory.
//
// Differences from the paper's own kernel layout (prior art for Xeon):
//  * the star matrices are applied as "inverse Jacobian, then physical
//    Jacobian" (same product, re-associated) from ~20 compact per-element
//    parameters instead of stored 9x9 / 6x9 matrices;
//  * the flux solvers are evaluated on the fly (Godunov state in the face
//    normal frame) instead of stored 9x9 / 6x9 matrices;
//  * every element's local vertices are sorted by global vertex id, so both
//    sides of a face parameterise it identically and the 12 neighbour flux
//    matrices F-_{j,h} collapse to the 4 F~_j: buffers are stored as face
//    traces (B F~_j, 9 x F per face), produced once by their owner;
//  * the local and neighbouring surface contributions of a step are applied
//    together at the end of the step (one Godunov solve and one lift per face)
//    from the element's own B1 trace and the neighbour data;
//  * ping-pong trace slots (by step parity) let one launch per finest level
//    finish the step of every active element and start its next one.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>
#include <type_traits>

#include "generated/refmats.h"
#include "kernels.hpp"
#include "device_common.hpp"

namespace edg {

namespace {

// ---------------------------------------------------------------------------
// The element update: a workgroup of W waves owns 7 elements.  Lane (e, q) of
// wave w keeps row q of element e for the modes [mb(w), mb(w + 1)) only
// (elementwise state is split W ways: no register spill, several workgroups
// per CU); the reference-matrix products that need a whole row read it from
// the LDS row exchange RX, and their outputs are split between the waves
// (stiffness and trace outputs balanced by non-zero count, the wave's own
// modes for the lift).  The gradient exchange holds only the 18 (row,
// direction) pairs that are read: all three directions of the velocities,
// d_i sigma_ij of each stress row.
//
// W (see LEVEL_W): a group's critical path shortens with more waves and the
// registers of a wave shrink, while what every wave repeats (parameters,
// addresses, whole-row reads) grows.
//
// What bounds it (O = 5, m = 3, FP32, 62k tets): latency at three waves per
// SIMD (168 registers; 128 spill: 4,493 us per cycle at 300k against 2,881).
// Of a wave's cycles vector issue takes 22% (66% of the SIMD's), LDS about 56%
// of its unit's, 43% wait on LDS, memory or barriers; 3.1-3.4 TB/s of memory
// traffic.  Fewer instructions alone (3,300 -> 3,053 a wave: one lift per face
// row, the memory recursion as one multiply-add) gain little at O = 5, but at
// O = 4 they brought a fourth wave per SIMD (41k tets 372 -> 341 us).
template <class R, int O, int M>
struct LevelLds {
  // Bank-conflict-free strides: with a row stride RS and an element stride
  // ES = 9 RS (mod 32), lane 9e+q addresses bank RS (9e + q) (mod 32), a
  // bijection for odd RS over the 63 working lanes.
  using RF = edg_gen::Ref<O>;
  static constexpr int B = RF::B, FP = RF::FP;
  static constexpr int up(int v, int m, int r) { return v + ((r - v % m) % m + m) % m; }
  static constexpr int BS = B % 2 ? B : B + 1;                 // row stride of mode rows (odd)
  // Face rows hold the F face modes at the least odd stride: the face area is
  // the larger one below O = 5, and its padding to FP kept a workgroup off the CU
  // (FP64 O = 4 55 -> 47 KB, two -> three; 41k tets m=0 279 -> 242 us per cycle,
  // 3.9k tets O = 3 plane wave check 667 -> 640 us; FP32 O = 4 m=0 303k 706 ->
  // 688).  FP32 O = 4 m=3 has no registers for a fifth (98k 418 -> 420): padded.
  static constexpr bool FPAD = sizeof(R) == 4 && O == 4 && M > 0;
  static constexpr int FS = FPAD ? FP + 1 : RF::F | 1;         // row stride of face rows (odd)
  static constexpr int FW = FPAD ? FP : RF::F;                 // words of a face row
  static constexpr int GRAD = 19 * BS;          // 18 used (row, dir) pairs + 1 dummy row
  static constexpr int COUP = 6 * BS;
  static constexpr int RX = LPE * BS;
  static constexpr int REST = GRAD + COUP + RX;
  static constexpr int REGION = up(REST, 32, (9 * BS) % 32);   // element stride of the mode areas
  static constexpr int FACE = up(4 * 2 * LPE * FS, 32, (9 * FS) % 32);  // element stride of the face area
  // At O = 5 the gradient, coupling and exchange areas are three arrays with
  // element strides of their own: the exchange keeps ES = 9 RS (mod 32) for
  // its row-wise accesses, while the gradient and coupling strides (7 and 24
  // mod 32) were chosen, with the slot table, for the fewest modelled
  // conflicts of their mode-owner and slot accesses (1,112 -> 813 cycles per
  // wave in the model).  At O = 4 that choice modelled worse: one region.
  static constexpr bool SPLIT = O == 5;
  static constexpr int GSTR = SPLIT ? up(GRAD, 32, 7) : REGION;
  static constexpr int CSTR = SPLIT ? up(COUP, 32, 24) : REGION;
  static constexpr int RSTR = SPLIT ? up(RX, 32, (9 * BS) % 32) : REGION;
  static constexpr int GOFF = 0;
  static constexpr int COFF = SPLIT ? EPW * GSTR : GRAD;
  static constexpr int ROFF = SPLIT ? COFF + EPW * CSTR : GRAD + COUP;
  static constexpr int MODES = SPLIT ? ROFF + EPW * RSTR : EPW * REGION;
  static constexpr int TOTAL = MODES > EPW * FACE ? MODES : EPW * FACE;
};

// An opaque copy of a lane index: addresses built from it are recomputed at
// the point of use instead of being kept live (as 64-bit register pairs)
// across the whole kernel.
__device__ __forceinline__ int fresh(int v) {
  asm volatile("" : "+v"(v));
  return v;
}

// slot of (row, direction) in the gradient exchange; 18 = not read (dummy).
// The assignment is the one with the fewest LDS bank conflicts (over the
// stiffness output writes, the strain reads of the memory variables and the
// star-product reads of a time-kernel step) found by a search over slot
// permutations for the strides above (one table per layout of LevelLds).
template <int O>
__device__ __forceinline__ int gslot(int row, int dir) {
  constexpr int T4[9][3] = {{1, 18, 18}, {18, 6, 18}, {18, 18, 13}, {17, 12, 18}, {18, 14, 7},
                            {16, 18, 15}, {0, 2, 5}, {11, 10, 3}, {4, 8, 9}};
  constexpr int T5[9][3] = {{16, 18, 18}, {18, 0, 18}, {18, 18, 10}, {15, 1, 18}, {18, 12, 9},
                            {17, 18, 11}, {7, 4, 2}, {8, 3, 14}, {6, 5, 13}};
  constexpr unsigned long long W0 = pack_rows5(O == 5 ? T5 : T4, 0), W1 = pack_rows5(O == 5 ? T5 : T4, 1),
                               W2 = pack_rows5(O == 5 ? T5 : T4, 2);
  const unsigned long long w = dir == 0 ? W0 : (dir == 1 ? W1 : W2);   // selects, no table in memory
  return (int)((w >> (5 * row)) & 31);
}

// Waves per SIMD the registers are budgeted for: four where the update fits 128
// registers without spills (left to itself the compiler takes up to 144 at
// O = 4 m=3, three waves: 16 runs of 18k tets 2,037 us per cycle against
// 1,879), two at O = 5 m=3 (it takes 168, three waves) and for the two-wave form
// of O >= 4; FP64 O >= 4 one, so that nothing spills (41k tets O = 5 m=0 919 ->
// 884 us, m=3 1,862 -> 1,835).
// (At least that many, up to the eight the hardware has: an upper bound of four,
// as before, is kept by allocating registers that nothing uses.  FP32 m=0, two
// clusters, us per cycle: O = 2 303k tets 247 -> 217, O = 4 762 -> 702.)
template <class R, int O, int M, int W>
constexpr int level_occ() {
  return sizeof(R) == 8 ? (O >= 4 ? 1 : 2) : (O <= 3 || (W == 4 && !(O == 5 && M > 0))) ? 4 : 2;
}

// Point sources: Q[stress] += -M phi(x_s) / |det J| * (S(t1) - S(t0)) for the
// step of the source's element.
__device__ __forceinline__ double stf_antiderivative(int kind, double p0, double p1, double t) {
  if (kind == 0) {  // Ricker moment rate: S = (t - t0) exp(-a (t - t0)^2), a = (pi fc)^2
    const double a = (M_PI * p0) * (M_PI * p0);
    const double tau = t - p1;
    return tau * exp(-a * tau * tau);
  }
  // Hann moment rate on [t0, t0 + T]
  const double tau = t - p0;
  if (tau <= 0.0) return 0.0;
  if (tau >= p1) return 1.0;
  return (tau - p1 / (2.0 * M_PI) * sin(2.0 * M_PI * tau / p1)) / p1;
}

// v of lane i (uniform)
__device__ __forceinline__ double lane_value(double v, int i) {
  const unsigned long long u = __builtin_bit_cast(unsigned long long, v);
  const unsigned lo = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)u, i);
  const unsigned hi = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)(u >> 32), i);
  return __builtin_bit_cast(double, (unsigned long long)hi << 32 | lo);
}

// The points of a level launch (see PointArgs), one wave each, beside the element
// groups.  As a launch of their own between two levels they cost 4.9 us per
// level of nothing but latency (three launches before that: 12); here nothing
// waits for them, since a sample reads the derivatives of the step before and a
// source is evaluated one level ahead.  Measured (us per shot): 5k tets O = 4 m=3
// 1,095 -> 885, five-cluster basin 8k O = 5 1,237 -> 1,105, 62k 4,985 -> 4,870,
// 997k 20,270 -> 20,160; a mesh without points pays 0.4 us a level for the branch
// and the longer argument block (plane wave check 642 -> 666).  The sources of
// one element are summed in packets of a wavefront, a lane each: 1,024 of them in
// one element, O = 4, 20 cycles, cost 6,099 us one after another and 305 so (272
// spread over the mesh).
// vals: LDS of O x 9 doubles per wave.
template <class R, int O, int KIND, int W>
__device__ __forceinline__ void level_points(const KPtrs& p, const LevelArgs& a, const PointArgs& pt, double* vals) {
  constexpr int B = edg_gen::Ref<O>::B, D = O * LPE;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int item = (int)blockIdx.x * W + w, run = a.run0 + (int)blockIdx.y;
  const long long level = *a.clock + a.level;
  const int n_rec = KIND != KIND_PREDICT ? pt.r.n : 0;
  if (item < n_rec) {
    // a receiver: evaluate the Taylor expansion predicted at level - 1 at the
    // sample times in its step, its lanes (d, q) forming the O x 9 derivative
    // values before nine of them sample
    const RecArgs& r = pt.r;
    const int elem = r.elem[item], cl = cluster_of(a, elem);
    if ((level - 1) & ((1ll << cl) - 1)) return;    // no step started there
    const double dt = a.dt[cl];
    const int n = (int)((level - 1) >> cl);
    const double t0 = (double)n * dt, t1 = (double)(n + 1) * dt;
    // step n takes the samples in [t0 - eps, t1 - eps), eps = 1e-9 dt: a sample
    // on (or within rounding of) a step boundary belongs to the step that
    // starts there, whichever way the two sides round the boundary
    const double eps = 1e-9 * dt, lo = t0 - eps, hi = t1 - eps;
    long long s = (long long)floor(lo / r.dt_sample) - 1;
    if (s < 0) s = 0;
    while (s < r.ns && (double)s * r.dt_sample < lo) ++s;
    if (!(s < r.ns && (double)s * r.dt_sample < hi)) return;   // (uniform over the wave)
    double* const v = vals + w * D;
    if (lane < D) {
      const R* x = reinterpret_cast<const R*>(p.recD) + (size_t)run * p.run_recd +
                   ((size_t)(r.slot[item] + (cl == 0 ? n & 1 : 0)) * D + lane) * B;
      const double* phi = r.phi + (size_t)item * B;
      double acc = 0.0;
#pragma unroll 5
      for (int b = 0; b < B; ++b) acc += (double)x[b] * phi[b];
      v[lane] = acc;
    }
    wave_lds_sync();
    double* const out = r.out + ((size_t)run * r.n + item) * r.ns * LPE;
    if (lane < LPE)
      for (; s < r.ns && (double)s * r.dt_sample < hi; ++s) {
        const double x = (double)s * r.dt_sample - t0;
        double acc = 0.0, pw = 1.0, fact = 1.0;
#pragma unroll
        for (int d = 0; d < O; ++d) {
          acc += pw / fact * v[d * LPE + lane];
          pw *= x;
          fact *= (double)(d + 1);
        }
        out[s * LPE + lane] = acc;
      }
  } else if (KIND != KIND_NEIGHBOR && pt.s.n > 0) {
    // a packet of sources of one element, in a step that ends at level + 1: each
    // lane evaluates the moment rate of one, then all of them form the words
    const SrcArgs& s = pt.s;
    const int se = s.run_first[run] + (item - n_rec);
    if (se >= s.run_first[run + 1]) return;
    const int cl = cluster_of(a, s.elem[se]);
    if ((level + 1) & ((1ll << cl) - 1)) return;
    const double dt = a.dt[cl];
    const int n = (int)((level + 1) >> cl) - 1;
    const double t0 = (double)n * dt, t1 = (double)(n + 1) * dt;
    constexpr int NW = (6 * B + 63) / 64;
    double acc[NW];
#pragma unroll
    for (int k = 0; k < NW; ++k) acc[k] = 0.0;
    const int src0 = s.first[se], m = s.first[se + 1] - src0;
    const int mine = src0 + (lane < m ? lane : 0);
    const double f = stf_antiderivative(s.kind[mine], s.par[2 * mine], s.par[2 * mine + 1], t1) -
                     stf_antiderivative(s.kind[mine], s.par[2 * mine], s.par[2 * mine + 1], t0);
    const double idet = s.inv_det[se];
    const double *mo[NW], *ph[NW];
#pragma unroll
    for (int k = 0; k < NW; ++k) {
      const int wd = lane + 64 * k < 6 * B ? lane + 64 * k : 0;
      mo[k] = s.moment + 6 * (size_t)src0 + wd / B;
      ph[k] = s.phi + (size_t)src0 * B + wd % B;
    }
    static_assert(SRC_PACKET == 64, "a lane per source");
#pragma unroll 8
    for (int i = 0; i < m; ++i) {
      const double fi = lane_value(f, i);
#pragma unroll
      for (int k = 0; k < NW; ++k) acc[k] += -mo[k][6 * i] * ph[k][i * B] * idet * fi;
    }
    R* const inc = reinterpret_cast<R*>(s.inc) + ((size_t)((level + 1) & 1) * s.n + se) * (6 * B);
#pragma unroll
    for (int k = 0; k < NW; ++k)
      if (lane + 64 * k < 6 * B) inc[lane + 64 * k] = R(acc[k]);
  }
}

// KIND is the launch kind (KIND_PREDICT, KIND_FUSED, KIND_NEIGHBOR) as a
// template parameter: one code path per kernel keeps the register allocation
// of the fused path free of the neighbour-only exit.  TM: the traces of faces
// 0 and 1 (the two densest) as one dense product on the matrix cores.
typedef float floatx16 __attribute__((ext_vector_type(16)));
template <class R, int O, int M, int KIND, int W, bool TM = false>
__global__ __launch_bounds__(64 * W) __attribute__((amdgpu_waves_per_eu(level_occ<R, O, M, W>(), 8)))
void k_level(LevelArgs a, KPtrs p, PointArgs pt) {
  using RF = edg_gen::Ref<O>;
  using L = LevelLds<R, O, M>;
  constexpr int B = RF::B, F = RF::F, FP = RF::FP;
  constexpr int MM = M > 0 ? M : 1;
  constexpr int NBX = RF::template nbx<W>;
  constexpr int NFW = 4 / W;                     // faces gathered per wave
  constexpr int NTC = RF::template ntc<W>, NCH = FP / 4;   // trace chunks per wave and per face
  constexpr int JW = (NBX + LPE - 1) / LPE;      // owned memory modes per lane
  constexpr int JB = (B + LPE - 1) / LPE;        // memory-variable layout
  __shared__ __align__(16) R lds[L::TOTAL];
  // per element and face: normal, area ratio, neighbour impedances (the face
  // words of the parameter table; a boundary face holds the element's own),
  // the inverse sums of both sides' impedances and the boundary kind, staged
  // for the Godunov items of the surface phase
  __shared__ R fdat[KIND != KIND_PREDICT ? EPW * 4 * 8 : 1];
  __shared__ int fbc[KIND != KIND_PREDICT ? EPW * 4 : 1];
  // per element: flags and own B3 slot, for the matrix-core trace's exports
  __shared__ int tme[TM ? EPW * 2 : 1];

  if ((int)blockIdx.x < a.points) {
    static_assert(W * O * LPE * sizeof(double) <= L::TOTAL * sizeof(R) && O * LPE <= 64, "a wave per point");
    level_points<R, O, KIND, W>(p, a, pt, reinterpret_cast<double*>(lds));
    return;
  }

  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);   // wave (uniform)
  const int lane = threadIdx.x & 63;
  const int e = lane / LPE, r = lane % LPE;
  const int ec = e < EPW ? e : EPW - 1;
  const int q = e < EPW ? r : 0;
  int g, run;
  group_and_run(a, g, run);
  select_run<R>(p, run);
  // the group's source packets (asked for here: their number is needed in mid-kernel)
  int src0 = 0, src1 = 0;
  if constexpr (KIND != KIND_PREDICT) {
    const int* const s = pt.s.group + (size_t)run * pt.s.row + (size_t)g * pt.s.col;
    src0 = s[0];
    src1 = s[1];
  }
  const int elem = g * EPW + ec;
  const int cl = cluster_of(a, g * EPW);        // one cluster per workgroup (uniform)
  const bool valid = (e < EPW) && (elem < a.cl_vend[cl]);
  const int slot = ec * LPE + q;
  const int base = RF::mb(W, w);
  const int nb = RF::mb(W, w + 1) - base;
  // the wave has its mode lb / the lane owns memory mode lb = q + 9 jw:
  // uniform (and decided here) but for the modes only some waves have
  auto has = [&](int lb) { return lb < RF::template nbn<W> || lb < nb; };
  auto owns = [&](int jw, int lb) { return LPE * jw + LPE <= RF::template nbn<W> || lb < nb; };
  // slot of owned mode b = base + q + 9 jw in the memory-variable layout:
  // lane b mod 9 of the element (the lane itself where waves start at
  // multiples of nine modes)
  const int mslot = RF::template nines<W> ? slot : ec * LPE + (base + q) % LPE;
  constexpr int BS = L::BS, FS = L::FS;
  R* const fac = lds + ec * L::FACE;          // face area (surface phase only)
  R* const grad = lds + L::GOFF + ec * L::GSTR;
  R* const coup = lds + L::COFF + ec * L::CSTR;
  R* const rx = lds + L::ROFF + ec * L::RSTR;

  // Global addresses are a per-workgroup (uniform, scalar) base plus a 32-bit
  // lane offset, so no 64-bit per-lane address has to stay live.
  constexpr int TS = 4 * LPE * FP;                // trace floats per element
  const size_t Kp = (size_t)p.Kp;
  const size_t tstride = (size_t)TS;
  R* const Qg = reinterpret_cast<R*>(p.Qe) + (size_t)g * B * NSLOT;
  R* const Qag = reinterpret_cast<R*>(p.Qa) + (size_t)g * JB * MM * 6 * NSLOT;
  const R* P = reinterpret_cast<const R*>(p.P) + (size_t)g * EPW * NPARAM + ec * NPARAM;
  const int* FI = p.FI + (size_t)g * EPW * FI_WORDS + ec * FI_WORDS;
  const size_t tg = (size_t)g * EPW * TS;        // this workgroup's first trace

  // The face records of the wave's two faces (and the face word codes to be
  // staged) are the first loads of the kernel: the neighbour gathers depend
  // on them, and loads complete in issue order.
  int fnb[NFW], fcd[NFW], fax[NFW];
  int fcode = 0;
  const bool stage = KIND != KIND_PREDICT && w == 0 && q < 4 && e < EPW;
  if constexpr (KIND != KIND_PREDICT) {
#pragma unroll
    for (int ii = 0; ii < NFW; ++ii) {
      fnb[ii] = FI[3 * (NFW * w + ii)];
      fcd[ii] = FI[3 * (NFW * w + ii) + 1];
      fax[ii] = FI[3 * (NFW * w + ii) + 2];
    }
    if (stage) fcode = FI[3 * q + 1];
  }

  const bool is_stress = q < 6;
  int qi = 0, qj = 0;
  if (q < 3) { qi = q; qj = q; }
  else if (q == 3) { qi = 0; qj = 1; }
  else if (q == 4) { qi = 1; qj = 2; }
  else if (q == 5) { qi = 0; qj = 2; }
  const R delta = q < 3 ? R(1) : R(0);

  R G[9];
#pragma unroll
  for (int c = 0; c < 9; ++c) G[c] = P[c];
  const R rho_inv = P[9], lam = P[10], mu = P[11], zp = P[12], zs = P[13];
  R al[MM], bl[MM], om[MM];
#pragma unroll
  for (int l = 0; l < MM; ++l) {
    al[l] = M > 0 ? P[14 + 2 * l] : R(0);
    bl[l] = M > 0 ? P[15 + 2 * l] : R(0);
    om[l] = M > 0 ? R(a.omega[l]) : R(0);
  }

  // LDS offsets (elements of `grad`) this lane writes and reads
  R* const gw0 = grad + gslot<O>(q, 0) * BS;
  R* const gw1 = grad + gslot<O>(q, 1) * BS;
  R* const gw2 = grad + gslot<O>(q, 2) * BS;
  // Star products without divergence: every lane forms
  //   wabc (g[sa] + g[sb] + g[sc]) + wde (g[sd] + g[se]) + wc coupling
  // stress row ij: lambda delta_ij div v + mu (d_j v_i + d_i v_j) + coupling,
  // velocity row i: (1/rho) sum_d d_d sigma_id (the last two reads unused).
  int sa, sb, sc, sd, se;
  R wabc, wde, wc;
  if (is_stress) {
    sa = gslot<O>(6, 0) * BS; sb = gslot<O>(7, 1) * BS; sc = gslot<O>(8, 2) * BS;
    sd = gslot<O>(6 + qi, qj) * BS; se = gslot<O>(6 + qj, qi) * BS;
    wabc = lam * delta; wde = mu; wc = R(1);
  } else {
    const int i = q - 6;
    sa = gslot<O>(sym_index(i, 0), 0) * BS; sb = gslot<O>(sym_index(i, 1), 1) * BS; sc = gslot<O>(sym_index(i, 2), 2) * BS;
    sd = sa; se = sb;
    wabc = rho_inv; wde = R(0); wc = R(0);
  }
  const int cs = (is_stress ? q : 0) * BS;     // coupling row read by this lane

  // The element state (elastic rows and the memory variables of the owned
  // modes) is loaded so that its latency overlaps the surface phase: after
  // the face-trace gathers are issued when there is one (they head the
  // critical path: face words, then the traces they point to), else here.
  R qe[NBX];
  R qa[JW][MM][6];
  auto load_state = [&]() {
#pragma unroll
    for (int lb = 0; lb < NBX; ++lb)
      qe[lb] = has(lb) ? Qg[(base + lb) * NSLOT + slot] : R(0);
#pragma unroll
    for (int jw = 0; jw < JW; ++jw) {
      const int lb = q + LPE * jw, b = base + lb;
      const int jb = b / LPE;
#pragma unroll
      for (int l = 0; l < MM; ++l)
#pragma unroll
        for (int c = 0; c < 6; ++c)
          qa[jw][l][c] = (M > 0 && owns(jw, lb)) ? Qag[((jb * MM + l) * 6 + c) * NSLOT + mslot] : R(0);
    }
  };
  if constexpr (KIND == KIND_PREDICT) load_state();

  // ------------------------------------------------ surface: finish step n
  bool coup_pending = false;
  if constexpr (KIND != KIND_PREDICT) {
    const int n = step_fin_of(a, cl);
    const R* T1 = reinterpret_cast<const R*>(p.T1);
    const R* T2 = reinterpret_cast<const R*>(p.T2);
    const R* T3 = reinterpret_cast<const R*>(p.T3);
    // the face words go to LDS after the gathers are issued (a store of a
    // loaded value waits for it)
    R fw[6] = {R(0), R(0), R(0), R(0), R(0), R(0)};
    if (stage)
#pragma unroll
      for (int k = 0; k < 6; ++k) fw[k] = P[20 + 6 * q + k];
    // Neighbour data of the wave's two faces.  Each lane selects its sources
    // by arithmetic (same cluster: the neighbour's B1; finer: its B3;
    // coarser: its B2 in the first half step, B1 - B2 in the second; none:
    // zeros) and every load of both faces is issued before any is used, so
    // the memory latency is paid once rather than once per source kind.
    R vown[NFW][FP], v1[NFW][FP], v2[NFW][FP];
    bool none[NFW];
#pragma unroll
    for (int ii = 0; ii < NFW; ++ii) {
      const int i = NFW * w + ii;
      const int nbr = fnb[ii];
      const int code = fcd[ii];
      const size_t aux = (size_t)fax[ii];
      const int j = code & 15, rel = ((code >> 8) & 15) - 1;
      const R* own = T1 + (size_t)(n & 1) * Kp * tstride + tg + (ec * TS + (i * LPE + q) * FP);
      const size_t fo = (size_t)(j * LPE + q) * FP;
      const int c = (n >> 1) & 1;
      const R* b1 = T1 + (size_t)(rel == 0 ? (n & 1) : c) * Kp * tstride + (size_t)nbr * tstride + fo;
      const R* b2 = T2 + ((size_t)c * p.N2 + aux) * tstride + fo;
      const R* b3 = T3 + ((size_t)(n & 1) * p.N3 + aux) * tstride + fo;
      const bool odd = (n & 1) != 0;
      const R* s1 = nbr < 0 ? own : (rel == 0 ? b1 : (rel < 0 ? b3 : (odd ? b1 : b2)));
      const bool sub = nbr >= 0 && rel > 0 && odd;
      none[ii] = nbr < 0;
      // (v2 is zeroed before its masked load: no write to a register with a
      // load in flight)
#pragma unroll
      for (int f = 0; f < FP; ++f) v2[ii][f] = R(0);
#pragma unroll
      for (int f = 0; f < FP; ++f) vown[ii][f] = own[f];
#pragma unroll
      for (int f = 0; f < FP; ++f) v1[ii][f] = s1[f];
      if (sub)
#pragma unroll
        for (int f = 0; f < FP; ++f) v2[ii][f] = b2[f];
    }
    if (stage) {
      R* d = fdat + (ec * 4 + q) * 8;
#pragma unroll
      for (int k = 0; k < 6; ++k) d[k] = fw[k];
      d[6] = R(1) / (zp + fw[4]);
      d[7] = R(1) / (zs + fw[5]);
      fbc[ec * 4 + q] = fcode;
    }
#pragma unroll
    for (int ii = 0; ii < NFW; ++ii) {
      const int i = NFW * w + ii;
      R* dmn = fac + ((i * 2 + 0) * LPE + q) * FS;
      R* dpl = fac + ((i * 2 + 1) * LPE + q) * FS;
#pragma unroll
      for (int f = 0; f < L::FW; ++f) {
        dmn[f] = vown[ii][f];
        dpl[f] = none[ii] ? R(0) : v1[ii][f] - v2[ii][f];
      }
    }
    // keep the state loads below behind these stores (the scheduler would
    // otherwise interleave them and wait for all loads before the barrier)
    __builtin_amdgcn_sched_barrier(0);
    load_state();
    __syncthreads();
#pragma unroll 2
    for (int rr = 0; rr < (4 * F + W * LPE - 1) / (W * LPE); ++rr) {
      const int t = q + LPE * (w + W * rr);
      if (t < 4 * F) {
        const int i = t / F, f = t % F;
        const int bc = (fbc[ec * 4 + i] >> 4) & 15;
        const R* fp = fdat + (ec * 4 + i) * 8;
        R qm[9], qp[9], v[4], tr[3], out[9];
#pragma unroll
        for (int k = 0; k < 9; ++k) {
          qm[k] = fac[((i * 2 + 0) * LPE + k) * FS + f];
          qp[k] = fac[((i * 2 + 1) * LPE + k) * FS + f];
        }
        godunov_state<R>(qm, qp, fp[0], fp[1], fp[2], zp, zs, fp[4], fp[5], fp[6], fp[7], bc, v, tr);
        if (M > 0) flux_strain<R>(v, fp[0], fp[1], fp[2], fp[3], out);
        else flux_stress<R>(v, fp[0], fp[1], fp[2], lam, mu, fp[3], out);
        flux_velocity<R>(tr, rho_inv, fp[3], out + 6);
#pragma unroll
        for (int k = 0; k < 9; ++k) fac[((i * 2 + 0) * LPE + k) * FS + f] = out[k];
      }
    }
    __syncthreads();
    R da[NBX];
    {
      R pf[4 * FP];
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int f = 0; f < FP; ++f) pf[i * FP + f] = f < L::FW ? fac[((i * 2 + 0) * LPE + q) * FS + f] : R(0);
      RF::template lift_w<W>(w, pf, da);
    }
    // the group's source packets, if any (uniform)
    for (int src = src0; src < src1; ++src) {
      const SrcArgs& s = pt.s;
      const R* const inc = reinterpret_cast<const R*>(s.inc) +
                           ((size_t)((*a.clock + a.level) & 1) * s.n + src) * (6 * B) + q * B + base;
      if (is_stress && s.elem[src] == elem)   // (lane 63 as lane 54: both write the exchange)
#pragma unroll
        for (int lb = 0; lb < NBX; ++lb)
          if (has(lb)) qe[lb] += inc[lb];
    }
    if (M > 0) {
      // the stress lanes hold the lifted strain-rate rows: the memory
      // variables of a mode take them (times omega) in the lane that owns the
      // mode, the stresses are lam tr I + 2 mu times them
      __syncthreads();
      if (is_stress && e < EPW)
#pragma unroll
        for (int lb = 0; lb < NBX; ++lb)
          if (has(lb)) coup[q * BS + base + lb] = da[lb];
      coup_pending = true;
      // coupling rows are read by their own wave (its modes)
      wave_lds_sync();
      const R w1 = is_stress ? R(2) * mu : R(1), w3 = is_stress ? wabc : R(0);
#pragma unroll
      for (int lb = 0; lb < NBX; ++lb) {
        const int b = base + lb;
        if (has(lb)) qe[lb] += w1 * da[lb] + w3 * (coup[b] + coup[BS + b] + coup[2 * BS + b]);
      }
    } else {
#pragma unroll
      for (int lb = 0; lb < NBX; ++lb) qe[lb] += da[lb];
      __syncthreads();
    }
  }

  if (M > 0 && coup_pending) {
#pragma unroll
    for (int jw = 0; jw < JW; ++jw) {
      const int lb = q + LPE * jw, b = base + lb;
      if (owns(jw, lb))
#pragma unroll
        for (int l = 0; l < MM; ++l)
#pragma unroll
          for (int c = 0; c < 6; ++c) qa[jw][l][c] += om[l] * coup[c * BS + b];
    }
  }
  // (the next LDS stores follow the workgroup barrier that forms need_b2)

  if constexpr (KIND == KIND_NEIGHBOR) {
    if (valid) {
#pragma unroll
      for (int lb = 0; lb < NBX; ++lb)
        if (has(lb)) Qg[(base + lb) * NSLOT + slot] = qe[lb];
      if (M > 0)
#pragma unroll
        for (int jw = 0; jw < JW; ++jw) {
          const int lb = q + LPE * jw, b = base + lb, jb = b / LPE;
          if (owns(jw, lb))
#pragma unroll
            for (int l = 0; l < MM; ++l)
#pragma unroll
              for (int c = 0; c < 6; ++c) Qag[((jb * MM + l) * 6 + c) * NSLOT + mslot] = qa[jw][l][c];
        }
    }
    return;
  }

  // the start-of-step state, recorded for the reverse sweep when asked
  // (every element slot of the group; padding slots get the zeros their state holds)
  if (a.rec_e != nullptr && e < EPW) {
    R* const Re = reinterpret_cast<R*>(a.rec_e) + (size_t)g * B * NSLOT;
#pragma unroll
    for (int lb = 0; lb < NBX; ++lb)
      if (has(lb)) Re[(base + lb) * NSLOT + slot] = valid ? qe[lb] : R(0);
    if (M > 0) {
      R* const Ra = reinterpret_cast<R*>(a.rec_a) + (size_t)g * JB * MM * 6 * NSLOT;
#pragma unroll
      for (int jw = 0; jw < JW; ++jw) {
        const int lb = q + LPE * jw, b = base + lb, jb = b / LPE;
        if (owns(jw, lb))
#pragma unroll
          for (int l = 0; l < MM; ++l)
#pragma unroll
            for (int c = 0; c < 6; ++c) Ra[((jb * MM + l) * 6 + c) * NSLOT + mslot] = valid ? qa[jw][l][c] : R(0);
      }
    }
  }

  // ------------------------------------------------ time kernel: predict step nn
  // The current derivative d^d Q lives only in the row exchange RX: each lane
  // adds its own modes of a new derivative to the time integrals when it forms
  // them and writes them there, so no register copy of it is kept across the
  // loop.
  const int nn = step_new_of(a, cl);
  const int eflags = FI[12];
  if constexpr (TM) {
    if (w == 0 && q == 0 && e < EPW) {
      tme[ec * 2] = eflags;
      tme[ec * 2 + 1] = FI[14];
    }
  }
  const bool need_b2 = __syncthreads_or((eflags & EF_HAS_FINER) != 0);
  const int rec_slot = FI[15];
  R te[NBX], t2[NBX];
  R dm[JW][MM][6];
  {
    const R c_0 = R(a.tc[cl][0]), h_0 = R(a.th[cl][0]);
#pragma unroll
    for (int lb = 0; lb < NBX; ++lb) {
      te[lb] = c_0 * qe[lb];
      t2[lb] = h_0 * qe[lb];
      if (has(lb)) rx[q * BS + base + lb] = qe[lb];
    }
  }
  R* const rd = reinterpret_cast<R*>(p.recD) +
                ((size_t)(rec_slot >= 0 ? rec_slot + (cl == 0 ? nn & 1 : 0) : 0) * O * LPE + q) * B + base;
  if (rec_slot >= 0 && valid)
#pragma unroll
    for (int lb = 0; lb < NBX; ++lb)
      if (has(lb)) rd[lb] = qe[lb];
#pragma unroll
  for (int jw = 0; jw < JW; ++jw)
#pragma unroll
    for (int l = 0; l < MM; ++l)
#pragma unroll
      for (int c = 0; c < 6; ++c) dm[jw][l][c] = qa[jw][l][c];

  // dm holds theta^l at d = 0 and z = (d^d theta^l) / omega_l after it, so that
  // its recursion, d^{d+1} theta = omega (d^d eps - d^d theta), is one
  // multiply-add z' = eps - omega z (the first step eps - theta); the weights
  // of the coupling carry the omega from then on
#pragma unroll 1
  for (int d = 0; d < O; ++d) {
    const R c_d = R(a.tc[cl][d]);
    const bool more = d + 1 < O;
    if (more) {
      __syncthreads();
      {
        R full[B];
#pragma unroll
        for (int b = 0; b < B; ++b) full[b] = rx[q * BS + b];
        RF::template ck_grad_w<W>(w, full, G, gw0, gw1, gw2);
      }
      __syncthreads();
    }
    if (M > 0) {
#pragma unroll
      for (int jw = 0; jw < JW; ++jw) {
        const int lb = q + LPE * jw, b = base + lb;
        if (owns(jw, lb)) {
          R eps[6];
          if (more) {
            eps[0] = grad[gslot<O>(6, 0) * BS + b];
            eps[1] = grad[gslot<O>(7, 1) * BS + b];
            eps[2] = grad[gslot<O>(8, 2) * BS + b];
            eps[3] = R(0.5) * (grad[gslot<O>(6, 1) * BS + b] + grad[gslot<O>(7, 0) * BS + b]);
            eps[4] = R(0.5) * (grad[gslot<O>(7, 2) * BS + b] + grad[gslot<O>(8, 1) * BS + b]);
            eps[5] = R(0.5) * (grad[gslot<O>(6, 2) * BS + b] + grad[gslot<O>(8, 0) * BS + b]);
          }
          R cp[6] = {R(0), R(0), R(0), R(0), R(0), R(0)};
#pragma unroll
          for (int l = 0; l < MM; ++l) {
            const R wz = d == 0 ? R(1) : om[l], wq = om[l] * c_d * wz;
            const R tr = dm[jw][l][0] + dm[jw][l][1] + dm[jw][l][2];
#pragma unroll
            for (int c = 0; c < 6; ++c) cp[c] -= bl[l] * dm[jw][l][c] + (c < 3 ? al[l] * tr : R(0));
#pragma unroll
            for (int c = 0; c < 6; ++c) {
              qa[jw][l][c] -= wq * dm[jw][l][c];
              if (more) dm[jw][l][c] = eps[c] - wz * dm[jw][l][c];
            }
          }
          if (e < EPW)
#pragma unroll
            for (int c = 0; c < 6; ++c) coup[c * BS + b] = cp[c];
        }
      }
      if (d == 0)
#pragma unroll
        for (int l = 0; l < MM; ++l) {
          al[l] *= om[l];
          bl[l] *= om[l];
        }
      // the coupling rows of a mode are read by the stress rows of the same
      // wave (the wave that owns the mode)
      wave_lds_sync();
    }
    // reads of three modes, then their stores of the next derivative (a store
    // into the row exchange between reads would, for the compiler, possibly
    // alias the next mode's reads and put an LDS wait behind every mode)
    const R c_n = more ? R(a.tc[cl][d + 1]) : R(0), h_n = more ? R(a.th[cl][d + 1]) : R(0);
    const R wcd = wc * c_d;
    constexpr int CH = 3;
#pragma unroll
    for (int l0 = 0; l0 < NBX; l0 += CH) {
      R nx[CH];
#pragma unroll
      for (int k = 0; k < CH; ++k) {
        const int lb = l0 + k, b = base + lb;
        nx[k] = R(0);
        if (lb < NBX && has(lb)) {
          const R cq = M > 0 ? coup[cs + b] : R(0);
          if (M > 0) qe[lb] += wcd * cq;
          if (more) {
            nx[k] = wabc * (grad[sa + b] + grad[sb + b] + grad[sc + b]) + wde * (grad[sd + b] + grad[se + b]);
            if (M > 0) nx[k] += wc * cq;
          }
        }
      }
      if (more)
#pragma unroll
        for (int k = 0; k < CH; ++k) {
          const int lb = l0 + k;
          if (lb < NBX && has(lb)) {
            rx[q * BS + base + lb] = nx[k];
            te[lb] += c_n * nx[k];
            t2[lb] += h_n * nx[k];
          }
        }
    }
    if (more && rec_slot >= 0 && valid)
#pragma unroll
      for (int lb = 0; lb < NBX; ++lb)
        if (has(lb)) rd[(size_t)(d + 1) * LPE * B + lb] = rx[q * BS + base + lb];
  }
  // (the barrier after the last products orders every read of RX before the
  // time integral is written there)

  // ------------------------------------------------ traces and volume
  // word offset of this wave's trace chunk ii in an element's trace (-1: none)
  auto chunk_off = [&](int ii) {
    const int c = RF::template tchunk<W>(w, ii);
    return ii >= RF::template ntn<W> && c < 0 ? -1 : (c / NCH) * LPE * FP + 4 * (c % NCH);
  };
  // (the matrix-core trace's coefficients are requested before the barrier,
  // so their latency overlaps it)
  float ftb[TM ? RF::MK : 1];
  if constexpr (TM)
#pragma unroll
    for (int st = 0; st < RF::MK; ++st) ftb[st] = RF::FT01[st * 64 + lane];
#pragma unroll
  for (int lb = 0; lb < NBX; ++lb)
    if (has(lb)) rx[q * BS + base + lb] = te[lb];
  __syncthreads();
  {
    R full[B];
#pragma unroll
    for (int b = 0; b < B; ++b) full[b] = rx[q * BS + b];
    if constexpr (!TM) {
    R pt[4 * NTC];
    RF::template trace_w<W>(w, full, pt);
    const int own = fresh(ec * TS + q * FP);
    if (valid) {
      R* T1 = reinterpret_cast<R*>(p.T1) + (size_t)(nn & 1) * Kp * tstride + tg;
#pragma unroll
      for (int ii = 0; ii < NTC; ++ii)
        if (const int o = chunk_off(ii); ii < RF::template ntn<W> || o >= 0)
#pragma unroll
          for (int k = 0; k < 4; ++k) T1[own + o + k] = pt[4 * ii + k];
    }
    if ((eflags & EF_HAS_COARSER) && valid) {
      R* T3 = reinterpret_cast<R*>(p.T3) + ((size_t)((nn >> 1) & 1) * p.N3 + (size_t)FI[14]) * tstride;
      if ((nn & 1) == 0) {
#pragma unroll
        for (int ii = 0; ii < NTC; ++ii)
          if (const int o = chunk_off(ii); ii < RF::template ntn<W> || o >= 0)
#pragma unroll
            for (int k = 0; k < 4; ++k) T3[q * FP + o + k] = pt[4 * ii + k];
      } else {
#pragma unroll
        for (int ii = 0; ii < NTC; ++ii)
          if (const int o = chunk_off(ii); ii < RF::template ntn<W> || o >= 0)
#pragma unroll
            for (int k = 0; k < 4; ++k) T3[q * FP + o + k] += pt[4 * ii + k];
      }
    }
    } else {
      // faces 0 and 1 on the matrix cores: wave w multiplies the group's rows
      // [32 w, 32 w + 32) (row 9 e + q of the exchange; row 63 is padding) by
      // the two faces' trace coefficients, 32 columns (face, face mode), two
      // modes per step; its sparse face (3, or 2) stays on the vector ALUs
      static_assert(W == 2 && sizeof(R) == 4 && FP <= 16, "matrix-core trace: FP32, at most 16 face modes");
      floatx16 acc;
#pragma unroll
      for (int j = 0; j < 16; ++j) acc[j] = 0.f;
      const int kh = lane >> 5;
      const int ar = 32 * w + (lane & 31), ae = ar / LPE, aq = ar - LPE * ae;
      const R* const arow = lds + L::ROFF + (ae < EPW ? ae : EPW - 1) * L::RSTR + aq * BS;
#pragma unroll
      for (int st = 0; st < RF::MK; ++st) {
        const int k = 2 * st + kh;
        const float av = (ar < EPW * LPE && k < B) ? arow[k] : 0.f;
        acc = __builtin_amdgcn_mfma_f32_32x32x2f32(av, ftb[st], acc, 0, 0, 0);
      }
      R pt[FP];
      if (w == 0) RF::trace_f3(full, pt); else RF::trace_f2(full, pt);
      const int fs = w == 0 ? 3 : 2;
      R* const T1 = reinterpret_cast<R*>(p.T1) + (size_t)(nn & 1) * Kp * tstride + tg;
      const int own = fresh(ec * TS + q * FP);
      if (valid)
#pragma unroll
        for (int f = 0; f < FP; ++f) T1[own + fs * LPE * FP + f] = pt[f];
      if ((eflags & EF_HAS_COARSER) && valid) {
        R* T3 = reinterpret_cast<R*>(p.T3) + ((size_t)((nn >> 1) & 1) * p.N3 + (size_t)FI[14]) * tstride;
        if ((nn & 1) == 0) {
#pragma unroll
          for (int f = 0; f < FP; ++f) T3[q * FP + fs * LPE * FP + f] = pt[f];
        } else {
#pragma unroll
          for (int f = 0; f < FP; ++f) T3[q * FP + fs * LPE * FP + f] += pt[f];
        }
      }
      // accumulator register j holds row 32 w + 8 (j / 4) + 4 (lane / 32) +
      // j % 4, column lane % 32 = 16 face + face mode
      const int col = lane & 31, fc = col >> 4, ff = col & 15;
      if (ff < FP)
#pragma unroll
        for (int j = 0; j < 16; ++j) {
          const int m = 32 * w + 8 * (j >> 2) + 4 * kh + (j & 3);
          const int e2 = m / LPE, q2 = m - LPE * e2;
          if (m < EPW * LPE && g * EPW + e2 < a.cl_vend[cl]) {
            T1[e2 * TS + (fc * LPE + q2) * FP + ff] = acc[j];
            if (tme[e2 * 2] & EF_HAS_COARSER) {
              R* T3 = reinterpret_cast<R*>(p.T3) + ((size_t)((nn >> 1) & 1) * p.N3 + (size_t)tme[e2 * 2 + 1]) * tstride;
              if ((nn & 1) == 0) T3[(fc * LPE + q2) * FP + ff] = acc[j];
              else T3[(fc * LPE + q2) * FP + ff] += acc[j];
            }
          }
        }
    }
    RF::template vol_grad_w<W>(w, full, G, gw0, gw1, gw2);
  }
  __syncthreads();
  if (M > 0) {
#pragma unroll
    for (int jw = 0; jw < JW; ++jw) {
      const int lb = q + LPE * jw, b = base + lb;
      if (owns(jw, lb)) {
        R eps[6];
        eps[0] = grad[gslot<O>(6, 0) * BS + b];
        eps[1] = grad[gslot<O>(7, 1) * BS + b];
        eps[2] = grad[gslot<O>(8, 2) * BS + b];
        eps[3] = R(0.5) * (grad[gslot<O>(6, 1) * BS + b] + grad[gslot<O>(7, 0) * BS + b]);
        eps[4] = R(0.5) * (grad[gslot<O>(7, 2) * BS + b] + grad[gslot<O>(8, 1) * BS + b]);
        eps[5] = R(0.5) * (grad[gslot<O>(6, 2) * BS + b] + grad[gslot<O>(8, 0) * BS + b]);
#pragma unroll
        for (int l = 0; l < MM; ++l)
#pragma unroll
          for (int c = 0; c < 6; ++c) qa[jw][l][c] -= om[l] * eps[c];
      }
    }
  }
#pragma unroll
  for (int lb = 0; lb < NBX; ++lb) {
    const int b = base + lb;
    if (has(lb))
      qe[lb] -= wabc * (grad[sa + b] + grad[sb + b] + grad[sc + b]) + wde * (grad[sd + b] + grad[se + b]);
  }
  if (need_b2) {   // B2 traces from the half-step integral (RX is free again)
#pragma unroll
    for (int lb = 0; lb < NBX; ++lb)
      if (has(lb)) rx[q * BS + base + lb] = t2[lb];
    __syncthreads();
    R full[B];
#pragma unroll
    for (int b = 0; b < B; ++b) full[b] = rx[q * BS + b];
    R pt[4 * NTC];
    RF::template trace_w<W>(w, full, pt);
    if (valid && (eflags & EF_HAS_FINER)) {
      R* T2 = reinterpret_cast<R*>(p.T2) + ((size_t)(nn & 1) * p.N2 + (size_t)FI[13]) * tstride;
      const int own = fresh(q * FP);
#pragma unroll
      for (int ii = 0; ii < NTC; ++ii)
        if (const int o = chunk_off(ii); ii < RF::template ntn<W> || o >= 0)
#pragma unroll
          for (int k = 0; k < 4; ++k) T2[own + o + k] = pt[4 * ii + k];
    }
  }

  if (KIND == KIND_FUSED && a.next != nullptr && g == 0 && run == a.run0 && threadIdx.x == 0)
    *a.next = *a.clock + a.tick;
  if (valid) {
    const int sl = fresh(slot);
    const int msl = RF::template nines<W> ? sl : fresh(mslot);
#pragma unroll
    for (int lb = 0; lb < NBX; ++lb)
      if (has(lb)) Qg[(base + lb) * NSLOT + sl] = qe[lb];
    if (M > 0)
#pragma unroll
      for (int jw = 0; jw < JW; ++jw) {
        const int lb = q + LPE * jw, b = base + lb, jb = b / LPE;
        if (owns(jw, lb))
#pragma unroll
          for (int l = 0; l < MM; ++l)
#pragma unroll
            for (int c = 0; c < 6; ++c) Qag[((jb * MM + l) * 6 + c) * NSLOT + msl] = qa[jw][l][c];
      }
  }
}

}  // namespace

__global__ void k_clock(long long* clock, long long set) {
  if (blockIdx.x == 0 && threadIdx.x == 0) *clock = set;
}

int launch_clock(long long* clock, long long set, hipStream_t st) {
  hipLaunchKernelGGL(k_clock, dim3(1), dim3(64), 0, st, clock, set);
  return (int)hipGetLastError();
}

__global__ __launch_bounds__(256) void k_scatter_pairs(int* p, const long long* at, const int* what, long long n) {
  const long long i = (long long)blockIdx.x * 256 + threadIdx.x;
  if (i >= n) return;
  p[2 * at[i]] = what[2 * i];
  p[2 * at[i] + 1] = what[2 * i + 1];
}

int launch_scatter_pairs(int* p, const long long* at, const int* what, long long n, hipStream_t st) {
  if (n <= 0) return 0;
  hipLaunchKernelGGL(k_scatter_pairs, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, p, at, what, n);
  return (int)hipGetLastError();
}

__global__ void k_zero_words(uint32_t* p, size_t words) {
  const size_t stride = (size_t)gridDim.x * blockDim.x;
  for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < words; i += stride) p[i] = 0u;
}

int launch_zero_words(void* p, size_t words, hipStream_t st) {
  if (words == 0) return 0;
  const size_t blocks = std::min<size_t>((words + 255) / 256, 4096);
  hipLaunchKernelGGL(k_zero_words, dim3((unsigned)blocks), dim3(256), 0, st, (uint32_t*)p, words);
  return (int)hipGetLastError();
}

// Waves per workgroup, measured in us per LTS cycle of three clusters (one
// wave was the form before, two at FP32 O >= 4):
//   O >= 4  four: FP32 O=5 m=3 2k / 41k / 300k tets 112 / 541 / 2,881 against
//           144 / 613 / 3,038 with two, m=0 300k 1,931 against 2,216; O=4 m=3
//           84 / 341 / 1,810 against 100 / 404 / 1,966, 16 runs of 18k 1,879
//           against 2,037.  FP64 O=4 m=3 41k 720 against 1,078 (one wave:
//           2,315).  FP64 O=5 m=0 1k / 11k / 101k 100 / 285 / 1,771 against 137 /
//           393 / 2,391; m=3 1k / 5k / 11k 126 / 225 / 525 against 189 / 270 /
//           565, but 41k / 101k 1,631 / 3,955 against 1,488 / 3,476: with two
//           rounds and more of workgroups the latency of one is hidden, and what
//           every wave repeats counts (one cluster, a longer launch: even at 41k).
//           FP64 at that order is run for convergence on small meshes, so four
//           stands for all sizes
//   O <= 3  two: FP32 m=3 300k O=3 1,062 against 1,313 (one: 3,207), O=2 631
//           against 891 (one: 1,092); FP64 O=3 m=3 41k 412 against 508 (785)
// Every split gives the same bits (no contraction across expressions).
template <int O>
constexpr int LEVEL_W = O >= 4 ? 4 : 2;

template <class R, int O, int M, int W, bool TM = false>
static void launch_kind(const LevelArgs& a, const PointArgs& pt, const KPtrs& p, hipStream_t st) {
  const dim3 grid((unsigned)(a.groups + a.points), a.runs);
  if (a.kind == KIND_FUSED)
    hipLaunchKernelGGL((k_level<R, O, M, KIND_FUSED, W, TM>), grid, dim3(64 * W), 0, st, a, p, pt);
  else if (a.kind == KIND_PREDICT)
    hipLaunchKernelGGL((k_level<R, O, M, KIND_PREDICT, W, TM>), grid, dim3(64 * W), 0, st, a, p, pt);
  else
    hipLaunchKernelGGL((k_level<R, O, M, KIND_NEIGHBOR, W>), grid, dim3(64 * W), 0, st, a, p, pt);
}

template <class R, int O, int M>
int launch_level(const KPtrs& p, LevelArgs a, const PointArgs& pt, int runs, hipStream_t st) {
  if (runs <= 0) return 0;
  const bool tm = std::is_same<R, float>::value && O >= 4 && a.trace_mfma;
  const int waves = tm ? 2 : LEVEL_W<O>;
  // a wave per point (a source packet is one); rows of a multiple of eight workgroups (see group_and_run)
  const long long items = (a.kind == KIND_PREDICT ? 0ll : pt.r.n) +
                          (a.kind == KIND_NEIGHBOR || pt.s.n == 0 ? 0 : pt.s.per_run);
  a.groups = (a.end + EPW - 1) / EPW;
  a.points = (int)(((items + waves - 1) / waves + 7) / 8 * 8);
  a.runs = runs;
  if (a.groups + a.points == 0) return 0;   // (a level of a cluster without elements still has its points)
  if constexpr (std::is_same<R, float>::value && O >= 4) {
    if (tm) {
      launch_kind<R, O, M, 2, true>(a, pt, p, st);
      return (int)hipGetLastError();
    }
  }
  launch_kind<R, O, M, LEVEL_W<O>>(a, pt, p, st);
  return (int)hipGetLastError();
}

#define EDG_INST(R, O, M) \
  template int launch_level<R, O, M>(const KPtrs&, LevelArgs, const PointArgs&, int, hipStream_t);

EDG_KERNEL_INSTANCES

}  // namespace edg
