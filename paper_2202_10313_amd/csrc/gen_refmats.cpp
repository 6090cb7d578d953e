// Build-time generator: writes straight-line device code that applies the
// reference-element matrices of the ADER-DG kernels (Sec. III-A (Discrete Formulation)) with their
// values as compile-time constants, so the sparse products cost one FMA per
// structural non-zero and no matrix loads.
//
//   ck_grad  : x_k = d K'_k^T (derivative coefficients along the reference
//              direction w_k, the time kernel's (d^d Q) K^T), combined to
//              physical gradients with the element's G' = V^-T G and stored
//              to LDS; K'_k = sum_c V[k][c] K_c for the three directions along
//              which the basis is sparsest (basis.hpp, sparse_directions)
//   vol_grad : z_k = t K'_k (the volume kernel's T K), combined the same way
//   trace    : p_i = t F~_i for the four faces (the surface kernel's T F~_i)
//   lift     : acc += sum_i p_i F^_i with F^_i = F~_i^T (orthonormal basis, so
//              the inverse mass matrix is the identity on the reference tet)
//   ck_grad_T, vol_grad_T : the transposes of ck_grad and vol_grad after the
//              combination with G' (adjoint kernels); trace and lift are each
//              other's transposes
//
// Usage: gen_refmats <out_header> <order>...
#include <cstdio>
#include <algorithm>
#include <cmath>
#include <cstdlib>
#include <string>
#include <vector>

#include "basis.hpp"

static const double ZERO_TOL = 1e-12;

static std::string hexf(double v) {
  char buf[64];
  std::snprintf(buf, sizeof buf, "%a", v);
  return buf;
}

static void term(std::string& s, bool& first, double c, const std::string& var) {
  if (!first) s += " + ";
  s += "R(" + hexf(c) + ")*" + var;
  first = false;
}

// faces traced by wave P of the two-wave split, in output order
static const int TFACE[2][2] = {{0, 3}, {1, 2}};

int main(int argc, char** argv) {
  if (argc < 3) {
    std::fprintf(stderr, "usage: %s out.h order...\n", argv[0]);
    return 2;
  }
  FILE* f = std::fopen(argv[1], "w");
  if (!f) return 1;
  std::fprintf(f, "// generated by gen_refmats.cpp: reference matrices as straight-line code\n");
  std::fprintf(f, "#pragma once\n#include <hip/hip_runtime.h>\nnamespace edg_gen {\n");
  std::fprintf(f, "template <int O> struct Ref;\n");
  for (int a = 2; a < argc; ++a) {
    const int O = std::atoi(argv[a]);
    edg::RefMats M = edg::reference_matrices(O);
    const edg::Directions Dir = edg::sparse_directions(O);
    const std::vector<double> Kd = edg::direction_matrices(M, Dir);
    const int B = M.B, F = M.F, FP = (F + 3) / 4 * 4;
    int nnzK[3] = {0, 0, 0}, nnzF[4] = {0, 0, 0, 0};
    for (int c = 0; c < 3; ++c)
      for (int i = 0; i < B * B; ++i) nnzK[c] += std::fabs(Kd[c * B * B + i]) > ZERO_TOL;
    for (int i = 0; i < 4; ++i)
      for (int j = 0; j < B * F; ++j) nnzF[i] += std::fabs(M.Ft[i * B * F + j]) > ZERO_TOL;
    std::fprintf(f, "// O=%d: directions V = [%g %g %g; %g %g %g; %g %g %g]; nnz(K'_k) = %d %d %d of %d; "
                 "nnz(F~_i) = %d %d %d %d of %d\n", O, Dir.V[0], Dir.V[1], Dir.V[2], Dir.V[3], Dir.V[4], Dir.V[5],
                 Dir.V[6], Dir.V[7], Dir.V[8], nnzK[0], nnzK[1], nnzK[2], B * B, nnzF[0], nnzF[1], nnzF[2], nnzF[3],
                 B * F);
    std::fprintf(f, "template <> struct Ref<%d> {\n", O);
    std::fprintf(f, "  static constexpr int B = %d, F = %d, FP = %d;\n", B, F, FP);
    std::fprintf(f, "  static constexpr int NNZ_K = %d, NNZ_F = %d;\n", nnzK[0] + nnzK[1] + nnzK[2],
                 nnzF[0] + nnzF[1] + nnzF[2] + nnzF[3]);
    // trace onto one sparse face: p[0..FP) for face i
    for (int i = 2; i < 4; ++i) {
      std::fprintf(f, "  template <class R> __device__ static __forceinline__ void trace_f%d(const R* __restrict__ t, R* __restrict__ p) {\n", i);
      for (int ff = 0; ff < FP; ++ff) {
        std::string s;
        bool first = true;
        if (ff < F)
          for (int b = 0; b < B; ++b) {
            const double v = M.Ft[(i * B + b) * F + ff];
            if (std::fabs(v) > ZERO_TOL) term(s, first, v, "t[" + std::to_string(b) + "]");
          }
        if (first) s = "R(0)";
        std::fprintf(f, "    p[%d] = %s;\n", ff, s.c_str());
      }
      std::fprintf(f, "  }\n");
    }
    // the traces of faces 0 and 1 as one dense product on the matrix cores
    // (v_mfma_f32_32x32x2f32: 32 rows x 32 columns, two modes per step): the
    // B operand of k-step s in lane l is the coefficient of mode 2 s + l / 32
    // onto face (l % 32) / 16, face mode l % 16 (zero past B or F)
    {
      const int MK = (B + 1) / 2;
      std::fprintf(f, "  static constexpr int MK = %d;  // k-steps of the matrix-core trace of faces 0 and 1\n", MK);
      std::fprintf(f, "  static constexpr float FT01[%d] = {", MK * 64);
      for (int st = 0; st < MK; ++st)
        for (int l = 0; l < 64; ++l) {
          const int b = 2 * st + l / 32, face = (l % 32) / 16, ff = l % 16;
          const double v = (b < B && ff < F) ? M.Ft[(face * B + b) * F + ff] : 0.0;
          std::fprintf(f, "%sfloat(%s)", (st == 0 && l == 0) ? "" : ", ", hexf(std::fabs(v) > ZERO_TOL ? v : 0.0).c_str());
        }
      std::fprintf(f, "};\n");
    }
    // ---- W-wave splits (W = 2, 4): wave P of W owns the elementwise modes
    // [mb(W, P), mb(W, P + 1)), computes a contiguous range of stiffness
    // outputs balanced by cost and the trace chunks tchunk(W, P, .).
    // X_w<W>(w, ...) runs wave w's part of X.
    const int NCH = FP / 4;   // chunks of four face modes per face
    std::vector<int> mbs[5], chunks[5][4];
    for (int W = 2; W <= 4; W += 2) {
      // modes: blocks of nine where they divide evenly enough (a memory-
      // variable mode is owned by one of nine lanes), else equal parts
      mbs[W].assign(W + 1, B);
      for (int P = 0; P < W; ++P)
        mbs[W][P] = W == 2 ? (P == 0 ? 0 : (B >= 18 ? 9 * ((B + 9) / 18) : (B + 1) / 2))
                           : (B > 27 ? 9 * P : (P * B + W - 1) / W);
      // trace chunks: W = 2 takes one of the two dense faces (0 and 1, the
      // faces through the reference vertex's two first edges) and one of the
      // sparse ones (2, 3) per wave; W = 4 deals chunks out, largest first
      if (W == 2) {
        for (int P = 0; P < 2; ++P)
          for (int ii = 0; ii < 2; ++ii)
            for (int k = 0; k < NCH; ++k) chunks[2][P].push_back(TFACE[P][ii] * NCH + k);
      } else {
        std::vector<std::pair<int, int>> cost;
        for (int c = 0; c < 4 * NCH; ++c) {
          int nz = 4;   // the chunk's stores
          for (int ff = 4 * (c % NCH); ff < std::min(F, 4 * (c % NCH) + 4); ++ff)
            for (int bb = 0; bb < B; ++bb) nz += std::fabs(M.Ft[(c / NCH * B + bb) * F + ff]) > ZERO_TOL;
          cost.push_back({-nz, c});
        }
        std::sort(cost.begin(), cost.end());
        int load[4] = {0, 0, 0, 0};
        for (auto& x : cost) {
          const int P = (int)(std::min_element(load, load + 4) - load);
          load[P] -= x.first;
          chunks[4][P].push_back(x.second);
        }
      }
    }
    size_t ntc[5] = {0};
    for (int W = 2; W <= 4; W += 2)
      for (int P = 0; P < W; ++P) ntc[W] = std::max(ntc[W], chunks[W][P].size());
    std::fprintf(f, "  // first mode of wave p of W (p = W: B); largest and smallest number of modes of a wave; every first mode a multiple of 9\n");
    std::fprintf(f, "  __host__ __device__ static constexpr int mb(int W, int p) { return W == 2 ? (p == 0 ? 0 : p == 1 ? %d : %d) : (p == 0 ? 0 : p == 1 ? %d : p == 2 ? %d : p == 3 ? %d : %d); }\n",
                 mbs[2][1], B, mbs[4][1], mbs[4][2], mbs[4][3], B);
    for (int W = 2; W <= 4; W += 2) {
      int nbx = 0, nbn = B, tn = 99;
      bool al = true;
      for (int P = 0; P < W; ++P) {
        nbx = std::max(nbx, mbs[W][P + 1] - mbs[W][P]);
        nbn = std::min(nbn, mbs[W][P + 1] - mbs[W][P]);
        tn = std::min(tn, (int)chunks[W][P].size());
        al = al && mbs[W][P] % 9 == 0;
      }
      std::fprintf(f, "  static constexpr int NBX%d = %d, NBN%d = %d, NTN%d = %d;\n  static constexpr bool NINES%d = %s;\n", W, nbx,
                   W, nbn, W, tn, W, al ? "true" : "false");
    }
    std::fprintf(f, "  template <int W> static constexpr int nbx = W == 2 ? NBX2 : NBX4;\n");
    std::fprintf(f, "  template <int W> static constexpr int nbn = W == 2 ? NBN2 : NBN4;\n  template <int W> static constexpr int ntn = W == 2 ? NTN2 : NTN4;\n");
    std::fprintf(f, "  template <int W> static constexpr bool nines = W == 2 ? NINES2 : NINES4;\n");
    std::fprintf(f, "  // trace chunks (four face modes each) of wave p of W: their number, at most ntc, at least ntn; chunk ii is face tchunk / %d, modes 4 (tchunk %% %d) ..\n", NCH, NCH);
    std::fprintf(f, "  template <int W> static constexpr int ntc = W == 2 ? %d : %d;\n", (int)ntc[2], (int)ntc[4]);
    std::fprintf(f, "  // (-1: none); 6 bits per entry\n");
    std::fprintf(f, "  template <int W> __device__ static __forceinline__ int tchunk(int p, int ii) {\n");
    for (int W = 2; W <= 4; W += 2) {
      std::fprintf(f, "    if (W == %d) {\n", W);
      for (int P = 0; P < W; ++P) {
        unsigned long long w = 0;
        for (size_t ii = 0; ii < ntc[W]; ++ii)
          w |= (unsigned long long)(ii < chunks[W][P].size() ? chunks[W][P][ii] : 63) << (6 * ii);
        std::fprintf(f, "      %sconst unsigned long long t%d = 0x%llxull;\n", "", P, w);
      }
      if (W == 2) std::fprintf(f, "      const unsigned long long t = p == 0 ? t0 : t1;\n");
      else std::fprintf(f, "      const unsigned long long t = p == 0 ? t0 : p == 1 ? t1 : p == 2 ? t2 : t3;\n");
      std::fprintf(f, "      const int c = (int)((t >> (6 * ii)) & 63);\n      return c == 63 ? -1 : c;\n    }\n");
    }
    std::fprintf(f, "    return -1;\n  }\n");
    // stiffness output ranges, balanced by cost
    auto split = [&](bool vol, int W) {
      std::vector<int> nz(B, 0);
      for (int b = 0; b < B; ++b)
        for (int c = 0; c < 3; ++c)
          for (int bb = 0; bb < B; ++bb) {
            const double k = vol ? Kd[(c * B + bb) * B + b] : Kd[(c * B + b) * B + bb];
            nz[b] += std::fabs(k) > ZERO_TOL;
          }
      // cost of an output mode: its FMAs + 9 for the physical combination
      // and stores; all-zero modes only store zeros (3)
      std::vector<double> cost(B);
      double tot = 0;
      for (int b = 0; b < B; ++b) { cost[b] = nz[b] ? nz[b] + 9.0 : 3.0; tot += cost[b]; }
      std::vector<int> cut(1, 0);
      double acc = 0;
      int s = 0;
      for (int P = 1; P < W; ++P) {
        while (s < B && acc + cost[s] / 2 < tot * P / W) acc += cost[s++];
        cut.push_back(s);
      }
      cut.push_back(B);
      return cut;
    };
    // emits X_w<W>(w, ...), the dispatch over the waves of both splits
    auto dispatch = [&](const char* name, const char* params, const char* call) {
      std::fprintf(f, "  template <int W, class R> __device__ static __forceinline__ void %s_w(int w, %s) {\n", name, params);
      std::fprintf(f, "    if constexpr (W == 2) {\n      if (w == 0) %s_w2p0(%s); else %s_w2p1(%s);\n    } else {\n", name, call,
                   name, call);
      std::fprintf(f, "      if (w < 2) { if (w == 0) %s_w4p0(%s); else %s_w4p1(%s); }\n", name, call, name, call);
      std::fprintf(f, "      else { if (w == 2) %s_w4p2(%s); else %s_w4p3(%s); }\n    }\n  }\n", name, call, name, call);
    };
    for (int W = 2; W <= 4; W += 2)
      for (int vol = 0; vol < 2; ++vol) {
        const std::vector<int> cut = split(vol != 0, W);
        for (int P = 0; P < W; ++P) {
          std::fprintf(f, "  template <class R> __device__ static __forceinline__ void %s_w%dp%d(const R* __restrict__ d, const R* __restrict__ G, R* g0, R* g1, R* g2) {\n",
                       vol ? "vol_grad" : "ck_grad", W, P);
          for (int b = cut[P]; b < cut[P + 1]; ++b) {
            bool any = false;
            for (int c = 0; c < 3; ++c) {
              std::string t;
              bool first = true;
              for (int bb = 0; bb < B; ++bb) {
                const double k = vol ? Kd[(c * B + bb) * B + b] : Kd[(c * B + b) * B + bb];
                if (std::fabs(k) > ZERO_TOL) term(t, first, k, "d[" + std::to_string(bb) + "]");
              }
              if (first) t = "R(0)";
              else any = true;
              std::fprintf(f, "    const R x%d_%d = %s;\n", c, b, t.c_str());
            }
            if (any) {
              std::fprintf(f, "    g0[%d] = G[0]*x0_%d + G[3]*x1_%d + G[6]*x2_%d;\n", b, b, b, b);
              std::fprintf(f, "    g1[%d] = G[1]*x0_%d + G[4]*x1_%d + G[7]*x2_%d;\n", b, b, b, b);
              std::fprintf(f, "    g2[%d] = G[2]*x0_%d + G[5]*x1_%d + G[8]*x2_%d;\n", b, b, b, b);
            } else {
              std::fprintf(f, "    g0[%d] = R(0); g1[%d] = R(0); g2[%d] = R(0);\n", b, b, b);
            }
          }
          std::fprintf(f, "  }\n");
        }
      }
    for (int W = 2; W <= 4; W += 2)
      for (int P = 0; P < W; ++P) {
        std::fprintf(f, "  template <class R> __device__ static __forceinline__ void trace_w%dp%d(const R* __restrict__ t, R* __restrict__ p) {\n", W, P);
        for (size_t ii = 0; ii < ntc[W]; ++ii)
          for (int k = 0; k < 4; ++k) {
            std::string t;
            bool first = true;
            if (ii < chunks[W][P].size()) {
              const int c = chunks[W][P][ii], i = c / NCH, ff = 4 * (c % NCH) + k;
              if (ff < F)
                for (int b = 0; b < B; ++b) {
                  const double v = M.Ft[(i * B + b) * F + ff];
                  if (std::fabs(v) > ZERO_TOL) term(t, first, v, "t[" + std::to_string(b) + "]");
                }
            }
            if (first) t = "R(0)";
            std::fprintf(f, "    p[%d] = %s;\n", (int)(4 * ii) + k, t.c_str());
          }
        std::fprintf(f, "  }\n");
        const int lo = mbs[W][P], hi = mbs[W][P + 1];
        // (assigned, not accumulated, and to all entries up to the largest
        // wave's: waves that touch different entries of a caller's array let
        // the compiler merge their accesses through a pointer select, which
        // keeps entries of it in scratch memory)
        std::fprintf(f, "  template <class R> __device__ static __forceinline__ void lift_w%dp%d(const R* __restrict__ p, R* __restrict__ out) {\n", W, P);
        int nbx = 0;
        for (int P2 = 0; P2 < W; ++P2) nbx = std::max(nbx, mbs[W][P2 + 1] - mbs[W][P2]);
        for (int lb = 0; lb < nbx; ++lb) {
          const int b = mbs[W][P] + lb;
          std::string t;
          bool first = true;
          if (b < mbs[W][P + 1])
            for (int i = 0; i < 4; ++i)
              for (int ff = 0; ff < F; ++ff) {
                const double v = M.Ft[(i * B + b) * F + ff];
                if (std::fabs(v) > ZERO_TOL) term(t, first, v, "p[" + std::to_string(i * FP + ff) + "]");
              }
          if (first) t = "R(0)";
          std::fprintf(f, "    out[%d] = %s;\n", lb, t.c_str());
        }
        std::fprintf(f, "  }\n");
      }
    // transposed stiffness: full input rows y0, y1, y2 (one per reference
    // direction: the physical-gradient adjoints combined with G'), outputs
    // for the wave's own modes (assigned, all entries: see lift)
    for (int W = 2; W <= 4; W += 2)
      for (int vol = 0; vol < 2; ++vol)
        for (int P = 0; P < W; ++P) {
          int nbx = 0;
          for (int P2 = 0; P2 < W; ++P2) nbx = std::max(nbx, mbs[W][P2 + 1] - mbs[W][P2]);
          std::fprintf(f, "  template <class R> __device__ static __forceinline__ void %s_w%dp%d(const R* y0, const R* y1, const R* y2, R* __restrict__ out) {\n",
                       vol ? "vol_grad_T" : "ck_grad_T", W, P);
          for (int lb = 0; lb < nbx; ++lb) {
            const int bb = mbs[W][P] + lb;
            std::string t;
            bool first = true;
            if (bb < mbs[W][P + 1])
              for (int c = 0; c < 3; ++c)
                for (int b = 0; b < B; ++b) {
                  const double k = vol ? Kd[(c * B + bb) * B + b] : Kd[(c * B + b) * B + bb];
                  if (std::fabs(k) > ZERO_TOL) term(t, first, k, "y" + std::to_string(c) + "[" + std::to_string(b) + "]");
                }
            if (first) t = "R(0)";
            std::fprintf(f, "    out[%d] = %s;\n", lb, t.c_str());
          }
          std::fprintf(f, "  }\n");
        }
    const char* gp = "const R* __restrict__ d, const R* __restrict__ G, R* g0, R* g1, R* g2";
    dispatch("ck_grad", gp, "d, G, g0, g1, g2");
    dispatch("vol_grad", gp, "d, G, g0, g1, g2");
    const char* gtp = "const R* y0, const R* y1, const R* y2, R* __restrict__ out";
    dispatch("ck_grad_T", gtp, "y0, y1, y2, out");
    dispatch("vol_grad_T", gtp, "y0, y1, y2, out");
    dispatch("trace", "const R* __restrict__ t, R* __restrict__ p", "t, p");
    dispatch("lift", "const R* __restrict__ p, R* __restrict__ out", "p, out");
    std::fprintf(f, "};\n");
  }
  std::fprintf(f, "}  // namespace edg_gen\n");
  std::fclose(f);
  return 0;
}
