// HIP kernels of libshp for gfx950: FP64 sum-factorisation stages on the matrix
// cores (v_mfma_f64_4x4x4_4b_f64).
//
// Every stage of the sum-factorised operators is a set of independent line
// contractions with one small table: Y[m] = sum_k T[m][k] X[k] for each line.
// v_mfma_f64_4x4x4_4b takes four blocks of 4 x 4 x 4; with the same 4 x 4
// piece of the table in all four blocks it is a 4 x 4 by 4 x 16 product, one
// column per line.  Lane l holds T[l % 4][l / 16] (A), X[l / 16][l % 16] (B) and
// Y[l / 16][l % 16] (C, D), a layout checked on gfx950 before use.  So
//  - B and D have the same layout: the result of one contraction is the input
//    of the next one along the same line without leaving the registers;
//  - rows are padded to multiples of 4, lines to multiples of 16 (a 64-wide
//    thread-per-line stage pads its lines to 64: at P = 10 one element's 144
//    lines keep 3 of 8 waves busy, here 9 sets of 16 lines);
//  - a wave holds K/4 values per lane of a set of lines instead of K, so u, D_0 u
//    and the factors of a set's points stay in registers at P = 10;
//  - the tables are vector operands read from LDS, not scalar loads that a
//    stage has to wait for.
// One instruction does 256 multiply-adds; it reached 62 TF where v_fma_f64
// reached 45 and v_mfma_f64_16x16x4 41 (dependent chains, two waves per SIMD).
// Each accumulates k = 0, 1, 2, 3 in order with one rounding per step, so a
// stage's results are bit for bit those of the thread-per-line stages with the
// same order of summation.
//
// The eta1 lines (e, j, k) carry u, D_0 u and the geometric factors of their
// points in registers, so that stage p, D_0, the metric, D_0^T and stage p^T run
// without a round trip of u and D_0 u through LDS (three point buffers per
// element instead of four).
//
// What bounds the tile: LDS and the matrix cores take turns rather than overlap,
// since all waves of a work-group are in the same stage (counters, P = 6 mesh: LDS
// busy 70 % of the time, matrix cores 24 %, VALU 32 %; P = 10 prisms 47, 20 and 17),
// so what matters is the padding.  Helmholtz on the mixed mesh (1 hex : 2 prisms : 6 pyramids : 6 tets,
// 8M points), thread-per-line / here, us:
//   P = 2 93 / 79, 6 119 / 95, 9 214 / 131, 10 220 / 141;
//   P = 1 101 / 104, 3 100 / 129, 4 114 / 125, 5 130 / 136, 7 150 / 156, 8 153 / 154.
// The first are the orders whose lines fill the blocks (Q = P + 2 = 4, 8, 12, and
// 11 of 12); the others stay with the thread-per-line tile.  Tried and slower:
// v_mfma_f64_16x16x4 (a third of the table reads, longer chains), tables read
// once for several sets of a wave and persistent work-groups that prefetch the
// next tile (both take registers that the second work-group of a CU needs).
#pragma once
#include "shp_kernels.hpp"

namespace shp {
namespace mf {

__device__ __forceinline__ double mma(double a, double b, double c) {
  return __builtin_amdgcn_mfma_f64_4x4x4f64(a, b, c, 0, 0, 0);
}

template <int SH, int P_>
struct MD {
  static constexpr int P = P_, n = P + 1, Q = P + 2, Q2 = Q * Q, Q3 = Q * Q * Q;
  static constexpr int KQ = (Q + 3) / 4, KN = (n + 3) / 4;  // groups of 4 rows
  // point buffers [i][j][k] with strides SI, SJ, 1; columns F[c][k] at c SJ + k
  static constexpr int SJ = qpad(Q);
  static constexpr int SI = Q * SJ;
  static constexpr int S3 = Q * SI;
  static constexpr int NP = num_modes(SH, P), NC = num_cols(SH, P);
  static constexpr TabLayout L = tab_layout(SH, P);
  static constexpr MfLayout H = mf_layout(SH, P);
  static constexpr int oA = H.A, oB = H.B, oC = H.C, oD = H.D;
  static constexpr int head(bool deriv) { return deriv ? H.total : H.D; }
};

struct Lane {
  int ln, lr, li;  // line of the set, row of a group, row of a table block
  int wv;          // wave (uniform)
};
__device__ __forceinline__ Lane lane_of() {
  const int l = threadIdx.x & 63;
  return Lane{l & 15, l >> 4, l & 3, __builtin_amdgcn_readfirstlane(threadIdx.x >> 6)};
}

// LDS view of a tile of E elements, NB point buffers per element
template <int SH, int P, int E_, int NB, bool DERIV>
struct View {
  using D = MD<SH, P>;
  static constexpr int E = E_, PER = NB * D::S3, HEAD = D::head(DERIV);
  double* tab;
  const int* cols;
  double* el;
  __device__ explicit View(double* smem)
      : tab(smem), cols(reinterpret_cast<const int*>(smem + D::H.cols)), el(smem + HEAD) {}
  static constexpr size_t BYTES = sizeof(double) * (size_t)(HEAD + E * PER);
};

// K rows of a line at byte-free offset o (stride st): b[g] = x[4 g + row], zero
// past the last row (read from the last row, so every read is initialised)
template <int K, int STRIDE, int KB>
__device__ __forceinline__ void load_rows(const double* x, const Lane& w, double (&b)[KB]) {
  constexpr int REM = K - 4 * (KB - 1);
  const double* p = x + w.lr * STRIDE;
#pragma unroll
  for (int g = 0; g < KB - 1; ++g) b[g] = p[4 * g * STRIDE];
  const int rl = REM == 4 ? w.lr : (w.lr < REM ? w.lr : REM - 1);
  const double v = x[(4 * (KB - 1) + rl) * STRIDE];
  b[KB - 1] = (REM == 4 || w.lr < REM) ? v : 0.0;
}

// rows m < M of the result to y (stride st); ok: this lane's line is in the tile
template <int M, int STRIDE, int MB>
__device__ __forceinline__ void store_rows(double* y, const Lane& w, const double (&a)[MB], bool ok) {
  double* p = y + w.lr * STRIDE;
  if (ok) {
#pragma unroll
    for (int g = 0; g < MB - 1; ++g) p[4 * g * STRIDE] = a[g];
    if (M == 4 * MB || 4 * (MB - 1) + w.lr < M) p[4 * (MB - 1) * STRIDE] = a[MB - 1];
  }
}

template <int MB>
__device__ __forceinline__ void zero(double (&a)[MB]) {
#pragma unroll
  for (int m = 0; m < MB; ++m) a[m] = 0.0;
}

// acc[m] += sum_k T[m][k] b[k]; table entry T[m][k] at t + m MS + k KS
template <int MS, int KS, int MB, int KB>
__device__ __forceinline__ void contract(const double* t, const Lane& w, const double (&b)[KB], double (&acc)[MB]) {
  const double* p = t + w.li * MS + w.lr * KS;
#pragma unroll
  for (int kb = 0; kb < KB; ++kb)
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) acc[mb] = mma(p[4 * mb * MS + 4 * kb * KS], b[kb], acc[mb]);
}
// table stored [k][m] (rows of Q): the forward stages, and D^T
template <int Q, int MB, int KB>
__device__ __forceinline__ void contract_km(const double* tab, const Lane& w, const double (&b)[KB],
                                            double (&acc)[MB]) {
  contract<1, Q>(tab, w, b, acc);
}
// table stored [m][k]: the transposed stages, and D
template <int Q, int MB, int KB>
__device__ __forceinline__ void contract_mk(const double* tab, const Lane& w, const double (&b)[KB],
                                            double (&acc)[MB]) {
  contract<Q, 1>(tab, w, b, acc);
}

// x y rounded on its own: not fused into a later addition, so that a value kept
// in registers is the one a stage through LDS would hold
__device__ __forceinline__ double mul_rn(double x, double y) {
#pragma clang fp contract(off)
  return x * y;
}

// ---------------------------------------------------------------------------
// stages r and q (modes <-> F[c][k] <-> G[p][j][k])
// ---------------------------------------------------------------------------

// The columns of the eta3 families have tables of their own, so a set holds
// columns of one family; the sets of a stage are numbered over its families, and
// wave w of NW takes the sets with number % NW = w.
constexpr int sets_of(int n) { return (n + 15) / 16; }

// x (modes at xb) -> F (columns at fb)
template <int SH, int P, int NW, int KAP = 0, int T0 = 0, class V>
__device__ __forceinline__ void stage_r(const V& T, const Lane& w, int xb, int fb) {
  if constexpr (KAP <= (SH == HEX ? 0 : P)) {
    using D = MD<SH, P>;
    constexpr int RL = P + 1 - KAP, ncol = fam_ncols(SH, P, KAP), c0 = fam_start(SH, P, KAP);
    // collapsed-vertex modes: the columns of family 1 also collect v1 (row 1 of
    // family 0) times one mode, as row RL of the contraction
    constexpr bool EXTRA = SH != HEX && KAP == 1;
    constexpr int K = RL + (EXTRA ? 1 : 0), KB = (K + 3) / 4, nl = V::E * ncol;
#pragma unroll
    for (int s = 0; s < sets_of(nl); ++s) {
      if (w.wv != (T0 + s) % NW) continue;
      const int l0 = 16 * s + w.ln, l = l0 < nl ? l0 : nl - 1;
      const int e = l / ncol, idx = l - e * ncol;
      const int pk = T.cols[c0 + idx];
      const double* x = T.el + e * V::PER + xb;
      const double* C3 = T.tab + D::oC + fam_index(P, KAP, 0) * D::Q;
      const int off = pk >> 8;
      double b[KB], acc[D::KQ];
#pragma unroll
      for (int g = 0; g < KB; ++g) {
        const int r = 4 * g + w.lr;
        int m = off + (r < RL ? r : RL - 1);
        if (EXTRA && r == RL) m = SH == PRISM ? idx * (P + 1) + 1 : 1;
        const double v = x[m];
        b[g] = (4 * g + 3 < K || r < K) ? v : 0.0;
      }
      zero(acc);
      if constexpr (EXTRA) {
#pragma unroll
        for (int g = 0; g < KB; ++g) {
          const int r = 4 * g + w.lr;
          const double* t = (r < RL ? C3 + r * D::Q : T.tab + D::oC + D::Q) + w.li;
#pragma unroll
          for (int mb = 0; mb < D::KQ; ++mb) acc[mb] = mma(t[4 * mb], b[g], acc[mb]);
        }
      } else {
        contract_km<D::Q>(C3, w, b, acc);
      }
      store_rows<D::Q, 1>(T.el + e * V::PER + fb + (pk & 255) * D::SJ, w, acc, l0 < nl);
    }
    stage_r<SH, P, NW, KAP + 1, T0 + sets_of(nl)>(T, w, xb, fb);
  }
}

// F (columns at fb) -> y (modes at yb)
template <int SH, int P, int NW, int KAP = 0, int T0 = 0, class V>
__device__ __forceinline__ void stage_rT(const V& T, const Lane& w, int fb, int yb) {
  if constexpr (KAP <= (SH == HEX ? 0 : P)) {
    using D = MD<SH, P>;
    constexpr int RL = P + 1 - KAP, ncol = fam_ncols(SH, P, KAP), c0 = fam_start(SH, P, KAP);
    constexpr int MB = (RL + 3) / 4, nl = V::E * ncol;
#pragma unroll
    for (int s = 0; s < sets_of(nl); ++s) {
      if (w.wv != (T0 + s) % NW) continue;
      const int l0 = 16 * s + w.ln, l = l0 < nl ? l0 : nl - 1;
      const int e = l / ncol, idx = l - e * ncol;
      const int pk = T.cols[c0 + idx];
      const double* F = T.el + e * V::PER + fb;
      double b[D::KQ], acc[MB];
      load_rows<D::Q, 1>(F + (pk & 255) * D::SJ, w, b);
      zero(acc);
      contract_mk<D::Q>(T.tab + D::oC + fam_index(P, KAP, 0) * D::Q, w, b, acc);
      if constexpr (SH != HEX && KAP == 0) {
        // adjoint of the collapsed-vertex modes: row r = 1 of family 0's columns
        // collects v1 on the neighbouring columns
        double s0[D::KQ], s1[D::KQ];
        load_rows<D::Q, 1>(F + (SH == PRISM ? P + 1 + idx : SH == PYR ? P + 1 : 1) * D::SJ, w, s0);
        if constexpr (SH != PRISM) {
          load_rows<D::Q, 1>(F + (SH == PYR ? 1 : P + 1) * D::SJ, w, s1);
#pragma unroll
          for (int g = 0; g < D::KQ; ++g) s0[g] += s1[g];
        }
        if constexpr (SH == PYR) {
          load_rows<D::Q, 1>(F + (P + 2) * D::SJ, w, s1);
#pragma unroll
          for (int g = 0; g < D::KQ; ++g) s0[g] += s1[g];
        }
        const double* v1 = T.tab + D::oC + D::Q + w.lr;
        // only row 1 takes the sum (zeros in the other rows of the table would make
        // an overflowed s0 NaN there)
        double a1 = acc[0];
#pragma unroll
        for (int g = 0; g < D::KQ; ++g) a1 = mma(v1[4 * g], s0[g], a1);
        acc[0] = w.lr == 1 ? a1 : acc[0];
      }
      store_rows<RL, 1>(T.el + e * V::PER + yb + (pk >> 8), w, acc, l0 < nl);
    }
    stage_rT<SH, P, NW, KAP + 1, T0 + sets_of(nl)>(T, w, fb, yb);
  }
}

// the tet's stage q: its eta2 functions depend on p, so a set holds lines of one p
template <int P, int NW, int PP = 0, class V>
__device__ __forceinline__ void stage_q_tet(const V& T, const Lane& w, int fb, int gb) {
  if constexpr (PP <= P) {
    using D = MD<TET, P>;
    constexpr int NQ = P + 1 - PP, K = NQ + (PP == 1 ? 1 : 0), KB = (K + 3) / 4;
    constexpr int cb = col_base(TET, P, PP), nl = V::E * D::Q, T0 = PP * sets_of(nl);
#pragma unroll
    for (int s = 0; s < sets_of(nl); ++s) {
      if (w.wv != (T0 + s) % NW) continue;
      const int l0 = 16 * s + w.ln, l = l0 < nl ? l0 : nl - 1;
      const int e = l / D::Q, k = l - e * D::Q;
      const double* F = T.el + e * V::PER + fb + k;
      const double* B2 = T.tab + D::oB + fam_index(P, PP, 0) * D::Q;
      double b[KB], acc[D::KQ];
#pragma unroll
      for (int g = 0; g < KB; ++g) {
        const int q = 4 * g + w.lr;
        int c = cb + (q < NQ ? q : NQ - 1);
        if (PP == 1 && q == NQ) c = 1;  // column (0, 1), through v1 (row 1 of family 0)
        const double v = F[c * D::SJ];
        b[g] = (4 * g + 3 < K || q < K) ? v : 0.0;
      }
      zero(acc);
      if constexpr (PP == 1) {
#pragma unroll
        for (int g = 0; g < KB; ++g) {
          const int q = 4 * g + w.lr;
          const double* t = (q < NQ ? B2 + q * D::Q : T.tab + D::oB + D::Q) + w.li;
#pragma unroll
          for (int mb = 0; mb < D::KQ; ++mb) acc[mb] = mma(t[4 * mb], b[g], acc[mb]);
        }
      } else {
        contract_km<D::Q>(B2, w, b, acc);
      }
      store_rows<D::Q, D::SJ>(T.el + e * V::PER + gb + PP * D::SI + k, w, acc, l0 < nl);
    }
    stage_q_tet<P, NW, PP + 1>(T, w, fb, gb);
  }
}

// F (columns at fb) -> G[p][j][k] (at gb)
template <int SH, int P, int NW, class V>
__device__ __forceinline__ void stage_q(const V& T, const Lane& w, int fb, int gb) {
  using D = MD<SH, P>;
  if constexpr (SH == TET) {
    stage_q_tet<P, NW>(T, w, fb, gb);
  } else {
    constexpr int nl = V::E * D::n * D::Q;
#pragma unroll
    for (int s = 0; s < sets_of(nl); s += NW) {
      if (s + w.wv >= sets_of(nl)) continue;
      const int l0 = 16 * (s + w.wv) + w.ln, l = l0 < nl ? l0 : nl - 1;
      const int e = l / (D::n * D::Q), rem = l - e * (D::n * D::Q);
      const int p = rem / D::Q, k = rem - p * D::Q;
      double* el = T.el + e * V::PER + k;
      double b[D::KN], acc[D::KQ];
      load_rows<D::n, D::SJ>(el + fb + p * (D::n * D::SJ), w, b);
      zero(acc);
      contract_km<D::Q>(T.tab + D::oB, w, b, acc);
      store_rows<D::Q, D::SJ>(el + gb + p * D::SI, w, acc, l0 < nl);
    }
  }
}

template <int P, int NW, int PP = 0, class V>
__device__ __forceinline__ void stage_qT_tet(const V& T, const Lane& w, int gb, int fb) {
  if constexpr (PP <= P) {
    using D = MD<TET, P>;
    constexpr int NQ = P + 1 - PP, MB = (NQ + 3) / 4, nl = V::E * D::Q, T0 = PP * sets_of(nl);
#pragma unroll
    for (int s = 0; s < sets_of(nl); ++s) {
      if (w.wv != (T0 + s) % NW) continue;
      const int l0 = 16 * s + w.ln, l = l0 < nl ? l0 : nl - 1;
      const int e = l / D::Q, k = l - e * D::Q;
      const double* G = T.el + e * V::PER + gb + k;
      double b[D::KQ], acc[MB];
      load_rows<D::Q, D::SJ>(G + PP * D::SI, w, b);
      zero(acc);
      contract_mk<D::Q>(T.tab + D::oB + fam_index(P, PP, 0) * D::Q, w, b, acc);
      if constexpr (PP == 0) {
        // adjoint of the extra eta2 term: column (0, 1) also collects v1 * G[1]
        load_rows<D::Q, D::SJ>(G + D::SI, w, b);
        const double* v1 = T.tab + D::oB + D::Q + w.lr;
        double a1 = acc[0];  // row 1 alone takes it, as in stage_rT
#pragma unroll
        for (int g = 0; g < D::KQ; ++g) a1 = mma(v1[4 * g], b[g], a1);
        acc[0] = w.lr == 1 ? a1 : acc[0];
      }
      store_rows<NQ, D::SJ>(T.el + e * V::PER + fb + col_base(TET, P, PP) * D::SJ + k, w, acc, l0 < nl);
    }
    stage_qT_tet<P, NW, PP + 1>(T, w, gb, fb);
  }
}

// G[p][j][k] (at gb) -> F (columns at fb)
template <int SH, int P, int NW, class V>
__device__ __forceinline__ void stage_qT(const V& T, const Lane& w, int gb, int fb) {
  using D = MD<SH, P>;
  if constexpr (SH == TET) {
    stage_qT_tet<P, NW>(T, w, gb, fb);
  } else {
    constexpr int nl = V::E * D::n * D::Q;
#pragma unroll
    for (int s = 0; s < sets_of(nl); s += NW) {
      if (s + w.wv >= sets_of(nl)) continue;
      const int l0 = 16 * (s + w.wv) + w.ln, l = l0 < nl ? l0 : nl - 1;
      const int e = l / (D::n * D::Q), rem = l - e * (D::n * D::Q);
      const int p = rem / D::Q, k = rem - p * D::Q;
      double* el = T.el + e * V::PER + k;
      double b[D::KQ], acc[D::KN];
      load_rows<D::Q, D::SJ>(el + gb + p * D::SI, w, b);
      zero(acc);
      contract_mk<D::Q>(T.tab + D::oB, w, b, acc);
      store_rows<D::n, D::SJ>(el + fb + p * (D::n * D::SJ), w, acc, l0 < nl);
    }
  }
}

// ---------------------------------------------------------------------------
// the tile's inputs
// ---------------------------------------------------------------------------

typedef double f64x2 __attribute__((ext_vector_type(2)));

// The modes of ne <= E elements (zero for the others) and the head's image,
// requested together and written to LDS once everything is requested: after()
// runs in between (one memory latency for all of the tile's inputs, where a
// loop that writes as it loads waits once per pass).
template <int SH, int P, bool DERIV, int NT, class V, class After>
__device__ __forceinline__ void load_tile(const V& T, const double* __restrict__ src, const double* __restrict__ img,
                                          int ne, int xb, After after) {
  using D = MD<SH, P>;
  constexpr int NP = D::NP, MX = (V::E * NP + NT - 1) / NT;
  constexpr int H2 = V::HEAD / 2, MH = (H2 + NT - 1) / NT;  // HEAD is even
  const int t0 = threadIdx.x, nm = ne * NP;
  double x[MX];
  f64x2 h[MH];
#pragma unroll
  for (int s = 0; s < MX; ++s) {
    const int t = t0 + s * NT;
    x[s] = src[t < nm ? t : nm - 1];
  }
  const f64x2* im = reinterpret_cast<const f64x2*>(img);
#pragma unroll
  for (int s = 0; s < MH; ++s) {
    const int t = t0 + s * NT;
    h[s] = im[t < H2 ? t : H2 - 1];
  }
  after();
#pragma unroll
  for (int s = 0; s < MX; ++s) {
    const int t = t0 + s * NT;
    if ((s + 1) * NT <= V::E * NP || t < V::E * NP) {
      const int e = t / NP;
      T.el[e * V::PER + xb + (t - e * NP)] = t < nm ? x[s] : 0.0;
    }
  }
  f64x2* hd = reinterpret_cast<f64x2*>(T.tab);
#pragma unroll
  for (int s = 0; s < MH; ++s) {
    const int t = t0 + s * NT;
    if ((s + 1) * NT <= H2 || t < H2) hd[t] = h[s];
  }
}

template <int SH, int P, int NT, class V>
__device__ __forceinline__ void store_y(const V& T, double* __restrict__ dst, int ne, int yb) {
  constexpr int NP = MD<SH, P>::NP;
  for (int t = threadIdx.x; t < ne * NP; t += NT) {
    const int e = t / NP;
    dst[t] = T.el[e * V::PER + yb + (t - e * NP)];
  }
}

// ---------------------------------------------------------------------------
// Laplacian / Helmholtz / advection-diffusion-reaction tile
// ---------------------------------------------------------------------------

// E elements on NW waves, at most SPW sets of 16 eta1 lines per wave.
// react: the reaction term lambda jw u (Helmholtz); ADR: the advection term too.
template <int SH, int P, int E, int SPW, int NW, bool ADR>
__device__ void helm_tile(const double* __restrict__ img, const double* __restrict__ fac,
                          const double* __restrict__ adv, const double* __restrict__ in, double* __restrict__ out,
                          int ne, double lam, bool react, double* smem) {
  using D = MD<SH, P>;
  using V = View<SH, P, E, 3, true>;
  constexpr int Q = D::Q, Q2 = D::Q2, Q3 = D::Q3, KQ = D::KQ, KN = D::KN, NT = 64 * NW;
  constexpr int U = 0, G1 = D::S3, G2 = 2 * D::S3, nl = E * Q2;
  // streamed past the caches when the sets' rows are whole cache lines; else a
  // line is shared by two waves' loads
  constexpr int AUX = Q % 4 == 0 ? 2 : 0;
  const V T(smem);
  const Lane w = lane_of();
  // the factors of this wave's eta1 lines, in flight during the stages before
  // the metric; points past the tile read out of range (zero, no access)
  double g[SPW][KQ][NFAC];
  load_tile<SH, P, true, NT>(T, in, img, ne, G1, [&]() {
    const __amdgpu_buffer_rsrc_t rs =
        __builtin_amdgcn_make_buffer_rsrc((void*)fac, (short)0, ne * (NFAC * Q3 * 8), 0x00020000);
#pragma unroll
    for (int s = 0; s < SPW; ++s) {
      const int l = (w.wv + s * NW) * 16 + w.ln;
      const int e = l / Q2, jk = l - e * Q2;
#pragma unroll
      for (int b = 0; b < KQ; ++b) {
        const int i = 4 * b + w.lr;
        const int off = (e < ne && i < Q) ? (e * (NFAC * Q3) + i * Q2 + jk) * 8 : E * (NFAC * Q3 * 8);
#pragma unroll
        for (int c = 0; c < NFAC; ++c) {
          // the Laplacian does without jw: a seventh of the factors, not read (with it,
          // 93750 hexahedra at P = 2 took as long as the Helmholtz action, 60 us)
          const int o = c == 0 && !react ? E * (NFAC * Q3 * 8) : off + c * Q3 * 8;
          g[s][b][c] = __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(rs, o, 0, AUX));
        }
      }
    }
  });
  __syncthreads();
  stage_r<SH, P, NW>(T, w, G1, G2);
  __syncthreads();
  stage_q<SH, P, NW>(T, w, G2, U);
  __syncthreads();
  // eta1 lines: u = stage p, D_0 u, both kept
  double u[SPW][KQ], d0[SPW][KQ];
  int oi[SPW];
  bool ok[SPW];
  constexpr int REM = Q - 4 * (KQ - 1);
#pragma unroll
  for (int s = 0; s < SPW; ++s) {
    const int l0 = (w.wv + s * NW) * 16 + w.ln;
    ok[s] = l0 < nl;
    const int l = ok[s] ? l0 : nl - 1;
    const int e = l / Q2, jk = l - e * Q2, j = jk / Q, k = jk - j * Q;
    oi[s] = e * V::PER + j * D::SJ + k;
    double b[KN];
    load_rows<D::n, D::SI>(T.el + U + oi[s], w, b);
    zero(u[s]);
    contract_km<Q>(T.tab + D::oA, w, b, u[s]);
    if (REM != 4 && w.lr >= REM) u[s][KQ - 1] = 0.0;
    store_rows<Q, D::SI>(T.el + U + oi[s], w, u[s], ok[s]);
    zero(d0[s]);
    contract_mk<Q>(T.tab + D::oD, w, u[s], d0[s]);
  }
  __syncthreads();
  // eta2 lines (e, i, k) and eta3 lines (e, i, j)
  int oj[SPW], ok3[SPW];
#pragma unroll
  for (int s = 0; s < SPW; ++s) {
    const int l0 = (w.wv + s * NW) * 16 + w.ln;
    const int l = ok[s] ? l0 : nl - 1;
    const int e = l / Q2, r = l - e * Q2, i = r / Q, a = r - i * Q;
    oj[s] = e * V::PER + i * D::SI + a;
    ok3[s] = e * V::PER + i * D::SI + a * D::SJ;
    double b[KQ], c[KQ];
    load_rows<Q, D::SJ>(T.el + U + oj[s], w, b);
    zero(c);
    contract_mk<Q>(T.tab + D::oD + Q2, w, b, c);
    store_rows<Q, D::SJ>(T.el + G1 + oj[s], w, c, ok[s]);
    load_rows<Q, 1>(T.el + U + ok3[s], w, b);
    zero(c);
    contract_mk<Q>(T.tab + D::oD + 2 * Q2, w, b, c);
    store_rows<Q, 1>(T.el + G2 + ok3[s], w, c, ok[s]);
  }
  __syncthreads();
  // the metric on the eta1 lines
#pragma unroll
  for (int s = 0; s < SPW; ++s) {
    double d1[KQ], d2[KQ];
    load_rows<Q, D::SI>(T.el + G1 + oi[s], w, d1);
    load_rows<Q, D::SI>(T.el + G2 + oi[s], w, d2);
    double av[ADR ? KQ : 1][3];
    if constexpr (ADR) {
      const int l0 = (w.wv + s * NW) * 16 + w.ln, l = ok[s] ? l0 : nl - 1;
      const int e = l / Q2, jk = l - e * Q2;
#pragma unroll
      for (int b = 0; b < KQ; ++b) {
        const int i0 = 4 * b + w.lr, i = i0 < Q ? i0 : Q - 1;
#pragma unroll
        for (int c = 0; c < 3; ++c) av[b][c] = adv[((e < ne ? e : ne - 1) * 3 + c) * Q3 + i * Q2 + jk];
      }
    }
#pragma unroll
    for (int b = 0; b < KQ; ++b) {
      const double* gg = g[s][b];
      const double x0 = d0[s][b], x1 = d1[b], x2 = d2[b];
      d0[s][b] = gg[1] * x0 + gg[2] * x1 + gg[3] * x2;
      d1[b] = gg[2] * x0 + gg[4] * x1 + gg[5] * x2;
      d2[b] = gg[3] * x0 + gg[5] * x1 + gg[6] * x2;
      if constexpr (ADR)
        u[s][b] = lam * gg[0] * u[s][b] + (av[b][0] * x0 + av[b][1] * x1 + av[b][2] * x2);
      else
        u[s][b] = mul_rn(lam * gg[0], u[s][b]);
    }
    if (REM != 4 && w.lr >= REM) d0[s][KQ - 1] = 0.0;
    store_rows<Q, D::SI>(T.el + G1 + oi[s], w, d1, ok[s]);
    store_rows<Q, D::SI>(T.el + G2 + oi[s], w, d2, ok[s]);
  }
  __syncthreads();
  // D_1^T and D_2^T in place
#pragma unroll
  for (int s = 0; s < SPW; ++s) {
    double b[KQ], c[KQ];
    load_rows<Q, D::SJ>(T.el + G1 + oj[s], w, b);
    zero(c);
    contract_km<Q>(T.tab + D::oD + Q2, w, b, c);
    store_rows<Q, D::SJ>(T.el + G1 + oj[s], w, c, ok[s]);
    load_rows<Q, 1>(T.el + G2 + ok3[s], w, b);
    zero(c);
    contract_km<Q>(T.tab + D::oD + 2 * Q2, w, b, c);
    store_rows<Q, 1>(T.el + G2 + ok3[s], w, c, ok[s]);
  }
  __syncthreads();
  // lambda jw u + D_0^T v_0 + the other two, then stage p^T
#pragma unroll
  for (int s = 0; s < SPW; ++s) {
    double a[KQ], w1[KQ], w2[KQ];
    load_rows<Q, D::SI>(T.el + G1 + oi[s], w, w1);
    load_rows<Q, D::SI>(T.el + G2 + oi[s], w, w2);
    zero(a);
    contract_km<Q>(T.tab + D::oD, w, d0[s], a);
#pragma unroll
    for (int b = 0; b < KQ; ++b) {
      double v = react ? u[s][b] + a[b] : a[b];
      v += w1[b];
      v += w2[b];
      a[b] = v;
    }
    if (REM != 4 && w.lr >= REM) a[KQ - 1] = 0.0;
    double y[KN];
    zero(y);
    contract_mk<Q>(T.tab + D::oA, w, a, y);
    store_rows<D::n, D::SI>(T.el + U + oi[s], w, y, ok[s]);
  }
  __syncthreads();
  stage_qT<SH, P, NW>(T, w, U, G1);
  __syncthreads();
  stage_rT<SH, P, NW>(T, w, G1, G2);
  __syncthreads();
  store_y<SH, P, NT>(T, out, ne, G2);
}

// Launch shape of the Laplacian / Helmholtz tile: elements per work-group, sets
// of eta1 lines per wave, waves.  Whole quarters of a CU's four SIMDs or fewer
// than four waves: five to seven waves put two on one SIMD, whose registers then
// limit the work-groups of the CU (P = 10 with five waves: 201 us against 141).
// Only the orders that run here are given (mf_helm_shape).
template <int P>
struct HelmShape {
  static constexpr int E = P == 2 ? 8 : 1;
  static constexpr int SPW = P == 2 ? 2 : P == 10 ? 3 : 1;
  static constexpr int NW = P == 2 || P == 6 ? 4 : P == 9 ? 8 : 3;
  static_assert(E * (P + 2) * (P + 2) <= 16 * SPW * NW, "every eta1 line needs a place");
};

// the block of work-group blockIdx.x and its first element there; false: none
__device__ __forceinline__ int pick_block(const MfMesh& m, int E, long long& e0) {
  int b = 0;
  while (b + 1 < m.nblk && (long long)blockIdx.x >= m.tile0[b + 1]) ++b;
  e0 = ((long long)blockIdx.x - m.tile0[b]) * E;
  return b;
}

template <int P, bool ADR>
__global__ void __launch_bounds__(64 * HelmShape<P>::NW) k_helm(MfMesh m, double lambda, int react) {
  using S = HelmShape<P>;
  extern __shared__ double smem[];
  long long e0;
  const MfBlock b = m.blk[pick_block(m, S::E, e0)];
  const long long rem = b.n_elem - e0;
  if (rem <= 0) return;
  const int ne = rem < S::E ? (int)rem : S::E;
  constexpr long long Q3 = (P + 2) * (P + 2) * (P + 2);
  const double* fac = b.fac + e0 * (NFAC * Q3);
  const double* av = ADR ? b.aux + e0 * (3 * Q3) : nullptr;
#define T_(SH)                                                                                    \
  helm_tile<SH, P, S::E, S::SPW, S::NW, ADR>(b.img, fac, av, b.in + e0 * num_modes(SH, P),          \
                                             b.out + e0 * num_modes(SH, P), ne, lambda, react != 0, smem)
  switch (b.shape) {
    case HEX: T_(HEX); break;
    case PRISM: T_(PRISM); break;
    case PYR: T_(PYR); break;
    default: T_(TET); break;
  }
#undef T_
}

// LDS of a work-group for a mesh with the shape
template <int P>
constexpr size_t helm_lds(int sh) {
  constexpr int E = HelmShape<P>::E;
  return sh == HEX ? View<HEX, P, E, 3, true>::BYTES : sh == PRISM ? View<PRISM, P, E, 3, true>::BYTES
       : sh == PYR ? View<PYR, P, E, 3, true>::BYTES : View<TET, P, E, 3, true>::BYTES;
}

}  // namespace mf
}  // namespace shp
