// HIP kernels of libshp for gfx950: Laplacian / Helmholtz actions of
// iso-parametric elements with the geometry recomputed in every launch.
//
// An iso-parametric element's map is a polynomial of the solution's degree in
// the element's own basis, x_c = sum_m X_cm phi_m (Sec. 2.1: J is then a
// polynomial; Sec. 4: curvilinear elements with iso-parametric mappings).
// Instead of streaming 7 precomputed FP64 factors per point (56 Q^3 bytes per
// element), a tile reads its 3 N_P coordinate coefficients (24 N_P bytes) and
// rebuilds them in FP64: each coordinate goes through the backward transform
// and the collocated derivatives (the stages of the Helmholtz tile), which
// give d x_c/d eta_d at the points; then per point the determinant, the
// inverse d eta/d x, jw = w |det| / prod (1 - eta_d)^alpha_d (the reference
// weight table wref) and g = jw (d eta/d x)(d eta/d x)^T.  Two forms, chosen by order
// (iso_shape): each coordinate by itself with the factors kept in registers, or the
// coordinates and the solution together.
#pragma once
#include "shp_kernels.hpp"

namespace shp {

// cofactors of d x_c/d eta_d (A, at c*3 + d): d eta_d/d x_i = C[d*3 + i] / det; returns det
__device__ __forceinline__ double iso_cofactors(const double* A, double* C) {
  C[0] = A[4] * A[8] - A[5] * A[7];
  C[1] = A[2] * A[7] - A[1] * A[8];
  C[2] = A[1] * A[5] - A[2] * A[4];
  C[3] = A[5] * A[6] - A[3] * A[8];
  C[4] = A[0] * A[8] - A[2] * A[6];
  C[5] = A[2] * A[3] - A[0] * A[5];
  C[6] = A[3] * A[7] - A[4] * A[6];
  C[7] = A[1] * A[6] - A[0] * A[7];
  C[8] = A[0] * A[4] - A[1] * A[3];
  return A[0] * C[0] + A[1] * C[3] + A[2] * C[6];
}

// d x_c/d eta_d and the reference weight of one point -> its 7 factors f; false when
// the determinant is not positive or a factor not finite.
__device__ __forceinline__ bool iso_factors(const double* A, double w, double* f) {
  double M[9];  // d eta_d / d x_i at d*3 + i
  const double det = iso_cofactors(A, M);
  const double id = 1.0 / det;
#pragma unroll
  for (int c = 0; c < 9; ++c) M[c] *= id;
  const double jw = w * det;
  f[0] = jw;
  f[1] = jw * (M[0] * M[0] + M[1] * M[1] + M[2] * M[2]);
  f[2] = jw * (M[0] * M[3] + M[1] * M[4] + M[2] * M[5]);
  f[3] = jw * (M[0] * M[6] + M[1] * M[7] + M[2] * M[8]);
  f[4] = jw * (M[3] * M[3] + M[4] * M[4] + M[5] * M[5]);
  f[5] = jw * (M[3] * M[6] + M[4] * M[7] + M[5] * M[8]);
  f[6] = jw * (M[6] * M[6] + M[7] * M[7] + M[8] * M[8]);
  bool good = det > 0.0 && isfinite(det);
#pragma unroll
  for (int c = 1; c < NFAC; ++c) good = good && isfinite(f[c]);
  return good;
}

// d x/d eta at the tile's points -> the 7 factors of each point a thread owns
// (slots as in the geometry prefetch); returns false when a determinant is not
// positive or a factor not finite.  Ends with a barrier (LDS free again).
template <int SH, int P, int PPT>
__device__ __forceinline__ bool iso_geometry(const double* __restrict__ xco, const double* __restrict__ wref, long long e0, int ne,
                             const Tile_<SH, P, double>& T, GeoRegs<PPT>& g) {
  using D = Dims<SH, P>;
  constexpr int Q3 = D::Q3, NP = D::NP;
  double J[PPT][9];  // d x_c / d eta_d at c*3 + d
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    for (int t = tid(); t < ne * NP; t += nthr()) {
      const int e = t / NP, m = t - e * NP;
      T.G(e, 0)[m] = xco[((e0 + e) * 3 + c) * NP + m];
    }
    __syncthreads();
    bwd_r<SH, P, false>(T, ne, 0, 1);
    __syncthreads();
    bwd_q<SH, P, false>(T, ne, 1, 2);
    __syncthreads();
    bwd_p_grad0<SH, P>(T, ne);  // U = x_c, G0 = d x_c / d eta_1
    __syncthreads();
    grad12<SH, P, false>(T, ne);  // G1, G2 = d x_c / d eta_2, d eta_3
    __syncthreads();
#pragma unroll
    for (int it = 0; it < PPT; ++it) {
      const int t = tid() + it * nthr();
      if (t < ne * Q3) {
        const int e = t / Q3, pt = t - e * Q3;
        const int lp = lds_pt<SH, P>(pt);
        J[it][c * 3 + 0] = T.G(e, 0)[lp];
        J[it][c * 3 + 1] = T.G(e, 1)[lp];
        J[it][c * 3 + 2] = T.G(e, 2)[lp];
      }
    }
    __syncthreads();
  }
  bool ok = true;
#pragma unroll
  for (int it = 0; it < PPT; ++it) {
    const int t = tid() + it * nthr();
    if (t < ne * Q3) {
      const int pt = t - (t / Q3) * Q3;
      const double* A = J[it];
      const bool good = iso_factors(A, wref[pt], g.v[it]);
      ok = ok && good;
    }
  }
  return ok;
}

// The block of work-group blockIdx.x, as an index into m: every offset is compared, so
// that they load together, in 32 bits (a grid is smaller), so that the scalar unit does
// it and the block's pointers stay in scalar registers.
__device__ __forceinline__ int iso_block(const IsoMesh& m) {
  int i = 0;
#pragma unroll
  for (int j = 1; j < ISO_MAX_BLK; ++j) i += blockIdx.x >= (unsigned)m.wg0[j] ? 1 : 0;
  return __builtin_amdgcn_readfirstlane(i);
}

// the tile of the work-group, whose block is b
template <int P>
__device__ __forceinline__ Tile iso_tile(const BlockStatic& b, const IsoMesh& m, int i) {
  constexpr int E = iso_shape(P).E;
  Tile tl;
  tl.blk = m.blk[i];
  tl.e0 = (blockIdx.x - m.wg0[i]) * E;
  const long long rem = b.n_elem - tl.e0;
  // at run time also where E = 1: as a constant it unrolls the stages of P = 10, 156 VGPRs
  // against 126, one work-group to a CU and not two (2315 hexahedra 285 us against 193)
  tl.ne = rem < E ? (int)rem : E;
  return tl;
}

template <int SH, int P, int OP, int PPT>
__device__ __forceinline__ void iso_helm(const BlockStatic& b, const Tile& tl, const double* in, double* out, double lambda,
                         double* smem) {
  OpArgs a;
  a.tab = b.tab;
  a.itab = b.itab;
  a.fac = nullptr;
  a.dxi = nullptr;
  a.n_elem = b.n_elem;
  a.in = in;
  a.out = out;
  a.in_cs = 0;
  a.out_cs = 0;
  a.lambda = lambda;
  a.E = 0;
  a.nt = 0;
  const Tile_<SH, P> T = make_tile_h<SH, P, double>(smem, b.tab);
  load_tables_helm<SH, P>(a, T);
  GeoRegs<PPT> g;
  iso_geometry<SH, P, PPT>(b.xco, b.wref, tl.e0, tl.ne, T, g);
  helm_tile<SH, P, OP, PPT>(a, tl.e0, tl.ne, T, g, false, []() {});
}

// ---------------------------------------------------------------------------
// one element per work-group, coordinates and solution through the stages together
// ---------------------------------------------------------------------------
// The three coordinates and the solution are the NF = 4 fields (3 for the geometry
// check) of one element and run through the forward stages as four "elements" of the
// tile: a stage has 4 Q^2 line tasks, one per thread, and the work-group waits on 11
// barriers instead of 28.  A coordinate takes three point buffers, G2 in place of U:
// 13 buffers an element against 16 (P = 4, 13.9k elements of mixed shapes: 103.7 us one
// field after the other, 91 with 16 buffers, 87 with 13).  At P = 4 the LDS is busy 61 %
// and the VALU 51 % of the time, 20 waves to a CU; padding the fields against
// bank conflicts changed nothing, 16-byte line accesses cost 4 us.

// the tile of the fields: field c at c * per
template <int SH, int P>
__device__ Tile_<SH, P> make_tile_iso(double* smem, const double* gtab) {
  Tile_<SH, P> T = make_tile_h<SH, P, double>(smem, gtab);
  T.per = 3 * T.bs;
  return T;
}

// eta2 and eta3 collocation derivatives of the fields: G1 = D_1 U and, in place of U,
// D_2 U; of field 3 (the solution, whose U stays) into G2
template <int SH, int P, int NF>
__device__ __forceinline__ void iso_grad12(const Tile_<SH, P>& T) {
  using D = Dims<SH, P>;
  constexpr int Q = D::Q, QP = D::QP;
  const int t = min(tid(), NF * Q * Q - 1);
  const int c = t / (Q * Q), r2 = t - c * (Q * Q), i = r2 / Q, b = r2 - i * Q;
  const double *s1 = T.U(c) + i * Q * QP + b, *s2 = T.U(c) + (i * Q + b) * QP;
  double v1[Q], v2[Q];
#pragma unroll
  for (int l = 0; l < Q; ++l) {
    v1[l] = s1[l * QP];
    v2[l] = s2[l];
  }
  __syncthreads();
  if (tid() < NF * Q * Q) {
    double* g = T.G(c, 1) + i * Q * QP + b;
    ctab_t Dm = launder(T.ct) + D::L.D + 1 * Q * Q;
#pragma unroll
    for (int m = 0; m < Q; ++m) {
      double s = 0.0;
#pragma unroll
      for (int l = 0; l < Q; ++l) s = fma(Dm[m * Q + l], v1[l], s);
      g[m * QP] = s;
    }
    g = (c < 3 ? T.U(c) : T.G(c, 2)) + (i * Q + b) * QP;
    Dm = launder(T.ct) + D::L.D + 2 * Q * Q;
#pragma unroll
    for (int m = 0; m < Q; ++m) {
      double s = 0.0;
#pragma unroll
      for (int l = 0; l < Q; ++l) s = fma(Dm[m * Q + l], v2[l], s);
      g[m] = s;
    }
  }
}

// coefficients -> the fields' collocated derivatives (and the solution's values);
// leaves the threads at a barrier
template <int SH, int P, int NF>
__device__ __forceinline__ void iso_fields(const double* __restrict__ xco, const double* __restrict__ in,
                                           long long e, const Tile_<SH, P>& T) {
  constexpr int NP = Dims<SH, P>::NP, NT = iso_shape(P).NT;
  constexpr int XS = (3 * NP + NT - 1) / NT, US = NF == 4 ? (NP + NT - 1) / NT : 0;
  const double *xs = xco + e * (3 * NP), *us = in + e * NP;
  double xv[XS], uv[US ? US : 1];
  // every slot loads (past the end the last coefficient, written to its own place)
#pragma unroll
  for (int s = 0; s < XS; ++s) xv[s] = xs[min(tid() + s * NT, 3 * NP - 1)];
#pragma unroll
  for (int s = 0; s < US; ++s) uv[s] = us[min(tid() + s * NT, NP - 1)];
#pragma unroll
  for (int s = 0; s < XS; ++s) {
    const int t = min(tid() + s * NT, 3 * NP - 1);
    const int c = t / NP;
    T.U(c)[t - c * NP] = xv[s];
  }
#pragma unroll
  for (int s = 0; s < US; ++s) T.U(3)[min(tid() + s * NT, NP - 1)] = uv[s];
  __syncthreads();
  // modes in U -> F in G0 -> G in G1 -> U, with G0 = D_0 U from the same task
  bwd_r<SH, P, false>(T, NF, -1, 0);
  __syncthreads();
  bwd_q<SH, P, false>(T, NF, 0, 1);
  __syncthreads();
  bwd_p_grad0<SH, P>(T, NF, 1);
  __syncthreads();
  iso_grad12<SH, P, NF>(T);
  __syncthreads();
}

// d x_c/d eta_d of the point at lp -> A[c*3 + d]
template <int SH, int P>
__device__ __forceinline__ void iso_derivs(const Tile_<SH, P>& T, int lp, double* A) {
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    A[c * 3 + 0] = T.G(c, 0)[lp];
    A[c * 3 + 1] = T.G(c, 1)[lp];
    A[c * 3 + 2] = T.U(c)[lp];
  }
}

template <int SH, int P, int OP>
__device__ __forceinline__ void iso_joint(const BlockStatic& b, const Tile& tl, const double* in, double* out,
                                          double lambda, double* smem) {
  using D = Dims<SH, P>;
  constexpr int Q3 = D::Q3, NT = iso_shape(P).NT, PPT = (Q3 + NT - 1) / NT;
  OpArgs a;
  a.tab = b.tab;
  a.itab = b.itab;
  const Tile_<SH, P> T = make_tile_iso<SH, P>(smem, b.tab);
  load_tables_helm<SH, P>(a, T);
  double w[PPT];
#pragma unroll
  for (int it = 0; it < PPT; ++it) w[it] = b.wref[min(tid() + it * NT, Q3 - 1)];
  iso_fields<SH, P, 4>(b.xco, in, tl.e0, T);
  Tile_<SH, P> S = T;  // the solution's buffers alone
  S.el += 3 * T.per;
#pragma unroll
  for (int it = 0; it < PPT; ++it) {
    const int pt = tid() + it * NT;
    if (pt < Q3) {
      const int lp = lds_pt<SH, P>(pt);
      double A[9], C[9], r[3];
      iso_derivs<SH, P>(T, lp, A);
      // jw (d eta/d x)(d eta/d x)^T d u/d eta = (w / det) C C^T d u/d eta: the factors
      // themselves are not formed
      const double det = iso_cofactors(A, C), wd = w[it] / det;
      double *p0 = S.G(0, 0) + lp, *p1 = S.G(0, 1) + lp, *p2 = S.G(0, 2) + lp;
      const double d0 = *p0, d1 = *p1, d2 = *p2;
#pragma unroll
      for (int i = 0; i < 3; ++i) r[i] = wd * (C[i] * d0 + C[3 + i] * d1 + C[6 + i] * d2);
      *p0 = C[0] * r[0] + C[1] * r[1] + C[2] * r[2];
      *p1 = C[3] * r[0] + C[4] * r[1] + C[5] * r[2];
      *p2 = C[6] * r[0] + C[7] * r[1] + C[8] * r[2];
      if (OP == OPK_HELM) {
        double* u = S.U(0) + lp;
        *u = lambda * (w[it] * det) * (*u);
      }
    }
  }
  __syncthreads();
  grad12<SH, P, true>(S, 1);
  __syncthreads();
  grad0T_ipr_p<SH, P>(S, 1, OP == OPK_HELM);
  __syncthreads();
  ipr_q<SH, P, false>(S, 1, -1, 0);
  __syncthreads();
  ipr_r<SH, P, false>(S, 1, 0, 1, false);
  __syncthreads();
  store_modes<false>(S, out, tl.e0, 1, 1);
}

template <int SH, int P>
__device__ __forceinline__ void iso_joint_check(const BlockStatic& b, const Tile& tl, double* smem, int* status) {
  using D = Dims<SH, P>;
  OpArgs a;
  a.tab = b.tab;
  a.itab = b.itab;
  const Tile_<SH, P> T = make_tile_iso<SH, P>(smem, b.tab);
  load_tables_helm<SH, P>(a, T);
  iso_fields<SH, P, 3>(b.xco, b.xco, tl.e0, T);
  bool ok = true;
  for (int pt = tid(); pt < D::Q3; pt += nthr()) {
    double A[9], f[NFAC];
    iso_derivs<SH, P>(T, lds_pt<SH, P>(pt), A);
    ok = iso_factors(A, b.wref[pt], f) && ok;
  }
  if (!ok) atomicOr(status, 1);
}

template <int SH, int P, int OP, int PPT>
__device__ __forceinline__ void iso_action(const BlockStatic& b, const Tile& tl, const double* in, double* out,
                                           double lambda, double* smem) {
  if constexpr (iso_shape(P).joint)
    iso_joint<SH, P, OP>(b, tl, in, out, lambda, smem);
  else
    iso_helm<SH, P, OP, PPT>(b, tl, in, out, lambda, smem);
}

// One field after the other, the kernels keep the register bound of 512 threads, though
// they run on 256 up to P = 3 (41.1 us at either bound, P = 1, 73k elements).
constexpr int iso_bounds(int P) { return iso_shape(P).joint ? iso_shape(P).NT : 512; }

// Laplacian (OP = OPK_LAP) or Helmholtz (OPK_HELM) action of iso-parametric
// blocks of order P, one tile per work-group.
template <int P, int OP, int PPT>
__global__ void __launch_bounds__(iso_bounds(P)) k_helm_iso(const BlockStatic* __restrict__ blocks, IsoMesh m,
                                                              const double* in, double* out, double lambda) {
  extern __shared__ double smem[];
  const int i = iso_block(m);
  const BlockStatic b = blocks[m.blk[i]];
  const Tile tl = iso_tile<P>(b, m, i);
  const double* bin = in + (m.whole ? b.coeff_off : 0);
  double* bout = out + (m.whole ? b.coeff_off : 0);
  switch (b.shape) {
    case HEX: iso_action<HEX, P, OP, PPT>(b, tl, bin, bout, lambda, smem); break;
    case PRISM: iso_action<PRISM, P, OP, PPT>(b, tl, bin, bout, lambda, smem); break;
    case PYR: iso_action<PYR, P, OP, PPT>(b, tl, bin, bout, lambda, smem); break;
    default: iso_action<TET, P, OP, PPT>(b, tl, bin, bout, lambda, smem); break;
  }
}

template <int SH, int P, int PPT>
__device__ __forceinline__ void iso_check_tile(const BlockStatic& b, const Tile& tl, double* smem, int* status) {
  if constexpr (iso_shape(P).joint) return iso_joint_check<SH, P>(b, tl, smem, status);
  OpArgs a;
  a.tab = b.tab;
  a.itab = b.itab;
  const Tile_<SH, P> T = make_tile_h<SH, P, double>(smem, b.tab);
  load_tables_helm<SH, P>(a, T);
  GeoRegs<PPT> g;
  if (!iso_geometry<SH, P, PPT>(b.xco, b.wref, tl.e0, tl.ne, T, g)) atomicOr(status, 1);
}

// The geometry only: status set to 1 when some point has a non-positive determinant or
// a non-finite factor.
template <int P, int PPT>
__global__ void __launch_bounds__(iso_bounds(P)) k_iso_check(const BlockStatic* __restrict__ blocks, IsoMesh m,
                                                               int* __restrict__ status) {
  extern __shared__ double smem[];
  const int i = iso_block(m);
  const BlockStatic b = blocks[m.blk[i]];
  const Tile tl = iso_tile<P>(b, m, i);
  switch (b.shape) {
    case HEX: iso_check_tile<HEX, P, PPT>(b, tl, smem, status); break;
    case PRISM: iso_check_tile<PRISM, P, PPT>(b, tl, smem, status); break;
    case PYR: iso_check_tile<PYR, P, PPT>(b, tl, smem, status); break;
    default: iso_check_tile<TET, P, PPT>(b, tl, smem, status); break;
  }
}

}  // namespace shp
