// Diagonal of the elemental Helmholtz operator H = lambda M + L, sum-factorised.
//
// With the collocated form (Sec. 2.2.1, eq. helm1) the derivatives of a mode
// at the points are those of its 1D factors, so for mode m = a(eta1) b(eta2)
// c(eta3)
//   H_mm = sum_q lambda jw phi_m^2 + sum_{d,e} g_de (d_d phi_m)(d_e phi_m),
// and every term is a point field f in {jw, g00, g01, g02, g11, g12, g22}
// contracted with one product of 1D values per direction: u^2, u w or w^2
// (u the factor, w its derivative).  Fields that share the products of the
// directions still to come are added up as soon as they do:
//   eta1, over the distinct eta1 factors a:
//     c0 = uu lambda jw + ww g00, c1 = uw 2 g01, c2 = uu g11   (phase 0)
//     c0 = uw 2 g02, c1 = uu 2 g12, c2 = uu g22                (phase 1)
//   eta2, over the distinct (eta1, eta2) pairs:
//     s0 = uu c0 + uw c1 + ww c2                               (phase 0)
//     s0 = uu c0 + uw c1, s1 = uu c2                           (phase 1)
//   eta3, per mode: uu s0 (phase 0) + uw s0 + ww s1 (phase 1).
//
// The launch reads each factor from HBM once.  15360 elements at P = 6 take 214 us where
// the factors' bytes need 95: eta2 reads 3 Q sums and 3 Q products from LDS for one or
// two results, and three waves a SIMD do not cover it (LDS busy 51 % of the time, 18 in
// bank conflicts, VALU 18 %).  The eta1 stage gives a lane one line (j, k), its fields'
// Q values in registers and the products as scalar operands; two waves share a line's
// factors a, so that an element has six tasks for the wave's 64 lines.  Products are
// tabulated per distinct factor and kept in LDS for eta2 and eta3 over the elements of a
// work-group (formed from global tables at every use, with Q a run-time value, the
// launch took 800 us).
#include <hip/hip_runtime.h>

#include <algorithm>

#include "shp_internal.hpp"

namespace shp {
namespace {

// elements side by side (full waves of lines at low order), threads
template <int Q>
struct DiagShape {
  static constexpr int E = Q == 3 ? 7 : Q == 4 ? 4 : Q == 5 ? 2 : 1;
  static constexpr int NT = Q >= 10 ? 512 : 256;
  static constexpr int NMAX = (Q - 1) * (Q - 1) * (Q - 1);
  static constexpr int MS = (E * NMAX + NT - 1) / NT;  // modes per thread
};

typedef const __attribute__((address_space(4))) double* ctab64;

// c[a] += sum_i T[a][i] v[i] for the eta1 factors a = h, h + 2, ...
template <int Q, bool TWO>
__device__ __forceinline__ void eta1(const double* t0, const double* t1, const double (&v0)[Q], const double (&v1)[Q],
                                     int h, int n1, double* __restrict__ out, int stride) {
  for (int a = h; a < n1; a += 2) {
    const ctab64 x = (ctab64)(t0 + a * Q), y = (ctab64)(t1 + a * Q);
    double s = 0.0;
#pragma unroll
    for (int i = 0; i < Q; ++i) s = fma(x[i], v0[i], s);
    if (TWO) {
#pragma unroll
      for (int i = 0; i < Q; ++i) s = fma(y[i], v1[i], s);
    }
    out[a * stride] = s;
  }
}

template <int Q>
__global__ void __launch_bounds__(DiagShape<Q>::NT) k_helm_diag(DiagMesh m, double lambda) {
  using S = DiagShape<Q>;
  constexpr int E = S::E, NT = S::NT, Q2 = Q * Q, Q3 = Q2 * Q, NL = E * Q2, CH = (NL + 63) / 64;
  extern __shared__ double sm[];
  int bi = 0;
  while (bi + 1 < m.nblk && (long long)blockIdx.x >= m.blk[bi + 1].wg0) ++bi;
  const DiagBlock b = m.blk[bi];
  const int n1 = b.n.n1, n2 = b.n.n2, n3 = b.n.n3, n12 = b.n.n12, NP = b.NP;
  double* T2 = sm;                       // [3][n2][Q]
  double* T3 = T2 + 3 * n2 * Q;          // [3][n3][Q]
  double* S1 = T3 + 3 * n3 * Q;          // [E][3][n1][Q^2]
  double* S2 = S1 + E * 3 * n1 * Q2;     // [E][2][n12][Q]
  const double* T1 = b.dt;               // [3][n1][Q]
  for (int t = threadIdx.x; t < 3 * (n2 + n3) * Q; t += NT) T2[t] = b.dt[3 * n1 * Q + t];
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), ln = threadIdx.x & 63;
  const int* pairs = b.di;
  const int* modes = b.di + n12;
  const long long g0 = ((long long)blockIdx.x - b.wg0) * m.per_wg;
  for (int it = 0; it < m.per_wg; ++it) {
    const long long e0 = (g0 + it) * E;
    const long long rem = b.n_elem - e0;
    if (rem <= 0) break;
    const int ne = rem < E ? (int)rem : E;
    double acc[S::MS];
#pragma unroll
    for (int s = 0; s < S::MS; ++s) acc[s] = 0.0;
#pragma unroll
    for (int ph = 0; ph < 2; ++ph) {
      // eta1: tasks (field sum c, half of the factors h, chunk of 64 lines)
      for (int t = wave; t < 6 * CH; t += NT / 64) {
        const int c = t % 3, h = (t / 3) & 1, l = (t / 6) * 64 + ln;
        const int e = l / Q2, jk = l - e * Q2;
        if (e < ne) {
          const double* f = b.fac + (e0 + e) * (long long)(NFAC * Q3) + jk;
          double* out = S1 + (e * 3 + c) * n1 * Q2 + jk;
          double v0[Q], v1[Q];
          // fields of (phase, c): 0: jw g00 | g01 | g11, 1: g02 | g12 | g22; the
          // off-diagonal ones count twice
          const int fi = ph == 0 ? (c == 0 ? 0 : c == 1 ? 2 : 4) : (c == 0 ? 3 : c == 1 ? 5 : 6);
          const double k0 = ph == 0 ? (c == 0 ? lambda : c == 1 ? 2.0 : 1.0) : (c == 2 ? 1.0 : 2.0);
          const int ty = (ph == 0 && c == 1) || (ph == 1 && c == 0) ? 1 : 0;
#pragma unroll
          for (int i = 0; i < Q; ++i) v0[i] = k0 * f[fi * Q3 + i * Q2];
          if (ph == 0 && c == 0) {
#pragma unroll
            for (int i = 0; i < Q; ++i) v1[i] = f[Q3 + i * Q2];
            eta1<Q, true>(T1, T1 + 2 * n1 * Q, v0, v1, h, n1, out, Q2);
          } else {
            eta1<Q, false>(T1 + ty * n1 * Q, T1, v0, v0, h, n1, out, Q2);
          }
        }
      }
      __syncthreads();
      // eta2 over the pairs
      for (int t = threadIdx.x; t < ne * n12 * Q; t += NT) {
        const int e = E == 1 ? 0 : t / (n12 * Q), r = t - e * (n12 * Q);
        const int p = r / Q, k = r - p * Q, pr = pairs[p];
        const double* c0 = S1 + (e * 3 * n1 + (pr & 65535)) * Q2 + k;
        const double* c1 = c0 + n1 * Q2;
        const double* c2 = c1 + n1 * Q2;
        const double* uu = T2 + (pr >> 16) * Q;
        const double* uw = uu + n2 * Q;
        const double* ww = uw + n2 * Q;
        double s0 = 0.0, s1 = 0.0;
#pragma unroll
        for (int j = 0; j < Q; ++j) {
          s0 = fma(uu[j], c0[j * Q], s0);
          s0 = fma(uw[j], c1[j * Q], s0);
          if (ph == 0)
            s0 = fma(ww[j], c2[j * Q], s0);
          else
            s1 = fma(uu[j], c2[j * Q], s1);
        }
        double* s2 = S2 + (e * 2 * n12 + p) * Q + k;
        s2[0] = s0;
        if (ph == 1) s2[n12 * Q] = s1;
      }
      __syncthreads();
      // eta3 per mode
#pragma unroll
      for (int s = 0; s < S::MS; ++s) {
        const int t = threadIdx.x + s * NT;
        if (t < ne * NP) {
          const int e = E == 1 ? 0 : t / NP, md = modes[t - e * NP];
          const double* s0 = S2 + (e * 2 * n12 + (md & 65535)) * Q;
          const double* s1 = s0 + n12 * Q;
          const double* uu = T3 + (md >> 16) * Q;
          const double* uw = uu + n3 * Q;
          const double* ww = uw + n3 * Q;
#pragma unroll
          for (int k = 0; k < Q; ++k) {
            if (ph == 0) {
              acc[s] = fma(uu[k], s0[k], acc[s]);
            } else {
              acc[s] = fma(uw[k], s0[k], acc[s]);
              acc[s] = fma(ww[k], s1[k], acc[s]);
            }
          }
          if (ph == 1) b.diag[e0 * NP + t] = acc[s];
        }
      }
    }
  }
}

template <int Q>
hipError_t run(DiagMesh& m, double lambda, hipStream_t s) {
  using S = DiagShape<Q>;
  size_t lds = 0;
  long long groups = 0;
  for (int b = 0; b < m.nblk; ++b) {
    const DiagDims& n = m.blk[b].n;
    lds = std::max(lds, sizeof(double) * (size_t)Q * (3 * (n.n2 + n.n3) + S::E * (3 * n.n1 * Q + 2 * n.n12)));
    groups += (m.blk[b].n_elem + S::E - 1) / S::E;
  }
  // the tables of eta2 and eta3 serve several groups once there is enough work
  // for eight work-groups per CU
  m.per_wg = (int)std::min<long long>(8, std::max<long long>(1, groups / (8LL * num_cus())));
  // grid x threads stays below 2^32
  while (groups / m.per_wg >= (1LL << 22)) m.per_wg *= 2;
  long long wg = 0;
  for (int b = 0; b < m.nblk; ++b) {
    m.blk[b].wg0 = wg;
    wg += ((m.blk[b].n_elem + S::E - 1) / S::E + m.per_wg - 1) / m.per_wg;
  }
  if (wg <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_helm_diag<Q>, dim3((unsigned)wg), dim3(S::NT), lds, s, m, lambda);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_helm_diag(DiagMesh& m, int Q, double lambda, hipStream_t s) {
  switch (Q) {
#define C_(q) case q: return run<q>(m, lambda, s);
    C_(3) C_(4) C_(5) C_(6) C_(7) C_(8) C_(9) C_(10) C_(11) C_(12)
#undef C_
  }
  return hipErrorInvalidValue;
}

}  // namespace shp
