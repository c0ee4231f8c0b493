// Launchers of the FP64 matrix-core sum-factorisation (shp_kernels_mf.hpp).
#include <algorithm>

#include "shp_kernels_mf.hpp"

namespace shp {

// Orders whose collocated FP64 actions run on the matrix cores: those whose
// lines fill the blocks of four rows (figures in shp_kernels_mf.hpp).
#define MF_HELM_CASES(X) X(2) X(6) X(9) X(10)

bool mf_helm_shape(int P, int* E, int* NT) {
  switch (P) {
#define C_(p)                        \
  case p:                            \
    *E = mf::HelmShape<p>::E;        \
    *NT = 64 * mf::HelmShape<p>::NW; \
    return true;
    MF_HELM_CASES(C_)
#undef C_
  }
  return false;
}

template <int P>
static hipError_t helm_p(MfMesh& m, double lambda, bool react, hipStream_t s) {
  using S = mf::HelmShape<P>;
  size_t lds = 0;
  long long tiles = 0;
  for (int b = 0; b < m.nblk; ++b) {
    lds = std::max(lds, mf::helm_lds<P>(m.blk[b].shape));
    m.tile0[b] = tiles;
    tiles += (m.blk[b].n_elem + S::E - 1) / S::E;
  }
  if (tiles <= 0) return hipSuccess;
  const dim3 g((unsigned)tiles), t(64 * S::NW);
  if (m.blk[0].aux)
    hipLaunchKernelGGL((mf::k_helm<P, true>), g, t, lds, s, m, lambda, react);
  else
    hipLaunchKernelGGL((mf::k_helm<P, false>), g, t, lds, s, m, lambda, react);
  return hipGetLastError();
}

hipError_t launch_mf_helm(int P, MfMesh& m, double lambda, bool react, hipStream_t s) {
  if (m.nblk < 1 || m.nblk > MF_MAX_BLK) return hipErrorInvalidValue;
  switch (P) {
#define C_(p) case p: return helm_p<p>(m, lambda, react, s);
    MF_HELM_CASES(C_)
#undef C_
  }
  return hipErrorInvalidValue;
}

}  // namespace shp
