// FP32 instantiations of the row pass of the PCG loop (nf_loop.hpp).
#include "nf_loop.hpp"

namespace nf {

hipError_t launch_row_flux32(const Geo& g, void* G0, void* G1, const float* m32, const float* r32, float* gd, int it,
                             double tol2, hipStream_t s) {
  const int rv = use_rv(g, true, it);
  const int nwg_col = rr_nwg(g, true);
#define L_(N)                                                                                               \
  return flux_var<N, float>(rv, g, (cx<float>*)G0, (cx<float>*)G1, m32, r32, it, (double*)nullptr, nwg_col, \
                            tol2, (float*)nullptr, gd, s)
  NF_DISPATCH(g.nx, L_)
#undef L_
  return hipErrorInvalidValue;
}
hipError_t launchb_row_flux32(const Geo& g, const FluxArgs* A, int count, int it, double tol2, hipStream_t s) {
  const int rv = use_rv(g, true, it);
  const int nwg_col = rr_nwg(g, true);
#define L_(N) return fluxb_var<N, float>(rv, g, A, count, it, nwg_col, tol2, s)
  NF_DISPATCH(g.nx, L_)
#undef L_
  return hipErrorInvalidValue;
}

}  // namespace nf
