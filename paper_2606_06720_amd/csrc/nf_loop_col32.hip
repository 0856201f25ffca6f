// FP32 instantiations of the column pass of the PCG loop (nf_loop.hpp).
#include "nf_loop.hpp"

namespace nf {

hipError_t launch_col_iter32(const Geo& g, void* M0, void* M1, void* xh, void* rh, void* dh, int it, int max_iter,
                             hipStream_t s) {
  typedef cx<float> V;
  const int cv = use_cv(g, true);
  const int nwg = row_nwg_var(g, use_rv(g, true, 0));
#define L_(N) \
  return iter_var<N, float>(cv, g, (V*)M0, (V*)M1, (V*)xh, (V*)rh, (V*)dh, (V*)nullptr, it, max_iter, nwg, s)
  NF_DISPATCH(g.ny, L_)
#undef L_
  return hipErrorInvalidValue;
}
hipError_t launchb_col_iter32(const Geo& g, const IterArgs* A, int count, int it, int max_iter, hipStream_t s) {
  const int cv = use_cv(g, true);
  const int nwg = row_nwg_var(g, use_rv(g, true, 0));
#define L_(N) return iterb_var<N, float>(cv, g, A, count, it, max_iter, nwg, s)
  NF_DISPATCH(g.ny, L_)
#undef L_
  return hipErrorInvalidValue;
}

}  // namespace nf
