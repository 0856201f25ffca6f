// FP64 instantiations of the row pass of the PCG loop (nf_loop.hpp).
#include "nf_loop.hpp"

namespace nf {

// The initial pass (it < 0, which may write the Kbar partials read with the
// default workgroup count) uses the default tile, the loop passes the chosen
// variant; the stopping test of the loop reads the partials of the column pass.
hipError_t launch_row_flux(const Geo& g, void* G0, void* G1, const double* m, const double* r, int it,
                           double* kslot, double tol2, hipStream_t s, float* lo) {
  const int rv = use_rv(g, false, it);
  const int nwg_col = rr_nwg(g, false);
#define L_(N) return flux_var<N, double>(rv, g, (cd*)G0, (cd*)G1, m, r, it, kslot, nwg_col, tol2, lo, (double*)nullptr, s)
  NF_DISPATCH(g.nx, L_)
#undef L_
  return hipErrorInvalidValue;
}
hipError_t launchb_row_flux64(const Geo& g, const FluxArgs* A, int count, int it, double tol2, hipStream_t s) {
  const int rv = use_rv(g, false, it);
  const int nwg_col = rr_nwg(g, false);
#define L_(N) return fluxb_var<N, double>(rv, g, A, count, it, nwg_col, tol2, s)
  NF_DISPATCH(g.nx, L_)
#undef L_
  return hipErrorInvalidValue;
}

}  // namespace nf
