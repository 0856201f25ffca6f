// FP64 instantiations of the small-grid team with 64 and 128 threads per member (nf_team.hpp).
#include "nf_team.hpp"

namespace nf {

hipError_t team_go64_64(const TeamGo& go, hipStream_t s) { return team_launch<double, 64>(go, s); }
hipError_t team_go64_128(const TeamGo& go, hipStream_t s) { return team_launch<double, 128>(go, s); }

}  // namespace nf
