// FP32 instantiations of the small-grid team with 256 and 512 threads per member (nf_team.hpp).
#include "nf_team.hpp"

namespace nf {

hipError_t team_go32_256(const TeamGo& go, hipStream_t s) { return team_launch<float, 256>(go, s); }
hipError_t team_go32_512(const TeamGo& go, hipStream_t s) { return team_launch<float, 512>(go, s); }

}  // namespace nf
