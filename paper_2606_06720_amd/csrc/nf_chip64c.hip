// FP64 instantiations of the team over the chip for rows of 200, 400, 800, 1600 (nf_chip.hpp).
#include "nf_chip.hpp"

namespace nf {

hipError_t chip_go64_200(const TeamGo& go, hipStream_t s) { return chip_launch<double, 200>(go, s); }
hipError_t chip_go64_400(const TeamGo& go, hipStream_t s) { return chip_launch<double, 400>(go, s); }
hipError_t chip_go64_800(const TeamGo& go, hipStream_t s) { return chip_launch<double, 800>(go, s); }
hipError_t chip_go64_1600(const TeamGo& go, hipStream_t s) { return chip_launch<double, 1600>(go, s); }

}  // namespace nf
