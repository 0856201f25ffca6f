// FP32 instantiations of the team over the chip for rows of 200, 400, 800, 1600 (nf_chip.hpp).
#include "nf_chip.hpp"

namespace nf {

hipError_t chip_go32_200(const TeamGo& go, hipStream_t s) { return chip_launch<float, 200>(go, s); }
hipError_t chip_go32_400(const TeamGo& go, hipStream_t s) { return chip_launch<float, 400>(go, s); }
hipError_t chip_go32_800(const TeamGo& go, hipStream_t s) { return chip_launch<float, 800>(go, s); }
hipError_t chip_go32_1600(const TeamGo& go, hipStream_t s) { return chip_launch<float, 1600>(go, s); }

}  // namespace nf
