// FP32 instantiations of the team over the chip for rows of 128, 256, 512 (nf_chip.hpp).
#include "nf_chip.hpp"

namespace nf {

hipError_t chip_go32_128(const TeamGo& go, hipStream_t s) { return chip_launch<float, 128>(go, s); }
hipError_t chip_go32_256(const TeamGo& go, hipStream_t s) { return chip_launch<float, 256>(go, s); }
hipError_t chip_go32_512(const TeamGo& go, hipStream_t s) { return chip_launch<float, 512>(go, s); }

}  // namespace nf
