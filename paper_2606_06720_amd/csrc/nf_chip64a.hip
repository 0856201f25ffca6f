// FP64 instantiations of the team over the chip for rows of 128, 256, 512 (nf_chip.hpp).
#include "nf_chip.hpp"

namespace nf {

hipError_t chip_go64_128(const TeamGo& go, hipStream_t s) { return chip_launch<double, 128>(go, s); }
hipError_t chip_go64_256(const TeamGo& go, hipStream_t s) { return chip_launch<double, 256>(go, s); }
hipError_t chip_go64_512(const TeamGo& go, hipStream_t s) { return chip_launch<double, 512>(go, s); }

}  // namespace nf
