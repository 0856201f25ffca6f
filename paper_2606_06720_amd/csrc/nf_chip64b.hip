// FP64 instantiations of the team over the chip for rows of 1024, 2048 (nf_chip.hpp).
#include "nf_chip.hpp"

namespace nf {

hipError_t chip_go64_1024(const TeamGo& go, hipStream_t s) { return chip_launch<double, 1024>(go, s); }
hipError_t chip_go64_2048(const TeamGo& go, hipStream_t s) { return chip_launch<double, 2048>(go, s); }

}  // namespace nf
