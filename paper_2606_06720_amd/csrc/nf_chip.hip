// The team over the chip: the split of a grid and the choice of its kernel (nf_chip.hpp).
#include "nf_chip.hpp"

namespace nf {

hipError_t chip_go64_128(const TeamGo& go, hipStream_t s);
hipError_t chip_go64_256(const TeamGo& go, hipStream_t s);
hipError_t chip_go64_512(const TeamGo& go, hipStream_t s);
hipError_t chip_go64_1024(const TeamGo& go, hipStream_t s);
hipError_t chip_go64_2048(const TeamGo& go, hipStream_t s);
hipError_t chip_go64_200(const TeamGo& go, hipStream_t s);
hipError_t chip_go64_400(const TeamGo& go, hipStream_t s);
hipError_t chip_go64_800(const TeamGo& go, hipStream_t s);
hipError_t chip_go64_1600(const TeamGo& go, hipStream_t s);
hipError_t chip_go32_128(const TeamGo& go, hipStream_t s);
hipError_t chip_go32_256(const TeamGo& go, hipStream_t s);
hipError_t chip_go32_512(const TeamGo& go, hipStream_t s);
hipError_t chip_go32_1024(const TeamGo& go, hipStream_t s);
hipError_t chip_go32_2048(const TeamGo& go, hipStream_t s);
hipError_t chip_go32_200(const TeamGo& go, hipStream_t s);
hipError_t chip_go32_400(const TeamGo& go, hipStream_t s);
hipError_t chip_go32_800(const TeamGo& go, hipStream_t s);
hipError_t chip_go32_1600(const TeamGo& go, hipStream_t s);

bool chip_shape(const Geo& g, ChipShape* cs) {
  if (g.nz != 1) return false;
  *cs = chip_split(g.nx, g.ny);
  return cs->G > 0;
}

hipError_t launch_chip(bool f32, const TeamGo& go, hipStream_t s) {
  switch (go.a.g.nx) {
    case 128: return f32 ? chip_go32_128(go, s) : chip_go64_128(go, s);
    case 256: return f32 ? chip_go32_256(go, s) : chip_go64_256(go, s);
    case 512: return f32 ? chip_go32_512(go, s) : chip_go64_512(go, s);
    case 1024: return f32 ? chip_go32_1024(go, s) : chip_go64_1024(go, s);
    case 2048: return f32 ? chip_go32_2048(go, s) : chip_go64_2048(go, s);
    case 200: return f32 ? chip_go32_200(go, s) : chip_go64_200(go, s);
    case 400: return f32 ? chip_go32_400(go, s) : chip_go64_400(go, s);
    case 800: return f32 ? chip_go32_800(go, s) : chip_go64_800(go, s);
    case 1600: return f32 ? chip_go32_1600(go, s) : chip_go64_1600(go, s);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace nf
