// FP32 instantiations of the plain H.x kernels.
#include "hv_impl.hpp"

namespace ftlm {
hipError_t launch_hv_f32(const SectorDev& s, const BondTable& B, const HvLaunch& h, hipStream_t st) {
    return launch_hv_typed<float>(s, B, h, st);
}
}  // namespace ftlm
