// FP64 instantiations of the H.x kernels.
#include "hv_impl.hpp"

namespace ftlm {
hipError_t launch_hv_f64(const SectorDev& s, const BondTable& B, const HvLaunch& h, hipStream_t st) {
    return launch_hv_typed<double>(s, B, h, st);
}
hipError_t launch_lanczos_f64(const LanczosLaunch& a, size_t lds, hipStream_t st) {
    return launch_lanczos_typed<double>(a.mode, a.n_sites, a, lds, st);
}
}  // namespace ftlm
