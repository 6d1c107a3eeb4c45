// FP32 instantiations of the Lanczos H.x kernels.
#include "lanczos_rows.hpp"

namespace ftlm {
hipError_t launch_lanczos_f32(const LanczosLaunch& a, hipStream_t st) { return launch_lanczos_rows_any(a, st); }
}  // namespace ftlm
