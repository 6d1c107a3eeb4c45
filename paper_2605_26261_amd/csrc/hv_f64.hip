// FP64 instantiations of the H.x kernels.
#include "hv_impl.hpp"
#include "lanczos_small.hpp"

namespace ftlm {
hipError_t launch_hv_f64(const SectorDev& s, const BondTable& B, const HvLaunch& h, hipStream_t st) {
    return launch_hv_typed<double>(s, B, h, st);
}
hipError_t launch_lanczos_f64(const LanczosLaunch& a, size_t lds, hipStream_t st) {
    const size_t small = small_lanczos_lds(a, lds, hv_slab_lds_bytes(a.n_sites, a.mode));
    return with_mode(a.mode, a.n_sites, [&](auto l, auto m) {
        using L = decltype(l);
        constexpr int MODE = decltype(m)::value;
        if (by_small_lanczos(a, small))
            return with_small_shape(a, [&](auto vb, auto nt) {
                constexpr int VB = decltype(vb)::value;
                return launch_small_lanczos(hv_small_lanczos_kernel<L, MODE, VB, decltype(nt)::value>, VB, a, small, st);
            });
        return with_vb<double>(a.vb, [&](auto vb) {
            return launch_lanczos_one<L, MODE, double, decltype(vb)::value>(a, lds, st);
        });
    });
}
}  // namespace ftlm
