// The IMEX step with dense or moment-projected scattering through azimuthal modes (sn_azimuth.h).
#include "sn_azimuth.h"

namespace snrt {

namespace {

template <typename R>
hipError_t launch(const snrt_mesh& m, const AzModes<R>& op, const StepEpi& se, hipStream_t st) {
    if (m.nc == 0) return hipSuccess;
    return az::by_shape(op, [&](auto shape) {
        using P = decltype(shape);
        auto go = [&](auto mfc, auto rc) {
            constexpr int MF = decltype(mfc)::value;
            constexpr bool RHO = decltype(rc)::value;
            static const int occ = az::az_resident(az::k_az_imex<P, R, MF, RHO>, P::THREADS);
            hipLaunchKernelGGL((az::k_az_imex<P, R, MF, RHO>), dim3(az::az_blocks(m, occ)),
                               dim3(P::THREADS), 0, st, op, se);
            return hipGetLastError();
        };
        using I3 = std::integral_constant<int, 3>;
        using I4 = std::integral_constant<int, 4>;
        if (m.mf == 4)
            return se.a.inv_rho ? go(I4{}, std::true_type{}) : go(I4{}, std::false_type{});
        return se.a.inv_rho ? go(I3{}, std::true_type{}) : go(I3{}, std::false_type{});
    });
}

}  // namespace

hipError_t launch_az_imex(const snrt_mesh& m, const AzModes<double>& op, const StepEpi& se,
                          hipStream_t st) {
    return launch(m, op, se, st);
}

hipError_t launch_az_imex(const snrt_mesh& m, const AzModes<float>& op, const StepEpi& se,
                          hipStream_t st) {
    return launch(m, op, se, st);
}

}  // namespace snrt
