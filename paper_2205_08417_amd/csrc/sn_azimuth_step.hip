// The azimuthal-mode scattering product and the explicit dense step on it (sn_azimuth.h).
#include "sn_azimuth.h"

namespace snrt {

hipError_t launch_az_product(const snrt_mesh& m, const AzModes<double>& op, const double* mats,
                             const float* in, float* out, hipStream_t st) {
    if (m.nc == 0) return hipSuccess;
    return az::by_shape(op, [&](auto shape) {
        using P = decltype(shape);
        static const int occ = az::az_resident(az::k_az_product<P>, P::THREADS);
        hipLaunchKernelGGL((az::k_az_product<P>), dim3(az::az_blocks(m, occ)), dim3(P::THREADS), 0,
                           st, op, mats, in, out, m.nc);
        return hipGetLastError();
    });
}

hipError_t launch_az_step(const snrt_mesh& m, const AzModes<double>& op, const StepEpi& se, double coeff,
                          double* dose, hipStream_t st) {
    if (m.nc == 0) return hipSuccess;
    return az::by_shape(op, [&](auto shape) {
        using P = decltype(shape);
        auto go = [&](auto mfc, auto rc, auto dc) {
            constexpr int MF = decltype(mfc)::value;
            constexpr bool R = decltype(rc)::value, D = decltype(dc)::value;
            static const int occ = az::az_resident(az::k_az_step<P, MF, R, D>, P::THREADS);
            hipLaunchKernelGGL((az::k_az_step<P, MF, R, D>), dim3(az::az_blocks(m, occ)),
                               dim3(P::THREADS), 0, st, op, se, coeff, dose);
            return hipGetLastError();
        };
        auto by_rho = [&](auto mfc, auto dc) {
            return se.a.inv_rho ? go(mfc, std::true_type{}, dc) : go(mfc, std::false_type{}, dc);
        };
        using I3 = std::integral_constant<int, 3>;
        using I4 = std::integral_constant<int, 4>;
        if (m.mf == 4)
            return dose ? by_rho(I4{}, std::true_type{}) : by_rho(I4{}, std::false_type{});
        return dose ? by_rho(I3{}, std::true_type{}) : by_rho(I3{}, std::false_type{});
    });
}

}  // namespace snrt
