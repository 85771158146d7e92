// The transposed dense step through azimuthal modes (sn_azimuth.h).
#include "sn_azimuth.h"

namespace snrt {
namespace {

template <typename GT, bool DA>
hipError_t launch(const snrt_mesh& m, const snrt_quad& q, const AzModes<double>& op, const StepArgs32& a,
                  const float* psi_n, const float* lam_np1, float* lam_n, GT* g_t, GT* g_s,
                  GT* g_r, const DoseAdj& da, hipStream_t st) {
    if (m.nc == 0) return hipSuccess;
    const az::AzAdjoint e{m.geom32, q.tab32, a, psi_n, lam_np1, lam_n, m.nc, q.nq, da};
    return az::by_shape(op, [&](auto shape) {
        using P = decltype(shape);
        auto go = [&](auto mfc) {
            constexpr int MF = decltype(mfc)::value;
            static const int occ = az::az_resident(az::k_az_adjoint<P, MF, GT, DA>, P::THREADS);
            hipLaunchKernelGGL((az::k_az_adjoint<P, MF, GT, DA>), dim3(az::az_blocks(m, occ)),
                               dim3(P::THREADS), 0, st, op, e, g_t, g_s, g_r);
            return hipGetLastError();
        };
        return m.mf == 4 ? go(std::integral_constant<int, 4>{}) : go(std::integral_constant<int, 3>{});
    });
}

}  // namespace

hipError_t launch_az_adjoint(const snrt_mesh& m, const snrt_quad& q, const AzModes<double>& op,
                             const StepArgs32& a, const float* psi_n, const float* lam_np1,
                             float* lam_n, float* g_t, float* g_s, float* g_r, const DoseAdj& da,
                             hipStream_t st) {
    if (da.g_dose) return hipErrorInvalidValue;
    return launch<float, false>(m, q, op, a, psi_n, lam_np1, lam_n, g_t, g_s, g_r, da, st);
}

hipError_t launch_az_adjoint(const snrt_mesh& m, const snrt_quad& q, const AzModes<double>& op,
                             const StepArgs32& a, const float* psi_n, const float* lam_np1,
                             float* lam_n, double* g_t, double* g_s, double* g_r,
                             const DoseAdj& da, hipStream_t st) {
    if (da.g_dose)
        return launch<double, true>(m, q, op, a, psi_n, lam_np1, lam_n, g_t, g_s, g_r, da, st);
    return launch<double, false>(m, q, op, a, psi_n, lam_np1, lam_n, g_t, g_s, g_r, da, st);
}

}  // namespace snrt
