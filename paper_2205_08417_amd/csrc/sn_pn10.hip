// The matrix-core P_N step of degree 10 (FP32), in a translation unit of its own like degree 13's.
#include "sn_pn_kernels.h"

namespace snrt {

hipError_t launch_pn_mfma32_10(const snrt_mesh& m, const snrt_pn& p, const StepArgs32& a,
                               const float* u, float* out, hipStream_t st) {
    if (p.degree != 10 || !p.wa) return hipErrorInvalidValue;
    return m.mf == 3 ? launch_mfma_t<10, 3>(m, p, a, u, out, st)
                     : launch_mfma_t<10, 4>(m, p, a, u, out, st);
}

}  // namespace snrt
