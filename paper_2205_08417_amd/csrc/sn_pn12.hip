// The matrix-core P_N step of degree 12 (FP32), in a translation unit of its own like degree 13's.
#include "sn_pn_kernels.h"

namespace snrt {

hipError_t launch_pn_mfma32_12(const snrt_mesh& m, const snrt_pn& p, const StepArgs32& a,
                               const float* u, float* out, hipStream_t st) {
    if (p.degree != 12 || !p.wa) return hipErrorInvalidValue;
    return m.mf == 3 ? launch_mfma_t<12, 3>(m, p, a, u, out, st)
                     : launch_mfma_t<12, 4>(m, p, a, u, out, st);
}

}  // namespace snrt
