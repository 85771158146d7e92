// The limited slope of the second-order scheme, used by the gradient kernel (sn_step2.hip) and by
// the fused stage (sn_step2_tile.hip).
#pragma once

#include "sn_step_kernels.h"

namespace snrt {

template <typename T> struct ReconOf;
template <> struct ReconOf<float> { using type = CellRecon32; };
template <> struct ReconOf<double> { using type = CellRecon64; };

namespace {

// the one operand that is a number where the other is not: one instruction, a compare and a
// select take two
__device__ __forceinline__ float larger(float a, float b) { return __builtin_fmaxf(a, b); }
__device__ __forceinline__ float smaller(float a, float b) { return __builtin_fminf(a, b); }
__device__ __forceinline__ double larger(double a, double b) { return __builtin_fmax(a, b); }
__device__ __forceinline__ double smaller(double a, double b) { return __builtin_fmin(a, b); }

template <int LIM, typename T>
__device__ __forceinline__ T limiter_eps2(T vk_k, T inv_area)
{
    if constexpr (LIM != SNRT_LIMITER_VENKATAKRISHNAN) return T(0);
    const T h = vk_k * sqrt(T(1) / inv_area);
    return h * h * h;
}

// a / d where every lane's d lies in [2^-96, 2^96]: the remainder of a * rcp(d) is exact, so the
// corrected quotient is the rounded one but for near ties (4 instructions and a reciprocal where
// the general division takes 10 and one).
__device__ __forceinline__ float ratio_in_range(float a, float d)
{
    const float r = __builtin_amdgcn_rcpf(d);
    const float q = a * r;
    return fmaf(fmaf(-d, q, a), r, q);
}
constexpr uint32_t kRatioLow = (127u - 96u) << 23, kRatioSpan = 192u << 23;
__device__ __forceinline__ uint32_t ratio_place(float d)   // <= kRatioSpan in that range
{
    return __builtin_bit_cast(uint32_t, d) - kRatioLow;
}

// gx, gy *= Psi.  Barth-Jespersen: d1 depends on the sign of d_f alone, and a rounded quotient
// falls with its divisor, so the smallest of d1 / d_f over the faces is that of the largest
// d_f > 0 or of the smallest d_f < 0: two quotients instead of one per face.  (ratio_in_range
// rounds otherwise than the divide near ties only: the limiter may differ by one bit there.)
// The gradient kernel is bound by its instructions (a Heun step of two kernels per stage, 198 450
// cells x 256 ordinates: 741 -> 726 us).
template <int V, int MF, int LIM, typename T>
__device__ __forceinline__ void limit_slope(T (&gx)[V], T (&gy)[V], const T (&u)[V],
                                            const T (&umax)[V], const T (&umin)[V],
                                            const T (&r)[4][2], T eps2)
{
    T lim[V];
    if constexpr (LIM == SNRT_LIMITER_VENKATAKRISHNAN) {
#pragma unroll
        for (int k = 0; k < V; ++k) lim[k] = T(1);
#pragma unroll
        for (int f = 0; f < MF; ++f) {
#pragma unroll
            for (int k = 0; k < V; ++k) {
                const T d2 = gx[k] * r[f][0] + gy[k] * r[f][1];
                const T d1 = d2 > T(0) ? umax[k] - u[k] : umin[k] - u[k];
                T t = T(1);
                // d1 d2 >= 0, so the denominator is at least 2 d2^2 > 0 whenever d2 != 0
                const T d11 = d1 * d1 + eps2;
                if (d2 != T(0)) t = (d11 + T(2) * d2 * d1) / (d11 + T(2) * d2 * d2 + d1 * d2);
                lim[k] = t < lim[k] ? t : lim[k];
            }
        }
    } else {
        T up[V], dn[V];      // largest d_f, largest -d_f
#pragma unroll
        for (int k = 0; k < V; ++k) {
            up[k] = dn[k] = T(0);
#pragma unroll
            for (int f = 0; f < MF; ++f) {
                const T d2 = gx[k] * r[f][0] + gy[k] * r[f][1];
                up[k] = larger(up[k], d2);
                dn[k] = larger(dn[k], -d2);
            }
        }
        const auto general = [&] {
#pragma unroll
            for (int k = 0; k < V; ++k) {
                const T tu = (umax[k] - u[k]) / up[k], td = (u[k] - umin[k]) / dn[k];
                lim[k] = smaller(up[k] > T(0) ? tu : T(1), T(1));
                lim[k] = smaller(dn[k] > T(0) ? td : T(1), lim[k]);
            }
        };
        if constexpr (sizeof(T) == 4) {
            uint32_t place = 0;
#pragma unroll
            for (int k = 0; k < V; ++k) place = max(place, max(ratio_place(up[k]), ratio_place(dn[k])));
            if (__builtin_expect(__ballot(place > kRatioSpan) == 0, 1)) {
#pragma unroll
                for (int k = 0; k < V; ++k)
                    lim[k] = smaller(smaller(ratio_in_range(umax[k] - u[k], up[k]),
                                             ratio_in_range(u[k] - umin[k], dn[k])), T(1));
            } else {
                general();
            }
        } else {
            general();
        }
    }
#pragma unroll
    for (int k = 0; k < V; ++k) {
        gx[k] *= lim[k];
        gy[k] *= lim[k];
    }
}

}  // namespace

}  // namespace snrt
