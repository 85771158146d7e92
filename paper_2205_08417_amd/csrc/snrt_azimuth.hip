// Host set-up of the azimuthal-mode scattering operators (sn_azimuth.h): finds the structure in
// an operator on a product rule and packs the transforms and polar matrices in lane order.
#include <algorithm>
#include <cmath>
#include <vector>

#include "snrt_internal.h"

namespace snrt {
namespace {

constexpr double kPi = 3.14159265358979323846;

// An operator counts as invariant if no entry is further than this from the mean over its
// azimuthal shifts, mirror images and (polar fold) reflection, relative to the largest entry of
// its polar pair: far above the FP64 rounding of a kernel evaluated from Omega_q . Omega_p, far
// below the FP32 rounding of the operands.
constexpr double kInvariant = 1e-11;

// Product-rule shape: na consecutive ordinates share each polar node, with one weight.  The
// kernels take up to 16 azimuths or an even count up to 32 (folded), and up to 16 polar nodes or an
// even count up to 32 (folded).
bool product_shape(const snrt_quad& q, int& np, int& na) {
    const int nq = q.nq;
    auto z = [&](int i) { return q.omega_host[(size_t)i * 3 + 2]; };
    na = 1;
    while (na < nq && std::fabs(z(na) - z(0)) <= 1e-12) ++na;
    if (na < 2 || nq % na != 0) return false;
    np = nq / na;
    if (na > 32 || (na > 16 && na % 2 != 0) || np > 32 || (np > 16 && np % 2 != 0)) return false;
    for (int k = 0; k < np; ++k)
        for (int l = 1; l < na; ++l)
            if (q.w_host[(size_t)k * na + l] != q.w_host[(size_t)k * na] ||
                std::fabs(z(k * na + l) - z(k * na)) > 1e-12)
                return false;
    return true;
}

int classes(int na) { return na > 16 ? 2 : 1; }

// Frequency and phase of mode slot m (0..15) of azimuthal class c (two classes: the even and the
// odd frequencies): pairs (2j, 2j + 1) are the cosine and sine of one frequency, except modes 0
// and na / 2 of class 0, which share its first pair.  f < 0: no mode in the slot.
struct Mode {
    int f;
    bool sine;
};
Mode mode_of(int na, int c, int m) {
    const int j = m / 2, s = m & 1, AZ = classes(na);
    const int f = AZ == 1 ? j : 2 * j + c;
    if (f == 0) {
        if (!s) return {0, false};
        return {na % 2 == 0 && (AZ == 1 || na / 2 % 2 == 0) ? na / 2 : -1, false};
    }
    if (2 * f < na) return {f, s == 1};
    // the odd class holds na / 2 where that is odd, as an ordinary pair without a sine
    return {2 * f == na && AZ == 2 && c == 1 && !s ? f : -1, false};
}

// Element l of the orthonormal real Fourier basis over na azimuths.
double basis(int na, const Mode& md, int l) {
    if (md.f < 0) return 0.0;
    const double x = 2.0 * kPi * (double)((md.f * l) % na) / na;
    if (md.f == 0 || 2 * md.f == na) return std::cos(x) / std::sqrt((double)na);
    return std::sqrt(2.0 / na) * (md.sine ? std::sin(x) : std::cos(x));
}

// The polar matrices M[class][pair][which] (h x h in a 16 x 16 frame, row-major) of the
// coefficients a; half: the polar fold's factor 1/2 included.
std::vector<double> polar_matrices(const std::vector<double>& a, int np, int na, bool half) {
    const int AZ = classes(na), MU = np > 16 ? 2 : 1, NC = AZ * MU, h = np / MU;
    std::vector<double> M((size_t)NC * 16 * 256, 0.0);
    std::vector<double> c(na);
    for (int f = 0; f <= na / 2; ++f) {
        for (int d = 0; d < na; ++d) c[d] = std::cos(2.0 * kPi * (double)((f * d) % na) / na);
        auto hat = [&](int k, int k2) {
            double s = 0.0;
            for (int d = 0; d < na; ++d) s += c[d] * a[((size_t)k * np + k2) * na + d];
            return s;
        };
        for (int cls = 0; cls < NC; ++cls)
            for (int j = 0; j < 8; ++j)
                for (int s = 0; s < 2; ++s) {
                    if (mode_of(na, cls % AZ, 2 * j + s).f != f) continue;
                    double* D = &M[((size_t)(cls * 8 + j) * 2 + s) * 256];
                    for (int i = 0; i < h; ++i)
                        for (int i2 = 0; i2 < h; ++i2) {
                            double v = hat(i, i2);
                            if (MU == 2) {
                                const double w = hat(i, np - 1 - i2);
                                v = cls < AZ ? v + w : v - w;
                                if (half) v *= 0.5;
                            }
                            D[i * 16 + i2] = v;
                        }
                }
    }
    return M;
}

// M [n][16][16] in the A-operand order of the kernels: lane (row = lane & 15), step s takes
// column 4 (lane >> 4) + s.
void pack(const double* M, size_t n, bool transpose, float* out) {
    for (size_t b = 0; b < n; ++b)
        for (int lane = 0; lane < 64; ++lane)
            for (int s = 0; s < 4; ++s) {
                const int r = lane & 15, c = 4 * (lane >> 4) + s;
                out[(b * 64 + lane) * 4 + s] =
                    (float)M[b * 256 + (transpose ? c * 16 + r : r * 16 + c)];
            }
}

snrt_status upload_operand(DenseB& B, int np, int na, std::vector<double> a) {
    const int AZ = classes(na), MU = np > 16 ? 2 : 1, NC = AZ * MU, half = na / AZ;
    const std::vector<double> M = polar_matrices(a, np, na, true);
    const size_t nf = (size_t)AZ * 256, nm = (size_t)NC * 16 * 256;
    std::vector<float> host(2 * nf + 2 * nm);
    for (int c = 0; c < AZ; ++c)
        for (int lane = 0; lane < 64; ++lane)
            for (int s = 0; s < 4; ++s) {
                const int lo = lane & 15, hi = lane >> 4;
                const size_t at = (size_t)(c * 64 + lane) * 4 + s;
                if (4 * hi + s < half) host[at] = (float)basis(na, mode_of(na, c, lo), 4 * hi + s);
                if (lo < half) host[nf + at] = (float)basis(na, mode_of(na, c, 4 * s + hi), lo);
            }
    pack(M.data(), (size_t)NC * 16, false, &host[2 * nf]);
    pack(M.data(), (size_t)NC * 16, true, &host[2 * nf + nm]);
    AzOperand op;
    snrt_status s = dev_alloc(&op.base, host.size(), "azimuthal modes");
    if (s == SNRT_OK) s = upload(op.base, host.data(), host.size(), "azimuthal modes: upload");
    if (s != SNRT_OK) {
        dev_free(op.base);
        return s;
    }
    op.np = np;
    op.na = na;
    op.f1 = op.base;
    op.f3 = op.base + nf;
    op.fwd = op.base + 2 * nf;
    op.adj = op.base + 2 * nf + nm;
    B.az = op;
    B.az_a = std::move(a);
    return SNRT_OK;
}

}  // namespace

snrt_status make_azimuth_dense(DenseB& B, const snrt_quad& q, const std::vector<double>& X) {
    int np = 0, na = 0;
    if (!tune().azimuth || !product_shape(q, np, na)) return SNRT_OK;
    const int nq = q.nq;
    // mean over the azimuthal shifts and the mirror image d -> -d (rows of X in order), then the
    // largest distance from it
    const size_t n = (size_t)np * np * na;
    std::vector<double> a(n, 0.0), top((size_t)np * np, 0.0);
    for (int k2 = 0; k2 < np; ++k2)
        for (int l2 = 0; l2 < na; ++l2) {
            const double* x = &X[(size_t)(k2 * na + l2) * nq];
            for (int k = 0; k < np; ++k, x += na) {
                double* m = &a[((size_t)k * np + k2) * na];
                double t = top[(size_t)k * np + k2];
                for (int l = 0; l < na; ++l) {
                    m[l - l2 + (l < l2 ? na : 0)] += x[l];
                    t = std::max(t, std::fabs(x[l]));
                }
                top[(size_t)k * np + k2] = t;
            }
        }
    for (size_t i = 0; i < n; i += na) {
        a[i] /= na;
        for (int d = 1; 2 * d <= na; ++d)
            a[i + d] = a[i + na - d] = 0.5 * (a[i + d] + a[i + na - d]) / na;
    }
    for (int k2 = 0; k2 < np; ++k2)
        for (int l2 = 0; l2 < na; ++l2) {
            const double* x = &X[(size_t)(k2 * na + l2) * nq];
            for (int k = 0; k < np; ++k, x += na) {
                const double* m = &a[((size_t)k * np + k2) * na];
                double far = 0.0;
                for (int l = 0; l < na; ++l) far = std::max(far, std::fabs(x[l] - m[l - l2 + (l < l2 ? na : 0)]));
                if (!(far <= kInvariant * top[(size_t)k * np + k2])) return SNRT_OK;
            }
        }
    if (np > 16) {
        for (int k = 0; k < np; ++k)
            for (int k2 = 0; k2 < np; ++k2) {
                const double* m = &a[((size_t)k * np + k2) * na];
                const double* r = &a[((size_t)(np - 1 - k) * np + np - 1 - k2) * na];
                const double top = std::max(*std::max_element(m, m + na), -*std::min_element(m, m + na));
                for (int d = 0; d < na; ++d)
                    if (!(std::fabs(m[d] - r[d]) <= kInvariant * top)) return SNRT_OK;
            }
    }
    // diag(r) A symmetric, r a function of the polar node: from the forward entries a_{0k}(0)
    std::vector<double> r(np, 1.0);
    for (int k = 1; k < np && !r.empty(); ++k) {
        const double ratio = a[(size_t)k * na] / a[(size_t)k * np * na];
        if (!(ratio > 0.0) || !std::isfinite(ratio)) r.clear();
        else r[k] = ratio;
    }
    B.az_r = std::move(r);
    return upload_operand(B, np, na, std::move(a));
}

snrt_status make_azimuth_moments(DenseB& B, const snrt_quad& q, const double* sigma_l) {
    int np = 0, na = 0;
    if (!tune().azimuth || !product_shape(q, np, na)) return SNRT_OK;
    // the ordinates themselves: equally spaced azimuths from one start, mirrored polar nodes;
    // then sum_j m_j(Omega) sigma_l(j) m_j(Omega') is a function of Omega . Omega'
    const double* om = q.omega_host.data();
    const double tol = 1e-13;
    for (int k = 0; k < np; ++k) {
        const double* o = om + (size_t)k * na * 3;
        if (std::fabs(o[0] * om[1] - o[1] * om[0]) > tol || o[0] * om[0] + o[1] * om[1] <= 0.0)
            return SNRT_OK;
        for (int l = 0; l < na; ++l) {
            const double c = std::cos(2.0 * kPi * l / na), s = std::sin(2.0 * kPi * l / na);
            if (std::fabs(o[3 * l] - (c * o[0] + s * o[1])) > tol ||
                std::fabs(o[3 * l + 1] - (c * o[1] - s * o[0])) > tol)
                return SNRT_OK;
        }
        const size_t r = (size_t)(np - 1 - k) * na;
        if (np > 16 && (std::fabs(om[r * 3 + 2] + o[2]) > tol ||
                        std::fabs(q.w_host[r] - q.w_host[(size_t)k * na]) > tol))
            return SNRT_OK;
    }
    std::vector<double> a((size_t)np * np * na), r(np);
    for (int k = 0; k < np; ++k) {
        r[k] = q.w_host[(size_t)k * na];
        for (int k2 = 0; k2 < np; ++k2)
            for (int d = 0; d < na; ++d) {
                const double* u = om + (size_t)(k * na + d) * 3;
                const double* v = om + (size_t)k2 * na * 3;
                const double mu = u[0] * v[0] + u[1] * v[1] + u[2] * v[2];
                double p0 = 1.0, p1 = mu, s = 0.0;          // Legendre recurrence
                for (int l = 0; l <= B.degree; ++l) {
                    s += sigma_l[l] * (2 * l + 1) / (4.0 * kPi) * p0;
                    const double p2 = ((2 * l + 3) * mu * p1 - (l + 1) * p0) / (l + 2);
                    p0 = p1;
                    p1 = p2;
                }
                a[((size_t)k * np + k2) * na + d] = s * q.w_host[(size_t)k2 * na];
            }
    }
    B.az_r = std::move(r);
    const snrt_status s = upload_operand(B, np, na, std::move(a));
    return s == SNRT_OK ? make_azimuth_implicit(B) : s;
}

snrt_status make_azimuth_implicit(DenseB& B) {
    AzOperand& op = B.az;
    if (op.na == 0 || op.imp_base || B.az_r.empty()) return SNRT_OK;
    const int np = op.np, na = op.na, AZ = classes(na), MU = np > 16 ? 2 : 1, h = np / MU;
    // A is symmetric after the scaling r of the polar nodes; under the polar fold r has to be
    // the same on both halves
    std::vector<double> sr(h);
    for (int k = 0; k < h; ++k) {
        if (MU == 2 && std::fabs(B.az_r[k] - B.az_r[np - 1 - k]) > 1e-10 * B.az_r[k]) return SNRT_OK;
        sr[k] = std::sqrt(B.az_r[k]);
    }
    const std::vector<double> M = polar_matrices(B.az_a, np, na, false);
    const size_t nb = (size_t)AZ * MU * 16;                    // matrices
    double top = 0.0;
    for (double v : M) top = std::max(top, std::fabs(v));
    std::vector<double> E1(nb * 256, 0.0), E2(nb * 256, 0.0), L(nb * 16, 0.0);
    std::vector<double> S((size_t)h * h), lam, zt;
    for (size_t b = 0; b < nb; ++b) {
        const double* D = &M[b * 256];
        for (int i = 0; i < h; ++i)
            for (int j = 0; j < h; ++j) S[(size_t)i * h + j] = sr[i] * D[i * 16 + j] / sr[j];
        for (int i = 0; i < h; ++i)
            for (int j = i + 1; j < h; ++j) {
                double &u = S[(size_t)i * h + j], &v = S[(size_t)j * h + i];
                if (!(std::fabs(u - v) <= 1e-10 * top)) return SNRT_OK;
                u = v = 0.5 * (u + v);
            }
        if (!symmetric_eigen(h, S, lam, zt)) return SNRT_OK;
        for (int j = 0; j < h; ++j) {
            L[b * 16 + j] = lam[j];
            for (int k = 0; k < h; ++k) {
                const double z = zt[(size_t)j * h + k];
                E1[b * 256 + j * 16 + k] = z * sr[k];
                E2[b * 256 + k * 16 + j] = lam[j] * z / sr[k] / MU;
            }
        }
    }
    const size_t nm = nb * 256;
    std::vector<float> host(2 * nm + L.size());
    pack(E1.data(), nb, false, host.data());
    pack(E2.data(), nb, false, &host[nm]);
    for (size_t i = 0; i < L.size(); ++i) host[2 * nm + i] = (float)L[i];
    float* base = nullptr;
    snrt_status s = dev_alloc(&base, host.size(), "azimuthal modes (implicit)");
    if (s == SNRT_OK) s = upload(base, host.data(), host.size(), "azimuthal modes: upload");
    if (s != SNRT_OK) {
        dev_free(base);
        return s;
    }
    op.imp_base = base;
    op.e1 = base;
    op.e2 = base + nm;
    op.lam = base + 2 * nm;
    return SNRT_OK;
}

}  // namespace snrt
