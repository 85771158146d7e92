// Host set-up of the azimuthal-mode scattering operators (sn_azimuth.h): finds the structure in
// an operator on a product rule and packs the transforms and polar matrices in lane order.
#include <algorithm>
#include <cmath>
#include <cstring>
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

// The modes' error is that of FP64 relative to the operator's norm (largest row or column sum), and
// has to stay below FP32 rounding in every element of S, which for psi >= 0 is at least the smallest
// entry times the sum of psi: entries below this share of the norm, zeros above all (a kernel that
// ends at an angle), leave the operator with the general products, whose error is relative to the
// element.  A Henyey-Greenstein kernel's are above 1e-6 up to g = 0.95 on 32 x 32 ordinates.
constexpr double kSmallest = 0x1p-25;

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

// The modes of azimuthal class c are those of half = na / classes azimuths, m = 0 .. half - 1, in a
// symmetric real basis: class 0 (the sums x_l + x_{l+half}, or the azimuths themselves) has
// cas(2 pi l m / half), cas = cos + sin, of frequency m; class 1 (the differences) has
// cas(pi (2 l + 1)(2 m + 1) / (2 half)) of frequency m + 1/2, both in periods per half azimuths.
// Two modes of one frequency (m and half - m, or half - 1 - m) share a polar matrix.
int frequency(int na, int c, int m) { return classes(na) == 1 ? m : 2 * m + c; }   // per na azimuths
double basis(int na, int c, int l, int m) {
    const int half = na / classes(na);
    if (l >= half || m >= half) return 0.0;
    const double x = c == 0 ? 2.0 * kPi * (double)((l * m) % half) / half
                            : kPi * (double)(((2 * l + 1) * (2 * m + 1)) % (4 * half)) / (2.0 * half);
    return (std::cos(x) + std::sin(x)) / std::sqrt((double)na);
}

// The accumulator row at a place, as the kernels' Modes<R>::row(); mode m lies in slot row(m).
template <typename R>
int row(int place) { return sizeof(R) == 8 ? 4 * (place & 3) + (place >> 2) : place; }

// The eight pairs of modes of class c that a wave takes together (modes from half on are empty
// slots).  Pair 0 of class 0: mode 0 and, where half is even, half / 2, each alone in its frequency.
std::vector<int> mode_pairs(int na, int c) {
    const int half = na / classes(na);
    std::vector<int> p, empty;
    for (int m = 15; m >= half; --m) empty.push_back(m);
    auto add = [&](int m, int partner) {
        if (partner < 0) {
            partner = empty.back();
            empty.pop_back();
        }
        p.push_back(m);
        p.push_back(partner);
    };
    if (c == 0) add(0, half % 2 == 0 ? half / 2 : -1);
    for (int m = c == 0 ? 1 : 0; m < half; ++m) {
        const int other = c == 0 ? half - m : half - 1 - m;
        if (m < other) add(m, other);
        else if (m == other && c == 1) add(m, -1);
    }
    while (!empty.empty()) {
        const int m = empty.back();
        empty.pop_back();
        add(m, -1);
    }
    return p;
}

// The polar matrices M[class][pair][which] (h x h in a 16 x 16 frame, row-major) of the
// coefficients a; half: the polar fold's factor 1/2 included.
std::vector<double> polar_matrices(const std::vector<double>& a, int np, int na, bool half) {
    const int AZ = classes(na), MU = np > 16 ? 2 : 1, NC = AZ * MU, h = np / MU;
    std::vector<double> M((size_t)NC * 16 * 256, 0.0);
    std::vector<double> c(na);
    for (int az = 0; az < AZ; ++az) {
        const std::vector<int> pairs = mode_pairs(na, az);
        for (int js = 0; js < 16; ++js) {
            if (pairs[js] >= na / AZ) continue;
            const int f = frequency(na, az, pairs[js]);
            for (int d = 0; d < na; ++d) c[d] = std::cos(2.0 * kPi * (double)((f * d) % na) / na);
            auto hat = [&](int k, int k2) {
                double s = 0.0;
                for (int d = 0; d < na; ++d) s += c[d] * a[((size_t)k * np + k2) * na + d];
                return s;
            };
            for (int mu = 0; mu < MU; ++mu) {
                double* D = &M[((size_t)(mu * AZ + az) * 16 + js) * 256];
                for (int i = 0; i < h; ++i)
                    for (int i2 = 0; i2 < h; ++i2) {
                        double v = hat(i, i2);
                        if (MU == 2) {
                            const double w = hat(i, np - 1 - i2);
                            v = mu == 0 ? v + w : v - w;
                            if (half) v *= 0.5;
                        }
                        D[i * 16 + i2] = v;
                    }
            }
        }
    }
    return M;
}

// M [n][16][16] in the A-operand order of the kernels: lane (row = lane & 15), step s takes
// column row(4 (lane >> 4) + s).
template <typename R>
void pack(const double* M, size_t n, bool transpose, std::vector<R>& out) {
    for (size_t b = 0; b < n; ++b)
        for (int lane = 0; lane < 64; ++lane)
            for (int s = 0; s < 4; ++s) {
                const int r = lane & 15, c = row<R>(4 * (lane >> 4) + s);
                out.push_back((R)M[b * 256 + (transpose ? c * 16 + r : r * 16 + c)]);
            }
}

// The transforms in that order, and the pairs' slots behind them.
constexpr size_t kTransform = 256;                     // elements of a class's transform
template <typename R>
void pack_transforms(int na, std::vector<R>& out) {
    std::vector<int32_t> slots;
    for (int c = 0; c < classes(na); ++c) {
        for (int lane = 0; lane < 64; ++lane)
            for (int s = 0; s < 4; ++s)
                out.push_back((R)basis(na, c, 4 * (lane >> 4) + s, row<R>(lane & 15)));
        for (int m : mode_pairs(na, c)) slots.push_back(row<R>(m));
    }
    const size_t at = out.size();
    out.resize(at + slots.size() * sizeof(int32_t) / sizeof(R));
    std::memcpy(&out[at], slots.data(), slots.size() * sizeof(int32_t));
}

template <typename R>
snrt_status upload_modes(DenseB& B, const std::vector<R>& host, const R** base) {
    R* p = nullptr;
    const snrt_status s = dev_alloc(&p, host.size(), "azimuthal modes");
    if (s != SNRT_OK) return s;
    B.az_mem.push_back(p);
    *base = p;
    return upload(p, host.data(), host.size(), "azimuthal modes: upload");
}

snrt_status upload_operand(DenseB& B, int np, int na, std::vector<double> a) {
    const int AZ = classes(na), NC = AZ * (np > 16 ? 2 : 1);
    const std::vector<double> M = polar_matrices(a, np, na, true);
    std::vector<double> host;
    pack(M.data(), (size_t)NC * 16, false, host);
    pack(M.data(), (size_t)NC * 16, true, host);
    pack_transforms(na, host);
    const double* base = nullptr;
    const snrt_status s = upload_modes(B, host, &base);
    if (s != SNRT_OK) return s;
    AzModes<double>& op = B.az;
    op.np = np;
    op.na = na;
    op.fwd = base;
    op.adj = base + M.size();
    op.f = base + 2 * M.size();
    op.slots = reinterpret_cast<const int32_t*>(op.f + AZ * kTransform);
    B.az_a = std::move(a);
    return SNRT_OK;
}

// The IMEX operands in precision R; E1, E2 [n][16][16], L [n][16].
template <typename R>
snrt_status upload_implicit(DenseB& B, AzModes<R>& op, const std::vector<double>& E1,
                            const std::vector<double>& E2, const std::vector<double>& L) {
    std::vector<R> host;
    pack(E1.data(), L.size() / 16, false, host);
    pack(E2.data(), L.size() / 16, false, host);
    for (size_t i = 0; i < L.size(); ++i) host.push_back((R)L[i / 16 * 16 + row<R>(i % 16)]);
    pack_transforms(B.az.na, host);
    const R* base = nullptr;
    const snrt_status s = upload_modes(B, host, &base);
    if (s != SNRT_OK) return s;
    op.np = B.az.np;
    op.na = B.az.na;
    op.e1 = base;
    op.e2 = base + E1.size();
    op.lam = base + 2 * E1.size();
    op.f = op.lam + L.size();
    op.slots = reinterpret_cast<const int32_t*>(op.f + classes(B.az.na) * kTransform);
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
    double least = INFINITY, norm = 0.0;
    bool positive = true;
    for (int k = 0; k < np; ++k) {
        double row = 0.0, column = 0.0;
        for (int k2 = 0; k2 < np; ++k2)
            for (int d = 0; d < na; ++d) {
                const double v = a[((size_t)k * np + k2) * na + d];
                row += std::fabs(v);
                column += std::fabs(a[((size_t)k2 * np + k) * na + d]);
                least = std::min(least, std::fabs(v));
                positive &= v > 0.0;
            }
        norm = std::max({norm, row, column});
    }
    if (!(least >= kSmallest * norm)) return SNRT_OK;
    B.az.positive = positive;
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
    if (B.az.na == 0 || B.az.e1 || B.az32.e1 || B.az_r.empty()) return SNRT_OK;
    const int np = B.az.np, na = B.az.na, AZ = classes(na), MU = np > 16 ? 2 : 1, h = np / MU;
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
    // the general solve of a 16-bit handle is further off than FP32 modes in every element, that of
    // an FP32 handle is not where the kernel is peaked
    return B.precision == SNRT_FP32 ? upload_implicit(B, B.az, E1, E2, L)
                                    : upload_implicit(B, B.az32, E1, E2, L);
}

}  // namespace snrt
