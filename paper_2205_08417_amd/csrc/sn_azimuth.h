// Scattering through azimuthal modes (kernel templates; instantiated by sn_azimuth_*.hip).
//
// A kernel k(Omega_q . Omega_p) on a product rule (q = k na + l: polar node k, equally spaced
// azimuth l) couples two ordinates through their polar nodes and the difference of their
// azimuths only: S[k,l] = sum_{k',l'} a_{kk'}(l - l') psi[k',l'], a even in the difference.  A
// real Fourier transform over the azimuths makes that one polar matrix per mode m,
// D_m[k][k'] = sum_d a_{kk'}(d) cos(2 pi f_m d / na), instead of one nq x nq matrix:
//     X = F psi,   Y_m = D_m X_m,   S = F Y   (F symmetric),
// 3 * 2 nq * 16 operations per cell after the two foldings below instead of 2 nq * nq (nq =
// 1024: 1/21).  The transforms mix signs, so that their error is relative to a row's norm, not to
// its elements: in FP32 an element of S that a peaked kernel makes small (Henyey-Greenstein 0.95 on
// 512 ordinates, one of them lit) was off by 6e-4 of itself and could be negative.  The modes are
// therefore FP64 (v_mfma_f64_16x16x4_f64), S is rounded to FP32 once, and every element is as good
// as with a product of nq positive terms (1.2e-7 at most in those cases).  The IMEX step of a 16-bit
// handle keeps FP32 modes: its general solve goes through eigenvectors of mixed sign as well, in
// less than FP32.
// Measured against the general products' one-launch steps (BF16x3): 100 352 cells x 1024 ordinates
// 0.305 against 0.653 ms (a copy of the state: 0.131; FP32 modes 0.232), FP32 handles 1.8 ms; 299 538
// x 512 with its dose 0.434 against 0.690 ms (FP32 modes 0.348).  What bounds it: the vector update
// (0.10 ms of issue at 1024 ordinates), the matrix instructions (0.13 ms: FP64 has half the FP32
// rate) and the row traffic overlap only across the waves between two barriers.
//
// Foldings, so that every contraction is at most 16 long (shorter ones are padded with zeros in
// the operands, empty azimuthal slots hold zeros):
//   * azimuth (16 < na <= 32, even): x_l +- x_{l+na/2}; the sums carry the even modes, the
//     differences the odd;
//   * polar (16 < np <= 32, np even, kernel unchanged by mu -> -mu): x_k +- x_{np-1-k}, k < np/2.
// A row is then 1, 2 or 4 classes of 16 polar x 16 azimuthal slots.
//
// One wave owns one cell (16 < np, 32 azimuths: one polar half of a cell, two waves per cell).
// Rows are read, updated and written in memory order, 1 KB per access of a wave; the matrix
// instructions want lane (kk = lane & 15, l4 = lane >> 4) to hold azimuths 4 l4 .. 4 l4 + 3 of
// polar slot kk, whose 16-byte pieces of 16 rows cost the address unit four times the accesses
// (0.35 against 0.24 ms per step at 100 352 x 1024), so rows change order through the wave's own
// corner of LDS.  The waves of eight cells form a block and exchange through LDS:
//   1. azimuthal fold (lane-local), X[k][m] = sum_l x[k][l] F[l][m] per class (4 MFMA), to LDS as
//      [class][polar half][slot of m][cell][k];
//   2. a wave takes two modes of one frequency of a class: their 2 x 8 cells are the 16 columns of
//      Y = D X (they share D), polar fold around it, in place;
//   3. S[l][k] = sum_m F[l][m] Y[k][m] per class, azimuthal unfold: S in the layout of the row.
// The K order of an MFMA and the order of its rows are free, so a lane group's four values are
// adjacent in LDS (Modes<R>), and the symmetric basis makes stages 1 and 3 use the same registers.
// One exchange buffer and a barrier before stage 1's stores: two FP64 buffers would not fit beside
// the corners (1024 ordinates: 66 KB), or would halve the blocks of a CU (512: 33 KB).
#pragma once

#include <cstddef>

#include "sn_step_kernels.h"

namespace snrt {
namespace az {

constexpr int kCells = 8;                    // cells of a block's tile, one wave each

// The precision R of the modes: FP64, or FP32 in the IMEX step of the 16-bit precisions.
// Accumulator rows of a lane group q (lane >> 4), as places 4 q .. 4 q + 3: the rows themselves in
// FP32, rows q, 4 + q, 8 + q, 12 + q in FP64.  row() is its own inverse.
// A cell's 16 polar places in a plane are 16-byte granules, granule g at g ^ turn(cell); planes are
// one granule longer than their eight cells: 8 cells at one g, and 8 planes, cover the banks once.
template <typename R>
struct Modes;
template <>
struct Modes<double> {
    typedef double V4 __attribute__((ext_vector_type(4)));
    typedef double V2 __attribute__((ext_vector_type(2)));
    static constexpr int PLANE = 130;
    __device__ static int row(int place) { return 4 * (place & 3) + (place >> 2); }
    __device__ static V4 mfma(double a, double b, const V4& c) {
        return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
    }
    // offset of a polar place of a cell, and places 4 q .. 4 q + 3
    __device__ static int at(int place, int cell) { return (((place >> 1) ^ cell) << 1) + (place & 1); }
    __device__ __forceinline__ static V4 load(const double* p, int q, int cell) {
        const V2 a = *reinterpret_cast<const V2*>(p + at(4 * q, cell));
        const V2 b = *reinterpret_cast<const V2*>(p + at(4 * q + 2, cell));
        return V4{a[0], a[1], b[0], b[1]};
    }
    __device__ __forceinline__ static void store(double* p, int q, int cell, const V4& v) {
        *reinterpret_cast<V2*>(p + at(4 * q, cell)) = V2{v[0], v[1]};
        *reinterpret_cast<V2*>(p + at(4 * q + 2, cell)) = V2{v[2], v[3]};
    }
};
template <>
struct Modes<float> {
    typedef f32x4 V4;
    static constexpr int PLANE = 132;
    __device__ static int row(int place) { return place; }
    __device__ static V4 mfma(float a, float b, const V4& c) {
        return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
    }
    __device__ static int at(int place, int cell) {
        return (((place >> 2) ^ ((cell ^ (cell >> 2)) & 3)) << 2) + (place & 3);
    }
    __device__ __forceinline__ static V4 load(const float* p, int q, int cell) {
        return *reinterpret_cast<const V4*>(p + at(4 * q, cell));
    }
    __device__ __forceinline__ static void store(float* p, int q, int cell, const V4& v) {
        *reinterpret_cast<V4*>(p + at(4 * q, cell)) = v;
    }
};
template <typename R>
using V4 = typename Modes<R>::V4;
template <typename R>
constexpr int kPlane = Modes<R>::PLANE;      // elements of a mode's plane
template <typename R>
constexpr int kClass = 16 * kPlane<R>;       // and of a class

template <typename R>
__device__ __forceinline__ V4<R> mfma4(const V4<R>& a, const V4<R>& b, V4<R> acc) {
#pragma unroll
    for (int s = 0; s < 4; ++s) acc = Modes<R>::mfma(a[s], b[s], acc);
    return acc;
}

// How a row is cut: AZ azimuthal classes, MU polar halves, WPC waves per cell, SEG segments per
// wave, ITEMS pairs of mode slots per wave in stage 2 (each with MU matrices).
// RV = 0: 16 AZ azimuths, rows in whole 16-byte pieces; else the azimuths do not fill their slots
// and a lane owns RV (even) ordinates of a wave's piece of the row, 64 apart (as in the step
// kernel's striped rows), the last RAGGED of which may lie past its end.
template <int AZ_, int MU_, int RV_ = 0>
struct Shape {
    static constexpr int AZ = AZ_, MU = MU_, RV = RV_;
    static constexpr int WPC = AZ * MU == 4 ? 2 : 1;
    static constexpr int SEG = AZ * MU / WPC;
    static constexpr int WAVES = kCells * WPC;
    static constexpr int THREADS = WAVES * kWave;
    static constexpr int ITEMS = AZ * 8 / WAVES;
    template <typename R>
    static constexpr int LDS = AZ * MU * kClass<R>;  // elements of the exchange
    static constexpr int RAGGED = 2;
    // eight values of every row in a lane (six do not fit either): the registers are full
    static constexpr bool FULL = SEG == 2 && (RV == 0 || RV >= 6);
    // waves per SIMD that the step's registers are bounded to
    static constexpr int STEP_WAVES = SEG == 1 && RV == 2 ? 6 : 4;
    // class of segment i; whether a lane has ordinate v of segment i at all
    static constexpr int az(int i) { return i % AZ; }
    static constexpr bool has(int i, int v) { return RV == 0 || 4 * i + v < RV; }
};

// The place of a wave's lane: its cell of the tile; for the row in memory order the byte offset
// (off) and LDS place (mem) of its ordinates and which exist (those past the end repeat the last
// one and are not stored); for the row in matrix order the LDS granule (mat) of each segment and
// whether the lane's polar slot exists (valid).
template <typename P>
struct Lane {
    static constexpr bool RAG = P::RV != 0;
    static constexpr int N = RAG ? P::RV : P::SEG;               // pieces in memory order
    int wave, lane, l4, kk, cell, mu0, half;
    bool valid, exists_[RAG ? P::RAGGED : P::SEG];
    uint32_t off[RAG ? 1 + P::RAGGED : P::SEG];
    int mem[N], mat[P::SEG];
    template <typename R>
    __device__ __forceinline__ Lane(const AzModes<R>& op) {
        wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
        lane = threadIdx.x & (kWave - 1);
        kk = lane & 15;
        l4 = lane >> 4;
        cell = wave & 7;
        mu0 = P::WPC == 2 ? wave >> 3 : 0;
        const int np = op.np, na = RAG ? op.na : 16 * P::AZ;
        half = na / P::AZ;
        const int h = P::MU == 2 ? np / 2 : np;
        const int rows = P::WPC == 2 ? h : np, k0 = mu0 * h;      // polar rows of this wave
        valid = kk < h;
        const int k = valid ? kk : h - 1;
        off[0] = 4u * (uint32_t)(k0 * na + lane);
#pragma unroll
        for (int n = 0; n < N; ++n) {
            int e = RAG ? n * kWave + lane : n * 256 + 4 * lane;
            const bool in = e < rows * na;
            e = in ? e : rows * na - (RAG ? 1 : 4);
            const int r = e / na, l = e % na;
            if constexpr (RAG) {
                if (n >= P::RV - P::RAGGED) {
                    exists_[n - (P::RV - P::RAGGED)] = in;
                    off[1 + n - (P::RV - P::RAGGED)] = 4u * (uint32_t)(k0 * na + e);
                }
                const int s = l < half ? l : 16 + l - half;       // azimuthal slot
                mem[n] = 4 * granule(r, s >> 2) + (s & 3);
            } else {
                exists_[n] = in;
                off[n] = 4u * (uint32_t)(k0 * na + e);
                mem[n] = granule(r, l >> 2);
            }
        }
#pragma unroll
        for (int i = 0; i < P::SEG; ++i) {
            const int mu = mu0 + i / P::AZ;
            mat[i] = granule((mu ? np - 1 - k : k) - k0, 4 * P::az(i) + l4);
        }
    }
    // 16-byte granule g of a row of 4 AZ granules: xor-ed so that 16 rows at one g, and 16
    // granules in memory order, each cover the banks once
    __device__ __forceinline__ static int granule(int r, int g) {
        constexpr int G = 4 * P::AZ;
        return r * G + (g ^ ((r >> (P::AZ == 2 ? 1 : 2)) & (G - 1)));
    }
    // ordinate v of segment i: whether the lane has it, and its byte offset in a row (striped)
    __device__ __forceinline__ bool exists(int i, int v) const {
        if constexpr (!RAG) return exists_[i];
        const int n = 4 * i + v;
        return P::has(i, v) && (n < P::RV - P::RAGGED || exists_[n - (P::RV - P::RAGGED)]);
    }
    __device__ __forceinline__ uint32_t at(int n) const {
        return n < P::RV - P::RAGGED ? off[0] + 256u * n : off[1 + n - (P::RV - P::RAGGED)];
    }
};

__device__ __forceinline__ f32x4 load4(__amdgpu_buffer_rsrc_t r, uint32_t voff, uint32_t soff) {
    return __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(r, voff, soff, 0));
}

__device__ __forceinline__ void store4(__amdgpu_buffer_rsrc_t r, uint32_t voff, uint32_t soff,
                                       const f32x4& v) {
    __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(i32x4, v), r, voff, soff,
                                           kAuxStream);
}

// Segment i of a row in memory order.
template <typename P>
__device__ __forceinline__ f32x4 load_piece(__amdgpu_buffer_rsrc_t r, const Lane<P>& ln, int i,
                                            uint32_t row) {
    if constexpr (P::RV == 0) {
        return load4(r, ln.off[i], row);
    } else {
        f32x4 x{0, 0, 0, 0};
#pragma unroll
        for (int v = 0; v < 4; ++v)
            if (P::has(i, v))
                x[v] = __builtin_bit_cast(
                    float, __builtin_amdgcn_raw_buffer_load_b32(r, ln.at(4 * i + v), row, 0));
        return x;
    }
}
template <typename P>
__device__ __forceinline__ void store_piece(__amdgpu_buffer_rsrc_t r, const Lane<P>& ln, int i,
                                            uint32_t row, const f32x4& x) {
    if constexpr (P::RV == 0) {
        if (ln.exists(i, 0)) store4(r, ln.off[i], row, x);
    } else {
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const float xv = x[v];
            if (ln.exists(i, v))
                __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(int32_t, xv), r,
                                                      ln.at(4 * i + v), row, kAuxStream);
        }
    }
}
// The same segment of a per-ordinate table in LDS (padded by a wave's width).
template <typename P, typename T>
__device__ __forceinline__ void table_piece(const T* tab, const Lane<P>& ln, int i, T (&x)[4]) {
    if constexpr (P::RV == 0) {
        __builtin_memcpy(x, __builtin_assume_aligned(tab + ln.off[i] / 4, 16), sizeof(x));
    } else {
#pragma unroll
        for (int v = 0; v < 4; ++v)
            x[v] = P::has(i, v) ? tab[ln.off[0] / 4 + kWave * (4 * i + v)] : T(0);
    }
}

// Between the two orders through the wave's LDS corner (LDS accesses of one wave stay in order).
// Azimuthal slots that no ordinate fills hold zeros: cleared at the start, and written as zeros
// even where a cell's modes are not finite.
template <typename P>
__device__ __forceinline__ void clear_corner(const Lane<P>& ln, f32x4* corner) {
    if constexpr (P::RV != 0) {
#pragma unroll
        for (int i = 0; i < P::SEG; ++i) corner[i * kWave + ln.lane] = f32x4{0, 0, 0, 0};
    }
}
template <typename P>
__device__ __forceinline__ void to_matrix_order(f32x4 (&x)[P::SEG], const f32x4 (&p)[P::SEG],
                                                const Lane<P>& ln, f32x4* corner) {
#pragma unroll
    for (int i = 0; i < P::SEG; ++i) {
        if constexpr (P::RV == 0) {
            if (ln.exists(i, 0)) corner[ln.mem[i]] = p[i];
        } else {
#pragma unroll
            for (int v = 0; v < 4; ++v)
                if (ln.exists(i, v)) reinterpret_cast<float*>(corner)[ln.mem[4 * i + v]] = p[i][v];
        }
    }
#pragma unroll
    for (int i = 0; i < P::SEG; ++i) x[i] = corner[ln.mat[i]];
}
template <typename P>
__device__ __forceinline__ void to_memory_order(f32x4 (&x)[P::SEG], const Lane<P>& ln,
                                                f32x4* corner) {
    if constexpr (P::RV != 0) {
#pragma unroll
        for (int i = 0; i < P::SEG; ++i)
#pragma unroll
            for (int v = 0; v < 4; ++v) x[i][v] = 4 * ln.l4 + v < ln.half ? x[i][v] : 0.0f;
    }
    if (ln.valid) {
#pragma unroll
        for (int i = 0; i < P::SEG; ++i) corner[ln.mat[i]] = x[i];
    }
#pragma unroll
    for (int i = 0; i < P::SEG; ++i) {
        if constexpr (P::RV == 0) {
            x[i] = corner[ln.mem[i]];
        } else {
#pragma unroll
            for (int v = 0; v < 4; ++v)
                x[i][v] = P::has(i, v) ? reinterpret_cast<float*>(corner)[ln.mem[4 * i + v]] : 0.0f;
        }
    }
}

// Azimuthal fold of a wave's segments and its inverse: the same sums.
template <typename P, typename V>
__device__ __forceinline__ void fold(V (&x)[P::SEG]) {
    if constexpr (P::AZ == 2) {
#pragma unroll
        for (int i = 0; i < P::SEG; i += 2) {
            const V a = x[i], b = x[i + 1];
            x[i] = a + b;
            x[i + 1] = a - b;
        }
    }
}

// The azimuthal transforms, the same numbers in stages 1 and 3 (the basis is symmetric), in
// registers or, in the kernels whose rows leave no room for them, in LDS.
template <typename P, typename R, bool IN_LDS>
struct Fourier {
    V4<R> f[IN_LDS ? 1 : P::AZ];
    const V4<R>* lds;
    // space: AZ kWave V4 of LDS (IN_LDS; a block barrier follows)
    __device__ __forceinline__ Fourier(const AzModes<R>& op, const Lane<P>& ln, V4<R>* space) {
        const V4<R>* src = reinterpret_cast<const V4<R>*>(op.f);
        if constexpr (IN_LDS) {
            for (int i = threadIdx.x; i < P::AZ * kWave; i += P::THREADS) space[i] = src[i];
            lds = space + ln.lane;
        } else {
#pragma unroll
            for (int a = 0; a < P::AZ; ++a) f[a] = src[a * kWave + ln.lane];
        }
    }
    __device__ __forceinline__ V4<R> at(int a) const {      // of azimuthal class a
        if constexpr (IN_LDS) return lds[a * kWave];
        else return f[a];
    }
};

// The polar matrices of a wave's pairs, and where their two modes lie in the exchange.
template <typename P, typename R>
struct Ops {
    V4<R> d[P::ITEMS][P::MU];
    int at[P::ITEMS];
    __device__ __forceinline__ Ops(const AzModes<R>& op, const R* __restrict__ mats,
                                   const Lane<P>& ln) {
        load(d, mats, ln);
#pragma unroll
        for (int i = 0; i < P::ITEMS; ++i) {
            const int az = az_of(ln, i);
            const int slot = op.slots[(az * 8 + (ln.wave & 7)) * 2 + ((ln.lane >> 3) & 1)];
            at[i] = az * P::MU * kClass<R> + slot * kPlane<R> + (ln.lane & 7) * 16;
        }
    }
    // mats: [class = mu * AZ + az][pair][which][lane] of V4
    __device__ __forceinline__ static void load(V4<R> (&d)[P::ITEMS][P::MU],
                                                const R* __restrict__ mats,
                                                const Lane<P>& ln) {
#pragma unroll
        for (int i = 0; i < P::ITEMS; ++i)
#pragma unroll
            for (int mu = 0; mu < P::MU; ++mu)
                d[i][mu] = reinterpret_cast<const V4<R>*>(
                    mats)[(((mu * P::AZ + az_of(ln, i)) * 8 + (ln.wave & 7)) * 2) * kWave + ln.lane];
    }
    __device__ __forceinline__ static int az_of(const Lane<P>& ln, int i) {
        return P::WPC == 2 ? ln.wave >> 3 : i;
    }
};

// Stage 1: the row segments x of this wave into LDS as modes, once the block has read the modes of
// the tile before.
template <typename P, typename R, bool FL>
__device__ __forceinline__ void to_modes(const f32x4 (&x)[P::SEG], const Fourier<P, R, FL>& fr,
                                         const Lane<P>& ln, R* __restrict__ lds) {
    V4<R> u[P::SEG];
#pragma unroll
    for (int i = 0; i < P::SEG; ++i) u[i] = __builtin_convertvector(x[i], V4<R>);
    fold<P>(u);
#pragma unroll
    for (int i = 0; i < P::SEG; ++i) u[i] = mfma4<R>(u[i], fr.at(P::az(i)), V4<R>{0, 0, 0, 0});
    lds_barrier();
    R* at = lds + ln.kk * kPlane<R> + ln.cell * 16;
#pragma unroll
    for (int i = 0; i < P::SEG; ++i)
        Modes<R>::store(at + (P::az(i) * P::MU + ln.mu0 + i / P::AZ) * kClass<R>, ln.l4, ln.cell,
                        u[i]);
}

// y = A x for a pair of modes.  The pair of modes 0 and half (pair 0 of class 0) has a matrix for
// each: second (LDS) is the other one's, null elsewhere.
template <typename R>
__device__ __forceinline__ V4<R> apply_pair(const V4<R>& d, const V4<R>* second, const V4<R>& x,
                                            int lane) {
    const V4<R> zero{0, 0, 0, 0};
    if (!second) return mfma4<R>(d, x, zero);
    const bool hi = (lane & 8) != 0;
    const V4<R> y = mfma4<R>(d, hi ? zero : x, zero);
    return mfma4<R>(second[lane], hi ? x : zero, y);
}

// Stage 2: f(item, polar class, column values) on this wave's mode pairs, in place.
template <typename P, typename R, typename F>
__device__ __forceinline__ void on_modes(const Ops<P, R>& op, const Lane<P>& ln,
                                         R* __restrict__ lds, F&& f) {
    using M = Modes<R>;
    const int cell = ln.lane & 7;
#pragma unroll
    for (int i = 0; i < P::ITEMS; ++i) {
        R* s = lds + op.at[i];
        const V4<R> a = M::load(s, ln.l4, cell);
        if constexpr (P::MU == 1) {
            M::store(s, ln.l4, cell, f(i, 0, a));
        } else {
            const V4<R> b = M::load(s + kClass<R>, ln.l4, cell);
            const V4<R> u = f(i, 0, a + b), v = f(i, 1, a - b);
            M::store(s, ln.l4, cell, u + v);
            M::store(s + kClass<R>, ln.l4, cell, u - v);
        }
    }
}

// The second matrices of the pair of modes 0 and half into LDS, one per polar class, and where a
// wave finds them (null if its item is another pair).  In LDS rather than read from memory at use:
// loads return in order, so a wait on one in the loop would also wait for the rows in flight.
template <typename P, typename R>
__device__ __forceinline__ void load_second(const R* __restrict__ mats, V4<R>* second) {
    if (threadIdx.x < kWave * P::MU)
        second[threadIdx.x] = reinterpret_cast<const V4<R>*>(
            mats)[((threadIdx.x >> 6) * P::AZ * 8 * 2 + 1) * kWave + (threadIdx.x & (kWave - 1))];
}
template <typename P, typename R, typename V>
__device__ __forceinline__ const V* second_of(const V* second, const Lane<P>& ln, int i, int mu) {
    return (ln.wave & 7) == 0 && Ops<P, R>::az_of(ln, i) == 0 ? second + mu * kWave : nullptr;
}

// Stage 3: the modes of this wave's segments back to azimuths, rounded to FP32.
template <typename P, typename R, bool FL>
__device__ __forceinline__ void from_modes(f32x4 (&x)[P::SEG], const Fourier<P, R, FL>& fr,
                                           const Lane<P>& ln, const R* __restrict__ lds) {
    const R* at = lds + ln.cell * 16 + Modes<R>::at(Modes<R>::row(ln.kk), ln.cell);
    V4<R> s[P::SEG];
#pragma unroll
    for (int i = 0; i < P::SEG; ++i) {
        const int cls = P::az(i) * P::MU + ln.mu0 + i / P::AZ;
        V4<R> y;
#pragma unroll
        for (int st = 0; st < 4; ++st)
            y[st] = at[cls * kClass<R> + Modes<R>::row(4 * ln.l4 + st) * kPlane<R>];
        s[i] = mfma4<R>(fr.at(P::az(i)), y, V4<R>{0, 0, 0, 0});
    }
    fold<P>(s);
#pragma unroll
    for (int i = 0; i < P::SEG; ++i) x[i] = __builtin_convertvector(s[i], f32x4);
}

// The tiles of a block: XCD x owns a contiguous range of tiles (cells in Hilbert order) and its
// blocks sweep it together, as in the step kernel.
struct Tiles {
    int32_t t, end, stride;
    __device__ __forceinline__ Tiles(int32_t ntiles) {
        const int32_t per = (ntiles + kNumXcd - 1) / kNumXcd;
        const int32_t x = (int32_t)(blockIdx.x % kNumXcd);
        t = x * per + (int32_t)(blockIdx.x / kNumXcd);
        end = x * per + per < ntiles ? x * per + per : ntiles;
        stride = (int32_t)(gridDim.x / kNumXcd);
    }
};

// The cell's data besides its rows.  All of it comes through vector loads, one word per lane, and
// is read back with readlane: the words of the geometry record (rec, two tiles ahead, for the
// neighbour list), then one tile ahead (mat) in lanes 0..3 sigma_t, sigma_s, source and 1/rho of
// the cell, in lanes 4.. the neighbours' 1/rho, in lanes 8, 9 the dose to add to.  Scalar loads
// would share their wait counter with the LDS exchange, which would then wait for memory.
struct CellWords {
    const float* base;
    bool nbr, dose;
    __device__ __forceinline__ CellWords(int lane, const StepArgs32& a, const float* src_arr,
                                         const double* dose_) {
        nbr = lane >= 4 && lane < 8 && a.inv_rho;
        dose = (lane == 8 || lane == 9) && dose_;
        base = lane == 1 ? a.sigma_s : lane == 2 ? src_arr : a.sigma_t;
        if ((lane == 3 && a.inv_rho) || nbr) base = a.inv_rho;
        if (dose) base = reinterpret_cast<const float*>(dose_) + (lane - 8);
    }
    __device__ __forceinline__ static float record(const CellGeom32* __restrict__ geom, int32_t c,
                                                   int lane) {
        return reinterpret_cast<const float*>(geom + c)[lane & 15];
    }
    template <int MF>
    __device__ __forceinline__ float material(float rec, int32_t c, int lane) const {
        int32_t i = c;
        if (nbr) {
#pragma unroll
            for (int f = 0; f < MF; ++f) {
                const int32_t j = word(rec, f);
                if (lane == 4 + f && j >= 0) i = j;
            }
        }
        return base[dose ? 2 * (int64_t)i : (int64_t)i];
    }
    __device__ __forceinline__ static int32_t word(float r, int l) {
        return __builtin_amdgcn_readlane(__builtin_bit_cast(int32_t, r), l);
    }
    __device__ __forceinline__ static float value(float r, int l) {
        return __builtin_bit_cast(float, word(r, l));
    }
};

// The update's coefficients, formed as fwd_load_stage forms them.
template <int MF>
struct CellData {
    float ghost[MF], nx[MF], ny[MF];
    float irho, cabs, cflux, cscat, srcv;
    bool scaled;      // some ghost scale may differ from 1 (densities, boundary faces)
    template <bool RHO>
    __device__ __forceinline__ void form(float rec, float mat, const StepArgs32& a,
                                         const FwdCtx<float>& x) {
        using W = CellWords;
        irho = RHO ? W::value(mat, 3) : 1.0f;
        const float bscale = x.dirichlet ? x.inflow_scale : (x.neumann ? irho : 0.0f);
        scaled = RHO;
#pragma unroll
        for (int f = 0; f < MF; ++f) {
            scaled |= W::word(rec, f) < 0;
            ghost[f] = W::word(rec, f) < 0 ? bscale : RHO ? W::value(mat, 4 + f) : 1.0f;
            nx[f] = W::value(rec, 4 + 2 * f);
            ny[f] = W::value(rec, 5 + 2 * f);
        }
        cabs = a.dt * a.alpha_t * W::value(mat, 0);
        cflux = a.dt * W::value(rec, 12);
        cscat = a.dt * a.alpha_s * W::value(mat, 1);
        srcv = W::value(mat, 2);
    }
};
static_assert(offsetof(CellGeom32, n) == 16 && offsetof(CellGeom32, inv_area) == 48, "record words");

// Per-ordinate tables in LDS, padded by a wave's width: the two direction rows, and for striped
// rows with a dose the FP64 weights (whole pieces have one weight per segment, in registers).
template <typename P>
constexpr int kTable = P::AZ * P::MU * 256 + (P::RV ? kWave : 0);
template <typename P, typename T>
__device__ __forceinline__ void load_table(const T* __restrict__ tab, int nq, T* dst) {
    for (int i = threadIdx.x; i < nq; i += P::THREADS) dst[i] = tab[i];
}
template <typename P>
__device__ __forceinline__ void load_dirs(const float* __restrict__ tab, int nq, float* dst) {
    load_table<P>(tab, nq, dst);
    load_table<P>(tab + nq, nq, dst + kTable<P>);
}
// sum over a lane's ordinates of w p, FP64
template <typename P>
__device__ __forceinline__ double weighted(const f32x4 (&p)[P::SEG], const double* wd,
                                           const Lane<P>& ln) {
    double sd = 0.0;
#pragma unroll
    for (int i = 0; i < P::SEG; ++i) {
        if constexpr (P::RV == 0) {
            sd += wd[i] *
                  (((double)p[i][0] + (double)p[i][1]) + ((double)p[i][2] + (double)p[i][3]));
        } else {
            double w[4];
            table_piece<P>(wd, ln, i, w);
#pragma unroll
            for (int v = 0; v < 4; ++v)
                if (ln.exists(i, v)) sd += w[v] * (double)p[i][v];
        }
    }
    return sd;
}

// Sum of a double over the wave, the same in every lane: DPP swaps inside rows of 16, the row
// sums through scalars (no LDS traffic, which the exchange needs).
template <int CTRL>
__device__ __forceinline__ double dpp_partner64(double v) {
    const uint64_t b = __builtin_bit_cast(uint64_t, v);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)b, CTRL, 0xF, 0xF, false);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(b >> 32), CTRL, 0xF, 0xF, false);
    return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}
__device__ __forceinline__ double lane64(double v, int l) {
    const uint64_t b = __builtin_bit_cast(uint64_t, v);
    return __builtin_bit_cast(
        double, ((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(b >> 32), l) << 32) |
                    (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)b, l));
}
__device__ __forceinline__ double wave_sum64(double v) {
    v += dpp_partner64<0xB1>(v);
    v += dpp_partner64<0x4E>(v);
    v += dpp_partner64<0x141>(v);
    v += dpp_partner64<0x140>(v);
    return (lane64(v, 0) + lane64(v, 16)) + (lane64(v, 32) + lane64(v, 48));
}

// The upwind candidate across a face to neighbour j of cell c (the step kernel's branch-free rule).
template <typename P>
__device__ __forceinline__ f32x4 load_face(int32_t j, int32_t c, const Lane<P>& ln, int i,
                                           const FwdCtx<float>& x) {
    const bool bnd = j < 0;
    const int32_t bidx = x.dirichlet ? -1 - j : c;
    return load_piece<P>(bnd && x.dirichlet ? x.inflow : x.psi, ln, i,
                         (uint32_t)(bnd ? bidx : j) * x.row_bytes);
}

// The upwind sum over the faces for one segment, in the explicit FMAs of fwd_compute; up: the
// upwind candidates times their ghost scales.
template <typename P, int MF, bool RHO>
__device__ __forceinline__ f32x4 flux4(int i, const f32x4& p, float irho, const float (&nx)[MF],
                                       const float (&ny)[MF], const f32x4 (&up)[MF],
                                       const float (&ox)[4], const float (&oy)[4]) {
    f32x4 acc{0, 0, 0, 0};
#pragma unroll
    for (int f = 0; f < MF; ++f)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            if (!P::has(i, v)) continue;
            const float u = RHO ? p[v] * irho : p[v];
            const float s = __builtin_fmaf(nx[f], ox[v], ny[f] * oy[v]);
            acc[v] = __builtin_fmaf(s, s > 0.0f ? u : up[f][v], acc[v]);
        }
    return acc;
}

__device__ __forceinline__ FwdCtx<float> make_ctx(const StepArgs32& a, const float* psi_in,
                                                  float* psi_out, int64_t nc, int32_t nq,
                                                  uint32_t nbf) {
    FwdCtx<float> cx;
    cx.row_bytes = (uint32_t)nq * (uint32_t)sizeof(float);
    const uint32_t state_bytes = (uint32_t)nc * cx.row_bytes;
    cx.psi = make_rsrc(psi_in, state_bytes);
    cx.out = make_rsrc(psi_out, state_bytes);
    cx.inflow = make_rsrc(a.inflow ? a.inflow : psi_in, a.inflow ? nbf * cx.row_bytes : 0u);
    cx.S = make_rsrc(psi_in, 0u);
    cx.src_arr = a.source ? a.source : a.sigma_t;
    cx.src_mul = a.source ? a.dt : 0.0f;
    cx.inflow_scale = a.inflow_scale;
    cx.dirichlet = a.inflow != nullptr && !a.neumann;
    cx.neumann = a.neumann != 0;
    cx.dpart = nullptr;
    return cx;
}

// A wave's cell in tile t, clamped to the mesh (a clamped cell is computed and not stored).
struct Cell {
    int32_t c;
    bool real;
    __device__ __forceinline__ Cell(int32_t t, int cell, int64_t nc) {
        const int64_t c0 = (int64_t)t * kCells + cell;
        real = c0 < nc;
        c = uniform_cell((int32_t)(real ? c0 : nc - 1));
    }
};

// A row with an infinity: the modes mix signs, so that its S comes out as NaN, where a product with
// a kernel of positive entries is infinite.  S of such a row is the plain sum of the row (NaN if it
// holds a NaN or both infinities).  x: S in memory order; some of a wave's first values are NaN then.
template <typename P>
__device__ __forceinline__ void keep_infinities(f32x4 (&x)[P::SEG], const AzModes<double>& op,
                                                __amdgpu_buffer_rsrc_t r, uint32_t row, int lane) {
    if (!op.positive || __builtin_amdgcn_ballot_w64(x[0][0] != x[0][0]) == 0) return;
    double t = 0.0;
    for (int q = lane; q < op.np * op.na; q += kWave)
        t += (double)__builtin_bit_cast(
            float, __builtin_amdgcn_raw_buffer_load_b32(r, 4u * (uint32_t)q, row, 0));
    const float sum = (float)wave_sum64(t);
#pragma unroll
    for (int i = 0; i < P::SEG; ++i) x[i] = f32x4{sum, sum, sum, sum};
}

// ------------------------------------------------------------------------------ the product

// S = Psi B (or Lambda B^T with the transposed matrices): [nc][nq] -> [nc][nq].
template <typename P>
__global__ __launch_bounds__(P::THREADS, 4) void k_az_product(AzModes<double> opd,
                                                              const double* __restrict__ mats,
                                                              const float* __restrict__ in,
                                                              float* __restrict__ out, int64_t nc)
{
    using R = double;
    __shared__ __attribute__((aligned(16))) R lds[P::template LDS<R>];
    __shared__ V4<R> second[P::MU * kWave];
    __shared__ f32x4 rows[P::WAVES][P::SEG * kWave];
    const Lane<P> ln(opd);
    const Ops<P, R> op(opd, mats, ln);
    const Fourier<P, R, false> fr(opd, ln, nullptr);
    load_second<P, R>(mats, second);
    clear_corner<P>(ln, rows[ln.wave]);
    const uint32_t row_bytes = (uint32_t)(opd.np * opd.na) * 4u;
    const auto rin = make_rsrc(in, (uint32_t)nc * row_bytes);
    const auto rout = make_rsrc(out, (uint32_t)nc * row_bytes);
    Tiles tl((int32_t)((nc + kCells - 1) / kCells));
    if (tl.t >= tl.end) return;
    f32x4 nx[P::SEG];
    auto fetch = [&](int32_t t) {
        const Cell c(t < tl.end ? t : tl.end - 1, ln.cell, nc);
#pragma unroll
        for (int i = 0; i < P::SEG; ++i)
            nx[i] = load_piece<P>(rin, ln, i, (uint32_t)c.c * row_bytes);
    };
    fetch(tl.t);
    for (; tl.t < tl.end; tl.t += tl.stride) {
        const Cell c(tl.t, ln.cell, nc);
        f32x4 x[P::SEG];
        to_matrix_order<P>(x, nx, ln, rows[ln.wave]);
        fetch(tl.t + tl.stride);
        to_modes(x, fr, ln, lds);
        lds_barrier();
        on_modes(op, ln, lds, [&](int i, int mu, const V4<R>& v) {
            return apply_pair<R>(op.d[i][mu], second_of<P, R>(second, ln, i, mu), v, ln.lane);
        });
        lds_barrier();
        from_modes(x, fr, ln, lds);
        to_memory_order<P>(x, ln, rows[ln.wave]);
        keep_infinities<P>(x, opd, rin, (uint32_t)c.c * row_bytes, ln.lane);
#pragma unroll
        for (int i = 0; i < P::SEG; ++i)
            if (c.real) store_piece<P>(rout, ln, i, (uint32_t)c.c * row_bytes, x[i]);
    }
}

// ------------------------------------------------------------------------ the explicit step

// The explicit dense step (and its dose) in one pass over the state: the wave's own row feeds the
// modes and stays in registers for the update.  The next tile's own row is fetched at the start
// of a tile, its neighbour rows segment by segment into the registers the update has just used
// (in flight during the next tile's exchange), cell data one tile ahead, neighbour lists two.  The update is fwd_compute's, in the same
// explicit FMAs: the state equals the product followed by the step kernel bit for bit.  A wave that
// is in the exchange has priority over one that updates, whose vector work fills the gaps
// (100 352 x 1024: 0.250 -> 0.231 ms; 299 538 x 512: 0.368 -> 0.350).
template <typename P, int MF, bool RHO, bool DOSE>
__global__ __launch_bounds__(P::THREADS, P::STEP_WAVES) void k_az_step(AzModes<double> opd, StepEpi se, double coeff,
                                                           double* __restrict__ dose)
{
    constexpr int SEG = P::SEG;
    using R = double;
    __shared__ __attribute__((aligned(16))) R lds[P::template LDS<R>];
    __shared__ V4<R> ftab[P::FULL ? P::AZ * kWave : 1];
    __shared__ double dsum[DOSE && P::WPC == 2 ? kCells : 1];
    __shared__ V4<R> second[P::MU * kWave];
    __shared__ __attribute__((aligned(16))) float dirs[2 * kTable<P>];
    __shared__ f32x4 rows[P::WAVES][SEG * kWave];
    const Lane<P> ln(opd);
    const Ops<P, R> op(opd, opd.fwd, ln);
    const Fourier<P, R, P::FULL> fr(opd, ln, ftab);
    load_second<P, R>(opd.fwd, second);
    load_dirs<P>(se.tab, se.nq, dirs);
    clear_corner<P>(ln, rows[ln.wave]);
    const FwdCtx<float> cx = make_ctx(se.a, se.psi_in, se.psi_out, se.nc, se.nq, se.nbf);
    const CellWords words(ln.lane, se.a, cx.src_arr, DOSE ? dose : nullptr);
    __shared__ double wtab[DOSE && P::RV ? kTable<P> : 1];
    double wd[DOSE ? SEG : 1];                                   // one weight per polar node
    if constexpr (DOSE && P::RV != 0) {
        load_table<P>(se.wq, se.nq, wtab);
    } else if constexpr (DOSE) {
#pragma unroll
        for (int i = 0; i < SEG; ++i) wd[i] = ln.exists(i, 0) ? se.wq[ln.off[i] / 4] : 0.0;
    }
    Tiles tl((int32_t)((se.nc + kCells - 1) / kCells));
    if (tl.t >= tl.end) return;
    auto cell_of = [&](int32_t t) { return Cell(t < tl.end ? t : tl.end - 1, ln.cell, se.nc); };
    auto record = [&](int32_t t) { return CellWords::record(se.geom, cell_of(t).c, ln.lane); };
    auto own = [&](f32x4 (&p)[SEG], int32_t t) {
        const uint32_t row = (uint32_t)cell_of(t).c * cx.row_bytes;
#pragma unroll
        for (int i = 0; i < SEG; ++i) p[i] = load_piece<P>(cx.psi, ln, i, row);
    };
    f32x4 p[SEG], pn[SEG], up[SEG][MF];
    float rec = record(tl.t), mat = words.template material<MF>(rec, cell_of(tl.t).c, ln.lane);
    own(p, tl.t);
#pragma unroll
    for (int i = 0; i < SEG; ++i)
#pragma unroll
        for (int f = 0; f < MF; ++f)
            up[i][f] = load_face<P>(CellWords::word(rec, f), cell_of(tl.t).c, ln, i, cx);
    float recn = record(tl.t + tl.stride);
    __syncthreads();                       // second, dirs
    for (;;) {
        const Cell c = cell_of(tl.t), cn = cell_of(tl.t + tl.stride);
        f32x4 x[SEG];
        __builtin_amdgcn_s_setprio(2);
        to_matrix_order<P>(x, p, ln, rows[ln.wave]);
        to_modes(x, fr, ln, lds);
        const float matn = words.template material<MF>(recn, cn.c, ln.lane);
        own(pn, tl.t + tl.stride);
        const float recn2 = record(tl.t + 2 * tl.stride);
        lds_barrier();
        on_modes(op, ln, lds, [&](int i, int mu, const V4<R>& v) {
            return apply_pair<R>(op.d[i][mu], second_of<P, R>(second, ln, i, mu), v, ln.lane);
        });
        double sd = 0.0;
        if constexpr (DOSE) {
            sd = weighted<P>(p, P::RV ? wtab : wd, ln);
            sd = wave_sum64(sd);
            if (P::WPC == 2 && ln.mu0 == 1 && ln.lane == 0) dsum[ln.cell] = sd;
        }
        lds_barrier();
        from_modes(x, fr, ln, lds);
        to_memory_order<P>(x, ln, rows[ln.wave]);
        keep_infinities<P>(x, opd, cx.psi, (uint32_t)c.c * cx.row_bytes, ln.lane);
        __builtin_amdgcn_s_setprio(0);
        CellData<MF> cd;
        cd.template form<RHO>(rec, mat, se.a, cx);
        if constexpr (DOSE) {
            const uint64_t d0 = ((uint64_t)(uint32_t)CellWords::word(mat, 9) << 32) |
                                (uint32_t)CellWords::word(mat, 8);
            if (ln.mu0 == 0 && ln.lane == 0 && c.real) {
                if (P::WPC == 2) sd += dsum[ln.cell];
                dose[c.c] = __builtin_bit_cast(double, d0) +
                            coeff * (RHO ? (double)cd.irho : 1.0) * sd;
            }
        }
        const uint32_t row = (uint32_t)c.c * cx.row_bytes;
#pragma unroll
        for (int i = 0; i < SEG; ++i) {
            float ox[4], oy[4];
            table_piece<P>(dirs, ln, i, ox);
            table_piece<P>(dirs + kTable<P>, ln, i, oy);
            if (cd.scaled) {
#pragma unroll
                for (int f = 0; f < MF; ++f) up[i][f] *= cd.ghost[f];
            }
            const f32x4 acc = flux4<P, MF, RHO>(i, p[i], cd.irho, cd.nx, cd.ny, up[i], ox, oy);
            f32x4 o;
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                if (!P::has(i, v)) continue;
                const float e =
                    __builtin_fmaf(-cd.cflux, acc[v], __builtin_fmaf(-p[i][v], cd.cabs, p[i][v]));
                o[v] = __builtin_fmaf(cx.src_mul, cd.srcv, __builtin_fmaf(cd.cscat, x[i][v], e));
            }
            if (c.real) store_piece<P>(cx.out, ln, i, row, o);
#pragma unroll
            for (int f = 0; f < MF; ++f)
                up[i][f] = load_face<P>(CellWords::word(recn, f), cn.c, ln, i, cx);
        }
        tl.t += tl.stride;
        if (tl.t >= tl.end) break;
#pragma unroll
        for (int i = 0; i < SEG; ++i) p[i] = pn[i];
        rec = recn;
        recn = recn2;
        mat = matn;
    }
}

// ---------------------------------------------------------------------- the transposed step

// The transposed dense step in one pass: G = Lambda B^T through the modes (transposed polar
// matrices), then adj_compute's update in the same explicit FMAs (lam_n equals the product followed
// by the transposed-step kernel bit for bit).  A wave holds its whole row (or polar half), so the
// gradient sums finish here: where two waves share a cell, their sums meet in LDS and are added
// after the next tile's first barrier.
struct AzAdjoint {
    const CellGeom32* geom;
    const float* tab;
    StepArgs32 a;
    const float *psi_n, *lam_np1;
    float* lam_n;
    int64_t nc;
    int32_t nq;
    DoseAdj da;
};

// Words of a cell for the transposed step: lanes 0..2 sigma_t, sigma_s, 1/rho; 4..7 the
// neighbours' 1/A; 8.. the gradients to add to; 14, 15 the dose functional's dJ/dD.
template <typename GT>
struct AdjWords {
    const float* base;
    int stride;
    bool nbr;
    __device__ __forceinline__ AdjWords(int lane, const AzAdjoint& e, const GT* g_t, const GT* g_s,
                                        const GT* g_r) {
        constexpr int W = sizeof(GT) / 4;
        base = lane == 1 ? e.a.sigma_s : lane == 2 && e.a.inv_rho ? e.a.inv_rho : e.a.sigma_t;
        stride = 1;
        nbr = lane >= 4 && lane < 8;
        if (nbr) {
            base = reinterpret_cast<const float*>(e.geom) + 12;
            stride = 16;
        }
        const int i = (lane - 8) / W, w = (lane - 8) % W;
        const GT* g = i == 0 ? g_t : i == 1 ? g_s : g_r;
        if (lane >= 8 && i < 3 && g) {
            base = reinterpret_cast<const float*>(g) + w;
            stride = W;
        }
        if ((lane == 14 || lane == 15) && e.da.g_dose) {
            base = reinterpret_cast<const float*>(e.da.g_dose) + (lane - 14);
            stride = 2;
        }
    }
    template <int MF>
    __device__ __forceinline__ float load(float rec, int32_t c, int lane) const {
        int32_t i = c;
        if (nbr) {
#pragma unroll
            for (int f = 0; f < MF; ++f) {
                const int32_t j = CellWords::word(rec, f);
                if (lane == 4 + f && j >= 0) i = j;
            }
        }
        return base[(int64_t)i * stride];
    }
    __device__ __forceinline__ static GT gradient(float mat, int i) {
        if constexpr (sizeof(GT) == 8)
            return __builtin_bit_cast(
                double, ((uint64_t)(uint32_t)CellWords::word(mat, 9 + 2 * i) << 32) |
                            (uint32_t)CellWords::word(mat, 8 + 2 * i));
        else
            return CellWords::value(mat, 8 + i);
    }
};

template <typename P, int MF, typename GT, bool DA>
__global__ __launch_bounds__(P::THREADS, 4) void k_az_adjoint(AzModes<double> opd, AzAdjoint e,
                                                              GT* __restrict__ g_t,
                                                              GT* __restrict__ g_s,
                                                              GT* __restrict__ g_r)
{
    constexpr int SEG = P::SEG;
    using R = double;
    __shared__ __attribute__((aligned(16))) R lds[P::template LDS<R>];
    __shared__ V4<R> second[P::MU * kWave];
    __shared__ __attribute__((aligned(16))) float dirs[2 * kTable<P>];
    __shared__ f32x4 rows[P::WAVES][SEG * kWave];
    __shared__ float gsum[P::WPC == 2 ? P::WAVES : 1][4];
    const Lane<P> ln(opd);
    __shared__ V4<R> ftab[P::AZ * kWave];
    const Ops<P, R> op(opd, opd.adj, ln);
    const Fourier<P, R, true> fr(opd, ln, ftab);
    load_second<P, R>(opd.adj, second);
    load_dirs<P>(e.tab, e.nq, dirs);
    clear_corner<P>(ln, rows[ln.wave]);
    const StepArgs32& a = e.a;
    const uint32_t row_bytes = (uint32_t)e.nq * 4u, state_bytes = (uint32_t)e.nc * row_bytes;
    const auto rlam = make_rsrc(e.lam_np1, state_bytes);
    const auto rpsi = make_rsrc(e.psi_n, state_bytes);
    const auto rout = make_rsrc(e.lam_n, state_bytes);
    const AdjWords<GT> words(ln.lane, e, g_t, g_s, g_r);
    __shared__ double wtab[DA && P::RV ? kTable<P> : 1];
    double wd[DA ? SEG : 1];                                     // one weight per polar node
    if constexpr (DA && P::RV != 0) {
        load_table<P>(e.da.w, e.nq, wtab);
    } else if constexpr (DA) {
#pragma unroll
        for (int i = 0; i < SEG; ++i) wd[i] = e.da.w[ln.off[i] / 4];
    }
    Tiles tl((int32_t)((e.nc + kCells - 1) / kCells));
    if (tl.t >= tl.end) return;
    auto cell_of = [&](int32_t t) { return Cell(t < tl.end ? t : tl.end - 1, ln.cell, e.nc); };
    auto record = [&](int32_t t) { return CellWords::record(e.geom, cell_of(t).c, ln.lane); };
    auto own = [&](f32x4 (&p)[SEG], int32_t t) {
        const uint32_t row = (uint32_t)cell_of(t).c * row_bytes;
#pragma unroll
        for (int i = 0; i < SEG; ++i) p[i] = load_piece<P>(rlam, ln, i, row);
    };
    // the rows of segment i that the update alone needs: psi and the neighbours' lambda (a
    // boundary face reads the cell's own row, with weight 0)
    f32x4 l[SEG], lnx[SEG], p[SEG], nl[SEG][MF];
    auto others = [&](int i, float rec, int32_t c) {
        p[i] = load_piece<P>(rpsi, ln, i, (uint32_t)c * row_bytes);
#pragma unroll
        for (int f = 0; f < MF; ++f) {
            const int32_t j = CellWords::word(rec, f);
            nl[i][f] = load_piece<P>(rlam, ln, i, (uint32_t)(j >= 0 ? j : c) * row_bytes);
        }
    };
    auto add_gradients = [&](float mat, int32_t c, float pt, float ps, float pr, float irho) {
        if (g_t) g_t[c] = AdjWords<GT>::gradient(mat, 0) + (GT)(-a.dt * a.alpha_t * pt);
        if (g_s) g_s[c] = AdjWords<GT>::gradient(mat, 1) + (GT)(a.dt * a.alpha_s * ps);
        if (g_r) g_r[c] = AdjWords<GT>::gradient(mat, 2) + (GT)(a.dt * irho * irho * pr);
    };
    auto shared_gradients = [&](float mat, const Cell& c) {
        if (ln.mu0 == 0 && c.real) {
            const float *u = gsum[ln.cell], *v = gsum[P::WPC == 2 ? ln.cell + 8 : 0];
            const float irho = a.inv_rho ? CellWords::value(mat, 2) : 1.0f;
            const float pt = u[0] + v[0], ps = u[1] + v[1], pr = u[2] + v[2];
            if (ln.lane == 0) add_gradients(mat, c.c, pt, ps, pr, irho);
        }
    };
    float rec = record(tl.t), mat = words.template load<MF>(rec, cell_of(tl.t).c, ln.lane);
    own(l, tl.t);
#pragma unroll
    for (int i = 0; i < SEG; ++i) others(i, rec, cell_of(tl.t).c);
    float recn = record(tl.t + tl.stride), matp = mat;
    Cell cp = cell_of(tl.t);
    bool first = true;
    __syncthreads();                       // second, dirs
    for (;;) {
        const Cell c = cell_of(tl.t), cn = cell_of(tl.t + tl.stride);
        f32x4 x[SEG];
        __builtin_amdgcn_s_setprio(2);
        to_matrix_order<P>(x, l, ln, rows[ln.wave]);
        to_modes(x, fr, ln, lds);
        const float matn = words.template load<MF>(recn, cn.c, ln.lane);
        own(lnx, tl.t + tl.stride);
        const float recn2 = record(tl.t + 2 * tl.stride);
        lds_barrier();
        if (P::WPC == 2 && !first) shared_gradients(matp, cp);
        on_modes(op, ln, lds, [&](int i, int mu, const V4<R>& v) {
            return apply_pair<R>(op.d[i][mu], second_of<P, R>(second, ln, i, mu), v, ln.lane);
        });
        lds_barrier();
        from_modes(x, fr, ln, lds);
        to_memory_order<P>(x, ln, rows[ln.wave]);
        keep_infinities<P>(x, opd, rlam, (uint32_t)c.c * row_bytes, ln.lane);
        __builtin_amdgcn_s_setprio(0);
        using W = CellWords;
        const float ia = W::value(rec, 12), irho = a.inv_rho ? W::value(mat, 2) : 1.0f;
        const float cabs = a.dt * a.alpha_t * W::value(mat, 0);
        const float cscat = a.dt * a.alpha_s * W::value(mat, 1), cstream = a.dt * irho;
        float ian[MF], nx[MF], ny[MF];
        bool all_signs[MF];
#pragma unroll
        for (int f = 0; f < MF; ++f) {
            const bool bnd = W::word(rec, f) < 0;
            ian[f] = bnd ? 0.0f : W::value(mat, 4 + f);
            all_signs[f] = bnd && a.neumann;
            nx[f] = W::value(rec, 4 + 2 * f);
            ny[f] = W::value(rec, 5 + 2 * f);
        }
        double gd = 0.0;
        if constexpr (DA) {
            const uint64_t g = ((uint64_t)(uint32_t)W::word(mat, 15) << 32) | (uint32_t)W::word(mat, 14);
            gd = e.da.coeff * (a.inv_rho ? (double)irho : 1.0) * __builtin_bit_cast(double, g);
        }
        float pt = 0.0f, ps = 0.0f, pr = 0.0f;
#pragma unroll
        for (int i = 0; i < SEG; ++i) {
            float ox[4], oy[4];
            double w[4];
            table_piece<P>(dirs, ln, i, ox);
            table_piece<P>(dirs + kTable<P>, ln, i, oy);
            if constexpr (DA && P::RV != 0) table_piece<P>(wtab, ln, i, w);
            f32x4 o;
            float t0 = 0.0f, s0 = 0.0f, r0 = 0.0f;
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                if (!P::has(i, v)) continue;
                float xs = 0.0f;
#pragma unroll
                for (int f = 0; f < MF; ++f) {
                    const float s = __builtin_fmaf(nx[f], ox[v], ny[f] * oy[v]);
                    const float dd = __builtin_fmaf(-nl[i][f][v], ian[f], l[i][v] * ia);
                    xs = (s > 0.0f || all_signs[f]) ? __builtin_fmaf(s, dd, xs) : xs;
                }
                const float lv = l[i][v], g = x[i][v];
                o[v] = __builtin_fmaf(cscat, g,
                                      __builtin_fmaf(-cstream, xs, __builtin_fmaf(-lv, cabs, lv)));
                if (P::RV == 0 || ln.exists(i, v)) {
                    t0 = __builtin_fmaf(lv, p[i][v], t0);
                    s0 = __builtin_fmaf(p[i][v], g, s0);
                    r0 = __builtin_fmaf(p[i][v], xs, r0);
                }
                if constexpr (DA)
                    o[v] = (float)__builtin_fma(gd, P::RV ? w[v] : wd[i], (double)o[v]);
            }
            if (P::RV != 0 || ln.exists(i, 0)) {
                pt += t0;
                ps += s0;
                pr += r0;
            }
            if (c.real) store_piece<P>(rout, ln, i, (uint32_t)c.c * row_bytes, o);
            others(i, recn, cn.c);
        }
        pt = wave_sum_dpp(pt);
        ps = wave_sum_dpp(ps);
        pr = wave_sum_dpp(pr);
        if constexpr (P::WPC == 2) {
            if (ln.lane == 0) {
                gsum[ln.wave][0] = pt;
                gsum[ln.wave][1] = ps;
                gsum[ln.wave][2] = pr;
            }
        } else if (ln.lane == 0 && c.real) {
            add_gradients(mat, c.c, pt, ps, pr, irho);
        }
        matp = mat;
        cp = c;
        first = false;
        tl.t += tl.stride;
        if (tl.t >= tl.end) break;
#pragma unroll
        for (int i = 0; i < SEG; ++i) l[i] = lnx[i];
        rec = recn;
        recn = recn2;
        mat = matn;
    }
    if constexpr (P::WPC == 2) {
        lds_barrier();
        shared_gradients(matp, cp);
    }
}

// ----------------------------------------------------------------------------- the IMEX step

// b / (a - b lam); in FP64 from the hardware's estimate of the reciprocal and a Newton step (2e-15
// measured).
__device__ __forceinline__ float ratio(float b, float a, float lam) { return b / (a - b * lam); }
__device__ __forceinline__ double ratio(double b, double a, double lam) {
    const double d = __builtin_fma(-b, lam, a), r = __builtin_amdgcn_rcp(d);
    return b * __builtin_fma(__builtin_fma(-d, r, 1.0), r, r);
}

// The IMEX step with a dense kernel or its moment projection (Sec. 4.2) in one pass: per cell
// (a I - b A) psi' = r with a = 1 + dt alpha_t sigma_t, b = dt alpha_s sigma_s, A = K W.  The modes
// decouple, D_m = V diag(lam) V^-1 per mode, so psi' = (r + V D V^-1 r) / a with
// D = diag(b lam / (a - b lam)).  r is the collision-free step, formed from the wave's rows and
// kept in registers; in stage 2 the two polar products follow each other without LDS (an MFMA's
// result rows are the next one's K order), the per-cell diagonal between them.  The next
// tile's rows are fetched as soon as r is formed and fly during the exchange.  R: FP64 for FP32
// handles, FP32 for the 16-bit ones.  Element-wise errors of a stiff step (g = 0.95, 512 ordinates,
// one of them lit): FP64 modes 1.1e-6 (the step's FP32 roundings), the general solve of an FP32
// handle 2.1e-4, FP32 modes 3.3e-4, the general solve of a BF16x3 handle 9.7e-3.  100 352 x 1024:
// 0.321 ms in FP32 and 0.49 in FP64, against 1.43 ms with two nq x nq products (BF16x3) and 0.53 ms
// with two products through 96 padded moments, each after a collision-free step of its own.
template <typename P, typename R, int MF, bool RHO>
__global__ __launch_bounds__(P::THREADS, 4) void k_az_imex(AzModes<R> opd, StepEpi se)
{
    constexpr int SEG = P::SEG;
    __shared__ __attribute__((aligned(16))) R lds[P::template LDS<R>];
    __shared__ V4<R> second[2][P::MU * kWave];
    __shared__ __attribute__((aligned(16))) float dirs[2 * kTable<P>];
    __shared__ f32x4 rows[P::WAVES][SEG * kWave];
    const Lane<P> ln(opd);
    __shared__ V4<R> ftab[P::AZ * kWave];
    const Ops<P, R> op(opd, opd.e1, ln);
    const Fourier<P, R, true> fr(opd, ln, ftab);
    V4<R> e2[P::ITEMS][P::MU];
    Ops<P, R>::load(e2, opd.e2, ln);
    __shared__ V4<R> lam[P::AZ * P::MU * 8 * 2 * 4];
    const V4<R>* lam_at[P::ITEMS];
    for (int i = threadIdx.x; i < P::AZ * P::MU * 8 * 2 * 4; i += P::THREADS)
        lam[i] = reinterpret_cast<const V4<R>*>(opd.lam)[i];
#pragma unroll
    for (int i = 0; i < P::ITEMS; ++i) {
        const int az = Ops<P, R>::az_of(ln, i), pair = ln.wave & 7;
        const int which = pair == 0 && az == 0 ? (ln.lane >> 3) & 1 : 0;
        lam_at[i] = lam + ((az * 8 + pair) * 2 + which) * 4 + ln.l4;
    }
    load_second<P, R>(opd.e1, second[0]);
    load_second<P, R>(opd.e2, second[1]);
    load_dirs<P>(se.tab, se.nq, dirs);
    clear_corner<P>(ln, rows[ln.wave]);
    const StepArgs32& a = se.a;
    const FwdCtx<float> cx = make_ctx(a, se.psi_in, se.psi_out, se.nc, se.nq, se.nbf);
    const CellWords words(ln.lane, a, cx.src_arr, nullptr);
    Tiles tl((int32_t)((se.nc + kCells - 1) / kCells));
    if (tl.t >= tl.end) return;
    auto cell_of = [&](int32_t t) { return Cell(t < tl.end ? t : tl.end - 1, ln.cell, se.nc); };
    auto record = [&](int32_t t) { return CellWords::record(se.geom, cell_of(t).c, ln.lane); };
    // the materials of this lane's column in stage 2
    auto column = [&](const float* __restrict__ v, int32_t t) {
        const int64_t c = (int64_t)(t < tl.end ? t : tl.end - 1) * kCells + (ln.lane & 7);
        return v[c < se.nc ? c : se.nc - 1];
    };
    f32x4 p[SEG], up[SEG][MF];
    auto fetch = [&](float rec, int32_t c) {
#pragma unroll
        for (int i = 0; i < SEG; ++i) {
            p[i] = load_piece<P>(cx.psi, ln, i, (uint32_t)c * cx.row_bytes);
#pragma unroll
            for (int f = 0; f < MF; ++f)
                up[i][f] = load_face<P>(CellWords::word(rec, f), c, ln, i, cx);
        }
    };
    float rec = record(tl.t), mat = words.template material<MF>(rec, cell_of(tl.t).c, ln.lane);
    float st = column(a.sigma_t, tl.t), ss = column(a.sigma_s, tl.t);
    fetch(rec, cell_of(tl.t).c);
    float recn = record(tl.t + tl.stride);
    __syncthreads();                       // second, dirs
    for (;;) {
        const Cell c = cell_of(tl.t), cn = cell_of(tl.t + tl.stride);
        CellData<MF> cd;
        cd.template form<RHO>(rec, mat, a, cx);
        f32x4 r[SEG], x[SEG];
#pragma unroll
        for (int i = 0; i < SEG; ++i) {
            float ox[4], oy[4];
            table_piece<P>(dirs, ln, i, ox);
            table_piece<P>(dirs + kTable<P>, ln, i, oy);
            if (cd.scaled) {
#pragma unroll
                for (int f = 0; f < MF; ++f) up[i][f] *= cd.ghost[f];
            }
            const f32x4 acc = flux4<P, MF, RHO>(i, p[i], cd.irho, cd.nx, cd.ny, up[i], ox, oy);
#pragma unroll
            for (int v = 0; v < 4; ++v)
                r[i][v] = P::has(i, v)
                              ? __builtin_fmaf(cx.src_mul, cd.srcv,
                                               __builtin_fmaf(-cd.cflux, acc[v], p[i][v]))
                              : 0.0f;
        }
        const float matn = words.template material<MF>(recn, cn.c, ln.lane);
        const float stn = column(a.sigma_t, tl.t + tl.stride);
        const float ssn = column(a.sigma_s, tl.t + tl.stride);
        fetch(recn, cn.c);
        const float recn2 = record(tl.t + 2 * tl.stride);
        __builtin_amdgcn_s_setprio(2);
        to_matrix_order<P>(x, r, ln, rows[ln.wave]);
        to_modes(x, fr, ln, lds);
        lds_barrier();
        const R ca = R(1) + (R)a.dt * a.alpha_t * st, cb = (R)a.dt * a.alpha_s * ss;
        on_modes(op, ln, lds, [&](int i, int mu, const V4<R>& v) {
            V4<R> z = apply_pair<R>(op.d[i][mu], second_of<P, R>(second[0], ln, i, mu), v, ln.lane);
            const V4<R> l = lam_at[i][mu * P::AZ * 8 * 2 * 4];
#pragma unroll
            for (int k = 0; k < 4; ++k) z[k] *= ratio(cb, ca, l[k]);
            return apply_pair<R>(e2[i][mu], second_of<P, R>(second[1], ln, i, mu), z, ln.lane);
        });
        lds_barrier();
        from_modes(x, fr, ln, lds);
        to_memory_order<P>(x, ln, rows[ln.wave]);
        __builtin_amdgcn_s_setprio(0);
        const float y = cd.cabs / (1.0f + cd.cabs);
#pragma unroll
        for (int i = 0; i < SEG; ++i) {
            const f32x4 s = r[i] + x[i];
            f32x4 o;
#pragma unroll
            for (int v = 0; v < 4; ++v) o[v] = __builtin_fmaf(-s[v], y, s[v]);
            if (c.real) store_piece<P>(cx.out, ln, i, (uint32_t)c.c * cx.row_bytes, o);
        }
        tl.t += tl.stride;
        if (tl.t >= tl.end) break;
        rec = recn;
        recn = recn2;
        mat = matn;
        st = stn;
        ss = ssn;
    }
}

// ------------------------------------------------------------------------------ launch shape

// Blocks of a kernel over the mesh's tiles: what the device holds at once (a multiple of the XCD
// count), never more than there are tiles.
inline unsigned az_blocks(const snrt_mesh& m, int resident) {
    const int64_t tiles = (m.nc + kCells - 1) / kCells;
    const int64_t cap = (int64_t)m.num_cu * (resident > 0 ? resident : 1);
    const int64_t b = tiles < cap ? tiles : cap;
    return (unsigned)((b + kNumXcd - 1) / kNumXcd * kNumXcd);
}

template <typename K>
int az_resident(K kernel, int threads) {
    int n = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, kernel, threads, 0) != hipSuccess) n = 0;
    return n;
}

// f(shape) for the class shape of an operand.
template <typename R, typename F>
hipError_t by_shape(const AzModes<R>& op, F&& f) {
    const bool two = op.na > 16, fold = op.np > 16;
    if (op.na == (two ? 32 : 16)) {
        if (two) return fold ? f(Shape<2, 2>{}) : f(Shape<2, 1>{});
        return fold ? f(Shape<1, 2>{}) : f(Shape<1, 1>{});
    }
    // ordinates of a wave's piece of the row per lane
    const int rv = ((two && fold ? op.np / 2 : op.np) * op.na + kWave - 1) / kWave;
    auto wide = [&](auto az, auto mu) {
        constexpr int AZ = decltype(az)::value, MU = decltype(mu)::value;
        if (rv <= 2) return f(Shape<AZ, MU, 2>{});
        if (rv <= 4) return f(Shape<AZ, MU, 4>{});
        return rv <= 6 ? f(Shape<AZ, MU, 6>{}) : f(Shape<AZ, MU, 8>{});
    };
    using I1 = std::integral_constant<int, 1>;
    using I2 = std::integral_constant<int, 2>;
    if (two) return fold ? wide(I2{}, I2{}) : wide(I2{}, I1{});
    if (fold) return wide(I1{}, I2{});
    return rv <= 2 ? f(Shape<1, 1, 2>{}) : f(Shape<1, 1, 4>{});
}

}  // namespace az
}  // namespace snrt
