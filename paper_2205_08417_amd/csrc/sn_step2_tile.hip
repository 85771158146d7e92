// A stage of the second-order scheme in one launch: limited gradients and the update that takes
// its face values from them (the formulas are in sn_step2.hip).
//
// The two-kernel stage writes the gradients, two rows per cell, and reads them back for the cell
// and each of its neighbours: of 350 us per stage (198 450 cells x 256 ordinates, 130 + 220) 32 are
// the time to copy a row per cell, and it moves seven of them.  Here a block owns a tile of up to
// 96 cells (StageTile) and sweeps the ordinates in chunks of 128, two per lane.  Per chunk its 16
// waves compute the slopes of the tile's cells and of its halo (1.36 slopes per cell), and write
// the flux through each face of the tile into LDS, an ordinate's by the side that it leaves; then
// they update the tile's cells with the sum over the faces.  The gradients take no memory, and
// the flux of a face is reconstructed once, by the upwind side alone: the two-kernel stage
// reconstructs both sides in both cells.  The rows of 158 faces take half of a CU's LDS (a G row
// per cell and halo cell instead would hold as few cells and take more arithmetic), so that the
// slopes of one block overlap the update of another.
// What bounds it is the arithmetic (105.7 million vector instructions per stage, at four cycles
// 413 000 of each SIMD's 540 000) and the latency of the scalar loads that precede a cell's rows:
// 16 waves a block 502 us per step, 12 waves 590, 8 waves 758; the records of a cell in one place
// and loaded ahead 447.  The step took 730 through two kernels.
#include "sn_slope.h"

namespace snrt {

namespace {

constexpr int kStageBlock = 1024;
constexpr int kStageWaves = kStageBlock / kWave;

__device__ __forceinline__ float row_ld(__amdgpu_buffer_rsrc_t r, uint32_t lane_off, uint32_t row) {
    return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(r, lane_off, row, 0));
}

struct StageCtx {
    __amdgpu_buffer_rsrc_t psi, inflow;
    uint32_t row_bytes;
    float inflow_scale;
    bool dirichlet, neumann;
};

// A cell whose slope is next: its own and its far sides' values, raw with their factors where
// there is a density, else u itself.
template <int V, int MF, bool RHO>
struct SlopeCell {
    uint32_t faces[2];
    float half_inv_area;
    float u[V], uf[MF][V];
    float irho, scale[MF];
};
template <int V, int MF, bool RHO>
__device__ __forceinline__ void load_slope_cell(SlopeCell<V, MF, RHO>& d, const StageRow& row,
                                                const uint32_t (&off)[V], const StepArgs32& a,
                                                const StageCtx& x)
{
    d.faces[0] = row.faces[0];
    d.faces[1] = row.faces[1];
    d.half_inv_area = row.half_inv_area;
    const int32_t c = row.cell;
    d.irho = RHO ? cell_val(a.inv_rho, c) : 1.0f;
#pragma unroll
    for (int k = 0; k < V; ++k) d.u[k] = row_ld(x.psi, off[k], (uint32_t)c * x.row_bytes);
    if (row.faces[0] & kFaceInterior) {
#pragma unroll
        for (int f = 0; f < MF; ++f) {
            const int32_t j = row.nbr[f];
            if constexpr (RHO) d.scale[f] = cell_val(a.inv_rho, j);
#pragma unroll
            for (int k = 0; k < V; ++k)
                d.uf[f][k] = row_ld(x.psi, off[k], (uint32_t)j * x.row_bytes);
        }
        return;
    }
    const float bscale = x.dirichlet ? x.inflow_scale : (x.neumann ? d.irho : 0.0f);
#pragma unroll
    for (int f = 0; f < MF; ++f) {
        const int32_t j = row.nbr[f];
        const bool bnd = j < 0;
        const int32_t from = bnd ? (x.dirichlet ? -1 - j : c) : j;
        d.scale[f] = bnd ? bscale : (RHO ? cell_val(a.inv_rho, bnd ? c : j) : 1.0f);
#pragma unroll
        for (int k = 0; k < V; ++k) {
            d.uf[f][k] = row_ld(bnd && x.dirichlet ? x.inflow : x.psi, off[k],
                                (uint32_t)from * x.row_bytes);
            if constexpr (!RHO) d.uf[f][k] *= d.scale[f];
        }
    }
}

// The slope of a cell, and through each face of the tile the flux of the ordinates that leave
// the cell there, out of the face's lower side.
template <int V, int MF, bool RHO, int LIM>
__device__ __forceinline__ void face_fluxes(SlopeCell<V, MF, RHO>& d, const StageGeom& g,
                                            const float (&ox)[V], const float (&oy)[V], float vk_k,
                                            float (&face)[kStageFaces][V][kWave], int lane)
{
    float gx[V], gy[V], umax[V], umin[V];
#pragma unroll
    for (int k = 0; k < V; ++k) {
        if constexpr (RHO) d.u[k] *= d.irho;
        gx[k] = gy[k] = 0.0f;
        umax[k] = umin[k] = d.u[k];
#pragma unroll
        for (int f = 0; f < MF; ++f) {
            if constexpr (RHO) d.uf[f][k] *= d.scale[f];
            const float sum = d.u[k] + d.uf[f][k];
            gx[k] = fmaf(sum, g.n[f][0], gx[k]);
            gy[k] = fmaf(sum, g.n[f][1], gy[k]);
            umax[k] = larger(umax[k], d.uf[f][k]);
            umin[k] = smaller(umin[k], d.uf[f][k]);
        }
        gx[k] *= d.half_inv_area;
        gy[k] *= d.half_inv_area;
    }
    limit_slope<V, MF, LIM>(gx, gy, d.u, umax, umin, g.r,
                            limiter_eps2<LIM>(vk_k, 2.0f * d.half_inv_area));
#pragma unroll
    for (int f = 0; f < MF; ++f) {
        const uint32_t e = d.faces[f / 2] >> (16 * (f % 2));
        if (e & kFaceSkip) continue;
        float* const to = &face[e & kFaceRow][0][lane];
        // Omega n of the lower side, exactly the negative of the upper side's
        const uint32_t flip = e & kFaceLower ? 0u : 0x80000000u;
        const float nx = __builtin_bit_cast(float, __builtin_bit_cast(uint32_t, g.n[f][0]) ^ flip);
        const float ny = __builtin_bit_cast(float, __builtin_bit_cast(uint32_t, g.n[f][1]) ^ flip);
        float s[V], ui[V];
#pragma unroll
        for (int k = 0; k < V; ++k) {
            s[k] = fmaf(oy[k], ny, ox[k] * nx);
            ui[k] = fmaf(gy[k], g.r[f][1], fmaf(gx[k], g.r[f][0], d.u[k]));
        }
        if (e & kFaceBoundary) {
#pragma unroll
            for (int k = 0; k < V; ++k) to[k * kWave] = s[k] * (s[k] > 0.0f ? ui[k] : d.uf[f][k]);
        } else if (e & kFaceLower) {
#pragma unroll
            for (int k = 0; k < V; ++k)
                if (s[k] >= 0.0f) to[k * kWave] = s[k] * ui[k];
        } else {
#pragma unroll
            for (int k = 0; k < V; ++k)
                if (s[k] < 0.0f) to[k * kWave] = s[k] * ui[k];
        }
    }
}

// A cell whose update is next: its own values.
template <int V>
struct UpdateCell {
    int32_t cell;
    uint32_t faces[2];
    float half_inv_area, sigma_t, sigma_s, source;
    float p[V], src[V], pn[V];
};
template <int V>
__device__ __forceinline__ void load_update_cell(UpdateCell<V>& d, const StageRow& row,
                                                 const StepArgs32& a,
                                                 const uint32_t (&off)[V], const float* S,
                                                 const float* psi_n, uint32_t state_bytes,
                                                 const StageCtx& x)
{
    d.cell = row.cell;
    d.faces[0] = row.faces[0];
    d.faces[1] = row.faces[1];
    d.half_inv_area = row.half_inv_area;
    d.sigma_t = cell_val(a.sigma_t, row.cell);
    d.sigma_s = cell_val(a.sigma_s, row.cell);
    d.source = a.source ? cell_val(a.source, row.cell) : 0.0f;
    const uint32_t own = (uint32_t)row.cell * x.row_bytes;
#pragma unroll
    for (int k = 0; k < V; ++k) d.p[k] = row_ld(x.psi, off[k], own);
    if (S) {
        const auto rs = make_rsrc(S, state_bytes);
#pragma unroll
        for (int k = 0; k < V; ++k) d.src[k] = row_ld(rs, off[k], own);
    }
    if (psi_n) {
        const auto rn = make_rsrc(psi_n, state_bytes);
#pragma unroll
        for (int k = 0; k < V; ++k) d.pn[k] = row_ld(rn, off[k], own);
    }
}

template <int V, int MF, bool RHO, int LIM>
__global__ __launch_bounds__(kStageBlock, 2 * kStageWaves / 4) void k_stage2(
    const StageTile* __restrict__ tile_of, const StageRow* __restrict__ rows,
    const StageGeom* __restrict__ geom,
    int32_t nc, int32_t nq, const float* __restrict__ tab, StepArgs32 a,
    const float* __restrict__ psi, const float* __restrict__ S, const float* __restrict__ psi_n,
    float* __restrict__ out, uint32_t nbf, int32_t parts, int32_t chunks_per_part, float vk_k)
{
    __shared__ float face[kStageFaces][V][kWave];      // the flux out of each face's lower side
    __shared__ float phi[kStageCells];
    const int32_t b = (int32_t)xcd_remap(blockIdx.x, gridDim.x);
    const StageTile t = tile_of[uniform_cell(b / parts)];
    const int part = b % parts;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int lane = threadIdx.x & (kWave - 1);
    const int nch = (nq + V * kWave - 1) / (V * kWave);

    StageCtx x;
    x.row_bytes = (uint32_t)nq * 4u;
    const uint32_t state_bytes = (uint32_t)nc * x.row_bytes;
    x.psi = make_rsrc(psi, state_bytes);
    x.inflow = make_rsrc(a.inflow ? a.inflow : psi, a.inflow ? nbf * x.row_bytes : 0u);
    x.inflow_scale = a.inflow_scale;
    x.dirichlet = a.inflow != nullptr && !a.neumann;
    x.neumann = a.neumann != 0;

    if (!S) {
        // three cells at a time: their loads overlap, and share the weights
        for (int i = wave; i < t.cells; i += 3 * kStageWaves) {
            uint32_t row[3];
            float sum[3] = {0.0f, 0.0f, 0.0f};
#pragma unroll
            for (int k = 0; k < 3; ++k)
                row[k] = (uint32_t)cell_rec(rows, t.rows + min(i + k * kStageWaves, t.cells - 1))->cell *
                         x.row_bytes;
#pragma unroll 4
            for (int q = lane; q < nq; q += kWave) {
                const float w = tab[3 * nq + q];
#pragma unroll
                for (int k = 0; k < 3; ++k)
                    sum[k] = fmaf(w, row_ld(x.psi, (uint32_t)q * 4u, row[k]), sum[k]);
            }
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                sum[k] = cell_sum(sum[k]);
                if (lane == 0 && i + k * kStageWaves < t.cells) phi[i + k * kStageWaves] = sum[k];
            }
        }
    }

    const int ch1 = min(nch, (part + 1) * chunks_per_part);
    for (int ch = part * chunks_per_part; ch < ch1; ++ch) {
        // lanes past the last ordinate repeat it and store nothing
        uint32_t off[V];
        float ox[V], oy[V];
#pragma unroll
        for (int k = 0; k < V; ++k) {
            const int q = min((ch * V + k) * kWave + lane, nq - 1);
            off[k] = (uint32_t)q * 4u;
            ox[k] = tab[q];
            oy[k] = tab[nq + q];
        }
        lds_barrier();      // the update of the chunk before has read its face values
        // in flight while a cell is worked on: the next cell's values and the row entry after it
        const int n = t.cells + t.halo;
        const auto row = [&](int i) { return *cell_rec(rows, t.rows + (i < n ? i : n - 1)); };
        const auto geo = [&](int i) { return *cell_rec(geom, t.rows + (i < n ? i : n - 1)); };
        {
            SlopeCell<V, MF, RHO> da, db;
            StageRow next = row(wave);
            StageGeom g;
            load_slope_cell<V, MF, RHO>(da, next, off, a, x);
            next = row(wave + kStageWaves);
            for (int i = wave; i < n; i += 2 * kStageWaves) {
                load_slope_cell<V, MF, RHO>(db, next, off, a, x);
                g = geo(i);
                next = row(i + 2 * kStageWaves);
                face_fluxes<V, MF, RHO, LIM>(da, g, ox, oy, vk_k, face, lane);
                if (i + kStageWaves >= n) break;
                load_slope_cell<V, MF, RHO>(da, next, off, a, x);
                next = row(i + 3 * kStageWaves);
                g = geo(i + kStageWaves);
                face_fluxes<V, MF, RHO, LIM>(db, g, ox, oy, vk_k, face, lane);
            }
        }
        UpdateCell<V> ua;
        StageRow next = row(wave);
        load_update_cell(ua, next, a, off, S, psi_n, state_bytes, x);
        next = row(wave + kStageWaves);
        lds_barrier();
        const auto update = [&](const UpdateCell<V>& d, int i) {
            const float cabs = a.dt * a.alpha_t * d.sigma_t;   // absorption as p - cabs p
            const float cflux = a.dt * (2.0f * d.half_inv_area);
            const float cscat = a.dt * a.alpha_s * d.sigma_s;
            const float csrc = a.dt * d.source;
            float acc[V];
#pragma unroll
            for (int k = 0; k < V; ++k) acc[k] = 0.0f;
#pragma unroll
            for (int f = 0; f < MF; ++f) {
                const uint32_t e = d.faces[f / 2] >> (16 * (f % 2));
                // an unused slot's row is another face's: no share of it
                const float side = e & kFaceLower ? 1.0f : e & kFaceSkip ? 0.0f : -1.0f;
#pragma unroll
                for (int k = 0; k < V; ++k) acc[k] = fmaf(side, face[e & kFaceRow][k][lane], acc[k]);
            }
            const auto ro = make_rsrc(out, state_bytes);
#pragma unroll
            for (int k = 0; k < V; ++k) {
                const float src = S ? d.src[k] : phi[i];
                float o = (d.p[k] - cabs * d.p[k]) - cflux * acc[k] + cscat * src + csrc;
                if (psi_n) o = 0.5f * (d.pn[k] + o);
                if ((ch * V + k) * kWave + lane < nq)
                    __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(int32_t, o), ro, off[k],
                                                          (uint32_t)d.cell * x.row_bytes, kAuxStream);
            }
        };
        for (int i = wave; i < t.cells; i += kStageWaves) {
            update(ua, i);
            load_update_cell(ua, next, a, off, S, psi_n, state_bytes, x);
            next = row(i + 2 * kStageWaves);
        }
    }
}

__global__ void k_stage_geom(const CellGeom32* __restrict__ cells,
                             const CellRecon32* __restrict__ recon,
                             const StageRow* __restrict__ rows, StageGeom* __restrict__ geom,
                             int64_t n)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const int32_t c = rows[i].cell;
    StageGeom g;
    for (int f = 0; f < 4; ++f)
        for (int d = 0; d < 2; ++d) {
            g.n[f][d] = cells[c].n[f][d];
            g.r[f][d] = recon[c].r_own[f][d];
        }
    geom[i] = g;
}

}  // namespace

hipError_t launch_stage_geom(const snrt_mesh& m, const StageRow* rows, StageGeom* geom, int64_t n,
                             hipStream_t st) {
    hipLaunchKernelGGL(k_stage_geom, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, m.geom32,
                       m.recon32, rows, geom, n);
    return hipGetLastError();
}

// Where the two kernels' gradients outgrow the caches, where there are enough cells for whole tiles,
// and where the launches are what costs.  Between these the gradients stay in the caches and the
// halo's slopes and the few blocks cost more.  Quadrilaterals have more faces to a tile, and
// Venkatakrishnan's limiter a quotient for each (Barth-Jespersen two per cell).  us per Heun step,
// tiles : two kernels, Barth-Jespersen on triangles | quadrilaterals, Venkatakrishnan on the same:
//     4 000 x   64   14 : 16  |   15 : 16       15 : 18  |   17 : 17
//     4 000 x  128   16 : 17  |   18 : 18       19 : 18  |   24 : 20
//     2 000 x  512   26 : 20  |   29 : 22       30 : 23  |   39 : 27
//     4 000 x  256   24 : 20  |   27 : 21       28 : 22  |   36 : 25
//    16 000 x  256   62 : 51  |   72 : 55       75 : 59  |   95 : 67
//    22 000 x  512  127 : 129 |  149 : 142     154 : 138 |  200 : 158     (45 MB)
//    32 800 x   64   45 : 43  |   45 : 47       51 : 46  |   54 : 52
//    32 800 x  100   56 : 65  |   55 : 74       72 : 67  |   78 : 79
//    32 800 x  256   87 : 93  |  104 : 101     107 : 105 |  138 : 116
//    32 800 x  512  164 : 203 |  199 : 228     202 : 216 |  265 : 243     (67 MB)
//    50 000 x  256  128 : 129 |  148 : 142     162 : 147 |  199 : 166
//    50 000 x  480  254 : 352 |  315 : 403     300 : 362 |  406 : 423     (96 MB)
//   100 000 x   32  100 : 117 |  116 : 129     113 : 118 |  137 : 133
//   100 000 x  256  220 : 358 |  270 : 393     279 : 372 |  380 : 423
bool stage2_tiled(const snrt_mesh& m, const snrt_quad& q, const Limiter& lim) {
    const int64_t bytes = m.nc * (int64_t)q.nq * 4;
    // 32-bit offsets, as in the persistent kernels
    if (m.tiles.count == 0 || bytes >= (int64_t(1) << 32) ||
        m.nbf * (int64_t)q.nq * 4 >= (int64_t(1) << 32))
        return false;
    const bool vk = lim.kind == SNRT_LIMITER_VENKATAKRISHNAN, quads = m.mf == 4;
    if (m.nc <= 4096 && q.nq <= (vk || quads ? 64 : 128)) return true;
    const int64_t mb = bytes >> 20;
    if (vk) return mb >= (quads ? 90 : 64);
    return mb >= 48 || m.nc >= 65536 || (m.nc >= 32768 && q.nq > 64);
}

hipError_t launch_stage2_32(const snrt_mesh& m, const snrt_quad& q, const StepArgs32& a,
                            const Limiter& lim, const float* psi, const float* S,
                            const float* psi_n, float* out, hipStream_t st) {
    if (m.nc == 0) return hipSuccess;
    const int v = q.nq <= kWave ? 1 : 2;
    const int nch = (q.nq + v * kWave - 1) / (v * kWave);
    // blocks of half a CU: the chunks are split over blocks until there are six rounds of them
    // (198 450 cells x 256: 441 us, one block per tile 438; 16 562 x 1 024 has 185 tiles)
    int parts = 1;
    while (parts < nch && (int64_t)m.tiles.count * parts < 12 * m.num_cu) ++parts;
    const int per = (nch + parts - 1) / parts;
    parts = (nch + per - 1) / per;
    const bool vk = lim.kind == SNRT_LIMITER_VENKATAKRISHNAN, rho = a.inv_rho != nullptr;
    auto go = [&](auto vc, auto mfc, auto rc, auto lc) {
        constexpr int V = decltype(vc)::value;
        constexpr int MF = decltype(mfc)::value;
        constexpr bool R = decltype(rc)::value;
        constexpr int L = decltype(lc)::value;
        hipLaunchKernelGGL((k_stage2<V, MF, R, L>), dim3((unsigned)(m.tiles.count * parts)),
                           dim3(kStageBlock), 0, st, m.tiles.tile, m.tiles.rows, m.tiles.geom, (int32_t)m.nc,
                           q.nq, q.tab32, a, psi, S, psi_n, out, (uint32_t)m.nbf, (int32_t)parts,
                           (int32_t)per, (float)lim.k);
        return hipGetLastError();
    };
    using std::integral_constant;
    auto by_lim = [&](auto vc, auto mfc, auto rc) {
        return vk ? go(vc, mfc, rc, integral_constant<int, SNRT_LIMITER_VENKATAKRISHNAN>{})
                  : go(vc, mfc, rc, integral_constant<int, SNRT_LIMITER_BARTH_JESPERSEN>{});
    };
    auto by_rho = [&](auto vc, auto mfc) {
        return rho ? by_lim(vc, mfc, std::true_type{}) : by_lim(vc, mfc, std::false_type{});
    };
    auto by_faces = [&](auto vc) {
        return m.mf == 4 ? by_rho(vc, integral_constant<int, 4>{})
                         : by_rho(vc, integral_constant<int, 3>{});
    };
    return v == 1 ? by_faces(integral_constant<int, 1>{}) : by_faces(integral_constant<int, 2>{});
}

}  // namespace snrt
