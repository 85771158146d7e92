// Tiles of the second-order stage kernel (sn_step2_tile.hip), laid out on the host: neighbouring
// cells, and the cells outside the tile that share a face with one inside (its halo), so that a
// block can hold the upwind value of every face of the tile in LDS, one row per face.
#pragma once

#include <algorithm>
#include <cstdint>
#include <vector>

namespace snrt {

// Per-cell geometry record, one 64-byte line: neighbours, n_ij (outward normal x length),
// 1/A_i and A_i.  An unused face slot points at the cell itself with a zero normal.
struct alignas(64) CellGeom32 {
    int32_t nbr[4];
    float n[4][2];
    float inv_area;
    float area;
    float pad[2];
};
static_assert(sizeof(CellGeom32) == 64, "one cache line per cell");

constexpr int kStageFaces = 158;       // face rows of a block, 64 lanes x 2 x 4 bytes each
constexpr int kStageCells = 96;        // cells of a tile at most
struct StageTile {
    int32_t rows;                      // first of its StageRows: its cells, then its halo
    int32_t cells, halo;
    int32_t pad;
};
// A cell of a tile or of its halo, in whole words for two scalar loads; the LDS row of face f, and
// who writes it, are the half word f % 2 of faces[f / 2].
struct alignas(32) StageRow {
    int32_t cell;
    uint32_t faces[2];
    float half_inv_area;
    int32_t nbr[4];
};
constexpr uint32_t kFaceRow = 0x1ff;        // the LDS row (an unused slot's: a used face's)
constexpr uint32_t kFaceInterior = 0x1000;  // on face 0: no face of the cell is a boundary's
constexpr uint32_t kFaceLower = 0x2000;     // the lower of the face's two cells, or the only one
constexpr uint32_t kFaceBoundary = 0x4000;  // this side writes the ghost value as well
constexpr uint32_t kFaceSkip = 0x8000;      // not a face of the tile, or an unused slot
struct alignas(64) StageGeom {
    float n[4][2], r[4][2];            // CellGeom32::n, CellRecon32::r_own
};

struct StageLayout {
    std::vector<StageTile> tiles;
    std::vector<StageRow> rows;
};

// Cells along order (null: as they are numbered), at most cap to a tile, as long as the faces fit
// a block's rows.  A face has one row and its two sides decide from their own normals which of them
// writes it: that takes normals that are exact negatives in FP32 and one face at most between two
// cells, in the slots of either.  false: the mesh is not like that, and has no tiles.
inline bool layout_stage_tiles(const CellGeom32* geom, int64_t nc, int mf, const int32_t* order,
                               int64_t cap, StageLayout& out)
{
    out.tiles.clear();
    out.rows.clear();
    const auto back = [&](int32_t j, int32_t k) {      // the slot of cell k in cell j
        int g = 0;
        while (g < mf && geom[j].nbr[g] != k) ++g;
        return g;
    };
    for (int32_t k = 0; k < nc; ++k)
        for (int f = 0; f < mf; ++f) {
            const int32_t j = geom[k].nbr[f];
            if (j < 0 || j == k) continue;             // a boundary, an unused slot
            for (int g = 0; g < f; ++g)
                if (geom[k].nbr[g] == j) return false;
            const float *n = geom[k].n[f], *nj = geom[j].n[back(j, k)];
            if (n[0] != -nj[0] || n[1] != -nj[1]) return false;
        }
    out.rows.reserve(nc + nc / 2);
    struct Faces {
        int32_t row[4];
    };
    std::vector<int32_t> local(nc, -1), cells;         // a cell's place among the tile's rows
    std::vector<Faces> face_row;                       // of those rows
    for (int64_t first = 0, end; first < nc; first = end) {
        cells.clear();
        int32_t faces = 0;
        for (end = first; end < nc && end - first < cap; ++end) {
            const int32_t k = order ? order[end] : (int32_t)end;
            int32_t add = 0;
            for (int f = 0; f < mf; ++f) {
                const int32_t j = geom[k].nbr[f];
                add += j != k && (j < 0 || local[j] < 0);
            }
            if (end > first && faces + add > kStageFaces) break;
            faces += add;
            local[k] = (int32_t)cells.size();
            cells.push_back(k);
        }
        StageTile t = {(int32_t)out.rows.size(), (int32_t)cells.size(), 0, 0};
        face_row.assign(cells.size(), {{-1, -1, -1, -1}});
        int32_t next = 0;
        for (int32_t i = 0; i < t.cells; ++i)
            for (int f = 0; f < mf; ++f) {
                const int32_t k = cells[i], j = geom[k].nbr[f];
                if (j == k || face_row[i].row[f] >= 0) continue;
                face_row[i].row[f] = next;
                if (j >= 0) {
                    if (local[j] < 0) {
                        local[j] = (int32_t)cells.size();
                        cells.push_back(j);
                        face_row.push_back({{-1, -1, -1, -1}});
                    }
                    face_row[local[j]].row[back(j, k)] = next;
                }
                ++next;
            }
        t.halo = (int32_t)cells.size() - t.cells;
        for (size_t i = 0; i < cells.size(); ++i) {
            const int32_t k = cells[i];
            local[k] = -1;
            StageRow r = {k, {0, 0}, 0.5f * geom[k].inv_area, {}};
            bool interior = true;
            const int32_t* rows = face_row[i].row;
            const int32_t any = *std::max_element(rows, rows + 4);
            for (int f = 0; f < 4; ++f) {
                const int32_t row = rows[f], j = geom[k].nbr[f];
                const uint32_t e = row < 0 ? (uint32_t)any | kFaceSkip
                                           : (uint32_t)row | (j < 0 ? kFaceBoundary : 0) |
                                                 (j < 0 || k < j ? kFaceLower : 0);
                interior &= j >= 0;
                r.faces[f / 2] |= e << (16 * (f % 2));
                r.nbr[f] = j;
            }
            r.faces[0] |= interior ? kFaceInterior : 0;
            out.rows.push_back(r);
        }
        out.tiles.push_back(t);
    }
    return true;
}

}  // namespace snrt
