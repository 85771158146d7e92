// Tiles of the second-order stage kernel (sn_step2_tile.hip), laid out on the host: neighbouring
// cells, and the cells outside the tile that share a face with one inside (its halo), so that a
// block can hold the upwind value of every face of the tile in LDS, one row per face.
#pragma once

#include <algorithm>
#include <cstdint>
#include <cstdlib>
#include <memory>
#include <new>
#include <vector>

#include "host_ranges.h"

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

struct StagePart {
    std::vector<StageTile> tiles;
    std::vector<StageRow> rows;
};
// The kernel reaches a row's StageGeom at a 32-bit byte offset.
constexpr int64_t kStageRows = (int64_t(1) << 32) / (int64_t)sizeof(StageGeom);

// The tiles of the cells order[first .. end) (order null: as they are numbered), at most cap cells to
// a tile, as long as the faces fit a block's rows.  A face has one row and its two sides decide from
// their own normals which of them writes it: that takes normals that are exact negatives in FP32 and
// one face at most between two cells, in the slots of either.  false: these cells are not like that.
inline bool layout_tiles_of(const CellGeom32* geom, int64_t nc, int mf, const int32_t* order,
                            int64_t cap, int64_t first, int64_t last, StagePart& out)
{
    const auto back = [&](int32_t j, int32_t k) {      // the slot of cell k in cell j
        int g = 0;
        while (g < mf && geom[j].nbr[g] != k) ++g;
        return g;
    };
    out.tiles.reserve((last - first) / 64 + 1);
    out.rows.reserve((last - first) * 3 / 2);
    struct Free {
        void operator()(int32_t* p) const { std::free(p); }
    };
    // a cell's place among the tile's rows, from 1 (calloc: only the part's pages are touched)
    std::unique_ptr<int32_t, Free> places(static_cast<int32_t*>(std::calloc(nc, sizeof(int32_t))));
    if (!places) throw std::bad_alloc();
    int32_t* const place = places.get();
    int32_t cells[kStageCells + kStageFaces], face_row[kStageCells + kStageFaces][4];
    const auto enter = [&](int32_t k, int32_t n) {
        cells[n] = k;
        for (int32_t& r : face_row[n]) r = -1;
        place[k] = n + 1;
    };
    while (first < last) {
        int32_t n = 0, faces = 0;
        for (; first < last && n < cap; ++first) {
            const int32_t k = order ? order[first] : (int32_t)first;
            int32_t add = 0;
            for (int f = 0; f < mf; ++f) {
                const int32_t j = geom[k].nbr[f];
                if (j == k) continue;                  // an unused slot
                add += j < 0 || !place[j];
                if (j < 0) continue;
                for (int g = 0; g < f; ++g)
                    if (geom[k].nbr[g] == j) return false;
                const float *a = geom[k].n[f], *b = geom[j].n[back(j, k)];
                if (a[0] != -b[0] || a[1] != -b[1]) return false;
            }
            if (n > 0 && faces + add > kStageFaces) break;
            enter(k, n);
            for (int f = 0; f < mf; ++f) {
                const int32_t j = geom[k].nbr[f];
                if (j == k) continue;
                face_row[n][f] = j >= 0 && place[j] ? face_row[place[j] - 1][back(j, k)] : faces++;
            }
            ++n;
        }
        StageTile t = {(int32_t)out.rows.size(), n, 0, 0};
        for (int32_t i = 0; i < t.cells; ++i)
            for (int f = 0; f < mf; ++f) {
                const int32_t k = cells[i], j = geom[k].nbr[f];
                if (j < 0 || j == k) continue;
                if (!place[j]) enter(j, n++);
                if (place[j] > t.cells) face_row[place[j] - 1][back(j, k)] = face_row[i][f];
            }
        t.halo = n - t.cells;
        for (int32_t i = 0; i < n; ++i) {
            const int32_t k = cells[i];
            place[k] = 0;
            StageRow r = {k, {0, 0}, 0.5f * geom[k].inv_area, {}};
            bool interior = true;
            const int32_t* rows = face_row[i];
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

// The tiles of a mesh, laid out and kept part by part (host_ranges), their rows numbered through.
// false: the mesh has none, because of its faces or because the rows exceed most.
struct StageLayout {
    StagePart part[kHostParts];
    int64_t ntiles = 0, nrows = 0;
};
inline bool layout_stage_tiles(const CellGeom32* geom, int64_t nc, int mf, const int32_t* order,
                               int64_t cap, StageLayout& out, int64_t most = kStageRows)
{
    bool ok[kHostParts];
    std::fill(ok, ok + kHostParts, true);
    host_ranges(nc, [&](int p, int64_t first, int64_t last) {
        ok[p] = layout_tiles_of(geom, nc, mf, order, cap, first, last, out.part[p]);
    });
    out.ntiles = out.nrows = 0;
    for (const StagePart& l : out.part) {
        out.ntiles += (int64_t)l.tiles.size();
        out.nrows += (int64_t)l.rows.size();
    }
    if (out.nrows > most || !std::all_of(ok, ok + kHostParts, [](bool b) { return b; })) return false;
    int32_t before = 0;
    for (StagePart& l : out.part) {
        for (StageTile& t : l.tiles) t.rows += before;
        before += (int32_t)l.rows.size();
    }
    return true;
}

}  // namespace snrt
