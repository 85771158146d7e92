"""The tiles of the second-order stage kernel, laid out on the host (no device): every face of a
tile has one LDS row and a writer on either side, rows and cells stay within a block's, and meshes
whose faces do not pair one to one have none."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

from paper_2205_08417_amd import inputs as I

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                    "paper_2205_08417_amd", "csrc")
SHIM = r"""
#include "sn_stage_tiles.h"
using namespace snrt;
static std::vector<StageTile> all_tiles;
static std::vector<StageRow> all_rows;
extern "C" int make(const void* geom, long nc, int mf, const int* order, long cap, long most) {
    StageLayout l;
    if (!layout_stage_tiles(static_cast<const CellGeom32*>(geom), nc, mf, order, cap, l,
                            most < 0 ? kStageRows : most))
        return 0;
    all_tiles.clear();
    all_rows.clear();
    for (const StagePart& p : l.part) {
        all_tiles.insert(all_tiles.end(), p.tiles.begin(), p.tiles.end());
        all_rows.insert(all_rows.end(), p.rows.begin(), p.rows.end());
    }
    return (long)all_tiles.size() == l.ntiles && (long)all_rows.size() == l.nrows;
}
extern "C" long ntiles() { return (long)all_tiles.size(); }
extern "C" long nrows() { return (long)all_rows.size(); }
extern "C" const void* tiles() { return all_tiles.data(); }
extern "C" const void* rows() { return all_rows.data(); }
"""
ROW, INTERIOR, LOWER, BOUNDARY, SKIP = 0x1ff, 0x1000, 0x2000, 0x4000, 0x8000
FACES = 158


@pytest.fixture(scope="module")
def shim(tmp_path_factory):
    d = tmp_path_factory.mktemp("stage_tiles")
    src, so = d / "shim.cpp", d / "shim.so"
    src.write_text(SHIM)
    subprocess.run(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", "-pthread", "-I", CSRC,
                    str(src), "-o", str(so)], check=True)
    lib = ctypes.CDLL(str(so))
    lib.make.argtypes = [ctypes.c_void_p, ctypes.c_long, ctypes.c_int, ctypes.c_void_p,
                         ctypes.c_long, ctypes.c_long]
    for f in (lib.ntiles, lib.nrows):
        f.restype = ctypes.c_long
    for f in (lib.tiles, lib.rows):
        f.restype = ctypes.c_void_p
    return lib


def _records(mesh):
    """The library's geometry records: unused slots are the cell itself with a zero normal."""
    g = np.zeros(mesh.ncells, dtype=[("nbr", "i4", 4), ("n", "f4", (4, 2)), ("inv", "f4"),
                                     ("area", "f4"), ("pad", "f4", 2)])
    g["nbr"] = np.arange(mesh.ncells)[:, None]
    nbr = mesh.face_nbr
    used = nbr != np.iinfo(np.int32).min
    mf = mesh.max_faces
    g["nbr"][:, :mf] = np.where(used, nbr, g["nbr"][:, :mf])
    g["n"][:, :mf] = np.where(used[..., None], mesh.face_normal, 0.0)
    g["inv"], g["area"] = 1.0 / mesh.area, mesh.area
    return g


def _layout(shim, g, mf, order=None, cap=96, most=-1):
    o = None if order is None else np.ascontiguousarray(order, dtype=np.int32)
    if not shim.make(g.ctypes.data, len(g), mf, None if o is None else o.ctypes.data, cap, most):
        return None
    tiles = np.ctypeslib.as_array((ctypes.c_int32 * (4 * shim.ntiles())).from_address(
        shim.tiles())).reshape(-1, 4).copy()
    rows = np.ctypeslib.as_array((ctypes.c_uint32 * (8 * shim.nrows())).from_address(
        shim.rows())).reshape(-1, 8).copy()
    return tiles, rows


def _check(g, mf, tiles, rows, order, cap):
    owners, at = [], 0
    for first, cells, halo, _ in tiles:
        assert first == at and 1 <= cells <= cap
        at += cells + halo
        writers = {}
        for i in range(first, first + cells + halo):
            k, nbr = int(rows[i, 0].astype(np.int32)), rows[i, 4:].astype(np.int32)
            assert np.array_equal(nbr, g["nbr"][k])
            assert rows[i, 3:4].view(np.float32)[0] == np.float32(0.5) * g["inv"][k]
            word = [(int(rows[i, 1 + f // 2]) >> (16 * (f % 2))) & 0xffff for f in range(4)]
            assert bool(word[0] & INTERIOR) == bool((nbr >= 0).all())
            if i < first + cells:
                owners.append(k)
            for f in range(4):
                e = word[f] & ~INTERIOR
                assert (e & ROW) < FACES
                if nbr[f] == k:
                    assert e & SKIP and not e & LOWER
                elif i < first + cells:
                    assert not e & SKIP
                if not e & SKIP:
                    side = "both" if nbr[f] < 0 else "lower" if k < nbr[f] else "upper"
                    assert bool(e & BOUNDARY) == (side == "both")
                    assert bool(e & LOWER) == (side != "upper")
                    pair = (k,) if nbr[f] < 0 else tuple(sorted((k, int(nbr[f]))))
                    writers.setdefault(e & ROW, []).append((side, pair))
        # a row is one face's: written by its two sides, or by the one of a boundary
        for w in writers.values():
            sides = sorted(s for s, _ in w)
            assert sides == ["both"] or (sides == ["lower", "upper"] and w[0][1] == w[1][1])
        assert sorted(writers) == list(range(len(writers))) and len(writers) <= FACES
    assert at == len(rows)
    assert np.array_equal(owners, np.arange(len(g)) if order is None else order)


MESHES = {
    "tri_2": lambda: I.jittered_delaunay_mesh(2, 0.0, 1.0, seed=281),
    "tri_1922": lambda: I.jittered_delaunay_mesh(32, 0.0, 1.0, seed=282),
    "quad_143": lambda: I.quad_grid_mesh(13, 11),
    "padded_512": lambda: I.pad_faces(I.jittered_delaunay_mesh(17, 0.0, 1.0, seed=283), 4),
    "tri_9800": lambda: I.jittered_delaunay_mesh(71, 0.0, 1.0, seed=286),      # two threads
    "quad_36481": lambda: I.quad_grid_mesh(191, 191),                          # eight
}


@pytest.mark.parametrize("name", list(MESHES))
@pytest.mark.parametrize("cap", [16, 96])
def test_every_face_row_has_its_writers(shim, name, cap):
    m = MESHES[name]()
    g = _records(m)
    rng = np.random.default_rng(284)
    for order in (None, rng.permutation(m.ncells)):    # any order, even one without neighbours
        tiles, rows = _layout(shim, g, m.max_faces, order, cap)
        _check(g, m.max_faces, tiles, rows, order, cap)


@pytest.mark.parametrize("side", ["lower", "higher"])
@pytest.mark.parametrize("slot", [0, 1, 2])
def test_a_neighbour_in_two_slots_of_one_cell_leaves_no_tiles(shim, side, slot):
    """A degenerate quadrilateral that lists a neighbour twice, the second time with a zero normal:
    the neighbour's one slot cannot be the other side of both."""
    m = I.pad_faces(I.jittered_delaunay_mesh(9, 0.0, 1.0, seed=285), 4)
    g = _records(m)
    assert _layout(shim, g, 4) is not None
    nbr = g["nbr"][:, slot]
    want = nbr > np.arange(m.ncells) if side == "lower" else (nbr >= 0) & (nbr < np.arange(m.ncells))
    k = int(np.flatnonzero(want)[3])
    g["nbr"][k, 3] = nbr[k]
    assert _layout(shim, g, 4) is None


def test_normals_that_do_not_cancel_leave_no_tiles(shim):
    m = MESHES["tri_1922"]()
    g = _records(m)
    k = int(np.flatnonzero((g["nbr"][:, :3] >= 0).all(1))[5])
    g["n"][k, 1, 0] *= np.float32(1.0 + 2.0 ** -22)
    assert _layout(shim, g, 3) is None


def test_rows_beyond_the_kernels_offsets_leave_no_tiles(shim):
    m = MESHES["tri_9800"]()
    g = _records(m)
    n = len(_layout(shim, g, 3)[1])
    assert n < 2 ** 26      # records of 64 bytes at 32-bit offsets
    assert _layout(shim, g, 3, most=n) is not None
    assert _layout(shim, g, 3, most=n - 1) is None
