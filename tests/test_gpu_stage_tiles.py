"""Second-order steps (FP32) of meshes and calls at the edges of the one-launch stage, against the
FP64 oracle.

Tolerance 3e-6 a step: two stages of about thirty FP32 roundings of values of an element's own size,
scaled by at most a half per face through the CFL number, and a row sum (512 ordinates: 1.4e-6 times
dt sigma < 1).
"""
import dataclasses

import numpy as np
import pytest

from _util import rel_l2, small_problem

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from paper_2205_08417_amd import inputs as I  # noqa: E402

TOL = 3e-6


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    from paper_2205_08417_amd import snrt
    snrt.lib()


def _heun(S, **kw):
    x = S.initial_state()
    out = torch.empty_like(x)
    S.step2(x, out, S.args(), **kw)
    return S.to_user(out).cpu().numpy()


def _oracle(P, **kw):
    from oracle import oracle as o
    return o.step2(o.OracleProblem.from_problem(P), P.psi0, P.dt, **kw)


@pytest.mark.parametrize("side", ["lower", "higher"])
def test_a_neighbour_in_two_slots_of_one_cell(side):
    """Degenerate quadrilaterals: the fourth slot repeats a neighbour, with a zero normal."""
    from paper_2205_08417_amd.solver import Solver
    m = I.pad_faces(I.jittered_delaunay_mesh(9, 0.0, 1.0, seed=291), 4)
    nbr, mid = np.array(m.face_nbr), np.array(m.face_mid)
    k = np.arange(m.ncells)
    for slot, cell in ((0, 20), (1, 71), (2, 104)):
        want = nbr[:, slot] > k if side == "lower" else (nbr[:, slot] >= 0) & (nbr[:, slot] < k)
        c = int(np.flatnonzero(want & (k >= cell))[0])
        nbr[c, 3], mid[c, 3] = nbr[c, slot], mid[c, slot]
    P = small_problem(dataclasses.replace(m, face_nbr=nbr, face_mid=mid), 8, 8, seed=292, rho=True,
                      inflow=True)
    S = Solver(P, reorder=False)
    assert rel_l2(_heun(S), _oracle(P)) <= TOL
    S.close()


@pytest.mark.parametrize("mesh", ["triangles", "quads"])
def test_a_captured_step_sees_midpoints_that_are_set_later(mesh):
    """The step's graph is replayed after new face midpoints, with eager work between: the mesh's
    records change in place, and every replay is the eager result."""
    from paper_2205_08417_amd import snrt
    from paper_2205_08417_amd.solver import Solver
    m = I.quad_grid_mesh(23, 19) if mesh == "quads" else I.jittered_delaunay_mesh(21, 0.0, 1.0, seed=293)
    P = small_problem(m, 8, 8, seed=294, inflow=True)
    S = Solver(P)
    x = S.initial_state()
    out, other = torch.empty_like(x), torch.empty_like(x)
    args = S.args()
    S.step2(x, out, args)
    torch.cuda.synchronize()
    assert rel_l2(S.to_user(out).cpu().numpy(), _oracle(P)) <= TOL
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        S.step2(x, out, args)
    rng = np.random.default_rng(295)
    for rep in range(3):
        # the face values of another point of every face
        moved = dataclasses.replace(m, face_mid=m.face_mid + 0.02 * rng.uniform(-1, 1, m.face_mid.shape)
                                    * np.abs(m.face_normal[..., ::-1]))
        snrt.snrt_mesh_set_face_midpoints(S.mesh, moved.face_mid)
        hold = [torch.full((1 << 14,), 1e30, device="cuda") for _ in range(8)]   # takes freed memory
        S.step2(x, other, args)
        out.fill_(float("nan"))
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, other), f"replay {rep}"
        assert rel_l2(S.to_user(out).cpu().numpy(), _oracle(dataclasses.replace(P, mesh=moved))) <= TOL
        del hold
    S.close()
