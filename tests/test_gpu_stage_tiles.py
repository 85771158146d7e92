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


# A block's chunks of 128 ordinates.  More than 3 072 tiles take all chunks in one block (240 ordinates:
# a full chunk and one of 112); 1 200 tiles split them, 480 ordinates into two and two, 640 into two,
# two and one, 500 ordinates of 600 tiles into one each.  The row sums of isotropic scattering are kept
# between a block's chunks.
@pytest.mark.parametrize("nx,npol,naz,dense", [(388, 12, 20, False), (224, 20, 24, False),
                                               (224, 20, 24, True), (224, 20, 32, False),
                                               (159, 20, 25, False)])
def test_several_ordinate_chunks_in_a_block(nx, npol, naz, dense):
    _large(I.jittered_delaunay_mesh(nx, 0.0, 1.0, seed=296), npol, naz, dense)


@pytest.mark.parametrize("limiter", ["barth-jespersen", "venkatakrishnan"])
def test_large_quadrilateral_meshes(limiter):
    _large(I.quad_grid_mesh(223, 221), 16, 32, False, limiter=limiter)


def _large(mesh, npol, naz, dense, **kw):
    """Sampled cells of one step against the oracle on the part of the mesh that they depend on."""
    from paper_2205_08417_amd.solver import Solver
    omega, w = I.product_quadrature(npol, naz)
    K = I.henyey_greenstein_kernel(omega, w, 0.7) if dense else None
    P = small_problem(mesh, omega_w=(omega, w), K=K, seed=297, rho=True, source=True, inflow=True)
    S = Solver(P)
    got = _heun(S, **kw)
    S.close()
    rng = np.random.default_rng(298)
    seeds = rng.choice(mesh.ncells, 60, replace=False)
    ring = [set(seeds.tolist())]
    for _ in range(4):                        # two stages of gradients and fluxes
        n = mesh.face_nbr[sorted(ring[-1])]
        ring.append(ring[-1] | set(n[n >= 0].tolist()))
    part = np.array(sorted(ring[-1]))
    to = np.full(mesh.ncells, -1)
    to[part] = np.arange(part.size)
    nbr = mesh.face_nbr[part]
    cut = (nbr >= 0) & (to[np.maximum(nbr, 0)] < 0)
    nbr = np.where(nbr >= 0, to[np.maximum(nbr, 0)], nbr)
    nbr[cut] = -1                             # beyond the rings: any boundary does
    sub = dataclasses.replace(mesh, cells=mesh.cells[part], face_nbr=nbr.astype(np.int32),
                              face_normal=mesh.face_normal[part], area=mesh.area[part],
                              centroid=mesh.centroid[part], face_mid=mesh.face_mid[part])
    Q = dataclasses.replace(P, mesh=sub, sigma_t=P.sigma_t[part], sigma_s=P.sigma_s[part],
                            rho=P.rho[part], source=P.source[part], psi0=P.psi0[part])
    want = _oracle(Q, **kw)
    err = rel_l2(got[seeds], want[to[seeds]])
    print(f"{mesh.ncells} x {P.nq} {kw}: {err:.2e}")
    assert err <= TOL
