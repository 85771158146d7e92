"""The second-order stage in one launch (FP32) against the FP64 oracle: one tile and many, their
halos and boundary faces, one and two ordinates per lane, last chunks that are partly empty, both
limiters, densities, every boundary kind, dense scattering, any numbering, and the sizes and meshes
that take the two kernels instead.

Tolerance: a step is two stages; each forms an element from about thirty FP32 roundings of values of
its own size, scaled by at most a half of it per face through the CFL number, and a row sum whose
error grows with the root of its length (512: 23 * 6e-8 = 1.4e-6, times dt sigma < 1): 3e-6 a step.
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


def _step(P, neumann=False, scale=1.0, limiter="barth-jespersen", k=1.0, **kw):
    from paper_2205_08417_amd import snrt
    from paper_2205_08417_amd.solver import Solver
    S = Solver(P, **kw)
    x = S.initial_state()
    out = torch.empty_like(x)
    S.step2(x, out, S.args(inflow_scale=scale, boundary=snrt.SNRT_BC_NEUMANN if neumann
                            else snrt.SNRT_BC_DIRICHLET), limiter=limiter, vk_k=k)
    r = S.to_user(out).cpu().numpy()
    S.close()
    return r


def _oracle(P, neumann=False, scale=1.0, limiter="barth-jespersen", k=1.0):
    from oracle import oracle as o
    op = o.OracleProblem.from_problem(P, neumann=neumann)
    return o.step2(op, P.psi0, P.dt, inflow_scale=scale, limiter=limiter, vk_k=k)


MESHES = {
    "tri_18": lambda: I.jittered_delaunay_mesh(4, 0.0, 1.0, seed=191),       # one or two tiles
    "tri_1922": lambda: I.jittered_delaunay_mesh(32, 0.0, 1.0, seed=192),
    "quad_143": lambda: I.quad_grid_mesh(13, 11),
    "padded_512": lambda: I.pad_faces(I.jittered_delaunay_mesh(17, 0.0, 1.0, seed=193), 4),
}


@pytest.mark.parametrize("npol,naz", [(2, 2), (8, 8), (5, 13), (8, 16), (3, 43), (12, 16), (16, 32)])
@pytest.mark.parametrize("mesh", list(MESHES))
def test_tiles_vs_oracle(mesh, npol, naz):
    m = MESHES[mesh]()
    for full in (True, False):
        P = small_problem(m, npol, naz, seed=194, rho=full, source=full, inflow=full)
        for kw in (dict(scale=0.7), dict(neumann=not full, limiter="venkatakrishnan", k=0.8)):
            err = rel_l2(_step(P, **kw), _oracle(P, **kw))
            print(f"{mesh} nq={npol * naz} full={full} {kw}: {err:.2e}")
            assert err <= TOL


@pytest.mark.parametrize("nx", [54, 130])      # 5 618 cells: two kernels; 33 282: tiles
def test_the_sizes_between_and_above(nx):
    P = small_problem(I.jittered_delaunay_mesh(nx, 0.0, 1.0, seed=195), 1, 65, seed=196, rho=True,
                      inflow=True)
    assert rel_l2(_step(P), _oracle(P)) <= TOL


def test_any_numbering_gives_the_same_bits():
    m = MESHES["tri_1922"]()
    P = small_problem(m, 8, 16, seed=197, source=True, inflow=True)
    assert np.array_equal(_step(P, reorder=True), _step(P, reorder=False))


def test_normals_that_do_not_cancel_exactly_take_the_two_kernels():
    m = I.jittered_delaunay_mesh(9, 0.0, 1.0, seed=198)
    n = np.array(m.face_normal)
    n[3, 0] *= 1.0 + 2.0 ** -22
    P = small_problem(dataclasses.replace(m, face_normal=n), 4, 8, seed=199, inflow=True)
    assert rel_l2(_step(P), _oracle(P)) <= TOL
