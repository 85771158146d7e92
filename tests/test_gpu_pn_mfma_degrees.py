"""P_N steps of degrees 10 to 12, whose FP32 step runs on the matrix cores: reflection classes
short of the 32 rows of a product (16 to 28 moments), both z parities, triangle, quadrilateral
and padded faces, a last tile that is partly empty and a mesh of less than one tile."""
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from paper_2205_08417_amd import inputs as I  # noqa: E402
import test_gpu_pn as P  # noqa: E402

MESHES = {
    "tri_392": lambda: I.jittered_delaunay_mesh(15, 0.0, 1.0, seed=170),
    "tri_32": lambda: I.jittered_delaunay_mesh(5, 0.0, 1.0, seed=171),
    "quad_247": lambda: I.quad_grid_mesh(19, 13),
    "padded_200": lambda: I.pad_faces(I.jittered_delaunay_mesh(11, 0.0, 1.0, seed=172), 4),
}
STEPS = 4
# FP32, per step: the round-off of u (2^-24), and the flux, at CFL 0.5 at most half of u per
# face, four faces, its operands held to 22 bits (2^-21): 6e-8 + 4 * 0.5 * 4.8e-7 < 1.1e-6
TOL = STEPS * 1.1e-6


@pytest.mark.parametrize("mesh_name", list(MESHES))
@pytest.mark.parametrize("degree", [10, 11, 12])
def test_matrix_core_degrees_vs_oracle(mesh_name, degree):
    mesh = MESHES[mesh_name]()
    kw = dict(alpha_t=1.1, alpha_s=0.9, inflow_scale=0.8)
    for full in (True, False):
        d = P._case(mesh, degree, seed=173 + degree, rho=full, source=full, ghost=full,
                    neumann=not full, sigma_l=I.hg_legendre_moments(0.7, degree))
        _, _, ref = P._oracle(d, STEPS, **kw)
        err = P.rel_l2(P._run(d, STEPS, torch.float32, **kw), ref)
        print(f"P{degree} {mesh_name} full={full}: {err:.2e}")
        assert err <= TOL
