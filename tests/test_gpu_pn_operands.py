"""The P_N step's coefficients per element: one moment of one cell is lit, and every moment that it
reaches in a neighbour is a short chain of products.

Tolerance: geometry (4 FP32 roundings), the face coefficient and P, Q (2), the coefficient of the
operator and its product (2), and a sum of four terms (3) of at most 2^-24 each of the terms'
magnitudes: 11 * 2^-24, however small the coefficient is beside the largest of its class.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from paper_2205_08417_amd import inputs as I  # noqa: E402

TOL = 11 * 2.0 ** -24


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")


@pytest.mark.parametrize("degree", [9, 10, 11, 12, 14])
@pytest.mark.parametrize("quads", [False, True])
def test_every_coefficient(degree, quads):
    from paper_2205_08417_amd import snrt
    from paper_2205_08417_amd.pn import PNSolver
    m = I.quad_grid_mesh(6, 5) if quads else I.jittered_delaunay_mesh(6, 0.0, 1.0, seed=311)
    nc, nm = m.ncells, (degree + 1) ** 2
    zero = np.zeros(nc)
    dt = 0.25 * float(m.area.min())
    S = PNSolver(m, degree, zero, zero, dt)
    ax, ay, ax_abs, ay_abs = (np.asarray(a).reshape(nm, nm) for a in snrt.snrt_pn_operators(degree))
    inner = int(np.flatnonzero((m.face_nbr >= 0).all(1))[3])
    out = S.to_tiled(torch.zeros(nc, nm, device="cuda"))
    worst = 0.0
    for mom in range(nm):
        v = np.float32(0.7 + 0.013 * mom)
        u = torch.zeros(nc, nm, device="cuda")
        u[inner, mom] = float(v)
        S.step(S.to_tiled(u), out)
        got = S.to_user(out).cpu().numpy().astype(np.float64)
        for i in m.face_nbr[inner]:
            n = m.face_normal[i, list(m.face_nbr[i]).index(inner)]
            s = -dt / m.area[i] * 0.5 * float(v)
            terms = [n[0] * ax[mom], n[1] * ay[mom], -abs(n[0]) * ax_abs[mom],
                     -abs(n[1]) * ay_abs[mom]]
            want, size = s * sum(terms), abs(s) * sum(np.abs(t) for t in terms)
            at = size > 1e-12 * size.max()        # structural zeros of the operators
            worst = max(worst, float((np.abs(got[i] - want)[at] / size[at]).max()))
            assert np.abs(got[i])[~at].max(initial=0.0) <= 1e-12
    print(f"P{degree} quads={quads}: {worst:.2e}")
    S.close()
    assert worst <= TOL
