"""GPU parity of rows that are not 64 * 2^k ordinates long, at the edges of the lanes' ordinate
counts (V = ceil(nq / 64) up to 8, then 16): every per-cell kernel against the FP64 oracle.

Tolerance: one step forms each element from about ten FP32 roundings of its own size and a sum
over the row whose error grows with the root of its length (1023 terms: 32 * 6e-8 = 2e-6, times
dt sigma < 1): 1e-6.  Gradients are such sums: 3e-6.  FP64 sums of FP32 states round the states
and materials only: 1e-6.
"""
import numpy as np
import pytest

from _util import rel_l2, small_problem

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from paper_2205_08417_amd import inputs as I  # noqa: E402

TOL = 1e-6
# 63 | 65 | 129 | 192 | 193 | 257 | 320 | 321 | 385 | 449 | 511 | 513 | 1023
COUNTS = [(7, 9), (5, 13), (3, 43), (12, 16), (1, 193), (1, 257), (16, 20), (3, 107), (5, 77),
          (1, 449), (7, 73), (19, 27), (31, 33)]


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    from paper_2205_08417_amd import snrt
    snrt.lib()


@pytest.mark.parametrize("npol,naz", COUNTS)
@pytest.mark.parametrize("quads", [False, True])
def test_every_row_kernel_vs_oracle(npol, naz, quads):
    from oracle import oracle as o
    from paper_2205_08417_amd import snrt
    from paper_2205_08417_amd.solver import Solver
    mesh = I.quad_grid_mesh(5, 4) if quads else I.jittered_delaunay_mesh(4, 0.0, 1.0, seed=91)
    P = small_problem(mesh, npol, naz, seed=92, rho=True, source=True, inflow=True)
    op = o.OracleProblem.from_problem(P)
    S = Solver(P)
    x, a = S.initial_state(), S.args(alpha_t=1.1, alpha_s=0.9, inflow_scale=0.6)
    out = torch.empty_like(x)
    user = lambda t: S.to_user(t.reshape(P.ncells, -1)).cpu().numpy()  # noqa: E731
    S.step(x, out, a)
    assert rel_l2(user(out), o.step(op, P.psi0, P.dt, 1.1, 0.9, 0.6)) <= TOL
    dose = torch.zeros(P.ncells, dtype=torch.float64, device="cuda")
    fused, again = dose.clone(), torch.empty_like(x)
    snrt.snrt_step_dose(S.mesh, S.quad, S.scatter, a, x, again, 0.37, fused, S.ws, S.ws_bytes)
    assert torch.equal(again, out)
    snrt.snrt_dose_accumulate(S.mesh, S.quad, x, S.mats32["inv_rho"], 0.37, dose)
    want = o.dose_accumulate(op, P.psi0, 0.37, np.zeros(P.ncells))
    assert rel_l2(user(fused)[:, 0], want) <= TOL and rel_l2(user(dose)[:, 0], want) <= TOL
    assert rel_l2(user(S.scalar_flux(x))[:, 0], o.scalar_flux(op, P.psi0)) <= TOL
    assert abs(S.mass(x) - o.mass(op, P.psi0)) <= TOL * o.mass(op, P.psi0)
    S.step_imex(x, out, a)
    assert rel_l2(user(out), o.step_imex(op, P.psi0, P.dt, 1.1, 0.9, 0.6)) <= TOL
    S.step2(x, out, a)
    assert rel_l2(user(out), o.step2(op, P.psi0, P.dt, 1.1, 0.9, 0.6)) <= TOL
    lam = np.random.default_rng(93).standard_normal((P.ncells, P.nq))
    g = [torch.zeros(P.ncells, device="cuda") for _ in range(3)]
    S.adjoint_step(x, S.to_internal(lam), out, *g, a)
    ref = [np.zeros(P.ncells) for _ in range(3)]
    assert rel_l2(user(out), o.adjoint_step(op, P.psi0, lam, P.dt, 1.1, 0.9, *ref)) <= TOL
    for got, r in zip(g, ref):
        assert rel_l2(user(got)[:, 0], r) <= 3 * TOL
    S.close()
