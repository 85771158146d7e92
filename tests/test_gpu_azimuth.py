"""GPU parity of the scattering through azimuthal modes (kernels that couple the ordinates of a
product rule through their polar nodes and azimuth difference only), against the FP64 oracle.

Tolerance: three chained FP32 contractions of 16 terms and four additions per value, every
rounding 2^-24, growing like the square root of their count: sqrt(52) 6e-8 = 4.3e-7 of the
product's norm, so 1e-6.  Gradients that are sums over a row of random sign get ten times that.
"""
import dataclasses

import numpy as np
import pytest

from _util import rel_l2, small_problem

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from paper_2205_08417_amd import inputs as I  # noqa: E402

TOL = 1e-6
# polar x azimuthal: every fold, full and partly filled polar slots, an odd count; then azimuths
# that leave slots empty (odd, even, folded with an even and an odd half), at the edges of the
# striped rows' lane counts (128 | 192 | 256 | 320 | 384 | 512 ordinates per wave)
SHAPES = [(8, 32), (13, 32), (16, 32), (18, 32), (32, 32), (9, 16), (16, 16), (20, 16), (32, 16),
          (12, 10), (13, 11), (16, 15), (20, 9), (26, 13), (32, 15), (13, 18), (16, 20), (16, 24),
          (15, 26), (16, 30), (18, 22), (28, 26), (32, 30)]


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    from paper_2205_08417_amd import snrt
    snrt.lib()


def _mesh(kind):
    if kind == "quads":
        return I.quad_grid_mesh(7, 5)
    return I.jittered_delaunay_mesh(kind, 0.0, 1.0, seed=71)


def _problem(npol, naz, mesh, K=None, rho=True, seed=72):
    omega, w = I.product_quadrature(npol, naz)
    K = I.henyey_greenstein_kernel(omega, w, 0.9) if K is None else K
    return small_problem(mesh, omega_w=(omega, w), K=K, rho=rho, source=True, inflow=True,
                         seed=seed, scatter=(0.5, 1.0))


def _apply(S, x, transpose):
    from paper_2205_08417_amd import snrt
    out = torch.empty_like(x)
    snrt.snrt_scatter_apply(S.mesh, S.quad, S.scatter, x, out, transpose, S.ws, S.ws_bytes)
    return out.cpu().numpy()


# 2, 8 and 18 triangles: a part of a tile of eight cells, one, two and a quarter
@pytest.mark.parametrize("npol,naz", SHAPES)
@pytest.mark.parametrize("kind", [2, 3, 4, "quads"])
def test_product_step_dose_and_transposed_step_vs_oracle(npol, naz, kind):
    from oracle import oracle as o
    from paper_2205_08417_amd import snrt
    from paper_2205_08417_amd.solver import Solver
    rho = kind != 3
    P = _problem(npol, naz, _mesh(kind), rho=rho)
    P = dataclasses.replace(P, psi0=I.random_state(P.ncells, P.nq, seed=73, decades=2.0))
    op = o.OracleProblem.from_problem(P)
    S = Solver(P, precision="fp32")
    x = S.initial_state()
    rows = x.cpu().numpy().astype(np.float64)
    for transpose in (0, 1):
        B = P.w[:, None] * P.K.T
        err = rel_l2(_apply(S, x, transpose), rows @ (B.T if transpose else B))
        print(f"{npol}x{naz} {kind} transpose={transpose}: {err:.2e}")
        assert err <= TOL
    # the step, and the step with its dose
    args = S.args(alpha_t=1.1, alpha_s=0.9, inflow_scale=0.6)
    out, out_d = torch.empty_like(x), torch.empty_like(x)
    S.step(x, out, args)
    dose = S.cells_to_internal(np.full(P.ncells, 0.25), torch.float64)
    snrt.snrt_step_dose(S.mesh, S.quad, S.scatter, args, x, out_d, 0.37, dose, S.ws, S.ws_bytes)
    assert torch.equal(out, out_d)
    want = o.step(op, P.psi0, P.dt, 1.1, 0.9, 0.6)
    assert rel_l2(S.to_user(out).cpu().numpy(), want) <= TOL
    dref = o.dose_accumulate(op, P.psi0, 0.37, np.full(P.ncells, 0.25))
    assert rel_l2(S.to_user(dose.reshape(-1, 1)).cpu().numpy().ravel(), dref) <= TOL
    # the transposed step and its gradients
    lam = np.random.default_rng(74).standard_normal((P.ncells, P.nq))
    l1, l0 = S.to_internal(lam), torch.empty_like(x)
    g = [torch.zeros(P.ncells, device="cuda") for _ in range(3)]
    S.adjoint_step(x, l1, l0, g[0], g[1], g[2] if rho else None,
                   S.args(alpha_t=1.2, alpha_s=0.8))
    gt, gs = np.zeros(P.ncells), np.zeros(P.ncells)
    gr = np.zeros(P.ncells) if rho else None
    want = o.adjoint_step(op, P.psi0, lam, P.dt, 1.2, 0.8, gt, gs, gr)
    assert rel_l2(S.to_user(l0).cpu().numpy(), want) <= TOL
    for got, ref in zip(g, (gt, gs, gr) if rho else (gt, gs)):
        assert rel_l2(S.to_user(got.reshape(-1, 1)).cpu().numpy().ravel(), ref) <= 10 * TOL
    S.close()


def _kernel(npol, naz):
    omega, w = I.product_quadrature(npol, naz)
    return omega, w, I.henyey_greenstein_kernel(omega, w, 0.9)


def _one_entry():
    omega, w, K = _kernel(16, 16)
    K[37, 101] *= 1.5
    return omega, w, K


def _no_mirror():
    omega, w, K = _kernel(32, 16)
    K[256:] *= 1.2                       # the upper half of the polar nodes as receivers
    return omega, w, K


def _odd_in_difference():
    omega, w, K = _kernel(16, 16)
    l = np.arange(16)
    skew = 1.0 + 0.3 * np.sin(2 * np.pi * (l[:, None] - l[None, :]) / 16)
    return omega, w, K * np.tile(skew, (16, 16))


def _uneven_weights():
    omega, w, K = _kernel(16, 16)
    return omega, w * (1.0 + 0.2 * np.cos(np.arange(256))), K


@pytest.mark.parametrize("make", [_one_entry, _no_mirror, _odd_in_difference, _uneven_weights,
                                  lambda: _kernel(16, 34), lambda: _kernel(17, 32),
                                  lambda: _kernel(32, 19), lambda: _kernel(4, 32)],
                         ids=["one-entry", "no-mirror", "odd-in-difference", "uneven-weights",
                              "34-azimuths", "17-polar", "19-azimuths", "4-polar"])
@pytest.mark.parametrize("precision,tol", [("fp32", TOL), ("bf16x3", 2e-5)])
def test_operators_without_the_structure_keep_the_general_products(make, precision, tol):
    """Kernels, weights and shapes outside the structure: their product, step and transposed step
    still match the full kernel (an operator averaged into the structure would be off by 1e-3 at
    the least)."""
    from oracle import oracle as o
    from paper_2205_08417_amd.solver import Solver
    omega, w, K = make()
    P = small_problem(_mesh(4), omega_w=(omega, w), K=K, seed=75, scatter=(0.5, 1.0))
    S = Solver(P, precision=precision)
    x = S.initial_state()
    rows = x.cpu().numpy().astype(np.float64)
    B = w[:, None] * K.T
    for transpose in (0, 1):
        assert rel_l2(_apply(S, x, transpose), rows @ (B.T if transpose else B)) <= tol
    op = o.OracleProblem.from_problem(P)
    out = torch.empty_like(x)
    S.step(x, out)
    assert rel_l2(S.to_user(out).cpu().numpy(), o.step(op, P.psi0, P.dt)) <= tol
    lam = np.random.default_rng(76).standard_normal((P.ncells, P.nq))
    g = [torch.zeros(P.ncells, device="cuda") for _ in range(2)]
    S.adjoint_step(x, S.to_internal(lam), out, g[0], g[1], None)
    ref = [np.zeros(P.ncells) for _ in range(2)]
    assert rel_l2(S.to_user(out).cpu().numpy(),
                  o.adjoint_step(op, P.psi0, lam, P.dt, 1.0, 1.0, ref[0], ref[1], None)) <= tol
    S.close()


# stiff: dt sigma of the order of ten.  The solve applies the modes' eigenvectors (condition
# number the root of the weights' ratio, below 4 here) around the diagonal: twice the product's
# roundings, each once more through the weights, 4 * TOL.
@pytest.mark.parametrize("npol,naz", [(8, 32), (13, 32), (18, 32), (9, 16), (16, 16), (20, 16),
                                      (12, 10), (20, 9), (13, 18), (16, 24), (18, 22)])
@pytest.mark.parametrize("kind", [3, 4, "quads"])
@pytest.mark.parametrize("moments", [False, True])
def test_imex_step_vs_oracle(npol, naz, kind, moments):
    from oracle import moments as mo
    from oracle import oracle as o
    from paper_2205_08417_amd.solver import Solver
    P = _problem(npol, naz, _mesh(kind), rho=kind != 3, seed=77)
    st = P.sigma_t * 10.0 / P.dt
    P = dataclasses.replace(P, sigma_t=st, sigma_s=0.9 * st)
    sig = I.hg_legendre_moments(0.8, 3) if moments else None
    K = mo.moment_kernel(P.omega, P.w, sig) if moments else P.K
    op = o.OracleProblem.from_problem(P, K=K)
    S = Solver(P, precision="fp32", moments=sig)
    out = torch.empty_like(S.initial_state())
    S.step_imex(S.initial_state(), out, S.args(alpha_t=1.1, alpha_s=0.9, inflow_scale=0.6))
    err = rel_l2(S.to_user(out).cpu().numpy(), o.step_imex(op, P.psi0, P.dt, 1.1, 0.9, 0.6))
    print(f"imex {npol}x{naz} {kind} moments={moments}: {err:.2e}")
    S.close()
    assert err <= 4 * TOL
