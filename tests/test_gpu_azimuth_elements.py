"""The azimuthal-mode scattering element by element, against FP64: peaked kernels on rows with one
lit ordinate, a beam and two decades of values, where an error relative to a row's norm would exceed
the small elements by orders of magnitude.

Tolerances: the product is formed in FP64 and rounded to FP32 once, with an operator whose smallest
entry is above 2^-25 of its norm: 2^-24 for the rounding and as much for the rest.
"""
import dataclasses

import numpy as np
import pytest

from _util import small_problem

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from paper_2205_08417_amd import inputs as I  # noqa: E402

EPS = 2.0 ** -24
# every fold, full and partly filled slots, striped rows
SHAPES = [(16, 32), (32, 32), (12, 16), (20, 16), (10, 10), (13, 18), (32, 15), (18, 22)]


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    from paper_2205_08417_amd import snrt
    snrt.lib()


def _rows(kind, omega, nc, seed):
    rng = np.random.default_rng(seed)
    nq = len(omega)
    if kind == "lit":
        x = np.zeros((nc, nq))
        x[np.arange(nc), rng.integers(0, nq, nc)] = 1.0
    elif kind == "beam":
        x = np.exp(-(omega[:, 1] + 1.0) ** 2 / 0.02)[None, :] * (0.5 + rng.random((nc, 1)))
    else:
        x = 10.0 ** (-2.0 * rng.random((nc, nq)))
    return x.astype(np.float32).astype(np.float64)


def _solver(omega, w, K, psi, precision, seed=301):
    from paper_2205_08417_amd.solver import Solver
    P = small_problem(I.jittered_delaunay_mesh(5, 0.0, 1.0, seed=seed), omega_w=(omega, w), K=K,
                      seed=seed, scatter=(0.5, 1.0))
    P = dataclasses.replace(P, psi0=psi(P.ncells))
    return P, Solver(P, precision=precision, reorder=False)


def _apply(S, x, transpose):
    from paper_2205_08417_amd import snrt
    out = torch.empty_like(x)
    snrt.snrt_scatter_apply(S.mesh, S.quad, S.scatter, x, out, transpose, S.ws, S.ws_bytes)
    return out.cpu().numpy().astype(np.float64)


@pytest.mark.parametrize("npol,naz", SHAPES)
@pytest.mark.parametrize("g", [0.5, 0.95])
@pytest.mark.parametrize("kind", ["lit", "beam", "two decades"])
def test_product_per_element(npol, naz, g, kind):
    omega, w = I.product_quadrature(npol, naz)
    K = I.henyey_greenstein_kernel(omega, w, g)
    precision = "bf16x3" if npol * naz % 32 == 0 and kind == "lit" else "fp32"
    P, S = _solver(omega, w, K, lambda nc: _rows(kind, omega, nc, 302), precision)
    x = S.initial_state()
    B = w[:, None] * K.T
    for transpose in (0, 1):
        got, want = _apply(S, x, transpose), P.psi0 @ (B.T if transpose else B)
        err = float((np.abs(got - want) / want).max())
        print(f"{npol}x{naz} g={g} {kind} transpose={transpose}: {err:.2e}")
        assert got.min() > 0.0 and err <= 2 * EPS
    S.close()


@pytest.mark.parametrize("npol,naz", [(16, 32), (12, 16), (10, 10)])
def test_a_kernel_that_ends_at_an_angle_scatters_nothing_beyond_it(npol, naz):
    omega, w = I.product_quadrature(npol, naz)
    K = I.henyey_greenstein_kernel(omega, w, 0.9)
    K[omega @ omega.T < 0.3] = 0.0
    P, S = _solver(omega, w, K, lambda nc: _rows("lit", omega, nc, 303), "fp32")
    x = S.initial_state()
    B = w[:, None] * K.T
    for transpose in (0, 1):
        got, want = _apply(S, x, transpose), P.psi0 @ (B.T if transpose else B)
        assert (want == 0.0).any() and np.array_equal(got == 0.0, want == 0.0)
        at = want > 0.0
        assert float((np.abs(got - want)[at] / want[at]).max()) <= 2 * EPS
    S.close()


@pytest.mark.parametrize("npol,naz", SHAPES)
def test_values_that_are_not_finite_stay_in_their_cell(npol, naz):
    """A positive kernel takes an infinite ordinate to an infinite row, a NaN or both infinities to
    a row of NaN, and no cell sees another's."""
    omega, w = I.product_quadrature(npol, naz)
    K = I.henyey_greenstein_kernel(omega, w, 0.8)
    P, S = _solver(omega, w, K, lambda nc: _rows("two", omega, nc, 304), "fp32")
    psi = P.psi0.copy()
    n = npol * naz
    psi[1, 0], psi[2, n - 1], psi[5, n // 2 + 1] = np.inf, -np.inf, np.nan
    psi[9, 3], psi[9, n // 2] = np.inf, -np.inf
    psi[12, n // 3] = psi[12, n // 4] = np.inf
    x = S.to_internal(psi)
    B = w[:, None] * K.T
    special = {1: np.inf, 2: -np.inf, 5: np.nan, 9: np.nan, 12: np.inf}
    for transpose in (0, 1):
        got, want = _apply(S, x, transpose), P.psi0 @ (B.T if transpose else B)
        for c, v in special.items():
            assert np.array_equal(got[c], np.full(n, v), equal_nan=True), c
        rest = [c for c in range(P.ncells) if c not in special]
        assert float((np.abs(got - want) / want)[rest].max()) <= 2 * EPS
    S.close()


# The solve's own error is that of FP64; a step adds the FP32 roundings of the collision-free part
# (four per face and six more, of positive terms: CFL 0.4) and of 1 / (1 + dt alpha_t sigma_t), whose
# rounding counts by that factor.
@pytest.mark.parametrize("npol,naz", [(16, 32), (12, 16), (20, 16), (10, 10), (13, 18)])
@pytest.mark.parametrize("kind", ["lit", "beam", "two decades"])
def test_imex_step_per_element(npol, naz, kind):
    from oracle import oracle as o
    omega, w = I.product_quadrature(npol, naz)
    K = I.henyey_greenstein_kernel(omega, w, 0.95)
    P, S = _solver(omega, w, K, lambda nc: _rows(kind, omega, nc, 305), "fp32")
    S.close()
    from paper_2205_08417_amd.solver import Solver
    s = (P.sigma_t * 10.0 / P.dt).astype(np.float32).astype(np.float64)
    P = dataclasses.replace(P, sigma_t=s, sigma_s=(0.9 * s).astype(np.float32).astype(np.float64))
    S = Solver(P, precision="fp32", reorder=False)
    out = torch.empty_like(S.initial_state())
    S.step_imex(S.initial_state(), out)
    got = out.cpu().numpy().astype(np.float64)
    S.close()
    want = o.step_imex(o.OracleProblem.from_problem(P), P.psi0, P.dt)
    err = float((np.abs(got - want) / want).max())
    bound = (4 * 3 + 6 + 1.0 + P.dt * P.sigma_t.max()) * EPS
    print(f"imex {npol}x{naz} {kind}: {err:.2e} of {bound:.2e}")
    assert got.min() > 0.0 and err <= bound


@pytest.mark.parametrize("npol,naz", [(16, 32), (12, 16), (10, 10)])
def test_dose_with_the_weights_of_another_rule_than_the_kernels(npol, naz):
    """A step whose ordinate set has other weights than the one its kernel was made with: dose and
    reverse dose take the step's (FP64 sums of FP32 states: 1e-12; the reverse one is stored in
    FP32)."""
    from paper_2205_08417_amd import snrt
    from paper_2205_08417_amd.solver import differentiable_rollout
    omega, w = I.product_quadrature(npol, naz)
    K = I.henyey_greenstein_kernel(omega, w, 0.8)
    P, S = _solver(omega, w, K, lambda nc: _rows("two", omega, nc, 306), "fp32")
    w2 = w * (1.0 + 0.3 * np.cos(np.arange(w.size)))
    own, S.quad = S.quad, snrt.snrt_quad_create(omega, w2)
    x = S.initial_state()
    outs = [torch.empty_like(x) for _ in range(2)]
    dose = torch.full((S.nc,), 0.25, dtype=torch.float64, device="cuda")
    S.step(x, outs[0])
    snrt.snrt_step_dose(S.mesh, S.quad, S.scatter, S.args(), x, outs[1], 0.37, dose, S.ws, S.ws_bytes)
    assert torch.equal(outs[0], outs[1])
    want = 0.25 + 0.37 * (P.psi0 @ w2)
    assert float(np.abs(dose.cpu().numpy() / want - 1.0).max()) <= 1e-12
    psi = x.clone().requires_grad_()
    rho = torch.ones(S.nc, device="cuda", requires_grad=True)
    _, D = differentiable_rollout(S, psi, 1, S.mats32["sigma_t"], S.mats32["sigma_s"], rho,
                                  ckpt_every=1, dose_coeff=[0.37])
    g = torch.linspace(0.5, 1.5, S.nc, dtype=torch.float64, device="cuda")
    torch.autograd.backward([D], [g])
    want = 0.37 * g.cpu().numpy()[:, None] * w2[None, :]
    assert float(np.abs(psi.grad.cpu().numpy() / want - 1.0).max()) <= 2 * EPS
    snrt.snrt_quad_destroy(S.quad)
    S.quad = own
    S.close()
