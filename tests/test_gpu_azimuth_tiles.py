"""The azimuthal-mode kernels where a block takes several tiles of eight cells: what is fetched a tile
or two ahead (rows, records, materials, dose), the exchange buffer and the waves' corners used again,
gradients that two waves of a cell add a tile late, and a last tile that is partly empty.

Sampled cells of 21 218 triangles (2 652 tiles) and 21 315 quadrilaterals: more than two tiles for each
block that the device holds at once (256 compute units, at most five blocks each) and a cell count that
is no multiple of eight.  One shape of every family of the kernels: azimuthal classes, polar halves,
and ordinates per lane where the azimuths leave slots empty.

Tolerances: the product per element 2^-23 (test_gpu_azimuth_elements.py), which the general products
do not reach; states 1e-6 of the norm, gradients of sums of random sign ten times that.
"""
import dataclasses

import numpy as np
import pytest

from _util import rel_l2, small_problem

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from paper_2205_08417_amd import inputs as I  # noqa: E402

TOL = 1e-6
SHAPES = [(8, 16), (10, 10), (16, 15), (20, 16), (18, 7), (26, 9), (26, 13), (32, 15), (8, 32),
          (5, 20), (10, 20), (15, 24), (15, 26), (32, 32), (18, 22), (22, 28), (32, 30)]
MESHES = {}


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    assert torch.cuda.get_device_properties(0).multi_processor_count <= 256
    yield
    MESHES.clear()


def _mesh(kind):
    if kind not in MESHES:
        MESHES[kind] = (I.quad_grid_mesh(145, 147) if kind == "quads" else
                        I.jittered_delaunay_mesh(104, 0.0, 1.0, seed=321))
    return MESHES[kind]


def _part(P, seeds):
    """The problem on the sampled cells and their neighbours (cells first), whose far sides are cut."""
    m = P.mesh
    n = m.face_nbr[seeds]
    part = np.concatenate([seeds, np.setdiff1d(n[n >= 0], seeds)])
    to = np.full(m.ncells, -1)
    to[part] = np.arange(part.size)
    nbr = m.face_nbr[part]
    nbr = np.where(nbr >= 0, np.where(to[np.maximum(nbr, 0)] < 0, -1, to[np.maximum(nbr, 0)]), nbr)
    sub = dataclasses.replace(m, cells=m.cells[part], face_nbr=nbr.astype(np.int32),
                              face_normal=m.face_normal[part], area=m.area[part],
                              centroid=m.centroid[part], face_mid=None)
    cell = lambda a: None if a is None else a[part]  # noqa: E731
    return part, dataclasses.replace(P, mesh=sub, sigma_t=P.sigma_t[part], sigma_s=P.sigma_s[part],
                                     rho=cell(P.rho), source=cell(P.source), psi0=P.psi0[part])


def _setup(npol, naz, kind, rho):
    omega, w = I.product_quadrature(npol, naz)
    m = _mesh(kind)
    P = small_problem(m, omega_w=(omega, w), K=I.henyey_greenstein_kernel(omega, w, 0.9), seed=322,
                      rho=rho, source=True, inflow=True, scatter=(0.5, 1.0))
    psi = (10.0 ** (-2.0 * P.psi0)).astype(np.float32).astype(np.float64)
    rng = np.random.default_rng(323)
    seeds = np.unique(np.concatenate([[0, 1, 7, 8, m.ncells - 9, m.ncells - 2, m.ncells - 1],
                                      rng.choice(m.ncells, 60, replace=False)]))
    return dataclasses.replace(P, psi0=psi), seeds


@pytest.mark.parametrize("npol,naz", SHAPES)
@pytest.mark.parametrize("kind", ["triangles", "quads"])
def test_product_step_dose_and_transposed_step(npol, naz, kind):
    from oracle import oracle as o
    from paper_2205_08417_amd import snrt
    from paper_2205_08417_amd.solver import Solver, differentiable_rollout
    rho = kind == "quads" or npol == 32
    P, seeds = _setup(npol, naz, kind, rho)
    part, Q = _part(P, seeds)
    op, ns = o.OracleProblem.from_problem(Q), len(seeds)
    S = Solver(P, precision="fp32", reorder=False)
    x = S.initial_state()
    B = P.w[:, None] * P.K.T
    out = torch.empty_like(x)
    for transpose in (0, 1):
        snrt.snrt_scatter_apply(S.mesh, S.quad, S.scatter, x, out, transpose, S.ws, S.ws_bytes)
        got = out.cpu().numpy().astype(np.float64)
        want = P.psi0 @ (B.T if transpose else B)
        assert float((np.abs(got - want) / want).max()) <= 2.0 ** -23
    args = S.args(alpha_t=1.1, alpha_s=0.9, inflow_scale=0.6)
    out_d = torch.full_like(x, float("nan"))
    S.step(x, out, args)
    dose = torch.full((S.nc,), 0.25, dtype=torch.float64, device="cuda")
    snrt.snrt_step_dose(S.mesh, S.quad, S.scatter, args, x, out_d, 0.37, dose, S.ws, S.ws_bytes)
    assert torch.equal(out, out_d)
    want = o.step(op, Q.psi0, P.dt, 1.1, 0.9, 0.6)[:ns]
    assert rel_l2(out.cpu().numpy()[seeds], want) <= TOL
    dref = 0.25 + 0.37 * (P.psi0 @ P.w) / (P.rho if rho else 1.0)
    assert rel_l2(dose.cpu().numpy(), dref) <= TOL
    # the transposed step and its gradients
    lam = np.random.default_rng(324).standard_normal((P.ncells, P.nq)).astype(np.float32)
    lam = lam.astype(np.float64)
    l1, l0 = S.to_internal(lam), torch.full_like(x, float("nan"))
    g = [torch.full((S.nc,), 0.5, device="cuda") for _ in range(3)]
    S.adjoint_step(x, l1, l0, g[0], g[1], g[2] if rho else None, S.args(alpha_t=1.2, alpha_s=0.8))
    ref = [np.full(len(part), 0.5) for _ in range(3)]
    want = o.adjoint_step(op, Q.psi0, lam[part], P.dt, 1.2, 0.8, ref[0], ref[1],
                          ref[2] if rho else None)[:ns]
    assert rel_l2(l0.cpu().numpy()[seeds], want) <= TOL
    for a, b in zip(g[:3 if rho else 2], ref):
        assert rel_l2(a.cpu().numpy()[seeds] - 0.5, b[:ns] - 0.5) <= 10 * TOL
    # a reverse step with the dose functional: FP64 gradients, dJ/dD added to the state
    leaf = [t.clone().requires_grad_() for t in (x, S.mats32["sigma_t"], S.mats32["sigma_s"])]
    dens = torch.ones(S.nc, device="cuda")
    if rho:
        dens = (1.0 / S.mats32["inv_rho"]).contiguous().requires_grad_()
    end, D = differentiable_rollout(S, leaf[0], 1, leaf[1], leaf[2], dens if rho else None,
                                    ckpt_every=1, dose_coeff=[0.37])
    gd = torch.linspace(-1.0, 1.0, S.nc, dtype=torch.float64, device="cuda")
    torch.autograd.backward([end, D], [l1, gd])
    ref = [np.zeros(len(part)) for _ in range(3)]
    want = o.adjoint_step(op, Q.psi0, lam[part], P.dt, 1.0, 1.0, ref[0], ref[1],
                          ref[2] if rho else None)
    want = want + (0.37 * gd.cpu().numpy()[part] / (Q.rho if rho else 1.0))[:, None] * P.w[None, :]
    assert rel_l2(leaf[0].grad.cpu().numpy()[seeds], want[:ns]) <= TOL
    for a, b in zip(leaf[1:], ref):
        assert rel_l2(a.grad.cpu().numpy()[seeds], b[:ns]) <= 10 * TOL
    S.close()


# FP64 modes (FP32 handles) and FP32 modes (the others); one material, so that the solve is one system.
# Stiff: dt sigma = 10, whose factor 1 / (1 + 10) is rounded once: ten roundings more.
@pytest.mark.parametrize("npol,naz", SHAPES)
@pytest.mark.parametrize("kind", ["triangles", "quads"])
def test_imex_step(npol, naz, kind):
    from oracle import oracle as o
    from paper_2205_08417_amd.solver import Solver
    rho = kind == "triangles"
    P, seeds = _setup(npol, naz, kind, rho)
    s = float(np.float32(10.0 / P.dt))
    P = dataclasses.replace(P, sigma_t=np.full(P.ncells, s), sigma_s=np.full(P.ncells, 0.5 * s))
    part, Q = _part(P, seeds)
    free = dataclasses.replace(Q, sigma_t=0.0 * Q.sigma_t, sigma_s=0.0 * Q.sigma_s)
    r = o.step(o.OracleProblem.from_problem(free), Q.psi0, P.dt, 1.0, 1.0, 0.6)[:len(seeds)]
    st = P.dt * s
    want = np.linalg.solve((1.0 + st) * np.eye(P.nq) - 0.5 * st * P.K * P.w[None, :], r.T).T
    for precision in ["fp32"] + (["bf16x3"] if P.nq % 32 == 0 else []):
        S = Solver(P, precision=precision, reorder=False)
        x = S.initial_state()
        out = torch.full_like(x, float("nan"))
        S.step_imex(x, out, S.args(inflow_scale=0.6))
        err = rel_l2(out.cpu().numpy()[seeds], want)
        print(f"imex {npol}x{naz} {kind} {precision}: {err:.2e}")
        S.close()
        assert err <= 2 * TOL
