"""The dense, moment-form, dose and IMEX tests once more on operators without azimuthal modes.

Kernels of the angle on product rules run through azimuthal modes, so that those tests no longer reach
the general products with them, which every other kernel and rule takes.  Here the ordinates' azimuths
are turned by 1e-11 from one polar node to the next, and a kernel's entries are scaled by 1 + 1e-8 s_q
s_p, which keeps it symmetrisable: below every tolerance, and above what counts as the structure.  The
tests that compare with child processes run in a process with SNRT_AZIMUTH=0 instead.  That the general
products run is checked on their rounding: the modes have none of BF16's.
"""
import os
import subprocess
import sys

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from paper_2205_08417_amd import inputs as I  # noqa: E402
import test_gpu_dense  # noqa: E402
import test_gpu_dose_fused  # noqa: E402
import test_gpu_graph  # noqa: E402
import test_gpu_imex  # noqa: E402
import test_gpu_moments  # noqa: E402

HERE = os.path.dirname(os.path.abspath(__file__))
CHILDREN = ["test_imex_separate_passes_in_a_fresh_process"]
ISOTROPIC = ["test_imex_rollout", "test_imex_per_step_scalars_and_quads",
             "test_imex_full_size_checkerboard"]

for _m in (test_gpu_dense, test_gpu_dose_fused, test_gpu_graph, test_gpu_imex, test_gpu_moments):
    for _name, _f in list(vars(_m).items()):
        if _name.startswith("test_") and _name not in CHILDREN + ISOTROPIC and callable(_f):
            globals()[_name.replace("test_", f"test_general_{_m.__name__[9:]}_", 1)] = _f


def _turned(n_polar, n_azimuth, rule=I.product_quadrature):
    omega, w = rule(n_polar, n_azimuth)
    a = 1e-11 * np.repeat(np.arange(n_polar) * (-1.0) ** np.arange(n_polar), n_azimuth)
    x, y = omega[:, 0].copy(), omega[:, 1].copy()
    omega[:, 0], omega[:, 1] = x + a * y, y - a * x
    return omega, w


def _scaled(omega, w, g, normalise=True, kernel=I.henyey_greenstein_kernel):
    s = np.random.default_rng(331).uniform(-1.0, 1.0, len(w))
    return kernel(omega, w, g, normalise) * (1.0 + 1e-8 * s[:, None] * s[None, :])


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    from paper_2205_08417_amd import snrt
    snrt.lib()
    patch = pytest.MonkeyPatch()
    patch.setattr(I, "product_quadrature", _turned)
    patch.setattr(I, "henyey_greenstein_kernel", _scaled)
    yield
    patch.undo()


def _one_bf16_product(moments):
    """The error of a BF16 product (one product, no split) on 162 cells."""
    from _util import rel_l2, small_problem
    from oracle import moments as mo
    from paper_2205_08417_amd import snrt
    from paper_2205_08417_amd.solver import Solver
    omega, w = I.product_quadrature(16, 16)
    sig = I.hg_legendre_moments(0.8, 3) if moments else None
    K = mo.moment_kernel(omega, w, sig) if moments else I.henyey_greenstein_kernel(omega, w, 0.8)
    P = small_problem(I.jittered_delaunay_mesh(10, 0.0, 1.0, seed=332), omega_w=(omega, w), K=K)
    S = Solver(P, precision="bf16x1", moments=sig, reorder=False)
    x = S.initial_state()
    out = torch.empty_like(x)
    snrt.snrt_scatter_apply(S.mesh, S.quad, S.scatter, x, out, 0, S.ws, S.ws_bytes)
    S.close()
    return rel_l2(out.cpu().numpy(), x.cpu().numpy().astype(np.float64) @ (w[:, None] * K.T))


@pytest.mark.parametrize("moments", [False, True])
def test_the_general_products_run(moments):
    assert 1e-5 < _one_bf16_product(moments) < 1e-2


def _child(*args):
    """pytest on the named tests in a process without azimuthal modes."""
    script = ("import sys, pytest; sys.path.insert(0, %r); import test_gpu_general_products as t; "
              "assert 1e-5 < t._one_bf16_product(False) < 1e-2; "
              "sys.exit(pytest.main(sys.argv[1:]))" % HERE)
    r = subprocess.run([sys.executable, "-c", script, "-x", "-q", "-p", "no:cacheprovider", *args],
                       env=dict(os.environ, SNRT_AZIMUTH="0"), cwd=os.path.dirname(HERE),
                       capture_output=True, text=True, timeout=170)
    print(r.stdout[-2000:])
    assert r.returncode == 0, r.stdout[-2000:] + r.stderr[-2000:]


@pytest.mark.timeout(180)
def test_fused_steps_against_two_launches():
    _child(os.path.join(HERE, "test_gpu_step_fused.py"))


@pytest.mark.timeout(180)
@pytest.mark.parametrize("name", CHILDREN)
def test_separate_passes(name):
    _child(os.path.join(HERE, "test_gpu_imex.py") + "::" + name)
