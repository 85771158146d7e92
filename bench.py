"""Throughput of the explicit S_N step on one MI355X.

Workload (default): the FP32 isotropic checkerboard -- seeded Delaunay mesh of 316 x 316
jittered points on [0, 7]^2 (198 450 triangles), 16 x 16 product quadrature (256 ordinates),
absorbers sigma_t = 10 in a checker pattern, source q = 1 in the centre square, vacuum
boundary, explicit Euler at CFL 0.5.  A step is one call of the library's step (upwind
flux over every face and ordinate, isotropic scattering, absorption, source) on states
resident in HBM.

Prints one JSON line: cell-ordinate updates/s over the timed steps, the roofline of the step
kernel (algorithmic bytes / measured kernel time vs 8 TB/s, and vs a measured device copy),
and the FP64 oracle timed on the host cores over a bounded sample of the same workload.
Further sections time the other paths on their own workloads: adjoint/forward, the dense BF16
hi+lo product (line source), the CSD dose step, moment-projected scattering, the
second-order Heun step, the IMEX step and the P_N solver step (P_5).

Usage: python bench.py [--gpus 1] [--steps K] [--warmup W] [--graph] [--no-cpu-baseline]
"""
from __future__ import annotations

import argparse
import hashlib
import json
import os
import sys
import time

ROOT = os.path.dirname(os.path.abspath(__file__))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)

METRIC = "cell-ordinate updates/s per S_N step (FP32 vs mixed) + adjoint/forward ratio"
HBM_PEAK_GBS = 8000.0           # MI355X HBM3E, vendor figure
BF16_PEAK_TFLOPS = 2500.0       # MI355X dense BF16 MFMA, vendor figure
FP32_VECTOR_PEAK_TFLOPS = 157.3 # MI355X FP32 vector, vendor figure
FP32_MFMA_PEAK_TFLOPS = 157.3   # MI355X dense FP32 MFMA, vendor figure
DENSE_WORKLOAD = "linesource_hg_s32"
WORKLOAD = "checkerboard_s16"
STEP_SOURCES = [os.path.join(ROOT, "paper_2205_08417_amd", "csrc", f)
                for f in ("sn_step_kernels.h", "sn_step_f32.hip")]
TRAFFIC_FILE = os.path.join(ROOT, "profiles", "sn_step_checkerboard_s16_traffic.json")


def kernel_source_sha() -> str:
    """Hash of the step kernel's sources: counter figures are only reused for this source."""
    h = hashlib.sha256()
    for f in STEP_SOURCES:
        h.update(open(f, "rb").read())
    return h.hexdigest()[:16]


def measured_traffic():
    """HBM bytes per launch from the committed rocprofv3 counter runs, if they were taken on
    the current step kernel source (else None)."""
    try:
        d = json.load(open(TRAFFIC_FILE))
    except (OSError, ValueError):
        return None
    if d.get("kernel_source_sha") != kernel_source_sha():
        return None
    return d.get("traffic_bytes_per_launch")


def cpu_baseline(P, budget_s: float = 36.0):
    """Oracle (FP64, OpenMP over cells) on the same mesh and quadrature: as many steps from
    the workload's initial state as fit the time budget (at least 2, at most 1000 in all).
    Also returns the oracle's state and its step count, for the parity figure."""
    from oracle import oracle as o
    op = o.OracleProblem.from_problem(P)
    psi = P.psi0
    t0 = time.perf_counter()
    psi = o.step(op, psi, P.dt)
    t1 = time.perf_counter() - t0
    n = max(2, min(999, int(budget_s / max(t1, 1e-6))))
    t0 = time.perf_counter()
    for _ in range(n):
        psi = o.step(op, psi, P.dt)
    el = time.perf_counter() - t0
    reference = (n + 1, psi)
    out = {"value": P.ncells * P.nq * n / el, "unit": "cell-ordinate updates/s",
           "cores": o.num_threads(), "cpu_model": host_cpu_model(), "kind": "oracle",
           "sample": f"{n} FP64 oracle steps of the full {WORKLOAD} workload "
                     f"({P.ncells} cells x {P.nq} ordinates), {el:.1f} s wall"}
    # the same oracle on one host thread, over a shorter sample
    prev = o.set_num_threads(1)
    try:
        n1 = max(1, min(n, int(0.25 * budget_s / max(el / n, 1e-6) / out["cores"])))
        t0 = time.perf_counter()
        for _ in range(n1):
            psi = o.step(op, psi, P.dt)
        el1 = time.perf_counter() - t0
    finally:
        o.set_num_threads(prev)
    out["single_thread"] = {"value": P.ncells * P.nq * n1 / el1, "cores": 1,
                            "sample": f"{n1} steps, {el1:.1f} s wall"}
    return out, reference


def host_cpu_model() -> str:
    """The host CPU's model name (from /proc/cpuinfo; empty if unavailable)."""
    try:
        for line in open("/proc/cpuinfo"):
            if line.startswith("model name"):
                return line.split(":", 1)[1].strip()
    except OSError:
        pass
    return ""


def sample_cells(nc: int, n: int = 256, seed: int = 0):
    import numpy as np
    return np.sort(np.random.default_rng(seed).choice(nc, min(n, nc), replace=False))


def oracle_error(got_rows, ref_rows, what: str) -> dict:
    """Error of GPU rows against the oracle's rows for the same cells and input state."""
    import numpy as np
    got = np.asarray(got_rows, dtype=np.float64)
    ref = np.asarray(ref_rows, dtype=np.float64)
    nr = float(np.linalg.norm(ref))
    return {"rel_l2": float(np.linalg.norm(got - ref)) / (nr if nr > 0 else 1.0),
            "max_abs_over_max_ref": float(np.max(np.abs(got - ref)) /
                                          max(float(np.max(np.abs(ref))), 1e-300)),
            "check": what}


def step_vs_oracle(S, psi, oracle_fn, n: int = 256, seed: int = 0,
                   step=None, what: str = "one step") -> dict:
    """One more step of the GPU path from the section's final state ``psi`` (internal order)
    against the FP64 oracle's step from the same state, on ``n`` seeded cells."""
    import torch
    out = torch.empty_like(psi)
    (step or S.step)(psi, out)
    cells = sample_cells(S.nc, n, seed)
    got = S.to_user(out).cpu().numpy()[cells]
    start = S.to_user(psi).cpu().numpy().astype("float64")
    ref = oracle_fn(start, cells)
    return oracle_error(got, ref, f"{what} from the final state, {cells.size} seeded cells")


def timed(fn, n, stream):
    """Average milliseconds of ``fn`` over n calls, bracketed by events on ``stream``."""
    import torch
    start, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    start.record(stream)
    for _ in range(n):
        fn()
    end.record(stream)
    torch.cuda.synchronize()
    return start.elapsed_time(end) / n


def product_rate(S, psi, reps: int = 10, passes: int = 3, kernel: str = "k_gemm_bf16",
                 peak: float = None):
    """Rate of the scattering product on state psi.  ``passes`` 0: through azimuthal modes
    (k_az_product: one read and one write of the state).  Else the executed TFLOP/s of a general
    product: BF16 or FP16 split (two or three passes, against the BF16 MFMA peak) or FP32 (one pass,
    FP32 MFMA peak)."""
    import torch
    from paper_2205_08417_amd import snrt
    peak = BF16_PEAK_TFLOPS if peak is None else peak
    sbuf = torch.empty_like(psi)
    stream = torch.cuda.current_stream()
    apply = lambda: snrt.snrt_scatter_apply(S.mesh, S.quad, S.scatter, psi, sbuf, 0, S.ws,  # noqa
                                            S.ws_bytes)
    apply()
    torch.cuda.synchronize()
    ms = timed(apply, reps, stream)
    if passes == 0:
        gbs = 2.0 * psi.element_size() * S.nc * S.nq / (ms * 1e-3) / 1e9
        return {"kernel": "k_az_product", "ms": ms, "gbs": gbs, "hbm_frac": gbs / HBM_PEAK_GBS}
    tflops = passes * 2.0 * S.nc * S.nq * S.nq / (ms * 1e-3) / 1e12
    return {"kernel": kernel, "ms": ms, "executed_tflops": tflops,
            "peak_tflops": peak, "mfma_utilization": tflops / peak}


def modes_on() -> bool:
    """Whether azimuth-invariant kernels run through azimuthal modes (read once per process)."""
    return os.environ.get("SNRT_AZIMUTH", "1") != "0"


MODES = ("FP64 azimuthal modes, S rounded to FP32 once (whatever the handle's precision: the kernel "
         "depends on the angle only, on a product rule)")


def arithmetic(general: str) -> str:
    """What the scattering product of a kernel of the angle is computed in; ``general``: the
    arithmetic of the general product of the handle's precision."""
    return MODES if modes_on() else general


def unstructured(P):
    """The same problem with a kernel that is not a function of the angle: its entries times 1 + 1e-8
    s_q s_p for random s, which the general products then run (nothing else changes above their
    rounding)."""
    import dataclasses
    import numpy as np
    s = np.random.default_rng(0).uniform(-1.0, 1.0, P.nq)
    return dataclasses.replace(P, K=P.K * (1.0 + 1e-8 * s[:, None] * s[None, :]))


def step_form(general: bool = False) -> str:
    """How the library runs an explicit dense step (SNRT_AZIMUTH, SNRT_STEP_FUSED, read once per
    process); ``general``: of an operator without azimuthal modes."""
    fused = os.environ.get("SNRT_STEP_FUSED", "1") != "0"
    if modes_on() and not general:
        return ("one launch: k_az_step, the scattering product through azimuthal modes and the "
                "update of the same cells" if fused else
                "two launches: k_az_product into the workspace, then k_step")
    if not fused:
        return "two launches: scattering product into the workspace, then k_step"
    return ("one launch: k_gemm_step, the scattering product whose tiles run the update of "
            "their cells and ordinates (triangles, nq % 256 == 0, BF16/FP16 products)")


def transposed_step_form() -> str:
    """How the library runs a dense transposed step (the same switches as the forward)."""
    fused = os.environ.get("SNRT_STEP_FUSED", "1") != "0"
    if not fused:
        return (f"two launches: transposed {'k_az_product' if modes_on() else 'product'} into the "
                "workspace, then k_adjoint_p, and the dose functional's term in a pass of its own")
    if modes_on():
        return ("one launch: k_az_adjoint, the transposed product through azimuthal modes, the "
                "update (with the dose functional's term) and the gradient sums")
    return ("one launch: k_gemm_adjoint, the transposed product whose tiles run the adjoint "
            "update (with the dose functional's term) of their cells and ordinates, then "
            "k_adjoint_fold adding the per-piece gradient sums")


def bench_dense(steps, warmup: int):
    """Anisotropic HG line source (100 352 cells x 1024 ordinates): the step as the library runs it
    (through azimuthal modes), then with the general scattering product in each mixed precision (BF16
    hi+lo in three and two products, FP16 hi+lo in three) and in FP32, on the same kernel without its
    azimuthal structure.  Each run but FP32's is timed over the whole 200-step workload from the
    initial pulse (steps=None; warm-up steps run on a separate copy first): early states are
    mostly exact zeros, on which the matrix cores draw less power and clock higher, so a
    window of early steps alone would flatter the rate.  The products' rates are
    measured on the run's final state and on a dense random state; every run's final
    state then takes one more step whose sampled cells are checked against the FP64 oracle."""
    import torch
    from oracle import oracle as o
    from paper_2205_08417_amd import inputs as I
    from paper_2205_08417_amd.solver import Solver

    P = I.build(DENSE_WORKLOAD)
    nsteps = P.nsteps if steps is None else steps
    general = unstructured(P)
    op = o.OracleProblem.from_problem(P)
    stream = torch.cuda.current_stream()

    def whole_run(precision, nrun, warm, Q=general):
        S = Solver(Q, precision=precision)
        args = S.args()
        st = [S.initial_state(), None]
        st[1] = torch.empty_like(st[0])

        def one_step():
            S.step(st[0], st[1], args)
            st.reverse()

        for _ in range(warm):
            one_step()
        st[0] = S.initial_state()
        torch.cuda.synchronize()
        return S, st[0], timed(one_step, nrun, stream)

    def oracle_rows(start, cells):
        return o.step(op, start, P.dt, cells=cells)

    out = {"workload": DENSE_WORKLOAD, "cells": P.ncells, "ordinates": P.nq,
           "scattering": "Henyey-Greenstein g=0.9, dense, column-normalised", "steps": nsteps,
           "unit": "cell-ordinate updates/s", "step_form": step_form()}
    # the headline figures of the section: the step as the library runs it
    S, final, ms = whole_run("bf16x3", nsteps, warmup, P)
    passes = 0 if modes_on() else 3
    vs = step_vs_oracle(S, final, oracle_rows)
    out.update({"precision": arithmetic("BF16 hi+lo, three products, FP32 accumulate"),
                "ms_per_step": ms, "value": P.ncells * P.nq / (ms * 1e-3),
                "scatter_product": product_rate(S, final, passes=passes),
                "scatter_product_dense_random_state":
                    product_rate(S, torch.rand_like(final), passes=passes),
                "vs_oracle": vs, "rel_l2_vs_oracle": vs["rel_l2"]})
    reference = final.clone()
    S.close()
    out["general_kernel"] = "the same kernel, its entries times 1 + 1e-8 s_q s_p"
    out["general_step_form"] = step_form(general=True)
    for precision, label in (("bf16x3", "BF16 hi+lo, three products"),
                             ("bf16x2", "BF16, operand hi+lo and state once: two products"),
                             ("fp16x3", "FP16 hi+lo with per-row power-of-2 scaling, three "
                                        "products")):
        S, final, ms = whole_run(precision, nsteps, warmup if precision == "bf16x3" else 3)
        passes = 2 if precision == "bf16x2" else 3
        kernel = "k_gemm_f16" if precision == "fp16x3" else "k_gemm_bf16"
        out[precision] = {
            "precision": label, "ms_per_step": ms, "steps": nsteps,
            "value": P.ncells * P.nq / (ms * 1e-3),
            "scatter_product": product_rate(S, final, passes=passes, kernel=kernel),
            "scatter_product_dense_random_state":
                product_rate(S, torch.rand_like(final), passes=passes, kernel=kernel),
            "vs_oracle": step_vs_oracle(S, final, oracle_rows),
            "rel_l2_vs_headline_final_state":
                float(torch.linalg.vector_norm((final - reference).double()) /
                      torch.linalg.vector_norm(reference.double()))}
        S.close()
    # the same step with the FP32 scattering product (on the matrix cores), 20 steps from the
    # initial state: the FP32 side of the FP32-vs-mixed comparison
    S32, final32, ms32 = whole_run("fp32", 20, 1)
    out["fp32"] = {"precision": "FP32", "ms_per_step": ms32, "steps": 20,
                   "scatter_product": product_rate(S32, final32, passes=1, kernel="k_gemm_f32",
                                                   peak=FP32_MFMA_PEAK_TFLOPS),
                   "vs_oracle": step_vs_oracle(S32, final32, oracle_rows)}
    S32.close()
    out["imex_dense"] = bench_imex_dense(P, op, nsteps, warmup)
    return out


def bench_imex_dense(P, op, nsteps: int, warmup: int):
    """IMEX steps with the dense HG kernel (implicit collisions through the kernel's
    eigendecomposition: collision-free step, V^-1, per-cell diagonal, V diag(lam), combine; one launch
    through azimuthal modes), a BF16x3 handle, over the whole run from the initial pulse; the
    one-time host set-up is timed on its own."""
    import time
    import torch
    from oracle import oracle as o
    from paper_2205_08417_amd.solver import Solver

    S = Solver(P, precision="bf16x3")
    t0 = time.perf_counter()
    S.prepare_implicit()
    torch.cuda.synchronize()
    setup_s = time.perf_counter() - t0
    args = S.args()
    st = [S.initial_state(), None]
    st[1] = torch.empty_like(st[0])

    def one_step():
        S.step_imex(st[0], st[1], args)
        st.reverse()

    for _ in range(min(warmup, 3)):
        one_step()
    st[0] = S.initial_state()
    torch.cuda.synchronize()
    ms = timed(one_step, nsteps, torch.cuda.current_stream())
    vs = step_vs_oracle(S, st[0], lambda start, c: o.step_imex(op, start, P.dt, cells=c), n=32,
                        step=lambda a_, b_: S.step_imex(a_, b_, args), what="one IMEX step")
    S.close()
    return {"precision": "FP32 azimuthal modes" if modes_on() else
                         "BF16 hi+lo, three products, FP32 accumulate",
            "steps": nsteps, "ms_per_step": ms,
            "value": P.ncells * P.nq / (ms * 1e-3), "setup_s": setup_s,
            "note": "implicit HG collisions through one eigendecomposition of K W (host FP64, "
                    "set-up), " + ("per azimuthal mode in one launch (k_az_imex)" if modes_on() else
                                   "two nq x nq products per step"),
            "vs_oracle": vs, "rel_l2_vs_oracle": vs["rel_l2"]}


def library_gemm_ceiling(M: int, nq: int, reps: int = 10):
    """Context only (not the product path): hipBLASLt BF16 GEMM of the scattering product's
    shape through torch.matmul, in TFLOP/s of its single product."""
    import torch
    a = torch.randn(M, nq, device="cuda", dtype=torch.bfloat16)
    b = torch.randn(nq, nq, device="cuda", dtype=torch.bfloat16)
    stream = torch.cuda.current_stream()
    torch.matmul(a, b)
    torch.cuda.synchronize()
    ms = timed(lambda: torch.matmul(a, b), reps, stream)
    return 2.0 * M * nq * nq / (ms * 1e-3) / 1e12


def copy_ceiling(nbytes: int, reps: int = 20, passes: int = 3):
    """Measured bandwidth ceilings, GB/s of read + write, for a copy of one state:
    (the library's nontemporal stream copy, run ping-pong like the step so that each copy
    reads the previous one's output, best of ``passes``; the runtime's device-to-device
    copy of torch's ``copy_``)."""
    import torch
    from paper_2205_08417_amd import snrt
    src = torch.ones(nbytes // 4, dtype=torch.float32, device="cuda")
    dst = torch.empty_like(src)
    stream = torch.cuda.current_stream()
    bufs = [src, dst]

    def pingpong():
        snrt.snrt_stream_copy(bufs[0], bufs[1], nbytes, stream.cuda_stream)
        bufs.reverse()

    for _ in range(3):
        pingpong()
    torch.cuda.synchronize()
    ms = min(timed(pingpong, reps, stream) for _ in range(passes))
    dst.copy_(src)
    torch.cuda.synchronize()
    ms_rt = timed(lambda: dst.copy_(src), reps, stream)
    return 2.0 * nbytes / (ms * 1e-3) / 1e9, 2.0 * nbytes / (ms_rt * 1e-3) / 1e9


def bench_csd(steps, warmup: int):
    """CSD dose workload: phantom of 388 x 388 points (299 538 cells), 16 x 32 = 512
    ordinates, HG g=0.95, densities in the streaming, the beam
    inflow scaled by S(E_n) G_E(E_n) at every energy step and the FP64 dose accumulated
    before every step.  The whole 500-step energy run is timed (steps=None; warm-up steps
    run on a separate copy first); the product's rate is measured on the final
    state and on a dense random state.  The general mixed-precision products run the same energy steps
    on the kernel without its azimuthal structure."""
    import torch
    from paper_2205_08417_amd import inputs as I
    from paper_2205_08417_amd import snrt
    from paper_2205_08417_amd.solver import Solver

    P = I.build("csd_phantom_s512")
    nsteps = P.nsteps if steps is None else min(steps, P.nsteps)
    S = Solver(P, precision="bf16x3")
    isc, coeff = P.meta["inflow_scale"], P.meta["dose_coeff"]
    args = [S.args(inflow_scale=float(isc[n])) for n in range(nsteps)]
    state = [S.initial_state(), None]
    state[1] = torch.empty_like(state[0])
    dose = torch.zeros(S.nc, dtype=torch.float64, device="cuda")
    stream = torch.cuda.current_stream()
    inv_rho = S.mats32["inv_rho"]
    counter = [0]

    def fused_step():
        n = counter[0]
        snrt.snrt_step_dose(S.mesh, S.quad, S.scatter, args[n], state[0], state[1],
                            float(coeff[n]), dose, S.ws, S.ws_bytes)
        state.reverse()
        counter[0] = n + 1

    def separate_step():
        n = counter[0]
        snrt.snrt_dose_accumulate(S.mesh, S.quad, state[0], inv_rho, float(coeff[n]), dose)
        S.step(state[0], state[1], args[n])
        state.reverse()
        counter[0] = n + 1

    def run(one_step):
        counter[0] = 0
        for _ in range(min(warmup, nsteps)):
            one_step()
        counter[0] = 0
        state[0] = S.initial_state()
        dose.zero_()
        torch.cuda.synchronize()
        return timed(one_step, nsteps, stream)

    ms_separate = run(separate_step)
    ms_step = run(fused_step)
    passes = 0 if modes_on() else 3
    final = product_rate(S, state[0], passes=passes)
    dense = product_rate(S, torch.rand_like(state[0]), passes=passes)
    dose_ref = dose.clone()
    from oracle import oracle as o
    op = o.OracleProblem.from_problem(P)
    last = nsteps - 1
    vs_oracle = step_vs_oracle(
        S, state[0], lambda start, cells: o.step(op, start, P.dt, inflow_scale=float(isc[last]),
                                                 cells=cells),
        step=lambda a_, b_: S.step(a_, b_, args[last]))
    S.close()
    # the general products over the same energy run: their doses against the one above
    general = unstructured(P)

    def general_run(precision):
        S2 = Solver(general, precision=precision)
        args2 = [S2.args(inflow_scale=float(isc[n])) for n in range(nsteps)]
        st = [S2.initial_state(), None]
        st[1] = torch.empty_like(st[0])
        d = torch.zeros(S2.nc, dtype=torch.float64, device="cuda")

        def one_step():
            n = counter[0]
            snrt.snrt_step_dose(S2.mesh, S2.quad, S2.scatter, args2[n], st[0], st[1],
                                float(coeff[n]), d, S2.ws, S2.ws_bytes)
            st.reverse()
            counter[0] = n + 1

        counter[0] = 0
        for _ in range(min(warmup, 5, nsteps)):
            one_step()
        counter[0] = 0
        st[0] = S2.initial_state()
        d.zero_()
        torch.cuda.synchronize()
        ms = timed(one_step, nsteps, stream)
        S2.close()
        return {"ms_per_step": ms, "step_form": step_form(general=True),
                "dose_rel_l2_vs_headline": float(torch.linalg.vector_norm(d - dose_ref) /
                                                 torch.linalg.vector_norm(dose_ref))}

    return {"workload": "csd_phantom_s512", "cells": P.ncells, "ordinates": P.nq,
            "scattering": "Henyey-Greenstein g=0.95, dense, column-normalised",
            "precision": arithmetic("BF16 hi+lo, three products, FP32 accumulate"), "steps": nsteps,
            "energy_MeV": [float(P.meta["energy"][0]), float(P.meta["energy"][nsteps - 1])],
            "value": P.ncells * P.nq / (ms_step * 1e-3), "unit": "cell-ordinate updates/s",
            "ms_per_step": ms_step,
            "note": "a step = snrt_step_dose: the scattering product, the flux/update and the "
                    "dose of the step's input",
            "step_form": step_form(),
            "ms_per_step_separate_dose_pass": ms_separate,
            "scatter_product": final, "scatter_product_dense_random_state": dense,
            "vs_oracle": vs_oracle, "rel_l2_vs_oracle": vs_oracle["rel_l2"],
            "general_kernel": "the same kernel, its entries times 1 + 1e-8 s_q s_p",
            **{p: general_run(p) for p in ("bf16x3", "bf16x2", "fp16x3")}}


def bench_dose_gradient(nsteps: int = 500, ckpt: int = 20):
    """Gradient of the target-minus-organ dose functional w.r.t. the per-cell density on
    the full CSD phantom (299 538 cells x 512 ordinates, the first 500 energy steps, checkpoints
    every 20): the differentiable rollout's forward pass (steps with the
    fused dose) against its backward pass (segment recompute, transposed steps with the
    transposed product and the dose's adjoint terms), each one library call."""
    import numpy as np
    import torch
    from paper_2205_08417_amd import inputs as I
    from paper_2205_08417_amd.solver import Solver, differentiable_rollout

    P = I.build("csd_phantom_s512")
    n = min(nsteps, P.nsteps)
    S = Solver(P, precision="bf16x3")
    isc = np.asarray(P.meta["inflow_scale"][:n])
    coeff = np.asarray(P.meta["dose_coeff"][:n])
    T = P.meta["target"].astype(float)
    O = P.meta["organ"].astype(float)
    wd = S.cells_to_internal(P.mesh.area * (T - O), torch.float64)
    r = S.cells_to_internal(P.rho).requires_grad_(True)
    psi0 = S.initial_state()
    stream = torch.cuda.current_stream()

    def one_pass():
        ev = [torch.cuda.Event(enable_timing=True) for _ in range(4)]
        torch.cuda.synchronize()
        ev[0].record(stream)
        _, dose = differentiable_rollout(S, psi0, n, rho=r, ckpt_every=ckpt, inflow_scale=isc,
                                         dose_coeff=coeff)
        ev[1].record(stream)
        J = torch.sum(wd * dose)
        ev[2].record(stream)
        J.backward()
        ev[3].record(stream)
        torch.cuda.synchronize()
        r.grad = None
        return ev[0].elapsed_time(ev[1]), ev[2].elapsed_time(ev[3])

    one_pass()
    fwd, bwd = one_pass()
    S.close()
    return {"workload": "csd_phantom_s512", "cells": P.ncells, "ordinates": P.nq, "steps": n,
            "checkpoint_every": ckpt,
            "precision": arithmetic("BF16 hi+lo, three products, FP32 accumulate"),
            "functional": "sum_T A D - sum_O A D, gradient w.r.t. per-cell density",
            "forward_ms": fwd, "backward_ms": bwd, "adjoint_forward_ratio": bwd / fwd,
            "step_form": step_form(), "transposed_step_form": transposed_step_form(),
            "parity": "the same path on the reduced CSD workload over the whole energy range, "
                      "and one transposed step on this full phantom, are checked against the "
                      "oracle in tests/test_gpu_fullsize.py"}


def bench_moments(steps, warmup: int, degree: int = 8):
    """Moment-projected scattering (eq. SNEqns2) on the HG line source (100 352 cells x
    1024 ordinates), HG g=0.9 to degree 8 (81 moments): the step rate over the whole 200-step run (steps=None) against the
    dense-kernel step of the same workload; then the same number of IMEX steps (implicit
    moment-form collisions).  Both run through azimuthal modes; with SNRT_AZIMUTH=0 through two
    products by way of the moments, padded to 96 for the MFMA kernel (BF16 hi+lo)."""
    import torch
    from paper_2205_08417_amd import inputs as I
    from paper_2205_08417_amd.solver import Solver

    P = I.build(DENSE_WORKLOAD)
    steps = P.nsteps if steps is None else steps
    sig = I.hg_legendre_moments(0.9, degree)
    S = Solver(P, precision="bf16x3", moments=sig)
    state = [S.initial_state(), None]
    state[1] = torch.empty_like(state[0])
    args = S.args()
    stream = torch.cuda.current_stream()

    def one_step():
        S.step(state[0], state[1], args)
        state.reverse()

    for _ in range(warmup):
        one_step()
    state[0] = S.initial_state()
    torch.cuda.synchronize()
    ms = timed(one_step, steps, stream)

    def one_imex():
        S.step_imex(state[0], state[1], args)
        state.reverse()

    state[0] = S.initial_state()
    for _ in range(min(warmup, 5)):
        one_imex()
    state[0] = S.initial_state()
    torch.cuda.synchronize()
    ms_imex = timed(one_imex, steps, stream)
    from oracle import moments as mo
    from oracle import oracle as o
    op = o.OracleProblem.from_problem(P, K=mo.moment_kernel(P.omega, P.w, sig))
    vs_oracle = step_vs_oracle(S, state[0], lambda st_, c: o.step(op, st_, P.dt, cells=c))
    vs_oracle_imex = step_vs_oracle(S, state[0],
                                    lambda st_, c: o.step_imex(op, st_, P.dt, cells=c), n=64,
                                    step=lambda a_, b_: S.step_imex(a_, b_, args),
                                    what="one IMEX step")
    nm = (degree + 1) ** 2
    products = {}
    if not modes_on():
        mid = ((nm + 31) // 32) * 32                     # the library's BF16 padding (K chunk)
        tile = ((mid + 127) // 128) * 128                # product 1's output tile width
        products = {"moment_dimension_padded": mid,      # two products, three BF16 passes
                    "product_flops_executed": 3 * 2.0 * P.ncells * P.nq * (tile + mid),
                    "product_flops_useful": 2 * 2.0 * P.ncells * P.nq * nm}
    S.close()
    return {"workload": DENSE_WORKLOAD, "cells": P.ncells, "ordinates": P.nq,
            "scattering": f"moment-projected O Sigma M, HG g=0.9, degree {degree} ({nm} moments)",
            "precision": arithmetic("BF16 hi+lo, three products, FP32 accumulate"),
            "imex_precision": "FP32 azimuthal modes" if modes_on() else
                              "BF16 hi+lo, three products, FP32 accumulate",
            "steps": steps, "ms_per_step": ms, "step_form": step_form(),
            "value": P.ncells * P.nq / (ms * 1e-3), "unit": "cell-ordinate updates/s",
            **products, "imex_ms_per_step": ms_imex,
            "vs_oracle": vs_oracle, "rel_l2_vs_oracle": vs_oracle["rel_l2"],
            "imex_vs_oracle": vs_oracle_imex}


def bench_second_order(steps: int, warmup: int):
    """Second-order scheme on the headline checkerboard (198 450 cells x 256 ordinates,
    isotropic, FP32): one Heun step = two stages, each one launch that keeps the limited
    gradients in LDS.  Algorithmic bytes per step: a stage reads psi and writes its result
    (8 B per update), the final one also reads psi^n (4 B): 20 B per update, plus 96 B of
    geometry per cell and stage."""
    import torch
    from paper_2205_08417_amd import inputs as I
    from paper_2205_08417_amd.solver import Solver

    P = I.build(WORKLOAD)
    S = Solver(P)
    state = [S.initial_state(), None]
    state[1] = torch.empty_like(state[0])
    args = S.args()
    stream = torch.cuda.current_stream()

    def run(limiter):
        def one_step():
            S.step2(state[0], state[1], args, limiter=limiter)
            state.reverse()

        for _ in range(warmup):
            one_step()
        torch.cuda.synchronize()
        return timed(one_step, steps, stream)

    ms = run("barth-jespersen")
    ms_vk = run("venkatakrishnan")
    alg = P.ncells * (20 * P.nq + 2 * 96)
    from oracle import oracle as o
    op = o.OracleProblem.from_problem(P)
    # the oracle's Heun step is taken over the whole state (it has no cell selection)
    vs_oracle = step_vs_oracle(S, state[0], lambda st_, c: o.step2(op, st_, P.dt)[c],
                               step=lambda a_, b_: S.step2(a_, b_, args),
                               what="one Heun step (Barth-Jespersen)")
    S.close()
    return {"workload": WORKLOAD, "cells": P.ncells, "ordinates": P.nq,
            "scheme": "second order: Green-Gauss + Barth-Jespersen reconstruction, Heun",
            "steps": steps, "ms_per_step": ms, "value": P.ncells * P.nq / (ms * 1e-3),
            "unit": "cell-ordinate updates/s", "algorithmic_bytes_per_step": alg,
            "achieved_gbs": alg / (ms * 1e-3) / 1e9,
            "hbm_frac": alg / (ms * 1e-3) / 1e9 / HBM_PEAK_GBS,
            "venkatakrishnan_ms_per_step": ms_vk, "vs_oracle": vs_oracle,
            "rel_l2_vs_oracle": vs_oracle["rel_l2"]}


def bench_imex(steps: int, warmup: int):
    """IMEX step (implicit isotropic collision) on the headline checkerboard: same bytes as
    the explicit step (8 B per update + 64 B per cell)."""
    import torch
    from paper_2205_08417_amd import inputs as I
    from paper_2205_08417_amd.solver import Solver

    P = I.build(WORKLOAD)
    S = Solver(P)
    state = [S.initial_state(), None]
    state[1] = torch.empty_like(state[0])
    args = S.args()
    stream = torch.cuda.current_stream()

    def one_step():
        S.step_imex(state[0], state[1], args)
        state.reverse()

    for _ in range(warmup):
        one_step()
    torch.cuda.synchronize()
    ms = timed(one_step, steps, stream)
    alg = P.ncells * (8 * P.nq + 64)
    from oracle import oracle as o
    op = o.OracleProblem.from_problem(P)
    vs_oracle = step_vs_oracle(S, state[0], lambda st_, c: o.step_imex(op, st_, P.dt, cells=c),
                               n=128, step=lambda a_, b_: S.step_imex(a_, b_, args),
                               what="one IMEX step")
    S.close()
    return {"workload": WORKLOAD, "scheme": "IMEX: implicit isotropic collision", "steps": steps,
            "ms_per_step": ms, "value": P.ncells * P.nq / (ms * 1e-3),
            "unit": "cell-ordinate updates/s", "hbm_frac": alg / (ms * 1e-3) / 1e9 / HBM_PEAK_GBS,
            "vs_oracle": vs_oracle, "rel_l2_vs_oracle": vs_oracle["rel_l2"]}


def bench_pn(steps: int, warmup: int, degree: int = 5):
    """P_N solver step (Sec. 4.3 flux with A^+/A^-) on the checkerboard mesh and materials:
    198 450 cells x (degree+1)^2 moments, FP32, tiled moment layout.  Algorithmic bytes per
    cell: the state in and out (8 B per moment), the 64-byte geometry record and sigma_t,
    sigma_s, source (12 B).  Algorithmic FLOPs per cell: one FMA per structurally non-zero
    entry of A_x, A_y, |A_x|, |A_y| plus the gather (per moment and face: a scale and four
    FMAs; per moment: five products)."""
    import numpy as np
    import torch
    from paper_2205_08417_amd import inputs as I
    from paper_2205_08417_amd import snrt
    from paper_2205_08417_amd.pn import PNSolver

    w = I.pn_checkerboard(degree=degree)
    mesh = w["mesh"]
    S = PNSolver(mesh, degree, w["sigma_t"], w["sigma_s"], w["dt"], source=w["source"])
    nm = S.nm
    state = [S.to_tiled(w["u0"]), None]
    state[1] = torch.empty_like(state[0])
    args = S.args()
    stream = torch.cuda.current_stream()

    def one_step():
        S.step(state[0], state[1], args)
        state.reverse()

    for _ in range(warmup):
        one_step()
    torch.cuda.synchronize()
    ms = timed(one_step, steps, stream)
    from oracle import oracle as o
    from oracle import pn as opn
    op = o.OracleProblem(mesh.face_nbr, mesh.face_normal, mesh.area, np.zeros((1, 3)),
                         np.ones(1), w["sigma_t"], w["sigma_s"], source=w["source"])
    system = opn.PNSystem(degree)
    final = state[0]
    nxt = torch.empty_like(final)
    S.step(final, nxt, args)
    cells = sample_cells(mesh.ncells, 256)
    got = S.to_user(nxt).cpu().numpy()[cells]
    start = S.to_user(final).cpu().numpy().astype(np.float64)
    vs_oracle = oracle_error(got, opn.pn_step(op, system, start, w["dt"], cells=cells),
                             f"one step from the final state, {cells.size} seeded cells")
    S.close()
    nc = mesh.ncells
    alg = nc * (8 * nm + 64 + 12)
    nnz = sum(int(np.count_nonzero(np.abs(a) > 1e-14)) for a in snrt.snrt_pn_operators(degree))
    mf = mesh.face_nbr.shape[1]
    flops = nc * (2 * nnz + nm * (5 + mf * 9))
    achieved = alg / (ms * 1e-3) / 1e9
    return {"workload": w["name"], "cells": nc, "moments": nm, "degree": degree,
            "steps": steps, "ms_per_step": ms, "value": nc * nm / (ms * 1e-3),
            "unit": "cell-moment updates/s", "precision": "fp32",
            "kernel": (f"k_pn_mfma<{degree},{mf}> (class blocks |A_x| P + |A_y| Q as FP16 "
                       "hi+lo matrix-core products, the rest FP32 vector FMAs)")
            if degree == 13 else f"k_pn_fused<{degree},{mf},float>" if degree <= 9 else
            f"k_pn_generic<16,{mf},float>",
            "algorithmic_bytes_per_step": alg, "achieved_gbs": achieved,
            "hbm_frac": achieved / HBM_PEAK_GBS, "flops_per_step": flops,
            "fp32_vector_tflops": flops / (ms * 1e-3) / 1e12,
            "fp32_vector_frac": flops / (ms * 1e-3) / 1e12 / FP32_VECTOR_PEAK_TFLOPS,
            "vs_oracle": vs_oracle, "rel_l2_vs_oracle": vs_oracle["rel_l2"]}


def bench_adjoint(nsteps: int = 400, ckpt: int = 20):
    """Checkerboard adjoint workload (51 842 cells x 256 ordinates, 400 steps): the forward
    rollout against the backward pass for J = integrated scalar flux over [5,6]x[3,4].
    Each pass is one library call (snrt_rollout / snrt_rollout_adjoint), so the host issues
    launches as fast as the device retires them and the event times are kernel-bound; the
    host wall time of each pass (to completion) is reported beside them.  With checkpoints
    every 20 steps the backward pass recomputes 380 states and runs 400 transposed steps;
    with every state kept (``ckpt_every=1``, 400 x 53 MB in HBM) it runs the 400 transposed
    steps alone."""
    import torch
    from paper_2205_08417_amd import inputs as I
    from paper_2205_08417_amd.solver import Solver, differentiable_rollout

    P = I.build("checkerboard_adjoint_s16", nsteps=nsteps)
    S = Solver(P)
    region = I.region_mask(P.mesh, P.meta["detector"])
    W = S.to_internal((region * P.mesh.area)[:, None] * P.w[None, :])
    st = S.mats32["sigma_t"].clone().requires_grad_(True)
    ss = S.mats32["sigma_s"].clone().requires_grad_(True)
    psi0 = S.initial_state()
    stream = torch.cuda.current_stream()

    def run_pass(k):
        """One forward + backward pass with checkpoints every k steps: (forward ms, backward
        ms) by events on the stream, and the same two by the host clock to completion."""
        torch.cuda.synchronize()
        ev = [torch.cuda.Event(enable_timing=True) for _ in range(4)]
        t0 = time.perf_counter()
        ev[0].record(stream)
        psiN = differentiable_rollout(S, psi0, nsteps, st, ss, ckpt_every=k)
        ev[1].record(stream)
        torch.cuda.synchronize()
        t1 = time.perf_counter()
        J = torch.sum(W * psiN)
        torch.cuda.synchronize()
        t2 = time.perf_counter()
        ev[2].record(stream)
        J.backward()
        ev[3].record(stream)
        torch.cuda.synchronize()
        t3 = time.perf_counter()
        st.grad = None
        ss.grad = None
        return (ev[0].elapsed_time(ev[1]), ev[2].elapsed_time(ev[3]), (t1 - t0) * 1e3,
                (t3 - t2) * 1e3)

    def timed_pass(k, reps=3):
        # two warm-up passes at the timed size settle clocks and leave the caching
        # allocator holding the checkpoint and segment buffers, so the timed passes allocate
        # nothing; each figure is the median of ``reps`` passes
        for _ in range(2):
            run_pass(k)
        runs = [run_pass(k) for _ in range(reps)]
        return tuple(float(sorted(r[i] for r in runs)[reps // 2]) for i in range(4))

    fwd, bwd, hfwd, hbwd = timed_pass(ckpt)
    fwd1, bwd1, hfwd1, hbwd1 = timed_pass(1)
    # the backward pass as its kernels add up: the recompute is (nsteps - nsteps/ckpt)
    # forward steps, the transposed steps are the store-everything backward pass
    recompute_steps = nsteps - (nsteps + ckpt - 1) // ckpt
    model = (recompute_steps / nsteps * fwd + bwd1) / fwd
    S.close()
    return {"workload": "checkerboard_adjoint_s16", "cells": P.ncells, "ordinates": P.nq,
            "steps": nsteps, "checkpoint_every": ckpt, "forward_ms": fwd, "backward_ms": bwd,
            "adjoint_forward_ratio": bwd / fwd,
            "host_wall_ms": {"forward": hfwd, "backward": hbwd, "ratio": hbwd / hfwd},
            "ratio_from_parts": model,
            "store_every_state": {"checkpoint_every": 1, "forward_ms": fwd1,
                                  "backward_ms": bwd1, "adjoint_forward_ratio": bwd1 / fwd1,
                                  "state_bytes_kept": nsteps * P.ncells * P.nq * 4},
            "note": "each pass is one library call; backward = segment recompute from the "
                    "checkpoints + transposed steps; ratio_from_parts = (recomputed steps x "
                    "forward step time + the store-every-state backward) / forward"}


def main():
    ap = argparse.ArgumentParser(description=__doc__.splitlines()[0])
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=1000)
    ap.add_argument("--warmup", type=int, default=20)
    ap.add_argument("--graph", action="store_true",
                    help="replay the timed steps from a captured HIP graph")
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--no-dense", action="store_true",
                    help="skip the mixed-precision anisotropic measurement")
    ap.add_argument("--dense-steps", type=int, default=None,
                    help="steps of the dense / CSD / moment runs (default: the whole workload)")
    ap.add_argument("--no-adjoint", action="store_true",
                    help="skip the adjoint/forward cost measurement")
    ap.add_argument("--no-second-order", action="store_true",
                    help="skip the second-order (Heun, reconstructed flux) measurement")
    ap.add_argument("--no-pn", action="store_true",
                    help="skip the P_N solver step measurement")
    ap.add_argument("--calibrate-copy", action="store_true",
                    help="run only a plain device copy of one state (for HBM counter scaling)")
    args = ap.parse_args()
    if args.gpus != 1 or int(os.environ.get("WORLD_SIZE", "1")) != 1:
        print("bench.py measures one GPU only: the S_N step library runs on a single device "
              "(a spatial decomposition across GPUs is described in the design notes but not "
              "built). Run with --gpus 1.", file=sys.stderr)
        sys.exit(2)

    import torch
    from paper_2205_08417_amd import inputs as I
    from paper_2205_08417_amd.solver import Solver

    if not torch.cuda.is_available():
        print("bench.py needs a HIP device", file=sys.stderr)
        sys.exit(1)
    torch.cuda.set_device(0)
    if args.calibrate_copy:
        n = 198450 * 256
        src = torch.ones(n, dtype=torch.float32, device="cuda")
        dst = torch.empty_like(src)
        for _ in range(args.steps):
            dst.copy_(src)
        torch.cuda.synchronize()
        print(json.dumps({"copy_bytes_read": 4 * n, "copy_bytes_written": 4 * n,
                          "launches": args.steps}))
        return
    P = I.build(WORKLOAD)
    S = Solver(P)
    a = S.initial_state()
    b = torch.empty_like(a)
    step_args = S.args()
    print(f"# {WORKLOAD}: {P.ncells} cells x {P.nq} ordinates, dt={P.dt:.4e}", file=sys.stderr,
          flush=True)

    def run(n, x, y):
        for _ in range(n):
            S.step(x, y, step_args)
            x, y = y, x
        return x, y

    stream = torch.cuda.current_stream()
    # the timed steps start from the developed state after the workload's 1000 steps (one
    # library call), not from the empty initial state
    a, _ = S.rollout(a, P.nsteps)
    a, b = run(args.warmup, a, b)
    torch.cuda.synchronize()
    K = args.steps
    if args.graph:
        K = 2 * ((K + 1) // 2)                      # pairs keep the ping-pong order fixed
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g):
            run(2, a, b)
        g.replay()
        torch.cuda.synchronize()
        start, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        start.record(stream)
        for _ in range(K // 2):
            g.replay()
        end.record(stream)
    else:
        start, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        start.record(stream)
        a, b = run(K, a, b)
        end.record(stream)
    torch.cuda.synchronize()
    ms = start.elapsed_time(end)
    ms_step = ms / K
    updates = P.ncells * P.nq
    value = updates * K / (ms * 1e-3)

    alg_bytes = P.ncells * (8 * P.nq + 64)          # 8 B per update + 64 B per cell record
    achieved = alg_bytes / (ms_step * 1e-3) / 1e9
    traffic = measured_traffic()
    out = {
        "metric": METRIC, "value": value, "unit": "cell-ordinate updates/s", "n_gpus": 1,
        "steps": K, "warmup": args.warmup, "ms_per_step": ms_step, "higher_is_better": True,
        "scaling": "weak", "vs_baseline": None, "dtype": "f32", "data": "synthetic",
        "config": {"workload": WORKLOAD, "cells": P.ncells, "ordinates": P.nq,
                   "scattering": "isotropic", "precision": "fp32", "mesh": "seeded jittered "
                   "Delaunay 316x316 points on [0,7]^2", "graph": bool(args.graph),
                   "timed_from": f"the state after {P.nsteps} steps from the initial state "
                                 f"plus {args.warmup} warm-up steps"},
        "roofline": {"bound": "hbm", "achieved": achieved, "peak": HBM_PEAK_GBS,
                     "unit": "GB/s", "frac": achieved / HBM_PEAK_GBS, "traffic": traffic,
                     "kernel": "k_step<4,true,3,false,false,float,false>",
                     "algorithmic_bytes_per_launch": alg_bytes},
    }
    S.close()
    copy_gbs, runtime_copy_gbs = copy_ceiling(P.ncells * P.nq * 4)
    out["roofline"]["copy_ceiling_gbs"] = copy_gbs
    out["roofline"]["frac_of_copy"] = achieved / copy_gbs
    out["roofline"]["runtime_copy_gbs"] = runtime_copy_gbs
    if not args.no_adjoint:           # first: its timing is sensitive to allocator history
        out["adjoint"] = bench_adjoint()
    if not args.no_dense:
        out["mixed_precision"] = bench_dense(args.dense_steps, 5)
        print("# mixed precision done", file=sys.stderr, flush=True)
        out["mixed_precision"]["hipblaslt_bf16_single_product_tflops_random"] = \
            library_gemm_ceiling(out["mixed_precision"]["cells"],
                                 out["mixed_precision"]["ordinates"])
        out["csd_dose"] = bench_csd(args.dense_steps, 5)
        print("# csd dose done", file=sys.stderr, flush=True)
        out["csd_dose_gradient"] = bench_dose_gradient()
        print("# csd dose gradient done", file=sys.stderr, flush=True)
        out["moments"] = bench_moments(args.dense_steps, 5)
    if not args.no_second_order:
        out["second_order"] = bench_second_order(min(args.steps, 200), 5)
        out["imex"] = bench_imex(min(args.steps, 200), 5)
    if not args.no_pn:
        out["pn"] = bench_pn(min(args.steps, 200), 5)
        # the degree of the paper's CSD P_N runs (Sec. 7), same mesh and materials
        out["pn_degree13"] = bench_pn(min(args.steps, 50), 3, degree=13)
    if not args.no_cpu_baseline:
        out["cpu_baseline"], (nref, ref) = cpu_baseline(P)
        # the FP32 path against the oracle after the same number of steps from the
        # workload's initial state
        import numpy as np
        Sp = Solver(P)
        psi_g, _ = Sp.rollout(Sp.initial_state(), nref)
        got = Sp.to_user(psi_g).cpu().numpy().astype(np.float64)
        Sp.close()
        out["parity_vs_oracle"] = {
            "workload": WORKLOAD, "steps": nref, "dtype": "f32",
            "rel_l2": float(np.linalg.norm(got - ref) / np.linalg.norm(ref))}
    print(json.dumps(out), flush=True)


if __name__ == "__main__":
    main()
