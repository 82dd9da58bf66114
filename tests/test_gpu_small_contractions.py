"""The contraction whose waves split K and that applies its epilogue itself (forced with
APC_TN_KS, 16 or 32 right-hand sides per workgroup): its epilogues and element types (the
FP32 reverse step in test_gpu_fp32_products.py), on sizes with one row tile, with fewer
steps of K than waves and with ragged ends."""

import math

import numpy as np
import pytest

from oracle import apc_oracle as O
from paper_1708_01413_amd import synth

pytestmark = pytest.mark.gpu


def _torch():
    import torch
    assert torch.cuda.is_available()
    return torch


def _system(N, n, k, seed):
    S = synth.gaussian_system(N, n, 5, k=k, seed=seed, scale=1 / math.sqrt(n), shift=2.0)
    torch = _torch()
    return S, torch.from_numpy(S.A).cuda(), torch.from_numpy(S.B).cuda()


SIZES = [(64, 64, 2), (300, 200, 33), (513, 260, 17)]


@pytest.mark.parametrize("ks", ["1", "2"])
@pytest.mark.parametrize("N,n,k", SIZES)
def test_trajectories(N, n, k, ks, monkeypatch):
    """18 updates (two anchors): FP64 to 1e-10 and anchored FP32 to 1e-5 of the oracle, and
    the rebuilt residual monitor's value to 1e-9 of the solution's own."""
    from paper_1708_01413_amd import apc
    S, A, b = _system(N, n, k, 7 * n + k)
    g, e, _ = O.optimal_params(*O.spectrum(S.A, S.off))
    ref = O.apc_run(S.A, S.B, S.off, T=18, gamma=g, eta=e, keep_traj=True)["traj"][18]
    monkeypatch.setenv("APC_TN_KS", ks)
    for prec, tol in (("f64", 1e-10), ("f32", 1e-5)):
        plan = apc.Plan(A, b, S.off, prec, gamma=g, eta=e)
        if k > 16 or ks == "1":
            assert plan.launch_shapes()["pass_a"]["rows_per_wg"] == 16
        plan.iterate(18)
        got = plan.xbar().cpu().numpy()
        dev = np.linalg.norm(got - ref) / np.linalg.norm(S.xstar)
        res = np.linalg.norm(S.B - S.A @ got) / np.linalg.norm(S.B)
        print(f"{prec} N={N} n={n} k={k} ks={ks}: dev {dev:.2e}", flush=True)
        assert dev <= tol
        assert abs(plan.residual() - res) <= 1e-9 * res + 1e-14


@pytest.mark.parametrize("ks", ["1", "2"])
def test_adjoint(ks, monkeypatch):
    """dL/dB to 1e-10 and dL/dgamma, dL/deta to 1e-9 of the oracle's adjoint (FP64)."""
    torch = _torch()
    from paper_1708_01413_amd import apc
    S, A, b = _system(300, 200, 33, 5)
    g, e, _ = O.optimal_params(*O.spectrum(S.A, S.off))
    dx = np.random.default_rng(1).standard_normal((S.n, S.k))
    rB, rg, re = O.apc_adjoint(S.A, S.B, S.off, 9, g, e, dx)
    monkeypatch.setenv("APC_TN_KS", ks)
    plan = apc.Plan(A, b, S.off, "f64", gamma=g, eta=e)
    dB, dg, de = plan.backward(torch.from_numpy(dx).cuda(), 9, 4)
    dev = np.linalg.norm(dB.cpu().numpy() - rB) / np.linalg.norm(rB)
    print(f"ks={ks}: dB {dev:.2e} dgamma {abs(dg - rg) / abs(rg):.2e} deta {abs(de - re) / abs(re):.2e}")
    assert dev <= 1e-10
    assert abs(dg - rg) <= 1e-9 * abs(rg) and abs(de - re) <= 1e-9 * abs(re)


@pytest.mark.parametrize("anchor", [0, 4])
def test_bf16_refinement(anchor, monkeypatch):
    """bf16 inner solves (with and without FP64 anchors) refined to the FP64 solution."""
    from paper_1708_01413_amd import apc
    S, A, b = _system(256, 256, 40, 9)
    monkeypatch.setenv("APC_TN_KS", "2")
    plan = apc.Plan(A, b, S.off, "bf16_ir", anchor_every=anchor)
    x, _, rr, st = plan.solve(1e-12, 2000)
    dev = np.linalg.norm(x.cpu().numpy() - S.xstar) / np.linalg.norm(S.xstar)
    print(f"anchor={anchor}: relres {rr:.2e} dev {dev:.2e}")
    assert st == 0 and dev <= 1e-10


@pytest.mark.parametrize("n,k", [(64, 2), (256, 16), (700, 24), (1000, 40), (512, 128), (1500, 16)])
def test_residual_takes_the_fastest_contraction(n, k):
    """An FP64 plan's residual is the contraction of pass A with a launch after it either
    way: its shape is the fastest one measured (one round of timing serves both), while
    pass A may take a slower one that saves that launch; residual() is right in it."""
    from paper_1708_01413_amd import apc
    S, A, b = _system(n, n, k, n + k)
    plan = apc.Plan(A, b, S.off, "f64", gamma=1.0, eta=1.0)
    shapes = plan.launch_shapes()
    print(f"n={n} k={k} {shapes}", flush=True)
    assert shapes["residual"]["tuned_us"] <= shapes["pass_a"]["tuned_us"]
    got = plan.xbar().cpu().numpy()
    res = np.linalg.norm(S.B - S.A @ got) / np.linalg.norm(S.B)
    assert abs(plan.residual() - res) <= 1e-9 * res + 1e-14


@pytest.mark.parametrize("g,e", [(1.2, 1.5), (4.0, 9.0)])
@pytest.mark.parametrize("prec,N,n,k", [("f64", 1290, 1290, 19), ("f32", 1290, 770, 37),
                                        ("f32", 1030, 1030, 11), ("bf16_ir", 1290, 770, 70)])
def test_first_plan_of_a_shape_equals_the_next(prec, N, n, k, g, e):
    """The first plan of a shape in a process times updates of its own start to choose its
    launch shapes, the next one takes that choice: the same bits after setup and after 18
    updates, also with parameters that diverge."""
    torch = _torch()
    from paper_1708_01413_amd import apc
    N, n = (v + 256 * (g > 2) for v in (N, n))  # (another padded shape: timed again)
    S, A, b = _system(N, n, k, N + n + k)
    plans = [apc.Plan(A, b, S.off, prec, gamma=g, eta=e) for _ in range(2)]
    first, second = ([p.launch_shapes()[q] for q in ("pass_a", "pass_b")] for p in plans)
    assert first == second
    for T in (0, 1, 17):
        for p in plans:
            p.iterate(T)
        x, y = (p.xbar() for p in plans)
        assert torch.equal(x, y) and bool(torch.isfinite(x).all())
