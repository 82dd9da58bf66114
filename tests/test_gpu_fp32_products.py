"""FP32 products of the k-RHS form on the bf16 matrix cores (operands split into three
bf16 parts): one plain FP32 update against the FP64 oracle."""

import math

import numpy as np
import pytest

from oracle import apc_oracle as O
from paper_1708_01413_amd import synth

pytestmark = pytest.mark.gpu

U = 2.0 ** -24  # FP32 unit roundoff


def _torch():
    import torch
    assert torch.cuda.is_available()
    return torch


def _one_update(S, g, e):
    Qt, R = O.factor(S.A, S.off)
    x = O.init_local(Qt, R, S.B, S.off)
    x0 = O.initial_average(x)
    return x0, O.apc_step(Qt, x, x0, g, e)[1]


# Row lengths around the 64-column step and the 256 padding, and right-hand sides around
# every column-tile count (16, 32, 64, 128) and a second column group.
@pytest.mark.parametrize("N,n,k,scale", [(64, 64, 2, 1.0), (65, 63, 16, 1.0), (130, 100, 17, 1.0),
                                         (256, 256, 32, 1.0), (300, 200, 33, 1.0),
                                         (257, 255, 64, 1.0), (192, 192, 65, 1.0),
                                         (300, 256, 128, 1.0), (140, 129, 130, 1.0),
                                         (200, 200, 24, 1e-30), (200, 200, 24, 1e30)])
def test_one_fp32_update(N, n, k, scale):
    """The inputs' rounding (C, y and W to FP32: 3 u) and the sums' (a random walk of at
    most K = 256 roundings per product: sqrt(K) u) bound the error of X y, which the
    update multiplies by eta: two products give 2 u (4 + sqrt(K)) eta ||X y|| / ||x_bar||.
    Leaving out the third part of either operand would cost about 2^-16."""
    torch = _torch()
    from paper_1708_01413_amd import apc
    S = synth.gaussian_system(N, n, 5, k=k, seed=3 * n + k, scale=1 / math.sqrt(n), shift=2.0)
    S.B *= scale
    g, e, _ = O.optimal_params(*O.spectrum(S.A, S.off))
    x0, ref = _one_update(S, g, e)
    plan = apc.Plan(torch.from_numpy(S.A).cuda(), torch.from_numpy(S.B).cuda(), S.off, "f32",
                    gamma=g, eta=e, anchor_every=0)
    plan.iterate(1)
    got = plan.xbar().cpu().numpy()
    # x_bar(1) = eta (x0 + y1 - X y1) + (1 - eta) x0 with y1 = gamma x0.
    Xy = x0 + g * x0 - (ref - (1 - e) * x0) / e
    amp = e * np.linalg.norm(Xy) / np.linalg.norm(ref)
    dev = np.linalg.norm(got - ref) / np.linalg.norm(ref)
    tol = 2 * U * (4 + math.sqrt(256)) * amp
    print(f"N={N} n={n} k={k} scale={scale}: dev {dev:.2e} tol {tol:.2e}", flush=True)
    assert dev <= tol


@pytest.mark.parametrize("k", [100, 128])
def test_mixed_batch_with_two_column_groups(k):
    """128 padded right-hand sides next to a k = 1 system, three plain FP32 updates against
    the oracle at the FP32 bar."""
    torch = _torch()
    from paper_1708_01413_amd import apc
    big = synth.gaussian_system(320, 300, 6, k=k, seed=k, scale=1 / math.sqrt(300), shift=2.0)
    small = synth.gaussian_system(90, 90, 4, seed=k + 1, scale=1 / math.sqrt(90), shift=2.0)
    plans, refs = [], []
    for S, kw in ((big, {"anchor_every": 0}), (small, {})):
        g, e, _ = O.optimal_params(*O.spectrum(S.A, S.off))
        refs.append(O.apc_run(S.A, S.B, S.off, T=3, gamma=g, eta=e, keep_traj=True)["traj"][3])
        plans.append(apc.Plan(torch.from_numpy(S.A).cuda(), torch.from_numpy(S.B).cuda(), S.off,
                              "f32", gamma=g, eta=e, **kw))
    batch = apc.Batch(plans)
    batch.iterate(3)
    for S, p, ref in zip((big, small), plans, refs):
        got = p.xbar().cpu().numpy().reshape(ref.shape)
        dev = np.linalg.norm(got - ref) / np.linalg.norm(S.xstar)
        print(f"k={k} n={S.n}: dev {dev:.2e}", flush=True)
        assert dev <= 1e-5
    batch.close()


def _worst_split_angles(count):
    """Angles whose cosine and sine, as FP32, have large middle and low thirds of one sign."""
    rng = np.random.default_rng(1)

    def worst(v):
        bits = int(np.float32(v).view(np.uint32))
        return 200 <= (bits >> 8 & 255) <= 254 and 96 <= (bits & 255) <= 126

    out = []
    while len(out) < count:
        t = rng.uniform(0.3, 1.27)
        if worst(math.cos(t)) and worst(math.sin(t)):
            out.append(t)
    return out


def test_products_of_sparse_rows():
    """Rows of two entries (2 x 2 rotations, a block per row), gamma = eta = 1: x_bar(1) =
    2 x0 - X x0 with x0 = x / m, so X x0 = 2 x0 - x_bar(1) is two FP32 contractions of two
    products each.  Their roundings have either sign, so the mean of the n k = 1536
    relative errors against 64 bits of the FP32 inputs is below 3 u / sqrt(n k) = 0.08 u
    (a third of it for a uniform rounding error); 0.5 u is six of that.  Entries whose
    middle and low thirds are large and of one sign make the parts that a product leaves
    out add up instead: a split by truncation has a mean of -1.6 u."""
    torch = _torch()
    from paper_1708_01413_amd import apc
    n, k = 64, 24
    A = np.zeros((n, n))
    for i, t in enumerate(_worst_split_angles(4) * 8):
        c, s = math.cos(t), math.sin(t)
        A[2 * i:2 * i + 2, 2 * i:2 * i + 2] = [[c, s], [-s, c]]
    rng = np.random.default_rng(2)
    x = ((rng.integers(128, 256, (n, k)) << 16) | (rng.integers(200, 255, (n, k)) << 8) |
         rng.integers(96, 127, (n, k))) / 2.0 ** 23
    plan = apc.Plan(torch.from_numpy(A).cuda(), torch.from_numpy(A @ x).cuda(),
                    np.arange(n + 1), "f32", gamma=1.0, eta=1.0, anchor_every=0)
    plan.iterate(1)
    z = n * (2 * x / n - plan.xbar().cpu().numpy())
    C = A.astype(np.float32).astype(np.float64)
    ref = C.T @ (C @ x) / n
    rel = (z - ref) / ref / U
    print(f"relative error in u: mean {rel.mean():.3f} rms {np.sqrt((rel ** 2).mean()):.3f} "
          f"max {abs(rel).max():.2f}", flush=True)
    assert abs(rel.mean()) <= 0.5


@pytest.mark.parametrize("ks", ["0", "1", "2"])
@pytest.mark.parametrize("exps", [(-36, -36), (-45, -45), (38, 38), (60, 60), (-60, 60)])
def test_one_fp32_update_far_from_one(exps, ks, monkeypatch):
    """Right-hand sides of 1e-60 to 1e60 (the last: every column of its own, one of them
    zero), each column to the bound of test_one_fp32_update.  A power of two changes no
    rounding, so the bound does not depend on the scale; the third parts of unscaled
    entries fall out of bf16's range below 1e-33."""
    torch = _torch()
    from paper_1708_01413_amd import apc
    k = 24
    S = synth.gaussian_system(200, 200, 5, k=k, seed=8, scale=1 / math.sqrt(200), shift=2.0)
    S.B *= 10.0 ** np.linspace(*exps, k)
    if exps[0] != exps[1]:
        S.B[:, 5] = 0.0
    monkeypatch.setenv("APC_TN_KS", ks)
    g, e, _ = O.optimal_params(*O.spectrum(S.A, S.off))
    x0, ref = _one_update(S, g, e)
    plan = apc.Plan(torch.from_numpy(S.A).cuda(), torch.from_numpy(S.B).cuda(), S.off, "f32",
                    gamma=g, eta=e, anchor_every=0)
    plan.iterate(1)
    got = plan.xbar().cpu().numpy()
    Xy = x0 + g * x0 - (ref - (1 - e) * x0) / e
    for c in range(k):
        norm = np.linalg.norm(ref[:, c])
        tol = 2 * U * (4 + math.sqrt(256)) * e * np.linalg.norm(Xy[:, c])
        dev = np.linalg.norm(got[:, c] - ref[:, c])
        assert dev <= tol, f"column {c}: dev {dev:.2e} tol {tol:.2e} of {norm:.2e}"
    # The next right-hand sides get scales of their own.
    plan.restart(torch.from_numpy(S.B / 10.0 ** np.linspace(*exps, k)).cuda())
    plan.iterate(1)
    back = plan.xbar().cpu().numpy() * 10.0 ** np.linspace(*exps, k)
    assert np.all(np.linalg.norm(back - ref, axis=0) <=
                  2 * U * (4 + math.sqrt(256)) * e * np.linalg.norm(Xy, axis=0))


@pytest.mark.parametrize("ks", ["0", "1", "2"])
@pytest.mark.parametrize("k", [12, 24])
def test_fp32_adjoint(k, ks, monkeypatch):
    """The FP32 reverse step, by itself and inside the contraction's launch, 16 and more
    right-hand sides, dL/dB, dL/dgamma and dL/deta to 1e-5 of the oracle's; with more than 16
    also for right-hand sides of 1e36 and cotangents of 1e-36."""
    torch = _torch()
    from paper_1708_01413_amd import apc
    S = synth.gaussian_system(300, 200, 5, k=k, seed=4, scale=1 / math.sqrt(200), shift=2.0)
    g, e, _ = O.optimal_params(*O.spectrum(S.A, S.off))
    dx = np.random.default_rng(1).standard_normal((S.n, k))
    rB, rg, re = O.apc_adjoint(S.A, S.B, S.off, 9, g, e, dx)
    monkeypatch.setenv("APC_TN_KS", ks)
    for f in (1.0, 1e36) if k > 16 else (1.0,):
        plan = apc.Plan(torch.from_numpy(S.A).cuda(), torch.from_numpy(S.B * f).cuda(), S.off,
                        "f32", gamma=g, eta=e)
        if ks == "1":
            assert plan.launch_shapes()["pass_b"]["rows_per_wg"] == 16
        dB, dg, de = plan.backward(torch.from_numpy(dx / f).cuda(), 9, 4)
        dev = np.linalg.norm(dB.cpu().numpy() * f - rB) / np.linalg.norm(rB)
        print(f"k={k} ks={ks} scale={f}: dB {dev:.2e} dgamma {abs(dg - rg) / abs(rg):.2e} "
              f"deta {abs(de - re) / abs(re):.2e}", flush=True)
        assert dev <= 1e-5
        assert abs(dg - rg) <= 1e-5 * abs(rg) and abs(de - re) <= 1e-5 * abs(re)


def test_scales_of_replayed_graphs_and_batches():
    """A captured graph's updates and a batch's take the scales of the last restart: three
    updates from right-hand sides of 1e-40 are those of 1 at the FP32 bar."""
    torch = _torch()
    from paper_1708_01413_amd import apc
    k = 24
    big = synth.gaussian_system(200, 200, 5, k=k, seed=8, scale=1 / math.sqrt(200), shift=2.0)
    small = synth.gaussian_system(90, 90, 4, seed=9, scale=1 / math.sqrt(90), shift=2.0)
    plans, stream = [], torch.cuda.Stream()
    for S, kw in ((big, {"anchor_every": 0}), (small, {})):
        g, e, _ = O.optimal_params(*O.spectrum(S.A, S.off))
        plans.append(apc.Plan(torch.from_numpy(S.A).cuda(), torch.from_numpy(S.B).cuda(), S.off,
                              "f32", gamma=g, eta=e, stream=stream, **kw))
    plan, b = plans[0], torch.from_numpy(big.B).cuda()
    g, e, _ = O.optimal_params(*O.spectrum(big.A, big.off))
    ref = O.apc_run(big.A, big.B, big.off, T=3, gamma=g, eta=e)["xbar"]
    batch = None
    for f in (1.0, 1e-40, 1.0, 1e40):
        for kind in ("graph", "batch"):
            plan.restart(b * f)
            if kind == "graph":
                plan.iterate(3, graph=True)
            else:
                batch = batch or apc.Batch(plans)
                batch.iterate(3)
            dev = np.linalg.norm(plan.xbar().cpu().numpy() / f - ref) / np.linalg.norm(big.xstar)
            print(f"{kind} scale {f}: dev {dev:.2e}", flush=True)
            assert dev <= 1e-5
    batch.close()
