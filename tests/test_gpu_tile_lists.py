"""The single pass's tile lists at their ends: combines on either side of what LDS holds,
and every user of an even split of the rows over the CUs (the eigenvalue estimate, both
heavy-ball forms, the orthogonality estimate)."""

import functools
import math

import numpy as np
import pytest

from oracle import apc_oracle as O

pytestmark = pytest.mark.gpu

LDS = 150 * 1024  # what the staged combine takes at most


def _torch():
    import torch
    assert torch.cuda.is_available()
    return torch


def _cuda(a):
    return _torch().from_numpy(np.ascontiguousarray(a)).cuda()


# Blocks of 1 to 20 rows have one or two tiles of 16: within 64 KB of LDS, above it, and past
# what the staged combine takes (partial rows read block by block).
@pytest.mark.parametrize("prec,tol,m,side", [("f64", 1e-10, 300, "small"), ("f64", 1e-10, 800, "staged"),
                                             ("f64", 1e-10, 1100, "read"),
                                             ("f32", 1e-5, 1500, "staged"),
                                             ("f32", 1e-5, 2300, "read")])
def test_combine_of_uneven_tile_counts(prec, tol, m, side, monkeypatch):
    """10 updates against the oracle's."""
    _torch()
    from paper_1708_01413_amd import apc
    n = 67
    p = np.random.default_rng(m).integers(1, 21, m)
    p[0], p[-1] = 1, 20
    off = np.concatenate([[0], np.cumsum(p)]).astype(np.int64)
    rng = np.random.default_rng(m + 1)
    A = rng.standard_normal((off[-1], n)) / math.sqrt(n)
    xs = rng.standard_normal((n, 1))
    B = A @ xs
    ref = O.apc_run(A, B, off, T=10, gamma=1.2, eta=1.1)["xbar"]
    monkeypatch.setenv("APC_FUSED_ROWS", "16")
    plan = apc.Plan(_cuda(A), _cuda(B), off, prec, gamma=1.2, eta=1.1)
    assert plan.single_pass_shape()["rows_per_wg"] == 16
    tiles = -(-p // 16)
    lds = int(tiles.sum()) * 16 * (8 if prec == "f64" else 4) + (m + 1) * 4
    assert set(tiles) == {1, 2}
    assert {"small": lds <= 64 * 1024, "staged": 64 * 1024 < lds <= LDS, "read": lds > LDS}[side]
    plan.iterate_timed(10)
    dev = np.linalg.norm(plan.xbar().cpu().numpy().reshape(n, 1) - ref) / np.linalg.norm(xs)
    print(f"{prec} m={m} tiles={tiles.sum()} lds={lds}: dev {dev:.2e}", flush=True)
    assert dev <= tol


@functools.lru_cache(maxsize=1)
def _tall():
    """8250 x 4100 in uneven blocks: FP64 rows take 16 chunks per thread and FP32 rows 8,
    and plain tiles of 32 rows would leave one CU with twice the mean, so both split their
    rows evenly."""
    rng = np.random.default_rng(3)
    p = rng.integers(3, 251, 70)
    off = [0, *np.cumsum(p)]
    while off[-1] < 8250:
        off.append(min(off[-1] + 250, 8250))
    off = np.array(off, dtype=np.int64)
    off = off[:np.searchsorted(off, 8250) + 1]
    off[-1] = 8250
    A = rng.standard_normal((8250, 4100)) / math.sqrt(4100)
    x = rng.standard_normal((4100, 8))
    return A, x, A @ x, off


def _even(plan, off):
    cus = _torch().cuda.get_device_properties(0).multi_processor_count
    if cus != 256:
        pytest.skip("the sizes are those of 256 CUs")
    return plan.single_pass_shape()["rows_per_wg"] == -(-int(off[-1]) // cus)


@functools.lru_cache(maxsize=1)
def _spectrum():
    A, _, _, off = _tall()
    return O.spectrum(A, off)


@pytest.mark.parametrize("prec,k", [("f64", 1), ("f32", 1), ("f32", 8)])
def test_eigenvalue_estimate(prec, k):
    """The estimate encloses the spectrum, with the margins of the small systems' test."""
    from paper_1708_01413_amd import apc
    A, _, B, off = _tall()
    mn, mx = _spectrum()
    plan = apc.Plan(_cuda(A), _cuda(B[:, :k] if k > 1 else B[:, 0]), off, prec)
    assert k > 1 or _even(plan, off)
    p = plan.params()
    print(f"{prec} k={k}: lo/mu_min {p['mu_min'] / mn:.4f} hi/mu_max {p['mu_max'] / mx:.6f}", flush=True)
    slack = 1e-12 if prec == "f64" else 1e-6
    assert 0.5 * mn <= p["mu_min"] <= mn * (1 + slack)
    assert mx * (1 - slack) <= p["mu_max"] <= min(1.0, 1.05 * mx)


@pytest.mark.parametrize("prec,tol", [("f64", 1e-10), ("f32", 1e-5)])
def test_heavy_ball(prec, tol):
    """12 preconditioned heavy-ball steps, FP64 and with an FP32 factor."""
    from paper_1708_01413_amd import apc
    A, x, B, off = _tall()
    ref = O.dhbm_run(A, B[:, :1], off, 12, preconditioned=True, alpha=0.2, beta=0.3,
                     keep_traj=True)["traj"][12, :, 0]
    plan = apc.Plan(_cuda(A), _cuda(B[:, 0]), off, prec, gamma=1.0, eta=1.0)
    assert _even(plan, off)
    h = apc.HeavyBall(plan, 1, alpha=0.2, beta=0.3)
    h.iterate(12)
    dev = np.linalg.norm(h.x().cpu().numpy() - ref) / np.linalg.norm(x[:, 0])
    print(f"{prec}: dev {dev:.2e}", flush=True)
    assert dev <= tol


def test_orthogonality_estimate(monkeypatch):
    """Blocks with a common part of 300 times their rows: the first CholeskyQR pass leaves a
    defect far above rounding, whose estimate over the even split (vector-unit setup) is that
    over plain tiles.  Both sum the same products in another order, with relative errors of
    about 1e-14 against a defect of 1e-10 or more: 1e-3."""
    from paper_1708_01413_amd import apc
    A, _, B, off = _tall()
    A = A.copy()
    for i in range(len(off) - 1):
        A[off[i]:off[i + 1]] += 300.0 * A[off[i]]
    monkeypatch.setenv("APC_SETUP_MFMA", "0")
    found = []
    for rows in (None, "32"):
        if rows:
            monkeypatch.setenv("APC_FUSED_ROWS", rows)
        plan = apc.Plan(_cuda(A), _cuda(B[:, 0]), off, "f32", gamma=1.0, eta=1.0)
        assert _even(plan, off) == (rows is None)
        found.append(plan.setup_info())
        plan.close()
    print(found, flush=True)
    a, b = (f["qr_defect"] for f in found)
    assert found[0]["qr_passes"] == found[1]["qr_passes"] == 2
    assert a > 1e-10 and abs(a - b) <= 1e-3 * b
