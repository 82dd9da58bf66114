"""Single right-hand side with blocks of different heights: the combine that stages every
partial row in LDS, tiles held whole, rows split evenly, the batch's combine."""

import numpy as np
import pytest

from oracle import apc_oracle as O

pytestmark = pytest.mark.gpu


def _blocks(m, lo, hi, seed):
    p = np.random.default_rng(seed).integers(lo, hi + 1, m)
    p[0], p[-1] = lo, hi
    return np.concatenate([[0], np.cumsum(p)]).astype(np.int64)


# m, smallest and largest block, n: up to three tiles of 16 rows per block; a ragged last
# column group; more blocks than the sums kept in registers; one tile per block.
@pytest.mark.parametrize("prec,tol", [("f64", 1e-10), ("f32", 1e-5)])
@pytest.mark.parametrize("m,lo,hi,n", [(3, 1, 40, 41), (17, 5, 33, 257), (131, 1, 20, 513),
                                       (500, 1, 3, 170)])
def test_trajectory(m, lo, hi, n, prec, tol):
    """20 updates against the oracle's."""
    import torch
    assert torch.cuda.is_available()
    from paper_1708_01413_amd import apc
    off = _blocks(m, lo, hi, 10 * m + n)
    rng = np.random.default_rng(m)
    A = rng.standard_normal((off[-1], n)) / np.sqrt(n)
    xs = rng.standard_normal((n, 1))
    B = A @ xs
    g, e = 1.2, 1.1
    ref = O.apc_run(A, B, off, T=20, gamma=g, eta=e, keep_traj=True)["traj"][20]
    plan = apc.Plan(torch.from_numpy(A).cuda(), torch.from_numpy(B).cuda(), off, prec,
                    gamma=g, eta=e)
    assert plan.resident_shape() or plan.single_pass_shape()
    plan.iterate_timed(20)
    got = plan.xbar().cpu().numpy().reshape(n, 1)
    dev = np.linalg.norm(got - ref) / np.linalg.norm(xs)
    print(f"{prec} m={m} n={n}: dev {dev:.2e}", flush=True)
    assert dev <= tol


# Rows of one 16-byte chunk and one wave; either side of a wave's width; the widest rows
# whose tiles are held whole, and one column more.
@pytest.mark.parametrize("prec,tol,n", [("f64", 1e-10, n) for n in (1, 127, 130, 2048, 2049)] +
                         [("f32", 1e-5, n) for n in (3, 255, 258, 4096, 4097)])
def test_tiles_held_whole(n, prec, tol):
    """20 updates on blocks of 1 to 65 rows (tiles of 16 and remainders), against
    the oracle's."""
    import torch
    assert torch.cuda.is_available()
    from paper_1708_01413_amd import apc
    p = [min(h, n) for h in (1, 65, 17, 15, 32)]
    while sum(p) < n:
        p.append(min(65, n))
    off = np.concatenate([[0], np.cumsum(p)]).astype(np.int64)
    rng = np.random.default_rng(n)
    A = rng.standard_normal((off[-1], n)) / np.sqrt(n)
    xs = rng.standard_normal((n, 1))
    B = A @ xs
    g, e = 1.2, 1.1
    ref = O.apc_run(A, B, off, T=20, gamma=g, eta=e, keep_traj=True)["traj"][20]
    plan = apc.Plan(torch.from_numpy(A).cuda(), torch.from_numpy(B).cuda(), off, prec,
                    gamma=g, eta=e)
    plan.iterate_timed(20)
    dev = np.linalg.norm(plan.xbar().cpu().numpy().reshape(n, 1) - ref) / np.linalg.norm(xs)
    print(f"{prec} n={n} N={off[-1]}: dev {dev:.2e}", flush=True)
    assert dev <= tol


def test_batch_combine():
    """One batch of systems with one row tile per block (fewer, exactly and more blocks than
    stay in registers; columns around a workgroup's 64) and with several: 20 updates."""
    import torch
    assert torch.cuda.is_available()
    from paper_1708_01413_amd import apc
    g, e = 1.2, 1.1
    plans, refs = [], []
    for s, (p, n) in enumerate([([1], 1), ([21, 22, 22], 65), ([4] * 15 + [3], 63),
                                ([9] * 16 + [1], 130), ([20] * 39 + [7], 700),
                                ([600, 1, 257] + [5] * 15, 640)]):
        off = np.concatenate([[0], np.cumsum(p)]).astype(np.int64)
        rng = np.random.default_rng(s)
        A = rng.standard_normal((off[-1], n)) / np.sqrt(n)
        xs = rng.standard_normal(n)
        refs.append((O.apc_run(A, (A @ xs)[:, None], off, T=20, gamma=g, eta=e)["xbar"][:, 0],
                     np.linalg.norm(xs)))
        plans.append(apc.Plan(torch.from_numpy(A).cuda(), torch.from_numpy(A @ xs).cuda(), off,
                              "f32", gamma=g, eta=e))
    batch = apc.Batch(plans)
    batch.iterate(20)
    for plan, (ref, xn) in zip(plans, refs):
        dev = np.linalg.norm(plan.xbar().cpu().numpy() - ref) / xn
        print(f"m={plan.m} n={plan.n}: dev {dev:.2e}", flush=True)
        assert dev <= 1e-5
    batch.close()


@pytest.mark.parametrize("prec,tol", [("f64", 1e-10), ("f32", 1e-5)])
@pytest.mark.parametrize("m,lo,hi,n", [(70, 3, 250, 4100), (4, 1000, 1100, 4100),
                                       (300, 20, 36, 4100)])
def test_rows_split_evenly(m, lo, hi, n, prec, tol):
    """Tall systems whose workgroups take consecutive rows across block boundaries (a few
    blocks per workgroup or workgroups per block): 12 updates."""
    import torch
    assert torch.cuda.is_available()
    from paper_1708_01413_amd import apc
    off = _blocks(m, min(lo, n), min(hi, n), m)
    while off[-1] < 8192:
        off = np.append(off, off[-1] + min(min(hi, n), 8250 - off[-1]))
    rng = np.random.default_rng(m)
    A = rng.standard_normal((off[-1], n)) / np.sqrt(n)
    xs = rng.standard_normal((n, 1))
    B = A @ xs
    g, e = 1.2, 1.1
    ref = O.apc_run(A, B, off, T=12, gamma=g, eta=e, keep_traj=True)["traj"][12]
    plan = apc.Plan(torch.from_numpy(A).cuda(), torch.from_numpy(B).cuda(), off, prec,
                    gamma=g, eta=e)
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    if prec == "f64" or 3 * m <= cus:
        assert plan.single_pass_shape()["rows_per_wg"] == -(-int(off[-1]) // cus)
    plan.iterate_timed(12)
    dev = np.linalg.norm(plan.xbar().cpu().numpy().reshape(n, 1) - ref) / np.linalg.norm(xs)
    print(f"{prec} m={len(off) - 1} N={off[-1]} n={n} {plan.single_pass_shape()}: dev {dev:.2e}",
          flush=True)
    assert dev <= tol


@pytest.mark.parametrize("m,n", [(1, 17), (259, 170), (600, 33)])
def test_heavy_ball_over_many_tiles(m, n):
    """15 heavy-ball steps over one, just over 256 and over 512 row tiles, FP64, against the
    oracle's."""
    import torch
    assert torch.cuda.is_available()
    from paper_1708_01413_amd import apc
    off = _blocks(m, 1, 2, m) if m > 1 else np.array([0, n], dtype=np.int64)
    rng = np.random.default_rng(m)
    A = rng.standard_normal((off[-1], n)) / np.sqrt(n)
    xs = rng.standard_normal((n, 1))
    B = A @ xs
    ref = O.dhbm_run(A, B, off, 15, preconditioned=True, alpha=0.9 / m, beta=0.3,
                     keep_traj=True)["traj"][15, :, 0]
    plan = apc.Plan(torch.from_numpy(A).cuda(), torch.from_numpy(B[:, 0]).cuda(), off, "f64",
                    gamma=1.0, eta=1.0)
    h = apc.HeavyBall(plan, 1, alpha=0.9 / m, beta=0.3)
    h.iterate(15)
    dev = np.linalg.norm(h.x().cpu().numpy() - ref) / np.linalg.norm(xs)
    print(f"m={m} n={n}: dev {dev:.2e}", flush=True)
    assert dev <= 1e-10


@pytest.mark.parametrize("n", [4096, 3300])
def test_wave_sums_of_whole_tiles(n):
    """One row product over 16 and 13 waves' columns, one entry per wave: a large product
    and then ones just below half a unit of its last place.  Added pairwise the product of
    the row is off by at most a rounding per product, four per sum and one of what is read
    back (6 u); added one after another every small one is lost (0.99 u each)."""
    import torch
    assert torch.cuda.is_available()
    from paper_1708_01413_amd import apc
    u = 2.0 ** -24
    at = np.arange(0, n, 256)
    a = np.zeros(n)
    a[at] = 1 / np.sqrt(len(at))
    # Block 0 is this row, with b = 0; the others are unit rows, so x_bar(0) = x / m.
    off = np.concatenate([[0], np.minimum(1 + np.arange(0, n, 64), n), [n + 1]]).astype(np.int64)
    m = len(off) - 1
    x = np.zeros(n)
    x[at] = m
    x[at[1:]] *= 0.99 * u
    A = np.concatenate([a[None], np.eye(n)])
    plan = apc.Plan(torch.from_numpy(A).cuda(), torch.from_numpy(np.concatenate([[0.0], x])).cuda(),
                    off, "f32", gamma=1.0, eta=1.0)
    d = plan.xbar().cpu().numpy()
    plan.iterate(1)
    # x_0(1) = x_bar(0) - C_0 w with w = C_0 . x_bar(0).
    C = a.astype(np.float32).astype(np.float64)
    w = (d - plan.local().cpu().numpy()[0].reshape(-1))[at] / C[at]
    ref = C @ d.astype(np.float32).astype(np.float64)
    print(f"n={n} {plan.single_pass_shape()}: w off by {(w / ref - 1) / u} u", flush=True)
    assert np.all(np.abs(w - ref) <= 6 * u * ref)


@pytest.mark.parametrize("prec,N,n,m,rows,group", [
    ("f32", 8192, 8192, 64, 32, 1), ("f32", 8300, 8192, 64, 33, 2), ("f32", 16384, 8192, 30, 64, 2), ("f32", 16384, 5000, 80, 64, 2),
    ("f64", 16384, 4000, 80, 64, 2), ("f32", 14000, 5000, 40, 32, 1), ("f32", 20000, 5000, 60, 64, 1),
    ("f64", 26000, 2500, 60, 64, 1)])
def test_split_and_groups_of_wide_rows(prec, N, n, m, rows, group):
    """FP32 and FP64 rows of eight chunks per thread in uneven blocks: one workgroup per CU
    over an even split of more than 32 rows reads two rows at a time; plain tiles (rows per
    workgroup 32 or 64) of between one and two per CU one row, two workgroups per CU.
    Rows that do not fill their chunks keep the plain tiles unless the fullest CU had
    nearly twice the mean."""
    import torch
    assert torch.cuda.is_available()
    from paper_1708_01413_amd import apc
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    if cus != 256:
        pytest.skip("the shapes are those of 256 CUs")
    p = np.random.default_rng(m).uniform(0.2, 1.0, m)
    off = np.concatenate([[0], np.round(np.cumsum(p) / p.sum() * N)]).astype(np.int64)
    g = torch.Generator(device="cuda").manual_seed(m)
    A = torch.randn(N, n, generator=g, dtype=torch.float64, device="cuda") / n ** 0.5
    plan = apc.Plan(A, A[:, 0].contiguous(), off, prec, gamma=1.2, eta=1.1)
    assert plan.single_pass_shape() == {"rows_per_wg": rows, "rows_per_group": group}
