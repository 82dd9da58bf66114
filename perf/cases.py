"""Workloads that time the solver through its public entry points.

Every case is a linear system A x = B of one of the two families this package's
generators and benchmark use -- tall Gaussian (A iid N(0, 1/n), N > n, shift 0) and
shifted square (A = G / sqrt(n) + shift * I, N = n) -- split into row blocks, and one way a program
uses the solver on it:

  updates     a plan that is kept: new right-hand sides, T updates, the estimate
  solve       the whole call: factor, parameters, updates to a tolerance
  refine      a kept mixed-precision plan: new right-hand sides, refinement to a tolerance
  heavy_ball  the heavy-ball comparison method on a kept plan
  batch       many small systems updated together
  adjoint     forward and backward of the unrolled iteration through torch.autograd

FP32 plans' results are handed on in FP32, the precision they carry.
"""

import math

import numpy as np
import torch

from paper_1708_01413_amd import apc, synth

# Above this size a factor does not stay in the last-level cache between updates.
CACHE_BYTES = 256 << 20


# ------------------------------------------------------------------ cases


def listed():
    return [
        # A small dense FP64 solve inside another program (the 512 x 512 system of the
        # benchmark): a new right-hand side, a few updates, latency throughout.
        dict(name="small_f64_updates", kind="updates", N=512, n=512, m=8, uneven=False, k=1,
             shift=2.0, precision="f64", T=20),
        # One cold FP64 solve of a mid-size overdetermined system with ragged blocks and
        # sizes that fit no tile: setup's launches and the eigenvalue estimate dominate.
        dict(name="ragged_f64_solve", kind="solve", N=1500, n=1200, m=11, uneven=True, k=1,
             shift=0.0, precision="f64", rtol=1e-11),
        # The benchmark system with its factorisation kept: the next right-hand side to 1e-6.
        dict(name="tall_f32_updates", kind="updates", N=16384, n=8192, m=64, uneven=False, k=1,
             shift=0.0, precision="f32", T=41),
        # The benchmark's own step: the same system from nothing to 1e-6.
        dict(name="tall_f32_solve", kind="solve", N=16384, n=8192, m=64, uneven=False, k=1,
             shift=0.0, precision="f32", rtol=1e-6),
        # The paper's closest competitor on the same shape, in FP64.
        dict(name="tall_f64_heavy_ball", kind="heavy_ball", N=16384, n=8192, m=64, uneven=False,
             k=1, shift=0.0, precision="f64", plain=True, T=42),
        # Several right-hand sides in FP64 on sizes that fit no tile (a small multi-source
        # problem), factorisation kept.
        dict(name="rhs20_f64_updates", kind="updates", N=3001, n=2403, m=17, uneven=True, k=20,
             shift=0.0, precision="f64", T=30),
        # The benchmark's batched system (64 right-hand sides, uneven blocks): next right-hand
        # sides on a kept factorisation, to 1e-6.
        dict(name="rhs64_f32_updates", kind="updates", N=8192, n=8192, m=64, uneven=True, k=64,
             shift=2.0, precision="f32", T=34),
        # The same system from nothing.
        dict(name="rhs64_f32_solve", kind="solve", N=8192, n=8192, m=64, uneven=True, k=64,
             shift=2.0, precision="f32", rtol=1e-6),
        # The mixed-precision section's system in FP32 (128 right-hand sides).
        dict(name="rhs128_f32_updates", kind="updates", N=16384, n=16384, m=64, uneven=False,
             k=128, shift=3.0, precision="f32", T=20),
        # The same system through bf16 products and FP64 refinement, to 1e-10.
        dict(name="rhs128_bf16_refine", kind="refine", N=16384, n=16384, m=64, uneven=False,
             k=128, shift=3.0, precision="bf16_ir", rtol=1e-10),
        # 256 independent systems of 64 to 1024 unknowns, one right-hand side each.
        dict(name="batch256_f32", kind="batch", count=256, lo=64, hi=1024, sizes=0, shift=2.0,
             precision="f32", T=64),
        # Differentiating a solve: the adjoint workload (200 updates unrolled).
        dict(name="adjoint_f32", kind="adjoint", N=4096, n=4096, m=32, uneven=False, k=16,
             shift=2.0, precision="f32", T=200),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["updates", "updates", "updates", "solve", "solve", "refine", "heavy_ball",
                       "batch", "adjoint"])
    if kind == "batch":
        return dict(kind=kind, count=_log_int(rng, 8, 256), lo=64, hi=rng.randint(128, 1024),
                    sizes=rng.randint(1, 10**6), shift=2.0, precision="f32",
                    T=rng.randint(48, 64))
    if kind == "adjoint":
        n = _log_int(rng, 512, 4096)
        return dict(kind=kind, N=n, n=n, m=max(4, n // rng.randint(96, 256)), uneven=False,
                    k=_log_int(rng, 4, 32), shift=rng.choice([2.0, 3.0]), precision="f32",
                    T=rng.randint(60, 150))
    k = 1
    if kind == "refine" or (kind in ("updates", "solve") and rng.random() < 0.5):
        k = _log_int(rng, 2, 128)
    square = k > 1 or rng.random() < 0.3
    top = 12288 if kind == "refine" else 8192
    n = _log_int(rng, 1024 if kind == "refine" else 200, top)
    N = n if square and rng.random() < 0.7 else min(16384, int(n * rng.uniform(1.5, 3.0)))
    # Blocks of about 40 to 300 rows, never more than half a row's width on average.
    m = max(4, N // rng.randint(40, 300), -(-2 * N // n) + 1)
    case = dict(kind=kind, N=N, n=n, m=m, uneven=rng.random() < 0.5, k=k,
                shift=(rng.choice([1.5, 2.0, 3.0]) if kind == "refine" else 2.0)
                if N == n else 0.0)
    if kind == "refine":
        return dict(case, precision="bf16_ir", rtol=1e-10)
    precision = rng.choice(["f32", "f32", "f64"])
    case = dict(case, precision=precision)
    if kind == "solve":
        return dict(case, rtol=1e-11 if precision == "f64" else 1e-6)
    if kind == "heavy_ball":
        return dict(case, k=1, plain=rng.random() < 0.5, T=rng.randint(20, 50))
    return dict(case, T=rng.randint(8, 40))


# ------------------------------------------------------------------ the systems


def _offsets(case):
    N, m, n = case["N"], case["m"], case["n"]
    if case["uneven"]:
        mean = max(1, N // m)
        sizes = synth.renormalised_sizes(np.random.default_rng(m), m, N, max(1, mean // 4),
                                         2 * mean)
    else:
        sizes = synth.even_sizes(N, m)
    return synth.offsets_from_sizes(np.minimum(sizes, min(n, 2048)))


def _edges(case):
    """The interval that the spectrum of A^T A fills for large sizes."""
    a = case["shift"]
    if a:
        q = math.sqrt(1.0 + 8.0 * a * a)
        return (q - 3.0) ** 3 / (8.0 * (q - 1.0)), (q + 3.0) ** 3 / (8.0 * (q + 1.0))
    r = math.sqrt(case["N"] / case["n"])
    return (r - 1.0) ** 2, (r + 1.0) ** 2


def _parameters(case):
    """gamma, eta of eq. (2) for an interval around the spectrum of X (Theorem 1)."""
    lo, hi = _edges(case)
    row = 1.0 + case["shift"] ** 2  # ||a row||^2
    lo, hi = 0.95 * lo / row / case["m"], min(1.0, 1.01 * hi / row / case["m"])
    a, c = math.sqrt(hi), math.sqrt(lo)
    rho, s = (a - c) / (a + c), 4.0 / (a + c) ** 2
    total = s - 1.0 - rho * rho
    v = 0.5 * (total + math.sqrt(max(total * total - 4.0 * rho * rho, 0.0)))
    return (1.0 + rho * rho / v if v > 0 else 1.0), 1.0 + v


def _heavy_ball(case):
    """Step and momentum of the heavy ball for the interval around its spectrum."""
    lo, hi = _edges(case)
    if not case["plain"]:
        row = 1.0 + case["shift"] ** 2
        lo, hi = lo / row, min(case["m"], hi / row)
    a, c = math.sqrt(1.05 * hi), math.sqrt(0.95 * lo)
    return 4.0 / (a + c) ** 2, ((a - c) / (a + c)) ** 2


def _system(N, n, k, shift, g):
    A = torch.randn(N, n, generator=g, dtype=torch.float64, device="cuda") / math.sqrt(n)
    if shift:
        A.diagonal().add_(shift)
    x = torch.randn(n, k, generator=g, dtype=torch.float64, device="cuda")
    B = A @ x
    return (A, B[:, 0].contiguous(), x[:, 0].contiguous()) if k == 1 else (A, B, x)


def _generator(seed):
    return torch.Generator(device="cuda").manual_seed(int(seed))


def _batch_sizes(case):
    rng = np.random.default_rng(case["sizes"])
    out = []
    for _ in range(case["count"]):
        n = int(rng.integers(case["lo"], case["hi"] + 1))
        out.append((n, int(rng.choice([4, 8, 16]))))
    return out


def _handed_on(case, x):
    return x.float() if case["precision"] == "f32" else x


# ------------------------------------------------------------------ the calls


def prepare(case, seed):
    g = _generator(seed)
    kind = case["kind"]
    if kind == "batch":
        plans = []
        for n, m in _batch_sizes(case):
            sub = dict(N=n, n=n, m=m, shift=case["shift"], uneven=False)
            A, b, _ = _system(n, n, 1, case["shift"], g)
            gamma, eta = _parameters(sub)
            plans.append(apc.Plan(A, b, _offsets(sub), case["precision"], gamma=gamma, eta=eta))
        return dict(case=case, plans=plans, batch=apc.Batch(plans))
    A, B, _ = _system(case["N"], case["n"], case["k"], case["shift"], g)
    off = _offsets(case)
    state = dict(case=case, A=A, B=B, off=off)
    if kind == "solve":
        return state
    if kind == "refine":
        state["plan"] = apc.Plan(A, B, off, case["precision"])
        return state
    gamma, eta = _parameters(case)
    state["plan"] = apc.Plan(A, B, off, case["precision"], gamma=gamma, eta=eta)
    if kind == "heavy_ball":
        alpha, beta = _heavy_ball(case)
        state["hbm"] = apc.HeavyBall(state["plan"],
                                     apc.APC_HBM_PLAIN if case["plain"]
                                     else apc.APC_HBM_PRECONDITIONED, alpha=alpha, beta=beta)
    if kind == "adjoint":
        state["params"] = (gamma, eta)
        state["target"] = torch.randn(_x_shape(case), generator=g, dtype=torch.float64,
                                      device="cuda")
    return state


def _x_shape(case):
    return (case["n"],) if case["k"] == 1 else (case["n"], case["k"])


def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "updates":
        plan = state["plan"]
        plan.restart(state["B"])
        plan.iterate(case["T"])
        return _handed_on(case, plan.xbar())
    if kind == "solve":
        plan = apc.Plan(state["A"], state["B"], state["off"], case["precision"])
        x = plan.solve(case["rtol"], 2000)[0]
        plan.close()
        return _handed_on(case, x)
    if kind == "refine":
        plan = state["plan"]
        plan.restart(state["B"])
        return plan.solve(case["rtol"], 5000)[0]
    if kind == "heavy_ball":
        h = state["hbm"]
        h.restart()
        h.iterate(case["T"])
        return _handed_on(case, h.x())
    if kind == "batch":
        state["batch"].iterate(case["T"])
        return _handed_on(case, torch.cat([p.xbar() for p in state["plans"]]))
    gamma, eta = state["params"]
    b = state["B"].detach().requires_grad_(True)
    x = apc.unrolled_apc(state["plan"], b, gamma, eta, case["T"])
    (0.5 * (x - state["target"]).square().sum()).backward()
    return _handed_on(case, x.detach()), _handed_on(case, b.grad)


# ------------------------------------------------------------------ what they amount to


def _factor_streams(nbytes, T):
    """Bytes of a factor over T updates: read by each one, or once when it can stay cached."""
    return nbytes * (T if nbytes > CACHE_BYTES else 1)


def work(case):
    sq = {"f64": 8, "f32": 4, "bf16_ir": 2}[case["precision"]]
    kind = case["kind"]
    if kind == "batch":
        T, nbytes, flops = case["T"], 0, 0
        for n, m in _batch_sizes(case):
            nbytes += n * n * sq
            flops += 4.0 * n * n * T
        return dict(bytes=float(_factor_streams(nbytes, T)), flops=flops)
    N, n, k = case["N"], case["n"], case["k"]
    factor, io = N * n * sq, 8.0 * (N + n) * k
    if kind in ("updates", "heavy_ball"):
        T = case["T"]
        return dict(bytes=_factor_streams(factor, T) + io, flops=4.0 * N * n * k * T)
    if kind == "adjoint":
        T = case["T"]  # forward, its recomputation from checkpoints, reverse
        return dict(bytes=_factor_streams(factor, 3 * T) + io, flops=4.0 * N * n * k * 3 * T)
    # to a tolerance: the updates Theorem 1's rate asks for
    lo, hi = _edges(case)
    kappa = hi / lo
    rho = (math.sqrt(kappa) - 1.0) / (math.sqrt(kappa) + 1.0)
    T = math.ceil(math.log(case["rtol"]) / math.log(rho))
    if kind == "refine":
        return dict(bytes=_factor_streams(factor, T) + 8.0 * N * n + io,
                    flops=4.0 * N * n * k * T)
    p2 = float(np.sum(np.diff(_offsets(case)).astype(np.float64) ** 2))
    return dict(bytes=8.0 * N * n + factor + _factor_streams(factor, T) + io,
                flops=2.0 * p2 * n + 4.0 * N * n * k * T)


# ------------------------------------------------------------------ in 64 bits, by torch alone


def _orthonormal_blocks(A, B, off):
    """Q_i^T (orthonormal rows spanning A_i's row space) and c_i with Q_i^T x = c_i."""
    out = []
    for i in range(len(off) - 1):
        Ai, Bi = A[off[i]:off[i + 1]], B[off[i]:off[i + 1]]
        L = torch.linalg.cholesky(Ai @ Ai.T)
        W = torch.linalg.solve_triangular(L, torch.cat([Ai, Bi], 1), upper=False)
        out.append((W[:, :A.shape[1]].contiguous(), W[:, A.shape[1]:].contiguous()))
    return out


def _exact_updates(A, B, off, gamma, eta, T):
    blocks = _orthonormal_blocks(A, B, off)
    m = len(blocks)
    x = [Q.T @ c for Q, c in blocks]
    xbar = sum(x) / m
    for _ in range(T):
        total = torch.zeros_like(xbar)
        for i, (Q, _) in enumerate(blocks):
            v = xbar - x[i]
            x[i] = x[i] + gamma * (v - Q.T @ (Q @ v))
            total += x[i]
        xbar = (eta / m) * total + (1.0 - eta) * xbar
    return xbar


def _exact_heavy_ball(A, B, off, plain, alpha, beta, T):
    blocks = _orthonormal_blocks(A, B, off)
    x = sum(Q.T @ c for Q, c in blocks) / len(blocks)
    z = torch.zeros_like(x)
    for _ in range(T):
        g = (A.T @ (A @ x - B) if plain
             else sum(Q.T @ (Q @ x - c) for Q, c in blocks))
        z = beta * z + g
        x = x - alpha * z
    return x


def exact(case, seed):
    g = _generator(seed)
    kind = case["kind"]
    if kind == "batch":
        return torch.cat([_system(n, n, 1, case["shift"], g)[2] for n, m in _batch_sizes(case)])
    A, B, x = _system(case["N"], case["n"], case["k"], case["shift"], g)
    off = [int(v) for v in _offsets(case)]
    B2 = B[:, None] if case["k"] == 1 else B
    if kind == "updates":
        gamma, eta = _parameters(case)
        return _exact_updates(A, B2, off, gamma, eta, case["T"]).reshape(x.shape)
    if kind == "heavy_ball":
        alpha, beta = _heavy_ball(case)
        return _exact_heavy_ball(A, B2, off, case["plain"], alpha, beta, case["T"]).reshape(x.shape)
    if kind == "adjoint":
        target = torch.randn(_x_shape(case), generator=g, dtype=torch.float64, device="cuda")
        return x, torch.linalg.solve(A.T, x - target)
    return x
