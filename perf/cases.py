"""Performance cases of the library, one pass per public entry point.

Each case is a plain dict: its kind (which entry point it calls) and the sizes,
storage type and options of that call. ``prepare`` makes what a user's program
holds before the call, ``run`` is one pass, ``work`` says what a pass cannot do
without and ``exact`` gives the same outputs in plain FP64 torch.

Kinds:

* ``nncp``    one whole decomposition call on a new problem (plan, graph and
              workspace are made inside it);
* ``run``     ``iters`` outer iterations of a plan that the program keeps, and
              the normalised result;
* ``batch``   ``iters`` ticks of a batch of many 3-way jobs;
* ``mttkrp``  the tree MTTKRP of one mode with given factors;
* ``pm``      a partial MTTKRP (one root branch of the tree);
* ``update``  one block update: a sweep, or the block NNLS problem solved to a
              tolerance;
* ``ingest``  a new FP32 tensor rounded to its storage type and its norm.
"""

from __future__ import annotations

import math

import numpy as np
import torch

from paper_1806_07985_amd import inputs, native

_TORCH = {"f32": torch.float32, "bf16": torch.bfloat16, "f16": torch.float16}
_SIZE = {"f32": 4, "bf16": 2, "f16": 2}
_HSI = (1024, 1344, 33, 9)


def _dims(text):
    return tuple(int(d) for d in text.split("x"))


def listed():
    return [
        # the smallest whole call of the tests: host work and launch latency count
        {"name": "nncp_60x50x40_r5", "kind": "nncp", "dims": "60x50x40", "dtype": "f32", "R": 5, "update": "hals",
         "iters": 20},
        # one ordinary job of the batch and serving ranges, on its own: ragged, a few MB
        {"name": "run_137x201x90_r16", "kind": "run", "dims": "137x201x90", "dtype": "f32", "R": 16,
         "update": "hals", "iters": 10},
        # bench.py's default workload: one process's share of the 4-way weak-scaling experiment
        {"name": "run_128x128x128x128_r32", "kind": "run", "dims": "128x128x128x128", "dtype": "f32", "R": 32,
         "update": "hals", "iters": 5},
        # the 5-way tensor of the large workloads: the deepest tree
        {"name": "run_64x64x64x64x64_r32", "kind": "run", "dims": "64x64x64x64x64", "dtype": "f32", "R": 32,
         "update": "hals", "iters": 3},
        # the time-lapse hyperspectral shape in 16-bit storage: long first modes, short last ones
        {"name": "run_1024x1344x33x9_bf16_r50", "kind": "run", "dims": "1024x1344x33x9", "dtype": "bf16", "R": 50,
         "update": "hals", "iters": 3},
        # the fMRI shape with fewer subjects: the largest tensor, low rank, columns tens of MB apart
        {"name": "run_30012x1200x48_bf16_r10", "kind": "run", "dims": "30012x1200x48", "dtype": "bf16", "R": 10,
         "update": "hals", "iters": 2},
        # the other 16-bit type, the other update rule, ragged in every mode
        {"name": "run_83x71x57x45_f16_r24_mu", "kind": "run", "dims": "83x71x57x45", "dtype": "f16", "R": 24,
         "update": "mu", "iters": 10},
        # the batch workload: 256 3-way jobs advanced together
        {"name": "batch_256_jobs", "kind": "batch", "jobs": 256, "iters": 2},
        # programs with an update loop of their own: one mode's MTTKRP of a ragged 5-way tensor
        {"name": "mttkrp_37x29x31x23x19_r16", "kind": "mttkrp", "dims": "37x29x31x23x19", "dtype": "f32", "R": 16,
         "split": 2, "mode": 2},
        # a partial MTTKRP past rank 64 (two column chunks)
        {"name": "pm_400x300x200_r96", "kind": "pm", "dims": "400x300x200", "dtype": "f32", "R": 96, "split": 1,
         "side": 1},
        # an exact block update at the size of the hyperspectral shape's longest mode
        {"name": "nls_solve_1344_r50", "kind": "update", "rows": 1344, "R": 50, "update": "hals", "sweeps": 50,
         "tol": 1e-6},
        # a tensor brought in for 16-bit storage
        {"name": "ingest_1024x1344x33_bf16", "kind": "ingest", "dims": "1024x1344x33", "dtype": "bf16"},
    ]


def _draw_dims(rng, lo, hi, orders):
    """Dims of a tensor of log-uniform size, log I split over the modes as a
    Dirichlet draw (the serving stream's recipe), each at least 4."""
    n = rng.choice(orders)
    log_i = rng.uniform(math.log(lo), math.log(hi))
    w = [rng.gammavariate(1.0, 1.0) for _ in range(n)]
    return [max(4, round(math.exp(log_i * v / sum(w)))) for v in w]


def draw(rng):
    kind = rng.choices(["run", "nncp", "batch", "mttkrp", "pm", "update", "ingest"], [45, 13, 10, 10, 10, 7, 5])[0]
    if kind == "batch":
        return {"kind": kind, "jobs": rng.randint(8, 256), "iters": rng.randint(1, 2)}
    if kind == "update":
        rows = round(math.exp(rng.uniform(math.log(9), math.log(30012))))
        sweeps = rng.choice([1, 1, 4, 50])
        return {"kind": kind, "rows": rows, "R": rng.choice([5, 8, 10, 16, 20, 32, 50, 64, 96]),
                "update": rng.choice(["hals", "hals", "hals", "mu"]), "sweeps": sweeps,
                "tol": 1e-6 if sweeps == 50 else 0.0}
    if kind == "ingest":
        d = _draw_dims(rng, 1e4, 2e8, (3, 4, 5))
        return {"kind": kind, "dims": "x".join(map(str, d)), "dtype": rng.choice(["bf16", "f16"])}
    small = kind in ("nncp", "mttkrp", "pm")
    d = _draw_dims(rng, 1e4 if small else 1e5, 3e7 if small else 2e8, (3, 4, 5))
    case = {"kind": kind, "dims": "x".join(map(str, d)), "dtype": rng.choice(["f32", "f32", "bf16", "f16"]),
            "R": rng.choice([5, 8, 10, 16, 20, 32, 50, 64])}
    if kind in ("run", "nncp"):
        case["update"] = rng.choice(["hals", "hals", "hals", "mu"])
        case["iters"] = rng.randint(5, 30) if kind == "nncp" else rng.randint(1, 5)
    else:
        case["split"] = rng.randint(1, len(d) - 1)
        if kind == "mttkrp":
            case["mode"] = rng.randrange(len(d))
        else:
            case["side"] = rng.randint(0, 1)
    return case


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------

def _tensor(case, seed):
    """The case's tensor in its storage type (flat, mode 1 fastest)."""
    dims, dt = _dims(case["dims"]), case["dtype"]
    R = case.get("R", 16)
    if dims == _HSI:
        X = inputs.hsi_like_device(dims, R, 0.02, seed=seed)
    elif math.prod(dims) > 1 << 30:
        return inputs.planted_device_slabs(dims, R, 0.01, seed=seed, dtype=dt)
    else:
        X = inputs.planted_device(dims, R, 0.01, seed=seed)
    return X if dt == "f32" else X.to(_TORCH[dt])


def _start(dims, R, seed):
    """Starting factors U[0, 1), each (R, I_n) on the device."""
    g = torch.Generator(device="cuda")
    g.manual_seed(seed + 1)
    return [torch.rand((R, d), generator=g, device="cuda") for d in dims]


def _batch_jobs(case, seed):
    """Shapes, tensors and starting factors of a batch. All factors are views
    into one flat buffer, 256 bytes aligned."""
    shapes = inputs.batch_shapes(case["jobs"], seed=9)
    total = sum((R * d + 63) // 64 * 64 for dims, R in shapes for d in dims)
    flat = torch.zeros(total, device="cuda")
    jobs, at = [], 0
    for j, (dims, R) in enumerate(shapes):
        X = inputs.planted_device(dims, R, 0.01, seed=seed * 1000 + j)
        H = []
        for h in _start(dims, R, seed * 1000 + j):
            v = flat[at:at + h.numel()].view(R, -1)
            v.copy_(h)
            H.append(v)
            at += (h.numel() + 63) // 64 * 64
        jobs.append((dims, R, X, H))
    return flat, jobs


def _block(case, seed):
    """One block subproblem: the other modes' Gram product S, M = W_true S plus
    noise, the factor before the update (unit columns) and its weights."""
    n, R = case["rows"], case["R"]
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    S = torch.ones((R, R), dtype=torch.float64, device="cuda")
    for d in (200, 150):
        A = torch.rand((d, R), generator=g, device="cuda", dtype=torch.float64)
        A /= torch.linalg.vector_norm(A, dim=0)
        S *= A.T @ A
    W = torch.rand((n, R), generator=g, device="cuda", dtype=torch.float64)
    W *= torch.rand((n, R), generator=g, device="cuda") < 0.7
    M = W @ S
    M += 0.01 * M.mean() * torch.randn((n, R), generator=g, device="cuda", dtype=torch.float64)
    H = torch.rand((n, R), generator=g, device="cuda", dtype=torch.float64)
    lam = torch.linalg.vector_norm(H, dim=0)
    return dict(S=S, M=M.T.contiguous(), H0=(H / lam).T.contiguous().float(), lam=lam)


def prepare(case, seed):
    kind = case["kind"]
    if kind == "batch":
        flat, jobs = _batch_jobs(case, seed)
        plans = [native.Plan(X, list(dims), R, H) for dims, R, X, H in jobs]
        batch = native.Batch()
        for p in plans:
            batch.add(p)
        return dict(case=case, flat=flat, plans=plans, batch=batch)
    if kind == "update":
        b = _block(case, seed)
        return dict(case=case, H=torch.empty_like(b["H0"]), **b)
    if kind == "ingest":
        return dict(case=case, X=_tensor(dict(case, dtype="f32"), seed))
    dims, R = list(_dims(case["dims"])), case["R"]
    state = dict(case=case, dims=dims, X=_tensor(case, seed), H=_start(dims, R, seed))
    if kind == "run":
        state["plan"] = native.Plan(state["X"], dims, R, state["H"], update=case["update"])
    return state


# ---------------------------------------------------------------------------
# one pass
# ---------------------------------------------------------------------------

def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "nncp":
        out = native.nncp(state["X"], state["dims"], case["R"], case["iters"], state["H"], update=case["update"])
        return {"H": state["H"], "lam": out["lam"], "fit": out["fit"]}
    if kind == "run":
        fit = state["plan"].run(case["iters"])
        return {"fit": fit, "lam": state["plan"].finish(), "H": state["H"]}
    if kind == "batch":
        state["batch"].run(case["iters"])
        return state["flat"]
    if kind == "mttkrp":
        return native.mttkrp(state["X"], state["dims"], case["split"], case["mode"], state["H"], case["R"])
    if kind == "pm":
        return native.partial_mttkrp(state["X"], state["dims"], case["split"], case["side"], state["H"], case["R"])
    if kind == "update":
        H = state["H"].copy_(state["H0"])  # the factor as the program's last iteration left it
        if case["sweeps"] == 1:
            lam, G = native.nls_update(state["M"], H, case["rows"], case["R"], state["S"], state["lam"],
                                       update=case["update"])
            return {"H": H, "lam": lam, "G": G}
        lam, G, W = native.nls_solve(state["M"], H, case["rows"], case["R"], state["S"], state["lam"],
                                     update=case["update"], max_sweeps=case["sweeps"], tol=case["tol"])
        return {"H": H, "lam": lam, "G": G, "W": W}
    Xq = native.quantize(state["X"], case["dtype"])
    return {"X": Xq, "norm_sq": native.norm_sq(Xq)}


# ---------------------------------------------------------------------------
# what a pass cannot do without
# ---------------------------------------------------------------------------

def _iteration_work(dims, R, size):
    """One outer iteration: the tensor read for each of the two root branches,
    every factor read and written; the products of both branches, and per mode
    the update and the Gram."""
    entries = math.prod(dims)
    b = 2 * entries * size + 8 * R * sum(dims)
    f = 4 * entries * R + sum(4 * d * R * R for d in dims)
    return b, f


def work(case):
    kind = case["kind"]
    if kind == "batch":
        b = f = 0
        for dims, R in inputs.batch_shapes(case["jobs"], seed=9):
            bj, fj = _iteration_work(dims, R, 4)
            b, f = b + bj, f + fj
        return {"bytes": b * case["iters"], "flops": f * case["iters"]}
    if kind == "update":
        n, R = case["rows"], case["R"]
        # (each row sweeps until it stops; one sweep is what none goes without)
        return {"bytes": n * R * (8 + 4 + 4 + (8 if case["sweeps"] > 1 else 0)) + 16 * R * R, "flops": 4 * n * R * R}
    entries = math.prod(_dims(case["dims"]))
    size = _SIZE[case["dtype"]]
    if kind == "ingest":
        return {"bytes": entries * (4 + size), "flops": 2 * entries}
    dims, R = _dims(case["dims"]), case["R"]
    if kind in ("run", "nncp"):
        b, f = _iteration_work(dims, R, size)
        return {"bytes": b * case["iters"], "flops": f * case["iters"]}
    if kind == "mttkrp":
        rows = dims[case["mode"]]
    else:
        rows = math.prod(dims[:case["split"]] if case["side"] == 0 else dims[case["split"]:])
    return {"bytes": entries * size + 4 * R * sum(dims) + 8 * R * rows, "flops": 2 * entries * R}


# ---------------------------------------------------------------------------
# the same outputs in 64 bits
# ---------------------------------------------------------------------------

def _krp(Hs):
    """Khatri-Rao rows of factors (I x R), the first one's index fastest."""
    K = Hs[0]
    for h in Hs[1:]:
        K = (h[:, None, :] * K[None, :, :]).reshape(-1, K.shape[1])
    return K


def _partial(X, dims, s, side, H):
    """Rows x R partial MTTKRP of the flat FP64 tensor X."""
    Xm = X.view(math.prod(dims[s:]), math.prod(dims[:s]))
    return Xm.T @ _krp(H[s:]) if side == 0 else Xm @ _krp(H[:s])


def _mttkrp(X, dims, n, H):
    """MTTKRP of mode n: the smaller of its two one-sided temporaries, then the
    other modes contracted column by column."""
    N, R = len(dims), H[0].shape[1]
    left, right = math.prod(dims[:n + 1]), math.prod(dims[n:])
    if n == 0 or (n < N - 1 and left <= right):
        T = _partial(X, dims, n + 1, 0, H)
        if n == 0:
            return T
        return (T.view(dims[n], -1, R) * _krp(H[:n])[None, :, :]).sum(1)
    T = _partial(X, dims, n, 1, H)
    if n == N - 1:
        return T
    return (T.view(-1, dims[n], R) * _krp(H[n + 1:])[:, None, :]).sum(0)


def _sweeps(W, M, S, update, sweeps=1, tol=0.0):
    """Up to `sweeps` update sweeps of every row, a row stopping once a sweep
    changes none of its entries by more than tol times its largest."""
    live = torch.ones(W.shape[0], dtype=torch.bool, device=W.device)
    for _ in range(sweeps):
        old = W
        if update == "mu":
            new = W * M / (W @ S).clamp_min(1e-16)
        else:
            new = W.clone()
            for r in range(W.shape[1]):
                d = S[r, r]
                step = (M[:, r] - new @ S[:, r]) / torch.where(d > 0, d, torch.ones_like(d))
                new[:, r] = torch.where(d > 0, (new[:, r] + step).clamp_min(0.0), torch.zeros_like(step))
        W = torch.where(live[:, None], new, old)
        if tol > 0:
            live &= (W - old).abs().amax(1) > tol * W.abs().amax(1)
            if not bool(live.any()):
                break
    return W


def _unit(W):
    lam = torch.linalg.vector_norm(W, dim=0)
    return torch.where(lam > 0, W / torch.where(lam > 0, lam, torch.ones_like(lam)), torch.zeros_like(W)), lam


def _decompose(X, dims, H, update, iters):
    """`iters` outer iterations from the factors H (R x I_n, any scaling, unit
    weights). Returns unit factors, weights, the fits and the unnormalised blocks."""
    X = X.double()
    alpha = float(X @ X)
    pairs = [_unit(h.double().T) for h in H]
    F = [p[0] for p in pairs]
    lam = torch.stack([p[1] for p in pairs]).prod(0)
    blocks, fits = [None] * len(dims), []
    for _ in range(iters):
        for n in range(len(dims)):
            S = torch.ones_like(F[0].T @ F[0])
            for k, f in enumerate(F):
                if k != n:
                    S = S * (f.T @ f)
            M = _mttkrp(X, dims, n, F)
            blocks[n] = _sweeps(F[n] * lam, M, S, update)
            F[n], lam = _unit(blocks[n])
        W = blocks[-1]
        num = alpha - 2.0 * float((M * W).sum()) + float((S * (W.T @ W)).sum())
        fits.append(1.0 - math.sqrt(max(0.0, num) / alpha))
    return F, lam, np.array(fits), blocks


def exact(case, seed):
    kind = case["kind"]
    if kind == "batch":
        flat, jobs = _batch_jobs(case, seed)
        out = flat.double()
        at = 0
        for dims, R, X, H in jobs:
            for W in _decompose(X, dims, H, "hals", case["iters"])[3]:
                out[at:at + W.numel()] = W.T.reshape(-1)
                at += (W.numel() + 63) // 64 * 64
        return out
    if kind == "update":
        b = _block(case, seed)
        S, M, W = b["S"], b["M"].T, b["H0"].double().T * b["lam"]
        W = _sweeps(W, M, S, case["update"], case["sweeps"], case["tol"])
        H, lam = _unit(W)
        out = {"H": H.T.contiguous(), "lam": lam, "G": H.T @ H}
        if case["sweeps"] > 1:
            out["W"] = W.T.contiguous()
        return out
    if kind == "ingest":
        X = _tensor(dict(case, dtype="f32"), seed)
        Xq = X.to(_TORCH[case["dtype"]]).double()
        return {"X": X.double(), "norm_sq": float(Xq @ Xq)}
    dims, R = _dims(case["dims"]), case["R"]
    X = _tensor(case, seed)
    H = _start(dims, R, seed)
    if kind in ("nncp", "run"):
        F, lam, fit, _ = _decompose(X, dims, H, case["update"], case["iters"])
        return {"H": [f.T.contiguous() for f in F], "lam": lam.cpu().numpy(), "fit": fit}
    H = [h.double().T for h in H]
    if kind == "mttkrp":
        return _mttkrp(X.double(), dims, case["mode"], H).T.contiguous()
    return _partial(X.double(), dims, case["split"], case["side"], H).T.contiguous()
