"""What the launches of an iteration write stays inside the region of the
workspace that was reserved for it (host check over random plans), and shapes
whose second chunk of 64 columns is split where the first is not, against the
oracle on the GPU."""

import os
import subprocess

import numpy as np
import pytest

import oracle as O

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB_DIR = os.path.join(ROOT, "paper_1806_07985_amd", "lib")


@pytest.fixture(scope="module")
def walker(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("ws") / "workspace_walker")
    cmd = [os.environ.get("HIPCC", "/opt/rocm/bin/hipcc"), "-O1", "-std=c++17", "-I", os.path.join(ROOT, "include"), "-I",
           os.path.join(ROOT, "paper_1806_07985_amd", "csrc"), os.path.join(ROOT, "tests", "workspace_walker.cpp"), "-o",
           exe, "-L", LIB_DIR, "-lnncp", f"-Wl,-rpath,{LIB_DIR}"]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    return exe


def _random_plans(n, ranks):
    rng = np.random.default_rng(4)
    lines = []
    for _ in range(n):
        N = int(rng.integers(2, 6))
        w = rng.gamma(1.0, 1.0, size=N)
        size = np.exp(rng.uniform(np.log(1e4), np.log(3e7)))
        dims = [max(1, round(size ** (v / w.sum()))) for v in w]
        lines.append(f"{rng.integers(0, 3)} {rng.choice(ranks)} {rng.integers(0, N)} {int(rng.random() < 0.3)} "
                     f"{rng.choice([0, 0, 0, 32, 16384])} {N} " + " ".join(map(str, dims)))
    return lines


# second chunk split over K, the first not (or less); ragged, every storage type
PAST_64 = [((101, 18, 33), 96, 0), ((100, 6, 8, 40), 96, 0), ((400, 300, 200), 96, 1), ((57, 31, 20), 72, 0),
           ((64, 40, 24, 10), 80, 0), ((20, 18, 22), 100, 0), ((33, 1100, 9), 128, 0), ((90, 33, 7, 5, 3), 65, 0)]


@pytest.mark.parametrize("ranks", [(5, 16, 20, 32, 33, 50, 64), (65, 72, 80, 96, 97, 112, 128)])
def test_every_write_ends_inside_its_region(walker, ranks):
    lines = _random_plans(6000, ranks)
    if ranks[-1] > 64:
        lines += [f"{dt} {R} {s} {nt} 0 {len(d)} " + " ".join(map(str, d)) for d, R, s in PAST_64 for dt in range(3)
                  for nt in (0, 1)]
    r = subprocess.run([walker], input="\n".join(lines) + "\n", capture_output=True, text=True, timeout=600)
    bad = [ln for ln in r.stdout.splitlines() if ln.startswith(("FAIL", "  "))]
    assert r.returncode == 0 and f"{len(lines)} cases, 0 failed" in r.stdout, "\n".join(x.split(" route")[0] for x in bad[:20])


@pytest.mark.gpu
@pytest.mark.parametrize("dims,R,s", PAST_64)
@pytest.mark.parametrize("dt", ["f32", "bf16", "f16"])
def test_mttkrp_past_rank_64(gpu_lib, dims, R, s, dt):
    import torch
    from paper_1806_07985_amd import native
    print(f"case past 64 {dt} dims={dims} R={R} s={s}", flush=True)
    rng = np.random.default_rng(sum(dims) + R)
    tdt = {"f32": torch.float32, "bf16": torch.bfloat16, "f16": torch.float16}[dt]
    X = torch.from_numpy(rng.random(int(np.prod(dims))).astype(np.float32)).to(tdt)
    X64 = X.double().numpy().reshape(dims, order="F")
    H = [rng.random((d, R)).astype(np.float32) for d in dims]
    H64 = [h.astype(np.float64) for h in H]
    Hd = [native.factor_to_device(h) for h in H]
    # positive data; the partial MTTKRP's own bound (1e-6 FP32, 2e-6 16-bit) plus the 16-bit path's FP32 temporaries
    tol = 1e-6 if dt == "f32" else 3e-6
    s = s or min(range(1, len(dims)), key=lambda k: int(np.prod(dims[:k])) + int(np.prod(dims[k:])))
    for side, fn in ((0, O.partial_mttkrp_left), (1, O.partial_mttkrp_right)):
        T = native.partial_mttkrp(X.cuda(), list(dims), s, side, Hd, R).cpu().numpy().T
        ref = fn(X64, H64, s).reshape(-1, R, order="F")
        assert np.all(np.abs(T - ref) <= tol * ref), (side, float(np.max(np.abs(T - ref) / ref)))
    for n in range(len(dims)):
        M = native.mttkrp(X.cuda(), list(dims), s, n, Hd, R).cpu().numpy().T
        ref = O.mttkrp_direct(X64, H64, n)
        assert np.all(np.abs(M - ref) <= tol * ref), (n, float(np.max(np.abs(M - ref) / ref)))


@pytest.mark.gpu
@pytest.mark.parametrize("dims,R", [((101, 18, 33), 96), ((100, 6, 8, 40), 96), ((57, 31, 20), 72)])
@pytest.mark.parametrize("no_tree", [False, True])
def test_whole_runs_past_rank_64(gpu_lib, dims, R, no_tree):
    from paper_1806_07985_amd import inputs, native
    print(f"case run past 64 dims={dims} R={R} no_tree={no_tree}", flush=True)
    X, _ = inputs.planted(dims, 5, 0.01, seed=3, dtype=np.float32)
    H0 = [h.astype(np.float32) for h in inputs.init_factors(dims, R, seed=4)]
    Hd = [native.factor_to_device(h) for h in H0]
    out = native.nncp(native.tensor_to_device(X), list(dims), R, 1, Hd, no_tree=no_tree)
    ref = O.nncp(X.astype(np.float64), [h.astype(np.float64) for h in H0], 1)
    # one iteration; the bound of whole trajectories (tolerances.py)
    assert abs(out["fit"][-1] - ref["fit"][-1]) <= 1e-5
    for h, hr in zip(Hd, ref["H"]):
        assert np.linalg.norm(native.factor_to_host(h) - hr) <= 1e-5 * np.linalg.norm(hr)
