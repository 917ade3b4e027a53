"""Range-checked tensor loads of the partial-MTTKRP kernels: a host walk of every
lane offset (FP32), and on the GPU ragged tensors that lie between NaNs."""

import os
import subprocess

import numpy as np
import pytest

import oracle as O

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB_DIR = os.path.join(ROOT, "paper_1806_07985_amd", "lib")
# (dims, R, split): ends of the tensor inside a k-step, a row group or a vector
SHAPES = [((1, 1, 1), 1, 1), ((1, 5, 1), 3, 2), ((3, 2), 2, 1), ((7, 11, 13), 5, 1), ((7, 11, 13), 17, 2),
          ((33, 47, 29), 16, 1), ((65, 17, 9), 33, 1), ((63, 31, 5), 20, 2), ((64, 16, 3), 8, 1), ((130, 33, 2), 50, 1),
          ((5, 3, 257), 12, 2), ((1001, 3), 64, 1)]


def test_every_offset_in_range(tmp_path):
    exe = str(tmp_path / "walker")
    cmd = [os.environ.get("HIPCC", "/opt/rocm/bin/hipcc"), "-O2", "-std=c++17", "-I", os.path.join(ROOT, "include"), "-I",
           os.path.join(ROOT, "paper_1806_07985_amd", "csrc"), os.path.join(ROOT, "tests", "pm_buffer_walker.cpp"), "-o",
           exe, "-L", LIB_DIR, "-lnncp", f"-Wl,-rpath,{LIB_DIR}"]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    lines = [f"{int(np.prod(d[:s]))} {int(np.prod(d[s:]))} {d[s]} {d[0]} {R}" for d, R, s in SHAPES]
    r = subprocess.run([exe], input="\n".join(lines) + "\n", capture_output=True, text=True, timeout=300)
    assert r.returncode == 0 and f"{len(lines)} cases" in r.stdout, r.stdout[-2000:]


@pytest.mark.gpu
@pytest.mark.parametrize("dims,R,s", SHAPES)
@pytest.mark.parametrize("side", [0, 1])
def test_ragged_tensor_between_nans(gpu_lib, dims, R, s, side):
    import torch
    from paper_1806_07985_amd import native
    print(f"case buffer loads dims={dims} R={R} s={s} side={side}", flush=True)
    rng = np.random.default_rng(sum(dims) + R + s)
    X = rng.random(dims).astype(np.float32)
    H = [rng.random((d, R)).astype(np.float32) for d in dims]
    room = torch.full((X.size + 20011,), float("nan"), device="cuda")
    Xd = room[10003:10003 + X.size]  # element-aligned only, NaN before and after
    Xd.copy_(torch.from_numpy(X.ravel(order="F")))
    T = native.partial_mttkrp(Xd, list(dims), s, side, [native.factor_to_device(h) for h in H], R).cpu().numpy().T
    fn = O.partial_mttkrp_left if side == 0 else O.partial_mttkrp_right
    ref = fn(X.astype(np.float64), [h.astype(np.float64) for h in H], s).reshape(-1, R, order="F")
    # positive data: FP32 chains of up to 2^7 products, each rounding at most 2^-24 of the sum
    assert np.all(np.abs(T - ref) <= 2.0 ** -17 * ref), float(np.max(np.abs(T - ref) / ref))


@pytest.mark.gpu
@pytest.mark.parametrize("dims,R,s", SHAPES + [((301, 70), 10, 1), ((129, 9001), 10, 1)])
@pytest.mark.parametrize("dt", ["bf16", "f16"])
def test_ragged_16bit_tensor_between_nans(gpu_lib, dims, R, s, dt):
    """The range check drops a dword that is half inside: a tensor of odd extents
    ends in one, and its last element has to count all the same."""
    import torch
    from paper_1806_07985_amd import native
    print(f"case buffer loads {dt} dims={dims} R={R} s={s}", flush=True)
    rng = np.random.default_rng(sum(dims) + R + s)
    tdt = {"bf16": torch.bfloat16, "f16": torch.float16}[dt]
    X = torch.from_numpy(rng.random(int(np.prod(dims))).astype(np.float32)).to(tdt)
    X[-1] = 100.0  # large: leaving the last element out would show
    X64 = X.double().numpy().reshape(dims, order="F")
    H = [rng.random((d, R)).astype(np.float32) for d in dims]
    Hd = [native.factor_to_device(h) for h in H]
    for at in (10002, 10003):  # even and odd element offsets
        room = torch.full((X.numel() + 20011,), float("nan"), device="cuda", dtype=tdt)
        Xd = room[at:at + X.numel()]
        Xd.copy_(X)
        for side, fn in ((0, O.partial_mttkrp_left), (1, O.partial_mttkrp_right)):
            T = native.partial_mttkrp(Xd, list(dims), s, side, Hd, R).cpu().numpy().T
            ref = fn(X64, [h.astype(np.float64) for h in H], s).reshape(-1, R, order="F")
            # the 16-bit path's bound: 2e-6 of sum |x||k| (all positive here)
            assert np.all(np.abs(T - ref) <= 2e-6 * ref), (side, at, float(np.max(np.abs(T - ref) / ref)))


@pytest.mark.gpu
@pytest.mark.parametrize("dims,s", [((33, 9, 150), 1), ((83, 3, 131), 2), ((5, 41, 301), 2), ((33, 4, 200), 2),
                                    ((33, 5, 200), 2), ((201, 90), 1), ((83, 71, 90), 2), ((129, 33001), 1),
                                    ((129, 66000), 1), ((1, 129), 1), ((15, 3, 300), 2), ((17, 3, 300), 2),
                                    ((257, 1, 3, 70), 2)])
@pytest.mark.parametrize("R", [5, 20, 40])
@pytest.mark.parametrize("dt", ["bf16", "f16"])
def test_right_node_of_odd_extent_between_nans(gpu_lib, dims, s, R, dt):
    """Columns that start in the middle of a dword: every one, or every other j."""
    import torch
    from paper_1806_07985_amd import native
    print(f"case odd extents {dt} dims={dims} R={R} s={s}", flush=True)
    rng = np.random.default_rng(sum(dims) + R + s)
    tdt = {"bf16": torch.bfloat16, "f16": torch.float16}[dt]
    X = torch.from_numpy(rng.random(int(np.prod(dims))).astype(np.float32)).to(tdt)
    X[-1] = X[0] = 100.0
    H = [rng.random((d, R)).astype(np.float32) for d in dims]
    room = torch.full((X.numel() + 20011,), float("nan"), device="cuda", dtype=tdt)
    Xd = room[10002:10002 + X.numel()]  # on a dword, NaN before and after
    Xd.copy_(X)
    T = native.partial_mttkrp(Xd, list(dims), s, 1, [native.factor_to_device(h) for h in H], R).cpu().numpy().T
    ref = O.partial_mttkrp_right(X.double().numpy().reshape(dims, order="F"), [h.astype(np.float64) for h in H], s)
    ref = ref.reshape(-1, R, order="F")
    # the 16-bit path's bound: 2e-6 of sum |x||k| (all positive here)
    assert np.all(np.abs(T - ref) <= 2e-6 * ref), float(np.max(np.abs(T - ref) / ref))
