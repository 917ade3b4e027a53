"""Partial MTTKRPs of tensors whose matricisation has columns of tens of MB and
more (masked loads: lane offsets past 31 bits) or a first contracted factor past 2^28
entries. Small integers, so that every product and sum is exact and the result has to
be equal; NaNs before and after the tensor."""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _check(dims, s, side, R, dt, density, offset=10003):
    import torch
    from paper_1806_07985_amd import native
    print(f"case exact integers {dt} dims={dims} s={s} side={side} R={R}", flush=True)
    tdt = {"f32": torch.float32, "bf16": torch.bfloat16, "f16": torch.float16}[dt]
    g = torch.Generator(device="cuda")
    g.manual_seed(sum(dims) + R)
    n = int(np.prod(dims))
    room = torch.full((n + 20011,), float("nan"), device="cuda", dtype=tdt)
    X = room[offset:offset + n]
    X.copy_((torch.rand(n, device="cuda", generator=g) < density) * torch.randint(1, 4, (n,), device="cuda", generator=g))
    X[0] = X[-1] = 3
    H = [torch.randint(0, 3, (R, d), device="cuda", generator=g).float() for d in dims]
    T = native.partial_mttkrp(X, list(dims), s, side, H, R)
    Xm = X.view(int(np.prod(dims[s:])), -1)  # row c: column c of the matricisation
    for r in range(R):
        k = torch.ones(1, device="cuda", dtype=torch.float64)
        for h in (H[s:] if side == 0 else H[:s]):  # first contracted mode fastest
            k = (h[r].double()[:, None] * k[None, :]).reshape(-1)
        if side == 1:
            ref = torch.stack([(row.double() * k).sum() for row in Xm]) if Xm.shape[0] < 64 else Xm.double() @ k
        else:
            ref = torch.zeros(Xm.shape[1], device="cuda", dtype=torch.float64)
            for c in range(Xm.shape[0]):
                ref += Xm[c].double() * k[c]
        assert float(ref.max()) < 2 ** 24  # FP32 sums stay exact
        assert torch.equal(T[r].double(), ref), (r, int((T[r].double() != ref).sum()))


@pytest.mark.parametrize("R", [5, 20])
def test_first_factor_past_31_bit_offsets(gpu_lib, R):
    _check((9000001 if R > 16 else 17000001, 3), 1, 1, R, "f32", 0.02)


# masked loads: ragged, lane offsets past 31 bits (one j and several, each column-block count)
@pytest.mark.parametrize("dims,s,side,R,dt", [
    ((9000001, 3), 1, 1, 5, "f32"), ((3001, 3001, 3), 2, 1, 20, "f32"), ((4201, 4201, 3), 2, 1, 40, "f32"),
    ((6001, 6001, 3, 2), 2, 0, 5, "f32"), ((6001, 6001, 3), 2, 0, 20, "f32"), ((6001, 6001, 2), 2, 0, 33, "f32"),
    ((4201, 4201, 3), 2, 1, 5, "bf16"), ((4201, 4201, 3), 2, 1, 20, "f16"), ((4201, 4201, 2), 2, 1, 40, "bf16"),
    ((17000001, 2), 1, 1, 5, "f16"), ((6001, 6001, 3, 2), 2, 0, 5, "f16"), ((6001, 6001, 3), 2, 0, 20, "bf16"),
    ((6001, 6001, 2), 2, 0, 33, "f16")])
def test_columns_past_31_bit_offsets(gpu_lib, dims, s, side, R, dt):
    _check(dims, s, side, R, dt, 0.02)


# 16-bit right nodes with one j, K split over i1 blocks, several tiles per group; the last
# i1 block, tile group and tile ragged, on a dword and not
@pytest.mark.parametrize("dims", [(6501, 33000), (6500, 33001), (3201, 70001)])
@pytest.mark.parametrize("R", [10, 20])
@pytest.mark.parametrize("dt", ["bf16", "f16"])
@pytest.mark.parametrize("offset", [10002, 10003])
def test_j1_nodes_that_split_k_over_several_tiles(gpu_lib, dims, R, dt, offset):
    _check(dims, 1, 1, R, dt, 0.5, offset)


@pytest.mark.parametrize("t", [1, 3, 4, 5, 15, 16, 17, 19, 20, 21, 31, 32, 37])
@pytest.mark.parametrize("R", [3, 40])
def test_split_sums_of_every_length(gpu_lib, t, R):
    """About t splits over K: the sum's runs of sixteen, of four and its rest."""
    _check((16, 64 * t, 7), 2, 1, R, "f32", 0.5)
    _check((16, 64 * t, 7), 2, 1, R, "bf16", 0.5)


@pytest.mark.parametrize("dims,dt", [((30013, 1200, 84), "f32"), ((30012, 1200, 168), "bf16"), ((30012, 1200, 168), "f16")])
@pytest.mark.parametrize("R", [10, 20, 33])
def test_left_nodes_of_tensors_past_12_gb(gpu_lib, dims, dt, R):
    """A left node that is streamed (12.1 GB) against the sum of its two halves along
    the last mode, which are not: exact integers, so the sums are equal."""
    import torch
    from paper_1806_07985_amd import native
    print(f"case past 12 GB {dt} dims={dims} R={R}", flush=True)
    g = torch.Generator(device="cuda")
    g.manual_seed(R)
    n, half = int(np.prod(dims)), int(np.prod(dims)) // 2
    X = torch.empty(n, device="cuda", dtype={"f32": torch.float32, "bf16": torch.bfloat16, "f16": torch.float16}[dt])
    for i in range(0, n, 1 << 29):
        part = X[i:i + (1 << 29)]
        part.copy_(torch.rand(part.numel(), device="cuda", generator=g) < 0.02)
    X[-1] = 3
    H = [torch.randint(0, 3, (R, d), device="cuda", generator=g).float() for d in dims]
    k = dims[2] // 2
    T = native.partial_mttkrp(X, list(dims), 1, 0, H, R)
    a = native.partial_mttkrp(X[:half], [dims[0], dims[1], k], 1, 0, [H[0], H[1], H[2][:, :k].contiguous()], R)
    b = native.partial_mttkrp(X[half:], [dims[0], dims[1], k], 1, 0, [H[0], H[1], H[2][:, k:].contiguous()], R)
    assert float(T.max()) < 2 ** 24 and float(T.max()) > 0
    assert torch.equal(T, a + b)
