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
