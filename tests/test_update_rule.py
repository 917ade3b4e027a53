"""The rows from which the update takes one lane per row: the line moves with the
sweeps, and both sides of it agree with the oracle."""

import ctypes

import numpy as np
import pytest

import oracle as O

UPDATE = {"hals": 0, "mu": 1}


def _line(R, update, sweeps, tol=0.0):
    from paper_1806_07985_amd import native
    f = native.lib()._ZN5nncpk16update_lane_rowsEiiid  # nncpk::update_lane_rows(int, int, int, double)
    f.argtypes, f.restype = [ctypes.c_int] * 3 + [ctypes.c_double], ctypes.c_int64
    return f(R, UPDATE[update], sweeps, tol)


def test_the_line_moves_with_the_sweeps():
    """A lane's work per sweep grows with R^2, a wave's with R: with many sweeps a
    wave per row is the faster one up to about 15000 rows (R = 16) or 30000 (R = 32)."""
    for R, one, many in ((1, 4096, 4096), (10, 4096, 9200), (16, 4096, 14720), (20, 8192, 24533), (32, 8192, 29440)):
        lines = [_line(R, "hals", s) for s in (1, 2, 4, 8, 50, 100000)]
        assert lines[0] == _line(R, "hals", 0) == one and lines == sorted(lines) and abs(lines[-1] - many) <= 2
        assert all(one <= _line(R, "hals", s, 1e-6) <= v for s, v in zip((1, 2, 4, 8, 50, 100000), lines))
    for R, one, many in ((5, 4096, 7667), (16, 6000, 24533), (32, 12000, 49067)):
        assert _line(R, "mu", 1) == one and abs(_line(R, "mu", 100000) - many) <= 2


@pytest.mark.gpu
@pytest.mark.parametrize("R", [3, 16, 17, 32])
@pytest.mark.parametrize("update,sweeps,tol", [("hals", 2, 0.0), ("hals", 4, 1e-7), ("hals", 30, 1e-7), ("mu", 1, 0.0), ("mu", 9, 0.0)])
@pytest.mark.parametrize("below", [0, 1])
def test_update_on_either_side_of_the_line(gpu_lib, R, update, sweeps, tol, below):
    import torch
    from paper_1806_07985_amd import native
    I = _line(R, update, sweeps, tol) - below
    print(f"case update line rows={I} R={R} {update} {sweeps} {tol}", flush=True)
    rng = np.random.default_rng(I + 7 * R + sweeps)
    K = rng.random((R + 20, R))
    S = K.T @ K
    M = rng.random((I, R)) * np.abs(S).sum(0) * 0.6
    H = rng.random((I, R)).astype(np.float32)
    lam = rng.random(R) + 0.5
    _, _, W = native.nls_solve(torch.from_numpy(np.ascontiguousarray(M.T)).cuda(), native.factor_to_device(H), I, R,
                               torch.from_numpy(S).cuda(), torch.from_numpy(lam).cuda(), update, max_sweeps=sweeps, tol=tol)
    ref = O.block_update(H.astype(np.float64) * lam, S, M, update, sweeps, tol)
    # FP64 throughout: R steps of R products, 2^-53 each, times the condition of S (< 1e4)
    assert np.max(np.abs(W.cpu().numpy().T - ref)) <= 1e-9 * np.max(np.abs(ref))
