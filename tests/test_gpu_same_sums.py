"""A job gives the same bits however it is advanced: a whole call, a plan in one
run or in pieces, with phase timers, and (rank <= 64) in a batch beside other jobs,
whose tick is a HIP graph."""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dims,R,kw", [((60, 50, 40), 5, {}), ((33, 21, 10, 9), 40, {"update": "mu"}),
                                       ((6, 5, 1100), 4, {"split": 1}), ((57, 31, 20), 72, {}),
                                       ((30, 20, 25), 8, {"no_tree": True}), ((24, 20, 17), 8, {"inner_sweeps": 7}),
                                       ((4, 3, 60001), 20, {"split": 2}),  # more than 32 row chunks
                                       ((9301, 8, 5), 10, {"inner_sweeps": 7, "split": 1}),  # either side of the update's line
                                       ((16, 640, 7), 5, {"split": 2, "pm_wg_kib": 4})])  # sums over many splits
@pytest.mark.parametrize("dt", ["f32", "bf16"])
def test_same_bits_by_every_route(gpu_lib, dims, R, kw, dt):
    import torch
    from paper_1806_07985_amd import native
    print(f"case same bits {dt} dims={dims} R={R} {kw}", flush=True)
    rng = np.random.default_rng(sum(dims) + R)
    X = torch.from_numpy(rng.random(int(np.prod(dims)), dtype=np.float32)).to({"f32": torch.float32, "bf16": torch.bfloat16}[dt]).cuda()
    H0 = [torch.from_numpy(rng.random((R, d), dtype=np.float32)).cuda() for d in dims]
    iters = 6
    H = [h.clone() for h in H0]
    out = native.nncp(X, list(dims), R, iters, H, **kw)
    routes = {}
    for name, extra, pieces in (("one run", {}, (6,)), ("pieces", {}, (1, 3, 2)), ("phase timers", {"phase_timers": True}, (6,))):
        Hp = [h.clone() for h in H0]
        plan = native.Plan(X, list(dims), R, Hp, **kw, **extra)
        fits = np.concatenate([plan.run(n) for n in pieces])
        routes[name] = (plan.finish(), fits, Hp)
        plan.close()
    if R <= 64:
        other = native.Plan(X, list(dims), R, [h.clone() for h in H0], update="hals")
        Hp = [h.clone() for h in H0]
        plan = native.Plan(X, list(dims), R, Hp, **kw)
        batch = native.Batch()
        batch.add(other)
        batch.add(plan)
        batch.run(2)
        batch.remove(other)  # members leave between ticks
        batch.run(4)
        batch.close()
        routes["batch"] = (plan.finish(), plan.fits(), Hp)
        other.close()
        plan.close()
    for name, (lam, fits, Hp) in routes.items():
        assert np.array_equal(lam, out["lam"]), name
        assert np.array_equal(fits, out["fit"]), name
        assert all(torch.equal(a, b) for a, b in zip(Hp, H)), name
