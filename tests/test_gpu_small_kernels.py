"""Dispatch edges of the small kernels against the FP64 oracle: the update with
one lane per row, the ranks at which a row's column steps are cut, the Gram's row
chunks and column-block pairs, trailing multi-TTVs over a long J, partial MTTKRPs of
small tensors cut into small groups, the 16-bit pack and scale table of one launch,
and the vector and block edges of ||X||^2 and of quantisation."""

import numpy as np
import pytest

import oracle as O

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("I", [4095, 4096, 8191, 8192, 9001])  # either side of the rule, a short last group
@pytest.mark.parametrize("R", [1, 15, 16, 17, 32])
@pytest.mark.parametrize("update,sweeps,tol", [("hals", 1, 0.0), ("mu", 2, 0.0), ("hals", 30, 1e-7)])
def test_update_of_many_rows(gpu_lib, I, R, update, sweeps, tol):
    import torch
    from paper_1806_07985_amd import native
    print(f"case update rows={I} R={R} {update} {sweeps} {tol}", flush=True)
    rng = np.random.default_rng(I + 7 * R + sweeps)
    K = rng.random((R + 20, R))
    S = K.T @ K
    if R > 2 and update == "hals":
        S[2, :] = S[:, 2] = 0.0  # a column that is zero in another mode
    M = rng.random((I, R)) * np.abs(S).sum(0) * 0.6
    M[3] = -M[3]
    H = rng.random((I, R)).astype(np.float32)
    lam = rng.random(R) + 0.5
    lam_t, G, W = native.nls_solve(torch.from_numpy(np.ascontiguousarray(M.T)).cuda(), native.factor_to_device(H), I, R,
                                   torch.from_numpy(S).cuda(), torch.from_numpy(lam).cuda(), update,
                                   max_sweeps=sweeps, tol=tol)
    ref = O.block_update(H.astype(np.float64) * lam, S, M, update, sweeps, tol)
    # FP64 throughout: R steps of R products, 2^-53 each, times the condition of S (< 1e4)
    assert np.max(np.abs(W.cpu().numpy().T - ref)) <= 1e-9 * np.max(np.abs(ref))


@pytest.mark.parametrize("R", [1, 7, 8, 9, 16, 17, 24, 25, 32, 33, 49, 56, 57, 64])
@pytest.mark.parametrize("sweeps,tol", [(1, 0.0), (30, 1e-7)])
def test_update_rank_edges(gpu_lib, R, sweeps, tol):
    import torch
    from paper_1806_07985_amd import native
    print(f"case update rank R={R} {sweeps} {tol}", flush=True)
    rng = np.random.default_rng(R + sweeps)
    I = 9
    K = rng.random((R + 20, R))
    S = K.T @ K
    if R > 2:
        S[R - 1, :] = S[:, R - 1] = 0.0
    M = rng.random((I, R)) * np.abs(S).sum(0) * 0.6
    M[3] = -M[3]
    H = rng.random((I, R)).astype(np.float32)
    lam = rng.random(R) + 0.5
    _, _, W = native.nls_solve(torch.from_numpy(np.ascontiguousarray(M.T)).cuda(), native.factor_to_device(H), I, R,
                               torch.from_numpy(S).cuda(), torch.from_numpy(lam).cuda(), "hals",
                               max_sweeps=sweeps, tol=tol)
    ref = O.block_update(H.astype(np.float64) * lam, S, M, "hals", sweeps, tol)
    assert np.max(np.abs(W.cpu().numpy().T - ref)) <= 1e-9 * np.max(np.abs(ref))  # as above


@pytest.mark.parametrize("R", [1, 16, 17, 32, 33, 48, 49, 64])
def test_gram_rows_and_chunks(gpu_lib, R):
    """Rows that end inside a group of 16 or of 4, one chunk and several."""
    from paper_1806_07985_amd import native
    rng = np.random.default_rng(R)
    for I in (1, 3, 15, 16, 17, 31, 33, 191, 193, 383, 385, 961, 3071, 3073, 50001):
        print(f"case gram I={I} R={R}", flush=True)
        H = (rng.random((I, R)) - 0.3).astype(np.float32)
        G = native.gram(native.factor_to_device(H), I, R).cpu().numpy()
        ref, size = O.gram(H.astype(np.float64)), O.gram(np.abs(H.astype(np.float64)))
        # exact products of FP32 values, FP64 sums: I roundings of 2^-53 at most
        assert np.all(np.abs(G - ref) <= 2.0 ** -53 * (I + 40) * size)
        assert np.array_equal(G, G.T)


@pytest.mark.parametrize("dims,R,split,dt", [((6, 5, 512), 3, 1, "f32"), ((6, 5, 511), 3, 1, "f32"),
                                             ((9, 65, 1100), 5, 1, "f32"), ((4, 7, 40, 37), 33, 1, "f32"),
                                             ((5, 700, 3, 2), 2, 2, "f32"), ((6, 5, 1100), 4, 1, "bf16"),
                                             ((6, 5, 383), 3, 1, "f32"), ((6, 5, 384), 3, 1, "f32"),
                                             ((4, 70, 437), 16, 1, "f32")])
def test_trailing_multi_ttv_over_long_j(gpu_lib, dims, R, split, dt):
    import torch
    from paper_1806_07985_amd import native
    print(f"case trail dims={dims} R={R} split={split} {dt}", flush=True)
    rng = np.random.default_rng(sum(dims) + R)
    X = torch.from_numpy(rng.random(int(np.prod(dims))).astype(np.float32)).to({"f32": torch.float32, "bf16": torch.bfloat16}[dt])
    X64 = X.double().numpy().reshape(dims, order="F")
    H = [rng.random((d, R)).astype(np.float32) for d in dims]
    Hd = [native.factor_to_device(h) for h in H]
    for n in range(len(dims)):
        M = native.mttkrp(X.cuda(), list(dims), split, n, Hd, R).cpu().numpy().T
        ref = O.mttkrp_direct(X64, [h.astype(np.float64) for h in H], n)
        # positive data; the partial MTTKRP's own bound (1e-6 FP32, 2e-6 16-bit plus its FP32 temporaries)
        assert np.all(np.abs(M - ref) <= 3e-6 * ref), float(np.max(np.abs(M - ref) / ref))
    # the same plan alone and in a batch, bitwise (both split the sum alike)
    out = []
    for batched in (False, True):
        Hb = [native.factor_to_device(h) for h in H]
        plan = native.Plan(X.cuda(), list(dims), R, Hb, split=split)
        if batched:
            b = native.Batch()
            b.add(plan)
            b.run(3)
            b.close()
        else:
            plan.run(3)
        out.append(Hb)
        plan.close()
    assert all(torch.equal(a, b) for a, b in zip(*out))


@pytest.mark.parametrize("dt", ["f32", "bf16", "f16"])
def test_ingest_edges(gpu_lib, dt):
    """Sizes around a vector, a group's run, and the largest grid; bases that are
    aligned to the element only."""
    import torch
    from paper_1806_07985_amd import native
    tdt = {"f32": torch.float32, "bf16": torch.bfloat16, "f16": torch.float16}[dt]
    X0 = (torch.rand(8192 * 1024 + 16400, generator=torch.Generator().manual_seed(3)) - 0.5)
    for n in (1, 3, 7, 8, 9, 255, 2047, 2049, 8191, 8192, 8193, 16383, 16385, 8192 * 1024 + 16385):
        for off in (0, 1, 3):
            print(f"case ingest {dt} n={n} offset={off}", flush=True)
            X = X0[off:off + n]
            Xd = X0.cuda()[off:off + n]
            if dt != "f32":
                Q = native.quantize(Xd, dt)
                assert torch.equal(Q.cpu().view(torch.int16), X.to(tdt).view(torch.int16))  # round to nearest even
            Xt = X0.to(tdt)
            got = native.norm_sq(Xt.cuda()[off:off + n])
            ref = float(np.sum(Xt[off:off + n].double().numpy() ** 2))
            # exact squares; at most 300 additions in a chain, 2^-53 each
            assert abs(got - ref) <= 1e-12 * ref


@pytest.mark.parametrize("dims", [(5, 4, 3), (32, 16, 16), (33, 16, 16), (64, 32, 8), (7, 90, 160), (128, 128, 127),
                                  (128, 128, 128), (512, 3, 700)])  # 240 B, 32 KiB, the ends of the rule at 8 MiB
@pytest.mark.parametrize("R", [3, 20, 40])
def test_small_tensors_in_small_groups(gpu_lib, dims, R):
    import torch
    from paper_1806_07985_amd import native
    print(f"case small groups dims={dims} R={R}", flush=True)
    rng = np.random.default_rng(sum(dims) + R)
    X = torch.from_numpy(rng.random(int(np.prod(dims))).astype(np.float32))
    H = [rng.random((d, R)).astype(np.float32) for d in dims]
    Hd = [native.factor_to_device(h) for h in H]
    X64 = X.double().numpy().reshape(dims, order="F")
    for n in range(3):
        M = native.mttkrp(X.cuda(), list(dims), 1, n, Hd, R).cpu().numpy().T
        ref = O.mttkrp_direct(X64, [h.astype(np.float64) for h in H], n)
        assert np.all(np.abs(M - ref) <= 1e-6 * ref), float(np.max(np.abs(M - ref) / ref))  # positive data, FP32 products


def test_step_calls_share_scratch_safely(gpu_lib):
    """Threads on their own streams, calls of growing and shrinking sizes: every
    result equals the one computed alone (the calls are deterministic)."""
    import threading
    import torch
    from paper_1806_07985_amd import native
    rng = np.random.default_rng(5)
    jobs = []
    for i, (dims, R) in enumerate([((9, 8, 7), 3), ((60, 50, 40), 20), ((200, 150, 130), 64), ((31, 2, 900), 48)]):
        X = torch.from_numpy(rng.random(int(np.prod(dims))).astype(np.float32)).cuda()
        H = [native.factor_to_device(rng.random((d, R)).astype(np.float32)) for d in dims]
        jobs.append((X, list(dims), R, H))

    def work(j):
        X, dims, R, H = jobs[j]
        T = [native.partial_mttkrp(X, dims, 1, side, H, R) for side in (0, 1)]
        M = [native.mttkrp(X, dims, 1, n, H, R) for n in range(3)]
        return T + M + [native.gram(H[0], dims[0], R)], native.norm_sq(X)

    alone = [work(j) for j in range(len(jobs))]
    torch.cuda.synchronize()
    bad = []

    def run(t):
        with torch.cuda.stream(torch.cuda.Stream()):
            for k in range(6):
                j = (t + k) % len(jobs)
                out, ns = work(j)
                torch.cuda.current_stream().synchronize()
                if ns != alone[j][1] or not all(torch.equal(a, b) for a, b in zip(out, alone[j][0])):
                    bad.append((t, k, j))

    threads = [threading.Thread(target=run, args=(t,)) for t in range(4)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not bad


@pytest.mark.parametrize("dims,s,side", [((3, 2100, 5), 1, 0), ((2049, 3, 7), 2, 1), ((3, 2048, 70), 1, 0),
                                         ((9, 8, 7), 1, 0), ((9, 16, 16), 1, 0), ((9, 16, 17, 2), 1, 0)])
@pytest.mark.parametrize("R", [1, 16, 33])
@pytest.mark.parametrize("dt", ["bf16", "f16"])
def test_pack_and_scale_table(gpu_lib, dims, s, side, R, dt):
    """Either size of group (first contracted extents around 2048), tables that end
    inside a group and on its end."""
    import torch
    from paper_1806_07985_amd import native
    print(f"case pack {dt} dims={dims} R={R} s={s} side={side}", flush=True)
    rng = np.random.default_rng(sum(dims) + R)
    tdt = {"bf16": torch.bfloat16, "f16": torch.float16}[dt]
    X = torch.from_numpy(rng.random(int(np.prod(dims))).astype(np.float32)).to(tdt)
    H = [rng.random((d, R)).astype(np.float32) for d in dims]
    T = native.partial_mttkrp(X.cuda(), list(dims), s, side, [native.factor_to_device(h) for h in H], R).cpu().numpy().T
    fn = O.partial_mttkrp_left if side == 0 else O.partial_mttkrp_right
    ref = fn(X.double().numpy().reshape(dims, order="F"), [h.astype(np.float64) for h in H], s).reshape(-1, R, order="F")
    # the 16-bit path's bound: 2e-6 of sum |x||k| (all positive here)
    assert np.all(np.abs(T - ref) <= 2e-6 * ref), float(np.max(np.abs(T - ref) / ref))
