"""The step calls' kept scratch is bounded and can be given back."""

import pytest


def test_release_without_a_device_or_kept_scratch():
    from paper_1806_07985_amd import native
    native.release_scratch()
    native.release_scratch()


@pytest.mark.gpu
def test_release_gives_the_memory_back(gpu_lib):
    import torch
    from paper_1806_07985_amd import native
    dims, R = [60, 50, 4000], 64
    X = torch.rand(60 * 50 * 4000, device="cuda")
    H = [torch.rand((R, d), device="cuda") for d in dims]
    first = native.mttkrp(X, dims, 1, 0, H, R)
    torch.cuda.synchronize()
    native.release_scratch()
    empty = torch.cuda.mem_get_info()[0]
    for d in ([60, 50, 4000], [60, 50, 40], [60, 50, 400]):  # blocks of several sizes
        n = d[0] * d[1] * d[2]
        native.mttkrp(X[:n], d, 1, 0, [h[:, :k].contiguous() for h, k in zip(H, d)], R)
    torch.cuda.synchronize()
    held = empty - torch.cuda.mem_get_info()[0]
    native.release_scratch()
    assert 0 <= held <= (2 * 64 << 20) + (64 << 20)  # two blocks, and what torch's own allocator took
    assert torch.cuda.mem_get_info()[0] >= empty - (64 << 20)
    assert torch.equal(native.mttkrp(X, dims, 1, 0, H, R), first)  # the next call allocates anew
    native.release_scratch()
