"""Every tensor load of the partial-MTTKRP kernels in the form that the launcher
picks (host walk, no GPU): inside the tensor, and the elements that count arrive as
themselves, over ragged, odd, tall and long shapes of every storage type."""

import math
import os
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB_DIR = os.path.join(ROOT, "paper_1806_07985_amd", "lib")

SHAPES = [(60, 50, 40), (33, 47, 29), (64, 40, 24, 10), (20, 18, 22), (128, 64, 33, 9), (300, 20, 10), (9, 8, 16), (7, 11, 13),
          (1, 1, 1), (1, 5, 1), (2, 3), (3, 2), (5, 1), (1, 7), (3, 1, 2), (12, 10, 9, 8, 7), (37, 29, 23), (63, 31, 5), (65, 17, 9),
          (83, 71, 57), (82, 71, 57), (83, 3, 131), (83, 4, 131), (301, 700), (15, 3, 300), (31, 5, 401), (1001, 3), (5, 3, 257),
          (1152, 70000), (200000, 40), (40, 200000), (199999, 37), (37, 199999), (333, 333, 333), (384, 1400, 16), (129, 33001),
          (64, 5, 8200), (128, 3, 4500)]
# 16-bit right node, J == 1, K split over i1 blocks with several tiles per group
J1_TILES = [(6501, 33000), (6500, 33001), (3201, 70001)]
# lane offsets past 31 bits: masked loads
LONG = [(9000001, 3), (3001, 3001, 4), (4201, 4201, 3), (6001, 6001, 3, 2), (36000001, 2), (17000001, 2)]


@pytest.fixture(scope="module")
def walk(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("walk") / "pm_load_walker")
    cmd = [os.environ.get("HIPCC", "/opt/rocm/bin/hipcc"), "-O2", "-std=c++17", "-I", os.path.join(ROOT, "include"), "-I",
           os.path.join(ROOT, "paper_1806_07985_amd", "csrc"), os.path.join(ROOT, "tests", "pm_load_walker.cpp"), "-o",
           exe, "-L", LIB_DIR, "-lnncp", f"-Wl,-rpath,{LIB_DIR}"]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]

    def run(shapes, ranks, lines=None):
        lines = lines or [f"{dt} {math.prod(d[:s])} {math.prod(d[s:])} {d[s]} {d[0]} {R} {off}" for d in shapes
                          for s in range(1, len(d)) for R in ranks for dt in range(3) for off in ((0, 1) if dt else (0,))]
        r = subprocess.run([exe], input="\n".join(lines) + "\n", capture_output=True, text=True, timeout=900)
        assert r.returncode == 0 and f"{len(lines)} cases" in r.stdout, r.stdout[-3000:]
        return {ln[6:] for ln in r.stdout.splitlines() if ln.startswith("cover")}
    return run


def test_loads_of_ragged_shapes(walk):
    rng = np.random.default_rng(1)
    shapes = SHAPES + [tuple(int(x) for x in rng.integers(2, 90, size=3)) for _ in range(12)]
    seen = walk(shapes, (5, 24, 50))
    for form in ("f32 side 0 form 1", "f32 side 0 form 2", "f32 side 0 form 3", "f32 side 1 form 2", "16 side 0 form 1",
                 "16 side 0 form 2", "16 side 1 form 1", "16 side 1 form 2", "16 side 1 form 3"):
        assert any(s.startswith(form) for s in seen), form


def test_loads_of_j1_nodes_that_split_k_over_several_tiles(walk):
    seen = walk(J1_TILES, (10, 20))
    for form in (2, 3):
        assert any(s.startswith(f"16 side 1 form {form} mt 1 split 1 j1 1") for s in seen), sorted(seen)


def test_loads_of_long_columns(walk):
    seen = walk(LONG, (5, 20, 40))
    for what in ("f32 side 0", "f32 side 1", "16 side 0", "16 side 1"):
        assert any(s.startswith(what + " form 0") for s in seen), what


@pytest.mark.parametrize("d,R,form", [((83, 71, 2565), 24, 3), ((301, 1, 40000), 10, 3), ((31, 5, 40001), 48, 3),  # the address unit is busy
                                      ((3, 2, 100000), 5, 2), ((1, 6, 7000), 20, 2),            # short columns
                                      ((363, 400, 5), 5, 2), ((363, 400, 20), 20, 2), ((363, 400, 28), 50, 2),  # few columns
                                      ((363, 400, 17), 5, 3), ((363, 400, 21), 20, 3), ((363, 400, 29), 50, 3),
                                      ((17, 50, 70), 20, 2), ((17, 50, 96), 20, 3), ((31, 10, 191), 50, 2),      # one group
                                      ((15, 20, 4001), 40, 2)])                                   # padding
def test_right_nodes_load_from_dword_starts_where_that_is_faster(walk, d, R, form):
    """16-bit right node (split 2) of odd first extent; a tensor off a dword never does."""
    for off, f in ((0, form), (1, 2)):
        seen = walk(None, None, [f"2 {d[0] * d[1]} {d[2]} {d[2]} {d[0]} {R} {off}"])
        assert any(s.startswith(f"16 side 1 form {f}") for s in seen), (off, sorted(seen))


@pytest.mark.parametrize("d,dt,form", [((30013, 1200, 83), 0, 2), ((30013, 1200, 84), 0, 3), ((255, 3000, 30000), 0, 2), ((257, 3000, 30000), 0, 3),
                                       ((30012, 1200, 166), 1, 2), ((30012, 1200, 167), 2, 4), ((511, 3000, 30000), 1, 2), ((513, 3000, 30000), 1, 4)])
def test_left_nodes_of_large_tensors_stream(walk, d, dt, form):
    """From 12 GB with columns of 1 KB and more (split 1)."""
    seen = walk(None, None, [f"{dt} {d[0]} {d[1] * d[2]} {d[1]} {d[0]} 10 0"])
    assert any(s.startswith(f"{'16' if dt else 'f32'} side 0 form {form} ") for s in seen), sorted(seen)
