"""The tile tests name the kernel that each of their shapes runs: the names are checked here against the library's own
selection (gm_plan.h, compiled for the host), and together they name every tile there is."""
import heapq
import os
import random
import shutil
import subprocess

import pytest

import test_gpu_backward_tiles as backward
import test_gpu_packed_tokens as tokens
import test_gpu_split_tiles as split
import test_gpu_square_sparse as sparse
import test_gpu_tiles as forward

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    cxx = shutil.which("g++") or shutil.which("c++")
    if cxx is None:
        pytest.skip("no host C++ compiler")
    exe = str(tmp_path_factory.mktemp("plan") / "tile_plan")
    subprocess.run([cxx, "-std=c++17", "-O1", "-Wall", "-Werror", "-o", exe, os.path.join(HERE, "tile_plan.cpp")], check=True)

    def ask(rows):
        text = "".join(" ".join(str(x) for x in r) + "\n" for r in rows)
        out = subprocess.run([exe], input=text, capture_output=True, text=True, check=True).stdout.splitlines()
        assert len(out) == len(rows)
        return out

    return ask


def _check(shapes, want, got):
    wrong = [f"{s}: named {w}, runs {g}" for s, w, g in zip(shapes, want, got) if w != g]
    assert not wrong, "\n".join(wrong)


def test_forward_tiles(plan):
    s = forward.FWD_TILES
    _check(s, [x[5] for x in s], plan([("fwd", *x[:5], 1) for x in s]))
    _check(s, [x[6] for x in s], plan([("packed", *x[:5], 1) for x in s]))
    assert {x[5] for x in s} == {"256x256", "256x128", "128x128"}
    assert {x[6] for x in s} >= {"256x256", "256x128", "128x128", "passes16"}
    # each width of the packed tiles and passes, with fractional selectors too (test_gpu_tiles.py runs every shape with both)
    tok = [x for x in plan([("packed", T, i, o, g, 1, 1) for T, i, o, g in tokens.PASSES])]
    assert set(tok) == {"passes16", "passes32"}


def test_backward_tiles(plan):
    s = backward.DX_TILES
    _check(s, [x[5] for x in s], plan([("dx", *x[:5], 0) for x in s]))
    lists = {"256x256", "256x128", "128x256", "128x128", "64x128", "64x256"}
    dense = {"dense 256x256", "dense 256x128", "dense 128x128"}
    assert {x[5] for x in s} == lists | dense
    assert all({x[3] for x in s if x[5] == t} == {16, 32} for t in dense)
    s = backward.DGATE_TILES
    _check(s, [x[5] for x in s], plan([("dgate", *x[:5], 0) for x in s]))
    assert {x[5] for x in s} == {"256x256", "256x128", "256x64"}
    s = backward.LM_TILES
    _check(s, [x[3] for x in s], plan([("lm", N, d, V, 0, 0, 0) for N, d, V, _ in s]))
    assert {x[3] for x in s} == {"256x256", "256x128", "128x128"}


def test_sparse_dx_tiles(plan):
    s = sparse.SHAPES
    _check(s, [x[4] for x in s], plan([("dx", T, i, o, g, g, 0) for T, i, o, g, _ in s]))
    assert {x[4] for x in s} == {"dense 256x256", "dense 256x128", "dense 128x128"}


def test_split_tiles(plan):
    s = split.SHAPES
    _check(s, [x[5] for x in s], plan([("fwd", *x[:5], x[6]) for x in s]))
    assert any(x[5] == "128x128 split" for x in s)


def test_end_of_a_launch_of_two_kinds_of_blocks(plan):
    # the closed form against 256 CUs that each take the next block when free
    r = random.Random(5)
    rows = [(r.randint(1, 1500), r.randint(1000, 200000), r.randint(1, 1500), r.randint(1000, 200000)) for _ in range(300)]
    rows += [(256, 5000, 256, 7000), (512, 5000, 1, 7000), (1, 9000, 1, 1000)]
    got = plan([("kinds", *x, 0, 0) for x in rows])
    for (n1, t1, n2, t2), g in zip(rows, got):
        free = [0] * 256
        end = 0
        for k in range(n1 + n2):
            t = heapq.heappop(free) + (t1 if k < n1 else t2)
            heapq.heappush(free, t)
            end = max(end, t)
        assert int(g) == end


def test_square_backward_takes_both_orders(plan):
    # the shapes of the parity tests run dX first and dgate first
    s = [x for x in backward.DX_TILES if x[5].startswith("dense")]
    assert set(plan([("first", *x[:5], 0) for x in s])) == {"dX", "dgate"}
