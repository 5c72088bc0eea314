"""Which kernels run the y and z operators of a single grid with the built-in
choice, on both sides of the lines drawn between tiles of whole pencils and
marches; and grids beside those lines, where tiles hold other numbers of
pencils than before, against the marches bit for bit."""
import re
import sys

import numpy as np
import pytest

from gpu_util import smooth_state
from launches import recorded

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def env():
    import torch
    from paper_1004_1680_amd import mhd
    mhd.load()
    return mhd, torch.cuda.Stream()


def say(*a):
    print(*a, flush=True)
    sys.stdout.flush()


# grid, tier, axis, operators (F, M, P pair, Z middle) that run in tiles
ROUTES = [((128, 128, 128), "f32", 1, "FP"), ((128, 128, 128), "f32", 2, "FPZ"), ((160, 128, 128), "f32", 2, "FPZ"),
          ((256, 128, 128), "f32", 2, "PZ"), ((128, 72, 256), "f32", 1, ""), ((80, 72, 64), "f32", 1, "FP"), ((124, 84, 64), "f32", 1, "FP"), ((148, 84, 76), "f32", 1, "P"),
          ((128, 72, 128), "f32", 1, "P"), ((160, 80, 208), "f32", 1, "P"), ((128, 96, 96), "f32", 1, "FP"), ((128, 96, 128), "f32", 1, "FP"), ((128, 96, 148), "f32", 1, "P"),
          ((128, 112, 128), "f32", 2, "FPZ"), ((192, 112, 128), "f32", 1, "P"), ((128, 64, 128), "f32", 1, "FMP"),
          ((256, 64, 256), "f32", 1, "FP"), ((384, 64, 256), "f32", 1, "FP"), ((256, 384, 64), "f32", 2, "Z"),
          ((384, 48, 256), "f32", 1, "FP"), ((384, 48, 260), "f32", 1, ""), ((384, 260, 48), "f32", 2, "Z"),
          ((512, 36, 256), "f32", 1, "F"), ((512, 36, 260), "f32", 1, ""),
          ((512, 32, 512), "f32", 1, "FP"), ((256, 16, 128), "f32", 1, "FMP"), ((256, 132, 64), "f32", 1, ""),
          ((128, 128, 128), "f64", 1, "P"), ((160, 128, 128), "f64", 1, ""), ((128, 64, 256), "f64", 1, "FMP"),
          ((256, 48, 256), "f64", 1, "P"), ((256, 256, 48), "f64", 2, ""), ((128, 72, 256), "f64", 1, ""), ((256, 64, 256), "f64", 2, ""),
          ((256, 256, 64), "f64", 2, "FP"),
          ((64, 132, 64), "f64", 1, "")]


@pytest.mark.parametrize("n,prec,d,tiled", ROUTES)
def test_kernels_of_the_operators(env, n, prec, d, tiled):
    M, side = env
    S = M.Solver(n, prec=prec, stream=side)
    S.set_relaxation_speed(1.0)
    S.set_reverse(1)
    if prec == "f32":
        S.set_launch(M.MHD_TUNE_MIDDLE, 1)
    calls = [("F", lambda: S.fluid(d, 0.1)), ("M", lambda: S.magnetic(d, 0.1)), ("P", lambda: S.sweep(3 + d, 0.1))]
    if d == 2 and prec == "f32":
        calls.append(("Z", lambda: S.sweep(7, 0.1)))
    got = ""
    for name, f in calls:
        runs = [k for k in recorded(side, f) if re.search("sweep_tile|march", k)]
        assert len(runs) == 1, runs
        got += name if "sweep_tile" in runs[0] else ""
    say(f"{n} {prec} axis {d}: tiles {got}")
    assert got == tiled
    S.close()


@pytest.mark.parametrize("prec", ["f32", "f64"])
@pytest.mark.parametrize("n", [(260, 64, 288), (260, 60, 308), (100, 20, 528), (116, 240, 40), (148, 148, 52)])
def test_other_tiles_are_the_marches(env, n, prec):
    # (more pencils to a tile than threads make whole waves, 32 to a tile, last
    # tiles partly empty)
    M, _ = env
    say(f"case: tiles n={n} {prec}")
    outs = []
    for march in (False, True):
        S = M.Solver(n, prec=prec)
        if march:
            for ax in (1, 2):
                S.set_chunk(ax, n[ax])
                S.set_pair_chunk(ax, n[ax])
            S.set_launch(M.MHD_TUNE_MIDDLE_CHUNK, n[2])
        S.set_state(smooth_state(n, seed=98))
        for _ in range(2):
            S.step_auto(0.5)
        outs.append(S.get_state())
        S.close()
    assert np.array_equal(*outs)


@pytest.mark.parametrize("n,d,chunk,pair", [((128, 128, 128), 1, 16, 32), ((128, 100, 128), 2, 16, 32),
                                            ((160, 68, 144), 1, 17, 34), ((160, 160, 160), 2, 32, 32), ((160, 88, 148), 1, 22, 44),
                                            ((64, 64, 1024), 2, 32, 64)])
def test_march_chunks_of_equal_estimate(env, n, d, chunk, pair):
    M, _ = env
    S = M.Solver(n)
    say(f"case: chunks n={n} axis {d}: {S.chunk(d)} {S.pair_chunk(d)}")
    assert (S.chunk(d), S.pair_chunk(d)) == (chunk, pair)
    S.close()
