"""The y and z tile kernels (tiles of whole pencils, the built-in choice for
short pencils) against the march kernels (a chunk length set by the caller):
the same device functions on the same values, so every operator, reverse
pair, middle and step comes out the same bit for bit.  Grids: pencils of one
wave and less, lengths that are no multiple of a wave, last tiles that are
partly empty, the longest pencils either rule takes and the first ones past
it, and a slab whose tiles hold 256 threads."""
import sys

import numpy as np
import pytest

from gpu_util import smooth_state

pytestmark = pytest.mark.gpu

GRIDS = [(8, 8, 8), (20, 12, 36), (12, 60, 64), (36, 64, 68), (20, 128, 124), (8, 132, 128), (256, 64, 64)]


@pytest.fixture(scope="module")
def M():
    from paper_1004_1680_amd import mhd
    mhd.load()
    return mhd


def say(*a):
    print(*a, flush=True)
    sys.stdout.flush()


def solver(M, n, prec, lim, march):
    S = M.Solver(n, prec=prec)
    S.set_limiter(lim)
    if march:
        for ax in (1, 2):
            S.set_chunk(ax, n[ax])
            S.set_pair_chunk(ax, n[ax])
        S.set_launch(M.MHD_TUNE_MIDDLE_CHUNK, n[2])
    return S


@pytest.mark.parametrize("prec", ["f32", "f64"])
@pytest.mark.parametrize("n", GRIDS)
def test_tiles_are_the_marches(M, n, prec):
    s = smooth_state(n, seed=61)
    limiters = (M.MHD_LIMITER_VANLEER,) if n[0] > 100 else (M.MHD_LIMITER_VANLEER, M.MHD_LIMITER_MINMOD,
                                                            M.MHD_LIMITER_MC, M.MHD_LIMITER_SUPERBEE)
    for lim in limiters:
        for what in ("F1", "F2", "M1", "M2", "P1", "P2", "mid", "step"):
            say(f"case: tiles n={n} {prec} limiter {lim} {what}")
            outs = []
            for march in (False, True):
                S = solver(M, n, prec, lim, march)
                S.set_state(s)
                dt = S.cfl_dt(0.5)
                if what == "mid":
                    S.sweep(7, dt)
                elif what == "step":
                    S.step(dt)
                else:
                    d = int(what[1])
                    (S.fluid if what[0] == "F" else S.magnetic if what[0] == "M" else
                     lambda d, dt: S.sweep(3 + d, dt))(d, dt)
                outs.append(S.get_state())
                S.close()
            assert np.array_equal(*outs), (what, lim)


@pytest.mark.parametrize("prec", ["f32", "f64"])
def test_tiles_keep_a_recorded_state(M, prec):
    n = (20, 24, 28)
    say(f"case: tiles under a record {prec}")
    s = smooth_state(n, seed=62)
    s[4, 3, 5, 7] = -1.0
    S = solver(M, n, prec, 0, False)
    S.set_state(s)
    before = S.get_state()
    S.step_auto(0.7)
    with pytest.raises(M.NonPhysicalState):
        S.status()
    assert np.array_equal(S.get_state(), before)
    S.close()


@pytest.mark.parametrize("prec,lim", [("f32", 0), ("f32", 2), ("f64", 0)])
@pytest.mark.parametrize("dims", [[(16, 8, 12), (20, 64, 36), (8, 60, 64)],
                                  [(16, 12, 8), (20, 64, 68), (24, 72, 64), (36, 132, 8)]])
def test_ensembles_with_tiles(M, dims, prec, lim):
    # boxes that run y and z in tiles, in marches, and one axis in each:
    # every box is the single grid bit for bit, eagerly and from the graph
    # (odd step counts: with the middle in one launch it holds two steps)
    say(f"case: ensemble with tiles {dims} {prec} limiter {lim}")
    states = [smooth_state(n, seed=63 + i) for i, n in enumerate(dims)]
    for graph in (False, True):
        B = M.Batch(dims, prec=prec)
        B.set_limiter(lim)
        for i, s in enumerate(states):
            B.set_state(i, s)
        for k in (1, 3, 2):
            B.run(k, 0.5, graph=graph)
        steps, _ = B.status()
        assert (steps == 6).all()
        times = B.times()
        for i, (n, s) in enumerate(zip(dims, states)):
            S = M.Solver(n, prec=prec)
            S.set_limiter(lim)
            S.set_state(s)
            for _ in range(6):
                S.step_auto(0.5)
            assert np.array_equal(B.get_state(i), S.get_state()) and times[i] == S.time(), (i, graph)
            S.close()
        B.close()
