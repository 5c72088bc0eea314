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
