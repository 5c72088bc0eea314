"""The march kernels on grids whose built-in choice is tiles: chunks set by the
caller (one and several to a pencil), 32-bit and 64-bit offsets.  Steps under a
record keep every field, and steps are the oracle's within the bounds of the
built-in choice (FP64 1e-12, FP32 3e-5 of a field family after three steps)."""
import sys

import numpy as np
import pytest

import oracle
from gpu_util import max_family_err
from paper_1004_1680_amd import inputs as I

pytestmark = pytest.mark.gpu

ONE, TWO = 1, 2


@pytest.fixture(scope="module")
def M():
    from paper_1004_1680_amd import mhd
    mhd.load()
    return mhd


def say(*a):
    print(*a, flush=True)
    sys.stdout.flush()


def solver(M, n, prec, reverse, middle, cuts, wide):
    """marches with `cuts` chunks to a pencil along y and z"""
    S = M.Solver(n, prec=prec)
    for ax in (1, 2):
        S.set_chunk(ax, n[ax] // cuts)
        S.set_pair_chunk(ax, n[ax] // cuts)
    S.set_launch(M.MHD_TUNE_MIDDLE_CHUNK, n[2] // cuts)
    S.set_reverse(reverse)
    S.set_launch(M.MHD_TUNE_MIDDLE, middle)
    S.set_launch(M.MHD_TUNE_WIDE_OFFSETS, wide)
    return S


WAYS = [("f32", TWO, TWO), ("f32", ONE, TWO), ("f32", ONE, ONE), ("f64", TWO, TWO), ("f64", ONE, TWO)]


@pytest.mark.parametrize("wide", [0, 1])
@pytest.mark.parametrize("cuts", [1, 2])
@pytest.mark.parametrize("prec,reverse,middle", WAYS)
def test_marches_keep_a_recorded_state(M, prec, reverse, middle, cuts, wide):
    n = (24, 16, 32)
    say(f"case: marches under a record {prec} reverse {reverse} middle {middle} x{cuts} wide {wide}")
    s = I.random_smooth(n, seed=6)
    s[4, 3, 5, 7] = -1.0
    S = solver(M, n, prec, reverse, middle, cuts, wide)
    S.set_state(s)
    before = S.get_state()
    for _ in range(2):
        S.step_auto(0.7)
        assert np.array_equal(S.get_state(), before)
    with pytest.raises(M.NonPhysicalState):
        S.status()
    S.close()


@pytest.mark.parametrize("cuts", [1, 2])
@pytest.mark.parametrize("prec,reverse,middle", WAYS)
def test_march_steps_match_the_oracle(M, prec, reverse, middle, cuts):
    n = (40, 24, 16)
    say(f"case: march steps vs oracle {prec} reverse {reverse} middle {middle} x{cuts}")
    s = I.random_smooth(n, seed=43).astype(np.float32).astype(np.float64)
    S = solver(M, n, prec, reverse, middle, cuts, 0)
    S.set_state(s)
    for _ in range(3):
        S.step_auto(0.7)
    assert S.status() == 3
    g, t = S.get_state(), S.time()
    S.close()
    o, to, _ = oracle.run(s, 3)
    err = max_family_err(g, o)
    say("err", err)
    assert err <= (1e-12 if prec == "f64" else 3e-5)
    assert t == pytest.approx(to, rel=1e-13 if prec == "f64" else 1e-6)
