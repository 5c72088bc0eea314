"""An ensemble in which one box has fields over 4 GiB and another has pencils
short enough for tiles: it steps, with 64-bit addressing throughout, and the
small box is the single grid bit for bit.  The large box is left as created
(rho = 0): its record keeps it unchanged, which needs no host copy of it."""
import sys

import numpy as np
import pytest

from gpu_util import smooth_state

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def M():
    from paper_1004_1680_amd import mhd
    mhd.load()
    return mhd


def say(*a):
    print(*a, flush=True)
    sys.stdout.flush()


@pytest.mark.parametrize("prec,big", [("f32", (1024, 1024, 1028)), ("f64", (1024, 1024, 516))])
def test_large_and_small_box(M, prec, big):
    small = (16, 12, 20)
    say(f"case: large and small box {big} {prec}")
    B = M.Batch([big, small], prec=prec)
    s = smooth_state(small, seed=91)
    B.set_state(1, s)
    S = M.Solver(small, prec=prec)
    S.set_state(s)
    for _ in range(2):
        B.step_auto(0.5)
        S.step_auto(0.5)
    steps, record = B.status(raise_on_nonphysical=False)
    assert list(steps) == [0, 2] and list(record) == [1, 0]
    assert np.array_equal(B.get_state(1), S.get_state()) and B.times()[1] == S.time()
    S.close()
    B.close()
