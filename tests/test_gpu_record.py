"""A record of the device CFL (non-physical state) that still stands when the
state has become physical again: the host's CFL call reports the state, and
once mhd_status has cleared the record device-dt steps run again."""
import sys

import numpy as np
import pytest

from paper_1004_1680_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def M():
    from paper_1004_1680_amd import mhd
    mhd.load()
    return mhd


def say(*a):
    print(*a, flush=True)
    sys.stdout.flush()


# (row lengths whose x kernels' workgroups are whole waves, and not)
@pytest.mark.parametrize("prec", ["f32", "f64"])
@pytest.mark.parametrize("n", [(16, 8, 8), (20, 12, 8)])
def test_record_of_a_state_that_is_gone(M, n, prec):
    say(f"case: a carried record n={n} {prec}")
    s = I.uniform(n)
    s[4, 3, 4, 5] *= 0.05                 # p < 0 in one cell; diffusion lifts it
    S = M.Solver(n, prec=prec)
    S.set_state(s)
    S.step_auto(0.5)                      # records, leaves the state
    S.set_relaxation_speed(4.0)
    for _ in range(3):
        S.step(0.1 / n[0])
    state = S.get_state()
    F = M.Solver(n, prec=prec)
    F.set_state(state)
    dt = F.cfl_dt(0.5)                    # (physical now)
    S.step_auto(0.5)                      # skipped: the record stands
    assert np.array_equal(S.get_state(), state)
    assert S.cfl_dt(0.5) == dt
    assert S.relaxation_speed() == F.relaxation_speed()
    S.step_auto(0.5)                      # still skipped
    with pytest.raises(M.NonPhysicalState):
        S.status()
    for X in (S, F):
        X.step_auto(0.5)
        X.step_auto(0.5)
    assert S.status() == 2 and F.status() == 2
    assert np.array_equal(S.get_state(), F.get_state())
    S.close()
    F.close()
