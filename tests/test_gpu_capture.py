"""Steps captured in a caller's HIP graph: every replay, with eager work
between the replays, is the eager step bit for bit, also on grids whose
steps run their middle in one launch (five writes of the faces a step)."""
import sys

import numpy as np
import pytest

from gpu_util import smooth_state

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def env():
    import torch
    from paper_1004_1680_amd import mhd
    mhd.load()
    return torch, mhd, torch.cuda.Stream()


def say(*a):
    print(*a, flush=True)
    sys.stdout.flush()


def capture(torch, side, f, times=1):
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side):
        for _ in range(times):
            f()
    return graph


def replay(torch, side, graph):
    with torch.cuda.stream(side):
        graph.replay()
    side.synchronize()


@pytest.mark.parametrize("n,prec,lim,times", [((32, 24, 28), "f32", 0, 1), ((148, 12, 64), "f32", 0, 1),
                                              ((24, 20, 16), "f32", 2, 1), ((32, 24, 28), "f64", 0, 1),
                                              ((128, 128, 128), "f32", 0, 2)])
@pytest.mark.parametrize("host_dt", [False, True])
def test_captured_steps(env, n, prec, lim, times, host_dt):
    torch, M, side = env
    say(f"case: captured steps n={n} {prec} limiter {lim} x{times} host dt {host_dt}")
    S, E = M.Solver(n, prec=prec, stream=side), M.Solver(n, prec=prec)
    for X in (S, E):
        X.set_limiter(lim)
        X.set_state(smooth_state(n, seed=81))
        dt = X.cfl_dt(0.3)
    step = (lambda X: X.step(dt)) if host_dt else (lambda X: X.step_auto(0.5))
    for X in (S, E):
        step(X)
    graph = capture(torch, side, lambda: step(S), times)
    for k in range(3):
        replay(torch, side, graph)
        for _ in range(times):
            step(E)
        assert np.array_equal(S.get_state(), E.get_state()), k
        assert S.time() == E.time()
        for X in (S, E):                          # the handle's own steps in between
            for _ in range(times):
                step(X)
    if times == 1 and not host_dt:                # and another state, after an odd number of them
        for X in (S, E):
            X.set_state(smooth_state(n, seed=80))
            step(X)
        replay(torch, side, graph)
        step(E)
        assert np.array_equal(S.get_state(), E.get_state())
    S.close()
    E.close()


@pytest.mark.parametrize("prec", ["f32", "f64"])
def test_operators_around_the_middle(env, prec):
    """The middle of a step in one launch and in two, in turn and repeated,
    between other operators: the same fields, read back at every point by the
    host and into a tensor."""
    torch, M, side = env
    n = (20, 12, 36)
    say(f"case: operators around the middle {prec}")
    runs = []
    for mode in (0, 2):
        S = M.Solver(n, prec=prec)
        S.set_launch(M.MHD_TUNE_MIDDLE, mode)
        S.set_state(smooth_state(n, seed=85))
        dt = 0.3 * S.cfl_dt(0.5)
        got = []
        for code in (7, 7, 7, 0, 7, 4, 3, 7, 6, 1, 7):
            S.sweep(code, dt)
            if len(got) == 2:
                S.magnetic(1, dt)
            got.append((S.get_state(), S.get_state_tensor(dtype=torch.float64).cpu().numpy()))
            assert np.array_equal(*got[-1])
        runs.append(got)
        S.close()
    for k, (a, b) in enumerate(zip(*runs)):
        assert np.array_equal(a[0], b[0]), k


@pytest.mark.parametrize("prec", ["f32", "f64"])
def test_captured_ensemble_step(env, prec):
    torch, M, side = env
    say(f"case: captured ensemble step {prec}")
    dims = [(16, 12, 24), (20, 64, 16)]
    C, E = M.Batch(dims, prec=prec, stream=side), M.Batch(dims, prec=prec)
    for X in (C, E):
        for i, n in enumerate(dims):
            X.set_state(i, smooth_state(n, seed=82 + i))
        X.step_auto(0.5)
    graph = capture(torch, side, lambda: C.step_auto(0.5))
    for k in range(4):
        if k == 2:                                # another state, after more steps of each kind
            for X in (C, E):
                X.run(2, 0.5)
                X.set_state(1, smooth_state(dims[1], seed=86))
                X.step_auto(0.5)
        replay(torch, side, graph)
        E.step_auto(0.5)
        for i in range(len(dims)):
            assert np.array_equal(C.get_state(i), E.get_state(i)), (k, i)
        C.step_auto(0.5)
        E.run(1, 0.5, graph=k > 0)
    C.close()
    E.close()


# (row lengths whose x kernels' workgroups are whole waves, and not)
@pytest.mark.parametrize("prec", ["f32", "f64"])
@pytest.mark.parametrize("n", [(32, 16, 8), (20, 16, 8)])
def test_cfl_around_captures(env, n, prec):
    """A time step is that of the state it meets: on replays that follow a new
    state, after a capture that has not run, and after replays that the host
    does not see."""
    torch, M, side = env
    say(f"case: CFL around captures n={n} {prec}")
    s0, s1 = smooth_state(n, seed=83), smooth_state(n, seed=84)
    s1[4] *= 2.0                                  # another largest signal speed

    def fresh(state):
        F = M.Solver(n, prec=prec)
        F.set_state(state)
        return F

    S = M.Solver(n, prec=prec, stream=side)
    S.set_state(s0)
    S.step_auto(0.5)
    one = capture(torch, side, lambda: S.step_auto(0.5))
    F = fresh(S.get_state())                      # recorded, not run
    assert S.cfl_dt(0.5) == F.cfl_dt(0.5)
    F.close()
    S.set_state(s1)
    F = fresh(s1)
    for k in range(2):
        replay(torch, side, one)
        F.step_auto(0.5)
        assert np.array_equal(S.get_state(), F.get_state()) and S.time() == F.time(), k
    F.close()

    S.set_state(s0)
    dt = S.cfl_dt(0.4)
    sweeps = capture(torch, side, lambda: (S.sweep(0, dt), S.sweep(3, dt)))
    S.step(dt)                                    # leaves the maximum of its state
    replay(torch, side, sweeps)
    F = fresh(S.get_state())
    assert S.cfl_dt(0.4) == F.cfl_dt(0.4)
    for k in range(2):
        S.step_auto(0.5)
        F.step_auto(0.5)
    assert np.array_equal(S.get_state(), F.get_state())
    F.close()

    S.set_state(s0)                               # two steps in one graph
    two = capture(torch, side, lambda: (S.step_auto(0.5), S.step_auto(0.5)))
    for s in (s1, s0):
        S.set_state(s)
        F = fresh(s)
        replay(torch, side, two)
        F.step_auto(0.5)
        F.step_auto(0.5)
        assert np.array_equal(S.get_state(), F.get_state())
        F.close()
    S.close()
