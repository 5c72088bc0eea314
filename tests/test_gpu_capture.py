"""Steps captured in a caller's HIP graph: every replay, with eager work
between the replays, is the eager step bit for bit, also on grids whose
eager steps run their middle in one launch (which moves the faces to the
other buffer)."""
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
    S.close()
    E.close()


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
    for k in range(3):
        replay(torch, side, graph)
        E.step_auto(0.5)
        for i in range(len(dims)):
            assert np.array_equal(C.get_state(i), E.get_state(i)), (k, i)
    C.close()
    E.close()
