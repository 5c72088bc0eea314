"""How many launches a step records under the launch settings: the built-in
choice on a small grid (pairs and, in FP32 with van Leer's limiter, the middle
in one launch each, by the tile kernels) and what a setting takes apart.  The
results do not depend on them, so the launches are counted in a captured step."""
import ctypes
import sys

import numpy as np
import pytest

from gpu_util import smooth_state

pytestmark = pytest.mark.gpu

N = (32, 24, 48)


@pytest.fixture(scope="module")
def env():
    import torch
    from paper_1004_1680_amd import mhd
    mhd.load()
    hip = ctypes.CDLL("libamdhip64.so")
    return torch, mhd, torch.cuda.Stream(), hip


def say(*a):
    print(*a, flush=True)
    sys.stdout.flush()


def recorded(side, hip, f):
    stream, graph, n = ctypes.c_void_p(side.cuda_stream), ctypes.c_void_p(), ctypes.c_size_t(0)
    assert hip.hipStreamBeginCapture(stream, 1) == 0            # thread-local mode
    f()
    assert hip.hipStreamEndCapture(stream, ctypes.byref(graph)) == 0
    assert hip.hipGraphGetNodes(graph, None, ctypes.byref(n)) == 0
    assert hip.hipGraphDestroy(graph) == 0
    return n.value


def launches(env, prec, settings):
    torch, M, side, hip = env
    S = M.Solver(N, prec=prec, stream=side)
    for key, value in settings:
        S.set_launch(key, value)
    S.set_state(smooth_state(N, seed=95))
    dt = S.cfl_dt(0.5)
    S.step(dt)
    state = S.get_state()
    n = recorded(side, hip, lambda: S.step(dt))
    S.close()
    return n - 1, state                                         # less the launch that opens a step


@pytest.mark.parametrize("prec", ["f32", "f64"])
def test_launches_of_a_step(env, prec):
    M = env[1]
    f32 = prec == "f32"
    one = 8 if f32 else 9
    cases = [("built in", [], one),
             ("z pair's chunk", [(M.MHD_TUNE_PAIR_CHUNK_Z, 16)], 9 if f32 else 10),
             ("z chunk", [(M.MHD_TUNE_CHUNK_Z, 16)], 9),
             ("middle's chunk", [(M.MHD_TUNE_MIDDLE_CHUNK, 16)], 9),
             ("z pair's chunk set and taken back", [(M.MHD_TUNE_PAIR_CHUNK_Z, 16), (M.MHD_TUNE_PAIR_CHUNK_Z, 0)], one),
             ("y pair's chunk", [(M.MHD_TUNE_PAIR_CHUNK_Y, 8)], one if f32 else 10),
             ("middle in two", [(M.MHD_TUNE_MIDDLE, 2)], 9),
             ("pairs in two", [(M.MHD_TUNE_REVERSE, 2)], 12),
             ("wide offsets", [(M.MHD_TUNE_WIDE_OFFSETS, 1)], 9 if f32 else 12)]
    states = []
    for name, settings, want in cases:
        n, state = launches(env, prec, settings)
        say(f"{prec} {name}: {n} launches")
        assert n == want, name
        states.append(state)
    assert all(np.array_equal(states[0], s) for s in states[1:])


def test_launches_of_an_ensemble_step(env):
    # (a step that a caller captures keeps the middle in two launches unless
    # one is asked for)
    torch, M, side, hip = env
    dims = [(16, 12, 24), (20, 16, 32)]
    states = []
    for name, settings, want in (("built in", [], 9), ("middle in one", [(M.MHD_BATCH_MIDDLE, 1)], 8),
                                 ("chunk target", [(M.MHD_BATCH_CHUNK, 8)], 9),
                                 ("pairs' target", [(M.MHD_BATCH_PAIR_CHUNK, 8)], 9),
                                 ("pairs in two", [(M.MHD_BATCH_REVERSE, 2)], 12)):
        B = M.Batch(dims, stream=side)
        for key, value in settings:
            B.set_launch(key, value)
        for i, n in enumerate(dims):
            B.set_state(i, smooth_state(n, seed=96 + i))
        B.step_auto(0.5)
        states.append([B.get_state(i) for i in range(len(dims))])
        got = recorded(side, hip, lambda: B.step_auto(0.5)) - 1
        say(f"ensemble {name}: {got} launches")
        assert got == want, name
        B.close()
    for s in states[1:]:
        assert all(np.array_equal(a, b) for a, b in zip(states[0], s))
