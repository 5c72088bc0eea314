"""Which kernels run the y and z sweeps of an ensemble: tiles of whole pencils
where every box has them short and the boxes are few enough cells in all (or
the pencils very short), marches otherwise; one launch per operator either
way, and the boxes evolve as single grids."""
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


CASES = [  # boxes, tier, the y and z sweeps run in tiles
    ([(16, 24, 36), (20, 64, 12)], "f32", True, True),
    ([(16, 24, 36), (20, 64, 12)], "f64", True, True),
    ([(16, 24, 36), (20, 64, 68)], "f32", True, False),         # one box with longer pencils
    ([(16, 72, 36), (20, 64, 12)], "f64", False, True),
    ([(64, 64, 64)] * 18, "f32", True, True),                   # 4.5 M cells in all, and one box more
    ([(64, 64, 64)] * 18 + [(16, 16, 16)], "f32", False, False),
    ([(64, 64, 64)] * 12, "f64", True, True),                   # 3 M
    ([(64, 64, 64)] * 12 + [(16, 16, 16)], "f64", False, False),
    ([(256, 32, 32)] * 20, "f32", True, True),                  # very short pencils: at any size
    ([(256, 32, 64)] * 10, "f32", True, False),
]


@pytest.mark.parametrize("dims,prec,ty,tz", CASES)
def test_kernels_of_an_ensemble_step(env, dims, prec, ty, tz):
    M, side = env
    say(f"case: kernels of {len(dims)} boxes {dims[-1]} {prec}")
    B = M.Batch(dims, prec=prec, stream=side)
    # (kernel, operator, axis), one launch per operator
    runs = [m.groups() for m in (re.search(r"batch_(tile|sweep)_kernelI[fd]Li(\d)ELi(\d)E", n)
                                 for n in recorded(side, lambda: B.step_auto(0.5))) if m]
    ops = sum((1, 1, 2, 3)[int(op)] for _, op, _ in runs)
    assert ops == 12 and len(runs) <= 12, runs
    for axis, tiled in (("1", ty), ("2", tz)):
        assert {k for k, _, d in runs if d == axis} == {"tile" if tiled else "sweep"}, runs
    B.close()


@pytest.mark.parametrize("prec", ["f32", "f64"])
@pytest.mark.parametrize("dims", [[(12, 48, 24), (20, 44, 36), (16, 20, 28)], [(16, 64, 68), (12, 36, 8)]])
def test_boxes_are_single_grids(env, dims, prec):
    # (pencils of which 256 threads hold no multiple of 8)
    M, _ = env
    say(f"case: boxes of {dims} {prec}")
    B = M.Batch(dims, prec=prec)
    for i, n in enumerate(dims):
        B.set_state(i, smooth_state(n, seed=97 + i))
    B.run(3, 0.5)
    for i, n in enumerate(dims):
        S = M.Solver(n, prec=prec)
        S.set_state(smooth_state(n, seed=97 + i))
        for _ in range(3):
            S.step_auto(0.5)
        assert np.array_equal(B.get_state(i), S.get_state()), i
        S.close()
    B.close()
