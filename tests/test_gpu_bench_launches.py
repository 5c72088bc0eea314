"""The launches of a step that bench.py names for its grids (pencils past the
tile kernels) are the ones a step records, in order, in both tiers."""
import os
import re
import sys

import pytest

from launches import recorded

pytestmark = pytest.mark.gpu

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def printed(mangled):
    """a kernel's name as the profiler prints it"""
    m = re.match(r"_ZN3mhd(\d+)", mangled)
    name = mangled[m.end():m.end() + int(m.group(1))]
    t, args = re.match(r"I([fd])((?:L[ib]\d+E)+)E", mangled[m.end() + len(name):]).groups()
    args = [("true" if v == "1" else "false") if k == "b" else v for k, v in re.findall(r"L([ib])(\d+)E", args)]
    return f"{name}<{', '.join([{'f': 'float', 'd': 'double'}[t]] + args)}>"


@pytest.mark.parametrize("prec,lim", [("f32", 0), ("f32", 2), ("f64", 0), ("f64", 3)])
def test_step_launches(prec, lim):
    import torch
    from paper_1004_1680_amd import mhd
    sys.path.insert(0, ROOT)
    import bench
    n, side = 160, torch.cuda.Stream()
    print("case: launches of a step", prec, lim, flush=True)
    S = mhd.Solver((n, n, n), prec=prec, stream=side)
    S.set_limiter(lim)
    S.set_relaxation_speed(1.0)
    names = [printed(k) for k in recorded(side, lambda: S.step(0.1)) if "begin_step" not in k]
    want = bench.step_launches(S, n, 8 if prec == "f64" else 4, S.reverse() == 1, "true", lim,
                               S.launch(mhd.MHD_TUNE_MIDDLE) == 1)
    assert names == [k for k, _ in want]
    S.close()
