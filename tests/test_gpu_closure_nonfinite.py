"""Infinities and NaN in the operands of single closure layers: they reach the
outputs whose 3x3x3 stencil holds them and no others, with the values that a
float64 sum of the same products has (sign of an infinity, NaN), and the finite
outputs stay those of the sum (bound 1e-5 of their scale, FP32 against FP64
accumulation).  Planted in odd and even rows and at the faces of the grid,
apart from one another; grids of one tile and of several per workgroup."""
import sys

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

GRIDS = [(32, 32, 64), (96, 64, 96)]


@pytest.fixture(scope="module")
def env():
    import torch
    from paper_1004_1680_amd import mhd
    mhd.load()
    return torch, mhd


def say(*a):
    print(*a, flush=True)
    sys.stdout.flush()


def operand(torch, n, c, seed, planted=True):
    """random BF16 values [nz][ny][nx][c] with some cells not finite"""
    g = torch.Generator(device="cuda").manual_seed(seed)
    x = torch.randn((n[2], n[1], n[0], c), generator=g, device="cuda").to(torch.bfloat16)
    if planted:
        inf, nan = float("inf"), float("nan")
        for q, (i, j, k) in enumerate([(3, 4, 5), (10, 9, 5), (20, 14, 8), (27, 19, 11), (5, 24, 15), (0, 0, 20),
                                       (n[0] - 1, n[1] - 1, 30), (15, 31, 40), (16, 7, 45), (8, 16, n[2] - 1)]):
            x[k, j, i, (5 * q + 1) % c] = (inf, -inf, nan)[q % 3]
    return x


def weights(torch, cin, cout, seed):
    w = np.random.default_rng(seed).normal(0.0, 0.1, (27, cin, cout)).astype(np.float32)
    wd = torch.from_numpy(w).to(torch.bfloat16)
    assert bool((wd != 0).all())                  # zero times infinity is no part of a layer here
    return w, wd.double().cuda()


def layer(torch, x, wd, order):
    """sum over offsets and input channels of the shifted cells times weights,
    in float64, product by product"""
    out = 0.0
    for o in range(27):
        p = order(o)
        sh = torch.roll(x, (1 - p // 9, 1 - (p // 3) % 3, 1 - p % 3), (0, 1, 2)).reshape(-1, x.shape[3])
        for c in range(sh.shape[1]):
            out = out + sh[:, c:c + 1] * wd[o][c]
    return out


def same(torch, got, ref, what):
    got = got.double()
    assert torch.equal(torch.isnan(got), torch.isnan(ref)), what
    assert torch.equal(torch.isposinf(got), torch.isposinf(ref)) and torch.equal(torch.isneginf(got), torch.isneginf(ref)), what
    ok = torch.isfinite(ref)
    err = float((got[ok] - ref[ok]).abs().max() / ref[ok].abs().max())
    say(f"{what}: {int((~ok).sum())} not finite, others {err:.2e}")
    assert 0 < int((~ok).sum()) < ok.numel() // 20 and err < 1e-5, what


@pytest.mark.parametrize("n", GRIDS)
@pytest.mark.parametrize("cin,cout", [(8, 32), (32, 32), (32, 8), (8, 8)])
def test_layers_keep_them_in_their_stencil(env, n, cin, cout):
    torch, mhd = env
    say(f"case: not finite n={n} {cin}->{cout}")
    N = n[0] * n[1] * n[2]
    w, wd = weights(torch, cin, cout, 6)
    x = operand(torch, n, cin, 7)
    y = torch.zeros((N, cout), device="cuda")
    mhd.conv3d_forward(n, x, w, None, y)
    same(torch, y, layer(torch, x.double(), wd, lambda o: o), "forward")
    dy = operand(torch, n, cout, 8)
    dx = torch.zeros((N, cin), device="cuda")
    mhd.conv3d_dgrad(n, dy, w, dx)
    same(torch, dx, layer(torch, dy.double(), wd.transpose(1, 2), lambda o: 26 - o), "dgrad")


@pytest.mark.parametrize("cin,cout", [(8, 32), (32, 32), (32, 8), (8, 8)])
def test_weight_gradients_keep_them_in_their_channels(env, cin, cout):
    # one input (output) channel that is not finite: its weights' gradients
    # are not, the others are those of the sum
    torch, mhd = env
    n = GRIDS[1]
    say(f"case: not finite wgrad {cin}->{cout}")
    N = n[0] * n[1] * n[2]
    x, dy = operand(torch, n, cin, 9, False), operand(torch, n, cout, 10, False)
    plain, bias = mhd.conv3d_wgrad(n, cin, cout, x.reshape(N, cin).T.contiguous(), dy.reshape(N, cout).T.contiguous())
    for which, ch in (("x", 3), ("x", cin - 1), ("dy", 2), ("dy", cout - 1)):
        xx, dd = x.clone(), dy.clone()
        (xx if which == "x" else dd)[17, 33, 31, ch] = float("nan")
        dw, db = mhd.conv3d_wgrad(n, cin, cout, xx.reshape(N, cin).T.contiguous(), dd.reshape(N, cout).T.contiguous())
        want = plain.copy()
        wantb = bias.copy()
        if which == "x":
            want[:, ch, :] = np.nan
        else:
            want[:, :, ch] = np.nan
            wantb[ch] = np.nan
        assert np.array_equal(dw, want, equal_nan=True) and np.array_equal(db, wantb, equal_nan=True), (which, ch)


@pytest.mark.parametrize("n", GRIDS)
def test_correction_keeps_them_in_its_stencil(env, n):
    """A cell of the state that is not finite, handed to the last layer at its
    place (the first two layers pass one field on; the NaN that they make of
    zero times infinity around it their ReLU drops): a layer and a curl on, the
    field's correction is not finite within 2 cells below and 1 above at most,
    and is another within one cell more (the fluid fields' corrections subtract
    a mean over the box)."""
    torch, mhd = env
    say(f"case: not finite state n={n}")
    w = [np.zeros((27, a, b), np.float32) for a, b in ((8, 32), (32, 32), (32, 8))]
    w[0][13, 2, 0] = w[1][13, 0, 0] = 1.0
    w[2][:] = np.random.default_rng(12).normal(0.0, 0.05, w[2].shape)
    g = torch.Generator(device="cuda").manual_seed(11)
    u = torch.randn((8, n[2], n[1], n[0]), generator=g, device="cuda") * 0.1 + 1.0
    cl = mhd.Closure(n)
    cl.set_params(np.concatenate([np.concatenate([x.ravel(), np.zeros(x.shape[2], np.float32)]) for x in w]))
    want = cl.forward(u)
    assert bool((want[5:] != 0).any())
    for i, j, k in ((12, 13, 20), (5, 18, 33)):
        bad = u.clone()
        bad[2, k, j, i] = float("inf")
        got = cl.forward(bad)
        def around(r):
            return (slice(None), slice(k - r, k + r), slice(j - r, j + r), slice(i - r, i + r))
        b, ref = got[5:].clone(), want[5:].clone()
        assert not bool(torch.isfinite(b[around(2)]).all())
        b[around(2)] = ref[around(2)] = 0.0
        assert bool(torch.isfinite(b).all()), (i, j, k)
        b[around(3)] = ref[around(3)] = 0.0
        assert torch.equal(b, ref), (i, j, k)
    cl.close()
