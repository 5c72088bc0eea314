"""The closure's own epilogues where a convolution's workgroup walks several
tiles (staged BF16 outputs stored two tiles late, masks of the tile that is
stored, gate and channel sums over tiles): gated corrections, losses and
gradients on grids with one to nine tiles to a workgroup, evenly and not,
against float64 layers with the kernels' BF16 rounding of activations and
gradients between them.

Bounds.  What differs is a rounding to BF16 of a value that FP32 and FP64 sums
place on two sides of a tie: with sums off by up to 5e-5 of their terms and a
BF16 step of 2^-8, one value in a hundred by one step, 2^-8 sqrt(1/100) = 4e-4
of a layer in L2, through three layers (and back, for gradients): 1e-3 and
2e-3, of the terms that are added up: a field's correction is a difference of
neighbouring outputs, and without a gate the last layer's bias gradient is a
sum that cancels to zero (the correction does not depend on it).  One misplaced
row of 16 cells is 0.5% or more of these grids."""
import sys

import numpy as np
import pytest

from oracle import closure as C
from paper_1004_1680_amd import inputs as I

pytestmark = pytest.mark.gpu

# tiles of 16 x 4 x 4 (32 -> 8 channels: x 8) over 256 workgroups: 1 (1/2), 2
# (1), 3 (1 or 2), 4 or 5 (2 or 3), 9 (4 or 5)
GRIDS = [(32, 32, 64), (64, 32, 64), (96, 32, 64), (96, 96, 32), (96, 64, 96)]


@pytest.fixture(scope="module")
def env():
    import torch
    from paper_1004_1680_amd import mhd
    mhd.load()
    return torch, mhd


def say(*a):
    print(*a, flush=True)
    sys.stdout.flush()


def rel(a, b):
    return float(np.linalg.norm(a - b) / np.linalg.norm(b))


class Net:
    """the three layers and their gradients in float64 on the device"""

    def __init__(self, torch, n, ps):
        self.t, self.n = torch, n
        self.w = [torch.from_numpy(p).to(torch.bfloat16).double().cuda() if p.ndim == 3 else
                  torch.from_numpy(p.astype(np.float32)).double().cuda() for p in ps]

    def bf16(self, x):
        return x.float().to(self.t.bfloat16).double()

    def shifted(self, x, o):
        n = self.n
        g = x.reshape(n[2], n[1], n[0], -1)
        return self.t.roll(g, (1 - o // 9, 1 - (o // 3) % 3, 1 - o % 3), (0, 1, 2)).reshape(x.shape)

    def conv(self, x, l):
        return sum(self.shifted(x, o) @ self.w[2 * l][o] for o in range(27)) + self.w[2 * l + 1]

    def dgrad(self, d, l):
        return sum(self.shifted(d, 26 - o) @ self.w[2 * l][o].T.contiguous() for o in range(27))

    def wgrad(self, x, d):
        return self.t.stack([self.shifted(x, o).T.contiguous() @ d for o in range(27)]), d.sum(0)


@pytest.mark.parametrize("gated", [True, False])
@pytest.mark.parametrize("n", GRIDS)
def test_network_over_many_tiles(env, n, gated):
    torch, mhd = env
    say(f"case: network over many tiles n={n} gated {gated}")
    N = n[0] * n[1] * n[2]
    rng = np.random.default_rng(21)
    f32 = lambda a: np.asarray(a, dtype=np.float32).astype(np.float64)
    u = f32(I.random_smooth(n, seed=22).reshape(8, N) + 0.02 * rng.normal(size=(8, N)))
    mean, std = f32(u.mean(1)), f32(u.std(1) + 1e-3)
    ps = C.init_params(23)
    ps[4] = ps[4] * 10.0
    for k in (1, 3, 5):
        ps[k] = rng.normal(0.0, 0.1, ps[k].shape)
    scale, tscale = f32(rng.uniform(0.5, 1.5, 8)), f32(rng.uniform(0.5, 1.5, 8))
    target = f32(rng.normal(size=(8, N)))
    rough = f32(rng.uniform(0.05, 0.2, 8))

    cl = mhd.Closure(n)
    cl.set_params(C.flatten(ps).astype(np.float32))
    cl.set_scales(mean, std, scale, tscale)
    if gated:
        cl.set_gate(rough)
    shape = (8, n[2], n[1], n[0])
    ud = torch.from_numpy(u.astype(np.float32)).reshape(shape).cuda()
    td = torch.from_numpy(target.astype(np.float32)).reshape(shape).cuda()
    delta = cl.forward(ud).cpu().double().numpy().reshape(8, N)
    loss, grads = cl.grad(ud, td)
    again = cl.forward(ud).cpu().double().numpy().reshape(8, N)
    cl.close()
    assert np.array_equal(delta, again)

    net = Net(torch, n, ps)
    x0 = net.bf16(torch.from_numpy(C.normalize(u, mean, std)).cuda())
    a1 = net.bf16(net.conv(x0, 0).clamp(min=0.0))
    a2 = net.bf16(net.conv(a1, 1).clamp(min=0.0))
    o = net.conv(a2, 2).cpu().numpy()
    g = C.gate(u, rough, n) if gated else np.ones(N)
    ref = C.project(o * g[:, None], scale, n)
    size = [np.linalg.norm(scale[f] * o[:, f] * g) for f in range(8)]
    terms = size[:5] + [2.0 * np.hypot(size[5 + (d + 1) % 3], size[5 + (d + 2) % 3]) for d in range(3)]
    worst = [np.linalg.norm(delta[f] - ref[f]) / terms[f] for f in range(8)]
    say("forward", rel(delta, ref), "by field", max(worst))
    assert rel(delta, ref) < 1e-3 and max(worst) < 1e-3

    r = (ref - target) / tscale[:, None]
    L = float(np.mean(r * r))
    go = C.project_T(2.0 * r / tscale[:, None] / r.size, scale, n) * g[:, None]
    # gradients of the mean over 8 N values are tiny: BF16 has FP32's range
    gob = net.bf16(torch.from_numpy(go).cuda())
    g2 = net.bf16(net.dgrad(gob, 2) * (a2 > 0))
    g1 = net.bf16(net.dgrad(g2, 1) * (a1 > 0))
    assert loss == pytest.approx(L, rel=1e-4)
    got = C.unflatten(grads.astype(np.float64))
    for l, (x, d) in enumerate(((x0, g1), (a1, g2), (a2, gob))):
        dw, db = [t.cpu().numpy() for t in net.wgrad(x, d)]
        ew = rel(got[2 * l], dw)
        eb = float((np.abs(got[2 * l + 1] - db) / d.abs().sum(0).cpu().numpy()).max())
        say("gradient of layer", l + 1, ew, "bias", eb)
        assert ew < 2e-3 and eb < 2e-3
