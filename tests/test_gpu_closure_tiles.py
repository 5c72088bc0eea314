"""The persistent convolution kernels where a workgroup walks several tiles
(two halo buffers, partial sums over tiles): single layers on a grid of more
tiles than workgroups and with halos that wrap and do not, against the same
sums in float64 torch on the same BF16 operands.  Bound 1e-5 of the output's
scale, FP32 against FP64 accumulation, as for the small grids."""
import sys

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

N3 = (96, 64, 96)


@pytest.fixture(scope="module")
def env():
    import torch
    from paper_1004_1680_amd import mhd
    mhd.load()
    return torch, mhd


def say(*a):
    print(*a, flush=True)
    sys.stdout.flush()


def operand(torch, c, seed):
    """random BF16 values as float64 [nz][ny][nx][c] and as the bits"""
    g = torch.Generator(device="cuda").manual_seed(seed)
    x = torch.randn((N3[2], N3[1], N3[0], c), generator=g, device="cuda").to(torch.bfloat16)
    return x.double(), x


def shifted(torch, x, o):
    return torch.roll(x, (1 - o // 9, 1 - (o // 3) % 3, 1 - o % 3), (0, 1, 2)).reshape(-1, x.shape[3])


def weights(cin, cout, seed):
    w = np.random.default_rng(seed).normal(0.0, 0.1, (27, cin, cout)).astype(np.float32)
    import torch
    return w, torch.from_numpy(w).to(torch.bfloat16).double().cuda()


def close(got, ref, what):
    err = float((got.double() - ref).abs().max() / ref.abs().max())
    say(f"{what}: {err:.2e}")
    assert err < 1e-5, what


@pytest.mark.parametrize("cin,cout", [(8, 32), (32, 32), (32, 8), (8, 8)])
def test_layers_over_many_tiles(env, cin, cout):
    torch, mhd = env
    say(f"case: layers over many tiles {cin}->{cout}")
    N = N3[0] * N3[1] * N3[2]
    x64, x = operand(torch, cin, 1)
    d64, dy = operand(torch, cout, 2)
    w, wd = weights(cin, cout, 3)
    bias = np.linspace(-0.2, 0.2, cout).astype(np.float32)

    y = torch.full((N, cout), float("nan"), device="cuda")
    mhd.conv3d_forward(N3, x, w, bias, y)
    ref = sum(shifted(torch, x64, o) @ wd[o] for o in range(27)) + torch.from_numpy(bias).double().cuda()
    close(y, ref, "forward")

    dx = torch.full((N, cin), float("nan"), device="cuda")
    mhd.conv3d_dgrad(N3, dy, w, dx)
    close(dx, sum(shifted(torch, d64, 26 - o) @ wd[o].T for o in range(27)), "dgrad")

    dw, db = mhd.conv3d_wgrad(N3, cin, cout, x.reshape(N, cin).T.contiguous(), dy.reshape(N, cout).T.contiguous())
    flat = d64.reshape(N, cout)
    close(torch.from_numpy(dw).cuda(), torch.stack([shifted(torch, x64, o).T @ flat for o in range(27)]), "wgrad")
    close(torch.from_numpy(db).cuda(), flat.sum(0), "bias gradient")


def test_forward_destinations(env):
    """The correction written over the state, at an address of 4 but not 16
    bytes, into pinned host memory and from a captured graph is the one of a
    plain call, bit for bit."""
    torch, mhd = env
    say("case: forward destinations")
    n = (32, 32, 64)
    g = torch.Generator(device="cuda").manual_seed(4)
    u = torch.randn((8, n[2], n[1], n[0]), generator=g, device="cuda") * 0.1 + 1.0
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        cl = mhd.Closure(n, stream=side)
        cl.set_params(np.random.default_rng(5).normal(0.0, 0.05, mhd.NPARAM).astype(np.float32))
        cl.set_gate(np.full(8, 0.5))
        want = cl.forward(u)
        over = u.clone()
        cl.forward(over, out=over)
        odd = torch.empty(u.numel() + 1, device="cuda")[1:].reshape(u.shape)
        cl.forward(u, out=odd)
        host = torch.empty(u.shape, pin_memory=True)
        cl.forward(u, out=host)
        side.synchronize()
        for name, got in (("over the state", over), ("odd address", odd), ("host", host.cuda())):
            say("destination:", name)
            assert torch.equal(got, want)
        replayed = torch.empty_like(u)
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=side):
            cl.forward(u, out=replayed)
        for _ in range(3):
            replayed.zero_()
            graph.replay()
            side.synchronize()
            assert torch.equal(replayed, want)
