"""Stride-1 convolutions at the edges of their bricks (4 x 4 x 16 and 4 x 8 x 16
voxels), of the channel chunks (16) and of the column blocks (16 and 32), against FP64 sums of
the same BF16 operands."""

import numpy as np
import pytest
import torch
import torch.nn.functional as F

from paper_2508_10743_amd import unet as N

pytestmark = pytest.mark.gpu


def operands(seed, n, dims, c0, c1, up, cout):
    g = torch.Generator().manual_seed(seed)
    r = lambda *s: torch.randn(*s, generator=g).to(torch.bfloat16)  # noqa: E731
    lo = tuple(d // 2 for d in dims) if up else dims
    x0 = r(n, *lo, c0)
    x1 = r(n, *dims, c1) if c1 else None
    w = N.bf16_round(torch.randn(cout, c0 + c1, 3, 3, 3, generator=g).numpy() * 0.1)
    full = x0.double()
    for a in (1, 2, 3):
        full = full.repeat_interleave(2, a) if up else full
    if c1:
        full = torch.cat([full, x1.double()], -1)
    return x0, x1, w, torch.randn(cout, generator=g), full


@pytest.mark.parametrize("dims,c0,c1,up,cout", [
    ((2, 2, 2), 16, 0, False, 16), ((4, 4, 16), 16, 0, False, 3), ((5, 3, 17), 32, 0, False, 17),
    ((6, 6, 18), 32, 16, True, 16), ((4, 8, 34), 16, 32, True, 33), ((9, 15, 16), 32, 0, False, 24),
    ((6, 24, 18), 16, 32, True, 72), ((5, 21, 33), 48, 0, False, 8), ((3, 5, 15), 16, 16, False, 40),
    ((4, 6, 20), 24, 8, False, 16), ((4, 4, 18), 8, 8, True, 20)])
def test_forward_and_input_gradient(dims, c0, c1, up, cout):
    n, cin = 2, c0 + c1
    x0, x1, w, bias, full = operands(dims[2] + cout, n, dims, c0, c1, up, cout)
    dev = torch.device("cuda", 0)
    y = N.conv3d(x0.to(dev), N.to_bf16_device(N.pack_weights(w), dev), bias.to(dev), cout,
                 x1=None if x1 is None else x1.to(dev), up0=up, out_planar=True).cpu().double()
    wd = torch.from_numpy(w).double()
    x = full.permute(0, 4, 1, 2, 3)
    ref = F.conv3d(x, wd, bias.double(), padding=1)
    # FP32 accumulation over 27 cin products and the bias
    tol = (27 * cin / 32 + 2) * 2.0 ** -24
    bound = tol * (F.conv3d(x.abs(), wd.abs(), padding=1) + bias.abs().view(-1, 1, 1, 1).double())
    assert bool(((y - ref).abs() <= 2 * bound).all())
    if cout % 8 == 0:  # BF16 channels-last outputs: one rounding of at most 2^-9 more
        y = N.conv3d(x0.to(dev), N.to_bf16_device(N.pack_weights(w), dev), bias.to(dev), cout,
                     x1=None if x1 is None else x1.to(dev), up0=up).cpu().double()
        y = y.permute(0, 4, 1, 2, 3)
        assert bool(((y - ref).abs() <= 2 * bound + 2.0 ** -8 * ref.abs()).all())

    cz = (cout + 7) // 8 * 8
    dz = torch.zeros((n,) + dims + (cz,), dtype=torch.bfloat16)
    dz[..., :cout] = torch.randn((n,) + dims + (cout,), generator=torch.Generator().manual_seed(1)).to(
        torch.bfloat16)
    dw, db, dx = N.conv3d_grad(dz.to(dev), x0.to(dev), torch.from_numpy(N.pack_weights(w)).to(dev),
                               cout, x1=None if x1 is None else x1.to(dev), up0=up)
    d = dz.double()[..., :cout].permute(0, 4, 1, 2, 3)
    gx = F.conv_transpose3d(d, wd, padding=1)
    gb = (27 * cz / 32 + 2) * 2.0 ** -24 * F.conv_transpose3d(d.abs(), wd.abs(), padding=1)
    assert bool(((dx.cpu().double().permute(0, 4, 1, 2, 3) - gx).abs() <= 2 * gb).all())


def test_infinite_input_stays_in_its_window():
    """An infinity in the input reaches the outputs whose window holds it, and
    no others (padding of bricks, chunks and K steps is not multiplied by it)."""
    dims, cin, cout = (6, 7, 19), 32, 16
    x0, _, w, bias, _ = operands(5, 1, dims, cin, 0, False, cout)
    w[w == 0] = 0.125
    x0[0, 3, 4, 10, 7] = float("inf")
    dev = torch.device("cuda", 0)
    y = N.conv3d(x0.to(dev), N.to_bf16_device(N.pack_weights(w), dev), bias.to(dev), cout,
                 out_planar=True).cpu()
    bad = ~torch.isfinite(y[0]).all(0)
    want = torch.zeros(dims, dtype=torch.bool)
    want[2:5, 3:6, 9:12] = True
    assert bool((bad == want).all())
    # each of those windows holds it once: an infinity of the weight's sign
    tap = torch.from_numpy(w[:, 7]).flip(1, 2, 3)
    assert bool((y[0, :, 2:5, 3:6, 9:12] == tap.sign() * float("inf")).all())


@pytest.mark.parametrize("dims,c0,c1,up,cout", [
    ((2, 2, 2), 16, 0, False, 16), ((3, 5, 7), 8, 8, False, 3), ((4, 3, 8), 32, 0, False, 17),
    ((2, 6, 34), 32, 32, True, 16), ((6, 10, 8), 16, 48, True, 33), ((5, 9, 40), 24, 0, False, 8),
    ((3, 7, 31), 64, 32, False, 24), ((2, 2, 3), 16, 0, False, 8), ((2, 4, 16), 16, 8, True, 40)])
def test_weight_gradient(dims, c0, c1, up, cout):
    """Every tap, channel group and output channel at ragged rows and both
    tensors, against FP64 sums; the bias gradient beside it."""
    n, cin = 3, c0 + c1
    x0, x1, w, _, full = operands(dims[2] + 7 * cout, n, dims, c0, c1, up, cout)
    dev = torch.device("cuda", 0)
    cz = (cout + 7) // 8 * 8
    dz = torch.zeros((n,) + dims + (cz,), dtype=torch.bfloat16)
    dz[..., :cout] = torch.randn((n,) + dims + (cout,), generator=torch.Generator().manual_seed(2)).to(
        torch.bfloat16)
    wp = torch.from_numpy(N.pack_weights(w)).to(dev)
    dw, db, _ = N.conv3d_grad(dz.to(dev), x0.to(dev), wp, cout, x1=None if x1 is None else x1.to(dev),
                              up0=up, input_grad=False)
    d = dz.double()[..., :cout]
    pad = F.pad(full, (0, 0, 1, 1, 1, 1, 1, 1))
    ref = torch.zeros(cout, 27, cin, dtype=torch.float64)
    mag = torch.zeros_like(ref)
    for t in range(27):
        a, b, c = t // 9, t // 3 % 3, t % 3
        x = pad[:, a:a + dims[0], b:b + dims[1], c:c + dims[2]].reshape(-1, cin)
        ref[:, t] = d.reshape(-1, cout).T @ x
        mag[:, t] = d.abs().reshape(-1, cout).T @ x.abs()
    got = dw.cpu().double()[:, :27 * cin].view(cout, 27, cin)
    # FP32 accumulation of every voxel's product, in any order
    tol = 2 * (n * dims[0] * dims[1] * dims[2] / 32 + 8) * 2.0 ** -24
    assert bool(((got - ref).abs() <= tol * mag).all())
    bref = d.reshape(-1, cout).sum(0)
    assert bool(((db.cpu().double() - bref).abs() <= 2 * tol * 32 * d.abs().reshape(-1, cout).sum(0)).all())
