"""Stride-1 convolutions with enough bricks for those of eight rows (one for each
CU), ragged and whole, with plain and upsampled inputs, against FP64 sums of the
same BF16 operands."""

import pytest
import torch
import torch.nn.functional as F

from paper_2508_10743_amd import unet as N

pytestmark = pytest.mark.gpu


# 288 bricks in 16 columns, 24 x 12 in two column blocks, 258 in one of 32, and 255
# (bricks of four rows)
@pytest.mark.parametrize("n,dims,c0,c1,up,cout", [
    (16, (5, 21, 33), 48, 0, False, 16), (12, (6, 24, 18), 16, 32, True, 40),
    (86, (4, 8, 34), 32, 16, True, 32), (85, (4, 8, 34), 16, 0, False, 8)])
def test_forward(n, dims, c0, c1, up, cout):
    assert torch.cuda.is_available(), "GPU tests need a ROCm GPU"
    g = torch.Generator().manual_seed(n + cout)
    r = lambda *s: torch.randn(*s, generator=g).to(torch.bfloat16)  # noqa: E731
    lo = tuple(d // 2 for d in dims) if up else dims
    x0, x1 = r(2, *lo, c0), r(2, *dims, c1) if c1 else None
    w = N.bf16_round(torch.randn(cout, c0 + c1, 3, 3, 3, generator=g).numpy() * 0.1)
    bias = torch.randn(cout, generator=g)
    full = x0.double()
    for a in (1, 2, 3):
        full = full.repeat_interleave(2, a) if up else full
    if c1:
        full = torch.cat([full, x1.double()], -1)
    wd = torch.from_numpy(w).double()
    x = full.permute(0, 4, 1, 2, 3)
    ref = F.conv3d(x, wd, bias.double(), padding=1)
    # FP32 accumulation over 27 cin products and the bias, then one BF16 rounding
    tol = 2 * (27 * (c0 + c1) / 32 + 2) * 2.0 ** -24
    bound = tol * (F.conv3d(x.abs(), wd.abs(), padding=1) + bias.abs().view(-1, 1, 1, 1).double())
    bound += 2.0 ** -8 * ref.abs()

    def many(t):
        return None if t is None else t.repeat(n // 2 + 1, 1, 1, 1, 1)[:n].cuda()

    y = N.conv3d(many(x0), N.to_bf16_device(N.pack_weights(w), torch.device("cuda", 0)), bias.cuda(),
                 cout, x1=many(x1), up0=up).cpu().double().permute(0, 4, 1, 2, 3)
    for k in range(n):
        assert bool(((y[k] - ref[k % 2]).abs() <= bound[k % 2]).all()), k
