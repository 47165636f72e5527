"""Outputs beyond the last-level cache, which are stored past it where their rows
allow: the same bits as from launches of half the subjects, which are not."""

import pytest
import torch

from paper_2508_10743_amd import darc as D

pytestmark = pytest.mark.gpu

N = 16


def halves(f, *tensors):
    return torch.cat([f(*(t[k:k + N // 2] for t in tensors)) for k in (0, N // 2)])


# 16 fields of 112 x 112 x 112 are 270 MB; rows of whole and of broken 64-byte
# pieces
@pytest.mark.parametrize("d2", [112, 113])
def test_same_bits_as_in_halves(d2):
    assert torch.cuda.is_available(), "GPU tests need a ROCm GPU"
    dims = (112, 112, d2)
    gen = torch.Generator("cuda").manual_seed(d2)

    def rand(shape, lo, hi):
        return torch.rand(shape, generator=gen, device="cuda") * (hi - lo) + lo

    img, g_img = rand((N,) + dims, 0.0, 1.0), rand((N,) + dims, -1.0, 1.0)
    v, g, acc = (rand((N, 3) + dims, -0.9, 0.9) for _ in range(3))
    assert v.numel() * 4 > 256 << 20

    for n_sq in (1, 2):  # both kinds of step
        u, ck = D.exp_svf(v, n_sq)
        assert torch.equal(u, halves(lambda x: D.exp_svf(x, n_sq)[0], v))
        assert torch.equal(D.exp_svf_bwd(v, ck, g, n_sq),
                           halves(lambda x, y: D.exp_svf_bwd(x, D.exp_svf(x, n_sq)[1], y, n_sq),
                                  v, g))
    assert torch.equal(D.gauss_smooth(v, 1.0), halves(lambda x: D.gauss_smooth(x, 1.0), v))
    assert torch.equal(D.warp3d_bwd(img, v, g_img), halves(D.warp3d_bwd, img, v, g_img))
    assert torch.equal(D.warp3d_bwd(img, v, g_img, acc.clone()),
                       halves(D.warp3d_bwd, img, v, g_img, acc.clone()))

    # a step with recorded cells
    def stepped(x, y):
        c = D.Cohort(x, D.SweepParams(metric="mse", n_sq=2, k2=1, batch=N), v0=y.clone())
        c.atlas.copy_(img[0])
        c.sweep()
        return c.v

    assert torch.equal(stepped(img, v), halves(stepped, img, v))
