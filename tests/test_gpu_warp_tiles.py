"""The warp and its adjoint at the edges of their 32 x 4 x 2 tiles, both forms of
the adjoint (accumulated and overwritten), and centring at the edges of the
register-held subject counts."""

import numpy as np
import pytest
import torch

from oracle import darc_oracle as O
from paper_2508_10743_amd import darc as D

pytestmark = pytest.mark.gpu

EPS = 2.0 ** -24


@pytest.mark.parametrize("dims", [(2, 2, 2), (2, 4, 32), (3, 5, 33), (5, 3, 31), (7, 9, 65)])
def test_warp_and_both_adjoints(dims):
    rng = np.random.default_rng(dims[2])
    img = rng.uniform(0.0, 1.0, (3,) + dims).astype(np.float32)
    u = rng.uniform(-3.0, 3.0, (3, 3) + dims).astype(np.float32)
    gr = rng.uniform(-1.0, 1.0, img.shape).astype(np.float32)
    acc = rng.uniform(-1.0, 1.0, u.shape).astype(np.float32)
    t = [torch.from_numpy(x).cuda() for x in (img, u, gr, acc)]
    out = D.warp3d(t[0], t[1]).cpu().numpy()
    fresh = D.warp3d_bwd(t[0], t[1], t[2]).cpu().numpy()
    total = D.warp3d_bwd(t[0], t[1], t[2], t[3]).cpu().numpy()
    for i in range(3):
        # seven interpolations of values in [0, 1], each a rounded difference
        # and a fused step, and a fraction rounded to 2^-25
        assert np.abs(out[i] - O.warp3d(img[i], u[i])).max() <= 32 * EPS
        ref = O.warp3d_bwd(img[i], u[i], gr[i])
        assert np.abs(fresh[i] - ref).max() <= 48 * EPS
        assert np.abs(total[i] - (acc[i] + ref)).max() <= 52 * EPS


@pytest.mark.parametrize("n", [1, 8, 9, 16, 17, 24, 25, 32, 33])
def test_center_counts(n):
    u = np.random.default_rng(n).uniform(-2.0, 2.0, (n, 3, 3, 5, 7)).astype(np.float32)
    t = torch.from_numpy(u).cuda()
    mean = D.center(t).cpu().numpy()
    ref = u.astype(np.float64).mean(0)
    assert np.abs(mean - ref).max() <= 2 * EPS * 2.0
    assert np.abs(t.cpu().numpy() - (u - ref)).max() <= 2 * EPS * 4.0
