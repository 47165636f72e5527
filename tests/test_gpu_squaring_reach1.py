"""The adjoint of a squaring step whose cells lie within one voxel (hat-function
gather, marching on 32 x 16 columns or on tiles of 32 x 8 x 2) at the edges of
its tiles, with positions clamped at the faces, and with gradients that are not
finite."""

import numpy as np
import pytest
import torch

from oracle import darc_oracle as O
from paper_2508_10743_amd import darc as D

pytestmark = pytest.mark.gpu

# at most 27 sources, each product and sum rounded once (about 32 roundings of
# 2^-24 relative to the terms, which do not cancel beyond their own size), twice
TOL = 2 * 32 * 2.0 ** -24


@pytest.fixture(autouse=True, params=[8, -1], ids=["march", "tiles"])
def shape(request):
    assert torch.cuda.is_available(), "GPU tests need a ROCm GPU"
    D.set_launch_shape("squaring", None, 0, request.param)
    yield request.param
    D.autotune_clear()


def noise_step(seed, n, dims):
    """u in (-1, 1) without any smoothness, zeros of both signs, and voxels on
    and next to the faces pointing far outwards (their cells stay in reach)."""
    rng = np.random.default_rng(seed)
    u = rng.uniform(-0.999, 0.999, (n, 3) + dims).astype(np.float32)
    u[rng.random(u.shape) < 0.05] = 0.0
    u[rng.random(u.shape) < 0.05] = -0.0
    for c in range(3):
        f = np.moveaxis(u[:, c], c + 1, 0)
        D0 = f.shape[0]
        far = rng.random(f.shape[1:]) < 0.3
        f[0][far], f[D0 - 1][far] = -5.5, 7.25
        if D0 > 3:
            f[1][far], f[D0 - 2][far] = -3.5, 1.0
    return u, rng.uniform(-1.0, 1.0, u.shape).astype(np.float32)


@pytest.mark.parametrize("dims", [(2, 2, 2), (3, 15, 31), (9, 16, 32), (8, 17, 33), (34, 18, 34),
                                  (5, 33, 65)])
def test_step_adjoint_matches_oracle(dims):
    u, gr = noise_step(500 + dims[2], 2, dims)
    for n_sq in (1, 2):  # the first step (scaled on the fly) and a later one
        v = u * 2.0 if n_sq == 1 else np.zeros_like(u)
        vd, gd = torch.from_numpy(v).cuda(), torch.from_numpy(gr).cuda()
        ck = torch.from_numpy(u[None].copy()).cuda() if n_sq == 2 else None
        got = D.exp_svf_bwd(vd, ck, gd, n_sq).cpu().numpy()
        for i in range(2):
            # with v = 0 the first step doubles the gradient, and the scale
            # 1/4 follows
            ref = O.squaring_step_bwd(u[i], gr[i]) * 0.5
            err = np.linalg.norm(got[i] - ref) / np.linalg.norm(ref)
            assert err <= TOL, (n_sq, i, err)


def test_non_finite_gradient_touches_the_same_voxels():
    """An infinite and a NaN gradient reach exactly the voxels that they reach
    in the oracle; the rest and another subject of the launch are unaffected."""
    dims = (10, 20, 40)
    u, gr = noise_step(77, 2, dims)
    gr[0, 1, 4, 9, 17] = np.inf
    gr[0, 2, 6, 3, 30] = np.nan
    vd, gd = torch.from_numpy(u * 2.0).cuda(), torch.from_numpy(gr).cuda()
    got = D.exp_svf_bwd(vd, None, gd, 1).cpu().numpy()
    for i in range(2):
        with np.errstate(invalid="ignore"):
            ref = O.squaring_step_bwd(u[i], gr[i]) * 0.5
        ok = np.isfinite(ref)
        assert np.array_equal(np.isfinite(got[i]), ok)
        assert (~ok).sum() < 200 and ((~ok).sum() > 0) == (i == 0)
        assert np.linalg.norm(got[i][ok] - ref[ok]) <= TOL * np.linalg.norm(ref[ok])
