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


def noise_step(seed, n, dims, beside=True):
    """u in (-1, 1) without any smoothness, zeros of both signs, and voxels on
    (and beside) the faces pointing far outwards (their cells stay in reach)."""
    rng = np.random.default_rng(seed)
    u = rng.uniform(-0.999, 0.999, (n, 3) + dims).astype(np.float32)
    u[rng.random(u.shape) < 0.05] = 0.0
    u[rng.random(u.shape) < 0.05] = -0.0
    for c in range(3):
        f = np.moveaxis(u[:, c], c + 1, 0)
        D0 = f.shape[0]
        far = rng.random(f.shape[1:]) < 0.3
        f[0][far], f[D0 - 1][far] = -5.5, 7.25
        if D0 > 3 and beside:
            f[1][far], f[D0 - 2][far] = -3.5, 1.0
    return u, rng.uniform(-1.0, 1.0, u.shape).astype(np.float32)


@pytest.mark.parametrize("dims", [(2, 2, 2), (3, 15, 31), (9, 16, 32), (8, 17, 33), (34, 18, 34),
                                  (5, 33, 65)])
@pytest.mark.parametrize("beside", [False, True])
def test_step_adjoint_matches_oracle(dims, beside):
    u, gr = noise_step(500 + dims[2], 2, dims, beside)
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
    u, gr = noise_step(77, 2, dims, beside=False)
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


@pytest.mark.parametrize("dims", [(3, 15, 31), (9, 17, 33), (20, 33, 40)])
def test_sweep_gradient_with_recorded_reaches(dims):
    """The same field inside a sweep, whose forward pass records the cells: the
    first moment after one step is (1 - beta1) times the gradient."""
    u, _ = noise_step(900 + dims[0], 2, dims)
    imgs = np.random.default_rng(901).uniform(0.0, 1.0, (2,) + dims).astype(np.float32)
    par = dict(metric="mse", lam=0.0, n_sq=1, k2=1)
    coh = D.Cohort(torch.from_numpy(imgs).cuda(), D.SweepParams(**par),
                   v0=torch.from_numpy(u * 2.0).cuda())
    atlas = coh.atlas.cpu().numpy().astype(np.float64)
    coh.sweep()
    got = coh.m.cpu().numpy() / 0.1
    for i in range(2):
        _, ref = O.subject_loss_grad(imgs[i].astype(np.float64), (u[i] * 2.0).astype(np.float64),
                                     atlas, O.SweepParams(**par))
        assert np.linalg.norm(got[i] - ref) <= 1e-4 * np.linalg.norm(ref)


def test_checkpoints_of_another_velocity():
    """The adjoint looks at the fields it is given, not at what the velocity
    suggests: steps of reach 1, 2 and beyond in any order, subjects mixed."""
    dims = (12, 21, 40)
    amp = [[0.5, 6.0], [1.7, 0.6], [0.4, 1.8], [9.0, 0.3]]  # u_0 .. u_3 per subject
    rng = np.random.default_rng(31)
    from synthetic.cohorts import random_velocity
    u = np.stack([np.concatenate([random_velocity(40 + 2 * t + i, 1, dims, a[i], corr_len=3.0)
                                  for i in range(2)]) for t, a in enumerate(amp)])
    gr = rng.uniform(-1.0, 1.0, u.shape[1:]).astype(np.float32)
    v = u[0] * 2.0 ** 4
    got = D.exp_svf_bwd(torch.from_numpy(v).cuda(), torch.from_numpy(u[1:].copy()).cuda(),
                        torch.from_numpy(gr).cuda(), 4).cpu().numpy()
    for i in range(2):
        ref = O.exp_svf_bwd([x[i].astype(np.float64) for x in u], gr[i].astype(np.float64))
        assert np.linalg.norm(got[i] - ref) <= 1e-4 * np.linalg.norm(ref)
