"""The adjoint of a squaring step without records, for subjects whose cells lie
beyond one voxel somewhere: blocks start on them, meet such a cell or another
block's mark, and leave them to the kernels after."""

import numpy as np
import pytest
import torch

from oracle import darc_oracle as O
from paper_2508_10743_amd import darc as D

pytestmark = pytest.mark.gpu

# at most 27 sources, each product and sum rounded once, twice
TOL = 2 * 32 * 2.0 ** -24


@pytest.fixture(autouse=True)
def march():
    assert torch.cuda.is_available(), "GPU tests need a ROCm GPU"
    D.set_launch_shape("squaring", None, 0, 8)
    yield
    D.autotune_clear()


def step(dims, peaks):
    """One field per peak: cells at offset -1 with one source each (but at the
    low faces), and the peak on a few voxels of the first planes."""
    rng = np.random.default_rng(5)
    u = rng.uniform(-0.4, -0.2, (len(peaks), 3) + dims).astype(np.float32)
    for i, p in enumerate(peaks):
        u[i, :, 2:4, 6:9, 10:14] = p
    return u, rng.uniform(-1.0, 1.0, u.shape).astype(np.float32)


def test_subjects_left_by_some_of_many_blocks():
    """More blocks than run at once (36 per subject), so that some start after
    their subject was marked and some meet its far cells themselves."""
    dims, copies = (48, 41, 40), 13
    peaks = [1.4, -0.3, 3.5]
    u, gr = step(dims, peaks)
    v = torch.from_numpy(np.tile(u * 2.0, (copies, 1, 1, 1, 1))).cuda()
    g = torch.from_numpy(np.tile(gr, (copies, 1, 1, 1, 1))).cuda()
    got = D.exp_svf_bwd(v, None, g, 1).cpu().numpy()
    for i in range(len(peaks)):
        ref = O.squaring_step_bwd(u[i], gr[i]) * 0.5
        for k in range(copies):
            err = np.linalg.norm(got[k * len(peaks) + i] - ref) / np.linalg.norm(ref)
            assert err <= TOL, (i, k, err)
