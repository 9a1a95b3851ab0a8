"""Reverse mode of the learned correction's CNN on the matrix cores, against the
FP64 oracle: every parameter block by itself, at a mesh of a few tiles (16) and
one where workgroups take several (64).

Tolerance: the GPU rounds weights and activations to BF16 (relative error at
most 2^-9 each); a gradient block sees at most four such roundings in a
product, so 4 x 2^-9 < 1e-2 bounds the relative L2 error.  db3 is the sum of a
mean-free field, zero up to rounding, and is left out."""
import numpy as np
import pytest
import torch

import oracle as O
from paper_2007_13394_amd import inputs as I
from test_gpu_net import _params, rel_l2, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("mesh", [16, 64])
def test_cnn_gradient_blocks_vs_oracle(dev, mesh):
    from paper_2007_13394_amd import pm
    cfg = I.config("C5_fd16", n_mesh=mesh, n_cdm=mesh // 2, n_sites=2, n_shell=3, n_fib=1)
    ctx = pm.Ctx(pm.make_config(cfg, flags=pm.PM_FLAG_LEARNED | pm.PM_FLAG_NO_SORT))
    sim = O.make_sim(cfg)
    x32, _ = I.synthetic_state(cfg, seed=81)
    th32 = _params(82)
    rng = np.random.default_rng(83)
    target = (O.force_cont(sim, x32.astype(np.float64)) * (1 + 0.2 * rng.standard_normal(x32.shape))).astype(np.float32)
    th, x, t = (torch.from_numpy(a).to(dev) for a in (th32, x32, target))
    d = torch.zeros_like(th)
    pm.pm_learned_loss(ctx, th, 0.6, x, t, d)
    _, rd = O.learned_loss(sim, th32.astype(np.float64), 0.6, x32.astype(np.float64), target.astype(np.float64))
    g = d.cpu().numpy()
    for k in ("C1W", "C1B", "C2W", "C2B", "C3W"):
        o, n = O.NET_OFF[k]
        e = rel_l2(g[o:o + n], rd[o:o + n])
        say(mesh, k, "rel L2", e)
        assert e < 1e-2, (mesh, k, e)
    # the gradient adds to what dtheta holds
    pm.pm_learned_loss(ctx, th, 0.6, x, t, d)
    assert rel_l2(d.cpu().numpy(), 2.0 * g) < 1e-5


@pytest.mark.parametrize("mesh", [16, 32])
def test_non_finite_force_gives_a_non_finite_gradient(dev, mesh):
    """A NaN that reaches the forces is not turned into numbers by the
    fixed-point cotangent paint (meshes of tiles) or the float one (16)."""
    from paper_2007_13394_amd import pm
    cfg = I.config("C5_fd16", n_mesh=mesh, n_cdm=8)
    ctx = pm.Ctx(pm.make_config(cfg, flags=pm.PM_FLAG_LEARNED | pm.PM_FLAG_NO_SORT))
    x32, _ = I.synthetic_state(cfg, seed=84)
    th32 = _params(85)
    th32[O.NET_OFF["B3"][0]] = np.nan
    th, x = torch.from_numpy(th32).to(dev), torch.from_numpy(x32).to(dev)
    d = torch.zeros_like(th)
    loss = pm.pm_learned_loss(ctx, th, 0.6, x, torch.ones_like(x), d)
    assert np.isnan(loss)
    o, n = O.NET_OFF["C3W"]
    assert torch.isnan(d[o:o + n]).all()
