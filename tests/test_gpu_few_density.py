"""The density of unsorted positions is painted by tile or, of few particles or onto
few tiles, with global atomics: on both sides of the lines pm_density's cells are
those of the painted integers, bit for bit, into aligned and unaligned meshes, and
pm_force and pm_power follow from the same cells.

Force: eight float32 products with weights of two roundings, 2e-6 of the largest
mesh value.  Power: the same float32 density through the same transforms as
pm_power_mesh, whose bins are summed in another order: 1e-12."""
import numpy as np
import pytest
import torch

from paper_2007_13394_amd import inputs as I
from test_gpu_sparse_readout import cic

pytestmark = pytest.mark.gpu


# whether positions in canonical and in sorted order go by tile
@pytest.mark.parametrize("n,nc,ns,canonical,in_order", [
    (32, 8, 0, False, False), (64, 16, 0, False, False), (128, 16, 0, False, False),   # up to 4096 particles
    (64, 8, 2, True, False), (64, 32, 0, True, True), (256, 8, 0, True, True),
    (32, 32, 0, False, False), (32, 16, 4, True, False), (32, 32, 16, False, True)])   # eight tiles
@pytest.mark.parametrize("offset", [0, 1])
def test_density(dev, n, nc, ns, canonical, in_order, offset):
    from paper_2007_13394_amd import pm
    cfg = I.config("C1", n_mesh=n, n_cdm=nc, n_sites=ns)
    ctx = pm.Ctx(pm.make_config(cfg))
    x32, p32 = I.synthetic_state(cfg, seed=97)
    x, p = torch.from_numpy(x32).to(dev), torch.from_numpy(p32).to(dev)
    delta = torch.full((n ** 3 + offset,), 7.0, device=dev)[offset:]
    off, mass, quantum = pm.pm_segments(ctx)
    F, acc = torch.empty(3, n, n, n, device=dev), torch.empty_like(x)
    for permuted, tiles in ((False, canonical), (True, in_order)):
        q = torch.zeros(n ** 3, dtype=torch.int64, device=dev)
        if permuted:
            pm.pm_step(ctx, x, p, 0.5, 0.4975, 0.5025, 0.505)
            pm.pm_paint(ctx, x, 0, ctx.nseg, q)
        else:
            for k in range(ctx.nseg):
                pm.pm_paint_q(ctx, x, int(off[k]), int(off[k + 1] - off[k]), int(quantum[k]), q)
        pm.pm_trace_begin(ctx)
        pm.pm_density(ctx, x, delta)
        names = [k for k, _ in pm.pm_trace_end(ctx)]
        assert names.count("sort_scatter") == (1 if tiles else 0), names
        assert torch.equal(delta, (q.double() * 2.0 ** -cfg["shift"] - 1.0).float())
        pm.pm_force_mesh(ctx, q, F)
        pm.pm_force(ctx, x, acc)
        assert float((acc.double() - cic(F, x)).abs().max()) <= 2e-6 * float(F.abs().max())
        # pm_power normalises by the painted mass itself
        scale = n ** 3 / float(sum(int(m) * int(c) for m, c in zip(quantum, np.diff(off))))
        d = (q.double() * scale - 1.0).float().view(n, n, n)
        _, pk, nm = pm.pm_power(ctx, x, 0, ctx.nseg, nbins=n // 2)
        _, ref, nr = pm.pm_power_mesh(ctx, d, d, n // 2)
        assert np.array_equal(nm, nr) and np.abs(pk - ref).max() <= 1e-12 * ref.max()


@pytest.mark.parametrize("n,nc,ns", [(32, 32, 0), (256, 32, 0), (64, 32, 8)])   # gathered twice, by tile
def test_loss_with_and_without_gradient(dev, n, nc, ns):
    """One loss, read out by tile for the gradient: the forces differ in the order
    of eight products, 1e-6 of a force, the loss in less."""
    from paper_2007_13394_amd import pm
    cfg = I.config("C1", n_mesh=n, n_cdm=nc, n_sites=ns)
    ctx = pm.Ctx(pm.make_config(cfg, flags=pm.PM_FLAG_LEARNED | pm.PM_FLAG_NO_SORT))
    x32, p32 = I.synthetic_state(cfg, seed=99)
    x, t = torch.from_numpy(x32).to(dev), torch.from_numpy(p32).to(dev)
    th = 0.05 * torch.randn(pm.pm_net_nparam(), device=dev, generator=torch.Generator(device=dev).manual_seed(4))
    alone = pm.pm_learned_loss(ctx, th, 0.5, x, t)
    assert abs(alone - pm.pm_learned_loss(ctx, th, 0.5, x, t, torch.zeros_like(th))) <= 1e-6 * alone
