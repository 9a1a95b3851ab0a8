"""A sorted step whose tile counts the caller made stale, in both guard modes.

Default guards find it out in the wait that ends the call, after the readout
was queued (which must then have left particles, momenta, ids and the next
step's counts alone); deferred guards before it is queued.  Either way the
step is done again from a fresh count.  After the caller moved the particles,
three steps (stale, counted afresh, counts taken over) must follow an unsorted
context: the density is the same integers and the readout differs in the order
of eight float32 products, so positions agree to 1e-5 of the largest move and
momenta to 1e-5 of the largest kick, plus two roundings, a step at a time.
The redone step reports nothing, and a momentum that then is NaN is still
reported: at once, or by pm_sync."""
import numpy as np
import pytest
import torch

from paper_2007_13394_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("name,over", [("C1", {}), ("C5", dict(n_mesh=256, n_cdm=64, n_sites=8))])
@pytest.mark.parametrize("deferred", [False, True])
def test_stale_counts(dev, name, over, deferred):
    from paper_2007_13394_amd import pm
    cfg = I.config(name, **over)
    n = cfg["n_mesh"]
    x32, p32 = I.synthetic_state(cfg, seed=81)
    free = pm.Ctx(pm.make_config(cfg, flags=pm.PM_FLAG_NO_SORT))
    ctx = pm.Ctx(pm.make_config(cfg, flags=pm.PM_FLAG_DEFER_GUARDS if deferred else 0))
    ids = torch.arange(ctx.P, dtype=torch.int32, device=dev)
    pm.pm_attach_ids(ctx, ids)
    xs, ps = torch.from_numpy(x32).to(dev), torch.from_numpy(p32).to(dev)
    call = (0.5, 0.4975, 0.5025, 0.505)
    pm.pm_step(ctx, xs, ps, *call)
    xs.add_(torch.tensor([[7.25], [19.5], [3.0]], device=dev)).remainder_(n)
    xs.masked_fill_(xs >= n, 0.0)
    drift = abs(pm.pm_kdk_factors(ctx, *call)[1])
    for _ in range(3):
        k = ids.long()
        x, p = torch.empty_like(xs), torch.empty_like(ps)
        x[:, k], p[:, k] = xs, ps
        p0 = p.clone()
        pm.pm_step(ctx, xs, ps, *call)
        pm.pm_step(free, x, p, *call)
        pm.pm_sync(ctx)
        k = ids.long()
        assert np.array_equal(np.sort(ids.cpu().numpy()), np.arange(ctx.P))
        pmax = float(p.abs().max())
        assert float((ps - p[:, k]).abs().max()) <= 1e-5 * float((p - p0).abs().max()) + 2 * pmax * 2.0 ** -23
        d = (xs - x[:, k]).abs()
        assert float(torch.minimum(d, n - d).max()) <= 1e-5 * drift * pmax + 2 * n * 2.0 ** -23
    ps[1, 1234] = float("nan")
    with pytest.raises(pm.PMError) as e:
        pm.pm_step(ctx, xs, ps, *call)
        pm.pm_sync(ctx)
    assert e.value.status == pm.PM_ERR_NAN
