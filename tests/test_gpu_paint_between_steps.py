"""pm_paint between sorted steps takes the counts that the last step left and
leaves them to the next one: that step counts nothing and sorts, paints and reads
out once, as without the paint, and its particles are the same bits (the density
is a sum of integers and a particle's readout depends on nothing else).  Counts
that the caller made stale are found out by the paint, and the step after it
counts its own."""
import numpy as np
import pytest
import torch

from paper_2007_13394_amd import inputs as I

pytestmark = pytest.mark.gpu

CALL = (0.5, 0.4975, 0.5025, 0.505)


def by_id(ids, x, p):
    k = ids.long()
    a, b = torch.empty_like(x), torch.empty_like(p)
    a[:, k], b[:, k] = x, p
    return a, b


@pytest.mark.parametrize("name,over", [("C1", {}), ("C5", dict(n_mesh=256, n_cdm=64, n_sites=8))])
@pytest.mark.parametrize("deferred", [False, True])
@pytest.mark.parametrize("paints", [1, 2])
@pytest.mark.parametrize("moved", [False, True])
def test_step_after_paint(dev, name, over, deferred, paints, moved):
    from paper_2007_13394_amd import pm
    cfg = I.config(name, **over)
    n = cfg["n_mesh"]
    x32, p32 = I.synthetic_state(cfg, seed=91)
    mesh = torch.zeros(n ** 3, dtype=torch.int64, device=dev)
    out = []
    for paint in (False, True):
        ctx = pm.Ctx(pm.make_config(cfg, flags=pm.PM_FLAG_DEFER_GUARDS if deferred else 0))
        ids = torch.arange(ctx.P, dtype=torch.int32, device=dev)
        pm.pm_attach_ids(ctx, ids)
        x, p = torch.from_numpy(x32).to(dev), torch.from_numpy(p32).to(dev)
        for _ in range(2):
            pm.pm_step(ctx, x, p, *CALL)
        if moved:
            x.add_(torch.tensor([[7.25], [19.5], [3.0]], device=dev)).remainder_(n)
            x.masked_fill_(x >= n, 0.0)
        for k in range(paints if paint else 0):
            mesh.zero_()
            pm.pm_paint(ctx, x, 0, ctx.nseg, mesh)
            off, _, quantum = pm.pm_segments(ctx)
            assert int(mesh.sum()) == int((np.diff(off) * quantum).sum())
        pm.pm_trace_begin(ctx)
        for _ in range(2):
            pm.pm_step(ctx, x, p, *CALL)
        names = [k for k, _ in pm.pm_trace_end(ctx)]
        pm.pm_sync(ctx)
        if not moved or paint:
            assert names.count("sort_count") == (1 if moved else 0), names
            assert names.count("sort_scatter") == names.count("paint") == names.count("readout_kick_drift") == 2, names
        out.append(by_id(ids, x, p))
    for a, b in zip(*out):
        assert torch.equal(a, b)
