"""The tile sort on both sides of the particle count where its passes change
(2^20), at counts that are no multiple of a chunk (2048) nor of a workgroup
(256), with spread positions and with half of the particles in one tile (one
key for whole chunks).

The records are checked through what is read from them: pm_density (positions
and segments) against pm_paint_q's integers, in every cell, bit for bit; then
two sorted steps (the second from canonical tags, ids and counts left by the
first) against unsorted ones: the ids are a permutation and each particle is
where its id says.  Both paths form the same integer density and differ in the
order of the readout's eight float32 products, some 1e-6 of a force; the
tolerance is 1e-5 of the largest change plus two roundings of the largest
value, and a misplaced record is off by the distance between two particles."""
import numpy as np
import pytest
import torch

from paper_2007_13394_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("clustered", [False, True])
@pytest.mark.parametrize("over", [dict(n_mesh=64, n_cdm=64, n_sites=1, n_shell=3, n_fib=1),     # P = 2^18 + 9
                                  dict(n_mesh=128, n_cdm=128, n_sites=1, n_shell=3, n_fib=1)])  # P = 2^21 + 9
def test_sorted_records(dev, over, clustered):
    from paper_2007_13394_amd import pm
    cfg = I.config("C5", **over)
    n = cfg["n_mesh"]
    x32, p32 = I.synthetic_state(cfg, seed=17)
    P = x32.shape[1]
    assert P % 256 != 0
    if clustered:
        rng = np.random.default_rng(18)
        x32[:, :P // 2] = (8 + 8 * rng.random((3, P // 2))).astype(np.float32)
    x, p = torch.from_numpy(x32).to(dev), torch.from_numpy(p32).to(dev)

    free = pm.Ctx(pm.make_config(cfg, flags=pm.PM_FLAG_NO_SORT))
    off, _, quanta = pm.pm_segments(free)
    q = torch.zeros(n ** 3, dtype=torch.int64, device=dev)
    for g in range(free.nseg):
        pm.pm_paint_q(free, x, int(off[g]), int(off[g + 1] - off[g]), int(quanta[g]), q)
    ref = (q.cpu().numpy().astype(np.float64) * 2.0 ** -cfg["shift"] - 1.0).astype(np.float32)
    delta = torch.empty(n ** 3, dtype=torch.float32, device=dev)
    pm.pm_density(free, x, delta)
    assert np.array_equal(delta.cpu().numpy(), ref)

    ctx = pm.Ctx(pm.make_config(cfg))
    ids = torch.arange(P, dtype=torch.int32, device=dev)
    pm.pm_attach_ids(ctx, ids)
    xs, ps = x.clone(), p.clone()
    for a in (0.5, 0.505):
        x0, p0 = x.clone(), p.clone()
        pm.pm_step(free, x, p, a, a - 0.0025, a + 0.0025, a + 0.005)
        pm.pm_step(ctx, xs, ps, a, a - 0.0025, a + 0.0025, a + 0.005)
        assert np.array_equal(np.sort(ids.cpu().numpy()), np.arange(P))
        k = ids.long()
        kick = float((p - p0).abs().max())
        assert float((ps - p[:, k]).abs().max()) <= 1e-5 * kick + 2 * float(p.abs().max()) * 2.0 ** -23
        d = (xs - x[:, k]).abs()
        d = torch.minimum(d, n - d)
        drift = abs(pm.pm_kdk_factors(ctx, a, a - 0.0025, a + 0.0025, a + 0.005)[1])
        move = float(p.abs().max()) * drift
        assert float(d.max()) <= 1e-5 * move + 2 * n * 2.0 ** -23
        # the same state for the next step, which then compares one step again
        x, p = torch.empty_like(xs), torch.empty_like(ps)
        x[:, k], p[:, k] = xs, ps

