"""The two forms of the tile sort's passes on both sides of the lines between them
on a 64^3 mesh (512 keys): 2^18 particles, 512 per key, in canonical order, 640 per key
in sorted order; and at 128^3 (4096 keys) sorted ones between 128 and 640 per key on both sides
of 2^20, at 256^3 (32768 keys) fewer than 128.  The checks are those of
test_gpu_sort_sizes."""
import pytest
import torch

import test_gpu_sort_sizes as sizes
from paper_2007_13394_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("clustered", [False, True])
@pytest.mark.parametrize("over", [
    dict(n_mesh=64, n_cdm=32, n_sites=4, n_shell=49, n_fib=36),    # P = 2^18 - 448
    dict(n_mesh=64, n_cdm=64, n_sites=1, n_shell=3, n_fib=1),      # P = 2^18 + 9
    dict(n_mesh=64, n_cdm=64, n_sites=4, n_shell=33, n_fib=15),    # P = 640 x 512 - 64
    dict(n_mesh=64, n_cdm=64, n_sites=4, n_shell=41, n_fib=12),    # P = 640 x 512 + 64
    dict(n_mesh=128, n_cdm=64, n_sites=4, n_shell=63, n_fib=98),   # P = 2^20 + 7872
    dict(n_mesh=128, n_cdm=64, n_sites=4, n_shell=25, n_fib=245),  # P = 2^20 - 832
    dict(n_mesh=256, n_cdm=128, n_sites=1, n_shell=3, n_fib=1)])   # P = 2^21 + 9
def test_records_at_the_lines(dev, over, clustered):
    sizes.test_sorted_records(dev, over, clustered)


def test_fewer_particles_sort_no_slower(dev):
    """Count and scatter from canonical order: 549 k particles, 1072 per key,
    against 1.12 M (one form above 2^20 at any density took 157 us there, the other
    177 at half the particles; 68 us now)."""
    from paper_2007_13394_amd import pm
    us = []
    for shell in (10, 30):
        cfg = I.config("C1", n_cdm=64, n_sites=16, n_shell=shell)
        ctx = pm.Ctx(pm.make_config(cfg, flags=pm.PM_FLAG_NO_SORT))
        x32, _ = I.synthetic_state(cfg, seed=98)
        x = torch.from_numpy(x32).to(dev)
        acc = torch.empty_like(x)
        t = []
        for _ in range(4):
            pm.pm_trace_begin(ctx)
            pm.pm_force(ctx, x, acc)
            t.append(sum(ms for k, ms in pm.pm_trace_end(ctx) if k in ("sort_count", "sort_scatter")) * 1e3)
        us.append(min(t))
    assert us[0] < us[1], us
