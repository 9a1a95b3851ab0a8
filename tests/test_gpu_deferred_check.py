"""With deferred guards the host waits, within a sorted step, for the check of the
counts it took over and for nothing queued behind it: the check follows the
scatter, before the paint and the solve, and the readout comes last."""
import pytest
import torch

from paper_2007_13394_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("learned", [False, True])
def test_check_follows_the_scatter(dev, learned):
    from paper_2007_13394_amd import pm
    cfg = I.config("C1")
    ctx = pm.Ctx(pm.make_config(cfg, flags=pm.PM_FLAG_DEFER_GUARDS | (pm.PM_FLAG_LEARNED if learned else 0)))
    x32, p32 = I.synthetic_state(cfg, seed=92)
    x, p = torch.from_numpy(x32).to(dev), torch.from_numpy(p32).to(dev)
    call = (0.5, 0.4975, 0.5025, 0.505)
    theta = torch.zeros(pm.pm_net_nparam(), device=dev)
    step = (lambda: pm.pm_learned_step(ctx, theta, x, p, *call)) if learned else (lambda: pm.pm_step(ctx, x, p, *call))
    for _ in range(2):
        step()
    pm.pm_trace_begin(ctx)
    step()
    names = [k for k, _ in pm.pm_trace_end(ctx)]
    pm.pm_sync(ctx)
    assert names.count("sort_count") == 0 and names.count("paint") == names.count("sort_scatter") == 1, names
    at = [names.index(k) for k in ("sort_scan", "sort_scatter", "sort_verify", "paint")]
    assert at == list(range(4)) and names[-1] == "readout_kick_drift", names
