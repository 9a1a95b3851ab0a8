"""A weak bin next to a strong one keeps its own precision.  The field 2^20 (1, 0,
-1, 0) + (1, -1, 1, -1) along the last axis is exact in float32, and so is every sum
of its transform but for the half-turn's cosine in float32 (6e-17 of a part): two
modes, N/4 and N/2, whose powers differ by 2^38, in neighbouring bins of one
wavefront; all others are zero.  A sum over the strong mode would cost the weak one
2^-53 x 2^38 = 3e-5; the bins are sums of few products in float64: 1e-12."""
import numpy as np
import pytest
import torch

from paper_2007_13394_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [32, 64])
@pytest.mark.parametrize("axis", [0, 1, 2])
def test_weak_bin(dev, n, axis):
    from paper_2007_13394_amd import pm
    cfg = I.config("C1", n_mesh=n, n_cdm=16, n_sites=2)
    ctx = pm.Ctx(pm.make_config(cfg))
    strong, weak = 2.0 ** 20 * np.array([1, 0, -1, 0]), np.array([1, -1, 1, -1])
    line = torch.from_numpy(np.tile(strong + weak, n // 4).astype(np.float32)).to(dev)
    shape = [1, 1, 1]
    shape[axis] = n
    d = line.view(shape).expand(n, n, n).contiguous()
    _, pk, nm = pm.pm_power_mesh(ctx, d, d, n // 2 + 1)
    norm = cfg["box"] ** 3 / float(n) ** 6
    m3 = float(n) ** 3
    # cos: two modes of half the amplitude; the alternating field one of the whole
    total = {n // 4: 2 * (2.0 ** 20 * m3 / 2) ** 2 * norm, n // 2: m3 ** 2 * norm}
    for b in range(1, n // 2 + 1):
        want = total.get(b, 0.0)
        assert abs(pk[b] * nm[b] - want) <= 1e-12 * want, (b, pk[b] * nm[b], want)
