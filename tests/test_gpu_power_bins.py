"""Binned powers of given meshes against float64 transforms and sums: below and
above the size (256^3) where the last axis pass is fused with the binning, auto
and cross, with and without the window, few, odd and many bins (the last ones
past the mesh's corner and empty).

Number of modes exactly.  Mean wavenumbers are float64 sums in another order:
1e-12.  A bin's power is a mean of products of float32 spectra, each within
about 1e-6 of the field's rms mode: 1e-5 of the white auto powers, which for the
cross power (its fields share half of their variance) is 2e-5 of the result."""
import math

import numpy as np
import pytest
import torch

from paper_2007_13394_amd import inputs as I

pytestmark = pytest.mark.gpu


def reference(da, db, nbins, compensate, box):
    n = da.shape[0]
    A = torch.fft.rfftn(da.double())
    B = A if db is da else torch.fft.rfftn(db.double())
    m = torch.fft.fftfreq(n, device=da.device, dtype=torch.float64) * n
    h = torch.arange(n // 2 + 1, device=da.device, dtype=torch.float64)
    nn = (m ** 2).view(n, 1, 1) + (m ** 2).view(1, n, 1) + (h ** 2).view(1, 1, -1)
    w = torch.full((n // 2 + 1,), 2.0, device=da.device, dtype=torch.float64)
    w[0] = w[-1] = 1.0
    p = (A * B.conj()).real * (box ** 3 / float(n) ** 6)
    if compensate:
        sinc = lambda k: torch.sinc(k / n) ** -4
        p = p * sinc(m).view(n, 1, 1) * sinc(m).view(1, n, 1) * sinc(h).view(1, 1, -1)
    k = nn.sqrt()
    b = k.floor().long()
    ok = (nn > 0) & (b < nbins)
    w = w.view(1, 1, -1).expand_as(nn)[ok]
    bins = b[ok].cpu().numpy()
    return [np.bincount(bins, weights=v.cpu().numpy(), minlength=nbins)
            for v in (w, w * k[ok] * (2 * math.pi / box), w * p[ok])]


@pytest.mark.parametrize("compensate", [False, True])
@pytest.mark.parametrize("n,nbins", [(32, 3), (32, 60), (64, 31), (128, 64), (256, 1), (256, 129), (256, 450), (512, 256)])
def test_power_of_meshes(dev, n, nbins, compensate):
    from paper_2007_13394_amd import pm
    cfg = I.config("C1", n_mesh=n, n_cdm=16, n_sites=2)
    ctx = pm.Ctx(pm.make_config(cfg))
    gen = torch.Generator(device=dev).manual_seed(n + nbins)
    da = torch.randn(n, n, n, device=dev, generator=gen)
    db = 0.5 ** 0.5 * (da + torch.randn(n, n, n, device=dev, generator=gen))
    auto = reference(da, da, nbins, compensate, cfg["box"])
    for second, tol in ((da, 1e-5), (db, 2e-5)):
        k, pk, nm = pm.pm_power_mesh(ctx, da, second, nbins, compensate=compensate)
        w, wk, wp = auto if second is da else reference(da, second, nbins, compensate, cfg["box"])
        assert np.array_equal(nm, w)
        some = w > 0
        assert np.allclose(k[some], wk[some] / w[some], rtol=1e-12, atol=0) and not k[~some].any()
        # against the typical power of the bin (its own auto power)
        assert np.abs(pk[some] - wp[some] / w[some]).max(initial=0) <= tol * (auto[2][some] / w[some]).max(initial=0)
        assert not pk[~some].any()
