"""Force meshes at the sizes whose last passes go through the mesh in plane
groups (512^3 in two, 1024^3 in sixteen), every component against float64
transforms.  Float32 transforms of three axes, about 1e-6 of the rms: bound
1e-5, the one of the smaller meshes; a group that was left out, taken twice or
mixed up is off by its share of the rms, at least 1/16."""
import math

import pytest
import torch

from paper_2007_13394_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [512, 1024])
def test_force_mesh_groups(dev, n):
    from paper_2007_13394_amd import pm
    cfg = I.config("C1", n_mesh=n, n_cdm=32, n_sites=8)
    ctx = pm.Ctx(pm.make_config(cfg))
    gen = torch.Generator(device=dev).manual_seed(n)
    delta = 0.5 * torch.randn(n, n, n, device=dev, generator=gen).double()
    q = torch.round((1.0 + delta).clamp_(min=0.0) * 2.0 ** 40).to(torch.int64)
    out = torch.empty(3 * n ** 3, dtype=torch.float32, device=dev)
    pm.pm_force_mesh(ctx, q.view(-1), out)
    got = out.view(3, n, n, n)
    spec = torch.fft.rfftn(q.double() * 2.0 ** -40 - 1.0)
    del q, delta
    full = torch.fft.fftfreq(n, device=dev, dtype=torch.float64) * 2 * math.pi
    half = torch.fft.rfftfreq(n, device=dev, dtype=torch.float64) * 2 * math.pi
    k = [full.view(n, 1, 1), full.view(1, n, 1), half.view(1, 1, -1)]
    k2 = k[0] ** 2 + k[1] ** 2 + k[2] ** 2
    k2[0, 0, 0] = 1.0
    spec = spec / k2 * (1.5 * cfg["omega_m"])
    spec[0, 0, 0] = 0.0
    for d in range(3):
        kd = k[d].clone()
        kd.view(-1)[n // 2] = 0.0   # no gradient at the Nyquist wavenumber
        ref = torch.fft.irfftn(spec * kd * 1j, s=(n, n, n))
        err = float((got[d] - ref).norm() / ref.norm())
        assert err < 1e-5, (d, err)
