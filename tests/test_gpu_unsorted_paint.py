"""Density of a context that keeps its particle order: painted by tile from
records sorted into the workspace where the mesh has at least two tiles per
side, with global atomics below.  The cells are integers either way, so
pm_density must equal (float)(Q 2^-shift - 1) of pm_paint_q's int64 mesh in
every cell, bit for bit: below and above the size where the sort takes more
rounds per thread, at meshes without tiles, and into a mesh that is not
aligned for 16-byte stores."""
import pytest
import torch

from paper_2007_13394_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("offset", [0, 1])
@pytest.mark.parametrize("name,over", [("C5_fd16", {}), ("C5_fd32", {}), ("C1", dict(n_shell=3, n_fib=1)),
                                       ("C5", dict(n_mesh=128, n_shell=7)),
                                       ("C1", dict(n_mesh=1024))])   # tiles in row-major order
def test_density_equals_atomic_paint(dev, name, over, offset):
    from paper_2007_13394_amd import pm
    cfg = I.config(name, **over)
    n = cfg["n_mesh"]
    ctx = pm.Ctx(pm.make_config(cfg, flags=pm.PM_FLAG_NO_SORT))
    off, _, quanta = pm.pm_segments(ctx)
    x32, _ = I.synthetic_state(cfg, seed=91)
    for g in range(ctx.nseg):   # tile faces in every segment
        k = int(off[g + 1] - off[g]) // 4
        if k:
            x32[:, off[g]:off[g] + k] = I.tile_face_positions(n, k, seed=92 + g)
    x = torch.from_numpy(x32).to(dev)
    q = torch.zeros(n ** 3, dtype=torch.int64, device=dev)
    for g in range(ctx.nseg):
        pm.pm_paint_q(ctx, x, int(off[g]), int(off[g + 1] - off[g]), int(quanta[g]), q)
    ref = (q.double() * 2.0 ** -cfg["shift"] - 1.0).float()
    delta = torch.full((n ** 3 + offset,), 7.0, dtype=torch.float32, device=dev)[offset:]
    pm.pm_density(ctx, x, delta)
    assert torch.equal(delta, ref)
