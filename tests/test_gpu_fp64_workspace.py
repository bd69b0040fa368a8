"""The FP64 plan's workspace holds the entries, the planes, the convolution's buffers and
the plan-time sort's scratch, and nothing besides for the shares of dense tiles, whose
scratch tiles lie in areas that are idle during the spread."""
import numpy as np
import pytest

import oracle
import synth
from gpu_helpers import TOL, host, make_plan, rel, say, to_dev

pytestmark = pytest.mark.gpu


def _parts(plan, prob):
    """Bytes of the areas that the operators need, from the plan's description."""
    i = plan.info()
    e, q = i["n_entries"], i["n_psf_entries"]
    px, nb, bb = prob.nx * prob.ny, prob.n_band, i["band_batch"]
    record, sort = 32 + 8 + 4 + 4, 32 + 8 + 3 * (8 + 4)        # (keys and positions: in, out, the radix sort's own)
    planes = bb * max(i["n_wplanes_max"] * i["grid_x"] * i["grid_y"], i["psf_grid_x"] * i["psf_grid_y"]) * 16
    half = bb * max(i["n_wplanes_max"] * i["grid_x"] * (prob.ny + 8), i["psf_grid_x"] * (2 * prob.ny + 8)) * 16
    keys = (i["grid_x"] // i["tile"]) * (i["grid_y"] // i["tile"]) * i["n_wplanes_max"] * nb
    conv = nb * i["grid_x"] * (i["grid_y"] // 2 + 16) * (16 + 8)
    return ((e + q) * record + max(planes + half, max(e, q) * sort) + conv + nb * px * (6 + 4 + 1) * 8 +
            prob.n_row * prob.n_chan * 20 + (keys + 4 * nb * px) * 64)


@pytest.mark.parametrize("nx,tile,flat,cell,n_band,batch", [
    (512, 64, True, 20.0, 1, 0), (512, 8, False, 80.0, 1, 0), (128, 8, False, 400.0, 1, 0), (64, 32, True, 20.0, 1, 0),
    (128, 16, False, 300.0, 4, 1)])
def test_dense_tiles_take_no_workspace(nx, tile, flat, cell, n_band, batch):
    import torch
    n_row = 160000 // n_band
    prob = synth.tiny_problem(seed=390, nx=nx, ny=nx, n_row=n_row, freqs=np.linspace(1.0e9, 1.2e9, 2 * n_band),
                              cell_arcsec=cell, n_band=n_band, w_frac=0.0 if flat else 0.3)
    prob.uvw[:, :2] *= np.random.default_rng(391).uniform(0.0, 1.0, (n_row, 1)) ** 2      # crowded centre
    plan = make_plan(prob, "fp64", support=9 if tile == 16 else 0, tile=tile, flat=flat, band_batch=batch)
    ws, parts = plan.info()["workspace_bytes"], _parts(plan, prob)
    say(f"fp64 workspace {nx}^2 T={tile} flat={flat} planes {plan.info()['n_wplanes_max']}: {ws / 2**20:.1f} MiB, parts {parts / 2**20:.1f}")
    assert ws < 1.1 * parts
    # and the shares in those areas give the right image, call after call
    vis = np.random.default_rng(392).normal(size=(n_row, 2 * n_band)) + 0.3j
    got = [host(plan.grid(to_dev(vis, torch.complex128))).copy() for _ in range(2)]
    pix = np.random.default_rng(393).choice(n_band * nx * nx, 24, replace=False)
    assert rel(got[0].ravel()[pix], oracle.grid(prob, vis, pix=pix, flat=flat)) < (1e-7 if tile == 16 else TOL["fp64"])
    assert np.array_equal(got[0], got[1])
    x = np.zeros((n_band, nx, nx))
    x[:, nx // 3, nx // 2] = 1.0
    h = [host(plan.hessian(to_dev(x, torch.float64))).copy() for _ in range(2)]
    assert rel(h[0].ravel()[pix], oracle.hessian(prob, x, pix=pix, flat=flat)) < (1e-7 if tile == 16 else TOL["fp64"])
    assert np.array_equal(h[0], h[1])
