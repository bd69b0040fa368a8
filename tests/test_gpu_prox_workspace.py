"""The prox workspace: the dual variable and six images, no more, and none of it read
before it is written."""
import numpy as np
import pytest

import synth
from gpu_helpers import host, make_plan, rel, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx,ny,n_band,nbasis,levels", [(64, 48, 2, 7, 4), (16, 32, 1, 2, 3), (96, 64, 3, 7, 5)])
def test_prox_workspace_holds_the_dual_and_six_images(nx, ny, n_band, nbasis, levels):
    """Guard words behind the workspace stay, and nothing of it is read before it is written."""
    import torch
    prob = synth.tiny_problem(seed=404, nx=nx, ny=ny, n_row=200, freqs=np.linspace(1.0e9, 1.4e9, n_band), cell_arcsec=20.0,
                              n_band=n_band)
    plan = make_plan(prob)
    plan.make_psf(want_image=False)
    img = n_band * nx * ny * 4
    need = plan.prox_workspace(nbasis).numel()
    assert need == (nbasis + 6) * img
    room = torch.full((need + 4096,), 0xFF, dtype=torch.uint8, device="cuda")       # NaN wherever read as float
    ws = room[:need]
    z = to_dev(np.random.default_rng(405).normal(size=(n_band, nx, ny)), torch.float32)
    x = plan.prox(z, torch.zeros_like(z), ws, 0.5, 1.0, 1.0, 1e4, 4, nbasis, levels)
    assert torch.isfinite(x).all() and bool((room[need:] == 0xFF).all())
    zeroed = torch.zeros(need, dtype=torch.uint8, device="cuda")
    assert torch.equal(x, plan.prox(z, torch.zeros_like(z), zeroed, 0.5, 1.0, 1.0, 1e4, 4, nbasis, levels))
    c = plan.wavelet_analysis(z, ws, nbasis, levels)
    back = plan.wavelet_synthesis(c, ws, nbasis, levels)
    assert rel(host(back), host(z)) < 1e-5 and bool((room[need:] == 0xFF).all())
