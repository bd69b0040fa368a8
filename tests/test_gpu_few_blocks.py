"""Launch shapes of small problems: the w-plane column passes that take several planes
of one column per block, the convolution's one-wave column blocks and short row blocks,
and the CG's reductions inside the kernels that make the partial sums."""
import numpy as np
import pytest

import oracle
import synth
from gpu_helpers import TOL, host, make_plan, rel, say, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["fp32", "fp64"])
@pytest.mark.parametrize("nx,ny", [(64, 512), (62, 500), (16, 512), (256, 512), (2048, 64)])
def test_plane_and_column_forms_agree(nx, ny, prec):
    """One band at a time (planes of a column per block) against eight bands in one
    launch (columns per block; the same at 2048 x 64, whose columns stay few)."""
    import torch
    R, C = (torch.float64, torch.complex128) if prec == "fp64" else (torch.float32, torch.complex64)
    n_band = 8
    prob = synth.tiny_problem(seed=330, nx=nx, ny=ny, n_row=200, freqs=np.linspace(1.0e9, 1.4e9, n_band),
                              cell_arcsec=60.0, w_frac=2.0 * 64 / max(nx, ny), n_band=n_band)
    rng = np.random.default_rng(331)
    vis = to_dev(rng.normal(size=(prob.n_row, n_band)) + 1j * rng.normal(size=(prob.n_row, n_band)), C)
    x = to_dev(rng.normal(size=(n_band, nx, ny)), R)
    one, all_ = make_plan(prob, prec, band_batch=1), make_plan(prob, prec, band_batch=n_band)
    e = (rel(host(one.grid(vis)), host(all_.grid(vis))), rel(host(one.degrid(x)), host(all_.degrid(x))))
    pix = rng.choice(n_band * nx * ny, 200, replace=False)
    ref = oracle.grid(prob, host(vis), pix=pix)
    r = rel(host(one.grid(vis)).ravel()[pix], ref)
    say(f"column forms {nx}x{ny} {prec}: planes {one.info()['n_wplanes_max']}, {e}, oracle {r:.1e}")
    # the same transforms in another order of sums: rounding only
    assert max(e) < (1e-6 if prec == "fp32" else 1e-14)
    assert r < TOL[prec]


@pytest.mark.parametrize("prec", ["fp32", "fp64"])
@pytest.mark.parametrize("nx,ny,n_band", [(32, 32, 1), (64, 512, 1), (128, 126, 3), (512, 256, 1), (256, 1024, 2)])
def test_cg_with_reductions_in_the_kernels(nx, ny, n_band, prec):
    import torch
    R = torch.float64 if prec == "fp64" else torch.float32
    prob = synth.tiny_problem(seed=332, nx=nx, ny=ny, n_row=400, freqs=np.linspace(1.0e9, 1.4e9, n_band),
                              cell_arcsec=20.0, n_band=n_band)
    plan = make_plan(prob, prec)
    psf = host(plan.make_psf()).astype(np.float64)
    x = np.random.default_rng(333).normal(size=(n_band, nx, ny))
    conv = oracle.psf_conv_op(psf)
    sigma = 0.3 * float(np.abs(np.fft.rfft2(psf)).max())
    g = conv(x)
    assert rel(host(plan.psf_conv(to_dev(x, R))), g) < TOL[prec]
    resid = torch.zeros(n_band, dtype=torch.float64, device="cuda")
    got = [host(plan.precond_solve(to_dev(g, R), sigma, it, resid=resid)).copy() for it in (1, 8, 8)]
    for it, y in ((1, got[0]), (8, got[1])):
        want = np.stack([oracle.cg(lambda v, b=b: conv.band(b, v) + sigma * v, g[b], it)[0] for b in range(n_band)])
        assert rel(y, want) < 10 * TOL[prec]       # the package's CG tolerance
    assert np.array_equal(got[1], got[2])          # fixed order of the sums: the same bits
