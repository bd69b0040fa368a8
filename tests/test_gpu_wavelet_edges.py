"""Wavelet levels with all bases in one launch: sides at and around the tiles
(16 x 32 coefficient positions), blocks smaller than a filter, one and many levels
and bases, rows that do and do not start on 16 bytes, one and several bands, against
the oracle; the dual projection over bands and the primal update included."""
import numpy as np
import pytest

import oracle
import synth
from oracle import wavelets
from gpu_helpers import TOL, host, make_plan, rel, say, to_dev

pytestmark = pytest.mark.gpu


def _plan(nx, ny, n_band, prec):
    prob = synth.tiny_problem(seed=320, nx=nx, ny=ny, n_row=300, freqs=np.linspace(1.0e9, 1.4e9, n_band),
                              cell_arcsec=20.0, n_band=n_band)
    return prob, make_plan(prob, prec)


@pytest.mark.parametrize("prec", ["fp32", "fp64"])
@pytest.mark.parametrize("nx,ny,n_band,nbasis,levels", [
    (16, 16, 1, 7, 4), (32, 64, 2, 7, 5), (34, 66, 1, 4, 1), (62, 130, 3, 7, 1), (64, 126, 2, 6, 1),
    (128, 72, 2, 7, 3), (96, 100, 1, 7, 2), (40, 264, 3, 5, 3), (64, 64, 2, 1, 2), (130, 34, 1, 2, 1)])
def test_analysis_synthesis_and_prox_at_tile_edges(nx, ny, n_band, nbasis, levels, prec):
    import torch
    R = torch.float64 if prec == "fp64" else torch.float32
    prob, plan = _plan(nx, ny, n_band, prec)
    rng = np.random.default_rng(321)
    x = rng.normal(size=(n_band, nx, ny))
    c = rng.normal(size=(nbasis, n_band, nx, ny))
    ws = plan.prox_workspace(nbasis)
    ana = host(plan.wavelet_analysis(to_dev(x, R), ws, nbasis, levels))
    syn = host(plan.wavelet_synthesis(to_dev(c, R), ws, nbasis, levels))
    e = dict(ana=rel(ana, wavelets.psi_adj(x, levels, nbasis)), syn=rel(syn, wavelets.psi(c, levels, nbasis)))
    # the primal-dual iteration, every band's dual and the iterate (the tolerances of the
    # package's prox test: five times the operators', ten times that for the dual)
    psf = oracle.psf(prob)
    conv = oracle.psf_conv_op(psf)
    plan.make_psf(want_image=False)
    z = rng.normal(size=(n_band, nx, ny)) * 0.05 + 0.02
    peak = float(psf.max())
    unorm, lam = 30.0 * peak, 2e-3 * peak
    xd = torch.zeros(n_band, nx, ny, dtype=R, device="cuda")
    plan.prox(to_dev(z, R), xd, ws, lam, 1.0, 0.1 * peak, unorm, 6, nbasis, levels)
    xr, vr = wavelets.prox_pd(conv, z, 0.1 * peak, 1.0, lam, unorm, levels, 6, nbasis)
    n = nbasis * n_band * nx * ny
    v = host(ws.view(R)[:n]).reshape(nbasis, n_band, nx, ny)
    ex, ev = rel(host(xd), xr), rel(v, vr)
    say(f"wavelets {nx}x{ny} bands {n_band} bases {nbasis} levels {levels} {prec}: {e} prox {ex:.1e} dual {ev:.1e}")
    assert max(e.values()) < TOL[prec], e
    assert ex < 5 * TOL[prec] and ev < 50 * TOL[prec]


def test_unaligned_images_match_aligned_ones():
    """Images that do not start on 16 bytes take the scalar accesses: the same bits."""
    import torch
    prob, plan = _plan(64, 72, 2, "fp32")
    plan.make_psf(want_image=False)
    ws = plan.prox_workspace(7)
    z = to_dev(np.random.default_rng(322).normal(size=(2, 64, 72)), torch.float32)
    room = torch.zeros(2 * (z.numel() + 4), device="cuda")
    off = lambda k: room[k * (z.numel() + 4) + 1:][: z.numel()].view(2, 64, 72)  # noqa: E731
    zo, xo, x = off(0), off(1), torch.zeros_like(z)
    zo.copy_(z)
    plan.prox(z, x, ws, 0.5, 1.0, 1.0, 1e4, 4, 7, 3)
    plan.prox(zo, xo, ws, 0.5, 1.0, 1.0, 1e4, 4, 7, 3)
    assert torch.equal(x, xo)
    c = plan.wavelet_analysis(z, ws, 7, 3)
    a = plan.wavelet_synthesis(c, ws, 7, 3)
    b = plan.wavelet_synthesis(c, ws, 7, 3, out=xo)
    assert torch.equal(a, b)
