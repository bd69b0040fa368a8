"""The FP32 flat gridder's fixed-point step: faint visibilities beside a bright one.

The step is 2^-26 of the largest |w V|, taken at every flush of a window's sums.  Faint
visibilities of equal sign, one to a window, lose up to a step in each of their cells,
all towards zero, so the error of the faint image shows the step: 0.31 % of it for
values 1e-5 of the largest and a step of 2^-26 (W = 7, the truncation simulated in 64
bits), 1.17 % for 2^-24."""
import numpy as np
import pytest

import oracle
import synth
from gpu_helpers import host, make_plan, rel, say, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("tile", [16, 32])
def test_faint_visibilities_beside_a_bright_one(tile):
    import torch
    n, gap = 128, 16                                   # 256 x 256 cells, one visibility per 16 x 16
    k = np.arange(15)
    rng = np.random.default_rng(360)
    at = np.stack(np.meshgrid(8 + gap * k, 8 + gap * k, indexing="ij"), -1).reshape(-1, 2) - 120 + rng.uniform(size=(225, 2))
    prob = synth.tiny_problem(seed=361, nx=n, ny=n, n_row=225, freqs=(1.0e9,), cell_arcsec=30.0)
    prob.uvw[:, :2] = at / (2 * n * prob.cellx) * synth.C_LIGHT / prob.freq[0]
    prob.uvw[:, 2] = 0.0
    prob.weight[:] = 1.0
    bright = np.zeros((225, 1), dtype=np.complex128)
    bright[112] = 1.0
    faint = np.full((225, 1), 1e-5 + 0j)
    faint[112] = 0.0
    plan = make_plan(prob, "fp32", tile=tile, flat=True)
    both, one = (host(plan.grid(to_dev(v, torch.complex64))).astype(np.float64) for v in (bright + faint, bright))
    e = rel(both - one, oracle.grid(prob, faint, flat=True))
    say(f"flat T={tile}: faint image beside a bright visibility {e:.2e}")
    assert e < 6e-3        # twice the error of a 2^-26 step, half that of 2^-24


@pytest.mark.parametrize("n_row", [27, 28, 29, 57, 4000])
def test_long_runs_of_one_window(n_row):
    """All visibilities in one window, at the ends of its runs: sums near the fixed-point
    range (equal values of largest modulus at one position) keep their value."""
    import torch
    prob = synth.tiny_problem(seed=362, nx=64, ny=64, n_row=n_row, freqs=(1.0e9,), cell_arcsec=30.0)
    prob.uvw[:] = 0.0
    prob.uvw[:, :2] = 5.0 / (128 * prob.cellx) * synth.C_LIGHT / prob.freq[0]   # on a cell: its weight is 1
    prob.weight[:] = 1.0
    vis = np.full((n_row, 1), 1.0 - 1.0j)
    plan = make_plan(prob, "fp32", flat=True)
    assert rel(host(plan.grid(to_dev(vis, torch.complex64))), oracle.grid(prob, vis, flat=True)) < 1e-5


@pytest.mark.parametrize("tile", [8, 16])
@pytest.mark.parametrize("support", [4, 7, 8])
@pytest.mark.parametrize("n_row,chunk", [(5, 0), (3000, 0), (3000, 64), (60000, 0), (60000, 1 << 20)])
def test_small_tiles_of_four_waves(tile, support, n_row, chunk):
    """Flat tiles of 8 and 16 cells, sparse, dense and shared between items, every support
    class; a given chunk bounds the shares (the default's where it is larger: same bits)."""
    import torch
    prob = synth.tiny_problem(seed=363, nx=64, ny=96, n_row=n_row, freqs=(1.0e9, 1.2e9), cell_arcsec=30.0, w_frac=0.0,
                              flag_frac=0.1)
    rng = np.random.default_rng(364)
    prob.uvw[n_row // 4:, :2] *= 0.2
    vis = rng.normal(size=(n_row, 2)) + 1j * rng.normal(size=(n_row, 2))
    x = rng.normal(size=(1, 64, 96))
    plan = make_plan(prob, "fp32", tile=tile, support=support, flat=True, chunk=chunk)
    got = [host(plan.grid(to_dev(vis, torch.complex64))).copy() for _ in range(2)]
    pix = rng.choice(64 * 96, 50, replace=False)
    tol = {4: 5e-3, 7: 1e-5, 8: 1e-5}[support]
    assert rel(got[0].ravel()[pix], oracle.grid(prob, vis, pix=pix, flat=True)) < tol
    assert rel(host(plan.hessian(to_dev(x, torch.float32))).ravel()[pix], oracle.hessian(prob, x, pix=pix, flat=True)) < tol
    assert np.array_equal(got[0], got[1])
    if chunk == 1 << 20:
        default = make_plan(prob, "fp32", tile=tile, support=support, flat=True)
        assert np.array_equal(got[0], host(default.grid(to_dev(vis, torch.complex64))))
