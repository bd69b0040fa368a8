"""The spread kernels at the edges of their forms, against the oracle: FP64 cells in
registers (tiles of one and of several 8 x 8 blocks, blocks of one and of four waves,
smallest and largest supports), FP32 flat windows on the matrix cores (PSF and flat
operators, tiles of 8 to 64 cells), short runs that touch few columns of a window."""
import numpy as np
import pytest

import oracle
import synth
from gpu_helpers import TOL, host, make_plan, rel, say, to_dev

pytestmark = pytest.mark.gpu


def _case(n_row, nx=32, ny=48, seed=340, w_frac=1.0, n_band=1):
    prob = synth.tiny_problem(seed=seed, nx=nx, ny=ny, n_row=n_row, freqs=(1.0e9, 1.2e9), cell_arcsec=150.0,
                              w_frac=w_frac, n_band=n_band, flag_frac=0.1)
    rng = np.random.default_rng(seed + 1)
    vis = rng.normal(size=(prob.n_row, 2)) + 1j * rng.normal(size=(prob.n_row, 2))
    return prob, vis, rng.normal(size=(n_band, nx, ny))


# supports reach their own accuracy: 9 is the FP64 path's coarsest (1e-8 class)
@pytest.mark.parametrize("support,tile,tol", [(9, 8, 1e-7), (9, 16, 1e-7), (13, 8, 1e-10), (16, 8, 1e-10)])
@pytest.mark.parametrize("n_row", [1, 3, 150, 6000])
def test_fp64_spread(support, tile, tol, n_row):
    import torch
    prob, vis, x = _case(n_row)
    plan = make_plan(prob, "fp64", support=support, tile=tile)
    g = [host(plan.grid(to_dev(vis, torch.complex128))).copy() for _ in range(2)]
    h = host(plan.hessian(to_dev(x, torch.float64)))
    e = rel(g[0], oracle.grid(prob, vis)), rel(h, oracle.hessian(prob, x))
    say(f"fp64 spread W={support} T={tile} rows={n_row}: entries {plan.info()['n_entries']}, {e}")
    assert max(e) < tol
    assert np.array_equal(g[0], g[1])         # fixed order of the sums


@pytest.mark.parametrize("prec", ["fp32", "fp64"])
@pytest.mark.parametrize("tile", [8, 16, 32, 64])
@pytest.mark.parametrize("n_row", [1, 40, 6000])
def test_flat_spread_and_psf(prec, tile, n_row):
    import torch
    R, C = (torch.float64, torch.complex128) if prec == "fp64" else (torch.float32, torch.complex64)
    prob, vis, x = _case(n_row, nx=64, ny=64, w_frac=0.0)
    # tiles whose w-stacked ring does not fit the LDS are refused without the flat option
    plan = make_plan(prob, prec, tile=tile, flat=True)
    e = dict(grid=rel(host(plan.grid(to_dev(vis, C))), oracle.grid(prob, vis, flat=True)),
             hess=rel(host(plan.hessian(to_dev(x, R))), oracle.hessian(prob, x, flat=True)),
             psf=rel(host(plan.make_psf()), oracle.psf(prob)))
    say(f"flat {prec} T={tile} rows={n_row}: {e}")
    assert max(e.values()) < TOL[prec]


@pytest.mark.parametrize("support,tol", [(4, 5e-3), (5, 1e-3), (6, 1e-4), (7, 1e-5), (8, 1e-5)])
def test_fp32_supports_flat_and_sparse(support, tol):
    """One to a few entries per window: flushes of runs that touch few columns."""
    import torch
    for n_row in (1, 2, 60):
        prob, vis, x = _case(n_row, nx=128, ny=64, seed=343)
        plan = make_plan(prob, "fp32", support=support)
        psf_ref = oracle.psf(prob)
        e = (rel(host(plan.grid(to_dev(vis, torch.complex64))), oracle.grid(prob, vis)),
             rel(host(plan.make_psf()), psf_ref))
        say(f"fp32 W={support} rows={n_row}: {e}")
        assert max(e) < tol
