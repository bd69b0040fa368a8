"""The interpolation's forms against the oracle: plane by plane with a block's entries in
registers (items of one to many entries, across base planes, gaps in w, tiles of 8 to 32
cells) and the plane ring, on either side of the density that divides them; FP64 flat."""
import numpy as np
import pytest

import oracle
import synth
from gpu_helpers import TOL, host, make_plan, rel, say, to_dev

pytestmark = pytest.mark.gpu


def _problem(n_row, nx=32, ny=48, w_frac=2.0, seed=350):
    prob = synth.tiny_problem(seed=seed, nx=nx, ny=ny, n_row=n_row, freqs=(1.0e9, 1.2e9), cell_arcsec=150.0,
                              w_frac=w_frac, flag_frac=0.1)
    return prob, np.random.default_rng(seed + 1).normal(size=(1, nx, ny))


def _check(plan, prob, x, prec, tol, flat=False):
    import torch
    R, C = (torch.float64, torch.complex128) if prec == "fp64" else (torch.float32, torch.complex64)
    model = oracle.degrid(prob, x, flat=flat)
    got = host(plan.degrid(to_dev(x, R)))
    start = to_dev(np.random.default_rng(9).normal(size=got.shape), C)
    added = host(plan.degrid_add(to_dev(x, R), start.clone()))
    on = prob.effective_weight() > 0
    e = dict(degrid=rel(got, model), add=rel((added - host(start))[on], model[on]),
             hess=rel(host(plan.hessian(to_dev(x, R))), oracle.hessian(prob, x, flat=flat)))
    assert np.all(got[~on] == 0)
    assert max(e.values()) < tol, e
    return e


@pytest.mark.parametrize("prec,support,tile,tol", [
    ("fp32", 4, 32, 5e-3), ("fp32", 7, 32, 1e-5), ("fp32", 8, 32, 1e-5), ("fp32", 7, 16, 1e-5), ("fp32", 7, 8, 1e-5),
    ("fp64", 9, 16, 1e-7), ("fp64", 13, 8, 1e-10), ("fp64", 16, 8, 1e-10)])
@pytest.mark.parametrize("n_row", [1, 33, 400, 9000])
def test_few_and_many_entries_per_tile(prec, support, tile, tol, n_row):
    prob, x = _problem(n_row)
    plan = make_plan(prob, prec, support=support, tile=tile)
    e = _check(plan, prob, x, prec, tol)
    say(f"interp {prec} W={support} T={tile} rows={n_row}: planes {plan.info()['n_wplanes_max']}, {e}")


@pytest.mark.parametrize("prec", ["fp32", "fp64"])
def test_items_across_w_gaps(prec):
    """Entries of one item many planes apart: planes between them are read past."""
    prob, x = _problem(60, w_frac=0.0)
    rng = np.random.default_rng(351)
    prob.uvw[:, 2] = rng.choice([0.0, 3.0e3, 9.0e3, -4.0e4], prob.n_row) + rng.uniform(0, 50.0, prob.n_row)
    plan = make_plan(prob, prec)
    e = _check(plan, prob, x, prec, TOL[prec])
    say(f"interp gaps {prec}: planes {plan.info()['n_wplanes_max']}, {e}")


@pytest.mark.parametrize("tile", [8, 32])
def test_fp64_flat(tile):
    prob, x = _problem(700, nx=64, ny=64, w_frac=0.0)
    _check(make_plan(prob, "fp64", flat=True, tile=tile), prob, x, "fp64", TOL["fp64"], flat=True)
