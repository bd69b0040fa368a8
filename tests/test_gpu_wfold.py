"""Folding of the w axis: where it saves planes, visibilities with w < 0 are listed
at -(u, v, w) with conjugated values (the image is real).  Every operator that reads
or writes visibilities is checked against the oracle for w of both signs (folded),
of one sign (not folded) and within one plane step (nothing to save)."""
import numpy as np
import pytest

import oracle
import synth
from gpu_helpers import TOL, host, make_plan, rel, say, to_dev

pytestmark = pytest.mark.gpu


def _problem(kind, seed):
    prob = synth.tiny_problem(seed=seed, nx=64, ny=48, n_row=500, freqs=(1.0e9, 1.1e9, 1.3e9, 1.4e9),
                              cell_arcsec=120.0, w_frac=3.0, n_band=2, flag_frac=0.15)
    if kind == "positive":
        prob.uvw[:, 2] = np.abs(prob.uvw[:, 2]) + 1.0
    elif kind == "negative":
        prob.uvw[:, 2] = -np.abs(prob.uvw[:, 2]) - 1.0
    elif kind == "narrow":
        prob.uvw[:, 2] *= 1e-4
    elif kind == "zeros":                       # exact zeros of either sign among both signs
        prob.uvw[::3, 2] = 0.0
        prob.uvw[1::3, 2] *= -1.0
        prob.uvw[0, 2] = -0.0
    return prob


@pytest.mark.parametrize("prec", ["fp32", "fp64"])
@pytest.mark.parametrize("kind", ["both", "positive", "negative", "narrow", "zeros"])
def test_folded_operators_match_the_oracle(kind, prec):
    import torch
    R, C = (torch.float64, torch.complex128) if prec == "fp64" else (torch.float32, torch.complex64)
    prob = _problem(kind, 310)
    rng = np.random.default_rng(311)
    vis = rng.normal(size=(prob.n_row, prob.n_chan)) + 1j * rng.normal(size=(prob.n_row, prob.n_chan))
    x = rng.normal(size=(2, prob.nx, prob.ny))
    plan = make_plan(prob, prec)
    model = oracle.degrid(prob, x)
    start = to_dev(vis, C)
    added = host(plan.degrid_add(to_dev(x, R), start.clone()))
    on = prob.effective_weight() > 0
    errs = dict(dirty=rel(host(plan.grid(to_dev(vis, C))), oracle.grid(prob, vis)),
                degrid=rel(host(plan.degrid(to_dev(x, R))), model),
                add=rel((added - host(start))[on], model[on]),
                hessian=rel(host(plan.hessian(to_dev(x, R))), oracle.hessian(prob, x)))
    say(f"w fold {kind} {prec}: {plan.info()['n_wplanes_max']} planes, {errs}")
    assert max(errs.values()) < TOL[prec], errs
    assert np.array_equal(added[~on], host(start)[~on])


def test_planes_span_the_absolute_range_only():
    both, one = _problem("both", 310), _problem("positive", 310)
    nb, n1 = make_plan(both).info()["n_wplanes_max"], make_plan(one).info()["n_wplanes_max"]
    # the same |w| (up to the 1 m shift): the same planes, where the signed range would take
    # nearly twice the steps
    assert abs(nb - n1) <= 1


def test_facets_with_w_of_both_signs():
    from paper_2101_08072_amd.facets import FacetedPlan
    import torch
    prob = synth.tiny_problem(seed=312, nx=128, ny=128, n_row=400, freqs=(1.3e9,), cell_arcsec=60.0, w_frac=3.0)
    rng = np.random.default_rng(313)
    vis = rng.normal(size=(prob.n_row, 1)) + 1j * rng.normal(size=(prob.n_row, 1))
    x = np.zeros((1, 128, 128))
    x[0, rng.integers(0, 128, 40), rng.integers(0, 128, 40)] = rng.uniform(0.1, 1.0, 40)
    fp = FacetedPlan.from_problem(prob, 2, 2)
    assert rel(host(fp.grid(to_dev(vis, torch.complex64))), oracle.grid(prob, vis)) < TOL["fp32"]
    assert rel(host(fp.degrid(to_dev(x, torch.float32))), oracle.degrid(prob, x)) < TOL["fp32"]
