"""Which form of a kernel a job takes, by what its results or the recorded kernel names show."""
import numpy as np
import pytest

import oracle
import synth
from gpu_helpers import TOL, host, make_plan, rel, say, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec,nx,ny,n_band", [("fp32", 62, 500, 9), ("fp32", 62, 508, 8), ("fp32", 32, 1020, 5),
                                               ("fp32", 128, 512, 8), ("fp64", 62, 500, 9), ("fp64", 34, 510, 8)])
def test_column_form_against_plane_form(prec, nx, ny, n_band):
    """One band at a time runs too few blocks for columns side by side and takes planes of
    one column; all bands in one launch do not.  The two add the planes in another order,
    so unequal bits show that two forms ran."""
    import torch
    R, C = (torch.float64, torch.complex128) if prec == "fp64" else (torch.float32, torch.complex64)
    prob = synth.tiny_problem(seed=400, nx=nx, ny=ny, n_row=300, freqs=np.linspace(1.0e9, 1.4e9, n_band),
                              cell_arcsec=60.0, w_frac=128.0 / max(nx, ny), n_band=n_band)
    rng = np.random.default_rng(401)
    vis = to_dev(rng.normal(size=(300, n_band)) + 1j * rng.normal(size=(300, n_band)), C)
    x = to_dev(rng.normal(size=(n_band, nx, ny)), R)
    one, every = make_plan(prob, prec, band_batch=1), make_plan(prob, prec, band_batch=n_band)
    a, b = one.grid(vis), every.grid(vis)
    e = rel(host(a), host(b)), rel(host(one.degrid(x)), host(every.degrid(x)))
    pix = rng.choice(n_band * nx * ny, 100, replace=False)
    r = (rel(host(b).ravel()[pix], oracle.grid(prob, host(vis), pix=pix)),
         rel(host(every.degrid(x)), oracle.degrid(prob, host(x))))
    say(f"column against plane form {nx}x{ny}x{n_band} {prec}: planes {every.info()['n_wplanes_max']}, {e}, oracle {r}")
    assert not torch.equal(a, b)
    assert max(e) < (1e-6 if prec == "fp32" else 1e-14)
    assert max(r) < TOL[prec]


@pytest.mark.parametrize("n_row,prec,kernel", [(300, "fp32", "interp_stream_kernel"), (60000, "fp32", "interp4_kernel"),
                                               (300, "fp64", "interp_stream_kernel"), (60000, "fp64", "interp_stream_kernel")])
def test_interpolation_form(n_row, prec, kernel):
    import torch
    prob = synth.tiny_problem(seed=402, nx=64, ny=64, n_row=n_row, freqs=(1.0e9,), cell_arcsec=150.0, w_frac=0.5)
    plan = make_plan(prob, prec)
    x = to_dev(np.random.default_rng(403).normal(size=(1, 64, 64)), torch.float64 if prec == "fp64" else torch.float32)
    plan.profile(True)
    plan.degrid(x)
    names = plan.profile_report()
    plan.profile(False)
    assert [k for k in names if k.startswith("interp")] == [kernel], names


@pytest.mark.parametrize("nx,ny,n_band,in_kernels", [(32, 32, 1, True), (64, 64, 1, True), (256, 256, 2, False),
                                                     (512, 512, 4, False)])
def test_cg_sums_by_launch_where_there_are_many_blocks(nx, ny, n_band, in_kernels):
    import torch
    prob = synth.tiny_problem(seed=406, nx=nx, ny=ny, n_row=300, freqs=np.linspace(1.0e9, 1.4e9, n_band), cell_arcsec=20.0,
                              n_band=n_band)
    plan = make_plan(prob)
    psf = host(plan.make_psf()).astype(np.float64)
    x = np.random.default_rng(407).normal(size=(n_band, nx, ny))
    conv = oracle.psf_conv_op(psf)
    sigma = 0.3 * float(np.abs(np.fft.rfft2(psf)).max())
    plan.profile(True)
    y = plan.precond_solve(to_dev(x, torch.float32), sigma, 5)
    names = plan.profile_report()
    plan.profile(False)
    assert names.get("reduce_kernel", (0, 0))[0] == (0 if in_kernels else 1 + 2 * 5)
    for b in range(n_band):
        want = oracle.cg(lambda v: conv.band(b, v) + sigma * v, x[b], 5)[0]
        assert rel(host(y)[b], want) < 10 * TOL["fp32"]
