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


@pytest.mark.parametrize("support", [4, 7, 8])
@pytest.mark.parametrize("tile", [16, 32])
@pytest.mark.parametrize("kind", ["centre", "corner", "edge"])
def test_dense_tiles_shared_between_items(kind, tile, support):
    """Most visibilities in one uv tile (its centre, a corner, across the periodic edge):
    several items share the tile's entries and their sums meet in a scratch tile.  A given
    chunk keeps one item per tile: the same sums but for where runs are cut."""
    import torch
    prob, vis, x = _case(3000, nx=64, ny=64, seed=345)
    rng = np.random.default_rng(346)
    lam = synth.C_LIGHT / prob.freq[0]
    at = {"centre": (48.0, 48.0), "corner": (32.0, 64.0), "edge": (0.0, 0.0)}[kind]
    spread = 6.0 if kind == "centre" else 3.0
    for k, (n, cell) in enumerate(((128, prob.cellx), (128, prob.celly))):
        prob.uvw[300:, k] = (at[k] + rng.normal(0, spread, prob.n_row - 300)) / (cell * n) * lam
    e = []
    for flat in (False, True):
        parts = make_plan(prob, "fp32", support=support, tile=tile, flat=flat)
        whole = make_plan(prob, "fp32", support=support, tile=tile, flat=flat, chunk=1 << 20)
        got = [host(p.grid(to_dev(vis, torch.complex64))).copy() for p in (parts, whole, parts)]
        hx = [host(p.hessian(to_dev(x, torch.float32))) for p in (parts, whole)]
        tol = {4: 5e-3, 7: 1e-5, 8: 1e-5}[support]
        e += [rel(got[0], oracle.grid(prob, vis, flat=flat)), rel(hx[0], oracle.hessian(prob, x, flat=flat))]
        # flush order differs (runs of a window end elsewhere): 2^-24 of the largest value each
        assert rel(got[0], got[1]) < 1e-6 and rel(hx[0], hx[1]) < 1e-6
        assert np.array_equal(got[0], got[2])
    say(f"shares {kind} W={support} T={tile}: {e}")
    assert max(e) < tol


@pytest.mark.parametrize("support", [4, 7, 8])
def test_w_planes_with_gaps_between_their_entries(support):
    """Entries in a few w clusters more than a support apart: planes without entries in
    reach lie between them, so ring slots are cleared, skipped and used again."""
    import torch
    prob, vis, x = _case(400, nx=64, ny=64, seed=345)
    rng = np.random.default_rng(346)
    step = 1.0 / (2.0 * 2.7e-4)                    # about one plane step at this field
    prob.uvw[:, 2] = (rng.choice([0, 9, 10, 21, 40], prob.n_row) + rng.uniform(0, 0.2, prob.n_row)) * step * 0.3
    plan = make_plan(prob, "fp32", support=support)
    tol = {4: 5e-3, 7: 1e-5, 8: 1e-5}[support]
    got = [host(plan.grid(to_dev(vis, torch.complex64))).copy() for _ in range(3)]
    e = rel(got[0], oracle.grid(prob, vis)), rel(host(plan.hessian(to_dev(x, torch.float32))), oracle.hessian(prob, x))
    say(f"w gaps W={support}: planes {plan.info()['n_wplanes_max']}, {e}")
    assert max(e) < tol
    assert np.array_equal(got[0], got[1]) and np.array_equal(got[0], got[2])


@pytest.mark.parametrize("support,tile", [(13, 8), (9, 16), (16, 8)])
def test_fp64_dense_tiles_shared_between_items(support, tile):
    import torch
    prob, vis, x = _case(6000, nx=64, ny=64, seed=347)
    prob.uvw[:, :2] *= 0.15                        # a handful of tiles around the centre
    tol = 1e-7 if support == 9 else 1e-10
    for flat in (False, True):
        plan = make_plan(prob, "fp64", support=support, tile=tile, flat=flat)
        got = [host(plan.grid(to_dev(vis, torch.complex128))).copy() for _ in range(3)]
        one = host(make_plan(prob, "fp64", support=support, tile=tile, flat=flat, chunk=1 << 20)
                   .grid(to_dev(vis, torch.complex128)))
        assert rel(got[0], oracle.grid(prob, vis, flat=flat)) < tol
        assert rel(got[0], one) < 1e-13
        assert np.array_equal(got[0], got[1]) and np.array_equal(got[0], got[2])
        assert rel(host(plan.hessian(to_dev(x, torch.float64))), oracle.hessian(prob, x, flat=flat)) < tol
    psf = host(plan.make_psf())
    assert rel(psf, oracle.psf(prob)) < tol


def test_shared_tiles_with_bands_in_batches():
    """Shared tiles of several bands, all at once and one band at a time; replays of a
    captured graph of the gridding give the eager result (the scratch is zero again)."""
    import torch
    prob = synth.tiny_problem(seed=348, nx=64, ny=64, n_row=5000, freqs=(1.0e9, 1.1e9, 1.2e9), cell_arcsec=60.0,
                              n_band=3, w_frac=1.0)
    prob.uvw[:, :2] *= 0.3
    vis = to_dev(np.random.default_rng(349).normal(size=(5000, 3)) + 0.5j, torch.complex64)
    one, every = make_plan(prob, band_batch=1), make_plan(prob)
    a, b = one.grid(vis), every.grid(vis)
    assert torch.equal(a, b)
    assert rel(host(a), oracle.grid(prob, host(vis))) < TOL["fp32"]
    out = torch.empty_like(a)
    stream = torch.cuda.Stream()
    stream.wait_stream(torch.cuda.current_stream())
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=stream):
        every.grid(vis, out=out)
    for _ in range(3):
        out.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, a)
        every.grid(vis)
        torch.cuda.synchronize()


@pytest.mark.parametrize("support,tile,tol", [(4, 32, 5e-3), (7, 32, 1e-5), (8, 32, 1e-5), (7, 16, 1e-5), (7, 8, 1e-5)])
@pytest.mark.parametrize("n_row", [3000, 40000])
def test_fp32_tiles_of_few_entries(support, tile, tol, n_row):
    """Many tiles of few entries (lanes own cells), some of them denser than that kernel
    takes (n_row = 40000); w of several planes with gaps."""
    import torch
    prob = synth.tiny_problem(seed=350, nx=512, ny=400, n_row=n_row, freqs=(1.3e9,), cell_arcsec=60.0, w_frac=0.3,
                              flag_frac=0.1)
    rng = np.random.default_rng(351)
    prob.uvw[n_row // 2:, :2] *= 0.2               # half of them in a few tiles
    prob.uvw[: n_row // 3, 2] += 4.0 * np.abs(prob.uvw[:, 2]).max()
    vis = rng.normal(size=(n_row, 1)) + 1j * rng.normal(size=(n_row, 1))
    plan = make_plan(prob, "fp32", support=support, tile=tile)
    got = [host(plan.grid(to_dev(vis, torch.complex64))).copy() for _ in range(2)]
    pix = rng.choice(512 * 400, 60, replace=False)
    x = np.zeros((1, 512, 400))
    x[0, rng.integers(0, 512, 50), rng.integers(0, 400, 50)] = rng.uniform(0.1, 1.0, 50)
    pix_h = np.concatenate([np.flatnonzero(x), pix])
    h = host(plan.hessian(to_dev(x, torch.float32)))
    e = rel(got[0].ravel()[pix], oracle.grid(prob, vis, pix=pix)), rel(h.ravel()[pix_h], oracle.hessian(prob, x, pix=pix_h))
    say(f"cells W={support} T={tile} rows={n_row}: planes {plan.info()['n_wplanes_max']}, {e}")
    assert max(e) < tol
    assert np.array_equal(got[0], got[1])


def test_fp32_tiles_of_few_entries_extreme_scales():
    """The scaled sums keep the range that the fixed-point kernel has; a NaN or infinite
    visibility is loud in every pixel."""
    import torch
    prob = synth.tiny_problem(seed=352, nx=512, ny=512, n_row=3000, freqs=(1.3e9,), cell_arcsec=60.0)
    rng = np.random.default_rng(353)
    vis = rng.normal(size=(3000, 1)) + 1j * rng.normal(size=(3000, 1))
    plan = make_plan(prob, "fp32")
    ref = host(plan.grid(to_dev(vis, torch.complex64))).astype(np.float64)
    for scale in (1e-20, 1e18):
        assert rel(host(plan.grid(to_dev(vis * scale, torch.complex64))).astype(np.float64) / scale, ref) < 1e-6
    for bad in (np.nan, np.inf):
        vis2 = vis.copy()
        vis2[7] = bad
        assert np.isnan(host(plan.grid(to_dev(vis2, torch.complex64)))).all()
    assert np.all(host(plan.grid(to_dev(0 * vis, torch.complex64))) == 0)
