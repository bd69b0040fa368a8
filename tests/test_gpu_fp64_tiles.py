"""FP64 spread of tiles larger than 8 x 8, one wave for each 8 x 8 block of an item's tile:
batches that miss a block are skipped, dense tiles shared, their shares summed in four runs
(fewer shares than runs, and many), against the oracle and bit for bit between calls."""
import numpy as np
import pytest

import oracle
import synth
from gpu_helpers import host, make_plan, rel, say, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("tile,flat,support", [(16, False, 9), (16, True, 13), (32, True, 13), (64, True, 13), (32, True, 16),
                                               (8, False, 13), (8, True, 9)])
@pytest.mark.parametrize("n_row,dense", [(1, False), (130, False), (700, True), (30000, True)])
def test_blocks_of_a_tile(tile, flat, support, n_row, dense):
    import torch
    prob = synth.tiny_problem(seed=380, nx=64, ny=96, n_row=n_row, freqs=(1.0e9, 1.2e9), cell_arcsec=150.0,
                              w_frac=0.0 if flat else 0.5, flag_frac=0.1 if n_row > 1 else 0.0)
    rng = np.random.default_rng(381)
    if dense:
        prob.uvw[n_row // 8:, :2] *= 0.1                # most of them in the tiles round the centre
    vis = rng.normal(size=(n_row, 2)) + 1j * rng.normal(size=(n_row, 2))
    x = rng.normal(size=(1, 64, 96))
    plan = make_plan(prob, "fp64", tile=tile, flat=flat, support=support)
    got = [host(plan.grid(to_dev(vis, torch.complex128))).copy() for _ in range(2)]
    pix = rng.choice(64 * 96, 100, replace=False)
    e = (rel(got[0].ravel()[pix], oracle.grid(prob, vis, pix=pix, flat=flat)),
         rel(host(plan.hessian(to_dev(x, torch.float64))).ravel()[pix], oracle.hessian(prob, x, pix=pix, flat=flat)))
    say(f"fp64 T={tile} W={support} flat={flat} rows={n_row}: {e}")
    assert max(e) < (1e-7 if support == 9 else 1e-10)
    assert np.array_equal(got[0], got[1])
    if flat:
        assert rel(host(plan.make_psf()), oracle.psf(prob)) < (1e-7 if support == 9 else 1e-10)


def test_large_tiles_keep_up_with_small_ones():
    """3.2e5 visibilities at 128^2: tiles of 64 cells against tiles of 8.  The blocks of a
    tile run side by side and its shares are summed by many threads, so the larger tiles
    take a few times as long (more entries are read past), not 35 times as when one wave
    went through a tile's 64 blocks."""
    import torch
    prob = synth.tiny_problem(seed=382, nx=128, ny=128, n_row=160000, freqs=(1.0e9, 1.2e9), cell_arcsec=20.0, w_frac=0.0)
    prob.uvw[:, :2] *= 0.3
    vis = torch.randn(160000, 2, dtype=torch.complex128, device="cuda")
    ms = {}
    for tile in (8, 64):
        plan = make_plan(prob, "fp64", tile=tile, flat=True)
        plan.grid(vis)
        t = []
        for _ in range(5):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            plan.grid(vis)
            b.record()
            torch.cuda.synchronize()
            t.append(a.elapsed_time(b))
        ms[tile] = min(t)
    say(f"flat FP64 dirty image, tiles of 8 and 64: {ms}")
    assert ms[64] < 8 * ms[8]


@pytest.mark.parametrize("flat", [False, True])
def test_a_given_chunk_keeps_dense_tiles_shared(flat):
    """chunk bounds the entries of an item: a large one leaves the default's shares (the
    same bits), a small one makes more of them."""
    import torch
    prob = synth.tiny_problem(seed=383, nx=64, ny=64, n_row=20000, freqs=(1.0e9, 1.2e9), cell_arcsec=150.0,
                              w_frac=0.0 if flat else 0.3)
    prob.uvw[:, :2] *= 0.15
    rng = np.random.default_rng(384)
    vis = to_dev(rng.normal(size=(20000, 2)) + 0.5j, torch.complex128)
    got = {c: host(make_plan(prob, "fp64", flat=flat, chunk=c).grid(vis)).copy() for c in (0, 64, 300, 1 << 20)}
    pix = rng.choice(64 * 64, 64, replace=False)
    ref = oracle.grid(prob, host(vis), pix=pix, flat=flat)
    for c, g in got.items():
        assert rel(g.ravel()[pix], ref) < 1e-10, c
    assert np.array_equal(got[0], got[1 << 20])
