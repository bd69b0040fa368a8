"""FP32 sums of tiles with few entries: a lane's register takes no more values than a
flush of the matrix-core kernel (124) before its sum goes to higher precision."""
import numpy as np
import pytest

import oracle
import synth
from gpu_helpers import host, make_plan, rel, say, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("support", [4, 5, 6, 7, 8])
@pytest.mark.parametrize("tile,n_row", [(8, 381), (16, 384), (32, 300), (32, 381)])
def test_small_values_after_a_large_one(tile, n_row, support):
    """One visibility of 1, then ones of 0.9 * 2^-25 at the same (u, v, w): an FP32 sum
    that holds the large value drops each of them.  Only those of the first run may be
    lost (124 of them, and one step of 2^-24 per later run), the rest adds up."""
    import torch
    n = 64
    prob = synth.tiny_problem(seed=370, nx=n, ny=n, n_row=n_row, freqs=(1.0e9,), cell_arcsec=30.0)
    prob.uvw[:] = 0.0
    # the middle of a tile: no neighbour's copies
    prob.uvw[:, :2] = (tile + tile // 2 + 0.3) / (2 * n * prob.cellx) * synth.C_LIGHT / prob.freq[0]
    prob.weight[:] = 1.0
    small = np.full((n_row, 1), 0.9 * 2.0 ** -25 * (1.0 + 1.0j))
    small[0] = 0.0
    large = np.zeros((n_row, 1), dtype=np.complex128)
    large[0] = 1.0 + 1.0j
    plan = make_plan(prob, "fp32", support=support, tile=tile)
    plan.profile(True)
    both, one = (host(plan.grid(to_dev(v, torch.complex64))).astype(np.float64) for v in (large + small, large))
    names = plan.profile_report()
    plan.profile(False)
    assert any("spread_cells" in k for k in names), names
    e = rel(both - one, oracle.grid(prob, small))
    say(f"small after large W={support} T={tile} n={n_row}: lost {e:.3f} of {n_row - 1} (one sum would lose all)")
    lost = 124.0 + 0.5 * 2.0 * (n_row // 124)      # values of 0.9 * 2^-25: a step of 2^-24 is about two
    assert e < lost / (n_row - 1) + 0.05           # and the FP32 transform's noise beside the large one
