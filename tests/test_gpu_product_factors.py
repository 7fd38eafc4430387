"""Factors of the float64 accumulation in float32 plans, matrix products (tile 32 and 64
from W = 5) and LDS atomics (else): they come from the sample's own cell outward, so the large taps carry the exponential's error at a
small argument, not at the footprint's edge (argument up to beta W^2 = 19, which alone
is 1.1e-6 of relative error).

Bound against the float64 oracle on the grid: a tap above 1 % of the peak is at most 4
cells out, four ratio steps from its exponential, under 10 roundings of 2^-24 over both
axes, the position's and the value's among them: 6e-7 relative L2.
"""
import numpy as np
import pytest
import torch

import oracle as O

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("W", [2, 3, 4, 5, 6, 7, 8])
@pytest.mark.parametrize("tile,copies", [(16, 1), (32, 1), (64, 1), (32, 2)])
@pytest.mark.parametrize("n", [64, 76])          # sigma = 2 and 1.68
def test_grid_error(W, tile, copies, n):
    from paper_1706_08575_amd.ftcg import Plan
    rng = np.random.default_rng(W + tile)
    m = 4000
    k = np.ascontiguousarray(rng.uniform(-0.5 * n, 0.5 * n, (m, 2)))
    f = (rng.standard_normal(m) + 1j * rng.standard_normal(m)).astype(np.complex64)
    with Plan(n, dim=2, W=W, sigma=128 / n, dtype="f32", weights="none") as P:
        P.set_tuning(tile, "f64", copies)
        P.set_points(torch.from_numpy(k).cuda())
        H = P.spread_only(torch.from_numpy(f).cuda()).cpu().numpy()
    err = O.rel_l2(H, O.spread(k, f.astype(np.complex128), n, 128 / n, W))
    print(f"W={W} tile={tile} copies={copies} n={n}: {err:.2e}")
    assert err < 6e-7
