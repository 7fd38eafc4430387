"""GPU parity of the density iterations on both sides of the line between the two
updates: in the interpolation, and (W <= 3 from 2^19 samples) a pass of its own.

Tolerances as for the whole transform: float64 1e-10 of a weight, float32 1e-4 (each
iteration divides by a product good to about 1e-6).
"""
import numpy as np
import pytest
import torch

import oracle as O

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("tile", [16, 32])
@pytest.mark.parametrize("dtype,tol", [("f32", 1e-4), ("f64", 1e-10)])
@pytest.mark.parametrize("W,m", [(2, (1 << 19) - 1), (2, 1 << 19), (3, (1 << 19) + 1), (4, 1 << 19)])
def test_line(W, m, dtype, tol, tile):
    from paper_1706_08575_amd.ftcg import Plan
    n = 128
    k = np.random.default_rng(W).uniform(-n / 2, n / 2, (m, 2))
    kd = torch.from_numpy(k).cuda()
    with Plan(n, dim=2, W=W, dtype=dtype, weights="density") as P:
        P.set_tuning(tile=tile)
        for iters in (1, 2):
            P.set_density_iterations(iters)
            P.set_points(kd)
            a = P.get_weights().cpu().numpy()
            ref = O.pipe_menon_weights(k, n, iters, W=W)
            assert np.max(np.abs(a - ref) / ref) < tol
