"""GPU parity of the frame approximation at the edges of the blocked QR: column
counts around the panel width 16, row counts around the panel kernels' limits
(512, 1024, 2048 and 4096 rows; above that the column-by-column form), both the
least-squares and the minimum-norm solve, on 1D jittered rasters whose spacing
keeps Psi well conditioned.

Tolerance: both sides are backward-stable float64 least-squares solvers, which
agree to about the condition number of Psi (below 1e4 here) times the float64
rounding; 1e-8 rel L2, as for the whole-image tests.
"""
import numpy as np
import pytest
import torch

import oracle as O
from paper_1706_08575_amd import synth as S

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,m", [(8, 7), (8, 8), (16, 15), (16, 16), (16, 17), (16, 40), (64, 33), (64, 63),
                                 (64, 512), (64, 513), (64, 1024), (64, 1025), (32, 2048), (32, 2049), (16, 4096),
                                 (16, 4097), (512, 100), (1024, 17), (1024, 300)])
def test_frame_at_panel_edges(n, m):
    from paper_1706_08575_amd.ftcg import Plan
    rng = np.random.default_rng(1000 * n + m)
    step = n / m if m > n else 1.0                 # fewer samples than modes: a window of the raster
    k = ((np.arange(m) - m / 2 + rng.uniform(-0.25, 0.25, m)) * step).reshape(m, 1)
    f = S.random_values(n + m, m)
    with Plan(n, dim=1, dtype="f64", weights="none") as P:
        kd, fd = torch.from_numpy(k).cuda(), torch.from_numpy(f).cuda()
        img = P.frame_approx(kd, fd)
        assert torch.equal(img, P.frame_approx(kd, fd))     # kept tables, same bits
        img = img.cpu().numpy()
    err = O.rel_l2(img, O.frame_image(k, f, n))
    print(f"n={n} m={m}: rel L2 {err:.2e}")
    assert err < 1e-8


def test_frame_square_2d_largest_register_panel():
    # 2 x (2048 .. 4096] rows: 2D modes 64 x 64 = 4096 rows, few samples
    from paper_1706_08575_amd.ftcg import Plan
    k = S.noisy_grid(S.seed_for(5), 6)
    f = S.random_values(3, len(k))
    with Plan(64, dim=2, dtype="f64", weights="none") as P:
        img = P.frame_approx(torch.from_numpy(k).cuda(), torch.from_numpy(f).cuda()).cpu().numpy()
    assert O.rel_l2(img, O.frame_image(k, f, 64)) < 1e-8
