"""GPU parity of the square interpolation on both sides of its rule: records listed (more
than 256 squares, W > 3) or taken in binning order. Grids of 256 and of 1024 squares,
all half-widths on the larger one, chunks of 512 records and their edges, one slot
holding every record, samples down one column.

Tolerances as for the whole transforms: forward float32 2e-5, float64 1e-9 rel
L2 (the oracle takes the plan's 2W taps, so W does not enter); density weights
1e-10 relative in float64, 1e-4 in float32.
"""
import numpy as np
import pytest
import torch

import oracle as O

pytestmark = pytest.mark.gpu


def dev(a, dtype=None):
    t = torch.from_numpy(np.ascontiguousarray(a))
    return (t if dtype is None else t.to(dtype)).cuda()


def raster(kind, m, n, rng):
    if kind == "spot":       # every footprint on the same cell
        return rng.uniform(0.05, 0.2, size=(m, 2))
    if kind == "column":     # a pulse down one column of cells
        return np.stack([np.sort(rng.uniform(-n / 2, n / 2, m)), np.full(m, 0.3)], axis=1)
    return rng.uniform(-n / 2, n / 2, size=(m, 2))


def forward(n, k, img, dtype, W=6, tile=32):
    from paper_1706_08575_amd.ftcg import Plan
    cd = torch.complex64 if dtype == "f32" else torch.complex128
    with Plan(n, dim=2, W=W, dtype=dtype, weights="none") as P:
        P.set_tuning(tile=tile)
        P.set_points(dev(k))
        return P.forward(dev(img, cd)).cpu().numpy()


@pytest.mark.parametrize("tile", [16, 32])
@pytest.mark.parametrize("dtype,tol", [("f32", 2e-5), ("f64", 1e-9)])
@pytest.mark.parametrize("kind,m", [("spot", 1), ("spot", 33), ("spot", 511), ("spot", 513), ("spot", 1500),
                                    ("column", 3000), ("spread", 5000)])
def test_listed(kind, m, dtype, tol, tile):
    n = 512                                  # 32 x 32 squares
    rng = np.random.default_rng(m + tile)
    k = raster(kind, m, n, rng)
    img = rng.standard_normal((n, n)) + 1j * rng.standard_normal((n, n))
    assert O.rel_l2(forward(n, k, img, dtype, tile=tile), O.forward(k, img, n)) < tol


@pytest.mark.parametrize("dtype,tol", [("f32", 2e-5), ("f64", 1e-9)])
@pytest.mark.parametrize("W", [2, 3, 4, 5, 6, 7, 8])
@pytest.mark.parametrize("n,tile", [(256, 32), (512, 32), (512, 64), (1024, 64)])
def test_half_widths(n, tile, W, dtype, tol):
    rng = np.random.default_rng(W)
    k = np.concatenate([raster("spread", 2000, n, rng), raster("column", 600, n, rng)])
    img = rng.standard_normal((n, n)) + 1j * rng.standard_normal((n, n))
    assert O.rel_l2(forward(n, k, img, dtype, W, tile), O.forward(k, img, n, W=W)) < tol


@pytest.mark.parametrize("dtype,tol", [("f32", 1e-4), ("f64", 1e-10)])
@pytest.mark.parametrize("kind,m", [("spot", 700), ("spread", 3000)])
def test_density_listed(kind, m, dtype, tol):
    from paper_1706_08575_amd.ftcg import Plan
    n = 512
    k = raster(kind, m, n, np.random.default_rng(m))
    with Plan(n, dim=2, dtype=dtype, weights="density") as P:
        P.set_density_iterations(4)
        P.set_points(dev(k))
        a = P.get_weights().cpu().numpy()
    ref = O.pipe_menon_weights(k, n, 4)
    assert np.max(np.abs(a - ref) / ref) < tol
