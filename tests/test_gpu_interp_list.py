"""GPU parity of the interpolation's record lists (forward transform, density
iterations) where they can go wrong: chunks of 512 records and their edges, one
LDS bank slot holding every record (more than the 32 listed rounds), all tile
sizes of the square kernel, both precisions, grids of the smallest size.

Tolerances as for the whole transforms: forward float32 2e-5, float64 1e-9 rel
L2; density weights 1e-10 relative in float64, 1e-4 in float32 (each iteration
divides by a product good to about 1e-6).
"""
import numpy as np
import pytest
import torch

import oracle as O
from paper_1706_08575_amd import synth as S

pytestmark = pytest.mark.gpu


def dev(a, dtype=None):
    t = torch.from_numpy(np.ascontiguousarray(a))
    return (t if dtype is None else t.to(dtype)).cuda()


def raster(kind, m, n, rng):
    if kind == "spot":       # every footprint on the same cell: one slot
        return rng.uniform(0.05, 0.2, size=(m, 2))
    if kind == "column":     # 43 cells apart on the window's rows: few slots
        return np.stack([rng.integers(-n // 2, n // 2, m) + 0.1, np.full(m, 0.3)], axis=1)
    return rng.uniform(-n / 2, n / 2, size=(m, 2))


@pytest.mark.parametrize("tile", [16, 32, 64])
@pytest.mark.parametrize("dtype,tol", [("f32", 2e-5), ("f64", 1e-9)])
@pytest.mark.parametrize("kind,m", [("spot", 1), ("spot", 33), ("spot", 511), ("spot", 513), ("spot", 1500),
                                    ("column", 700), ("spread", 5000)])
def test_forward_lists(kind, m, dtype, tol, tile):
    from paper_1706_08575_amd.ftcg import Plan
    n = 64
    rng = np.random.default_rng(m + tile)
    k = raster(kind, m, n, rng)
    img = rng.standard_normal((n, n)) + 1j * rng.standard_normal((n, n))
    cd = torch.complex64 if dtype == "f32" else torch.complex128
    with Plan(n, dim=2, dtype=dtype, weights="none") as P:
        P.set_tuning(tile=tile)
        P.set_points(dev(k))
        out = P.forward(dev(img, cd)).cpu().numpy()
    assert O.rel_l2(out, O.forward(k, img, len(img))) < tol


@pytest.mark.parametrize("tile", [16, 32, 64])
@pytest.mark.parametrize("dtype,tol", [("f32", 1e-4), ("f64", 1e-10)])
@pytest.mark.parametrize("kind,m", [("spot", 40), ("spot", 700), ("spread", 3000)])
def test_density_lists(kind, m, dtype, tol, tile):
    from paper_1706_08575_amd.ftcg import Plan
    n = 64
    rng = np.random.default_rng(m + tile + 1)
    k = raster(kind, m, n, rng)
    with Plan(n, dim=2, dtype=dtype, weights="density") as P:
        P.set_tuning(tile=tile)
        P.set_density_iterations(4)
        P.set_points(dev(k))
        a = P.get_weights().cpu().numpy()
        P.set_points(dev(k))
        assert np.array_equal(a, P.get_weights().cpu().numpy()) or dtype == "f64"   # fixed-point spread
    ref = O.pipe_menon_weights(k, n, 4)
    assert np.max(np.abs(a - ref) / ref) < tol


def test_forward_smallest_grid():
    from paper_1706_08575_amd.ftcg import Plan
    rng = np.random.default_rng(3)
    k = rng.uniform(-4, 4, size=(50, 2))
    img = rng.standard_normal((8, 8)) + 1j * rng.standard_normal((8, 8))
    with Plan(8, dim=2, dtype="f64", weights="none") as P:
        P.set_points(dev(k))
        out = P.forward(dev(img)).cpu().numpy()
    assert O.rel_l2(out, O.forward(k, img, len(img))) < 1e-9
