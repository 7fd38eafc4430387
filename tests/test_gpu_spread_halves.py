"""Fixed-point spread with a tile's records in two lists (more than W of the 2W
rows inside the tile, or W and fewer) against the float64 accumulation: every
half-width, tiles of 16, 32 and 64, record counts around the chunk of 256, and
samples whose footprint ends on each row of a tile edge.

Bound: both form a tap from float32 factors by at most 15 recursion steps
(2^-24 each on the value and on the ratio: under 120 of them, 7.2e-6 of a tap),
and the fixed-point quantum is below 2^-31 of the tile's records' sum, 300 times
the largest value at most: 1e-5 of the largest cell.
"""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

N, G = 64, 128


def points(count, W, tile, seed):
    """samples whose first rows run over every offset to the tile's edges, the rest anywhere in two tiles"""
    rng = np.random.default_rng(seed)
    u = rng.uniform(0, 2 * min(tile, 32), (count, 2))
    edge = np.arange(-2 * W, 2 * W + 1) + tile + 0.25
    u[: min(count, len(edge)), 0] = edge[:count]
    return np.ascontiguousarray((u - G / 2) * N / G)


@pytest.mark.parametrize("tile", [16, 32, 64])
@pytest.mark.parametrize("W", [2, 3, 4, 5, 6, 7, 8])
@pytest.mark.parametrize("count", [1, 40, 255, 256, 257, 700])
def test_lists(tile, W, count):
    from paper_1706_08575_amd.ftcg import Plan
    k = points(count, W, tile, count + W)
    rng = np.random.default_rng(1)
    f = rng.standard_normal(count) + 1j * rng.standard_normal(count)
    out = []
    for accum in ("fixed", "f64"):
        with Plan(N, dim=2, W=W, sigma=G / N, dtype="f32", weights="none") as P:
            P.set_tuning(tile, accum, 1)
            P.set_points(torch.from_numpy(k).cuda())
            out.append(P.spread_only(torch.from_numpy(f).cuda().to(torch.complex64)).cpu().numpy())
    assert np.max(np.abs(out[0] - out[1])) <= 1e-5 * np.max(np.abs(out[1]))
