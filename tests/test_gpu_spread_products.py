"""Float64 spread as matrix products (tiles of 32 and 64, one partial tile)
against the LDS-atomic kernel (two partial tiles) over all half-widths, record
counts of a tile around the chunk of 64 records and the groups of four, samples
on tile and block edges, and non-finite values.

Bound: both kernels form a cell from at most 400 taps, each tap from the same
three exponentials' factors by recursions of at most 16 steps (under 2^-45
relative), and add them in float64 in some order: 1e-11 of the largest cell.
"""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

N, G = 64, 128


def points(count, seed):
    """count samples within one tile (0 .. 32 cells), every fourth on an edge of a tile or a block of 16"""
    rng = np.random.default_rng(seed)
    u = rng.uniform(0, 32, (count, 2))
    u[::4] = rng.choice([0.0, 15.999, 16.0, 31.999, 32.0], (len(u[::4]), 2))
    return np.ascontiguousarray((u - G / 2) * N / G)


def grids(k, f, W, tile, dtype=torch.complex128):
    from paper_1706_08575_amd.ftcg import Plan
    out = []
    for copies in (1, 2):
        with Plan(N, dim=2, W=W, sigma=G / N, dtype="f64" if dtype == torch.complex128 else "f32",
                  weights="none") as P:
            P.set_tuning(tile, "f64", copies)
            P.set_points(torch.from_numpy(k).cuda())
            out.append(P.spread_only(torch.from_numpy(f).cuda().to(dtype)).cpu().numpy())
    return out


@pytest.mark.parametrize("tile", [32, 64])
@pytest.mark.parametrize("W", [2, 3, 4, 5, 6, 7, 8])
@pytest.mark.parametrize("count", [1, 4, 5, 63, 64, 65, 200])
def test_counts(tile, W, count):
    k = points(count, count + W)
    rng = np.random.default_rng(1)
    f = rng.standard_normal(count) + 1j * rng.standard_normal(count)
    a, b = grids(k, f, W, tile)
    assert np.max(np.abs(a - b)) <= 1e-11 * np.max(np.abs(b))


@pytest.mark.parametrize("tile", [32, 64])
def test_float32_values(tile):
    k = points(150, 3)
    f = np.random.default_rng(2).standard_normal(150) + 0j
    a, b = grids(k, f, 6, tile, torch.complex64)
    assert np.max(np.abs(a - b)) <= 1e-5 * np.max(np.abs(b))   # float32 factors: 16 steps of 2^-24


@pytest.mark.parametrize("bad", [np.nan, np.inf, -np.inf])
def test_non_finite_values_stay_in_their_footprint(bad):
    k = points(100, 4)
    f = np.random.default_rng(3).standard_normal(100) + 0j
    f[37] = complex(bad, 1.0)
    a, b = grids(k, f, 6, 32)
    assert np.array_equal(np.isfinite(a.real), np.isfinite(b.real))
    assert not np.isfinite(b.real).all()
    ok = np.isfinite(b.real) & np.isfinite(a.imag) & np.isfinite(b.imag)
    assert np.max(np.abs(a - b)[ok]) <= 1e-11 * np.max(np.abs(b[ok]))
