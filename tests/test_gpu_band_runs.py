"""GPU parity of the banded coefficient matrix at the edges of its run layout:
runs of 16 / 14 / 8 samples with one, two or three blocks (r = 1 .. 16), sample
counts around a run, pulses that end inside a run (a jump in k), rasters in
shuffled order (whose runs are left to the per-sample kernel), and a mix of both.

Tolerance: C is the float64 solution of each column's normal equations on both
sides; the sums differ by the order of addition and, in the per-sample kernel,
by products rounded to 2^-36 (below 1e-11 of a sum), amplified by the
normal matrix's condition number (about 10^2 at these spacings): 1e-8 of the
largest entry, as for the whole-raster tests.
"""
import numpy as np
import pytest
import torch

import oracle as O
from paper_1706_08575_amd import synth as S

pytestmark = pytest.mark.gpu


def gpu_band(k, r):
    from paper_1706_08575_amd.ftcg import Plan
    with Plan(64, dim=2, dtype="f64", weights="band") as P:
        P.set_band(r)
        kd = torch.from_numpy(np.ascontiguousarray(k)).cuda()
        P.set_points(kd)
        B = P.get_band().cpu().numpy()
        P.set_points(kd)
        assert np.array_equal(B, P.get_band().cpu().numpy())      # fixed order of addition
        f = S.random_values(9, len(k))
        img = P.execute(torch.from_numpy(f).cuda()).cpu().numpy()
    ref = O.ftcg_image(k, O.band_apply(B, f, r), np.ones(len(k)), 64)
    assert O.rel_l2(img, ref) < 1e-9
    return B


def check(k, r):
    B, Bref = gpu_band(k, r), O.band_columns(k, r, 8.0)
    err = np.max(np.abs(B - Bref)) / np.max(np.abs(Bref))
    print(f"m={len(k)} r={r}: {err:.2e}")
    assert err < 1e-8


def pulses(seed, per, count, m=None):
    k, _, _ = S.make_sas(seed, n=64, pulses=count, per_pulse=per, m=m)
    return k


@pytest.mark.parametrize("r", list(range(1, 17)))
def test_band_every_half_width(r):
    check(pulses(100 + r, 50, 7), r)           # pulses end inside runs


@pytest.mark.parametrize("m", [1, 2, 15, 16, 17, 31, 33])
@pytest.mark.parametrize("r", [2, 8, 12])
def test_band_few_samples(m, r):
    check(pulses(7, 48, 2, m=m), r)


@pytest.mark.parametrize("r", [1, 3, 8, 11])
def test_band_shuffled_order(r):
    k = pulses(11, 48, 6)
    rng = np.random.default_rng(r)
    check(k[rng.permutation(len(k))], r)
    half = len(k) // 2
    check(np.concatenate([k[:half], k[half:][rng.permutation(len(k) - half)]]), r)
