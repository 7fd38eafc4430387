"""GPU parity of the banded coefficient matrix where a run of samples is one block
of the matrix-core form (r = 4, 5: runs of 10 and 8 samples): sample counts around
one and two runs, pulses that end inside a run, and rasters in shuffled or half
shuffled order, whose runs go to the per-sample form at those strides.

Tolerance: C is the float64 solution of each column's normal equations on both
sides; the sums differ by the order of addition and, in the per-sample form, by
products rounded to 2^-36 (below 1e-11 of a sum), amplified by the normal matrix's
condition number (about 10^2 at these spacings): 1e-8 of the largest entry.
"""
import numpy as np
import pytest
import torch

import oracle as O
from paper_1706_08575_amd import synth as S

pytestmark = pytest.mark.gpu


def check(k, r):
    from paper_1706_08575_amd.ftcg import Plan
    k = np.ascontiguousarray(k)
    with Plan(64, dim=2, dtype="f64", weights="band") as P:
        P.set_band(r)
        kd = torch.from_numpy(k).cuda()
        P.set_points(kd)
        B = P.get_band().cpu().numpy()
        P.set_points(kd)
        assert np.array_equal(B, P.get_band().cpu().numpy())      # fixed order of addition
    ref = O.band_columns(k, r, 8.0)
    err = np.max(np.abs(B - ref)) / np.max(np.abs(ref))
    print(f"m={len(k)} r={r}: {err:.2e}")
    assert err < 1e-8


@pytest.mark.parametrize("r", [4, 5])
@pytest.mark.parametrize("m", [1, 7, 8, 9, 10, 11, 15, 16, 17, 19, 20, 21, 33])
def test_few_samples(m, r):
    check(S.make_sas(7, n=64, pulses=2, per_pulse=48, m=m)[0], r)


@pytest.mark.parametrize("r", [4, 5])
@pytest.mark.parametrize("per", [13, 16, 21])
def test_pulses_end_inside_runs(per, r):
    check(S.make_sas(21, n=64, pulses=6, per_pulse=per)[0], r)


@pytest.mark.parametrize("r", [4, 5])
def test_shuffled_order(r):
    k = S.make_sas(11, n=64, pulses=6, per_pulse=48)[0]
    rng = np.random.default_rng(r)
    check(k[rng.permutation(len(k))], r)
    half = len(k) // 2
    check(np.concatenate([k[:half], k[half:][rng.permutation(len(k) - half)]]), r)
