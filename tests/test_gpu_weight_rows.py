"""Frame weights where candidates of the own and of later bin rows meet: the
symmetric pair sum tells the two apart (a later row's coordinate on axis 0 is
never the own one), so equal coordinates on either axis, exact repeats, and
neighbours just across a bin boundary all have to come out of the right form.
Every samples-per-lane and lanes-per-sample choice is compared with the
float64 oracle (eq:difopt); points differ by 2^-20 or are equal.

Bound: a term sinc(d)^2 carries about 2^-51 absolute error in the sine
difference over pi |d|, so at d = 2^-20 about 2^-30 relative of a term that is
at most 1; the smallest sum is 1 and 1e-8 holds any mix of them.
"""
import numpy as np
import pytest
import torch

import oracle as O

pytestmark = pytest.mark.gpu

N = 64


def raster(kind):
    rng = np.random.default_rng(5)
    if kind == "lattice":        # integer and half-integer lattice: equal on both axes, across all rows
        a = np.arange(-24, 24.5, 0.5)
        return np.stack(np.meshgrid(a, a, indexing="ij"), -1).reshape(-1, 2)
    if kind == "columns":        # equal on axis 0, 2^-20 apart on axis 1
        a = np.repeat(rng.integers(-30, 30, 40).astype(float), 25)
        return np.stack([a, rng.integers(-30, 30, 1000) + 2.0**-20 * rng.integers(0, 9, 1000)], 1)
    if kind == "rows":           # equal on axis 1, 2^-20 apart on axis 0 around every integer
        b = np.repeat(rng.integers(-30, 30, 40).astype(float), 25)
        return np.stack([rng.integers(-30, 30, 1000) + 2.0**-20 * rng.integers(-9, 9, 1000), b], 1)
    a = rng.uniform(-31, 31, (700, 2))   # repeats of scattered points, in another order
    return np.concatenate([a, a[rng.permutation(700)[:300]]])


@pytest.mark.parametrize("kind", ["lattice", "columns", "rows", "repeats"])
@pytest.mark.parametrize("samples,lanes", [(1, 1), (1, 2), (1, 4), (2, 1), (2, 2), (2, 4)])
def test_rows(kind, samples, lanes):
    from paper_1706_08575_amd.ftcg import Plan
    k = np.ascontiguousarray(raster(kind))
    with Plan(N, dim=2) as P:
        P.set_weight_tuning(samples, lanes)
        P.set_points(torch.from_numpy(k).cuda())
        a = P.get_weights()
        torch.cuda.synchronize()
        a = a.cpu().numpy()
    ref = O.frame_weights_at(k, np.arange(len(k)), 8.0)
    assert np.max(np.abs(a - ref) / ref) < 1e-8
