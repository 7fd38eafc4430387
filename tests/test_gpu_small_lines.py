"""1D rasters with plain weights in one launch (up to 4096 samples) against the
general launches and the oracle: sizes around a workgroup's samples and the
limit, float32 and float64, samples on tile edges and the periodic seam, equal
samples, several tiles, a second call on the same plan, rejected points, and
the calls that read what the launch leaves.

The weights are sums of squares rounded to one quantum, so those of the general
launches (reached with more tiles than the one launch takes) are equal bit for
bit. Images: the bars of the oracle comparisons, 1e-10 and 1e-4 relative.
"""
import numpy as np
import pytest
import torch

import oracle as O

pytestmark = pytest.mark.gpu


def line(n, m, seed):
    rng = np.random.default_rng(seed)
    k = rng.uniform(-n / 2, n / 2, m)
    k[::7] = np.round(k[::7])                  # grid points and repeats
    k[: min(m, 3)] = [-n / 2, n / 2 - 1e-9, 0.0][: min(m, 3)]
    f = rng.standard_normal(m) + 1j * rng.standard_normal(m)
    return k, f


@pytest.mark.parametrize("dtype,bar", [("f32", 1e-4), ("f64", 1e-10)])
@pytest.mark.parametrize("n,m", [(8, 1), (16, 15), (32, 33), (256, 512), (256, 513), (1024, 2047), (2048, 4096),
                                 (2048, 4097)])
def test_image_and_weights(n, m, dtype, bar):
    from paper_1706_08575_amd.ftcg import Plan
    with Plan(n, dim=1, dtype=dtype) as P:
        for seed in (1, 2):
            k, f = line(n, m, seed)
            kd = torch.from_numpy(k).cuda()
            P.set_points(kd)
            img = P.execute(torch.from_numpy(f).cuda().to(P.cdtype)).cpu().numpy()
            a = P.get_weights().cpu().numpy()
            ref = O.frame_weights_at(k.reshape(-1, 1), np.arange(m), 8.0)
            assert np.max(np.abs(a - ref) / ref) < 1e-10
            # the oracle's footprint is closed (2W + 1 cells about a grid point), the
            # kernels' half open (2W): 2^-40 to the right the two agree (a change below 1e-11)
            want = O.ftcg_image(k.reshape(-1, 1) + 2.0**-40, f, a, n)
            assert O.rel_l2(img.ravel(), np.asarray(want).ravel()) < bar
            back = P.execute(torch.from_numpy(f).cuda().to(P.cdtype)).cpu().numpy()
            assert np.allclose(back, img, rtol=0, atol=1e-12 * np.abs(img).max() if dtype == "f64" else
                               1e-6 * np.abs(img).max())


@pytest.mark.parametrize("bad", [np.nan, np.inf, -(2.0**41)])
def test_rejected_points(bad):
    from paper_1706_08575_amd import _lib as L
    from paper_1706_08575_amd.ftcg import Plan
    k, f = line(64, 100, 3)
    with Plan(64, dim=1, dtype="f64") as P:
        k[57] = bad
        with pytest.raises(L.FtcgError):
            P.set_points(torch.from_numpy(k).cuda())
        k[57] = 1.25
        P.set_points(torch.from_numpy(k).cuda())     # the plan goes on
        assert np.isfinite(P.execute(torch.from_numpy(f).cuda()).cpu().numpy()).all()


@pytest.mark.parametrize("dtype", ["f32", "f64"])
@pytest.mark.parametrize("m", [1, 31, 1000, 4096])
def test_against_the_general_launches(m, dtype):
    from paper_1706_08575_amd.ftcg import Plan
    k, f = line(2048, m, 4)
    out = []
    for tile in (0, 32):           # 4 tiles of 1024 cells, 128 of 32
        with Plan(2048, dim=1, dtype=dtype) as P:
            if tile:
                P.set_tuning(tile, "fixed" if dtype == "f32" else "f64", 1)
            P.set_points(torch.from_numpy(k).cuda())
            img = P.execute(torch.from_numpy(f).cuda().to(P.cdtype))
            back = P.forward(img)
            out.append([x.cpu().numpy() for x in (P.get_weights(), img, back)])
    assert np.array_equal(out[0][0], out[1][0])
    tol = 1e-12 if dtype == "f64" else 1e-5
    for a, b in zip(out[0][1:], out[1][1:]):
        assert np.linalg.norm(a - b) <= tol * np.linalg.norm(b)
