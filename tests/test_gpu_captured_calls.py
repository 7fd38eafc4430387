"""Calls captured into a graph: a capture only records, so it leaves the plan's
weights as they were, and a replay takes the points the plan has by then (the same
number of samples, so that no buffer moves).

Float32 plans add integers, so equal points give equal images bit for bit;
float64 accumulation adds in any order: 1e-12 relative in float64, 1e-6 where the
tiles are rounded to float32.
"""
import ctypes as C

import numpy as np
import pytest
import torch

from paper_1706_08575_amd import synth as S

pytestmark = pytest.mark.gpu

N = 128
# dtype, set_tuning arguments: kernels that form the weights from the sums, and
# (tile 16, several partial tiles) kernels that read the records' weights
SUMS = [("f32", None), ("f64", None), ("f64", (64, "f64", 1)), ("f32", (32, "f64", 1))]
RECORDS = [("f64", (16, "f64", 1)), ("f64", (32, "f64", 2)), ("f32", (16, "f64", 1)), ("f32", (32, "f64", 2))]


def raster(seed, m=7001):
    k, f, _ = S.make_sas(seed, n=N, pulses=60, per_pulse=120, m=m)
    return torch.from_numpy(k).cuda(), torch.from_numpy(f).cuda()


def same(a, b, dtype, tuning):
    a, b = a.cpu().numpy(), b.cpu().numpy()
    if dtype == "f32" and (tuning is None or tuning[1] == "fixed"):
        return np.array_equal(a, b)
    return np.linalg.norm(a - b) <= (1e-12 if dtype == "f64" else 1e-6) * np.linalg.norm(b)


def plan(dtype, tuning, stream=None, dim=2, n=N):
    from paper_1706_08575_amd.ftcg import Plan
    P = Plan(n, dim=dim, dtype=dtype, stream=stream)
    if tuning:
        P.set_tuning(*tuning)
    return P


def fresh(dtype, tuning, k, f, dim=2, n=N):
    """image and weights of a plan of its own"""
    with plan(dtype, tuning, dim=dim, n=n) as P:
        P.set_points(k)
        w = P.get_weights()
        img = P.execute(f.to(P.cdtype))
        torch.cuda.synchronize()
        return img, w


@pytest.mark.parametrize("dtype,tuning", SUMS + RECORDS)
@pytest.mark.parametrize("before", [0, 2, 4])
def test_replay_takes_new_points(dtype, tuning, before):
    k1, f1 = raster(11)
    k2, f2 = raster(12)
    ref1, _ = fresh(dtype, tuning, k1, f1)
    ref2, w2 = fresh(dtype, tuning, k2, f2)
    s = torch.cuda.Stream()
    with torch.cuda.stream(s), plan(dtype, tuning, stream=s) as P:
        P.set_points(k1)
        f = f1.to(P.cdtype)
        for _ in range(before):
            P.execute(f)
        out = torch.zeros_like(ref1)
        s.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=s):
            P.execute(f, out=out)
        g.replay()
        s.synchronize()
        assert same(out, ref1, dtype, tuning)
        P.set_points(k2)
        f.copy_(f2)
        for _ in range(3):
            out.zero_()
            g.replay()
            s.synchronize()
            assert same(out, ref2, dtype, tuning)
            assert same(P.execute(f), ref2, dtype, tuning)
        assert torch.equal(P.get_weights(), w2)


@pytest.mark.parametrize("dtype,tuning", SUMS + RECORDS)
@pytest.mark.parametrize("call", ["execute", "get_weights"])
def test_capture_does_not_finish_the_weights(dtype, tuning, call):
    from paper_1706_08575_amd import _lib as L
    k, f = raster(13)
    ref, w = fresh(dtype, tuning, k, f)
    s = torch.cuda.Stream()
    with torch.cuda.stream(s), plan(dtype, tuning, stream=s) as P:
        f = f.to(P.cdtype)
        out, wout = torch.zeros_like(ref), torch.zeros_like(w)
        P.set_points(k)
        s.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=s):
            if call == "execute":
                P.execute(f, out=out)
            else:   # without the fallback flag, which would synchronise
                L.check(L.call("ftcg_get_weights", P._h, C.c_void_p(wout.data_ptr()), None), "ftcg_get_weights")
        assert torch.equal(P.get_weights(), w)              # before the graph has run
        assert same(P.execute(f), ref, dtype, tuning)
        for _ in range(3):
            out.zero_()
            wout.zero_()
            g.replay()
            s.synchronize()
            if call == "execute":
                assert same(out, ref, dtype, tuning)
            else:
                assert torch.equal(wout, w)
            assert same(P.execute(f), ref, dtype, tuning)
