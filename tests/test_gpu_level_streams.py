"""k-means levels on several streams of one handle, beside its uniform weighting, and under capture: results are those of
the same calls one after another (bitwise; the sums and their order do not depend on the path)."""

import math

import numpy as np
import pytest
import torch

import sims

pytestmark = pytest.mark.gpu

N, LEVELS = 300, 6


@pytest.fixture()
def handle(gpu):
    from paper_2310_09200_amd import Context, StandardSynthesis
    ctx = Context(0)
    s = StandardSynthesis(ctx, np.array([[0.0, 0.0, 1.0]]), LEVELS, 1, N, 32)
    yield s
    torch.cuda.synchronize()
    s.close()
    ctx.close()


def spectra(count):
    g = np.random.default_rng(5)
    return [torch.as_tensor(np.concatenate([np.exp(g.normal(0, 1.5, N - 40)), -g.random(40)]), device="cuda")
            for _ in range(count)]


def weighting(s):
    g = np.random.default_rng(6)
    x = torch.as_tensor(sims.disk_layout(N, 900.0, g, z_sigma_m=1.0), device="cuda")
    V = torch.view_as_complex(torch.as_tensor(g.normal(size=(N, N, 2)), device="cuda"))
    return lambda: s.uniform_weighting(x, 2.0, V, [1.0, 0, 0], [0, 1.0, 0], math.radians(5.0))


def test_streams(handle):
    s, lams, weigh = handle, spectra(4), weighting(handle)
    want = []
    for lam in lams:
        want.append([t.clone() for t in s.levels_kmeans(lam)])
        s.sync()
    want_v = weigh().clone()
    s.sync()
    busy = torch.randn(4096, 4096, device="cuda")
    streams = [torch.cuda.Stream() for _ in range(4)]
    for rnd in range(6):
        torch.cuda.synchronize()
        got = []
        for i, st in enumerate(streams):
            with torch.cuda.stream(st):
                for _ in range(3):
                    busy @ busy  # the calls are queued before any of them runs
                if (i + rnd) % 4 == 3:
                    v = weigh()
                for _ in range(2):
                    got.append((i, s.levels_kmeans(lams[i])))
        torch.cuda.synchronize()
        print("case streams, round", rnd, flush=True)
        for i, (iv, lev) in got:
            assert torch.equal(iv, want[i][0]) and torch.equal(lev, want[i][1])
        assert torch.equal(v, want_v)
    s.sync()


def test_capture(handle):
    s, lams, weigh = handle, spectra(2), weighting(handle)
    want = [[t.clone() for t in s.levels_kmeans(lam)] for lam in lams]
    want_v = weigh().clone()
    s.sync()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        iv, lev = s.levels_kmeans(lams[0])
    other = torch.cuda.Stream()
    for rnd in range(4):
        print("case capture, replay", rnd, flush=True)
        iv.zero_()
        torch.cuda.synchronize()
        graph.replay()
        with torch.cuda.stream(other):
            iv1, lev1 = s.levels_kmeans(lams[1])
            v = weigh()
        torch.cuda.synchronize()
        assert torch.equal(iv, want[0][0]) and torch.equal(lev, want[0][1])
        assert torch.equal(iv1, want[1][0]) and torch.equal(lev1, want[1][1])
        assert torch.equal(v, want_v)
    s.sync()
