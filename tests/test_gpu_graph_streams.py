"""Graphs of one stream replayed beside each other: an assignment, or a
transform whose dims are not split, captured on a stream that has run it
before, keeps nothing in that stream's buffers, so its graphs may replay on
several streams at once and beside eager calls.  A transform whose dims are split
can be captured after one uncaptured call."""
import numpy as np
import pytest
import torch

from test_gpu_kmeans import DEV, as_keys, say, unit
from test_gpu_transform import make_case

pytestmark = pytest.mark.gpu


def _assign(seed):
    from paper_2502_15572_amd import kmeans_assign
    rng = np.random.default_rng(seed)
    x = as_keys(unit(rng, 60000, 64), "f16").to(DEV)
    c = torch.from_numpy(unit(rng, 500, 64).astype(np.float32)).to(DEV)
    return lambda s: kmeans_assign(x, c, stream=s)


def _transform(seed, M=70000, D=128, l=128):
    from paper_2502_15572_amd import transform
    args = [torch.from_numpy(a).to(DEV) for a in make_case(M, D, l, seed=seed)]
    return lambda s: transform(*args, stream=s)


def _capture(call, s):
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=s):
        out = call(s)
    return g, out


@pytest.mark.parametrize("make", [_assign, _transform], ids=["assign", "transform"])
def test_graphs_of_one_stream_replay_together(gpu_lib, make):
    say("graphs of one stream", make.__name__)
    calls = [make(1), make(2)]
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        eager = [c(s) for c in calls]  # the stream's buffers exist now
    torch.cuda.synchronize()
    graphs = [_capture(c, s) for c in calls]
    want = []
    for g, out in graphs:
        out.zero_()
        g.replay()
        torch.cuda.synchronize()
        want.append(out.clone())
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    for _ in range(5):
        for g, out in graphs:
            out.zero_()
        torch.cuda.synchronize()
        again = []
        for _ in range(4):
            for (g, out), r in zip(graphs, streams):
                with torch.cuda.stream(r):
                    g.replay()
            with torch.cuda.stream(s):
                again.append(calls[0](s))
        torch.cuda.synchronize()
        for (g, out), w in zip(graphs, want):
            assert torch.equal(out, w)
        for a in again:
            assert torch.equal(a, eager[0])
    for w, e in zip(want, eager):
        if w.dtype == torch.int32:
            assert (w != e).float().mean() <= 1e-4  # near-ties: other sums
        else:
            assert torch.allclose(w, e, rtol=0, atol=(128 + 10) * 2.0 ** -22)


def test_split_transform_captured_after_a_call(gpu_lib):
    say("split transform captured")
    M, D, l = 1100, 4096, 128
    call = _transform(3, M, D, l)
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        want = call(s)
    torch.cuda.synchronize()
    g, out = _capture(call, s)
    for _ in range(3):
        out.zero_()
        g.replay()
        torch.cuda.synchronize()
        assert torch.allclose(out, want, rtol=0, atol=(D + 10) * 2.0 ** -22)
