"""Calls from several host threads on one stream (torch's default stream is
one for all threads, and the binding releases the interpreter's lock): the
transform, the k-means assignment and the k-means update use a workspace per
stream, and each call's kernels must find there what that call wrote.  Every
result equals the one computed alone, bit for bit."""
import threading

import numpy as np
import pytest
import torch

from test_gpu_kmeans import DEV, as_keys, say, unit
from test_gpu_transform import make_case

pytestmark = pytest.mark.gpu


def _transform(seed, M, D, l):
    from paper_2502_15572_amd import transform
    x, mean, var, W = make_case(M, D, l, seed=seed)
    args = [torch.from_numpy(a).to(DEV) for a in (x, mean, var, W)]
    return lambda: (transform(*args),)


def _assign(seed, n, d, P, dt):
    from paper_2502_15572_amd import kmeans_assign
    rng = np.random.default_rng(seed)
    x = as_keys(unit(rng, n, d), dt).to(DEV)
    c = torch.from_numpy(unit(rng, P, d).astype(np.float32)).to(DEV)
    return lambda: kmeans_assign(x, c, with_score=True)


def _update(seed, n, d, P):
    from paper_2502_15572_amd import kmeans_update
    rng = np.random.default_rng(seed)
    x = as_keys(unit(rng, n, d), "f16").to(DEV)
    a = torch.from_numpy(rng.integers(0, P, n).astype(np.int32)).to(DEV)
    c0 = torch.from_numpy(unit(rng, P, d).astype(np.float32)).to(DEV)

    def call():
        c = c0.clone()
        return c, kmeans_update(x, a, c)
    return call


CASES = {
    # the same shapes with other weights, and other shapes
    "transform": lambda: [_transform(1, 2100, 4096, 128), _transform(2, 2100, 4096, 128),
                          _transform(3, 20001, 512, 200), _transform(4, 30, 2048, 100)],
    "assign": lambda: [_assign(1, 30000, 128, 300, "f16"), _assign(2, 30000, 128, 300, "f16"),
                       _assign(3, 9000, 64, 900, "bf16"), _assign(4, 3000, 256, 2000, "f32")],
    "update": lambda: [_update(1, 140000, 128, 300), _update(2, 140000, 128, 300),
                       _update(3, 270000, 64, 70000), _update(4, 5000, 64, 50)],
}


@pytest.mark.parametrize("op", list(CASES))
def test_threads_on_one_stream(gpu_lib, op):
    say("threads on one stream", op)
    calls = CASES[op]()
    want = [c() for c in calls]
    torch.cuda.synchronize()
    outs = [[] for _ in calls]
    gate = threading.Barrier(len(calls))

    def work(i):
        gate.wait()
        for _ in range(20):
            outs[i].append(calls[i]())

    threads = [threading.Thread(target=work, args=(i,)) for i in range(len(calls))]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    torch.cuda.synchronize()
    for got, ref in zip(outs, want):
        assert len(got) == 20
        for g in got:
            for a, b in zip(g, ref):
                assert torch.equal(a, b)
