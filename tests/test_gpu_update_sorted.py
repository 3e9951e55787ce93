"""The k-means update over rows sorted by partition (from 2^24 elements on):
within the fixed-point bound of the oracle, and bit for bit the sums of the
row-order kernel, which a first call inside a capture (no sort workspace on
that stream yet) takes."""
import numpy as np
import pytest
import torch

import oracle
from datagen import to_numpy_bits
from test_gpu_kmeans import DEV, as_keys, say, unit

pytestmark = pytest.mark.gpu

SHAPES = [
    # dtype, n, d, P, how rows are assigned
    ("f16", 131077, 128, 1, "even"),        # one run across every wave
    ("bf16", 170000, 100, 70000, "even"),   # runs of a few rows, three sort digits, empty partitions
    ("f32", 66001, 257, 256, "skew"),       # five steps of 64 dims, half of the rows in one
    ("f16", 262145, 65, 300, "even"),       # one row in the last wave
]


@pytest.mark.parametrize("dt,n,d,P,how", SHAPES, ids=["%s-n%d-d%d-P%d-%s" % s for s in SHAPES])
def test_update_sorted(gpu_lib, dt, n, d, P, how):
    from paper_2502_15572_amd import kmeans_update
    assert n * d >= 1 << 24
    say("update sorted", dt, n, d, P, how)
    rng = np.random.default_rng(n + P)
    keys = as_keys(unit(rng, n, d), dt)
    a = rng.integers(0, P, n).astype(np.int32)
    if how == "skew":
        a[rng.random(n) < 0.5] = P // 3
    old = unit(rng, P, d).astype(np.float32)
    x = oracle.decode_keys(to_numpy_bits(keys)[0], dt)
    want = oracle.kmeans_update(x, a, old.astype(np.float64))
    xd, ad = keys.to(DEV), torch.from_numpy(a).to(DEV)
    c = torch.from_numpy(old).to(DEV)
    start = c.clone()
    counts = kmeans_update(xd, ad, c)
    # row order: the sums' workspace exists on the stream (a small update), the sort's does not
    s = torch.cuda.Stream()
    small = torch.zeros(P, d, device=DEV)
    with torch.cuda.stream(s):
        kmeans_update(xd[:1], ad[:1], small, stream=s)
    torch.cuda.synchronize()
    ref = start.clone()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=s):
        ref_counts = kmeans_update(xd, ad, ref, stream=s)
    for _ in range(2):
        ref.copy_(start)
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(ref, c) and torch.equal(ref_counts, counts)
    assert np.array_equal(counts.cpu().numpy(), np.bincount(a, minlength=P))
    assert np.max(np.abs(c.cpu().numpy() - want)) <= 1e-6
