"""Memory that the library keeps for later calls is bounded and goes back:
blocks of closed indexes, and the operand and sorting buffers of uncaptured
transforms, assignments and updates, to the driver by release_cached; an
outgrown buffer of that kind at once.  Calls afterwards allocate again and
give the same results."""
import gc

import numpy as np
import pytest
import torch

from test_gpu_failure import datastore, free_bytes
from test_gpu_kmeans import DEV, as_keys, say, unit

pytestmark = pytest.mark.gpu
SLACK = 4 << 20  # small allocations come from blocks of 2 MiB


def _release():
    from paper_2502_15572_amd import release_cached
    gc.collect()
    torch.cuda.empty_cache()
    release_cached()


def test_blocks_of_closed_indexes(gpu_lib):
    from paper_2502_15572_amd import Index, PartitionedIndex
    say("blocks of closed indexes")
    x, cont, q = datastore(N=1 << 20, d=256)  # 512 MiB of keys, 40 MiB of values
    for make in (Index, PartitionedIndex.by_first_token):
        make(x[:100], cont[:100]).close()  # loads the kernels
    _release()
    before = free_bytes()
    total = torch.cuda.mem_get_info()[1]
    for make in (Index, PartitionedIndex.by_first_token):
        for _ in range(3):
            ix = make(x, cont)
            torch.cuda.synchronize()
            ix.close()
            kept = before - free_bytes()
            assert (512 << 20) - SLACK <= kept <= total // 128 + SLACK
        _release()
        assert abs(before - free_bytes()) <= SLACK
    ix = Index(x, cont)
    want = ix.search(q[:4], 10)
    ix.close()
    _release()
    ix = Index(x, cont)
    for a, b in zip(ix.search(q[:4], 10), want):
        assert torch.equal(a, b)
    ix.close()
    _release()


def test_buffers_of_uncaptured_calls(gpu_lib):
    from paper_2502_15572_amd import kmeans_assign, kmeans_update, transform
    from test_gpu_transform import make_case
    say("buffers of uncaptured calls")
    rng = np.random.default_rng(3)
    x = as_keys(unit(rng, 1 << 19, 32), "f16").to(DEV)
    big = torch.from_numpy(unit(rng, 1 << 18, 64).astype(np.float32)).to(DEV)
    rows = torch.nn.functional.normalize(torch.randn(4096, 64, device=DEV)).half()
    args = [torch.from_numpy(a).to(DEV) for a in make_case(600, 4096, 1024, seed=3)]
    streams = [torch.cuda.Stream() for _ in range(2)]
    torch.cuda.synchronize()

    def calls(s):
        with torch.cuda.stream(s):
            out = [kmeans_assign(rows, big[: 1 << 15].contiguous(), stream=s)]
            grown = [kmeans_assign(rows, big, stream=s)]  # outgrows the buffer
            a = torch.arange(1 << 19, dtype=torch.int32, device=DEV) % 64
            c = torch.ones(64, 32, device=DEV)
            kmeans_update(x, a, c, stream=s)
            return out + grown + [c, transform(*args, stream=s)]

    want = [calls(s) for s in streams]  # (kernels loaded, k-means sums allocated)
    _release()
    before = free_bytes()
    got = [calls(s) for s in streams]
    torch.cuda.synchronize()
    # 96 MiB of assignment operands per stream, 8 of sorting and 24 of transform ones
    held = before - free_bytes()
    assert held >= 2 * (120 << 20)
    for g, w in zip(got, want):
        for a, b in zip(g, w):
            assert torch.equal(a, b)
    del got, g, a, b
    _release()
    assert abs(before - free_bytes()) <= SLACK
    # the outgrown buffer (12 MiB) is not held beside its successor
    s = streams[0]
    with torch.cuda.stream(s):
        kmeans_assign(rows, big, stream=s)
    _hold = before - free_bytes()
    _release()
    with torch.cuda.stream(s):
        kmeans_assign(rows, big[: 1 << 17].contiguous(), stream=s)
        kmeans_assign(rows, big, stream=s)
    gc.collect()
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    assert before - free_bytes() <= _hold + SLACK
    _release()


def test_transform_workspace_is_bounded(gpu_lib):
    """Partial sums of a batch that is split over D take at most 256 MiB (eight
    slices, which the split would take otherwise, 264) beside the operands."""
    from paper_2502_15572_amd import transform
    say("transform workspace")
    M, D, l = 8448, 16384, 1024
    x = torch.randn(M, D, device=DEV)
    mean, var = torch.zeros(D, device=DEV), torch.ones(D, device=DEV)
    W = torch.randn(D, l, device=DEV) / 128
    out = torch.empty(M, l, device=DEV)
    s = torch.cuda.Stream()
    torch.cuda.synchronize()
    with torch.cuda.stream(s):
        transform(x[:600], mean, var, W, out=out[:600], stream=s)  # loads the kernels
    _release()
    before = free_bytes()
    with torch.cuda.stream(s):
        transform(x, mean, var, W, out=out, stream=s)
    torch.cuda.synchronize()
    assert 6 * D * l <= before - free_bytes() <= 6 * D * l + (256 << 20) + SLACK
    _release()
