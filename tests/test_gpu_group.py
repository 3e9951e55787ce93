"""The device grouping behind the partitioned indexes (radix sort of the rows,
slot table) and the tiled layout's row loads, at the edges where they can go
wrong: rows around a sort block, tokens that differ in any of the four
digits, empty partitions, row pitches of every alignment.

A query for a token must return exactly the rows whose value starts with it
(all of them, k at least their number), each with its own score and value, in
the order of the fp64 scores up to the fp32 bound."""
import numpy as np
import pytest
import torch

from test_gpu_kmeans import DEV, as_keys, say

pytestmark = pytest.mark.gpu


def tokens(rng, kind, n):
    if kind == "one":
        return np.full(n, 7, np.int32)
    if kind == "wide":  # every digit varies, both ends of the range among them
        pool = rng.integers(-2 ** 31, 2 ** 31, max(1, n // 3), dtype=np.int64)
        pool[0] = -2 ** 31
        pool[-1] = 2 ** 31 - 1
        return pool[rng.integers(0, pool.size, n)].astype(np.int32)
    if kind == "high":  # only the top digit varies
        return (rng.integers(-3, 3, n) << 24).astype(np.int32)
    r = rng.zipf(1.3, n)
    return np.minimum(r, 31999).astype(np.int32)


def check(idx, score, tok, x, q, cont, rows):
    got = idx[idx >= 0]
    assert np.array_equal(np.sort(got), rows)
    m = rows.size
    assert np.all(idx[m:] == -1) and np.all(np.isneginf(score[m:])) and not tok[m:].any()
    want = x[got] @ q
    assert np.all(np.abs(score[:m] - want) <= 1e-5)
    assert np.all(np.diff(score[:m]) <= 0)
    assert np.array_equal(tok[:m], cont[got])


@pytest.mark.parametrize("kind", ["one", "wide", "high", "zipf"])
@pytest.mark.parametrize("dt,n,d,L", [("f16", 1, 8, 1), ("f16", 1000, 9, 3), ("bf16", 4095, 6, 2),
                                      ("f32", 4097, 5, 1), ("f16", 12289, 34, 4),
                                      ("f16", 70001, 16, 2)])
def test_group_by_token(gpu_lib, kind, dt, n, d, L):
    from paper_2502_15572_amd import PartitionedIndex
    say("group by token", kind, dt, n, d, L)
    rng = np.random.default_rng(n + d)
    keys = as_keys(rng.standard_normal((n, d)) / np.sqrt(d), dt)
    x = keys.to(torch.float64).numpy()
    cont = rng.integers(-5, 5, (n, L)).astype(np.int32)
    cont[:, 0] = tokens(rng, kind, n)
    ix = PartitionedIndex.by_first_token(keys.to(DEV), torch.from_numpy(cont).to(DEV))
    present, counts = np.unique(cont[:, 0], return_counts=True)
    assert ix.P == present.size
    assert ix.info()["tiles"] == np.sum((counts + 15) // 16)
    small = present[counts <= 1024]
    if small.size == 0:
        ix.close()
        return
    ask = np.concatenate([small[:3], small[-3:], [present[0] - 1 if present[0] > -2 ** 31
                                                  else 123456789]]).astype(np.int32)
    q = rng.standard_normal((ask.size, d)).astype(np.float32) / np.float32(np.sqrt(d))
    k = min(n, 1024)
    idx, score, tok = ix.search_next_token(torch.from_numpy(q).to(DEV),
                                           torch.from_numpy(ask).to(DEV), k)
    torch.cuda.synchronize()
    idx, score, tok = idx.cpu().numpy(), score.cpu().numpy(), tok.cpu().numpy()
    for b, t in enumerate(ask):
        rows = np.nonzero(cont[:, 0] == t)[0]
        check(idx[b], score[b], tok[b], x, q[b].astype(np.float64), cont, rows)
    ix.close()


@pytest.mark.parametrize("n,P", [(1, 1), (5000, 3), (5000, 70000), (20000, 300)])
def test_group_by_partition(gpu_lib, n, P):
    """Partitions given by the caller, most of them empty where P > n; an id
    outside [0, P) is refused."""
    from paper_2502_15572_amd import DresdError, PartitionedIndex
    say("group by partition", n, P)
    rng = np.random.default_rng(n + P)
    d = 32
    keys = as_keys(rng.standard_normal((n, d)) / np.sqrt(d), "f16")
    x = keys.to(torch.float64).numpy()
    cont = rng.integers(0, 9, (n, 2)).astype(np.int32)
    a = rng.integers(0, P, n).astype(np.int32)
    a[n // 2] = P - 1
    cents = rng.standard_normal((P, d)).astype(np.float32)
    dev = [torch.from_numpy(v).to(DEV) for v in (cont, cents, a)]
    ix = PartitionedIndex(keys.to(DEV), *dev)
    counts = np.bincount(a, minlength=P)
    assert ix.info()["tiles"] == np.sum((counts + 15) // 16)
    pick = np.array([P - 1, 0, a[0], P // 2], np.int32)
    k = min(n, 1024)
    q = rng.standard_normal((4, d)).astype(np.float32) / np.float32(np.sqrt(d))
    idx, score, tok = ix.search_probes(torch.from_numpy(q).to(DEV),
                                       torch.from_numpy(pick[:, None].copy()).to(DEV), k)
    torch.cuda.synchronize()
    idx, score, tok = idx.cpu().numpy(), score.cpu().numpy(), tok.cpu().numpy()
    for b, t in enumerate(pick):
        rows = np.nonzero(a == t)[0]
        if rows.size <= k:
            check(idx[b], score[b], tok[b], x, q[b].astype(np.float64), cont, rows)
    ix.close()
    for bad in (-1, P):
        a[n - 1] = bad
        with pytest.raises(DresdError, match="outside"):
            PartitionedIndex(keys.to(DEV), dev[0], dev[1], torch.from_numpy(a).to(DEV))


def test_released_blocks_are_bounded(gpu_lib):
    """Large blocks of destroyed indexes are kept for the next build, never
    more than 1/128 of the device's memory, and builds on them give the same
    answers (also from two threads at once)."""
    import threading
    from paper_2502_15572_amd import Index, PartitionedIndex
    say("released blocks")
    d, L = 64, 2
    torch.cuda.synchronize()
    total = torch.cuda.mem_get_info()[1]
    q = torch.randn(2, d, device=DEV)
    data = []
    for n in (700000, 701000, 1500000):  # 90 MB keys and up
        keys = torch.randn(n, d, device=DEV).to(torch.float16)
        cont = torch.randint(0, 50, (n, L), device=DEV, dtype=torch.int32)
        ix = Index(keys, cont)
        data.append((keys, cont, ix.search(q, 5)))
        ix.close()
    torch.cuda.synchronize()
    free0 = torch.cuda.mem_get_info()[0]
    bad = []

    def build(order):
        s = torch.cuda.Stream()
        for i in order:
            keys, cont, ref = data[i]
            with torch.cuda.stream(s):
                ix = Index(keys, cont, stream=s)
                tix = PartitionedIndex.by_first_token(keys, cont, stream=s)
                got = ix.search(q, 5, stream=s)
                nt = got[2][:, 0, 0].contiguous()
                best = tix.search_next_token(q, nt, 1, stream=s)
                s.synchronize()
            if not all(torch.equal(a, b) for a, b in zip(got, ref)) or \
                    not torch.equal(best[0][:, 0], ref[0][:, 0]):
                bad.append(i)
            ix.close()
            tix.close()

    threads = [threading.Thread(target=build, args=(o,)) for o in ((0, 1, 2, 0), (2, 1, 0, 1))]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not bad
    torch.cuda.synchronize()
    # (torch may have taken a few MB of its own meanwhile)
    assert free0 - torch.cuda.mem_get_info()[0] <= total // 128 + (64 << 20)
