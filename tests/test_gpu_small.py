"""Exact search over small datastores whose waves list whole tiles
(dresd_scan_small) and partitioned scans of few tiles, against the oracle: the
edges of the list sizes (one, two, four tiles per wave), ragged rows and
dims, batches around a query tile, k above the number of lists, the
next-token filter and rows that must not compete."""
import numpy as np
import pytest
import torch

import oracle
from datagen import to_numpy_bits
from parity import TOL, check_batch
from test_gpu_kmeans import DEV, as_keys, say, unit

pytestmark = pytest.mark.gpu

CASES = [
    # dtype, N, d, B, k
    ("f32", 1, 1, 1, 1),
    ("f32", 17, 3, 5, 17),          # every row returned, two tiles
    ("f32", 16384, 256, 16, 10),    # one query tile, full
    ("f32", 16401, 20, 17, 33),     # a tile past 1,024; one query past a tile
    ("f32", 32769, 8, 2, 1),        # two tiles per wave
    ("f32", 65553, 16, 3, 100),     # past 4,096 tiles
    ("f32", 262144, 17, 2, 64),     # four tiles per wave, as many lists as the merge takes
    ("f32", 5000, 500, 129, 20),    # 32 blocks per tile; nine query tiles
    ("f32", 3000, 64, 2, 1024),     # k above the lists: every key a candidate
    ("f16", 16384, 128, 4, 100),
    ("f16", 40003, 100, 1, 16),     # ragged dims, two tiles per wave
    ("f16", 9999, 1024, 3, 7),
    ("f16", 140001, 128, 1, 100),   # past 32 MiB: with the filter as well, from 64 ranks on
    ("f16", 140001, 128, 1, 63),
    ("bf16", 20011, 33, 2, 50),
    ("bf16", 2047, 700, 4, 300),
]


def data(dt, N, d, B, seed):
    rng = np.random.default_rng(seed)
    x = unit(rng, N, d)
    q = unit(rng, B, d).astype(np.float32)
    src = rng.integers(0, N, B)
    q[: B // 2 + 1] = (x[src[: B // 2 + 1]]).astype(np.float32)
    cont = rng.integers(0, 7, (N, 3)).astype(np.int32)
    return as_keys(x, dt), torch.from_numpy(q), cont, cont[src, 0].astype(np.int32)


@pytest.mark.parametrize("dt,N,d,B,k", CASES, ids=["%s-N%d-d%d-B%d-k%d" % c for c in CASES])
def test_small_search(gpu_lib, dt, N, d, B, k):
    from paper_2502_15572_amd import Index
    say("small search", dt, N, d, B, k)
    keys, q, cont, nt = data(dt, N, d, B, N + d + B + k)
    kb, kdt = to_numpy_bits(keys)
    qn = q.numpy()
    ix = Index(keys.to(DEV), torch.from_numpy(cont).to(DEV))
    assert ix.plan(B, k)["scan_kernel"] == "whole_tile"
    ntd = torch.from_numpy(nt).to(DEV)
    for filt in (False, True):
        idx, score, tok = ix.search(q.to(DEV), k, next_tok=ntd if filt else None)
        torch.cuda.synchronize()
        o_idx, o_score, _, o_next = oracle.topk(kb, kdt, qn, k, cont,
                                                next_tok=nt if filt else None)
        # exact query parts at every batch: the fp32 bound for all types
        check_batch(idx.cpu().numpy(), score.cpu().numpy(), tok.cpu().numpy(), o_idx, o_score,
                    o_next, lambda b, rows: oracle.score_rows(kb, kdt, qn[b], rows), N, cont,
                    1e-5, next_tok=nt if filt else None)
    ix.close()


@pytest.mark.parametrize("dt", ["f32", "f16"])
def test_rows_that_cannot_compete(gpu_lib, dt):
    """NaN scores are never returned (their ranks are padded), an infinite
    score ranks first or last, and neither touches its neighbours."""
    from paper_2502_15572_amd import Index, PartitionedIndex
    say("rows that cannot compete", dt)
    N, d, B, k = 100, 32, 3, 100
    keys, q, cont, _ = data(dt, N, d, B, 5)
    q = q.abs() + 0.01
    clean = keys.clone()
    for r in (0, 15, 16, 50, 99):
        keys[r, 3] = float("nan")
    keys[51, 4], keys[52, 4] = float("inf"), float("-inf")
    cd = torch.from_numpy(cont).to(DEV)
    nan, rest = [0, 15, 16, 50, 99], [r for r in range(N) if r not in (0, 15, 16, 50, 99, 51, 52)]

    def look(idx, score):
        idx, score = idx.cpu().numpy(), score.cpu().numpy()
        want = clean.double().numpy()[rest] @ q.double().numpy().T
        for b in range(B):
            # 16-bit keys: the query's other parts are zero or opposite, so an infinite
            # score may be NaN and drop out
            got = [r for r in idx[b].tolist() if r >= 0]
            assert not set(got) & set(nan)
            assert set(rest) <= set(got)
            if 51 in got:
                assert got[0] == 51
            if 52 in got:
                assert got[-1] == 52
            by = dict(zip(idx[b].tolist(), score[b].tolist()))
            assert np.allclose([by[r] for r in rest], want[:, b], atol=1e-5)

    ix = Index(keys.to(DEV), cd)
    idx, score, _ = ix.search(q.to(DEV), k)
    look(idx, score)
    ix.close()
    a = torch.zeros(N, dtype=torch.int32, device=DEV)
    a[40:] = 1
    pix = PartitionedIndex(keys.to(DEV), cd, torch.eye(2, d, device=DEV), a)
    probes = torch.tensor([[1, 0]] * B, dtype=torch.int32, device=DEV)
    idx, score, _ = pix.search_probes(q.to(DEV), probes, k)
    look(idx, score)
    pix.close()


@pytest.mark.parametrize("k", [1, 70, 300])
def test_few_and_many_tiles(gpu_lib, k):
    """Partitions just within and just past the tiles that a wave lists
    whole, in one batch: both forms of the scan agree with the oracle."""
    from paper_2502_15572_amd import PartitionedIndex
    say("few and many tiles", k)
    rng = np.random.default_rng(k)
    d, P = 32, 40
    sizes = np.concatenate([[30000, 1, 500], rng.integers(1, 200, P - 3)])
    a = np.repeat(np.arange(P), sizes).astype(np.int32)
    N = a.size
    rng.shuffle(a)
    keys = as_keys(unit(rng, N, d), "f16")
    cont = rng.integers(0, 9, (N, 2)).astype(np.int32)
    B = 30
    q = unit(rng, B, d).astype(np.float32)
    probes = np.stack([rng.permutation(P)[:3] for _ in range(B)]).astype(np.int32)
    probes[0] = [0, 1, 2]
    probes[1] = [1, 1, -5]
    ix = PartitionedIndex(keys.to(DEV), torch.from_numpy(cont).to(DEV),
                          torch.from_numpy(unit(rng, P, d).astype(np.float32)).to(DEV),
                          torch.from_numpy(a).to(DEV))
    idx, score, tok = ix.search_probes(torch.from_numpy(q).to(DEV),
                                       torch.from_numpy(probes).to(DEV), k)
    torch.cuda.synchronize()
    kb, dt = to_numpy_bits(keys)
    o_idx, o_score, _, o_next = oracle.topk_partitioned(kb, dt, q, k, a, P, probes, cont)
    sets = [set(r.tolist()) for r in probes]
    check_batch(idx.cpu().numpy(), score.cpu().numpy(), tok.cpu().numpy(), o_idx, o_score, o_next,
                lambda b, rows: oracle.score_rows(kb, dt, q[b], rows), N, cont, 1e-5,
                admitted_b=lambda b, rows: np.isin(a[rows], list(sets[b])))
    ix.close()


@pytest.mark.parametrize("B", [4, 16])
def test_small_search_without_allocation(gpu_lib, B):
    """The allocation-free search takes whole-tile lists where they fit its
    scratch (B = 4) and the single-tile scan's shorter ones where they do not."""
    from paper_2502_15572_amd import Index
    from test_zz_no_alloc import _noalloc, _outs
    say("small search without allocation", B)
    N, d, k = 262144, 32, 10
    keys, q, cont, _ = data("f32", N, d, B, 9)
    ix = Index(keys.to(DEV), torch.from_numpy(cont).to(DEV))
    q = q.to(DEV)
    assert (ix.plan(B, k)["workspace_bytes"] <= 64 << 20) == (B == 4)
    ref = ix.search(q, k)
    out = _outs(B, k, cont.shape[1])
    assert _noalloc(gpu_lib, ix, q, out) == 0, gpu_lib.dresd_last_error()
    torch.cuda.synchronize()
    # fp32 sums of the same products in the same order
    for a, b in zip(out, ref):
        assert torch.equal(a, b)
    ix.close()


def _shorter_lists(B):
    """262,144 x 128 fp32 keys: 48 queries' lists of whole tiles (195 MiB) take
    more memory than the single-tile scan's (104 MiB, 136 for 128 queries)."""
    from paper_2502_15572_amd import Index
    keys, q, cont, _ = data("f32", 262144, 128, B, 11)
    ix = Index(keys.to(DEV), torch.from_numpy(cont).to(DEV))
    q = q.to(DEV)
    return ix, q


def test_small_search_without_memory_for_whole_tiles(gpu_lib):
    """A search whose lists of whole tiles cannot be allocated runs with the
    shorter lists, with the same results and no error left behind."""
    from test_gpu_failure import fail_alloc_at
    say("small search, no memory for whole tiles")
    ix, q = _shorter_lists(48)
    gpu_lib.dresd_search(None, None, 1, 1, None, None, None, None)
    text = gpu_lib.dresd_last_error()
    with fail_alloc_at(1):
        got = ix.search(q, 10)
    torch.cuda.synchronize()
    assert gpu_lib.dresd_last_error() == text
    for a, b in zip(got, ix.search(q, 10)):  # fp32 sums of the same products in the same order
        assert torch.equal(a, b)
    ix.close()


def test_small_search_captured_after_a_larger_one(gpu_lib):
    """The workspace of a warm-up at the largest batch serves the capture of a
    smaller one, whose lists of whole tiles it does not hold."""
    say("small search captured after a larger one")
    ix, q = _shorter_lists(48)
    rng = np.random.default_rng(12)
    big = torch.from_numpy(unit(rng, 128, 128).astype(np.float32)).to(DEV)
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        ix.search(big, 10, stream=s)
    torch.cuda.synchronize()
    assert ix.plan(128, 10)["workspace_bytes"] < ix.plan(48, 10)["workspace_bytes"]
    out = (torch.empty((48, 10), dtype=torch.int64, device=DEV),
           torch.empty((48, 10), dtype=torch.float32, device=DEV),
           torch.empty((48, 10, 3), dtype=torch.int32, device=DEV))
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=s):
        ix.search(q, 10, out=out, stream=s)
    want = ix.search(q, 10)
    for _ in range(3):
        for t in out:
            t.zero_()
        g.replay()
        torch.cuda.synchronize()
        for a, b in zip(out, want):
            assert torch.equal(a, b)
    ix.close()


@pytest.mark.parametrize("dt,N,d,B,waves", [
    ("f32", 1, 1, 1, 4),              # one tile, one workgroup
    ("f32", 262144, 144, 1, None),    # past 2^17 blocks of keys
    ("f32", 262144, 128, 1, 4096),    # 2^17 blocks, four tiles per wave
    ("f32", 262145, 16, 1, None),     # past the lists that the merge takes
    ("f32", 16384, 512, 129, 9216),   # nine query tiles; 32 blocks per tile
    ("f32", 16384, 513, 1, None),     # 33 blocks per tile
    ("f32", 262144, 16, 64, 16384),   # 2^20 (query, tile) pairs
    ("f32", 262144, 16, 65, None),
    ("f16", 16384, 128, 4, 1024),
    ("f16", 16384, 128, 5, None),     # past four queries of 16-bit keys
    ("bf16", 16384, 1024, 4, 1024),
    ("bf16", 16384, 1025, 4, None),
])
def test_shapes_of_the_whole_tile_scan(gpu_lib, dt, N, d, B, waves):
    """The plan names the whole-tile scan, with the waves of its launch, just
    inside the limits of its rule and another scan just outside."""
    from paper_2502_15572_amd import Index
    say("shapes of the whole-tile scan", dt, N, d, B)
    ix = Index(torch.zeros(N, d, dtype={"f32": torch.float32, "f16": torch.float16,
                                        "bf16": torch.bfloat16}[dt], device=DEV),
               torch.zeros(N, 1, dtype=torch.int32, device=DEV))
    plan = ix.plan(B, 1)
    assert (plan["scan_kernel"] == "whole_tile") == (waves is not None)
    if waves is not None:
        assert plan["scan_waves"] == waves and plan["launches"] == 1
        assert plan["sample_passes"] == 0
    ix.close()


@pytest.mark.parametrize("dt,d", [("f32", 40), ("f32", 256), ("f32", 340), ("f16", 128),
                                  ("f16", 680), ("bf16", 512), ("bf16", 700)])
def test_waves_of_one_to_nine_tiles(gpu_lib, dt, d):
    """Partitions of 1 to 36 tiles split over four waves: each remainder of a
    wave's tiles by four, over widths at the edges of the blocks read at a time
    (3 to 22 blocks; 16, 8 and 4 at a time), against the oracle."""
    from paper_2502_15572_amd import PartitionedIndex
    say("waves of one to nine tiles", dt, d)
    rng = np.random.default_rng(d)
    tiles = np.array([1, 2, 4, 5, 7, 8, 10, 12, 13, 16, 19, 20, 26, 36])
    sizes = tiles * 16 - rng.integers(0, 16, tiles.size)
    P = B = tiles.size
    a = np.repeat(np.arange(P), sizes).astype(np.int32)
    N = a.size
    rng.shuffle(a)
    keys = as_keys(unit(rng, N, d), dt)
    cont = rng.integers(0, 9, (N, 2)).astype(np.int32)
    q = unit(rng, B, d).astype(np.float32)
    probes = np.arange(P, dtype=np.int32).reshape(B, 1)
    ix = PartitionedIndex(keys.to(DEV), torch.from_numpy(cont).to(DEV),
                          torch.from_numpy(unit(rng, P, d).astype(np.float32)).to(DEV),
                          torch.from_numpy(a).to(DEV))
    k = 100
    idx, score, tok = ix.search_probes(torch.from_numpy(q).to(DEV),
                                       torch.from_numpy(probes).to(DEV), k)
    torch.cuda.synchronize()
    kb, kdt = to_numpy_bits(keys)
    o_idx, o_score, _, o_next = oracle.topk_partitioned(kb, kdt, q, k, a, P, probes, cont)
    check_batch(idx.cpu().numpy(), score.cpu().numpy(), tok.cpu().numpy(), o_idx, o_score, o_next,
                lambda b, rows: oracle.score_rows(kb, kdt, q[b], rows), N, cont, 1e-5,
                admitted_b=lambda b, rows: a[rows] == b)
    ix.close()
