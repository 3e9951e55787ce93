"""The k-means assignment on the 16-bit matrix cores (rows of at most 256
dims, from 2^25 multiply-adds on) against the fp64 oracle, at the edges of its
variants, and against the library's own fp32 contraction where the split into
16-bit parts does not hold the values.

Tolerance: (d + 2) 2^-24, the bound of an fp32 sum of d exact products of unit
vectors, as for the fp32 contraction; the split drops less than 2^-26 of a
product and sums in fewer steps."""
import numpy as np
import pytest
import torch

import oracle
from datagen import to_numpy_bits
from test_gpu_kmeans import DEV, as_keys, say, unit

pytestmark = pytest.mark.gpu

SHAPES = [
    # dtype, n, d, P: one of each built width, ragged rows and centroids
    ("f16", 1060000, 1, 40),      # one dim; enough rows that no centroid split is needed
    ("bf16", 16001, 32, 66),      # one block of 32 dims, two split groups
    ("f16", 8191, 33, 129),       # two blocks, one dim in the second
    ("f32", 4099, 64, 130),
    ("bf16", 2049, 65, 300),      # three blocks
    ("f32", 5000, 96, 71),
    ("f16", 513, 128, 513),       # four blocks, one row past a workgroup
    ("f32", 1025, 100, 330),      # rows not a multiple of 16 bytes apart in blocks
    ("f16", 1000, 129, 270),      # six blocks (five rounded up)
    ("f32", 700, 190, 256),
    ("bf16", 511, 193, 400),      # eight blocks
    ("f32", 63, 256, 2100),
    ("f16", 1, 256, 131072),      # one row, the centroids split over all workgroups
]


@pytest.mark.parametrize("dt,n,d,P", SHAPES, ids=["%s-n%d-d%d-P%d" % s for s in SHAPES])
def test_assign_split(gpu_lib, dt, n, d, P):
    from paper_2502_15572_amd import kmeans_assign
    assert n * P * d >= 1 << 25
    say("assign split", dt, n, d, P)
    rng = np.random.default_rng(n + d + P)
    x64 = unit(rng, n, d)
    if n > 2:
        x64[n // 2] = 0.0           # a zero row: every score 0, id 0
    keys = as_keys(x64, dt)
    c = unit(rng, P, d).astype(np.float32)
    c[P - 1] = c[1]                 # an exact tie: its rows go to id 1
    c[P // 3] = 0.0                 # a zero centroid
    a, sc = kmeans_assign(keys.to(DEV), torch.from_numpy(c).to(DEV), with_score=True)
    a0 = kmeans_assign(keys.to(DEV), torch.from_numpy(c).to(DEV))
    torch.cuda.synchronize()
    assert torch.equal(a, a0)       # with and without the scores
    a, sc = a.cpu().numpy(), sc.cpu().numpy()
    x = oracle.decode_keys(to_numpy_bits(keys)[0], dt)
    tol = (d + 2) * 2.0 ** -24
    step = max(1, 4000000 // P)
    for r in range(0, n, step):
        oa, ob, S = oracle.kmeans_assign(x[r:r + step], c.astype(np.float64))
        g, m = a[r:r + step], len(oa)
        assert np.all((g >= 0) & (g < P))
        assert np.all(np.abs(sc[r:r + step] - ob) <= tol)
        got = S[np.arange(m), g]
        assert np.all(got >= ob - tol)
        srt = np.partition(S, P - 2, axis=1)
        clear = srt[:, P - 1] - srt[:, P - 2] >= tol
        assert np.array_equal(g[clear], oa[clear])
        assert not np.any(g == P - 1)
    if n > 2:
        assert a[n // 2] == 0 and sc[n // 2] == 0.0


def _wide(t, d):
    """Zero-padded to more than 256 dims: the fp32 contraction computes it."""
    return torch.nn.functional.pad(t, (0, 257 - d)).contiguous()


@pytest.mark.parametrize("dt", ["f16", "bf16", "f32"])
@pytest.mark.parametrize("n,d,P", [(3001, 128, 100), (1100000, 32, 4)])
def test_rows_left_to_fp32(gpu_lib, dt, n, d, P):
    """Rows with infinities or NaN (and fp32 rows past bf16's range or of
    vanishing size) come out bit for bit as the fp32 contraction gives them,
    the others as without them."""
    from paper_2502_15572_amd import kmeans_assign
    say("rows left to fp32", dt, n, d, P)
    rng = np.random.default_rng(n)
    keys = as_keys(unit(rng, n, d), dt)
    clean = keys.clone()
    inf, nan = float("inf"), float("nan")
    odd = {0: (3, inf), 17: (0, -inf), 64: (d - 1, nan), 515: (5, inf), n - 1: (2, nan)}
    for r, (j, v) in odd.items():
        keys[r, j] = v
    keys[515, 6] = -inf
    if dt == "f32":
        keys[700] = 1e-30 * clean[700]
        keys[701, 4] = 3.4e38
        odd.update({700: None, 701: None})
    c = torch.from_numpy(unit(rng, P, d).astype(np.float32)).to(DEV)
    a, sc = kmeans_assign(keys.to(DEV), c, with_score=True)
    ra, rs = kmeans_assign(clean.to(DEV), c, with_score=True)
    rows = sorted(odd)
    wa, ws = kmeans_assign(_wide(keys[rows], d).to(DEV), _wide(c, d), with_score=True)
    torch.cuda.synchronize()
    assert torch.equal(a[rows], wa)
    assert torch.equal(sc[rows].view(torch.int32), ws.view(torch.int32))
    rest = torch.ones(n, dtype=torch.bool)
    rest[rows] = False
    rest = rest.to(DEV)
    assert torch.equal(a[rest], ra[rest]) and torch.equal(sc[rest], rs[rest])


@pytest.mark.parametrize("n,d,P,share", [(70001, 64, 300, 0.5), (600001, 40, 64, 0.3),
                                         (1100000, 32, 4, 0.01), (4097, 200, 300, 1.0)])
def test_many_rows_left_to_fp32(gpu_lib, n, d, P, share):
    """Rows left over in every chunk, more than one block of 64 of them in
    some: bit for bit as the fp32 contraction gives them, the others as without."""
    from paper_2502_15572_amd import kmeans_assign
    say("many rows left to fp32", n, d, P, share)
    rng = np.random.default_rng(n + P)
    keys = as_keys(unit(rng, n, d), "f16")
    c = torch.from_numpy(unit(rng, P, d).astype(np.float32)).to(DEV)
    left = rng.random(n) < share
    left[: n // 3] &= np.arange(n // 3) % 97 == 0   # few there
    dirty = keys.clone()
    dirty[torch.from_numpy(left), 7] = float("inf")
    a, sc = kmeans_assign(dirty.to(DEV), c, with_score=True)
    ra, rs = kmeans_assign(keys.to(DEV), c, with_score=True)
    wa, ws = kmeans_assign(_wide(dirty[torch.from_numpy(left)], d).to(DEV), _wide(c, d),
                           with_score=True)
    torch.cuda.synchronize()
    left = torch.from_numpy(left).to(DEV)
    assert torch.equal(a[left], wa)
    assert torch.equal(sc[left].view(torch.int32), ws.view(torch.int32))
    assert torch.equal(a[~left], ra[~left]) and torch.equal(sc[~left], rs[~left])


@pytest.mark.parametrize("dt", ["f16", "bf16", "f32"])
@pytest.mark.parametrize("value", [float("inf"), float("nan"), 3e38, 1e-25])
def test_centroids_left_to_fp32(gpu_lib, dt, value):
    """A centroid that the split does not hold takes the whole call to the
    fp32 contraction."""
    from paper_2502_15572_amd import kmeans_assign
    n, d, P = 2500, 64, 300
    say("centroids left to fp32", dt, value)
    rng = np.random.default_rng(7)
    keys = as_keys(unit(rng, n, d), dt).to(DEV)
    c = torch.from_numpy(unit(rng, P, d).astype(np.float32))
    c[200] = 0.0
    c[200, 9] = value
    c = c.to(DEV)
    a, sc = kmeans_assign(keys, c, with_score=True)
    wa, ws = kmeans_assign(_wide(keys, d), _wide(c, d), with_score=True)
    torch.cuda.synchronize()
    assert torch.equal(a, wa)
    assert torch.equal(sc.view(torch.int32), ws.view(torch.int32))


@pytest.mark.parametrize("dt", ["f16", "bf16", "f32"])
def test_centroid_scales(gpu_lib, dt):
    """Centroids of sizes 2^-50 .. 2^50 beside each other: every row's best
    score within the fp32 bound of its own magnitude."""
    from paper_2502_15572_amd import kmeans_assign
    n, d, P = 3000, 96, 200
    say("centroid scales", dt)
    rng = np.random.default_rng(11)
    keys = as_keys(unit(rng, n, d), dt)
    x = oracle.decode_keys(to_numpy_bits(keys)[0], dt)
    for e in (-50, 0, 50):
        c = (unit(rng, P, d) * 2.0 ** (e + rng.integers(-3, 4, (P, 1)))).astype(np.float32)
        a, sc = kmeans_assign(keys.to(DEV), torch.from_numpy(c).to(DEV), with_score=True)
        torch.cuda.synchronize()
        oa, ob, S = oracle.kmeans_assign(x, c.astype(np.float64))
        tol = (d + 2) * 2.0 ** -24 * 2.0 ** (e + 3)
        assert np.all(np.abs(sc.cpu().numpy() - ob) <= tol)
        assert np.all(S[np.arange(n), a.cpu().numpy()] >= ob - tol)


@pytest.mark.parametrize("dt,ex,ec", [("f32", -95, 60), ("f32", -118, 70), ("f32", -122, 100),
                                      ("f32", -130, 110), ("bf16", -130, 110),
                                      ("f16", -18, 30)])
def test_vanishing_rows_large_centroids(gpu_lib, dt, ex, ec):
    """Rows so small that bf16 does not hold their lower parts, against
    centroids that bring the scores back into range: no further from 64 bits
    than an fp32 sum of the rows' own values."""
    from paper_2502_15572_amd import kmeans_assign
    n, d, P = 3000, 96, 200
    say("vanishing rows, large centroids", dt, ex, ec)
    rng = np.random.default_rng(13)
    keys = as_keys(unit(rng, n, d) * 2.0 ** ex, dt)
    c = (unit(rng, P, d) * 2.0 ** ec).astype(np.float32)
    x = oracle.decode_keys(to_numpy_bits(keys)[0], dt)
    a, sc = kmeans_assign(keys.to(DEV), torch.from_numpy(c).to(DEV), with_score=True)
    torch.cuda.synchronize()
    oa, ob, S = oracle.kmeans_assign(x.astype(np.float64), c.astype(np.float64))
    tol = (d + 2) * 2.0 ** -24 * 2.0 ** (ex + ec)
    assert np.all(np.abs(sc.cpu().numpy() - ob) <= tol)
    assert np.all(S[np.arange(n), a.cpu().numpy()] >= ob - tol)


def test_assign_on_two_streams(gpu_lib):
    """Assignments on two streams, each with its own workspace, equal the
    ones computed alone."""
    from paper_2502_15572_amd import kmeans_assign
    rng = np.random.default_rng(3)
    data = []
    for n, d, P in ((30000, 128, 300), (9000, 64, 900)):
        keys = as_keys(unit(rng, n, d), "f16").to(DEV)
        c = torch.from_numpy(unit(rng, P, d).astype(np.float32)).to(DEV)
        data.append((keys, c, kmeans_assign(keys, c)))
    torch.cuda.synchronize()
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    outs = [[], []]
    for _ in range(6):
        for i, s in enumerate(streams):
            with torch.cuda.stream(s):
                outs[i].append(kmeans_assign(data[i][0], data[i][1], stream=s))
    torch.cuda.synchronize()
    for i in range(2):
        for a in outs[i]:
            assert torch.equal(a, data[i][2])


def test_first_call_inside_capture(gpu_lib):
    """A first call on a capturing stream has no workspace yet: it runs (and
    replays) on the fp32 contraction instead of failing."""
    from paper_2502_15572_amd import kmeans_assign
    rng = np.random.default_rng(5)
    n, d, P = 20000, 64, 128
    keys = as_keys(unit(rng, n, d), "f16").to(DEV)
    c = torch.from_numpy(unit(rng, P, d).astype(np.float32)).to(DEV)
    ref = kmeans_assign(_wide(keys, d), _wide(c, d))
    s = torch.cuda.Stream()
    g = torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(g, stream=s):
        a = kmeans_assign(keys, c, stream=s)
    for _ in range(3):
        a.zero_()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(a, ref)
