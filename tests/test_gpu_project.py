"""The transform of datastore-sized batches on the 16-bit matrix cores (from
about 2^30 multiply-adds on) in every instance of its kernel (column tiles, copy
width, whole rows or partial sums) and at their edges: several column groups, ragged rows, dims (with 16- and 4-byte
copies) and columns, D split or not, whole rows normalised in the kernel or
after it.  Bound: the fp32 bound of test_gpu_transform, per element; rows that
the split into bf16 parts does not hold come out as the fp32 kernels give them
(rows computed by themselves, below the path's size)."""
import numpy as np
import pytest
import torch

import oracle
from test_gpu_transform import DEV, bound, make_case, run

pytestmark = pytest.mark.gpu

SHAPES = [
    # M, D, l
    (66000, 1024, 16),     # one column tile; whole rows
    (40001, 512, 32),      # two
    (16385, 1030, 33),     # three; rows of x 8 bytes off 16
    (9000, 999, 64),       # four; 4-byte copies
    (7001, 1001, 80),      # five, the last dims past D
    (1025, 4096, 128),     # D split, one row past four blocks
    (2049, 2500, 107),     # seven tiles, a column short
    (66049, 128, 127),     # four blocks of dims, whole rows, one row in the last block
    (70001, 64, 130),      # two column groups of five tiles, not split
    (513, 2048, 1025),     # nine groups
    (600, 3333, 300),
]


@pytest.mark.parametrize("M,D,l", SHAPES, ids=["M%d-D%d-l%d" % s for s in SHAPES])
def test_project_split(gpu_lib, M, D, l):
    print("project split", M, D, l, flush=True)
    assert M * D * l >= 2 ** 29
    x, mean, var, W = make_case(M, D, l, seed=M + D + l)
    x[M // 2] = mean
    got = run(x, mean, var, W)
    step = max(1, 40000000 // D)
    for r in range(0, M, step):
        want = oracle.transform(x[r:r + step], mean, var, W, 1e-5, 1e-12)
        err = np.abs(got[r:r + step] - want)
        tol = bound(x[r:r + step], mean, var, W, 1e-5, want)
        assert np.all(err <= tol), (float(err.max()), float((err / tol).max()))
    assert not got[M // 2].any()


@pytest.mark.parametrize("whole", [True, False], ids=["whole", "split"])
@pytest.mark.parametrize("vec", [True, False], ids=["16B", "4B"])
@pytest.mark.parametrize("nt", range(1, 9))
def test_every_instance(gpu_lib, nt, vec, whole):
    """Each instance of the kernel once: nt tiles of 16 columns (a few columns
    short), rows copied 16 or 4 bytes a lane, rows normalised in the kernel (four
    blocks of dims, too few to split) or partial sums of slices (32 blocks, fewer
    row blocks than half the CUs)."""
    l = 16 * nt - nt % 3
    D = (128 if whole else 1024) - (0 if vec else 1)
    even = D % 4 == 0 and l % 64 == 0  # twice the work before this path is taken
    M = -(-(2 ** 30 if even else 2 ** 29) // (D * l))
    test_project_split(gpu_lib, M, D, l)


@pytest.mark.parametrize("M,D,l", [(66000, 128, 128), (1030, 4096, 256)])
def test_rows_computed_again(gpu_lib, M, D, l):
    """Infinities, NaN, values past bf16's rounding range and rows of
    vanishing size: as computed by themselves (fp32 kernels)."""
    from paper_2502_15572_amd import transform
    print("rows computed again", M, D, l, flush=True)
    x, mean, var, W = make_case(M, D, l, seed=3)
    mean[:] = 0.0
    var[:] = 1.0
    W[7] = 0.0               # an infinity there meets zero weights
    odd = {0: (7, np.inf), 31: (5, np.inf), 33: (D - 1, -np.inf), 300: (2, np.nan),
           M - 2: (9, 3.4e38)}
    clean = x.copy()
    for r, (j, v) in odd.items():
        x[r, j] = v
    x[300 + 1, 3], x[300 + 1, 4] = np.inf, -np.inf
    x[M - 1] = clean[M - 1] * np.float32(1e-25)
    rows = sorted(list(odd) + [301, M - 1])
    t = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(DEV)
    args = (t(mean), t(var), t(W))
    got = transform(t(x), *args, eps_z=0.0, eps_n=0.0)
    ref = transform(t(clean), *args, eps_z=0.0, eps_n=0.0)
    alone = transform(t(x[rows]), *args, eps_z=0.0, eps_n=0.0)
    torch.cuda.synchronize()
    g, a = got[rows].cpu().numpy(), alone.cpu().numpy()
    assert np.array_equal(np.isnan(g), np.isnan(a))
    assert np.array_equal(np.isinf(g), np.isinf(a))
    fin = np.isfinite(a)
    assert np.array_equal(g[~fin & ~np.isnan(a)], a[~fin & ~np.isnan(a)])
    assert np.all(np.abs(g[fin] - a[fin]) <= (D + 10) * 2.0 ** -22)
    rest = torch.ones(M, dtype=torch.bool)
    rest[rows] = False
    rest = rest.to(DEV)
    assert torch.equal(got[rest], ref[rest])


@pytest.mark.parametrize("ez,ew", [(-95, 30), (-118, 65), (-118, 90), (-140, 120), (60, -105),
                                   (75, -115)])
@pytest.mark.parametrize("M,D,l", [(16500, 1024, 64), (1030, 4096, 128), (9001, 515, 250)],
                         ids=["whole", "split", "groups"])
def test_scales_the_split_does_not_hold(gpu_lib, M, D, l, ez, ew):
    """z-scores or weights so small that bf16 does not hold their lower parts,
    beside weights or z-scores that bring the sums back into range: within the
    fp32 bound of 64 bits per element, and together within what the rounding of
    D / 4 fp32 partial sums adds up to as a random walk (2^-24 sqrt(D / 4); with
    bf16's loss 1e-6 to 1e-5).  A row of zeros stays one."""
    say = "scales z 2^%d W 2^%d" % (ez, ew)
    print(say, M, D, l, flush=True)
    rng = np.random.default_rng(M + D)
    x = (rng.standard_normal((M, D)) * 2.0 ** ez).astype(np.float32)
    W = (rng.standard_normal((D, l)) * 2.0 ** ew).astype(np.float32)
    x[M - 2] = 0.0
    mean, var = np.zeros(D, np.float32), np.ones(D, np.float32)
    got = run(x, mean, var, W, eps_z=0.0, eps_n=1e-30)
    rows = np.r_[0:300, M - 300:M]
    want = oracle.transform(x[rows], mean, var, W, 0.0, 1e-30)
    err = np.abs(got[rows] - want)
    tol = bound(x[rows], mean, var, W, 0.0, want)
    if ez < -126:  # x itself holds so few bits that z W can cancel further than bound() says
        tol = tol + 2.0 ** -20
    assert np.all(err <= tol), (float(err.max()), float((err / tol).max()))
    if ez >= -126:
        assert np.linalg.norm(err) <= 2.0 ** -24 * np.sqrt(D / 4) * np.linalg.norm(want)
    assert not got[M - 2].any()


@pytest.mark.parametrize("M,D,l", [(9000, 999, 64), (1030, 4096, 128), (5000, 1000, 200)],
                         ids=["whole", "split", "groups"])
def test_every_row_computed_again(gpu_lib, M, D, l):
    """A value past bf16's rounding range in most rows: as the fp32 kernels
    give them (a captured call), the clean rows as without them."""
    from paper_2502_15572_amd import transform
    print("every row computed again", M, D, l, flush=True)
    x, mean, var, W = make_case(M, D, l, seed=17)
    mean[:] = 0.0
    var[:] = 1.0
    t = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(DEV)
    clean = t(x)
    args = (t(mean), t(var), t(W))
    ref = transform(clean, *args, eps_z=0.0)
    keep = np.arange(M) % 7 == 3
    x[~keep, 5] = 3.395e38
    dirty = t(x)
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        got = transform(dirty, *args, eps_z=0.0, stream=s)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=s):
        fp32 = transform(dirty, *args, eps_z=0.0, stream=s)
    g.replay()
    torch.cuda.synchronize()
    got, fp32, ref = got.cpu().numpy(), fp32.cpu().numpy(), ref.cpu().numpy()
    assert np.array_equal(got[keep], ref[keep])
    fin = np.isfinite(fp32)
    assert np.array_equal(np.isfinite(got[~keep]), fin[~keep])
    assert np.all(np.abs(got - fp32)[~keep & fin.all(axis=1)] <= (D + 10) * 2.0 ** -22)


def test_project_first_call_inside_capture(gpu_lib):
    """No workspace yet on a capturing stream: the fp32 kernels run."""
    from paper_2502_15572_amd import transform
    M, D, l = 70000, 128, 128   # D not split: those kernels need no workspace
    x, mean, var, W = make_case(M, D, l, seed=5)
    t = lambda a: torch.from_numpy(a).to(DEV)
    args = (t(x), t(mean), t(var), t(W))
    want = transform(*args)
    s = torch.cuda.Stream()
    g = torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(g, stream=s):
        y = transform(*args, stream=s)
    for _ in range(3):
        y.zero_()
        g.replay()
        torch.cuda.synchronize()
        assert torch.allclose(y, want, rtol=0, atol=(D + 10) * 2.0 ** -22)
