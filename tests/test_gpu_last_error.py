"""A call that goes on without a workspace it could not get succeeds, with the
fp32 kernels' results, and leaves the thread's error text as it was."""
import numpy as np
import pytest
import torch

from test_gpu_failure import fail_alloc_at
from test_gpu_kmeans import DEV, as_keys, say, unit
from test_gpu_transform import make_case

pytestmark = pytest.mark.gpu


def _assign():
    from paper_2502_15572_amd import kmeans_assign
    rng = np.random.default_rng(1)
    x = as_keys(unit(rng, 60000, 64), "f16").to(DEV)
    c = torch.from_numpy(unit(rng, 500, 64).astype(np.float32)).to(DEV)
    return lambda s: kmeans_assign(x, c, stream=s)


def _transform():
    from paper_2502_15572_amd import transform
    args = [torch.from_numpy(a).to(DEV) for a in make_case(70000, 128, 128, seed=1)]
    return lambda s: transform(*args, stream=s)


def _update():
    from paper_2502_15572_amd import kmeans_update
    rng = np.random.default_rng(2)
    x = as_keys(unit(rng, 1 << 17, 128), "f16").to(DEV)
    a = torch.from_numpy(rng.integers(0, 50, 1 << 17).astype(np.int32)).to(DEV)

    def call(s):
        c = torch.zeros(50, 128, device=DEV)
        kmeans_update(x, a, c, stream=s)
        return c
    return call


# the update's sums are its first allocation on a stream, its sort the second
@pytest.mark.parametrize("make,n", [(_assign, 1), (_transform, 1), (_update, 2)],
                         ids=["assign", "transform", "update"])
def test_no_error_left_behind(gpu_lib, make, n):
    say("no error left behind", make.__name__)
    call = make()
    s = torch.cuda.Stream()
    torch.cuda.synchronize()
    gpu_lib.dresd_search(None, None, 1, 1, None, None, None, None)
    text = gpu_lib.dresd_last_error()
    with fail_alloc_at(n), torch.cuda.stream(s):
        got = call(s)
    assert gpu_lib.dresd_last_error() == text
    with torch.cuda.stream(s):
        want = call(s)
    torch.cuda.synchronize()
    if make is _assign:
        assert (got != want).float().mean() <= 1e-4  # near-ties: other sums
    elif make is _transform:
        assert torch.allclose(got, want, rtol=0, atol=(128 + 10) * 2.0 ** -22)
    else:
        assert torch.equal(got, want)  # the sums do not depend on the order
