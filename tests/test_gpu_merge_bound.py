"""Merges whose lists' best keys lie close together while other lists are empty
or hold negative scores only: keys in tight clusters, some of them opposite
the queries, with and without the next-token filter and grouped by first token.
The bound over the lists' best keys must neither lose a result nor depend on
the empty lists; every rank is compared with the oracle."""
import numpy as np
import pytest
import torch

import oracle
from datagen import to_numpy_bits
from parity import check_batch
from test_gpu_kmeans import DEV, as_keys, say

pytestmark = pytest.mark.gpu

CASES = [
    # dtype, N, d, B, k, clusters, noise
    ("f32", 65536, 64, 2, 100, 16, 1e-3),
    ("f32", 16384, 32, 8, 10, 1, 1e-4),
    ("f16", 200001, 64, 1, 100, 16, 1e-3),
    ("f16", 100003, 100, 13, 30, 2, 1e-3),
]


@pytest.mark.parametrize("dt,N,d,B,k,ncl,noise", CASES,
                         ids=["%s-N%d-d%d-B%d-k%d-c%d-n%g" % c for c in CASES])
def test_concentrated_scores(gpu_lib, dt, N, d, B, k, ncl, noise):
    from paper_2502_15572_amd import Index, PartitionedIndex
    say("concentrated scores", dt, N, d, B, k, ncl, noise)
    rng = np.random.default_rng(N + d)
    cen = rng.standard_normal((ncl, d))
    cen /= np.linalg.norm(cen, axis=1, keepdims=True)
    cen[ncl // 2:] *= -1.0 if ncl > 1 else 1.0
    # runs of rows of one cluster, so that whole lists lie in it
    which = np.repeat(rng.integers(0, ncl, N // 64 + 1), 64)[:N]
    x = cen[which] + noise * rng.standard_normal((N, d))
    x /= np.linalg.norm(x, axis=1, keepdims=True)
    x[N // 3] = x[N // 3 + 1]            # an exact tie
    q = (np.sign(cen[rng.integers(0, ncl, B), :1]) * cen[rng.integers(0, ncl, B)])
    q = np.ascontiguousarray(q, np.float32)
    cont = rng.integers(0, 30, (N, 2)).astype(np.int32)
    nt = rng.integers(0, 30, B).astype(np.int32)
    keys = as_keys(x, dt)
    kb, kdt = to_numpy_bits(keys)
    exact = dt == "f32" or B <= 4
    kd, cd, qd, nd = keys.to(DEV), torch.from_numpy(cont).to(DEV), torch.from_numpy(q).to(DEV), \
        torch.from_numpy(nt).to(DEV)
    ix = Index(kd, cd)
    tix = PartitionedIndex.by_first_token(kd, cd)
    got = {"plain": ix.search(qd, k), "filtered": ix.search(qd, k, next_tok=nd),
           "by token": tix.search_next_token(qd, nd, k)}
    torch.cuda.synchronize()
    for how, (idx, score, tok) in got.items():
        f = None if how == "plain" else nt
        o_idx, o_score, _, o_next = oracle.topk(kb, kdt, q, k, cont, next_tok=f)
        # (a batch of more than four takes 16-bit keys' queries in 16 bits)
        tol = 1e-5 if exact or how == "by token" else 2e-3
        check_batch(idx.cpu().numpy(), score.cpu().numpy(), tok.cpu().numpy(), o_idx, o_score,
                    o_next, lambda b, rows: oracle.score_rows(kb, kdt, q[b], rows), N, cont, tol,
                    next_tok=f)
    ix.close()
    tix.close()
