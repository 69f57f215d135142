"""Candidate selection of the batched path where a query has to look through clusters of several chunks (needs an MI355X)."""

import numpy as np
import pytest
import torch

from oracle import oracle as O
from paper_2410_18926_amd.synth import random_index
from paper_2410_18926_amd.synth.workloads import Workload

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def B():
    from paper_2410_18926_amd import binding
    assert torch.cuda.is_available(), "these tests need the GPU"
    return binding


def _index(metric, n, L, r=16, d=32, seed=3):
    wl = Workload("big-clusters", seed, n=n, d=d, nq=1, G=1, alpha=None, normalize=False, lognormal_norms=None, metric=metric,
                  L=L, dp=d, r=r, w=1, m=1)
    rng = np.random.default_rng(seed)
    corpus = torch.from_numpy(rng.standard_normal((n, d)).astype(np.float32))
    return random_index(corpus, wl)


@pytest.mark.parametrize("metric", [0, 1])
@pytest.mark.parametrize("m", [10, 200, 1500])
def test_clusters_of_many_chunks(B, metric, m):
    """Clusters of 4000 points: the survivor list fills up and is compacted several times inside one cluster, so every wavefront
    of the block has to see the same number of survivors at every step."""
    ix = _index(metric, n=24_000, L=6)
    queries = np.random.default_rng(9).standard_normal((700, 32)).astype(np.float32)
    gix = B.Index.from_arrays(ix.to("cuda"))
    oix = O.OracleIndex(ix.numpy())
    _, _, ost = O.search(oix, queries, 5, 3, m, stages=True)
    q = torch.from_numpy(queries).cuda()
    for _ in range(3):
        _, _, st = gix.search_stages(q, 5, 3, m)
        np.testing.assert_array_equal(np.sort(st["cand_rows"].astype(np.int64), axis=1), np.sort(ost["cand_rows"], axis=1))
    gix.close()
