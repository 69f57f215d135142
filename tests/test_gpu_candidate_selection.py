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


@pytest.mark.parametrize("scheme", ["cluster", "columns", "mixed"])
@pytest.mark.parametrize("metric,r,m,nq", [(0, 16, 200, 2049), (1, 40, 10, 2100), (1, 24, 352, 2060), (2, 64, 353, 2050), (0, 32, 864, 2051), (1, 8, 865, 2049),
                                           (1, 24, 200, 300), (0, 48, 600, 2048)])
def test_one_cluster_holds_most_points(B, metric, r, m, nq, scheme):
    """A cluster of 41 111 points (81 work items, the last one ragged) beside small and empty ones: most of it is dismissed by the
    best scores of its quarters (batches beyond 2048 queries and m up to 864; below and above four wavefronts share a query).  Half of its points repeat the codes of the other half, so scores tie at every threshold."""
    ix = _index(metric, n=48_000, L=7, r=r, seed=11 + r)
    rng = np.random.default_rng(r)
    ix.cluster_offsets[:] = torch.tensor([0, 1500, 1500, 42_611, 44_700, 46_749, 46_750, 48_000])
    ix.B[1500 + 20_000:1500 + 40_000] = ix.B[1500:1500 + 20_000]
    if metric == 1:
        ix.corpus[1500 + 20_000:1500 + 40_000] = ix.corpus[1500:1500 + 20_000]
    if scheme != "cluster":
        ix.scale_A_columns = torch.from_numpy(rng.uniform(0.5, 2.0, (7, r)).astype(np.float32)) * 1e-3
        ix.scale_B_points = torch.ones(48_000)
        ix.scale_B_points[::3] = 1.25
    if scheme == "mixed":
        ix.first_row_A = torch.from_numpy(rng.normal(size=(7, r)).astype(np.float32))
        ix.first_row_B = torch.from_numpy((rng.integers(-3, 4, 48_000) / 4).astype(np.float32))
    queries = rng.standard_normal((nq, 32)).astype(np.float32)
    gix = B.Index.from_arrays(ix.to("cuda"))
    _, _, st = gix.search_stages(torch.from_numpy(queries).cuda(), 5, 5, m)
    some = np.concatenate([np.arange(0, nq, 16), np.arange(nq - 5, nq)])         # (the oracle on the CPU: a sample)
    _, _, ost = O.search(O.OracleIndex(ix.numpy()), queries[some], 5, 5, m, stages=True)
    st = {f: st[f][some] for f in ("cand_rows", "pmax")}
    np.testing.assert_array_equal(np.sort(st["cand_rows"].astype(np.int64), axis=1), np.sort(ost["cand_rows"], axis=1))
    np.testing.assert_array_equal(st["pmax"], ost["pair_best"])
    gix.close()


@pytest.mark.parametrize("metric,m,scheme", [(0, 10, "cluster"), (0, 352, "cluster"), (2, 353, "cluster"), (0, 864, "cluster"), (1, 352, "cluster"), (1, 700, "mixed"), (0, 300, "columns")])
def test_more_ties_than_the_list_holds(B, metric, m, scheme):
    """Thousands of points share the m-th score of nearly every query, a few hundred score higher: the list is cut back to the m best
    (ties to the lower rows) as often as it fills, and no query is handed to the exhaustive kernel."""
    ix = _index(metric, n=24_000, L=6, r=16, seed=5)
    ix.cluster_offsets[:] = torch.tensor([0, 9000, 9000, 13_000, 13_500, 17_600, 24_000])
    ix.B[:] = 1
    ix.B[7::90] = 100                                     # (a score is this code times the sum of the query's)
    ix.corpus[:] = ix.corpus / ix.corpus.norm(dim=1, keepdim=True)
    if metric == 1:
        ix.corpus[:] = ix.corpus[0]                       # equal norms to the last bit
    if scheme != "cluster":
        ix.scale_A_columns, ix.scale_B_points = torch.full((6, 16), 1e-3), torch.full((24_000,), 1.25)
    if scheme == "mixed":
        ix.first_row_A, ix.first_row_B = torch.full((6, 16), 0.5), torch.ones(24_000)
    queries = np.random.default_rng(m).standard_normal((2100, 32)).astype(np.float32)
    gix = B.Index.from_arrays(ix.to("cuda"))
    _, _, st = gix.search_stages(torch.from_numpy(queries).cuda(), 5, 4, m)
    gix.close()
    some = np.arange(0, 2100, 20)
    _, _, ost = O.search(O.OracleIndex(ix.numpy()), queries[some], 5, 4, m, stages=True)
    np.testing.assert_array_equal(np.sort(st["cand_rows"][some].astype(np.int64), axis=1), np.sort(ost["cand_rows"], axis=1))
    assert (st["n_survivors"] >= 0).all()


@pytest.mark.parametrize("m", [10, 400])
def test_scores_that_are_no_numbers(B, m):
    """Norms that are NaN with every bit set give scores with the largest key there is: each query still gets exactly m distinct rows."""
    ix = _index(1, n=12_000, L=6, r=16, seed=8)
    ix.cluster_offsets[:] = torch.tensor([0, 3000, 6000, 8000, 9000, 10_000, 12_000])
    ix.corpus[::5, 0] = torch.tensor([-1], dtype=torch.int32).view(torch.float32)
    queries = np.random.default_rng(m).standard_normal((2100, 32)).astype(np.float32)
    gix = B.Index.from_arrays(ix.to("cuda"))
    _, _, st = gix.search_stages(torch.from_numpy(queries).cuda(), 5, 6, m)
    gix.close()
    rows = np.sort(st["cand_rows"], axis=1)
    assert rows.min() >= 0 and rows.max() < 12_000 and (rows[:, 1:] > rows[:, :-1]).all()


@pytest.mark.parametrize("m", [250, 700])
def test_points_of_infinite_norm_fill_up_the_candidates(B, m):
    """Squared Euclidean, most points of a large cluster with a norm beyond the float range (score -inf): with fewer finite scores than
    candidates asked for, the lowest rows of the others follow, also where the walk goes by the best scores of quarters."""
    ix = _index(1, n=43_000, L=2, r=16, seed=13)
    ix.cluster_offsets[:] = torch.tensor([0, 41_111, 43_000])
    far = torch.ones(43_000, dtype=torch.bool)
    far[130::137] = False                                 # 300 of the large cluster, 13 of the other
    ix.corpus[far] *= 1e20
    queries = np.random.default_rng(m).standard_normal((2100, 32)).astype(np.float32)
    gix = B.Index.from_arrays(ix.to("cuda"))
    q = torch.from_numpy(queries).cuda()
    _, _, st = gix.search_stages(q, 5, 1, m)
    gix.set_exact_selection(True)
    _, _, e_st = gix.search_stages(q, 5, 1, m)
    gix.close()
    np.testing.assert_array_equal(np.sort(st["cand_rows"], axis=1), np.sort(e_st["cand_rows"], axis=1))
