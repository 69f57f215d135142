"""The screened re-rank (all candidates at half width, the few that can matter in full) against the kernel that evaluates every
candidate of one query per block: bit-identical results (needs an MI355X)."""
import numpy as np
import pytest
import torch

from oracle import oracle as O
from tests.parity_util import assert_topk_equal, oracle_distance_of, rounding_abs_tol
from tests.test_gpu_parity import _random_index

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def B():
    from paper_2410_18926_amd import binding
    assert torch.cuda.is_available(), "these tests need the GPU"
    return binding


# row lengths around the k-steps of 32, the register slices of 256 and their limits; candidate counts around the group sizes (16, 10,
# 4, 1 queries), the wavefront and the block finish; k at the edge of the rule (4 k <= m); batches that end inside a group
CASES = [(1, 0, 70, 100, 25), (3, 1, 65, 204, 10), (31, 2, 200, 205, 10), (32, 0, 129, 64, 16), (33, 1, 100, 300, 7), (255, 1, 90, 256, 64),
         (256, 0, 333, 257, 10), (301, 2, 81, 777, 100), (516, 1, 66, 512, 128), (768, 0, 500, 200, 10), (768, 2, 30, 513, 1), (1023, 1, 70, 1024, 200),
         (1024, 2, 111, 300, 10), (1028, 0, 66, 1025, 9), (1029, 1, 20, 1638, 11), (2000, 0, 70, 200, 10), (2050, 2, 67, 40, 10), (64, 1, 80, 4096, 1000),
         (64, 0, 1, 600, 10), (96, 2, 9, 60, 15)]


@pytest.mark.parametrize("half", [False, True])
@pytest.mark.parametrize("d,metric,nq,m,k", CASES)
def test_same_bits_as_the_plain_rerank(B, d, metric, nq, m, k, half):
    rng = np.random.default_rng(31 * d + metric)
    dp = 16 if d < 32 else 32
    ix = _random_index(rng, n=7000, d=max(d, 16) if d < 16 else d, L=9, r=8, metric=metric, dp=dp)
    d = ix["d"]
    if metric != 2:       # heavy-tailed norms, elements in binary16's subnormal range, rows that are all zero
        ix["corpus"] = (ix["corpus"] * np.exp(rng.normal(size=(7000, 1)) * 1.5)).astype(np.float32)
        ix["corpus"][::53, ::3] *= np.float32(1e-6)
        ix["corpus"][::701] = 0
    ix["corpus"][1::2] = ix["corpus"][0::2] * np.float32(1 + 2.0 ** -9 if metric == 0 else 1)      # near-ties and ties
    q = rng.normal(size=(nq, d)).astype(np.float32)
    q[::7] *= np.float32(1e-4)
    q[nq // 2] = 0
    if nq > 3:
        q[3] = ix["corpus"][4242]
    gix = B.Index(**ix)
    if half:
        gix.set_rerank(B.RERANK_F16)
    gix.set_rerank_screening(B.RERANK_SCREEN_ALWAYS)
    s_ids, s_d = gix.search(q, k, 6, m)
    assert gix.profile_gather_plan()[1] == (nq > 64 or m > 512 or d > 1536)      # (small batches share full rows where they can)
    gix.set_exact_selection(True)
    e_ids, e_d = gix.search(q, k, 6, m)
    gix.set_exact_selection(False)
    np.testing.assert_array_equal(s_ids, e_ids)
    np.testing.assert_array_equal(s_d, e_d)
    a = O.with_half_precision_corpus(ix) if half else ix
    o_ids, o_d = O.search(O.OracleIndex(a), q, k, 6, m)
    rows = a.get("rerank_corpus", ix["corpus"])
    assert_topk_equal(s_ids, s_d, o_ids, o_d, f"d={d} metric={metric}", abs_tol=rounding_abs_tol(q, rows, metric) + (1e-6 if metric == 2 else 0.0),
                      exact=oracle_distance_of(ix, q, rows))
    gix.close()


# beyond 2048 queries one wavefront finishes a query (m <= 512; four above): every register slice, rows that are and are not a multiple of
# four elements, both candidate budgets, a ragged last block
WIDE = [(50, 2, 257, 10), (128, 1, 100, 10), (255, 0, 200, 40), (301, 1, 300, 7), (516, 0, 256, 12), (768, 0, 200, 10), (1023, 1, 512, 60), (1024, 2, 300, 10),
        (1028, 1, 200, 10), (2001, 0, 60, 15), (96, 0, 700, 100)]


@pytest.mark.parametrize("half", [False, True])
@pytest.mark.parametrize("d,metric,m,k", WIDE)
def test_same_bits_in_large_batches(B, d, metric, m, k, half):
    rng = np.random.default_rng(77 * d + metric)
    ix = _random_index(rng, n=5000, d=d, L=9, r=8, metric=metric, dp=32)
    if metric != 2:
        ix["corpus"] = (ix["corpus"] * np.exp(rng.normal(size=(5000, 1)) * 0.5)).astype(np.float32)
    ix["corpus"][1::2] = ix["corpus"][0::2] * np.float32(1 + 2.0 ** -9 if metric == 0 else 1)      # near-ties and ties
    q = torch.from_numpy(rng.normal(size=(2051, d)).astype(np.float32)).cuda()
    gix = B.Index(**ix)
    if half:
        gix.set_rerank(B.RERANK_F16)
    gix.set_rerank_screening(B.RERANK_SCREEN_ALWAYS)
    s_ids, s_d = gix.search(q, k, 4, m)
    assert gix.profile_gather_plan()[1]
    gix.set_exact_selection(True)
    e_ids, e_d = gix.search(q, k, 4, m)
    gix.close()
    assert torch.equal(s_ids, e_ids) and torch.equal(s_d, e_d)


def test_queries_that_are_no_numbers_keep_every_candidate(B):
    """An infinite or NaN query gives bounds that are no numbers: nothing may be dropped for the other queries of its group, and the call ends."""
    rng = np.random.default_rng(5)
    ix = _random_index(rng, n=3000, d=64, L=6, r=8, metric=0, dp=32)
    q = rng.normal(size=(70, 64)).astype(np.float32)
    clean = q.copy()
    q[11, 3], q[40, 9] = np.nan, np.inf
    q[50] *= np.float32(1e30)
    q[51] *= np.float32(1e-30)
    gix = B.Index(**ix)
    gix.set_rerank_screening(B.RERANK_SCREEN_ALWAYS)
    ids, dist = gix.search(q, 5, 3, 100)
    assert gix.profile_gather_plan()[1]
    ref_ids, ref_d = gix.search(clean, 5, 3, 100)
    good = np.setdiff1d(np.arange(70), [11, 40, 50, 51])
    np.testing.assert_array_equal(ids[good], ref_ids[good])
    np.testing.assert_array_equal(dist[good], ref_d[good])
    gix.set_exact_selection(True)
    e_ids, e_d = gix.search(q[50:52], 5, 3, 100)
    np.testing.assert_array_equal(ids[50:52], e_ids)
    np.testing.assert_array_equal(dist[50:52], e_d)
    gix.close()


@pytest.mark.parametrize("nq", [65, 67, 400, 401, 4097, 5003])
def test_few_queries_per_cluster(B, nq):
    """Up to two queries per cluster the groups are smaller (4 queries; 5 from 4097 on where the clusters are that many): batches
    that end inside a group and on both sides of the rule, against the plain re-rank."""
    L = 2600 if nq > 4000 else 200
    rng = np.random.default_rng(nq)
    ix = _random_index(rng, n=9000, d=48, L=L, r=8, metric=nq % 3, dp=32)
    q = rng.normal(size=(nq, 48)).astype(np.float32)
    gix = B.Index(**ix)
    gix.set_rerank_screening(B.RERANK_SCREEN_ALWAYS)
    s_ids, s_d = gix.search(q, 10, 40, 100)
    assert gix.profile_gather_plan() == (4 if nq <= 4096 else 5, True) or nq > 2 * L
    gix.set_exact_selection(True)
    e_ids, e_d = gix.search(q, 10, 40, 100)
    np.testing.assert_array_equal(s_ids, e_ids)
    np.testing.assert_array_equal(s_d, e_d)
    gix.close()


@pytest.mark.parametrize("half", [False, True])
@pytest.mark.parametrize("metric,scales", [(0, (3e36, 1e37, 3e37)), (1, (1e18, 2e18, 4e18, 1e20, 1e24)), (2, (2e18, 3e18, 1e20, 1e30))])
def test_distances_that_overflow_tie_by_id(B, metric, scales, half):
    """Queries so long that an exact distance - or the norm a cosine is divided by - is infinite in float: the plain re-rank then
    orders many candidates by their id, and so must the screened one, whose scaled products stay finite."""
    rng = np.random.default_rng(40 + metric)
    ix = _random_index(rng, n=4000, d=64, L=6, r=8, metric=metric, dp=32)
    ix["scale_A"] = (ix["scale_A"] * 1e-6).astype(np.float32)            # (the estimated scores stay finite)
    q = rng.normal(size=(70, 64)).astype(np.float32)
    if metric == 0:       # positive elements: sums run into +inf, never into inf - inf
        ix["corpus"] = (np.abs(ix["corpus"]) * np.exp(rng.normal(size=(4000, 1)))).astype(np.float32)
        q = np.abs(q)
    for i, s in enumerate(scales):
        q[i::len(scales) + 1] *= np.float32(s)
    gix = B.Index(**ix)
    if half:
        gix.set_rerank(B.RERANK_F16)
    gix.set_rerank_screening(B.RERANK_SCREEN_ALWAYS)
    s_ids, s_d = gix.search(q, 10, 4, 100)
    assert gix.profile_gather_plan()[1]
    gix.set_exact_selection(True)
    e_ids, e_d = gix.search(q, 10, 4, 100)
    gix.close()
    np.testing.assert_array_equal(s_d, e_d)
    np.testing.assert_array_equal(s_ids, e_ids)
    tied = (e_d[:, 1:] == e_d[:, :-1]).all(axis=1)
    assert tied.any() and not tied.all()


@pytest.mark.parametrize("metric,nq,m,w", [(0, 32768, 4096, 6), (1, 16384, 2000, 4)])
def test_search_without_room_for_the_screening_lists(B, metric, nq, m, w):
    """Little free memory: the lists of the screened re-rank (and the quarter maxima) do not fit beside what every search needs.  The search then
    goes without them, on this call and on later ones, with the same results."""
    rng = np.random.default_rng(m)
    ix = _random_index(rng, n=24_000, d=32, L=6, r=8, metric=metric)
    q = torch.from_numpy(rng.normal(size=(nq, 32)).astype(np.float32)).cuda()
    ref = B.Index(**ix)
    r_ids, r_d = ref.search(q, 10, w, m)
    ref.close()
    gix = B.Index(**ix)
    outs = [(torch.empty(nq, 10, dtype=torch.int64, device="cuda"), torch.empty(nq, 10, device="cuda")) for _ in range(3)]
    torch.cuda.empty_cache()
    needed = int(1.3 * (nq * (m * 4 + 500) + (32 << 20)))        # candidates and the small buffers, with the workspace's slack of 1/8
    free = torch.cuda.mem_get_info()[0]
    assert free > needed
    hog = torch.empty(free - needed, dtype=torch.uint8, device="cuda")
    try:
        gix.search(q, 10, w, m, out=outs[0])
        gix.search(q, 10, w, m, out=outs[1], asynchronous=True)
        gix.search(q[:500], 10, w, m, out=(outs[2][0][:500], outs[2][1][:500]))       # small enough for the lists
        torch.cuda.synchronize()
    finally:
        del hog
        torch.cuda.empty_cache()
    for ids, d in outs[:2]:
        assert torch.equal(ids, r_ids) and torch.equal(d, r_d)
    assert torch.equal(outs[2][0][:500], r_ids[:500]) and torch.equal(outs[2][1][:500], r_d[:500])
    gix.close()


@pytest.mark.parametrize("what,metric,screened", [("plain", 0, True), ("plain", 1, True), ("plain", 2, True), ("mean", 0, False), ("mean", 1, False),
                                                  ("one long row", 0, False), ("one row near zero", 1, False)])
@pytest.mark.parametrize("half", [False, True])
def test_screening_is_left_out_where_its_bound_keeps_everything(B, what, metric, screened, half):
    """A mean of a thousand times the spread, one row a thousand times as long as the others (inner product), one row whose elements are all
    subnormal in binary16 (Euclidean): the bound excludes hardly a candidate, which the search of a sample at load finds out.  The three
    settings give the same results."""
    rng = np.random.default_rng(17 + metric)
    ix = _random_index(rng, n=20_000, d=96, L=12, r=8, metric=metric, dp=32)
    q = rng.normal(size=(300, 96)).astype(np.float32)
    if what == "mean":
        ix["corpus"] = ix["corpus"] + np.float32(1000)
        q = q + np.float32(1000)
    elif what == "one long row":
        ix["corpus"][12_345] *= np.float32(1000)
    elif what == "one row near zero":
        ix["corpus"][12_345] = np.float32(3e-5) * np.sign(ix["corpus"][12_345])
    gix = B.Index(**ix)
    if half:
        gix.set_rerank(B.RERANK_F16)
    a_ids, a_d = gix.search(q, 10, 5, 200)
    assert gix.profile_gather_plan()[1] == screened
    for mode in (B.RERANK_SCREEN_ALWAYS, B.RERANK_SCREEN_NEVER):
        gix.set_rerank_screening(mode)
        ids, d = gix.search(q, 10, 5, 200)
        assert gix.profile_gather_plan()[1] == (mode == B.RERANK_SCREEN_ALWAYS)
        np.testing.assert_array_equal(ids, a_ids)
        np.testing.assert_array_equal(d, a_d)
    gix.close()


def test_the_half_precision_copy_is_given_back(B):
    """NEVER frees the copy, the other settings and the half-precision re-rank make it again."""
    rng = np.random.default_rng(3)
    ix = _random_index(rng, n=200_000, d=128, L=40, r=8, metric=1)
    q = rng.normal(size=(100, 128)).astype(np.float32)
    gix = B.Index(**ix)
    copy = 200_000 * 128 * 2
    ids, d = gix.search(q, 10, 5, 100)
    free = torch.cuda.mem_get_info()[0]
    gix.set_rerank_screening(B.RERANK_SCREEN_NEVER)
    assert torch.cuda.mem_get_info()[0] - free > 0.9 * copy
    n_ids, n_d = gix.search(q, 10, 5, 100)
    gix.set_rerank(B.RERANK_F16)
    h_ids, _ = gix.search(q, 10, 5, 100)
    assert (h_ids == ids).mean() > 0.9 and not gix.profile_gather_plan()[1]
    gix.set_rerank(B.RERANK_F32)
    assert torch.cuda.mem_get_info()[0] - free > 0
    gix.set_rerank_screening(B.RERANK_SCREEN_AUTO)
    a_ids, a_d = gix.search(q, 10, 5, 100)
    for i, x in ((n_ids, n_d), (a_ids, a_d)):
        np.testing.assert_array_equal(i, ids)
        np.testing.assert_array_equal(x, d)
    with pytest.raises(B.LorannError):
        gix.set_rerank_screening(3)
    gix.close()


@pytest.mark.parametrize("nq,screened", [(2, False), (64, False), (65, True)])
def test_a_few_dozen_queries_share_full_rows(B, nq, screened):
    """Whatever the kernels in front of it - column-wise step sizes take the batched ones at any size - up to 64 queries are not screened."""
    rng = np.random.default_rng(nq)
    ix = _random_index(rng, n=5000, d=64, L=6, r=8, metric=0, dp=32)
    ix["scale_A_columns"] = rng.uniform(0.01, 0.1, (6, 8)).astype(np.float32)
    ix["scale_B_points"] = rng.uniform(0.01, 0.1, 5000).astype(np.float32)
    q = rng.normal(size=(nq, 64)).astype(np.float32)
    gix = B.Index(**ix)
    gix.set_rerank_screening(B.RERANK_SCREEN_ALWAYS)
    ids, d = gix.search(q, 10, 4, 100)
    assert gix.profile_gather_plan()[1] == screened
    gix.set_exact_selection(True)
    e_ids, e_d = gix.search(q, 10, 4, 100)
    gix.close()
    np.testing.assert_array_equal(ids, e_ids)
    np.testing.assert_array_equal(d, e_d)
