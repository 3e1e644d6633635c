"""Search with derived quantizers (chapter 6, Alg. 5) on the GPU against the oracle.

Stage-wise bit-exactness: the compact float tables are taken from the GPU (pq_build_luts, the same
kernel the search runs inside) and handed to the oracle, so that qmax, the 8-bit tables, every
integer distance, the bucket b* and the candidate set must agree bit for bit; the precise distances
of Step 2 agree within 1e-5 and the final ids up to ties inside that tolerance."""
import numpy as np
import pytest
import torch

from oracle import derived_oracle as dq
from oracle import pq_oracle as orc
from paper_1712_02912_amd import binding
from util import check_float_topk_ranked

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    c = binding.Context(0)
    yield c
    torch.cuda.synchronize()
    c.close()


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def make_problem(seed, n, k, dsub, nq, distinct=None):
    """Codebooks with property P1 by construction (index low byte = cluster), random codes."""
    r = np.random.default_rng(seed)
    m, kbar = 4, 256
    centres = r.normal(size=(m, kbar, dsub)) * 4
    cb = (centres[:, np.arange(k) % kbar, :] + r.normal(size=(m, k, dsub)) * 0.7).astype(np.float32)
    cbar = np.stack([np.stack([cb[j, l::kbar].astype(np.float64).mean(0) for l in range(kbar)]) for j in range(m)])
    if distinct:
        pool = r.integers(0, k, (distinct, m))
        codes = pool[r.integers(0, distinct, n)].astype(np.uint16)
    else:
        codes = r.integers(0, k, (n, m)).astype(np.uint16)
    queries = (r.normal(size=(nq, m * dsub)) * 4).astype(np.float32)
    return cb, cbar.astype(np.float32), codes, queries


def run_case(ctx, cb, cbar, codes, queries, r2, topk):
    n, nq = len(codes), len(queries)
    d_cbar, d_cb, d_q = dev(cbar), dev(cb), dev(queries)
    d_codes = dev(codes.view(np.int16)) if n else torch.empty((0, 4), dtype=torch.int16, device="cuda")
    # oracle from the GPU's compact tables
    dluts = ctx.pq_build_luts(d_q, d_cbar)
    torch.cuda.synchronize()
    dluts = dluts.cpu().numpy()
    np.testing.assert_allclose(dluts, orc.build_luts(queries, cbar), rtol=1e-5, atol=1e-30)
    qmax = dq.derived_qmax(codes, dluts, r2)
    qluts, _, _ = orc.quantize_luts(dluts, qmax)
    od, oi, s_star, cands = dq.search_from_tables(codes, qluts, cb, queries, r2, topk)
    cap = max([len(c) for c in cands] + [1])
    gd, gi, bucket, ncand, cand = ctx.pq_derived_search(d_codes, d_cbar, d_cb, d_q, r2, topk, cand_cap=cap)
    torch.cuda.synchronize()
    gd, gi, bucket, ncand, cand = (t.cpu().numpy() for t in (gd, gi, bucket, ncand, cand))
    for q in range(nq):
        assert ncand[q] == len(cands[q]), f"query {q}: candidate count"
        if n:
            assert bucket[q] == s_star[q], f"query {q}: bucket"
        got = np.sort(cand[q][:ncand[q]])
        assert np.array_equal(got, cands[q]), f"query {q}: candidate set"
        assert np.all(cand[q][ncand[q]:] == -1)
        check_float_topk_ranked(gd[q], gi[q], od[q], oi[q])
    return ncand


def test_derived_search_several_tiles_ragged_tail_two_query_groups(ctx):
    cb, cbar, codes, queries = make_problem(3, 50_003, 1024, 8, 13)
    ncand = run_case(ctx, cb, cbar, codes, queries, 500, 10)
    assert ncand.min() >= 500
    # the same context again with a smaller problem (workspace kept, counters reset)
    run_case(ctx, cb, cbar, codes[:4097], queries[:3], 64, 5)


def test_derived_search_short_subvectors_direct_tables_kernel(ctx):
    cb, cbar, codes, queries = make_problem(5, 20_000, 512, 4, 9)
    run_case(ctx, cb, cbar, codes, queries, 300, 20)


@pytest.mark.parametrize("n,r2,topk", [(300, 1000, 10), (5000, 1, 1), (129, 129, 128), (2048, 2048, 7), (1, 5, 3)])
def test_derived_search_edges(ctx, n, r2, topk):
    cb, cbar, codes, queries = make_problem(7 + n, n, 768, 8, 4)
    run_case(ctx, cb, cbar, codes, queries, r2, topk)


def test_derived_search_empty_database(ctx):
    cb, cbar, codes, queries = make_problem(9, 0, 256, 8, 3)
    gd, gi, bucket, ncand, _ = ctx.pq_derived_search(torch.empty((0, 4), dtype=torch.int16, device="cuda"), dev(cbar),
                                                     dev(cb), dev(queries), 10, 4)
    torch.cuda.synchronize()
    assert torch.isinf(gd).all() and (gi == -1).all() and (ncand == 0).all()


def test_derived_search_huge_buckets_of_identical_codes(ctx):
    """40 distinct codes only: the bucket of the r2-th vector holds thousands of vectors, all of
    them candidates; precise distances tie massively and ids decide."""
    cb, cbar, codes, queries = make_problem(11, 60_000, 1024, 8, 10, distinct=40)
    ncand = run_case(ctx, cb, cbar, codes, queries, 700, 50)
    assert ncand.max() > 1400


def test_derived_search_full_size_codebooks(ctx):
    """k = 65536 centroids of 32 dimensions per sub-quantizer (d = 128), as in Section 6.3."""
    cb, cbar, codes, queries = make_problem(13, 200_000, 65536, 32, 16)
    run_case(ctx, cb, cbar, codes, queries, 2000, 100)


def test_derived_search_descending_order_worst_case_for_the_bound(ctx):
    """Codes ordered from far to near for query 0: every vector passes the bound of its time."""
    cb, cbar, codes, queries = make_problem(15, 40_000, 1024, 8, 2)
    dl = orc.build_luts(queries[:1], cbar)[0]
    low = (codes & 255).astype(np.int64)
    dist = sum(dl[j][low[:, j]].astype(np.float64) for j in range(4))
    codes = codes[np.argsort(-dist, kind="stable")]
    run_case(ctx, cb, cbar, codes, queries, 400, 10)


def test_derived_search_errors(ctx):
    cb, cbar, codes, queries = make_problem(17, 3000, 256, 8, 2)
    args = (dev(codes.view(np.int16)), dev(cbar), dev(cb), dev(queries))
    with pytest.raises(binding.PqError) as e:
        ctx.pq_derived_search(*args, 500, 10, cand_cap=100)     # every query has at least 500 candidates
    assert e.value.code == -2
    with pytest.raises(binding.PqError) as e:
        ctx.pq_derived_search(*args, 500, 200)                  # topk above 128
    assert e.value.code == -3
    with pytest.raises(binding.PqError) as e:
        ctx.pq_derived_search(*args, 0, 10)                     # r2 < 1
    assert e.value.code == -1
    z = lambda *s, dt=torch.float32: torch.zeros(s, dtype=dt, device="cuda")
    with pytest.raises(binding.PqError) as e:                   # m = 8 is outside the covered shapes
        ctx.pq_derived_search(z(10, 8, dt=torch.int16), z(8, 256, 4), z(8, 256, 4), z(1, 32), 5, 2)
    assert e.value.code == -3
    # the context still works after the errors
    run_case(ctx, cb, cbar, codes, queries, 100, 10)


def test_derived_search_bench_configuration_sampled(ctx):
    """The workload bench.py --derived times (25 M codes, 1000 queries, k = 65536, r2 = 10000, top-100):
    bucket, candidate count, candidate set and result of three sampled queries against the oracle."""
    from paper_1712_02912_amd import datagen
    mix = datagen.sift_like()
    n, nq, r2, topk = 25_000_000, 1000, 10000, 100
    cb, cbar = datagen.clustered_codebooks(mix, 4, 65536)
    queries = mix.sample(nq, datagen.SEED_QUERIES)
    gen = torch.Generator(device="cuda").manual_seed(datagen.SEED_CODES + 5)
    d_codes = torch.randint(-32768, 32768, (n, 4), dtype=torch.int16, device="cuda", generator=gen)
    d_cbar, d_cb, d_q = dev(cbar), dev(cb), dev(queries)
    cap = 40000
    gd, gi, bucket, ncand, cand = ctx.pq_derived_search(d_codes, d_cbar, d_cb, d_q, r2, topk, cand_cap=cap)
    dluts = ctx.pq_build_luts(d_q, d_cbar)
    torch.cuda.synchronize()
    codes = d_codes.cpu().numpy().view(np.uint16)
    dluts = dluts.cpu().numpy()
    sample = [0, 499, 999]
    qmax = dq.derived_qmax(codes, dluts[sample], r2)
    qluts, _, _ = orc.quantize_luts(dluts[sample], qmax)
    od, oi, s_star, cands = dq.search_from_tables(codes, qluts, cb, queries[sample], r2, topk)
    gd, gi, bucket, ncand = gd.cpu().numpy(), gi.cpu().numpy(), bucket.cpu().numpy(), ncand.cpu().numpy()
    assert ncand.min() >= r2 and ncand.max() <= cap
    for i, q in enumerate(sample):
        assert bucket[q] == s_star[i] and ncand[q] == len(cands[i])
        assert np.array_equal(np.sort(cand[q, :ncand[q]].cpu().numpy()), cands[i])
        check_float_topk_ranked(gd[q], gi[q], od[i], oi[i])


# ------------------------------------------------------------ 640 queries and more: 16 queries per pass over the codes
# (the last case has more queries than the 1024 that the offsets of the candidate lists are summed over at a time)
@pytest.mark.parametrize("n,nq,r2,topk", [(30_003, 650, 300, 10), (8_193, 641, 2000, 50), (300, 640, 1000, 5),
                                          (70_001, 777, 64, 128), (4_001, 2_301, 150, 5)])
def test_derived_search_many_queries(ctx, n, nq, r2, topk):
    cb, cbar, codes, queries = make_problem(21 + n, n, 1024, 8, nq)
    run_case(ctx, cb, cbar, codes, queries, r2, topk)


def test_derived_search_many_queries_identical_codes_and_worst_case_order(ctx, opts):
    # 40 distinct codes: buckets of thousands of vectors, all candidates
    cb, cbar, codes, queries = make_problem(23, 40_000, 1024, 8, 643, distinct=40)
    ncand = run_case(ctx, cb, cbar, codes, queries, 700, 20)
    assert ncand.max() > 1400
    # far to near for query 0: every vector passes the bound of its time
    cb, cbar, codes, queries = make_problem(25, 40_000, 1024, 8, 640)
    dl = orc.build_luts(queries[:1], cbar)[0]
    low = (codes & 255).astype(np.int64)
    dist = sum(dl[j][low[:, j]].astype(np.float64) for j in range(4))
    codes = codes[np.argsort(-dist, kind="stable")]
    run_case(ctx, cb, cbar, codes, queries, 400, 10)
    # the 8-query kernel for the same input (switch)
    opts.set("scan_q8", 0)
    run_case(ctx, cb, cbar, codes, queries, 400, 10)


@pytest.mark.parametrize("dsub,nq,n,r2,topk,shift", [(5, 3, 3001, 1024, 7, 0), (32, 2, 40_000, 33_000, 128, 1), (33, 1, 5000, 2049, 1, 0),
                                                     (36, 17, 2500, 1025, 100, 0), (1, 2, 300, 64, 3, 0)])
def test_derived_search_rerank_pieces(ctx, dsub, nq, n, r2, topk, shift):
    """Step 2 at the edges of its pieces (512 candidates) and tiles (1024) and rows: dimensions below, at and above the 32 that eight
    lanes read at once, rows that do not start on 16 bytes, lists of several pieces, a handful of candidates."""
    cb, cbar, codes, queries = make_problem(dsub * 7 + nq, n, 512, dsub, nq, distinct=200 if nq == 17 else None)
    if shift:   # codebooks that start on 4 bytes only
        buf = torch.empty(cb.size + 4, device="cuda")
        d_cb = buf[shift:shift + cb.size].view(*cb.shape)
        d_cb.copy_(torch.from_numpy(cb))
        args = dev(codes.view(np.int16)), dev(cbar), d_cb, dev(queries)
        plain = ctx.pq_derived_search(args[0], args[1], dev(cb), args[3], r2, topk)
        moved = ctx.pq_derived_search(*args, r2, topk)
        assert torch.equal(plain[0], moved[0]) and torch.equal(plain[1], moved[1])
    run_case(ctx, cb, cbar, codes, queries, r2, topk)


@pytest.mark.parametrize("dsub,k,nq,n,r2,topk", [(8, 256, 129, 4000, 300, 17), (32, 1024, 5, 70_000, 60_000, 100), (12, 300, 260, 2100, 2100, 128), (8, 65536, 300, 1500, 400, 20)])
def test_derived_search_rerank_on_complete_tables(ctx, opts, dsub, k, nq, n, r2, topk):
    """The queries' complete tables, as for lists that are long for the number of centroids: ragged pieces, one and
    several dies' shares, more queries than a block takes and, with 65 536 centroids, than one batch of tables."""
    cb, cbar, codes, queries = make_problem(dsub + nq, n, k, dsub, nq)
    opts.set("derived_tables", 1)
    run_case(ctx, cb, cbar, codes, queries, r2, topk)


def exact_case(ctx, cb, cbar, codes, queries, topk):
    """Every code is a candidate (r2 = n): distances and rows of Step 2 exactly as the oracle has them."""
    with np.errstate(over="ignore"):   # (infinite components: infinite distances)
        want = [dq.rerank_exact(codes, np.arange(len(codes)), cb, y, topk) for y in queries]
    gd, gi = ctx.pq_derived_search(dev(codes.view(np.int16)), dev(cbar), dev(cb), dev(queries), len(codes), topk)[:2]
    torch.cuda.synchronize()
    assert np.array_equal(gd.cpu().numpy(), np.stack([w[0] for w in want]))
    assert np.array_equal(gi.cpu().numpy(), np.stack([w[1] for w in want]))
    return gd, gi


@pytest.mark.parametrize("dsub", [8, 32, 60])
@pytest.mark.parametrize("nq", [1, 40, 129])
def test_derived_search_rerank_near_hits(ctx, opts, nq, dsub):
    """Queries that nearly hit a vector (5e-5 of its length away): the terms are sums of squared differences in double, where
    norms and products of that size would have lost the distance.  The same bits for a query alone and among others."""
    cb, cbar, codes, _ = make_problem(nq + dsub, 3000, 1024, dsub, 1)
    near = cb[np.arange(4)[None, :], codes[:nq].astype(np.int64)].reshape(nq, 4 * dsub)
    queries = (near * np.float32(1 + 5e-5)).astype(np.float32)
    opts.set("derived_tables", 1)
    gd, gi = exact_case(ctx, cb, cbar, codes, queries, 20)
    opts.set("derived_tables", 0)
    assert np.array_equal(gi[:, 0].cpu().numpy(), np.arange(nq))
    for q in (0, nq - 1):
        d1, i1 = exact_case(ctx, cb, cbar, codes, queries[q:q + 1], 20)
        assert torch.equal(d1[0], gd[q]) and torch.equal(i1[0], gi[q])


@pytest.mark.parametrize("tables", [0, 1])
def test_derived_search_rerank_infinite_components(ctx, opts, tables):
    """Centroids with infinite components: their codes are infinitely far and stand behind the finite ones, by row."""
    cb, cbar, codes, queries = make_problem(31, 120, 256, 32, 130)
    cb[1, 7, 3] = np.inf
    cb[2, 9, 31] = -np.inf
    codes[::3, 1] = 7
    codes[1::7, 2] = 9
    opts.set("derived_tables", tables)
    gd, _ = exact_case(ctx, cb, cbar, codes, queries, 128)
    assert torch.isinf(gd[:, 60:]).any() and not torch.isnan(gd).any()


@pytest.mark.parametrize("dsub,nq,n,r2", [(8, 3, 3000, 1024), (32, 9, 20_000, 5000), (36, 650, 4000, 900), (7, 650, 2500, 300), (60, 2, 5000, 5000)])
def test_derived_search_forms_of_step_2(ctx, opts, dsub, nq, n, r2):
    """Complete tables or centroid rows, codes copied beside the lists or read from the database (what calls short of memory
    take): the same distances and rows bit for bit, and those of the oracle."""
    cb, cbar, codes, queries = make_problem(dsub + nq, n, 512, dsub, nq)
    first = None
    for tables, copies in ((0, 1), (1, 1), (1, 0), (0, 0)):
        opts.set("derived_tables", tables)
        opts.set("derived_code_copy", copies)
        if first is None or not copies:
            run_case(ctx, cb, cbar, codes, queries, r2, 20)
        got = ctx.pq_derived_search(dev(codes.view(np.int16)), dev(cbar), dev(cb), dev(queries), r2, 20)[:2]
        first = first or got
        assert torch.equal(got[0], first[0]) and torch.equal(got[1], first[1]), (tables, copies)


@pytest.mark.parametrize("n,nq", [(300_000_000, 8), (3_400_000, 640)])
def test_derived_search_lists_beyond_two_to_the_31(ctx, n, nq):
    """Equal codes, all of them candidates of every query: more than 2^31 places in the candidate lists (8 and 16 queries per
    pass over the codes); the first rows are the result, and every list holds every row once."""
    cb, cbar, codes, queries = make_problem(43, 1, 256, 8, nq)
    d_codes = torch.empty((n, 4), dtype=torch.int16, device="cuda")
    d_codes[:] = dev(codes.view(np.int16))[0]
    big = binding.Context(0)   # (its lists are given back at the end)
    cap = n if nq == 640 else 0
    gd, gi, _, ncand, cand = big.pq_derived_search(d_codes, dev(cbar), dev(cb), dev(queries), 1000, 10, cand_cap=cap)
    torch.cuda.synchronize()
    big.close()
    assert n * nq > 2**31 and (ncand == n).all()
    for q in (0, nq - 1):
        assert np.array_equal(gi[q].cpu().numpy(), np.arange(10))
        assert (gd[q] == float(dq.rerank_exact(codes, np.zeros(1, np.int64), cb, queries[q], 1)[0][0])).all()
        if cap:
            assert torch.equal(cand[q].sort().values, torch.arange(n, device="cuda"))
    del d_codes, cand
    torch.cuda.empty_cache()


def test_derived_search_every_code_of_a_full_bucket(ctx):
    """Nearly 2^32 equal codes in one bucket: all of them are candidates, the first rows are the result."""
    n = 2**32 - 100
    if torch.cuda.mem_get_info()[0] < 150 << 30:
        pytest.skip("needs 150 GB of device memory")
    cb, cbar, codes, queries = make_problem(41, 1, 256, 8, 1)
    d_codes = torch.empty((n, 4), dtype=torch.int16, device="cuda")
    d_codes[:] = dev(codes.view(np.int16))[0]
    big = binding.Context(0)   # (its lists are given back at the end)
    gd, gi, _, ncand, _ = big.pq_derived_search(d_codes, dev(cbar), dev(cb), dev(queries), 1000, 10)
    torch.cuda.synchronize()
    big.close()
    del d_codes
    torch.cuda.empty_cache()
    want = dq.rerank_exact(codes, np.zeros(1, np.int64), cb, queries[0], 1)[0][0]
    assert ncand[0].item() == n
    assert np.array_equal(gi.cpu().numpy()[0], np.arange(10)) and np.all(gd.cpu().numpy()[0] == want)


def sample_rows(n, r2):
    """Rows that the sample of pq_derived_search looks at (one of every `step`, picked by a hash of its number)."""
    step = min(r2 // 150, 16)
    i = np.arange(n // step, dtype=np.uint64)
    return (i * step + ((i * 2654435761) % 2 ** 32 >> 16) % step).astype(np.int64), step


@pytest.mark.parametrize("nq", [260, 645])
@pytest.mark.parametrize("order", ["random", "sorted", "equal", "sample_nearer", "sample_farther", "few_near"])
def test_derived_search_on_the_bounds_of_a_sample(ctx, opts, order, nq):
    """One collecting pass on the bounds of a sample against the two passes: the same distances, rows, buckets and candidate sets, also
    where the sample misleads (too few vectors up to its bucket, lists that do not fit) and the call falls back."""
    n, r2, topk = 330_007, 10_000, 20
    cb, cbar, codes, queries = make_problem(71, n, 512, 4, nq)
    rows, step = sample_rows(n, r2)
    if order == "sorted":
        codes = codes[np.lexsort(codes.T & 255)]
    if order == "equal":
        codes[:] = codes[17]
    if order != "random" and order != "sorted" and order != "equal":
        # `near`: codes of centroids close to all queries, whose scatter is small here
        queries = (queries * 1e-2).astype(np.float32)
        centre = queries.mean(0).reshape(4, 4)
        best = np.stack([((cbar[j] - centre[j]) ** 2).sum(1).argsort()[:4] for j in range(4)])
        r = np.random.default_rng(5)
        near = lambda count: np.stack([best[j][r.integers(0, 4, count)] for j in range(4)], 1).astype(np.uint16)
        if order == "sample_nearer":      # 900 near vectors, all of them in the sample, which takes them for 14 400
            codes[rows[:900]] = near(900)
        if order == "sample_farther":     # the vectors between the sample's near ones and the rest are near too: 16 times its estimate and more
            codes[:] = near(n)
            far = np.setdiff1d(rows, rows[::23])
            codes[far] = np.stack([((cbar[j] - centre[j]) ** 2).sum(1).argsort()[-4:][r.integers(0, 4, len(far))] for j in range(4)], 1)
        if order == "few_near":           # r2 - 1 near vectors, anywhere
            codes[r.permutation(n)[:r2 - 1]] = near(r2 - 1)
    args = (dev(codes.view(np.int16)), dev(cbar), dev(cb), dev(queries), r2, topk)
    opts.set("derived_sample", 0)
    two = [t.cpu().numpy() for t in ctx.pq_derived_search(*args)[:4]]
    cap = int(two[3].max())
    assert (two[3] >= r2).all()
    # the candidate sets, as sums over the rows of a hash each (all rows: up to 660 MB a call)
    def sets():
        out = ctx.pq_derived_search(*args, cand_cap=cap)
        ids = out[4]
        h = (ids + 1) * 2654435761 % 4294967291 * (ids >= 0)
        return [t.cpu().numpy() for t in out[:4]] + [h.sum(1).cpu().numpy(), (ids >= 0).sum(1).cpu().numpy()]
    ref = sets()
    opts.set("derived_sample", 1)
    ctx.pq_set_profiling(True)
    got = ctx.pq_derived_search(*args)[:4]
    kernel = ctx.pq_last_scan_info()["kernel"]
    ctx.pq_set_profiling(False)
    # the last scan that was timed: the sampled call's collecting pass, or the counting pass of the call that went back to two
    assert ("buckets of a sample" if order not in ("sample_nearer", "sample_farther") else "<count>") in kernel, kernel
    for got, want in zip(got, two):
        assert np.array_equal(got.cpu().numpy(), want)
    for got, want in zip(sets(), ref):
        assert np.array_equal(got, want)
    if cap > 0:
        with pytest.raises(RuntimeError, match="cand_cap"):
            ctx.pq_derived_search(*args, cand_cap=cap - 1)


def test_derived_search_without_memory_for_the_sample():
    """The sample is a convenience: a call that cannot have its memory makes the two passes."""
    ctx = binding.Context(0)
    n, nq, r2 = 1_320_011, 64, 450   # 440 003 codes of 8 bytes in the sample
    cb, cbar, codes, queries = make_problem(3, n, 512, 4, nq)
    args = (dev(codes.view(np.int16)), dev(cbar), dev(cb), dev(queries), r2, 10)
    ctx.pq_set_profiling(True)
    ctx.pq_set_option("alloc_limit_mib", 3)
    got = [t.cpu().numpy() for t in ctx.pq_derived_search(*args)[:4]]
    assert "<count>" in ctx.pq_last_scan_info()["kernel"]
    ctx.pq_set_option("alloc_limit_mib", None)
    sampled = [t.cpu().numpy() for t in ctx.pq_derived_search(*args)[:4]]
    assert "buckets of a sample" in ctx.pq_last_scan_info()["kernel"]
    for a, b in zip(got, sampled):
        assert np.array_equal(a, b)
    torch.cuda.synchronize()
    ctx.close()
