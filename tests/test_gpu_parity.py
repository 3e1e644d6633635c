"""Parity of the HIP path (through the C ABI) against the CPU oracle, element by element.

Float distances: 1e-5 relative, top-k sets identical up to ties inside that band.
Integer sums, quantised tables and ids: bit-exact.
"""
import math

import numpy as np
import pytest
import torch

from oracle import pq_oracle as orc
from paper_1712_02912_amd import binding, datagen
from util import RTOL, check_exact_topk, check_float_topk, sift_pq

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    c = binding.Context(0)
    yield c
    torch.cuda.synchronize()
    c.close()


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def host(t):
    torch.cuda.synchronize()
    return t.cpu().numpy()


# ----------------------------------------------------------------------------- Tables step
@pytest.mark.parametrize("m,k,d,nq", [(8, 256, 128, 16), (16, 16, 128, 37), (16, 256, 960, 21), (4, 7, 20, 3),
                                       (1, 256, 16, 1), (8, 1, 64, 5)])
def test_build_luts(ctx, m, k, d, nq):
    r = np.random.default_rng(m * 1000 + k)
    mix = datagen.sift_like() if d == 128 else None
    queries = mix.sample(nq, 5) if mix else (r.random((nq, d)).astype(np.float32))
    cb = datagen.sampled_codebooks(mix, m, k) if mix else r.random((m, k, d // m)).astype(np.float32)
    ref = orc.build_luts(queries, cb)
    got = host(ctx.pq_build_luts(dev(queries), dev(cb)))
    assert got.shape == ref.shape
    np.testing.assert_allclose(got, ref, rtol=4e-6, atol=1e-30)  # (dsub+1)*2^-24 at dsub=60 is 3.6e-6


def test_build_luts_exact_zero_distance(ctx):
    cb = np.arange(2 * 4 * 3, dtype=np.float32).reshape(2, 4, 3)
    queries = np.concatenate([cb[0, 2], cb[1, 1]])[None, :]
    got = host(ctx.pq_build_luts(dev(queries), dev(cb)))
    assert got[0, 0, 2] == 0.0 and got[0, 1, 1] == 0.0
    assert np.array_equal(got, orc.build_luts(queries, cb))  # small integers: exact in float


# Launches of 512 and more tiles of 128 x 128 entries take a kernel of their own (other tile, other
# block numbering, results written through LDS): ragged tiles on both sides, one and several chunks
# of 16 dimensions, a last chunk of 4 and of 12 dimensions, and rows of a length that rules out
# 16-byte stores.  Sub-vectors of 64 dimensions and more whose rows serve 8 tiles and more are converted to doubles
# by a pass of their own first (cases 3 and 7, the latter with rows padded from 68 to 80 dimensions).
@pytest.mark.parametrize("m,k,d,nq", [(32, 256, 256, 1100), (8, 300, 96, 4500), (1, 5000, 128, 1700), (4, 250, 80, 9000),
                                       (16, 256, 960, 2100), (2, 1100, 56, 8000), (2, 1100, 136, 4000)])
def test_build_luts_many_tiles(ctx, m, k, d, nq):
    r = np.random.default_rng(m * 1000 + k + nq)
    queries = (r.random((nq, d)) * 4 - 1).astype(np.float32)
    cb = (r.random((m, k, d // m)) * 4 - 1).astype(np.float32)
    # some queries lie exactly on centroids of their sub-spaces: these entries must be exact zeros
    ds = d // m
    hits = [(int(q), int(r.integers(0, m)), int(r.integers(0, k))) for q in r.integers(0, nq, 40)]
    for q, j, c in hits:
        queries[q, j * ds:(j + 1) * ds] = cb[j, c]
    ref = orc.build_luts(queries, cb)
    got = host(ctx.pq_build_luts(dev(queries), dev(cb)))
    assert got.shape == ref.shape
    np.testing.assert_allclose(got, ref, rtol=4e-6, atol=1e-30)
    for q, j, c in hits:
        assert got[q, j, c] == 0.0


# ----------------------------------------------------------------------------- quantiser
@pytest.mark.parametrize("m,k", [(16, 16), (8, 256), (3, 5)])
def test_quantize_luts_bit_exact(ctx, m, k):
    r = np.random.default_rng(11)
    nq = 33
    luts = (r.random((nq, m, k)) * 1000 + 3).astype(np.float32)
    qmax = (luts.min(axis=(1, 2)) + r.random(nq) * 2000).astype(np.float32)
    qmax[0] = luts[0].min()          # empty range
    qmax[1] = np.inf
    qmax[2] = luts[2].min() - 1.0    # negative range
    ref_q, ref_min, ref_scale = orc.quantize_luts(luts, qmax)
    q, qmin, scale = ctx.pq_quantize_luts(dev(luts), dev(qmax))
    assert np.array_equal(host(q), ref_q)
    assert np.array_equal(host(qmin), ref_min)
    assert np.array_equal(host(scale), ref_scale)


def test_qmax_prescan(ctx):
    _, queries, cb, codes16 = sift_pq(16, 16, 100000, 16)
    packed = orc.pack_u4(codes16)
    luts = ctx.pq_build_luts(dev(queries), dev(cb))
    luts_h = host(luts)
    for init, kq in ((200, 1), (1000, 1000), (4096, 1000), (3000, 77)):
        got = host(ctx.pq_qmax_prescan(dev(packed), binding.CODES_U4_PACKED, luts, init, kq))
        ref = orc.qmax_prescan(packed, orc.CODES_U4_PACKED, luts_h, init, kq)
        np.testing.assert_allclose(got, ref, rtol=2e-6)


# ----------------------------------------------------------------------------- float scan
def run_float_scan(ctx, codes, fmt, luts_h, topk):
    d, i = ctx.pq_adc_scan_topk(dev(codes) if len(codes) else torch.empty((0, codes.shape[1]), dtype=torch.uint8, device="cuda"),
                                fmt, dev(luts_h), topk)
    gd, gi = host(d), host(i)
    od, oi = orc.adc_scan_topk_f32(codes, fmt, luts_h, topk)
    for q in range(luts_h.shape[0]):
        check_float_topk(gd[q], gi[q], od[q], oi[q], codes, fmt, luts_h[q], len(codes))
    return gd, gi, od, oi


def test_scan_config0_pq8x8(ctx):
    """Config 0: d=128 mixture, 8x8 trained codebooks, N=100k encoded codes, 16 queries, top-100."""
    _, queries, cb, codes = sift_pq(8, 256, 100000, 16)
    luts_h = host(ctx.pq_build_luts(dev(queries), dev(cb)))
    gd, gi, od, oi = run_float_scan(ctx, codes, orc.CODES_U8, luts_h, 100)
    # encoded data holds many identical codes: their distances tie up to the rounding of the float
    # sum, so ids may swap inside the tolerance band, but the distance profile must match rank by rank
    np.testing.assert_allclose(gd, od, rtol=RTOL)


@pytest.mark.parametrize("n", [0, 1, 63, 127, 128, 129, 1023, 1025, 8191, 8193, 50001])
@pytest.mark.parametrize("nq,topk", [(1, 1), (3, 10), (5, 100), (8, 128)])
def test_scan_f32_ragged(ctx, n, nq, topk):
    r = np.random.default_rng(n * 7 + nq)
    codes = r.integers(0, 256, (n, 8), dtype=np.uint8)
    luts_h = (r.random((nq, 8, 256)) * 100).astype(np.float32)
    run_float_scan(ctx, codes, orc.CODES_U8, luts_h, topk)


@pytest.mark.parametrize("topk", [129, 500, 1024])
def test_scan_f32_large_topk(ctx, topk):
    r = np.random.default_rng(topk)
    n = 30011
    codes = r.integers(0, 256, (n, 8), dtype=np.uint8)
    luts_h = (r.random((6, 8, 256)) * 100).astype(np.float32)
    run_float_scan(ctx, codes, orc.CODES_U8, luts_h, topk)


def test_scan_f32_pq16x8(ctx):
    r = np.random.default_rng(3)
    n = 70007
    codes = r.integers(0, 256, (n, 16), dtype=np.uint8)
    luts_h = r.random((7, 16, 256)).astype(np.float32)
    run_float_scan(ctx, codes, orc.CODES_U8, luts_h, 100)


def test_scan_f32_many_chunks_and_groups(ctx):
    """Several chunks per query and several query groups: exercises the shared bounds and the merge."""
    r = np.random.default_rng(4)
    n = 1_000_003
    codes = r.integers(0, 256, (n, 8), dtype=np.uint8)
    luts_h = (r.random((13, 8, 256)) * 10).astype(np.float32)
    run_float_scan(ctx, codes, orc.CODES_U8, luts_h, 100)


def test_scan_f32_all_equal_and_ties(ctx):
    n = 20000
    codes = np.zeros((n, 8), np.uint8)
    luts_h = np.ones((2, 8, 256), np.float32)
    d, i = ctx.pq_adc_scan_topk(dev(codes), binding.CODES_U8, dev(luts_h), 50)
    assert np.array_equal(host(i), np.tile(np.arange(50), (2, 1)))  # equal values: smallest ids
    assert np.all(host(d) == 8.0)
    # few distinct values (exact in float, so ties are exact and the (value, id) order is unique)
    r = np.random.default_rng(5)
    codes = r.integers(0, 256, (n, 8), dtype=np.uint8)
    luts_h = r.integers(0, 3, (3, 8, 256)).astype(np.float32)
    d, i = ctx.pq_adc_scan_topk(dev(codes), binding.CODES_U8, dev(luts_h), 100)
    od, oi = orc.adc_scan_topk_f32(codes, orc.CODES_U8, luts_h, 100)
    assert np.array_equal(host(i), oi) and np.array_equal(host(d), od)


def test_scan_f32_descending_order_worst_case(ctx):
    """Distances strictly decreasing with position: every code beats the current bound."""
    n = 40000
    codes = np.zeros((n, 8), np.uint8)
    idx = np.arange(n)
    codes[:, 0] = idx % 256
    codes[:, 1] = idx // 256
    lut = np.zeros((1, 8, 256), np.float32)
    lut[0, 0] = 255 - np.arange(256)
    lut[0, 1] = (255 - np.arange(256)) * 256.0
    d, i = ctx.pq_adc_scan_topk(dev(codes), binding.CODES_U8, dev(lut), 100)
    od, oi = orc.adc_scan_topk_f32(codes, orc.CODES_U8, lut, 100)
    assert np.array_equal(host(i), oi) and np.array_equal(host(d), od)


@pytest.mark.parametrize("m,k,fmt", [(4, 16, orc.CODES_U8), (32, 16, orc.CODES_U4_PACKED), (2, 256, orc.CODES_U8),
                                     (16, 16, orc.CODES_U4_PACKED)])
def test_scan_f32_general_shapes(ctx, m, k, fmt):
    r = np.random.default_rng(m + k)
    n = 9001
    cb = m // 2 if fmt == orc.CODES_U4_PACKED else m
    hi = 256 if fmt == orc.CODES_U4_PACKED else k
    codes = r.integers(0, hi, (n, cb), dtype=np.uint8)
    luts_h = r.random((3, m, k)).astype(np.float32)
    run_float_scan(ctx, codes, fmt, luts_h, 20)


# ----------------------------------------------------------------------------- integer scan
# ------------------------------------------------------------- 8x8 float scan, pruned path
# Databases of 65536 codes and more take the scan that dismisses codes by 16-bit lower bounds
# before any float work; these cases aim at what is specific to it.
@pytest.mark.parametrize("n", [65535, 65536, 65537, 300_001])
def test_scan_f32_pruned_path_sizes(ctx, n):
    r = np.random.default_rng(n)
    codes = r.integers(0, 256, (n, 8), dtype=np.uint8)
    luts_h = (r.random((11, 8, 256)) * 50 + r.random((11, 8, 1)) * 200).astype(np.float32)
    run_float_scan(ctx, codes, orc.CODES_U8, luts_h, 100)


@pytest.mark.parametrize("topk", [1, 128, 129, 1000])
def test_scan_f32_pruned_topk_range(ctx, topk):
    r = np.random.default_rng(topk + 77)
    codes = r.integers(0, 256, (200_003, 8), dtype=np.uint8)
    luts_h = (r.random((5, 8, 256)) * 100).astype(np.float32)
    run_float_scan(ctx, codes, orc.CODES_U8, luts_h, topk)


def test_scan_f32_pruned_degenerate_tables(ctx):
    r = np.random.default_rng(21)
    n = 70_001
    # (a) every code is the per-table minimiser: the first bound equals the sum of the minima,
    #     which leaves no range for the 16-bit tables (nothing can be pruned)
    luts_h = (r.random((3, 8, 256)) * 10 + 1).astype(np.float32)
    codes = np.tile(luts_h[0].argmin(axis=1).astype(np.uint8), (n, 1))
    run_float_scan(ctx, codes, orc.CODES_U8, luts_h, 100)
    # (b) a large common offset with a tiny spread: too little fp32 resolution for a threshold
    codes = r.integers(0, 256, (n, 8), dtype=np.uint8)
    luts_h = (1.0e7 + r.random((2, 8, 256))).astype(np.float32)
    run_float_scan(ctx, codes, orc.CODES_U8, luts_h, 100)
    # (c) a huge dynamic range: most 16-bit entries clamp at their maximum
    luts_h = np.exp(r.random((4, 8, 256)) * 30 - 10).astype(np.float32)
    run_float_scan(ctx, codes, orc.CODES_U8, luts_h, 100)
    # (d) constant tables: all distances equal, the smallest ids win
    luts_h = np.full((2, 8, 256), 3.0, np.float32)
    d, i = ctx.pq_adc_scan_topk(dev(codes), binding.CODES_U8, dev(luts_h), 100)
    assert np.array_equal(host(i), np.tile(np.arange(100), (2, 1))) and np.all(host(d) == 24.0)
    # (e) few distinct table values: exact float sums, massive exact ties, unique (value, id) order
    luts_h = r.integers(0, 3, (9, 8, 256)).astype(np.float32)
    d, i = ctx.pq_adc_scan_topk(dev(codes), binding.CODES_U8, dev(luts_h), 100)
    od, oi = orc.adc_scan_topk_f32(codes, orc.CODES_U8, luts_h, 100)
    assert np.array_equal(host(i), oi) and np.array_equal(host(d), od)


def test_scan_f32_pruned_descending_order_worst_case(ctx):
    """Distances strictly decreasing with position over 2^17 codes: every code beats the bound."""
    n = 1 << 17
    codes = np.zeros((n, 8), np.uint8)
    idx = np.arange(n)
    codes[:, 0] = idx % 256
    codes[:, 1] = (idx // 256) % 256
    codes[:, 2] = idx // 65536
    lut = np.zeros((1, 8, 256), np.float32)
    lut[0, 0] = 255 - np.arange(256)
    lut[0, 1] = (255 - np.arange(256)) * 256.0
    lut[0, 2] = (255 - np.arange(256)) * 65536.0
    d, i = ctx.pq_adc_scan_topk(dev(codes), binding.CODES_U8, dev(lut), 100)
    od, oi = orc.adc_scan_topk_f32(codes, orc.CODES_U8, lut, 100)
    assert np.array_equal(host(i), oi) and np.array_equal(host(d), od)


@pytest.mark.parametrize("n,nq,topk", [(65536, 3, 100), (200_001, 9, 128), (131_072, 2, 1000)])
def test_scan_f32_pruned_16_tables(ctx, n, nq, topk):
    """16 x 256 float tables on the pruned path: random tables, then tables with exact ties."""
    r = np.random.default_rng(n + topk)
    codes = r.integers(0, 256, (n, 16), dtype=np.uint8)
    luts_h = (r.random((nq, 16, 256)) * 40 + r.random((nq, 16, 1)) * 300).astype(np.float32)
    run_float_scan(ctx, codes, orc.CODES_U8, luts_h, topk)
    luts_h = r.integers(0, 3, (nq, 16, 256)).astype(np.float32)
    d, i = ctx.pq_adc_scan_topk(dev(codes), binding.CODES_U8, dev(luts_h), topk)
    od, oi = orc.adc_scan_topk_f32(codes, orc.CODES_U8, luts_h, topk)
    assert np.array_equal(host(i), oi) and np.array_equal(host(d), od)


def test_scan_f32_pruned_encoded_duplicates(ctx):
    """Encoded mixture data (many identical codes), 37 queries: not a multiple of the group size."""
    _, queries, cb, codes = sift_pq(8, 256, 100000, 16)
    mix = datagen.sift_like()
    q2 = mix.sample(37, datagen.SEED_QUERIES + 5)
    luts_h = host(ctx.pq_build_luts(dev(q2), dev(cb)))
    gd, gi, od, oi = run_float_scan(ctx, codes, orc.CODES_U8, luts_h, 100)
    np.testing.assert_allclose(gd, od, rtol=RTOL)


def run_int_scan(ctx, codes, fmt, qluts_h, topk):
    s, i = ctx.pq_adc_scan_topk(dev(codes), fmt, dev(qluts_h), topk)
    os_, oi = orc.adc_scan_topk_u8(codes, fmt, qluts_h, topk)
    gs, gi = host(s), host(i)
    check_exact_topk(gs, gi, os_, oi)


@pytest.mark.parametrize("n", [1, 127, 129, 4097, 60001])
@pytest.mark.parametrize("nq,topk", [(1, 1), (7, 100), (9, 128), (3, 1000)])
def test_scan_u4_bit_exact(ctx, n, nq, topk):
    r = np.random.default_rng(n + nq)
    packed = r.integers(0, 256, (n, 8), dtype=np.uint8)
    qluts = r.integers(0, 256, (nq, 16, 16), dtype=np.uint8)
    run_int_scan(ctx, packed, orc.CODES_U4_PACKED, qluts, topk)


def test_scan_u4_heavy_ties_and_extremes(ctx):
    r = np.random.default_rng(6)
    n = 200_003
    packed = r.integers(0, 256, (n, 8), dtype=np.uint8)
    qluts = r.integers(0, 4, (10, 16, 16), dtype=np.uint8)      # sums in 0..48: thousands of ties
    qluts[1] = 255                                               # every sum = 4080
    qluts[2] = 0
    run_int_scan(ctx, packed, orc.CODES_U4_PACKED, qluts, 100)
    run_int_scan(ctx, packed, orc.CODES_U4_PACKED, qluts, 1000)


def test_scan_u8_general_shapes(ctx):
    r = np.random.default_rng(8)
    codes = r.integers(0, 256, (5003, 8), dtype=np.uint8)
    qluts = r.integers(0, 256, (4, 8, 256), dtype=np.uint8)
    run_int_scan(ctx, codes, orc.CODES_U8, qluts, 64)
    packed = r.integers(0, 256, (5003, 4), dtype=np.uint8)
    run_int_scan(ctx, packed, orc.CODES_U4_PACKED, r.integers(0, 256, (2, 8, 16), dtype=np.uint8), 10)


# ----------------------------------------------------------------------------- config 2 pipeline
def test_quick_adc_pipeline_config2_small(ctx):
    """16x4 codes: tables -> qmax pre-scan -> 8-bit tables -> integer scan top-1000 -> float rerank top-100.

    Stage-wise parity: each oracle stage is fed the GPU output of the previous stage, so that
    float rounding in the tables cannot move an integer decision.
    """
    _, queries, cb, codes16 = sift_pq(16, 16, 100000, 16)
    packed = orc.pack_u4(codes16)
    fmt = orc.CODES_U4_PACKED
    dpacked = dev(packed)
    luts = ctx.pq_build_luts(dev(queries), dev(cb))
    qmax = ctx.pq_qmax_prescan(dpacked, fmt, luts, 2000, 1000)
    qluts, qmin, scale = ctx.pq_quantize_luts(luts, qmax)
    sums, cand = ctx.pq_adc_scan_topk(dpacked, fmt, qluts, 1000)
    dist, ids = ctx.pq_rerank_f32(dpacked, fmt, luts, cand, 100)
    luts_h, qmax_h, qluts_h, cand_h = host(luts), host(qmax), host(qluts), host(cand)
    np.testing.assert_allclose(luts_h, orc.build_luts(queries, cb), rtol=4e-6)
    ref_q, ref_min, ref_scale = orc.quantize_luts(luts_h, qmax_h)
    assert np.array_equal(qluts_h, ref_q) and np.array_equal(host(qmin), ref_min) and np.array_equal(host(scale), ref_scale)
    os_, oi = orc.adc_scan_topk_u8(packed, fmt, qluts_h, 1000)
    check_exact_topk(host(sums), cand_h, os_, oi)
    od, oid = orc.rerank_f32(packed, fmt, luts_h, cand_h, 100)
    gd, gi = host(dist), host(ids)
    for q in range(len(queries)):
        np.testing.assert_allclose(gd[q], od[q], rtol=RTOL)
        exact = orc.adc_all_f32(packed[gi[q]], fmt, luts_h[q])
        np.testing.assert_allclose(gd[q], exact, rtol=RTOL)
        assert np.all(exact <= od[q][-1] * (1 + RTOL))
    # none of the top-1000 candidates has a clamped table entry (qmax = 1000-th distance of the pre-scan)
    un = np.stack([packed & 15, packed >> 4], axis=2).reshape(len(packed), 16)
    for q in range(len(queries)):
        assert np.all(qluts_h[q][np.arange(16)[None, :], un[cand_h[q, :100]]] < 255)


def test_rerank_matches_oracle(ctx):
    r = np.random.default_rng(10)
    n = 5000
    codes = r.integers(0, 256, (n, 8), dtype=np.uint8)
    luts_h = r.random((4, 8, 256)).astype(np.float32)
    cand = np.stack([r.choice(n, 300, replace=False) for _ in range(4)]).astype(np.int64)
    cand[2, 5:9] = -1
    d, i = ctx.pq_rerank_f32(dev(codes), binding.CODES_U8, dev(luts_h), dev(cand), 40)
    od, oi = orc.rerank_f32(codes, orc.CODES_U8, luts_h, cand, 40)
    assert np.array_equal(host(i), oi)
    np.testing.assert_allclose(host(d), od, rtol=RTOL)


# ----------------------------------------------------------------------------- error handling
def test_errors_are_reported_not_raised_in_kernels(ctx):
    codes = torch.zeros((10, 8), dtype=torch.uint8, device="cuda")
    luts = torch.zeros((1, 8, 256), dtype=torch.float32, device="cuda")
    with pytest.raises(binding.PqError) as e:
        ctx.pq_adc_scan_topk(codes, binding.CODES_U8, luts, 0)
    assert e.value.code == -1
    with pytest.raises(binding.PqError) as e:
        ctx.pq_adc_scan_topk(codes, binding.CODES_U8, luts, 5000)
    assert e.value.code == -3
    with pytest.raises(binding.PqError) as e:
        ctx.pq_build_luts(torch.zeros((1, 10), device="cuda"), torch.zeros((3, 4, 3), device="cuda"))
    assert e.value.code == -2
    with pytest.raises(binding.PqError) as e:
        ctx.pq_adc_scan_topk(codes[:, :4].contiguous(), binding.CODES_U4_PACKED, torch.zeros((1, 7, 16), device="cuda"), 5)
    assert e.value.code == -2
    # the context stays usable
    d, i = ctx.pq_adc_scan_topk(codes, binding.CODES_U8, luts, 3)
    assert host(i).tolist() == [[0, 1, 2]]


def test_scan_f32_plain_loop_on_a_large_database(ctx, opts):
    """The plain float loop (no pruning) normally serves small databases only; here it scans a large one."""
    opts.set("scan_prune", 0)
    r = np.random.default_rng(31)
    codes = r.integers(0, 256, (400_003, 8), dtype=np.uint8)
    luts_h = (r.random((9, 8, 256)) * 100).astype(np.float32)
    run_float_scan(ctx, codes, orc.CODES_U8, luts_h, 100)
    run_float_scan(ctx, codes, orc.CODES_U8, luts_h[:2], 700)


def test_switches_general_kernel_and_launch_shapes(ctx, opts):
    """The general kernel on the shapes the tuned kernels normally take, and unusual launch shapes."""
    r = np.random.default_rng(33)
    codes = r.integers(0, 256, (120_001, 8), dtype=np.uint8)
    luts_h = (r.random((6, 8, 256)) * 100).astype(np.float32)
    qluts = r.integers(0, 256, (5, 16, 16), dtype=np.uint8)
    opts.set("scan_force_general", 1)
    run_float_scan(ctx, codes, orc.CODES_U8, luts_h, 100)
    run_int_scan(ctx, codes, orc.CODES_U4_PACKED, qluts, 100)
    opts.set("scan_force_general", None)
    for blocks, items in ((3, 1), (1000, 7), (1, 1)):
        opts.set("scan_blocks", blocks)
        opts.set("scan_items_per_block", items)
        run_float_scan(ctx, codes, orc.CODES_U8, luts_h, 100)
        run_int_scan(ctx, codes, orc.CODES_U4_PACKED, qluts, 1000)


def test_build_luts_without_matrix_cores(ctx, opts):
    opts.set("lut_mfma", 0)
    r = np.random.default_rng(34)
    q = (r.random((19, 128)) * 255).astype(np.float32)
    cb = (r.random((8, 256, 16)) * 255).astype(np.float32)
    np.testing.assert_allclose(host(ctx.pq_build_luts(dev(q), dev(cb))), orc.build_luts(q, cb), rtol=4e-6, atol=0)


# ----------------------------------------------------------------------------- OPQ rotation
# the last two cases have 512 and more tiles of 128 x 128 outputs and take the kernel for large launches
@pytest.mark.parametrize("n,d", [(1000, 128), (77, 960), (4097, 20), (1, 8), (0, 16), (70001, 128), (9000, 960)])
def test_rotate_matches_oracle(ctx, n, d):
    r = np.random.default_rng(n + d)
    x = (r.random((n, d)) * 255).astype(np.float32)
    Q, _ = np.linalg.qr(r.standard_normal((d, d)))
    R = Q.astype(np.float32)
    got = host(ctx.pq_rotate(dev(x) if n else torch.empty((0, d), device="cuda"), dev(R)))
    ref = orc.rotate(x, R)
    # both sides add in double and round once; the orders differ, so the last float bit may
    np.testing.assert_allclose(got, ref, rtol=2e-7, atol=1e-30 + 2e-7 * np.abs(ref).max() if n else 0)
    if n:
        assert (got == ref).mean() > 0.99
        perm = r.permutation(d)
        P = np.zeros((d, d), np.float32)
        P[np.arange(d), perm] = 1.0
        assert np.array_equal(host(ctx.pq_rotate(dev(x), dev(P))), x[:, perm])


def test_opq_search_equals_search_on_rotated_data(ctx):
    """opq(x) = pq(R x): rotating database and queries, encoding and scanning on the GPU gives the
    oracle's results for the rotated data (rotation, encoder, tables and scan chained)."""
    mix = datagen.sift_like()
    r = np.random.default_rng(91)
    Q, _ = np.linalg.qr(r.standard_normal((128, 128)))
    R = Q.astype(np.float32)
    x = mix.sample(70_000, datagen.SEED_DATA + 5)
    y = mix.sample(9, datagen.SEED_QUERIES + 5)
    xr, yr = ctx.pq_rotate(dev(x), dev(R)), ctx.pq_rotate(dev(y), dev(R))
    cb = orc.rotate(mix.sample(256, 5), R).reshape(256, 8, 16).transpose(1, 0, 2).copy()   # centroids = rotated samples
    codes = ctx.pq_encode(xr, dev(cb))
    luts = ctx.pq_build_luts(yr, dev(cb))
    d, i = ctx.pq_adc_scan_topk(codes, binding.CODES_U8, luts, 100)
    xr_h, yr_h = host(xr), host(yr)
    codes_h = orc.pq_encode(xr_h, cb)
    assert np.array_equal(host(codes), codes_h)
    luts_h = host(luts)
    np.testing.assert_allclose(luts_h, orc.build_luts(yr_h, cb), rtol=4e-6)
    od, oi = orc.adc_scan_topk_f32(codes_h, orc.CODES_U8, luts_h, 100)
    gd, gi = host(d), host(i)
    for q in range(len(y)):
        check_float_topk(gd[q], gi[q], od[q], oi[q], codes_h, orc.CODES_U8, luts_h[q], len(codes_h))


# ----------------------------------------------------------------------------- encoder
@pytest.mark.parametrize("m,k,d,n,fmt", [(8, 256, 128, 100_000, orc.CODES_U8), (16, 16, 128, 33_333, orc.CODES_U4_PACKED),
                                         (16, 256, 960, 5_001, orc.CODES_U8), (4, 7, 20, 1_000, orc.CODES_U8),
                                         (2, 16, 6, 129, orc.CODES_U4_PACKED), (1, 200, 33, 63, orc.CODES_U8)])
def test_encode_bit_exact(ctx, m, k, d, n, fmt):
    """Codes of mixture data against trained-like codebooks equal the oracle's, index for index."""
    mix = datagen.sift_like() if d == 128 else (datagen.gist_like() if d == 960 else None)
    r = np.random.default_rng(m * 1000 + k)
    if mix is not None:
        x = mix.sample(n, datagen.SEED_DATA + 3)
        cb = datagen.sampled_codebooks(mix, m, k)
    else:
        x = (r.random((n, d)) * 10).astype(np.float32)
        cb = (r.random((m, k, d // m)) * 10).astype(np.float32)
    ref = orc.pq_encode(x, cb)
    if fmt == orc.CODES_U4_PACKED:
        ref = orc.pack_u4(ref)
    got = host(ctx.pq_encode(dev(x), dev(cb), fmt))
    assert np.array_equal(got, ref)


def test_encode_ties_and_exact_hits(ctx):
    """Duplicate centroids tie exactly (smallest index wins); vectors that are centroids encode to themselves."""
    r = np.random.default_rng(77)
    cb = (r.random((8, 256, 16)) * 255).astype(np.float32)
    cb[:, 200:] = cb[:, :56]                      # duplicates of centroids 0..55
    pick = r.integers(0, 256, (5000, 8))
    x = np.concatenate([cb[j][pick[:, j]] for j in range(8)], axis=1)
    got = host(ctx.pq_encode(dev(x), dev(cb)))
    assert np.array_equal(got, orc.pq_encode(x, cb))
    assert np.array_equal(got, np.where(pick >= 200, pick - 200, pick).astype(np.uint8))
    assert host(ctx.pq_encode(dev(x[:0]), dev(cb))).shape == (0, 8)


@pytest.mark.parametrize("ds,m,k,n", [(1, 8, 256, 1), (2, 8, 256, 65), (7, 4, 255, 511), (8, 16, 16, 513), (15, 6, 16, 1000),
                                      (16, 8, 256, 263_001), (17, 3, 33, 130), (30, 32, 16, 3001), (32, 2, 256, 64), (33, 5, 241, 700),
                                      (60, 16, 256, 2049), (64, 2, 17, 129), (65, 2, 40, 200)])
def test_encode_edges_of_tiles(ctx, ds, m, k, n):
    """Ragged numbers of vectors, dimensions and centroids, every alignment of a sub-vector, and vectors that the ranking
    on 16-bit halves cannot settle: not finite, far larger or smaller than the codebook, exactly between two centroids."""
    r = np.random.default_rng(ds * 100 + k)
    fmt = orc.CODES_U4_PACKED if k == 16 else orc.CODES_U8
    for scale in (1.0, 1e-30, 1e25):
        cb = ((r.random((m, k, ds)) - 0.3) * scale).astype(np.float32)
        x = ((r.random((n, m, ds)) - 0.3) * scale).astype(np.float32)
        x[n // 3] = np.nan
        x[n // 2, 0, 0] = np.inf
        x[n // 4] *= np.float32(1e5)
        x[n // 5] *= np.float32(1e-9)
        x[n // 6] = (cb[:, 0] + cb[:, k - 1]) / 2
        if k > 2:
            cb[:, k // 2] = cb[:, 1]
        x = x.reshape(n, m * ds)
        with np.errstate(invalid="ignore", over="ignore"):
            ref = orc.pq_encode(x, cb)
        ref = orc.pack_u4(ref) if fmt == orc.CODES_U4_PACKED else ref
        for shift in (0, 1):   # vectors that start on 16 bytes or only on 4
            buf = torch.empty(n * m * ds + 4, device="cuda")
            xd = buf[shift:shift + n * m * ds].view(n, m * ds)
            xd.copy_(torch.from_numpy(x))
            assert np.array_equal(host(ctx.pq_encode(xd, dev(cb), fmt)), ref), (scale, shift)


@pytest.mark.parametrize("ds,m,k,n", [(16, 8, 256, 1025), (16, 8, 256, 16_321), (46, 12, 256, 11_003), (50, 8, 256, 129), (64, 4, 256, 33_001), (8, 16, 16, 9_001),
                                      (15, 8, 16, 1)])
def test_encode_code_bytes_dealt_to_blocks(ctx, ds, m, k, n):
    """Few vectors: the bytes of a code are written by several blocks (also where it has whole words), of 2 waves and of 8."""
    r = np.random.default_rng(ds * 1000 + n)
    x = (r.standard_normal((n, m * ds)) * 50).astype(np.float32)
    cb = (r.standard_normal((m, k, ds)) * 50).astype(np.float32)
    fmt = orc.CODES_U4_PACKED if k == 16 else orc.CODES_U8
    ref = orc.pq_encode(x, cb)
    assert np.array_equal(host(ctx.pq_encode(dev(x), dev(cb), fmt)), orc.pack_u4(ref) if fmt == orc.CODES_U4_PACKED else ref)


@pytest.mark.parametrize("ds,m,k", [(8, 4, 256), (16, 2, 40), (5, 4, 16), (33, 2, 256)])
def test_encode_codebooks_of_extreme_magnitude(ctx, ds, m, k):
    """Codebooks at both ends of fp32 (subnormal numbers, spreads too small to be scaled into fp16's range, components near
    the greatest number), some with centroids of widely different size: the nearest centroid is decided in double."""
    r = np.random.default_rng(ds + k)
    fmt = orc.CODES_U4_PACKED if k == 16 else orc.CODES_U8
    n = 3000
    for scale in (1e-31, 1e-33, 1e-34, 1e-35, 1e-36, 1e-37, 1e-40, 1e-44, 1e30, 1e35, 4e38):
        for mixed in (False, True):
            unit = r.random((m, k, ds)) - 0.3
            if mixed:   # one centroid in four is 2^-90 times as large as the others
                unit[:, ::4] *= 2.0 ** -90
            cb = (unit * scale).astype(np.float32)
            x = ((r.random((n, m, ds)) - 0.3) * scale).astype(np.float32)
            if mixed:
                x[::2] *= np.float32(2.0 ** -90)
            x = x.reshape(n, m * ds)
            ref = orc.pq_encode(x, cb)
            got = host(ctx.pq_encode(dev(x), dev(cb), fmt))
            assert np.array_equal(got, orc.pack_u4(ref) if fmt == orc.CODES_U4_PACKED else ref), (scale, mixed)


@pytest.mark.parametrize("ds,m,k,n", [(1, 8, 256, 65), (7, 4, 255, 511), (8, 16, 16, 513), (16, 8, 256, 3001), (17, 3, 33, 130),
                                      (30, 32, 16, 301), (60, 2, 16, 200), (64, 2, 17, 129)])
def test_encode_without_scratch(ctx, opts, ds, m, k, n):
    """The form that captured calls and calls without memory take, and the one by ranking: the same codes, packed ones too."""
    r = np.random.default_rng(ds + m)
    fmt = orc.CODES_U4_PACKED if k == 16 else orc.CODES_U8
    cb = r.normal(size=(m, k, ds)).astype(np.float32)
    cb[:, k // 2] = cb[:, 1]   # ties
    x = r.normal(size=(n, m, ds)).astype(np.float32)
    x[n // 3] = cb[:, k - 1]
    x[n // 2] = cb[:, 1]
    x[n // 4] *= np.float32(1e5)
    x = x.reshape(n, m * ds)
    ref = orc.pq_encode(x, cb)
    ref = orc.pack_u4(ref) if fmt == orc.CODES_U4_PACKED else ref
    for split in (1, 0):
        opts.set("encode_split16", split)
        assert np.array_equal(host(ctx.pq_encode(dev(x), dev(cb), fmt)), ref), split


@pytest.mark.parametrize("ds,m,k,n", [(16, 4, 256, 2000), (7, 4, 16, 500), (1, 8, 256, 300), (40, 2, 100, 700)])
@pytest.mark.parametrize("distinct", [1, 2, 37])
def test_encode_equal_centroids(ctx, ds, m, k, n, distinct):
    """Codebooks with copies of centroids, one with an infinite component among them: the first copy is the code."""
    r = np.random.default_rng(ds + distinct)
    fmt = orc.CODES_U4_PACKED if k == 16 else orc.CODES_U8
    pool = r.normal(size=(m, distinct, ds)).astype(np.float32)
    if distinct == 37:
        pool[1, 5, ds - 1] = np.inf
    cb = pool[:, r.integers(0, distinct, k)]
    x = r.normal(size=(n, m, ds)).astype(np.float32)
    x[::3] = cb[:, r.integers(0, k)]
    x = x.reshape(n, m * ds)
    with np.errstate(invalid="ignore"):
        ref = orc.pq_encode(x, cb)
    assert np.array_equal(host(ctx.pq_encode(dev(x), dev(cb), fmt)), orc.pack_u4(ref) if fmt == orc.CODES_U4_PACKED else ref)


@pytest.mark.parametrize("m,k,warm", [(8, 256, True), (8, 256, False), (16, 16, True)])
def test_encode_in_a_captured_graph(m, k, warm):
    """A graph with pq_encode is replayed on new vectors while later calls on the context, eager ones with larger codebooks
    among them, make its buffers grow: every replay gives the codes of its vectors."""
    r = np.random.default_rng(m)
    stream = torch.cuda.Stream()
    g_ctx = binding.Context(0, stream)
    fmt = orc.CODES_U4_PACKED if k == 16 else orc.CODES_U8
    n, ds = 5000, 16
    cb = r.normal(size=(m, k, ds)).astype(np.float32)
    with torch.cuda.stream(stream):
        x, d_cb = torch.empty((n, m * ds), device="cuda"), dev(cb)
        if warm:
            g_ctx.pq_encode(x.zero_(), d_cb, fmt)
        stream.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=stream):
            codes = g_ctx.pq_encode(x, d_cb, fmt)
        for i in range(4):
            host_x = r.normal(size=(n, m * ds)).astype(np.float32)
            x.copy_(torch.from_numpy(host_x))
            graph.replay()
            # eager work between the replays: the encoder's own buffer and that of the Tables step grow
            big_m = 16 << i
            big_x, big_cb = torch.randn((300, big_m * 64), device="cuda"), torch.randn((big_m, 256, 64), device="cuda")
            g_ctx.pq_encode(big_x, big_cb)
            g_ctx.pq_build_luts(torch.randn((1024 << i, 128), device="cuda"), torch.randn((2, 1024 << i, 64), device="cuda"))
            torch.empty(1 << 24, dtype=torch.uint8, device="cuda").fill_(255)
            ref = orc.pq_encode(host_x, cb)
            assert np.array_equal(host(codes), orc.pack_u4(ref) if fmt == orc.CODES_U4_PACKED else ref), i
    g_ctx.close()


# ----------------------------------------------------------------------------- full size (bench configuration)
FULL_N, FULL_NQ = 25_000_000, 1000
SAMPLE_Q = [0, 1, 7, 8, 123, 500, 640, 777, 998, 999]


def test_full_size_config1_sampled(ctx):
    """Config 1 as bench.py runs it (25 M random codes, 1000 queries, top-100): complete results of a
    sample of the queries against the oracle."""
    mix = datagen.sift_like()
    queries = dev(mix.sample(FULL_NQ, datagen.SEED_QUERIES))
    cb = dev(datagen.sampled_codebooks(mix, 8, 256))
    codes_h = datagen.random_codes(FULL_N, 8)
    luts = ctx.pq_build_luts(queries, cb)
    d, i = ctx.pq_adc_scan_topk(dev(codes_h), binding.CODES_U8, luts, 100)
    gd, gi, luts_h = host(d), host(i), host(luts)
    od, oi = orc.adc_scan_topk_f32(codes_h, orc.CODES_U8, np.ascontiguousarray(luts_h[SAMPLE_Q]), 100)
    for r, q in enumerate(SAMPLE_Q):
        check_float_topk(gd[q], gi[q], od[r], oi[r], codes_h, orc.CODES_U8, luts_h[q], FULL_N)
    # properties that hold for every query: ascending, ids valid and distinct
    assert np.all(np.diff(gd, axis=1) >= 0) and gi.min() >= 0 and gi.max() < FULL_N
    assert all(len(set(row.tolist())) == 100 for row in gi[::50])


def test_full_size_config2_sampled(ctx):
    """Config 2 as bench.py runs it (25 M packed codes, 1000 queries, top-1000 by integer sums, rerank
    to top-100): stage-wise parity on a sample of the queries."""
    mix = datagen.sift_like()
    queries = dev(mix.sample(FULL_NQ, datagen.SEED_QUERIES))
    cb = dev(datagen.sampled_codebooks(mix, 16, 16))
    packed_h = datagen.random_codes(FULL_N, 8, seed=datagen.SEED_CODES + 1)
    fmt = orc.CODES_U4_PACKED
    dpacked = dev(packed_h)
    luts = ctx.pq_build_luts(queries, cb)
    qmax = ctx.pq_qmax_prescan(dpacked, fmt, luts, 2000, 1000)
    qluts, _, _ = ctx.pq_quantize_luts(luts, qmax)
    sums, cand = ctx.pq_adc_scan_topk(dpacked, fmt, qluts, 1000)
    dist, ids = ctx.pq_rerank_f32(dpacked, fmt, luts, cand, 100)
    luts_h, qmax_h, qluts_h, cand_h = host(luts), host(qmax), host(qluts), host(cand)
    ref_q, _, _ = orc.quantize_luts(np.ascontiguousarray(luts_h[SAMPLE_Q]), np.ascontiguousarray(qmax_h[SAMPLE_Q]))
    assert np.array_equal(qluts_h[SAMPLE_Q], ref_q)
    os_, oi = orc.adc_scan_topk_u8(packed_h, fmt, np.ascontiguousarray(qluts_h[SAMPLE_Q]), 1000)
    check_exact_topk(host(sums)[SAMPLE_Q], cand_h[SAMPLE_Q], os_, oi)
    od, oid = orc.rerank_f32(packed_h, fmt, np.ascontiguousarray(luts_h[SAMPLE_Q]), np.ascontiguousarray(cand_h[SAMPLE_Q]), 100)
    gd, gi = host(dist), host(ids)
    for r, q in enumerate(SAMPLE_Q):
        np.testing.assert_allclose(gd[q], od[r], rtol=RTOL)
        exact = orc.adc_all_f32(packed_h[gi[q]], fmt, luts_h[q])
        np.testing.assert_allclose(gd[q], exact, rtol=RTOL)
        assert np.all(exact <= od[r][-1] * (1 + RTOL))


def test_config3_gist_like_16x8_sampled(ctx):
    """Config 3 shape: d=960 mixture in [0,1], 16 x 256 codebooks (60 dims each), 1 M 16-byte codes, 1000
    queries, top-100.  Tables against the oracle for a sample of queries (the oracle's table build is slow),
    scan results for the same sample."""
    mix = datagen.gist_like()
    queries_h = mix.sample(FULL_NQ, datagen.SEED_QUERIES)
    cb_h = datagen.sampled_codebooks(mix, 16, 256)
    codes_h = datagen.random_codes(1_000_000, 16, seed=datagen.SEED_CODES + 4)
    luts = ctx.pq_build_luts(dev(queries_h), dev(cb_h))
    d, i = ctx.pq_adc_scan_topk(dev(codes_h), binding.CODES_U8, luts, 100)
    luts_h, gd, gi = host(luts), host(d), host(i)
    ref = orc.build_luts(np.ascontiguousarray(queries_h[SAMPLE_Q]), cb_h)
    np.testing.assert_allclose(luts_h[SAMPLE_Q], ref, rtol=4e-6, atol=0)
    od, oi = orc.adc_scan_topk_f32(codes_h, orc.CODES_U8, np.ascontiguousarray(luts_h[SAMPLE_Q]), 100)
    for r, q in enumerate(SAMPLE_Q):
        check_float_topk(gd[q], gi[q], od[r], oi[r], codes_h, orc.CODES_U8, luts_h[q], len(codes_h))



def test_scan_f32_few_queries_large_database_wide_first_bound(ctx):
    """Few query groups over a database large enough for the first bound to come from n / 64 codes
    (several seed slices): 8 x 256 tables, 3 and 17 queries, ragged size; top-100 and top-1."""
    r = np.random.default_rng(47)
    n = 9_000_011
    codes = r.integers(0, 256, (n, 8), dtype=np.uint8)
    codes[n // 2:n // 2 + 300] = codes[:300]          # exact ties across slices
    luts_h = (r.random((17, 8, 256)) * 100).astype(np.float32)
    run_float_scan(ctx, codes, orc.CODES_U8, luts_h[:3], 100)
    run_float_scan(ctx, codes, orc.CODES_U8, luts_h, 1)
    # distances descending with the row number for query 0: the first bound (from the front of the
    # database) is the loosest possible
    d0 = orc.adc_all_f32(codes[:2_000_000], orc.CODES_U8, luts_h[0])
    worst = np.ascontiguousarray(codes[:2_000_000][np.argsort(-d0, kind="stable")])
    big = np.concatenate([worst, codes[2_000_000:5_000_000]])
    run_float_scan(ctx, big, orc.CODES_U8, luts_h[:2], 100)


def test_scan_u4_few_queries_large_database_wide_first_bound(ctx):
    """The integer scan's first bound from n / 64 codes (several seed slices): bit-exact top-100 and top-1000."""
    r = np.random.default_rng(49)
    n = 9_000_011
    packed = r.integers(0, 256, (n, 8), dtype=np.uint8)
    qluts = r.integers(0, 256, (11, 16, 16), dtype=np.uint8)
    run_int_scan(ctx, packed, orc.CODES_U4_PACKED, qluts[:2], 100)
    run_int_scan(ctx, packed, orc.CODES_U4_PACKED, qluts, 1000)
    qluts[0, :, :] = 7                                  # every code has the same sum: ids decide
    run_int_scan(ctx, packed, orc.CODES_U4_PACKED, qluts[:1], 100)


# --------------------------------------------- packed 4-bit codes on the matrix cores
def run_on_matrix_cores(ctx, packed, qluts, topk, again, passes=None):
    """run_int_scan of a call that takes the matrix cores and scans `again` of its queries once more."""
    ctx.pq_set_profiling(True)
    try:
        run_int_scan(ctx, packed, orc.CODES_U4_PACKED, qluts, topk)
        info = ctx.pq_last_scan_info()
    finally:
        ctx.pq_set_profiling(False)
    kernel, nq = info["kernel"], len(qluts)
    assert kernel.startswith("scan_onehot_kernel"), kernel
    assert kernel.endswith(f"; {again} queries again by the other loops") == (again > 0) and ("again" in kernel) == (again > 0), kernel
    # every query's results are among the keys inserted, which are at most a full list (and, again, every code)
    room = 16384 if topk <= 128 else 65536
    assert nq * topk <= info["inserted_keys"] <= nq * room + again * len(packed)
    assert info["passes"] == (passes or math.ceil(nq / info["queries_per_pass"]))


# Sums are integers: results are bit-exact, ties by row.  Sizes around a load of codes (1024 bytes), the groups of 32 queries and the widths
# of 32, 64 and 128 queries; tables of few values (ties by the thousand) beside ordinary ones.
@pytest.mark.parametrize("m", [16, 32])
@pytest.mark.parametrize("n,nq,topk", [(65_536, 1, 1), (65_537, 31, 100), (66_001, 33, 129), (70_019, 65, 1000), (131_073, 129, 100), (65_664, 257, 10)])
def test_scan_u4_on_matrix_cores_sizes(ctx, opts, m, n, nq, topk):
    opts.set("scan_onehot", 1)
    r = np.random.default_rng(n + nq + m)
    packed = r.integers(0, 256, (n, m // 2), dtype=np.uint8)
    qluts = np.minimum(255, r.standard_normal((nq, m, 16)) ** 2 * r.uniform(5, 60, (nq, m, 1))).astype(np.uint8)
    qluts[::3] //= 32
    run_on_matrix_cores(ctx, packed, qluts, topk, 0)


@pytest.mark.parametrize("value", [0, 1, 255])
def test_scan_u4_on_matrix_cores_constant_tables(ctx, opts, value):
    """All codes tie: rows decide, within the sums that are counted."""
    opts.set("scan_onehot", 1)
    r = np.random.default_rng(value)
    packed = r.integers(0, 256, (131_073, 8), dtype=np.uint8)
    qluts = r.integers(0, 256, (40, 16, 16), dtype=np.uint8)
    qluts[::9] = value
    run_on_matrix_cores(ctx, packed, qluts, 100, 0)


@pytest.mark.parametrize("m", [16, 32])
@pytest.mark.parametrize("order", ["copies", "ascending", "descending"])
def test_scan_u4_on_matrix_cores_misleading_samples(ctx, opts, m, order):
    """Few distinct codes, and codes sorted by their distance: the sample bounds them all the same."""
    opts.set("scan_onehot", 1)
    r = np.random.default_rng(m)
    qluts = np.repeat(r.integers(0, 256, (1, m, 16), dtype=np.uint8), 40, axis=0)
    if order == "copies":
        packed = r.integers(0, 256, (7, m // 2), dtype=np.uint8)[r.integers(0, 7, 150_001)]
        qluts = r.integers(0, 256, (40, m, 16), dtype=np.uint8)
    else:
        packed = r.integers(0, 256, (150_001, m // 2), dtype=np.uint8)
        nib = np.stack([packed & 15, packed >> 4], 2).reshape(len(packed), m)
        sums = qluts[0][np.arange(m), nib].astype(np.int64).sum(1)
        packed = packed[np.argsort(sums if order == "ascending" else -sums)]
    run_on_matrix_cores(ctx, np.ascontiguousarray(packed), qluts, 100, 0)


# With 32 tables a query whose sums all lie beyond the bins that are counted gets no bound, and so no list of its own: it alone is scanned
# again.  Forms of that scan: short and long results, coarse and fine tiles (many codes per block or few), one group of queries and several.
@pytest.mark.parametrize("n,nq,topk,bad", [(70_001, 40, 100, [7]), (263_000, 300, 1000, [0, 7, 299]), (530_000, 16, 129, [3]), (1_100_003, 64, 10, list(range(1, 64, 5))),
                                           (66_000, 33, 128, list(range(33)))])
def test_scan_u4_on_matrix_cores_scans_only_queries_without_bound_again(ctx, opts, n, nq, topk, bad):
    opts.set("scan_onehot", 1)
    r = np.random.default_rng(n + nq)
    packed = r.integers(0, 256, (n, 16), dtype=np.uint8)
    qluts = np.minimum(255, r.standard_normal((nq, 32, 16)) ** 2 * r.uniform(5, 40, (nq, 32, 1))).astype(np.uint8)
    qluts[bad] = 255
    run_on_matrix_cores(ctx, packed, qluts, topk, len(bad))


def sampled_rows(n, shift):
    """The rows that bound a scan on the matrix cores (onehot_sample_row)."""
    i = np.arange(n >> shift, dtype=np.uint64)
    mix = np.uint64(0x9e3779b9)
    x = ((i ^ (i >> np.uint64(15))) * mix) & np.uint64(0xffffffff)
    x = ((x ^ (x >> np.uint64(15))) * mix) & np.uint64(0xffffffff)
    return (i << np.uint64(shift) | x >> np.uint64(32 - shift)).astype(np.int64)


def int_sums(packed, m, qlut):
    nib = np.stack([packed & 15, packed >> 4], 2).reshape(len(packed), m)
    return sum(qlut[j].astype(np.int32)[nib[:, j]] for j in range(m))


# The sample is made to mislead: all results of some queries lie in it, so that it bounds too few.  Every form of the other loops that these
# queries are left to (8 and 16 queries per pass, 32 tables, short and long results, coarse and fine tiles).
@pytest.mark.parametrize("m,n,nq,topk,bad", [(16, 263_001, 300, 1000, [0, 7, 299]), (16, 263_000, 300, 100, list(range(2, 40, 2))), (16, 70_001, 40, 100, [39]),
                                             (16, 1_100_003, 64, 128, [5, 60]), (16, 530_000, 9, 200, [8]), (32, 263_000, 300, 129, [1]), (32, 70_001, 100, 64, [3, 90])])
def test_scan_u4_on_matrix_cores_scans_misled_queries_again(ctx, opts, m, n, nq, topk, bad):
    opts.set("scan_onehot", 1)
    r = np.random.default_rng(n + nq + m)
    packed = r.integers(0, 256, (n, m // 2), dtype=np.uint8)
    qluts = np.minimum(255, r.standard_normal((nq, m, 16)) ** 2 * r.uniform(5, 40, (nq, m, 1))).astype(np.uint8)
    places = r.permutation(sampled_rows(n, 3))
    for b, q in enumerate(bad):
        best = np.argpartition(int_sums(packed, m, qluts[q]), topk)[:topk]
        best = best[~np.isin(best, places[:(b + 1) * topk])]
        to = places[b * topk:b * topk + len(best)]
        packed[best], packed[to] = packed[to].copy(), packed[best].copy()
    run_on_matrix_cores(ctx, packed, qluts, topk, len(bad))


# Neighbours stored side by side: the sample bounds every query as it does for rows in any other order.
@pytest.mark.parametrize("m,n,nq,topk,group", [(16, 300_000, 300, 1000, 64), (16, 300_032, 300, 100, 1024), (16, 2_200_000, 60, 100, 64), (32, 300_000, 100, 1000, 64), (16, 131_072, 100, 10, 16)])
def test_scan_u4_on_matrix_cores_neighbours_side_by_side(ctx, opts, m, n, nq, topk, group):
    opts.set("scan_onehot", 1)
    r = np.random.default_rng(n + nq + m)
    nib = np.repeat(r.integers(0, 16, (n // group, m), dtype=np.uint8), group, 0)
    moved = r.random(nib.shape) < 0.15
    nib[moved] = r.integers(0, 16, int(moved.sum()), dtype=np.uint8)
    packed = np.ascontiguousarray(nib[:, 0::2] | nib[:, 1::2] << 4)
    qluts = np.minimum(255, r.standard_normal((nq, m, 16)) ** 2 * r.uniform(5, 40, (nq, m, 1))).astype(np.uint8)
    run_on_matrix_cores(ctx, packed, qluts, topk, 0)


# Equal codes stored side by side, far from the start: their rows, not their sum, end the results.  They are the nearest codes of half of the queries: of the
# least sum that the tables allow, or of a greater one.
@pytest.mark.parametrize("m,nq,topk,least", [(16, 40, 100, True), (16, 40, 1000, False), (32, 20, 1000, True), (32, 20, 50, False)])
def test_scan_u4_on_matrix_cores_equal_codes_side_by_side(ctx, opts, m, nq, topk, least):
    opts.set("scan_onehot", 1)
    n, r = 2_200_003, np.random.default_rng(nq + m + topk)
    packed = r.integers(0, 256, (n, m // 2), dtype=np.uint8)
    code = r.integers(0, 16, m, dtype=np.uint8)
    packed[2_000_000:2_090_000] = code[0::2] | code[1::2] << 4
    qluts = (1 + np.minimum(254, r.standard_normal((nq, m, 16)) ** 2 * r.uniform(5, 40, (nq, m, 1)))).astype(np.uint8)
    qluts[::2, np.arange(m), code] = 0
    if not least:
        qluts[::2, 0, (code[0] + 1) % 16] = qluts[::2, 1, (code[1] + 1) % 16] = 0
        qluts[::2, 0, code[0]] = 1
        packed[:, 0] = np.where((packed[:, 0] & 15) == (code[0] + 1) % 16, packed[:, 0] & 0xf0 | code[0], packed[:, 0])
    run_on_matrix_cores(ctx, packed, qluts, topk, 0)


# More queries than their lists have room for: equal slices of them, all of which take the matrix cores (32 tables: room for half as many).
@pytest.mark.parametrize("m,n,nq,topk,passes", [(16, 65_600, 3000, 3, 2 * 12), (32, 65_536, 1501, 100, 2 * 12), (32, 65_536, 2100, 130, 2 * 17)])
def test_scan_u4_on_matrix_cores_in_slices_of_queries(ctx, opts, m, n, nq, topk, passes):
    opts.set("scan_onehot", 1)
    r = np.random.default_rng(77 + nq)
    packed = r.integers(0, 256, (n, m // 2), dtype=np.uint8)
    qluts = np.minimum(255, r.standard_normal((nq, m, 16)) ** 2 * 20).astype(np.uint8)
    if m == 32:
        qluts[700], qluts[-1] = 255, 255          # (no bound: scanned again, one of each slice)
    run_on_matrix_cores(ctx, packed, qluts, topk, 2 if m == 32 else 0, passes)


# Which loop serves a call by default, on both sides of the lines (results are compared elsewhere: here the codes are few and far between).
@pytest.mark.parametrize("m,n,nq,topk,served", [
    (16, 262_144, 249, 129, False), (16, 262_144, 249, 480, True), (16, 720_896, 249, 129, True), (16, 327_680, 1000, 1, True), (16, 262_144, 1100, 1, False),
    (16, 262_144, 1100, 100, True), (16, 1 << 20, 248, 100, False), (16, 1 << 23, 88, 100, True), (16, 1 << 23, 88, 1000, True), (16, 1 << 22, 180, 1000, False),
    (32, 262_144, 249, 129, True), (32, 262_144, 600, 31, False), (32, 262_144, 600, 32, True), (32, 1 << 23, 48, 100, False), (32, 1 << 23, 48, 300, True),
    (32, 1 << 19, 1500, 100, False), (32, 983_040, 1500, 100, True), (16, 1 << 19, 3000, 99, False), (16, 1 << 19, 3000, 100, True)])
def test_scan_u4_calls_that_take_the_matrix_cores(ctx, m, n, nq, topk, served):
    codes = datagen.random_codes_device(n, m // 2, seed=n + m)
    qluts = torch.randint(0, 40, (nq, m, 16), dtype=torch.uint8, device="cuda", generator=torch.Generator(device="cuda").manual_seed(nq))
    ctx.pq_set_profiling(True)
    try:
        v, _ = ctx.pq_adc_scan_topk(codes, orc.CODES_U4_PACKED, qluts, topk)
        kernel = ctx.pq_last_scan_info()["kernel"]
    finally:
        ctx.pq_set_profiling(False)
    assert kernel.startswith("scan_onehot_kernel") == served and "again" not in kernel, kernel
    assert bool((v[:, 1:] >= v[:, :-1]).all())


def test_scan_u4_batches_that_the_matrix_cores_do_not_serve_stay_whole(ctx, opts):
    """Tables that are not on 16 bytes: the other loops take the batch in one go, whatever its size."""
    opts.set("scan_onehot", 1)
    r = np.random.default_rng(5)
    n, nq = 65_600, 3000
    packed = r.integers(0, 256, (n, 8), dtype=np.uint8)
    qluts = np.minimum(255, r.standard_normal((nq, 16, 16)) ** 2 * 20).astype(np.uint8)
    moved = torch.empty(qluts.size + 4, dtype=torch.uint8, device="cuda")[4:].view(nq, 16, 16)
    moved.copy_(dev(qluts))
    ctx.pq_set_profiling(True)
    try:
        s, i = ctx.pq_adc_scan_topk(dev(packed), orc.CODES_U4_PACKED, moved, 3)
        info = ctx.pq_last_scan_info()
    finally:
        ctx.pq_set_profiling(False)
    check_exact_topk(host(s), host(i), *orc.adc_scan_topk_u8(packed, orc.CODES_U4_PACKED, qluts, 3))
    assert info["kernel"].startswith("scan_tuned_kernel<U4Q_M16") and info["passes"] == math.ceil(nq / 16), info


# --------------------------------------------- 8x8 float scan, 8-bit lower bounds, 16 queries per pass
# 512 queries and more (enough groups of 16 to fill the GPU) take the loop on 8-bit lower bounds; these
# cases aim at what is specific to it: ragged last group, saturating entries, degenerate ranges, ties.
def many_queries(r, nq, spread=50.0, offset=200.0):
    return (r.random((nq, 8, 256)) * spread + r.random((nq, 8, 1)) * offset).astype(np.float32)


@pytest.mark.parametrize("n,nq,topk", [(65536, 512, 100), (70_001, 520, 1), (90_003, 777, 128), (66_000, 513, 1000),
                                       (75_001, 530, 129), (100_003, 512, 512), (80_001, 249, 100), (66_000, 250, 1000)])
def test_scan_f32_16_queries_per_pass_sizes(ctx, n, nq, topk):
    r = np.random.default_rng(n + nq)
    codes = r.integers(0, 256, (n, 8), dtype=np.uint8)
    run_float_scan(ctx, codes, orc.CODES_U8, many_queries(r, nq), topk)


def test_scan_f32_16_queries_per_pass_degenerate_tables(ctx, opts):
    r = np.random.default_rng(23)
    n, nq = 70_001, 515
    codes = r.integers(0, 256, (n, 8), dtype=np.uint8)
    # a huge dynamic range: most 8-bit entries saturate
    luts_h = np.exp(r.random((nq, 8, 256)) * 30 - 10).astype(np.float32)
    run_float_scan(ctx, codes, orc.CODES_U8, luts_h, 100)
    # a large common offset with a tiny spread: no fp32 resolution for a threshold (no pruning for those queries),
    # mixed with ordinary queries in the same groups
    luts_h = many_queries(r, nq)
    luts_h[::3] = (1.0e7 + r.random((len(luts_h[::3]), 8, 256))).astype(np.float32)
    run_float_scan(ctx, codes, orc.CODES_U8, luts_h, 100)
    # few distinct table values: exact sums, massive exact ties, unique (value, id) order
    luts_h = r.integers(0, 3, (nq, 8, 256)).astype(np.float32)
    d, i = ctx.pq_adc_scan_topk(dev(codes), binding.CODES_U8, dev(luts_h), 100)
    od, oi = orc.adc_scan_topk_f32(codes, orc.CODES_U8, luts_h, 100)
    assert np.array_equal(host(i), oi) and np.array_equal(host(d), od)
    # every code is the per-table minimiser of query 0: its first bound leaves no range
    luts_h = many_queries(r, nq)
    same = np.tile(luts_h[0].argmin(axis=1).astype(np.uint8), (n, 1))
    run_float_scan(ctx, same, orc.CODES_U8, luts_h, 100)
    # the 16-bit loop for the same inputs (switch), as a cross-check of the switch itself
    opts.set("scan_q8", 0)
    run_float_scan(ctx, codes, orc.CODES_U8, luts_h, 100)


def test_scan_f32_16_queries_per_pass_worst_case_order_and_duplicates(ctx):
    r = np.random.default_rng(29)
    n, nq = 80_000, 512
    codes = r.integers(0, 256, (n, 8), dtype=np.uint8)
    luts_h = many_queries(r, nq)
    d0 = orc.adc_all_f32(codes, orc.CODES_U8, luts_h[0])
    worst = np.ascontiguousarray(codes[np.argsort(-d0, kind="stable")])    # far to near for query 0
    worst[40_000:40_500] = worst[-500:]                                    # duplicates of the best codes
    run_float_scan(ctx, worst, orc.CODES_U8, luts_h, 100)


# ------------------------------------------------- integer scan of many queries (8-bit lower bounds, 16 per pass)
def quantized_like_tables(r, nq):
    """u8 tables shaped like quantised distance tables: a spread of small values per component and a few
    saturated entries."""
    base = r.integers(0, 40, (nq, 16, 1))
    t = base + (r.random((nq, 16, 16)) ** 2 * 60).astype(np.int64)
    t[r.random((nq, 16, 16)) < 0.05] = 255
    return np.clip(t, 0, 255).astype(np.uint8)


@pytest.mark.parametrize("n,nq,topk", [(65536, 512, 100), (70_001, 520, 1), (90_003, 777, 128), (66_001, 513, 1000),
                                       (75_001, 530, 129), (100_003, 512, 512), (80_001, 249, 100), (66_000, 250, 1000)])
def test_scan_u4_16_queries_per_pass_sizes(ctx, n, nq, topk):
    r = np.random.default_rng(n + nq)
    packed = r.integers(0, 256, (n, 8), dtype=np.uint8)
    run_int_scan(ctx, packed, orc.CODES_U4_PACKED, quantized_like_tables(r, nq), topk)


def test_scan_u4_16_queries_per_pass_degenerate_tables(ctx, opts):
    r = np.random.default_rng(31)
    n, nq = 70_001, 515
    packed = r.integers(0, 256, (n, 8), dtype=np.uint8)
    # uniform bytes: wide sums, the 8-bit entries saturate for most codes
    run_int_scan(ctx, packed, orc.CODES_U4_PACKED, r.integers(0, 256, (nq, 16, 16), dtype=np.uint8), 100)
    # sums in 0..48 (thousands of ties at the bound), constant tables (no range at all), all 255, all 0
    qluts = r.integers(0, 4, (nq, 16, 16), dtype=np.uint8)
    qluts[1] = 255
    qluts[2] = 0
    qluts[3] = 7
    qluts[20:40] = quantized_like_tables(r, 20)
    run_int_scan(ctx, packed, orc.CODES_U4_PACKED, qluts, 100)
    run_int_scan(ctx, packed, orc.CODES_U4_PACKED, qluts, 400)
    # every code is the minimiser of query 0: its first bound equals the sum of the minima
    qluts = quantized_like_tables(r, nq)
    best = qluts[0].argmin(axis=1)
    same = np.tile((best[0::2] | (best[1::2] << 4)).astype(np.uint8), (n, 1))
    run_int_scan(ctx, same, orc.CODES_U4_PACKED, qluts, 100)
    # the 16-bit loop for the same inputs (switch)
    opts.set("scan_q8", 0)
    run_int_scan(ctx, packed, orc.CODES_U4_PACKED, qluts, 100)


def test_scan_u4_16_queries_per_pass_worst_case_order_and_duplicates(ctx):
    r = np.random.default_rng(37)
    n, nq = 80_000, 512
    packed = r.integers(0, 256, (n, 8), dtype=np.uint8)
    qluts = quantized_like_tables(r, nq)
    d0 = orc.adc_all_u8(packed, orc.CODES_U4_PACKED, qluts[0]).astype(np.int64)
    worst = np.ascontiguousarray(packed[np.argsort(-d0, kind="stable")])   # far to near for query 0
    worst[40_000:40_500] = worst[-500:]                                    # duplicates of the best codes
    run_int_scan(ctx, worst, orc.CODES_U4_PACKED, qluts, 100)
    run_int_scan(ctx, worst, orc.CODES_U4_PACKED, qluts, 500)


def test_scan_16_queries_per_pass_first_round_of_short_items(ctx, opts):
    """Long result lists start with a round of short chunks (one per block) before the long ones: here forced onto a
    small database (one block tile per short chunk, few blocks), ragged end, float and integer scans."""
    opts.set("scan_head", 1)
    opts.set("scan_blocks", 20)   # one short chunk per group (513 queries), two (300 queries)
    r = np.random.default_rng(43)
    for n, nq, topk in [(100_003, 513, 1000), (140_001, 300, 300)]:
        codes = r.integers(0, 256, (n, 8), dtype=np.uint8)
        run_float_scan(ctx, codes, orc.CODES_U8, many_queries(r, nq), topk)
        run_int_scan(ctx, codes, orc.CODES_U4_PACKED, quantized_like_tables(r, nq), topk)


@pytest.mark.parametrize("n,nq,topk", [(1, 1, 1), (63, 3, 100), (1023, 4, 128), (1024, 5, 128), (1023, 300, 600), (3000, 300, 1000), (4097, 9, 128), (65_535, 8, 129), (65_537, 11, 1000), (200_003, 260, 100),
                                      (140_001, 70, 1024), (2_200_001, 2, 1000)])
def test_scan_u4_32_tables(ctx, n, nq, topk):
    """32 x 4 codes: tables like quantised distances (small sums), uniform bytes (sums around 4080, where the bins of the
    bounds end), large entries (all sums beyond the bins), and ties far beyond k."""
    r = np.random.default_rng(n + nq)
    packed = r.integers(0, 256, (n, 16), dtype=np.uint8)
    qluts = np.concatenate([quantized_like_tables(r, nq), quantized_like_tables(r, nq)], axis=1)
    kinds = [lambda: r.integers(0, 256, (32, 16)), lambda: r.integers(200, 256, (32, 16)), lambda: np.full((32, 16), 255),
             lambda: r.integers(0, 2, (32, 16))]
    for q in range(1, nq, 2):
        qluts[q] = kinds[(q // 2) % len(kinds)]()
    run_int_scan(ctx, packed, orc.CODES_U4_PACKED, qluts, topk)


@pytest.mark.parametrize("n,nq,topk", [(511, 3, 100), (512, 9, 100), (512, 300, 256), (513, 2, 257), (8191, 30, 1000), (8193, 30, 100),
                                      (20_000, 260, 1000), (4097, 300, 100), (40_000, 7, 1024)])
def test_scan_u4_first_bound_of_small_databases(ctx, n, nq, topk):
    """16 x 4 codes from where the integer scan takes a first bound on: one and several slices, few and many queries, k
    half of the codes and more."""
    r = np.random.default_rng(n + nq)
    packed = r.integers(0, 256, (n, 8), dtype=np.uint8)
    qluts = quantized_like_tables(r, nq)
    qluts[0] = 255
    run_int_scan(ctx, packed, orc.CODES_U4_PACKED, qluts, topk)


@pytest.mark.parametrize("m", [16, 32])
def test_scan_u4_ties_in_the_slices_of_a_wide_first_bound(ctx, m):
    """Few queries, more than 2^21 codes: the first bound comes from slices of 65 536 codes.  Ties at the k-th sum end in
    the first slice, in a later one, or only beyond the sample; sums beyond the bins that are kept per slice."""
    r = np.random.default_rng(m)
    n = 2_300_011
    packed = r.integers(0, 256, (n, m // 2), dtype=np.uint8)
    packed[:70_000] = 0x11            # sum m for query 1, no ties with the zeros
    packed[70_000:70_500] = 0x00      # in the second slice of the sample
    packed[n - 3000:] = 0x00          # beyond the sample
    qluts = r.choice(np.array([0, 1, 40], dtype=np.uint8), size=(4, m, 16), p=[0.4, 0.2, 0.4])
    qluts[1] = np.arange(16)[None, :]
    qluts[2] = 60                     # every sum 60 m: a tie of all codes, above the bins of the slices
    qluts[3] = 7                      # the same below them for 16 tables
    for topk in (100, 1000):
        run_int_scan(ctx, packed, orc.CODES_U4_PACKED, qluts, topk)


def test_scan_u4_32_tables_copies_and_fixed_scratch(ctx):
    """A hundred thousand copies of a query's best code (rows decide), and the call that allocates nothing."""
    r = np.random.default_rng(5)
    n, nq, topk = 150_003, 20, 100
    packed = r.integers(0, 256, (n, 16), dtype=np.uint8)
    qluts = np.concatenate([quantized_like_tables(r, nq), quantized_like_tables(r, nq)], axis=1)
    best = qluts[0].argmin(axis=1)
    packed[r.choice(n, 100_000, replace=False)] = (best[0::2] | (best[1::2] << 4)).astype(np.uint8)
    for k in (topk, 1000):   # (1000: the tuned kernel's lists do not fit the fixed scratch, the general kernel's do)
        run_int_scan(ctx, packed, orc.CODES_U4_PACKED, qluts, k)
        s, i = ctx.pq_adc_scan_topk(dev(packed), orc.CODES_U4_PACKED, dev(qluts), k)
        s2, i2 = ctx.pq_adc_scan_topk(dev(packed), orc.CODES_U4_PACKED, dev(qluts), k, noalloc=True)
        assert torch.equal(s, s2) and torch.equal(i, i2)


@pytest.mark.parametrize("fmt,m,k,nq,n", [(orc.CODES_U8, 8, 256, 16, 1_000_003), (orc.CODES_U4_PACKED, 16, 16, 9, 500_001), (orc.CODES_U8, 16, 256, 8, 300_007)])
def test_scan_long_results_with_fixed_scratch(ctx, fmt, m, k, nq, n):
    """Long results of a database that plain calls spread over the chip: with the fixed scratch, which has no room for as
    many blocks' lists, the call is served in fewer."""
    r = np.random.default_rng(m + nq)
    codes = dev(r.integers(0, 256, (n, m // 2 if fmt == orc.CODES_U4_PACKED else m), dtype=np.uint8))
    luts = dev(quantized_like_tables(r, nq) if fmt == orc.CODES_U4_PACKED else (r.random((nq, m, k)) * 50).astype(np.float32))
    v, i = ctx.pq_adc_scan_topk(codes, fmt, luts, 1000)
    v2, i2 = ctx.pq_adc_scan_topk(codes, fmt, luts, 1000, noalloc=True)
    assert torch.equal(i, i2) and torch.equal(v, v2)


@pytest.mark.parametrize("fmt,m,k,nq,n,topk", [(orc.CODES_U8, 8, 256, 3, 524_289, 129), (orc.CODES_U8, 8, 256, 8, 600_001, 1000), (orc.CODES_U4_PACKED, 16, 16, 9, 700_003, 513),
                                               (orc.CODES_U4_PACKED, 32, 16, 6, 540_003, 1024), (orc.CODES_U8, 16, 256, 29, 2_100_001, 300)])
def test_scan_long_results_on_part_of_the_blocks(ctx, opts, fmt, m, k, nq, n, topk):
    """Long results of a few groups of queries, served in large tiles by half or a quarter of the blocks: the same lists
    whatever the number of blocks, integer sums against the oracle."""
    r = np.random.default_rng(n + nq)
    codes = r.integers(0, 256, (n, m // 2 if fmt == orc.CODES_U4_PACKED else m), dtype=np.uint8)
    if fmt == orc.CODES_U4_PACKED:
        luts = np.concatenate([quantized_like_tables(r, nq)] * (m // 16), axis=1)
        run_int_scan(ctx, codes, fmt, luts, topk)
    else:
        luts = (r.random((nq, m, k)) * 50).astype(np.float32)
    v, i = ctx.pq_adc_scan_topk(dev(codes), fmt, dev(luts), topk)
    opts.set("scan_blocks", 37)
    v2, i2 = ctx.pq_adc_scan_topk(dev(codes), fmt, dev(luts), topk)
    assert torch.equal(i, i2) and torch.equal(v, v2)


# ----------------------------------------------------------------------------- encoded data at full size
ENC_UNIQUE = 400_000   # vectors encoded by the oracle; the 25 M rows are drawn from them (so every code has ~60 exact copies)


def test_full_size_config1_encoded_sampled(ctx):
    """Config 1 on encoded data: mixture vectors encoded by the oracle against codebooks trained by the oracle's
    k-means, rows drawn from them to fill 25 M (clustered distances, heavy duplicates: what a pruning scan finds
    hardest), 1000 queries, top-100; complete results of a sample of the queries against the oracle."""
    _, _, cb, unique = sift_pq(8, 256, ENC_UNIQUE, 16)
    codes_h = datagen.tile_rows(unique, FULL_N)
    queries = dev(datagen.sift_like().sample(FULL_NQ, datagen.SEED_QUERIES))
    luts = ctx.pq_build_luts(queries, dev(cb))
    d, i = ctx.pq_adc_scan_topk(dev(codes_h), binding.CODES_U8, luts, 100)
    gd, gi, luts_h = host(d), host(i), host(luts)
    od, oi = orc.adc_scan_topk_f32(codes_h, orc.CODES_U8, np.ascontiguousarray(luts_h[SAMPLE_Q]), 100)
    for r, q in enumerate(SAMPLE_Q):
        check_float_topk(gd[q], gi[q], od[r], oi[r], codes_h, orc.CODES_U8, luts_h[q], FULL_N)
        np.testing.assert_allclose(gd[q], od[r], rtol=RTOL)
    assert np.all(np.diff(gd, axis=1) >= 0) and gi.min() >= 0 and gi.max() < FULL_N
    assert all(len(set(row.tolist())) == 100 for row in gi[::50])


def test_full_size_config2_encoded_sampled(ctx):
    """Config 2 on encoded data (16 x 4, packed; rows drawn from oracle-encoded vectors): 8-bit tables are coarse where
    the codes crowd, so thousands of codes tie at the 1000th integer sum and rows decide; stage-wise, bit-exact."""
    _, _, cb, unique = sift_pq(16, 16, ENC_UNIQUE, 16)
    fmt = orc.CODES_U4_PACKED
    packed_h = datagen.tile_rows(orc.pack_u4(unique), FULL_N)
    queries = dev(datagen.sift_like().sample(FULL_NQ, datagen.SEED_QUERIES))
    dpacked = dev(packed_h)
    luts = ctx.pq_build_luts(queries, dev(cb))
    qmax = ctx.pq_qmax_prescan(dpacked, fmt, luts, 2000, 1000)
    qluts, _, _ = ctx.pq_quantize_luts(luts, qmax)
    luts_h, qmax_h, qluts_h = host(luts), host(qmax), host(qluts)
    ref_q, _, _ = orc.quantize_luts(np.ascontiguousarray(luts_h[SAMPLE_Q]), np.ascontiguousarray(qmax_h[SAMPLE_Q]))
    assert np.array_equal(qluts_h[SAMPLE_Q], ref_q)
    for topk in (1000, 100):
        sums, cand = ctx.pq_adc_scan_topk(dpacked, fmt, qluts, topk)
        os_, oi = orc.adc_scan_topk_u8(packed_h, fmt, np.ascontiguousarray(qluts_h[SAMPLE_Q]), topk)
        check_exact_topk(host(sums)[SAMPLE_Q], host(cand)[SAMPLE_Q], os_, oi)
    # every query: sums ascending, rows valid, distinct, and ascending inside runs of equal sums
    gs, gc = host(sums).astype(np.int64), host(cand)
    assert np.all(np.diff(gs, axis=1) >= 0) and gc.min() >= 0 and gc.max() < FULL_N
    order_key = gs * (1 << 32) + gc
    assert np.all(np.diff(order_key, axis=1) > 0)


@pytest.mark.parametrize("nq", [20, 300])
def test_scan_u4_ties_at_the_kth_sum_far_beyond_k(ctx, nq):
    """Tables with entries 0 / 1 / 40: sums take a handful of values and tens of thousands of codes tie at the
    k-th; the result is the tied codes with the smallest rows.  Both integer loops, short and long lists."""
    r = np.random.default_rng(91 + nq)
    n = 400_003
    packed = r.integers(0, 256, (n, 8), dtype=np.uint8)
    qluts = r.choice(np.array([0, 1, 40], dtype=np.uint8), size=(nq, 16, 16), p=[0.5, 0.3, 0.2])
    qluts[1] = 0          # every code ties
    qluts[2, :, 1:] = 7   # one cheap entry per table: sums 0, 7, 14, ...
    qluts[2, :, 0] = 0
    for topk in (100, 1000, 1):
        run_int_scan(ctx, packed, orc.CODES_U4_PACKED, qluts, topk)


@pytest.mark.parametrize("m,nq", [(8, 5), (8, 300), (16, 5), (16, 40)])
def test_scan_f32_first_bound_equal_to_the_sum_of_the_table_minima(ctx, m, nq):
    """More than k codes are exact copies of a query's best possible code (every table entry at its minimum), as
    happens with encoded high-dimensional data: the first bound leaves no range for the lower-bound tables.
    Query 0: thousands of copies; query 1: k - 1 copies (the k-th result is an ordinary code); the others: none."""
    r = np.random.default_rng(300 + m + nq)
    n, topk = 200_003, 100
    codes = r.integers(0, 256, (n, m), dtype=np.uint8)
    luts_h = (r.random((nq, m, 256)) * 50 + r.random((nq, m, 1)) * 100).astype(np.float32)
    best0 = luts_h[0].argmin(axis=1).astype(np.uint8)
    best1 = luts_h[1].argmin(axis=1).astype(np.uint8)
    codes[r.choice(n, 5000, replace=False)] = best0
    rows1 = r.choice(n, topk - 1, replace=False)
    codes[rows1] = best1
    gd, gi, od, oi = run_float_scan(ctx, codes, orc.CODES_U8, luts_h, topk)
    assert np.all(gd[0] == gd[0][0])                       # a hundred copies of the best code
    np.testing.assert_allclose(gd, od, rtol=RTOL)
    run_float_scan(ctx, codes, orc.CODES_U8, luts_h, 1000 if nq <= 40 else 300)


@pytest.mark.parametrize("m", [8, 16])
@pytest.mark.parametrize("n,nq,topk,kind", [(65_536, 1, 1, "random"), (65_537, 248, 3, "random"), (100_003, 17, 1024, "random"), (300_001, 5, 100, "far"),
                                            (70_000, 9, 100, "infinite"), (66_000, 2, 128, "mostly_infinite"), (90_001, 40, 1000, "equal"), (80_000, 3, 10, "negative")])
def test_scan_f32_first_bound_from_slices_of_small_samples(ctx, opts, m, n, nq, topk, kind):
    """The float scans of few queries start from a bound found on slices of a sample: against the oracle and the one-block
    first bound, with a far centroid, infinite entries (also so many that fewer than topk distances are finite), equal codes and tables
    that are no distances."""
    r = np.random.default_rng(n + m)
    codes = r.integers(0, 256, (n, m), dtype=np.uint8)
    luts = (r.random((nq, m, 256)) * 100).astype(np.float32)
    if kind == "far":
        luts[:, 2, 7] = 3e20
    if kind == "infinite":
        luts[:, 1, 9] = np.inf
    if kind == "mostly_infinite":
        luts[:, 0, 1:] = np.inf
        codes[:, 0] = np.maximum(codes[:, 0], 1)
        codes[r.permutation(n)[:50], 0] = 0
    if kind == "equal":
        codes[:] = codes[5]
    if kind == "negative":
        luts -= 60.0
    got = [host(t) for t in ctx.pq_adc_scan_topk(dev(codes), binding.CODES_U8, dev(luts), topk)]
    opts.set("scan_wide_seed", 0)
    ref = [host(t) for t in ctx.pq_adc_scan_topk(dev(codes), binding.CODES_U8, dev(luts), topk)]
    assert np.array_equal(got[0], ref[0]) and np.array_equal(got[1], ref[1])
    if kind in ("random", "far", "equal"):
        od, oi = orc.adc_scan_topk_f32(codes, orc.CODES_U8, luts, topk)
        for q in range(0, nq, 7):
            check_float_topk(got[0][q], got[1][q], od[q], oi[q], codes, orc.CODES_U8, luts[q], n)


@pytest.mark.parametrize("n,nq,topk,kind", [(4096, 1, 1, "random"), (4097, 4, 100, "random"), (4351, 5, 1024, "random"), (8192, 3, 128, "equal"),
                                            (70_001, 9, 129, "few_values"), (100_003, 7, 100, "far"), (50_000, 2, 100, "infinite"),
                                            (60_000, 6, 128, "mostly_infinite"), (300_001, 17, 100, "negative"), (40_000, 4, 1000, "overflow"),
                                            (500_003, 33, 1024, "random"), (20_000, 1100, 10, "random")])
def test_scan_f32_four_byte_codes(ctx, opts, n, nq, topk, kind):
    """32-bit codes: values and ids are those of the general kernel, whatever order the filter adds in: with ties, a far centroid,
    infinite entries (also so many that fewer than topk distances are finite), tables that are no distances and sums that
    overflow in one order of the additions but not in another."""
    r = np.random.default_rng(n)
    codes = r.integers(0, 256, (n, 4), dtype=np.uint8)
    luts = (r.random((nq, 4, 256)) * 100).astype(np.float32)
    if kind == "equal":
        codes[:] = codes[5]
    if kind == "few_values":
        luts = np.round(luts / 20)
    if kind == "far":
        luts[:, 2, 7] = 3e20
    if kind == "infinite":
        luts[:, 1, 9] = np.inf
        luts[:, 3, 2] = -np.inf
        luts[:, 0, 5] = np.nan
    if kind == "mostly_infinite":
        luts[:, 0, 1:] = np.inf
        codes[:, 0] = np.maximum(codes[:, 0], 1)
        codes[r.permutation(n)[:50], 0] = 0
    if kind == "negative":
        luts -= 60.0
    if kind == "overflow":
        luts[:, 0, :128] = 3e38
        luts[:, 1, :128] = -3e38
        luts[:, 2, :64] = 3e38
        luts[:, 3, :64] = -3e38
    got = [host(t) for t in ctx.pq_adc_scan_topk(dev(codes), binding.CODES_U8, dev(luts), topk)]
    opts.set("scan_force_general", 1)
    ref = [host(t) for t in ctx.pq_adc_scan_topk(dev(codes), binding.CODES_U8, dev(luts), topk)]
    assert np.array_equal(got[0], ref[0]) and np.array_equal(got[1], ref[1])
    if kind == "random":
        od, oi = orc.adc_scan_topk_f32(codes, orc.CODES_U8, luts, topk)
        for q in range(0, nq, 7):
            check_float_topk(got[0][q], got[1][q], od[q], oi[q], codes, orc.CODES_U8, luts[q], n)


@pytest.mark.parametrize("n,nq,topk,m", [(8191, 1, 1, 8), (8192, 1, 1, 16), (8193, 4, 100, 8), (8200, 3, 1024, 16), (12_288, 5, 512, 8), (24_601, 30, 1000, 16),
                                         (24_576, 600, 1024, 8), (9001, 513, 3, 16), (65_535, 2, 128, 8)])
@pytest.mark.parametrize("kind", ["random", "few_values", "negative", "infinite"])
def test_scan_f32_pruned_small_databases(ctx, opts, n, nq, topk, m, kind):
    """Small databases that are pruned, and their neighbours: against the oracle and the plain loop."""
    r = np.random.default_rng(n + nq)
    codes = r.integers(0, 256, (n, m), dtype=np.uint8)
    luts = (r.random((nq, m, 256)) * 100).astype(np.float32)
    if kind == "few_values":
        luts = np.round(luts / 30)
    if kind == "negative":
        luts -= 60.0
    if kind == "infinite":
        luts[:, 1, 9:200] = np.inf
    got = [host(t) for t in ctx.pq_adc_scan_topk(dev(codes), binding.CODES_U8, dev(luts), topk)]
    opts.set("scan_prune", 0)
    plain = [host(t) for t in ctx.pq_adc_scan_topk(dev(codes), binding.CODES_U8, dev(luts), topk)]
    # (entries of at most 100, m of them: two orders of the additions differ by less than 2 m roundings of 100 m)
    np.testing.assert_allclose(got[0], plain[0], rtol=0, atol=2 * m * 100 * m * 2.0 ** -24)
    if kind == "few_values":   # (whole numbers: no rounding, ids are decided)
        assert np.array_equal(got[0], plain[0]) and np.array_equal(got[1], plain[1])
    if kind == "random":
        od, oi = orc.adc_scan_topk_f32(codes, orc.CODES_U8, luts, topk)
        for q in range(0, nq, 97):
            check_float_topk(got[0][q], got[1][q], od[q], oi[q], codes, orc.CODES_U8, luts[q], n)


@pytest.mark.parametrize("kind", ["random", "far", "infinite", "negative", "cancelling"])
@pytest.mark.parametrize("m", [8, 16])
@pytest.mark.parametrize("n", [8192, 30_001, 65_535])
def test_scan_f32_one_order_of_additions_whatever_the_batch(ctx, opts, m, n, kind):
    """Databases below 65 536 codes are served by the pruned or by the plain loop: a query's distances and ids have the same bits
    in either, alone, in a batch of any size, with any topk, and in the call that allocates nothing."""
    r = np.random.default_rng(n + m)
    codes = dev(r.integers(0, 256, (n, m), dtype=np.uint8))
    tables = (r.random((600, m, 256)) * 100).astype(np.float32)
    if kind == "far":
        tables[:, 2, 7] = 3e20
    if kind == "infinite":
        tables[:, 1, 9:200] = np.inf
    if kind == "negative":
        tables -= 60.0
    if kind == "cancelling":
        tables[:, 0] += 3e5
        tables[:, 5] -= 3e5
    luts = dev(tables)

    def scan(nq, topk, **kw):
        out = ctx.pq_adc_scan_topk(codes, binding.CODES_U8, luts[:nq].contiguous(), topk, **kw)
        return [host(t) for t in out]

    opts.set("scan_prune", 0)
    want_v, want_i = scan(600, 1024)
    opts.set("scan_prune", 1)
    for nq, topk in [(1, 1), (1, 100), (1, 511), (1, 1024), (4, 100), (5, 100), (2, 512), (5, 341), (5, 512), (40, 1000), (100, 512), (150, 800), (300, 512), (400, 800), (512, 100), (600, 100), (600, 1024)]:
        v, i = scan(nq, topk)
        assert np.array_equal(v, want_v[:nq, :topk]) and np.array_equal(i, want_i[:nq, :topk]), (nq, topk)
    for nq, topk in [(1, 1), (1, 100), (4, 100), (5, 128)]:
        out = (torch.empty((nq, topk), dtype=torch.float32, device="cuda"), torch.empty((nq, topk), dtype=torch.int64, device="cuda"))
        v, i = scan(nq, topk, out=out, noalloc=True)
        assert np.array_equal(v, want_v[:nq, :topk]) and np.array_equal(i, want_i[:nq, :topk]), (nq, topk)


@pytest.mark.parametrize("shift", [3e4, 1e6])
@pytest.mark.parametrize("m", [8, 16])
@pytest.mark.parametrize("n,nq,topk", [(4096, 7, 1), (4097, 3, 1000), (5000, 40, 100), (9001, 5, 10), (8192, 1, 100), (30_001, 600, 512), (30_001, 300, 1),
                                       (65_536, 3, 1), (70_000, 300, 512), (70_000, 520, 1), (100_000, 20, 100), (150_000, 4, 1024)])
def test_scan_f32_tables_that_cancel(ctx, m, n, nq, topk, shift):
    """Tables of large entries that cancel (no distances): first bounds and lower bounds must allow for the roundings of the entries'
    magnitudes, not of the distance, else results are lost.  Bit by bit against sums in the order of the scan."""
    r = np.random.default_rng(n + nq)
    codes = r.integers(0, 256, (n, m), dtype=np.uint8)
    tables = (r.random((nq, m, 256)) * 100).astype(np.float32)
    tables[:, 0] += np.float32(shift)
    tables[:, m - 3] -= np.float32(shift)
    v, i = [host(t) for t in ctx.pq_adc_scan_topk(dev(codes), binding.CODES_U8, dev(tables), topk)]
    rows = np.arange(n)
    first = (0 if n >= 65_536 else rows >> 2 if m == 8 else rows) + np.zeros(n, np.int64)
    for q in range(0, nq, 41):
        want = np.zeros(n, np.float32)
        for s in range(m):
            j = (first + s) % m
            want += tables[q, j, codes[rows, j]]
        order = np.lexsort((rows, want))[:topk]
        assert np.array_equal(v[q], want[order]) and np.array_equal(i[q], order), q


@pytest.mark.parametrize("kind", ["both_infinities", "minus_infinity", "nan_with_sign", "nan_rows", "minus_zero"])
@pytest.mark.parametrize("m", [4, 8, 16])
@pytest.mark.parametrize("n,nq,topk", [(100, 3, 20), (4096, 5, 100), (4200, 2, 1000), (9001, 4, 1), (20_001, 600, 300), (33_000, 40, 1000), (66_000, 5, 1), (70_000, 300, 100), (300_001, 2, 1024)])
def test_scan_f32_sums_that_are_no_numbers(ctx, m, n, nq, topk, kind):
    """Tables with infinities of both signs and with NaN of either sign: the result holds the smallest sums that are numbers, minus
    infinity among them, no NaN and nothing at plus infinity, and neither takes the place of a sum in a first bound.  Sums of minus
    zero are results like others."""
    r = np.random.default_rng(n + m)
    codes = r.integers(0, 256, (n, m), dtype=np.uint8)
    tables = (r.random((nq, m, 256)) * 100).astype(np.float32)
    if kind == "both_infinities":
        tables[:, 0, :100] = np.inf
        tables[:, 1, :100] = -np.inf
    if kind == "minus_infinity":
        tables[:, 1, 9] = -np.inf
    if kind == "nan_with_sign":
        tables[:, 2, :64] = np.copysign(np.float32(np.nan), np.float32(-1))
        tables[:, 3, 7] = np.nan
    if kind == "nan_rows":   # every sum but those of 50 codes
        tables[:, 0, 1:] = np.copysign(np.float32(np.nan), np.float32(-1))
        codes[:, 0] = np.maximum(codes[:, 0], 1)
        codes[r.permutation(n)[:50], 0] = 0
    if kind == "minus_zero":
        tables[:] = -0.0
    v, i = [host(t) for t in ctx.pq_adc_scan_topk(dev(codes), binding.CODES_U8, dev(tables), topk)]
    rows = np.arange(n)
    first = (0 if n >= 65_536 or m == 4 else rows >> 2 if m == 8 else rows) + np.zeros(n, np.int64)
    for q in range(0, nq, 41):
        sums = np.zeros(n, np.float32)
        with np.errstate(invalid="ignore"):
            for s in range(m):
                j = (first + s) % m
                sums += tables[q, j, codes[rows, j]]
        number = rows[sums < np.inf]
        order = number[np.lexsort((number, sums[number]))][:topk]
        want_v, want_i = np.full(topk, np.inf, np.float32), np.full(topk, -1, np.int64)
        want_v[:len(order)], want_i[:len(order)] = sums[order], order
        assert np.array_equal(v[q], want_v) and np.array_equal(i[q], want_i), q


@pytest.mark.parametrize("order", ["none", "sorted"])
@pytest.mark.parametrize("topk", [100, 1000])
def test_scan_u4_full_size_both_loops(ctx, opts, order, topk):
    """Config 2's scan on the matrix cores (the default) and by the 16-query loop: the same keys for every query, also where equal
    codes and neighbours are stored side by side."""
    mix = datagen.sift_like()
    cb = dev(datagen.sampled_codebooks(mix, 16, 16))
    codes = torch.cat([ctx.pq_encode(mix.sample_device(1 << 20, 900 + i), cb, orc.CODES_U4_PACKED) for i in range(24)])
    if order == "sorted":
        codes = codes.view(torch.int64).view(-1).sort()[0].view(torch.uint8).view(-1, 8)
    luts = ctx.pq_build_luts(dev(mix.sample(1000, datagen.SEED_QUERIES)), cb)
    qluts, _, _ = ctx.pq_quantize_luts(luts, luts.amin(2).sum(1) * 1.5 + 1.0)
    got = {}
    for option, kernel in ((None, "scan_onehot_kernel"), (0, "scan_tuned_kernel<U4Q_M16")):
        if option is not None:
            opts.set("scan_onehot", option)
        ctx.pq_set_profiling(True)
        try:
            got[kernel] = ctx.pq_adc_scan_topk(codes, orc.CODES_U4_PACKED, qluts, topk)
            name = ctx.pq_last_scan_info()["kernel"]
        finally:
            ctx.pq_set_profiling(False)
        assert name.startswith(kernel) and "again" not in name, name
    (sa, ia), (sb, ib) = got.values()
    assert torch.equal(sa, sb) and torch.equal(ia, ib)


@pytest.mark.parametrize("m", [16, 32])
def test_scan_u4_on_matrix_cores_in_a_captured_graph(m):
    """Every replay gives the results of the tables that it finds, those of queries that are scanned again (32 tables) among them."""
    stream = torch.cuda.Stream()
    g_ctx = binding.Context(0, stream)
    g_ctx.pq_set_option("scan_onehot", 1)
    r = np.random.default_rng(m)
    n, nq, topk = 70_001, 40, 100
    with torch.cuda.stream(stream):
        packed_h = r.integers(0, 256, (n, m // 2), dtype=np.uint8)
        packed, qluts = dev(packed_h), torch.zeros((nq, m, 16), dtype=torch.uint8, device="cuda")
        g_ctx.pq_adc_scan_topk(packed, orc.CODES_U4_PACKED, qluts, topk)   # (the workspace)
        stream.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=stream):
            s, i = g_ctx.pq_adc_scan_topk(packed, orc.CODES_U4_PACKED, qluts, topk)
        for turn in range(4):
            tables = np.minimum(255, r.standard_normal((nq, m, 16)) ** 2 * r.uniform(5, 40, (nq, m, 1))).astype(np.uint8)
            tables[::7 + turn] = 255
            qluts.copy_(torch.from_numpy(tables))
            graph.replay()
            gs, gi = host(s), host(i)
            check_exact_topk(gs, gi, *orc.adc_scan_topk_u8(packed_h, orc.CODES_U4_PACKED, tables, topk))
            # eager work on the same workspace between the replays
            es, ei = g_ctx.pq_adc_scan_topk(packed, orc.CODES_U4_PACKED, qluts[: 3 + turn].contiguous(), topk)
            assert np.array_equal(host(es), gs[: 3 + turn]) and np.array_equal(host(ei), gi[: 3 + turn])
    g_ctx.close()
