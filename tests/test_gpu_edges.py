"""Edges of what the kernels accept: the last bytes of their LDS, values that overflow, grid limits,
batches and candidate buffers at which another route takes over.  Everything is compared with the
oracle bit for bit (same operation order: no tolerance)."""
import numpy as np
import pytest
import torch

import oracle
from paper_2312_01712_amd import workloads as wl

pytestmark = pytest.mark.gpu


def _binding():
    from paper_2312_01712_amd import binding
    return binding


def _index(rng, D, M, sizes, spread=0.3, centre=1.0):
    offs = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
    N, nlist = int(offs[-1]), len(sizes)
    return wl.Index(N=N, D=D, nlist=nlist, M=M, centroids=(centre * rng.normal(size=(nlist, D))).astype(np.float32),
                    codebooks=(spread * rng.normal(size=(M, 256, D // M))).astype(np.float32), list_offsets=offs,
                    codes=rng.integers(0, 256, size=(N, M), dtype=np.uint8), ids=rng.permutation(N).astype(np.int64))


def _same(got, want, what):
    torch.cuda.synchronize()
    assert np.array_equal(got[0].cpu().numpy(), want[0]), f"{what}: ids differ"
    assert np.array_equal(got[1].cpu().numpy().view(np.uint32), want[1].view(np.uint32)), f"{what}: distances differ"


@pytest.mark.parametrize("M,D", [(100, 100), (100, 300), (100, 400), (64, 256)])
def test_inner_product_last_suffix_sums(M, D):
    """Inner products where the suffix sums of the row minima lie at the very end of the LDS: with
    100 subspaces of 4 the allocation's rounding leaves 40 bytes behind what is asked for."""
    b = _binding()
    rng = np.random.default_rng(D)
    idx = _index(rng, D, M, rng.integers(100, 900, size=40))
    q = rng.normal(size=(40, D)).astype(np.float32)
    gi = b.IvfPqIndex.from_index(idx, metric=b.METRIC_IP)
    for radii in (np.full(M, np.inf, np.float32), np.full(M, 0.8 * np.sqrt(D / M), np.float32)):
        for k in (1, 10, 100):
            _same(gi.search(torch.from_numpy(q).cuda(), 12, k, radii), oracle.search(q, idx, 12, k, radii, threads=8, metric=1), (M, D, k))
    gi.close()


@pytest.mark.parametrize("nlist", [200, 700])
@pytest.mark.parametrize("Q", [1, 9])
def test_filtering_with_infinite_centroids(nlist, Q):
    """Inner products with centroids that are infinite where the query is zero are NaN: the other lists
    come first, in order, as where every distance is formed and sorted."""
    b = _binding()
    rng = np.random.default_rng(nlist)
    cent = np.zeros((nlist, 2), np.float32)
    cent[:, 1] = rng.permutation(nlist) - nlist // 2
    bad = rng.permutation(nlist)[:nlist // 3]
    cent[bad, 0] = np.inf
    q = np.tile(np.array([[0.0, 1.0]], np.float32), (Q, 1))
    real = np.setdiff1d(np.arange(nlist), bad)
    score = np.float32(0) - cent[real, 1]
    order = real[np.lexsort((real, score))]
    gi = b.IvfPqIndex(cent, rng.normal(size=(1, 256, 2)).astype(np.float32), np.arange(nlist + 1, dtype=np.int64),
                      np.zeros((nlist, 1), dtype=np.uint8), metric=b.METRIC_IP)
    for nprobe in (1, 60, 90, 101):
        pid, pd = gi.coarse(torch.from_numpy(q).cuda(), nprobe)
        torch.cuda.synchronize()
        for row, dist in zip(pid.cpu().numpy(), pd.cpu().numpy()):
            assert np.array_equal(row, order[:nprobe]), nprobe
            assert np.array_equal(dist, np.sort(score)[:nprobe]), nprobe
    gi.close()


# (at 8 probes the proposals come from keys from 4481 lists on)
@pytest.mark.parametrize("nlist,D,Q", [(4481, 32, 257), (5000, 64, 100), (4737, 260, 90)])
@pytest.mark.parametrize("what", ["plain", "worst"])
@pytest.mark.parametrize("metric", [0, 1])
def test_split_product_bound(nlist, D, Q, what, metric):
    """Depths of whole slices and with 16-byte loads, and values whose split product drops most: all
    of one sign and near 1 + 2^-8, so that the dropped parts add up instead of averaging out."""
    b = _binding()
    rng = np.random.default_rng(nlist + D)
    if what == "plain":
        c = rng.normal(size=(nlist, D)).astype(np.float32)
        q = (c[rng.integers(0, nlist, Q)] + 0.5 * rng.normal(size=(Q, D))).astype(np.float32)
    else:   # two populations: mantissas that drop 3e-5 and ones that drop nothing, norms alike
        c = np.where(rng.random((nlist, 1)) < 0.5, 1.0039136, 1.0).astype(np.float32) * np.ones((1, D), np.float32)
        c += (2e-5 * rng.normal(size=c.shape)).astype(np.float32)
        q = np.full((Q, D), 1.0039136, np.float32) + (2e-5 * rng.normal(size=(Q, D))).astype(np.float32)
    gi = b.IvfPqIndex(c, rng.normal(size=(1, 256, D)).astype(np.float32), np.arange(nlist + 1, dtype=np.int64),
                      np.zeros((nlist, 1), dtype=np.uint8), metric=metric)
    b.coarse_fallbacks(reset=True)
    got = gi.coarse(torch.from_numpy(q).cuda(), 8)
    torch.cuda.synchronize()
    fb = b.coarse_fallbacks()
    _same(got, oracle.coarse(q, c, 8, metric=metric), (nlist, D, what))
    if what == "plain" and metric == 0:
        assert fb <= Q // 20, f"{fb} of {Q} queries were not accepted from the proposal"
    gi.close()


@pytest.mark.parametrize("metric", [0, 1])
def test_filtering_of_more_than_a_million_queries(metric):
    """Few lists and dimensions leave a batch of millions within what is done without a matrix product:
    65 536 tiles of 16 queries and one more."""
    b = _binding()
    rng = np.random.default_rng(3)
    nlist, D, Q = 40, 3, 65_536 * 16 + 1
    c = rng.normal(size=(nlist, D)).astype(np.float32)
    some = rng.normal(size=(4096, D)).astype(np.float32)
    q = torch.from_numpy(some).cuda().repeat(257, 1)[:Q].contiguous()
    gi = b.IvfPqIndex(c, rng.normal(size=(1, 256, D)).astype(np.float32), np.arange(nlist + 1, dtype=np.int64),
                      np.zeros((nlist, 1), dtype=np.uint8), metric=metric)
    pid, pd = gi.coarse(q, 5)
    o_pid, o_pd = oracle.coarse(some, c, 5, metric=metric)
    _same((pid[:4096], pd[:4096]), (o_pid, o_pd), "first queries")
    for got in (pid, pd.view(torch.int32)):
        assert torch.equal(got, got[:4096].repeat(257, 1)[:Q])
    gi.close()


@pytest.mark.parametrize("M,dsub", [(2, 10), (3, 12), (5, 7), (7, 9), (9, 16), (17, 14), (33, 20), (65, 11), (1, 40)])
@pytest.mark.parametrize("mode", [0, 1, 2])
def test_run_time_dimension_of_the_subspaces(M, dsub, mode):
    """Codebook rows in loads of 4, 8 and 16 bytes: dsub odd, even and a multiple of 4, beyond the ones
    whose entries are whole 16-byte pieces; short last groups of every kind of length."""
    b = _binding()
    rng = np.random.default_rng(M * 100 + dsub)
    D = M * dsub
    idx = _index(rng, D, M, np.array([0, 1, 64, 65, 700, 300, 129, 1000, 63, 400]))
    q = (idx.centroids[rng.integers(0, 10, 40)] + 0.3 * rng.normal(size=(40, D))).astype(np.float32)
    radii = np.full(M, 0.45 * np.sqrt(dsub), dtype=np.float32)
    gi = b.IvfPqIndex.from_index(idx)
    for Q, nprobe, k in ((40, 6, 10), (2, 9, 128), (40, 9, 300)):
        _same(gi.search(torch.from_numpy(q[:Q]).cuda(), nprobe, k, radii, mode=mode),
              oracle.search(q[:Q], idx, nprobe, k, radii, threads=8, mode=mode), (M, dsub, k))
    gi.close()


def _rounds(q, idx, pid, k, radii, mode, first_probes, cap):
    """How the list-major scan sees each query: overflows in the first round of its main pass (probes 1 to
    first_probes, filtered by the k-th distance of the nearest list), only in the second (the other
    probes, filtered by the k-th distance so far), or never."""
    offs, dist, _ = oracle.scan_all(q, idx, pid, radii, mode=mode)
    lens = np.diff(idx.list_offsets)[pid]
    out = []
    for i in range(q.shape[0]):
        d, ends = dist[offs[i]:offs[i + 1]], np.concatenate([[0], np.cumsum(lens[i])])
        head, near = d[:ends[1]], d[:ends[1 + first_probes]]
        tau = np.sort(head)[k - 1] if head.size >= k else np.inf
        if (near[ends[1]:] <= tau).sum() > cap:
            out.append("first")
            continue
        tau = np.sort(near)[k - 1] if near.size >= k else np.inf
        out.append("second" if (d[ends[1 + first_probes]:] <= tau).sum() > cap else "never")
    return out


@pytest.mark.parametrize("D,M", [(96, 48), (128, 64), (64, 16)])
@pytest.mark.parametrize("mode", [0, 1, 2])
def test_candidates_that_overflow_in_either_round(D, M, mode):
    """Enough probes for two rounds of the list-major main pass and candidate buffers of 64 slots: queries
    that overflow in the first round stay out of the second and are still redone, like those that overflow
    in the second; over 4096 queries, so that the redoing workgroups serve several queries each."""
    b = _binding()
    rng = np.random.default_rng(M + mode)
    nlist, k, cap, nprobe, distinct = 70, 10, 64, 52, 200
    idx = _index(rng, D, M, rng.integers(40, 260, size=nlist), centre=0.04)
    q = (idx.centroids[rng.integers(0, nlist, distinct)] + 0.25 * rng.normal(size=(distinct, D))).astype(np.float32)
    q[::3] = idx.centroids[rng.integers(0, nlist, len(q[::3]))]
    radii = np.full(M, (0.6 if mode == 0 else 0.45) * np.sqrt(D / M), dtype=np.float32)
    want = oracle.search(q, idx, nprobe, k, radii, threads=8, mode=mode)
    pid, _ = oracle.coarse(q, idx.centroids, nprobe)
    kinds = _rounds(q, idx, pid, k, radii, mode, 7, cap)
    assert min(kinds.count(x) for x in ("first", "second", "never")) >= 3, {x: kinds.count(x) for x in set(kinds)}
    gi = b.IvfPqIndex.from_index(idx)
    try:
        b.set_option("lm_cap", cap)
        for reps in (1, 22):
            Q = distinct * reps
            got = gi.search(torch.from_numpy(q).cuda().repeat(reps, 1), nprobe, k, radii, mode=mode, strategy=b.SCAN_LIST_MAJOR)
            _same(got, (np.tile(want[0], (reps, 1)), np.tile(want[1], (reps, 1))), (D, M, mode, Q))
    finally:
        b.set_option("lm_cap", 0)
        gi.close()


@pytest.mark.parametrize("metric", [0, 1])
@pytest.mark.parametrize("name", ["all equal", "two values", "tiny jitter", "duplicates", "zero"])
def test_row_proposals_that_are_not_accepted(name, metric):
    """Few lists (up to 4096), and a batch too large for the path without a matrix product (more than 4.5e8
    query x list x dimension products): degenerate centroids, where the proposal's window cannot separate the
    lists, its collection overflows, and the flagged queries go to the second line."""
    b = _binding()
    rng = np.random.default_rng(len(name))
    D, distinct, reps = 16, 40, 235
    cent = {
        "all equal": lambda: np.tile(rng.normal(size=(1, D)), (4000, 1)),
        "two values": lambda: np.repeat(rng.normal(size=(2, D)), 1800, axis=0),
        "tiny jitter": lambda: rng.normal(size=(1, D)) + 1e-7 * rng.normal(size=(3000, D)),
        "duplicates": lambda: np.concatenate([rng.normal(size=(300, D)), rng.normal(size=(300, D))[rng.integers(0, 300, 3300)]]),
        "zero": lambda: np.zeros((3100, D)),
    }[name]().astype(np.float32)
    nlist = len(cent)
    assert distinct * reps * nlist * D > 450_000_000
    q = rng.normal(size=(distinct, D)).astype(np.float32)
    dq = torch.from_numpy(q).cuda().repeat(reps, 1)
    gi = b.IvfPqIndex(cent, rng.normal(size=(1, 256, D)).astype(np.float32), np.arange(nlist + 1, dtype=np.int64),
                      np.zeros((nlist, 1), dtype=np.uint8), metric=metric)
    b.coarse_fallbacks(reset=True)
    for nprobe in (1, 10, 100, 200):
        o_pid, o_pd = oracle.coarse(q, cent, nprobe, metric=metric)
        _same(gi.coarse(dq, nprobe), (np.tile(o_pid, (reps, 1)), np.tile(o_pd, (reps, 1))), (name, nprobe))
    assert name == "duplicates" or b.coarse_fallbacks() > 0
    gi.close()


@pytest.mark.parametrize("D,M", [(96, 48), (128, 64), (64, 16)])
@pytest.mark.parametrize("k,cap,radius", [(129, 8192, 0.6), (500, 8192, 0.6), (1000, 8192, 0.6), (700, 1024, 0.6), (300, 2048, np.inf)])
def test_more_than_128_neighbours_of_large_batches(D, M, k, cap, radius):
    """k above 128 in batches whose later probes are scanned list-major behind the first few: queries that one list
    answers, queries between the lists, many equal distances, empty lists, probes that hold fewer than k
    points at first, shared and per-query radii, and the query-major scan of the same call.  (1024 slots do not hold
    twice the first lists of k = 700: query-major throughout, with slots that overflow.)"""
    b = _binding()
    rng = np.random.default_rng(M + k)
    nlist, nprobe, distinct, reps = 60, 40, 100, 5
    sizes = rng.integers(100, 420, size=nlist)
    sizes[:3] = (0, 1, 64)
    idx = _index(rng, D, M, sizes, centre=0.15)
    idx.codes[idx.list_offsets[5]:idx.list_offsets[8]] = idx.codes[0]   # runs of equal distances
    q = (idx.centroids[rng.integers(0, nlist, distinct)] + 0.25 * rng.normal(size=(distinct, D))).astype(np.float32)
    q[::3] = idx.centroids[rng.integers(0, nlist, len(q[::3]))]
    radii = np.full(M, radius * np.sqrt(D / M), dtype=np.float32)
    per_query = np.where(np.isinf(radius), np.inf, rng.uniform(0.3, 0.9, size=(distinct, M)) * np.sqrt(D / M)).astype(np.float32)
    gi = b.IvfPqIndex.from_index(idx)
    dq = torch.from_numpy(q).cuda().repeat(reps, 1)
    try:
        b.set_option("wide_cap", cap)
        for own in (None, per_query):
            want = oracle.search(q, idx, nprobe, k, radii if own is None else own, threads=8)
            want = (np.tile(want[0], (reps, 1)), np.tile(want[1], (reps, 1)))
            rq = None if own is None else torch.from_numpy(own).cuda().repeat(reps, 1)
            for strategy in (b.SCAN_AUTO, b.SCAN_QUERY_MAJOR):
                got = gi.search(dq, nprobe, k, radii if own is None else None, query_radii=rq, strategy=strategy)
                _same(got, want, (D, M, k, cap, own is not None, strategy))
    finally:
        b.set_option("wide_cap", 8192)
        gi.close()


@pytest.mark.parametrize("D,M", [(96, 48), (128, 64), (64, 16)])
@pytest.mark.parametrize("k,cap,radius", [(1, 0, 0.6), (100, 0, 0.6), (128, 64, 0.6), (10, 0, np.inf)])
def test_long_lists_shared_by_many_queries(D, M, k, cap, radius):
    """Lists above 4096 points on average and batches that share them: the head pass with byte tables (histogram of the
    byte sums, candidates up to the k-th and what the bytes can have lost).  Nearest lists that are empty or hold fewer
    points than k, queries between the lists, runs of equal distances, candidate buffers of 64 slots, infinite, shared and
    per-query radii; groups of eight queries and of fewer; the query-major scan of the same call."""
    b = _binding()
    rng = np.random.default_rng(7 * M + k)
    sizes = np.array([9100, 0, 8300, 90, 12_000, 1, 8800, 9900])
    nlist, nprobe, distinct, reps = len(sizes), 6, 60, 46
    idx = _index(rng, D, M, sizes, centre=0.2)
    idx.codes[idx.list_offsets[2] + 50:idx.list_offsets[2] + 400] = idx.codes[0]   # runs of equal distances
    q = (idx.centroids[rng.integers(0, nlist, distinct)] + 0.25 * rng.normal(size=(distinct, D))).astype(np.float32)
    q[::3] = idx.centroids[rng.integers(0, nlist, len(q[::3]))]
    radii = np.full(M, radius * np.sqrt(D / M), dtype=np.float32)
    per_query = np.where(np.isinf(radius), np.inf, rng.uniform(0.3, 0.9, size=(distinct, M)) * np.sqrt(D / M)).astype(np.float32)
    gi = b.IvfPqIndex.from_index(idx)
    try:
        b.set_option("lm_cap", cap)
        assert gi.resolve_strategy(distinct * reps, nprobe, k) == b.SCAN_LIST_MAJOR
        assert gi.resolve_strategy(distinct, nprobe, k) == b.SCAN_QUERY_MAJOR
        small = gi.workspace(distinct * reps, nprobe, k, strategy=b.SCAN_QUERY_MAJOR)   # serves AUTO query-major
        want = oracle.search(q, idx, nprobe, k, radii, threads=8)
        _same(gi.search(torch.from_numpy(q).cuda().repeat(reps, 1), nprobe, k, radii, workspace=small),
              (np.tile(want[0], (reps, 1)), np.tile(want[1], (reps, 1))), (D, M, k, cap, "small workspace"))
        for own in (None, per_query):
            want = oracle.search(q, idx, nprobe, k, radii if own is None else own, threads=8)
            for n, strategy in ((reps, b.SCAN_AUTO), (reps - 20, b.SCAN_LIST_MAJOR), (1, b.SCAN_LIST_MAJOR), (1, b.SCAN_QUERY_MAJOR)):
                dq = torch.from_numpy(q).cuda().repeat(n, 1)
                rq = None if own is None else torch.from_numpy(own).cuda().repeat(n, 1)
                got = gi.search(dq, nprobe, k, radii if own is None else None, query_radii=rq, strategy=strategy)
                _same(got, (np.tile(want[0], (n, 1)), np.tile(want[1], (n, 1))), (D, M, k, cap, n, own is not None, strategy))
    finally:
        b.set_option("lm_cap", 0)
        gi.close()


@pytest.mark.parametrize("D,M,spread,sigma,radius,wide", [
    (64, 16, 0.3, 1.0, 0.049, 1.0), (64, 16, 0.3, 1.0, 0.053, 1.0), (64, 16, 0.3, 3.0, 0.1, 1.0), (64, 16, 0.3, 3.0, 0.164, 1.0),
    (64, 16, 1.0, 1.0, 0.1, 1.0), (64, 16, 1.0, 0.3, 0.6, 35.0), (96, 48, 0.3, 3.0, 0.122, 1.0), (96, 48, 0.3, 3.0, 0.05, 1.0),
    (128, 64, 0.3, 3.0, 0.09, 1.0), (128, 64, 0.3, 1.0, 0.0, 1.0)])
def test_long_lists_with_radii_far_below_the_residuals(D, M, spread, sigma, radius, wide):
    """The nearest list ranked with byte tables where squared distances to the entries lie a thousand times and more above
    the largest squared radius (values in the tables' units beyond 2^16, where a byte is cut from bits that wrap), and
    where one subspace is much wider than the others."""
    b = _binding()
    rng = np.random.default_rng(M + int(1000 * radius))
    sizes = np.array([9100, 0, 8300, 90, 12_000, 1, 8800, 9900])
    nlist, nprobe, distinct, reps = len(sizes), 6, 60, 46
    idx = _index(rng, D, M, sizes, spread=spread, centre=0.01)
    idx.codebooks[0] *= np.float32(wide)
    q = (idx.centroids[rng.integers(0, nlist, distinct)] + sigma * rng.normal(size=(distinct, D))).astype(np.float32)
    radii = np.full(M, radius, dtype=np.float32)
    gi = b.IvfPqIndex.from_index(idx)
    dq = torch.from_numpy(q).cuda().repeat(reps, 1)
    try:
        b.set_option("lm_cap", 65536)   # (no query is redone for want of slots, which would cover up what the tables miss)
        assert gi.resolve_strategy(distinct * reps, nprobe, 10) == b.SCAN_LIST_MAJOR
        for k in (1, 10, 100):
            want = oracle.search(q, idx, nprobe, k, radii, threads=8)
            _same(gi.search(dq, nprobe, k, radii), (np.tile(want[0], (reps, 1)), np.tile(want[1], (reps, 1))), (D, M, sigma, radius, k))
    finally:
        b.set_option("lm_cap", 0)
        gi.close()


@pytest.mark.parametrize("D,M", [(96, 48), (128, 64), (64, 16)])
@pytest.mark.parametrize("radius", [0.0, 0.02, 0.06])
def test_more_candidates_than_a_task_holds(D, M, radius):
    """Radii that hold next to nothing: most points of most lists are candidates of all eight queries of a task, more than
    its queue takes and, of all lists, more than a query has slots."""
    b = _binding()
    rng = np.random.default_rng(M)
    nlist, nprobe, distinct, reps = 40, 32, 64, 8
    idx = _index(rng, D, M, rng.integers(600, 1100, size=nlist), centre=0.05)
    q = (idx.centroids[rng.integers(0, nlist, distinct)] + 0.3 * rng.normal(size=(distinct, D))).astype(np.float32)
    radii = np.full(M, radius, dtype=np.float32)
    gi = b.IvfPqIndex.from_index(idx)
    dq = torch.from_numpy(q).cuda().repeat(reps, 1)
    try:
        for cap in (0, 65536):
            b.set_option("lm_cap", cap)
            assert gi.resolve_strategy(distinct * reps, nprobe, 10) == b.SCAN_LIST_MAJOR
            for k in (1, 10, 100):
                want = oracle.search(q, idx, nprobe, k, radii, threads=8)
                _same(gi.search(dq, nprobe, k, radii), (np.tile(want[0], (reps, 1)), np.tile(want[1], (reps, 1))), (D, M, radius, cap, k))
    finally:
        b.set_option("lm_cap", 0)
        gi.close()


@pytest.mark.parametrize("D,M", [(96, 48), (128, 64), (64, 16)])
@pytest.mark.parametrize("k,radius", [(1, 0.6), (100, 0.6), (100, 1.5), (100, 0.05), (10, np.inf)])
def test_long_lists_in_two_main_passes(D, M, k, radius):
    """Enough probes for two main passes behind a head pass with byte tables: queries whose nearest list it ranks, queries it
    only finds any k points for (wide, infinite and very small radii), lists shorter than k, empty ones and runs of equal
    distances; radii per query that are NaN (they cut nothing off)."""
    b = _binding()
    rng = np.random.default_rng(M + k)
    nlist, nprobe, distinct, reps = 56, 50, 40, 110
    sizes = rng.integers(3900, 5000, size=nlist)
    sizes[:3] = (0, 40, 11_000)
    idx = _index(rng, D, M, sizes, centre=0.05)
    idx.codes[idx.list_offsets[9] + 50:idx.list_offsets[9] + 400] = idx.codes[0]
    q = (idx.centroids[rng.integers(0, nlist, distinct)] + 0.25 * rng.normal(size=(distinct, D))).astype(np.float32)
    q[::3] = idx.centroids[rng.integers(0, nlist, len(q[::3]))]
    radii = np.full(M, radius * np.sqrt(D / M), dtype=np.float32)
    gi = b.IvfPqIndex.from_index(idx)
    dq = torch.from_numpy(q).cuda().repeat(reps, 1)
    assert gi.resolve_strategy(distinct * reps, nprobe, k) == b.SCAN_LIST_MAJOR
    want = oracle.search(q, idx, nprobe, k, radii, threads=8)
    want = (np.tile(want[0], (reps, 1)), np.tile(want[1], (reps, 1)))
    for strategy in (b.SCAN_AUTO, b.SCAN_LIST_MAJOR, b.SCAN_QUERY_MAJOR):
        _same(gi.search(dq, nprobe, k, radii, strategy=strategy), want, (D, M, k, radius, strategy))
    own = np.tile(radii, (distinct, 1))
    own[::2, 3] = np.nan
    rq = torch.from_numpy(own).cuda().repeat(reps, 1)
    ref = gi.search(dq, nprobe, k, None, query_radii=rq, strategy=b.SCAN_QUERY_MAJOR)
    ref = (ref[0].cpu().numpy(), ref[1].cpu().numpy())
    _same(gi.search(dq, nprobe, k, None, query_radii=rq), ref, (D, M, k, radius, "NaN radii"))
    gi.close()


@pytest.mark.parametrize("D,M", [(96, 48), (64, 16)])
def test_long_lists_with_entries_that_are_nan(D, M):
    """Codebook entries that are NaN count as outside of every radius: list-major as query-major."""
    b = _binding()
    rng = np.random.default_rng(D)
    sizes = np.array([9100, 8300, 5000, 12_000, 8800, 9900])
    nprobe, distinct, reps = 5, 50, 56
    idx = _index(rng, D, M, sizes, centre=0.2)
    idx.codebooks[2, 5:40] = np.nan
    idx.codebooks[M - 1, 100, 0] = np.nan
    q = (idx.centroids[rng.integers(0, len(sizes), distinct)] + 0.25 * rng.normal(size=(distinct, D))).astype(np.float32)
    gi = b.IvfPqIndex.from_index(idx)
    dq = torch.from_numpy(q).cuda().repeat(reps, 1)
    for radius in (0.6, 3.0, 20.0):
        radii = np.full(M, radius, dtype=np.float32)
        for k in (1, 100):
            ref = gi.search(dq, nprobe, k, radii, strategy=b.SCAN_QUERY_MAJOR)
            ref = (ref[0].cpu().numpy(), ref[1].cpu().numpy())
            _same(gi.search(dq, nprobe, k, radii, strategy=b.SCAN_LIST_MAJOR), ref, (D, M, radius, k))
    gi.close()


@pytest.mark.parametrize("D,M", [(96, 48), (128, 64), (64, 16)])
def test_which_batches_are_selected_list_major_above_128_neighbours(D, M):
    """The stages' tables are asked for where the batch is large against the share of a list that k is, and not for small
    batches of few neighbours, which the query-major scan serves in fewer launches; both return the same."""
    b = _binding()
    rng = np.random.default_rng(M)
    nlist, nprobe, distinct = 60, 32, 64
    idx = _index(rng, D, M, rng.integers(900, 1050, size=nlist), centre=0.3)
    gi = b.IvfPqIndex.from_index(idx)

    def staged(Q, k):
        return gi.workspace_bytes(Q, nprobe, k) > gi.workspace_bytes(Q, nprobe, k, strategy=b.SCAN_QUERY_MAJOR)

    assert not staged(512, 129) and not staged(512, 300)
    assert staged(512, 1000) and staged(8192, 129) and staged(8192, 300)
    assert staged(1200, 129) == (M > 16)
    q = (idx.centroids[rng.integers(0, nlist, distinct)] + 0.25 * rng.normal(size=(distinct, D))).astype(np.float32)
    radii = np.full(M, 0.6 * np.sqrt(D / M), dtype=np.float32)
    dq = torch.from_numpy(q).cuda()
    for k, reps in ((129, 8), (600, 8), (300, 35)):
        want = oracle.search(q, idx, nprobe, k, radii, threads=8)
        _same(gi.search(dq.repeat(reps, 1), nprobe, k, radii), (np.tile(want[0], (reps, 1)), np.tile(want[1], (reps, 1))), (D, M, k, reps))
    gi.close()


def test_large_batches_on_long_lists_go_in_pieces():
    """AUTO on long lists: the workspace's candidate slots do not grow with the batch beyond 1 GiB (or 4096 queries), and
    batches beyond that return what the query-major scan does: two pieces, the last one short, shared and per-query
    radii, search and scan_topk."""
    b = _binding()
    rng = np.random.default_rng(11)
    D, M, nprobe, k, distinct, reps = 64, 16, 6, 10, 60, 75
    sizes = np.array([9100, 0, 8300, 90, 12_000, 1, 8800, 9900])
    idx = _index(rng, D, M, sizes, centre=0.2)
    q = (idx.centroids[rng.integers(0, len(sizes), distinct)] + 0.25 * rng.normal(size=(distinct, D))).astype(np.float32)
    radii = np.full(M, 1.2, dtype=np.float32)
    per_query = rng.uniform(0.6, 1.8, size=(distinct, M)).astype(np.float32)
    gi = b.IvfPqIndex.from_index(idx)

    def slots(Q, nprobe):
        return gi.workspace_bytes(Q, nprobe, k) - gi.workspace_bytes(Q, nprobe, k, strategy=b.SCAN_QUERY_MAJOR)

    try:
        for Q in (8192, 100_000, 1_000_000):
            assert gi.resolve_strategy(Q, nprobe, k) == b.SCAN_LIST_MAJOR
            assert slots(Q, nprobe) < (1 << 30) + (16 << 20), Q
        b.set_option("lm_cap", 65536)   # 4096 queries a piece
        assert slots(1_000_000, nprobe) == slots(distinct * reps, nprobe) == slots(4096, nprobe) > slots(4000, nprobe)
        assert gi.resolve_strategy(distinct * reps, nprobe, k) == b.SCAN_LIST_MAJOR
        dq = torch.from_numpy(q).cuda().repeat(reps, 1)
        for own in (None, per_query):
            want = oracle.search(q, idx, nprobe, k, radii if own is None else own, threads=8)
            want = (np.tile(want[0], (reps, 1)), np.tile(want[1], (reps, 1)))
            rq = None if own is None else torch.from_numpy(own).cuda().repeat(reps, 1)
            shared = radii if own is None else None
            _same(gi.search(dq, nprobe, k, shared, query_radii=rq), want, "search")
            _same(gi.scan_topk(dq, gi.coarse(dq, nprobe)[0], k, shared, query_radii=rq), want, "scan_topk")
    finally:
        b.set_option("lm_cap", 0)
        gi.close()


@pytest.mark.parametrize("D,M", [(96, 48), (128, 64), (64, 16)])
@pytest.mark.parametrize("radius", [0.6, np.inf])
def test_first_lists_that_the_wide_slots_do_not_hold(D, M, radius):
    """k above 128 selected list-major in stages where some queries' first lists are several times the mean and alone hold
    more points than a query has slots (those queries start over query-major), beside queries whose first lists fit."""
    b = _binding()
    rng = np.random.default_rng(M)
    nlist, nprobe, distinct, reps, k, cap, first = 60, 40, 96, 6, 300, 2048, 3
    sizes = rng.integers(100, 300, size=nlist)
    sizes[:6] = rng.integers(950, 1250, size=6)
    idx = _index(rng, D, M, sizes, centre=0.3)
    near = np.float32(0.05) * rng.normal(size=(6, D)).astype(np.float32)
    idx.centroids[:6] = idx.centroids[0] + near        # the long lists lie together
    assert -(-2 * k * nlist // int(sizes.sum())) == first and first * 2 * sizes.sum() <= cap * nlist
    q = (idx.centroids[rng.integers(0, nlist, distinct)] + 0.25 * rng.normal(size=(distinct, D))).astype(np.float32)
    q[::3] = idx.centroids[0] + np.float32(0.1) * rng.normal(size=(len(q[::3]), D)).astype(np.float32)
    radii = np.full(M, radius * np.sqrt(D / M), dtype=np.float32)
    gi = b.IvfPqIndex.from_index(idx)
    dq = torch.from_numpy(q).cuda()
    try:
        b.set_option("wide_cap", cap)
        seeds = sizes[gi.coarse(dq, nprobe)[0].cpu().numpy()[:, :first]].sum(1)
        assert np.any(seeds > cap) and np.any(seeds <= cap)
        dq = dq.repeat(reps, 1)
        assert gi.workspace_bytes(len(dq), nprobe, k) > gi.workspace_bytes(len(dq), nprobe, k, strategy=b.SCAN_QUERY_MAJOR)
        want = oracle.search(q, idx, nprobe, k, radii, threads=8)
        _same(gi.search(dq, nprobe, k, radii), (np.tile(want[0], (reps, 1)), np.tile(want[1], (reps, 1))), (D, M, radius))
    finally:
        b.set_option("wide_cap", 8192)
        gi.close()


@pytest.mark.parametrize("D,M", [(96, 48), (64, 16)])
def test_stages_above_128_neighbours_in_two_chunks(D, M):
    """So many slots a query that the batch goes through them in two chunks, the second one short: counters and tables of
    the stages serve both, with shared and with per-query radii."""
    b = _binding()
    rng = np.random.default_rng(M + 1)
    nlist, nprobe, distinct, reps, k = 60, 32, 60, 25, 300
    idx = _index(rng, D, M, rng.integers(150, 400, size=nlist), centre=0.15)
    q = (idx.centroids[rng.integers(0, nlist, distinct)] + 0.25 * rng.normal(size=(distinct, D))).astype(np.float32)
    radii = np.full(M, 0.6 * np.sqrt(D / M), dtype=np.float32)
    per_query = (rng.uniform(0.3, 0.9, size=(distinct, M)) * np.sqrt(D / M)).astype(np.float32)
    gi = b.IvfPqIndex.from_index(idx)
    dq = torch.from_numpy(q).cuda().repeat(reps, 1)
    try:
        b.set_option("wide_cap", 65536)
        chunk = (1 << 30) // (65536 * 12)
        assert chunk < len(dq) < 2 * chunk
        assert gi.workspace_bytes(len(dq), nprobe, k) > gi.workspace_bytes(len(dq), nprobe, k, strategy=b.SCAN_QUERY_MAJOR)
        for own in (None, per_query):
            want = oracle.search(q, idx, nprobe, k, radii if own is None else own, threads=8)
            rq = None if own is None else torch.from_numpy(own).cuda().repeat(reps, 1)
            _same(gi.search(dq, nprobe, k, radii if own is None else None, query_radii=rq),
                  (np.tile(want[0], (reps, 1)), np.tile(want[1], (reps, 1))), (D, M, own is not None))
    finally:
        b.set_option("wide_cap", 8192)
        gi.close()


@pytest.mark.parametrize("D,M", [(96, 48), (128, 64), (64, 16), (200, 100), (160, 80)])
@pytest.mark.parametrize("lm_cap", [0, 64])
def test_candidates_settled_together(D, M, lm_cap):
    """Byte tables in batches of one query, of fewer and of more than one per workgroup, of 4097 (queries to be redone are
    listed) and of more than 64 per workgroup (a wavefront a query); queries without candidates, with a few and with
    thousands, in one main pass and in two, and buffers of 64 slots that overflow; 80 subspaces (fp32
    tables) hand over by a map instead of a list."""
    b = _binding()
    rng = np.random.default_rng(M + lm_cap)
    nlist, distinct = 72, 41
    idx = _index(rng, D, M, rng.integers(600, 1100, size=nlist), centre=0.05)
    idx.centroids[:20] *= np.float32(8.0)   # lists of their own: nothing elsewhere is near their queries
    q = (idx.centroids[rng.integers(0, nlist, distinct)] + 0.3 * rng.normal(size=(distinct, D))).astype(np.float32)
    radii = np.full(M, 0.5 * np.sqrt(D / M), dtype=np.float32)
    gi = b.IvfPqIndex.from_index(idx)
    try:
        b.set_option("lm_cap", lm_cap)
        for nprobe, k in ((24, 10), (64, 100)):
            want = oracle.search(q, idx, nprobe, k, radii, threads=8)
            for Q in (1, 255, 257, 4097, 16_385 if nprobe == 24 else 1000):
                rows = np.arange(Q) % distinct
                got = gi.search(torch.from_numpy(q[rows]).cuda(), nprobe, k, radii, strategy=b.SCAN_LIST_MAJOR)
                _same(got, (want[0][rows], want[1][rows]), (D, M, lm_cap, nprobe, k, Q))
    finally:
        b.set_option("lm_cap", 0)
        gi.close()
