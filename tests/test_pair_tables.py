"""fp32 tables of two queries that go by in parts (lm_pair_kernel): searches that take them, at the edges of blocks, segments
and of what the head pass holds, against the oracle bit for bit."""
import numpy as np
import pytest

import oracle
from paper_2312_01712_amd import workloads as wl


def _index(rng, D, M, sizes, spread=0.3, centre=0.05):
    offs = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
    N, nlist = int(offs[-1]), len(sizes)
    return wl.Index(N=N, D=D, nlist=nlist, M=M, centroids=(centre * rng.normal(size=(nlist, D))).astype(np.float32),
                    codebooks=(spread * rng.normal(size=(M, 256, D // M))).astype(np.float32), list_offsets=offs,
                    codes=rng.integers(0, 256, size=(N, M), dtype=np.uint8), ids=rng.permutation(N).astype(np.int64))


def _same(got, want, what):
    got = [x.cpu().numpy() for x in got]
    assert np.array_equal(got[0], want[0]) and np.array_equal(got[1].view(np.uint32), want[1].view(np.uint32)), what


@pytest.mark.gpu
@pytest.mark.parametrize("D,M", [(96, 48), (128, 64), (200, 100), (146, 73), (80, 80), (246, 82), (256, 128), (255, 85), (95, 95)])
@pytest.mark.parametrize("k,radius", [(1, 0.6), (128, 0.6), (10, 0.05), (100, np.inf)])
def test_segments_and_groups(D, M, k, radius):
    """Lists of a block, of whole segments and one point more or less, of what the head pass holds (4600 to 4750 points) and
    more; groups of one and two queries; points alike; radii per query, some of them not a number; few candidate slots."""
    import torch
    from paper_2312_01712_amd import binding as b
    rng = np.random.default_rng(M + k)
    sizes = np.array([2048, 2047, 2049, 4097, 4600, 4672, 4750, 6200, 64, 65, 63, 1, 0, 128, 129, 300, 513, 511, 1100, 700] + [90] * 12)
    nprobe, distinct, reps = 9, 61, 17   # 1037 queries
    idx = _index(rng, D, M, sizes)
    idx.codes[100:1500] = idx.codes[100]   # more equal distances than the head pass can rank
    q = (idx.centroids[rng.integers(0, len(sizes), distinct)] + 0.3 * rng.normal(size=(distinct, D))).astype(np.float32)
    radii = np.full(M, radius * np.sqrt(D / M), dtype=np.float32)
    gi = b.IvfPqIndex.from_index(idx)
    try:
        dq = torch.from_numpy(q).cuda().repeat(reps, 1)
        want = oracle.search(q, idx, nprobe, k, radii, threads=8)
        tiled = (np.tile(want[0], (reps, 1)), np.tile(want[1], (reps, 1)))
        own = np.tile(radii, (distinct, 1)) * rng.uniform(0.7, 1.3, (distinct, M)).astype(np.float32)
        own[::2, 3] = np.nan
        rq = torch.from_numpy(own).cuda().repeat(reps, 1)
        ref = [x.cpu().numpy() for x in gi.search(dq, nprobe, k, None, query_radii=rq, strategy=b.SCAN_QUERY_MAJOR)]
        for cap in (0, 64):
            b.set_option("lm_cap", cap)
            _same(gi.search(dq, nprobe, k, radii, strategy=b.SCAN_LIST_MAJOR), tiled, (cap, "whole batch"))
            _same(gi.search(dq[:distinct].contiguous(), nprobe, k, radii, strategy=b.SCAN_LIST_MAJOR), want, (cap, "small batch"))
            _same(gi.search(dq, nprobe, k, None, query_radii=rq, strategy=b.SCAN_LIST_MAJOR), ref, (cap, "radii per query"))
    finally:
        b.set_option("lm_cap", 0)
        gi.close()


@pytest.mark.gpu
def test_100_subspaces_with_little_workspace():
    """AUTO, and a request for the list-major scan, with a workspace that only has room for the query-major one; hit counts."""
    import torch
    from paper_2312_01712_amd import binding as b
    rng = np.random.default_rng(5)
    D, M, nprobe, k, Q = 200, 100, 16, 10, 1100
    idx = _index(rng, D, M, rng.integers(40, 400, size=64))
    q = (idx.centroids[rng.integers(0, 64, Q)] + 0.3 * rng.normal(size=(Q, D))).astype(np.float32)
    radii = np.full(M, 0.6 * np.sqrt(2), dtype=np.float32)
    gi = b.IvfPqIndex.from_index(idx)
    dq = torch.from_numpy(q).cuda()
    small = gi.workspace(Q, nprobe, k, strategy=b.SCAN_QUERY_MAJOR)
    want = oracle.search(q, idx, nprobe, k, radii, threads=8)
    assert gi.resolve_strategy(Q, nprobe, k) == b.SCAN_LIST_MAJOR
    assert gi.resolve_strategy(Q, nprobe, k, mode=1) == b.SCAN_QUERY_MAJOR
    for strategy in (b.SCAN_AUTO, b.SCAN_LIST_MAJOR):
        _same(gi.search(dq, nprobe, k, radii, strategy=strategy), want, (strategy, "own workspace"))
        _same(gi.search(dq, nprobe, k, radii, strategy=strategy, workspace=small), want, (strategy, "small workspace"))
    ref = oracle.search(q, idx, nprobe, k, radii, threads=8, mode=1)
    _same(gi.search(dq, nprobe, k, radii, mode=1, strategy=b.SCAN_LIST_MAJOR), ref, "hit counts")
    gi.close()


@pytest.mark.gpu
@pytest.mark.parametrize("D,M", [(96, 48), (128, 64), (200, 100), (146, 73), (80, 80), (246, 82), (256, 128), (255, 85), (95, 95)])
@pytest.mark.parametrize("centre", [0.1, 0.3, 3.0])
def test_bounds_that_end_early(D, M, centre):
    """Lists that are ruled out by few of their subspaces, by many and not at all; probes that name no list, or an empty one;
    with and without the grid of nearest entries; a number of pairs that fills no workgroup."""
    import torch
    from paper_2312_01712_amd import binding as b
    rng = np.random.default_rng(M)
    nlist, nprobe, k, Q = 90, 50, 10, 333
    idx = _index(rng, D, M, rng.integers(0, 200, size=nlist), centre=centre)
    q = (idx.centroids[rng.integers(0, nlist, Q)] + 0.3 * rng.normal(size=(Q, D))).astype(np.float32)
    radii = np.full(M, 0.7 * np.sqrt(2), dtype=np.float32)
    pid, _ = oracle.coarse(q, idx.centroids, nprobe)
    pid[::7, 3] = -1
    pid[1::7, 5] = nlist
    gi = b.IvfPqIndex.from_index(idx)
    dq, dp = torch.from_numpy(q).cuda(), torch.from_numpy(pid.astype(np.int32)).cuda()
    try:
        want = [x.cpu().numpy() for x in gi.scan_topk(dq, dp, k, radii, strategy=b.SCAN_QUERY_MAJOR)]
        for grid in (1, 2):
            b.set_option("bound_grid", grid)
            _same(gi.scan_topk(dq, dp, k, radii, strategy=b.SCAN_LIST_MAJOR), want, ("grid", grid))
            _same(gi.search(dq, nprobe, k, radii, strategy=b.SCAN_LIST_MAJOR), oracle.search(q, idx, nprobe, k, radii, threads=8), ("search", grid))
    finally:
        b.set_option("bound_grid", 0)
        gi.close()


@pytest.mark.gpu
def test_batches_around_what_one_workgroup_sorts():
    """1024 and 2048 queries and one more or less; all of them with the same nearest list, or none with any."""
    import torch
    from paper_2312_01712_amd import binding as b
    rng = np.random.default_rng(9)
    D, M, nlist, nprobe, k = 128, 64, 1100, 16, 10
    idx = _index(rng, D, M, rng.integers(0, 60, size=nlist), centre=0.5)
    q = (idx.centroids[rng.integers(0, nlist, 2049)] + 0.3 * rng.normal(size=(2049, D))).astype(np.float32)
    radii = np.full(M, 0.7 * np.sqrt(2), dtype=np.float32)
    pid, _ = oracle.coarse(q, idx.centroids, nprobe)
    gi = b.IvfPqIndex.from_index(idx)
    dq = torch.from_numpy(q).cuda()
    for first in (None, int(np.argmax(np.diff(idx.list_offsets))), -1):
        p = pid.astype(np.int32).copy()
        if first is not None:
            p[:, 0] = first
        dp = torch.from_numpy(p).cuda()
        for Q in (1023, 1024, 1025, 2047, 2048, 2049):
            want = [x.cpu().numpy() for x in gi.scan_topk(dq[:Q].contiguous(), dp[:Q].contiguous(), k, radii, strategy=b.SCAN_QUERY_MAJOR)]
            _same(gi.scan_topk(dq[:Q].contiguous(), dp[:Q].contiguous(), k, radii, strategy=b.SCAN_LIST_MAJOR), want, (first, Q))
    gi.close()


@pytest.mark.gpu
@pytest.mark.parametrize("D,M,line", [(128, 64, 6144), (64, 16, 4096), (200, 100, 9600)])
def test_small_batches_that_go_list_major(D, M, line):
    """Either side of the line of AUTO, with a workspace of their own and one that only has room for the query-major scan;
    lists too long for the head pass, few probes and k near its limit stay query-major."""
    import torch
    from paper_2312_01712_amd import binding as b
    rng = np.random.default_rng(M)
    nprobe, k = 16, 10
    sizes = rng.integers(20, 300, size=80)
    for longest in (300, 9000):
        sizes[7] = longest
        idx = _index(rng, D, M, sizes, centre=0.3)
        Q = line // nprobe
        q = (idx.centroids[rng.integers(0, len(sizes), Q)] + 0.3 * rng.normal(size=(Q, D))).astype(np.float32)
        radii = np.full(M, 0.7 * np.sqrt(D / M), dtype=np.float32)
        gi = b.IvfPqIndex.from_index(idx)
        assert gi.resolve_strategy(Q, nprobe, k) == (b.SCAN_LIST_MAJOR if longest == 300 else b.SCAN_QUERY_MAJOR)
        for other in ((Q - 1, nprobe, k), (line // 4, 4, k), (Q, nprobe, 113)):
            assert gi.resolve_strategy(*other) == b.SCAN_QUERY_MAJOR, other
        want = oracle.search(q, idx, nprobe, k, radii, threads=8)
        dq = torch.from_numpy(q).cuda()
        _same(gi.search(dq, nprobe, k, radii), want, (longest, "own workspace"))
        _same(gi.search(dq, nprobe, k, radii, workspace=gi.workspace(Q, nprobe, k, strategy=b.SCAN_QUERY_MAJOR)), want, (longest, "small workspace"))
        for kk in (100, 112):
            _same(gi.search(dq, nprobe, kk, radii), oracle.search(q, idx, nprobe, kk, radii, threads=8), (longest, kk))
        gi.close()


@pytest.mark.gpu
@pytest.mark.parametrize("D,M,mean,longest,Q,nprobe,k,mode,list_major", [
    (64, 16, 400, 500, 256, 32, 25, 0, True), (64, 16, 400, 500, 256, 32, 26, 0, False),       # mean lists of 16 k points
    (64, 16, 400, 500, 512, 32, 26, 0, True),                                                  # (16 384 pairs: always)
    (64, 16, 400, 500, 256, 24, 64, 1, True), (64, 16, 400, 500, 255, 32, 64, 1, False),       # hit counts: queries ...
    (64, 16, 400, 500, 256, 23, 64, 2, False), (64, 16, 400, 500, 256, 32, 65, 1, False),      # ... pairs and neighbours
    (96, 48, 800, 900, 256, 32, 100, 0, True), (96, 48, 900, 999, 256, 32, 101, 0, False),
    (128, 64, 400, 500, 256, 32, 50, 0, True), (128, 64, 400, 500, 256, 32, 51, 0, False),     # mean lists of 8 k points
    (128, 64, 400, 500, 256, 32, 51, 1, True), (128, 64, 400, 500, 512, 32, 51, 0, True),      # (not hit counts, nor larger batches)
    (160, 80, 1100, 4000, 512, 32, 10, 0, True),
    (200, 100, 400, 500, 512, 32, 112, 0, True), (200, 100, 400, 500, 512, 32, 113, 0, False),
    (160, 80, 1000, 5000, 1024, 32, 10, 0, True), (160, 80, 1000, 5000, 1023, 32, 10, 0, False),   # a list that the head pass does not hold
    (160, 80, 1100, 5000, 4096, 32, 10, 0, True), (160, 80, 1100, 5000, 4095, 32, 10, 0, False)])
def test_lines_of_auto(D, M, mean, longest, Q, nprobe, k, mode, list_major):
    """Either side of what AUTO asks of the lists, the batch and the neighbours."""
    from paper_2312_01712_amd import binding as b
    rng = np.random.default_rng(M)
    sizes = np.full(70, mean)
    sizes[7] += longest - mean
    sizes[8:68] -= (longest - mean) // 60 + 1
    sizes[9] += 70 * mean - sizes.sum()   # (the mean is what it says)
    gi = b.IvfPqIndex.from_index(_index(rng, D, M, sizes))
    try:
        assert gi.resolve_strategy(Q, nprobe, k, mode=mode) == (b.SCAN_LIST_MAJOR if list_major else b.SCAN_QUERY_MAJOR)
    finally:
        gi.close()


@pytest.mark.gpu
@pytest.mark.parametrize("D,M", [(200, 100), (160, 80)])
def test_large_batches_go_in_pieces(D, M):
    """Shapes without byte tables for everything: what a workspace holds for candidates stops growing at 2 GiB (or what 4096
    queries want), however the scan is asked for; batches of two pieces, the last one short, return what the oracle does."""
    import torch
    from paper_2312_01712_amd import binding as b
    rng = np.random.default_rng(M)
    nprobe, k, distinct, reps = 8, 10, 60, 75
    idx = _index(rng, D, M, rng.integers(40, 400, size=70))
    q = (idx.centroids[rng.integers(0, 70, distinct)] + 0.3 * rng.normal(size=(distinct, D))).astype(np.float32)
    radii = np.full(M, 0.6 * np.sqrt(2), dtype=np.float32)
    gi = b.IvfPqIndex.from_index(idx)

    def slots(Q, nprobe, strategy):
        return gi.workspace_bytes(Q, nprobe, k, strategy=strategy) - gi.workspace_bytes(Q, nprobe, k, strategy=b.SCAN_QUERY_MAJOR)

    try:
        for strategy in (b.SCAN_AUTO, b.SCAN_LIST_MAJOR):
            assert gi.resolve_strategy(1_000_000, 64, k, strategy=strategy) == b.SCAN_LIST_MAJOR
            assert slots(1_000_000, 64, strategy) == slots(16_384, 64, strategy) < (2 << 30) + (64 << 20), strategy
        b.set_option("lm_cap", 65536)   # 4096 queries a piece
        assert slots(distinct * reps, nprobe, b.SCAN_AUTO) == slots(4096, nprobe, b.SCAN_AUTO) > slots(4000, nprobe, b.SCAN_AUTO)
        dq = torch.from_numpy(q).cuda().repeat(reps, 1)
        own = np.tile(radii, (distinct, 1)) * rng.uniform(0.7, 1.3, (distinct, M)).astype(np.float32)
        for per_query in (None, own):
            want = oracle.search(q, idx, nprobe, k, radii if per_query is None else per_query, threads=8)
            want = (np.tile(want[0], (reps, 1)), np.tile(want[1], (reps, 1)))
            rq = None if per_query is None else torch.from_numpy(per_query).cuda().repeat(reps, 1)
            shared = radii if per_query is None else None
            for strategy in (b.SCAN_AUTO, b.SCAN_LIST_MAJOR):
                _same(gi.search(dq, nprobe, k, shared, query_radii=rq, strategy=strategy), want, ("search", strategy))
            _same(gi.scan_topk(dq, gi.coarse(dq, nprobe)[0], k, shared, query_radii=rq), want, "scan_topk")
    finally:
        b.set_option("lm_cap", 0)
        gi.close()
