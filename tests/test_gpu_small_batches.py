"""Small batches, where the probes of a query are split over several workgroups: the merge of their
lists, the bounds they share, and the filtering stage without a matrix product.  Everything is
compared with the oracle bit for bit (same operation order: no tolerance)."""
import numpy as np
import pytest
import torch

import oracle
from paper_2312_01712_amd import workloads as wl

pytestmark = pytest.mark.gpu


def _index(rng, D, M, nlist, mean, spread=0.3, distinct=256):
    """Random codes over clustered centroids; `distinct` < 256 makes equal distances common."""
    sizes = rng.integers(0, 2 * mean + 1, nlist)
    sizes[:2] = (0, 1)
    offs = np.zeros(nlist + 1, dtype=np.int64)
    offs[1:] = np.cumsum(sizes)
    N = int(offs[-1])
    cb = (rng.normal(size=(M, 256, D // M)) * spread).astype(np.float32)
    return wl.Index(N=N, D=D, nlist=nlist, M=M, centroids=rng.normal(size=(nlist, D)).astype(np.float32), codebooks=cb,
                    list_offsets=offs, codes=rng.integers(0, distinct, size=(N, M), dtype=np.uint8),
                    ids=rng.permutation(N).astype(np.int64))


def _check(idx, q, nprobe, k, radii, metric=0, mode=0, query_radii=None):
    from paper_2312_01712_amd import binding as b
    gi = b.IvfPqIndex.from_index(idx, metric=metric)
    dq = torch.from_numpy(q).cuda()
    rq = None if query_radii is None else torch.from_numpy(query_radii).cuda()
    o_ids, o_dist = oracle.search(q, idx, nprobe, k, radii if query_radii is None else query_radii, threads=8, mode=mode,
                                  metric=metric)
    for _ in range(2):   # twice: the second call finds the workspace as the first one left it
        ids, dist = gi.search(dq, nprobe, k, radii, mode=mode, query_radii=rq)
        torch.cuda.synchronize()
        assert np.array_equal(ids.cpu().numpy(), o_ids), "ids differ"
        assert np.array_equal(dist.cpu().numpy().view(np.uint32), o_dist.view(np.uint32)), "distances differ"
    gi.close()


# probe groups per query: min(ceil(2048 / Q), nprobe, 64), so these cover 2, 4, 5, 16, 17, 33 and 64 of them
@pytest.mark.parametrize("Q,nprobe", [(1, 2), (3, 5), (1024, 9), (511, 9), (129, 20), (123, 33), (1, 33), (5, 80)])
@pytest.mark.parametrize("D,M", [(128, 64), (64, 16), (30, 10)])
def test_split_probes(Q, nprobe, D, M):
    rng = np.random.default_rng(Q * 100 + nprobe)
    idx = _index(rng, D, M, 90, 40 if Q > 100 else 150)
    q = (idx.centroids[rng.integers(0, idx.nlist, Q)] + 0.4 * rng.normal(size=(Q, D))).astype(np.float32)
    radii = np.full(M, 0.5, dtype=np.float32)
    for k in (1, 64, 65, 128):
        _check(idx, q, nprobe, k, radii)


@pytest.mark.parametrize("mode,metric", [(0, 0), (1, 0), (2, 0), (0, 1)])
def test_split_probes_ties_and_more_passes(mode, metric):
    """Two codes only (masses of equal scores across workgroups) and k above one pass."""
    rng = np.random.default_rng(5)
    idx = _index(rng, 128, 64, 60, 120, distinct=2)
    q = (idx.centroids[rng.integers(0, 60, 37)] + 0.2 * rng.normal(size=(37, 128))).astype(np.float32)
    for k in (10, 128, 200):
        _check(idx, q, 24, k, np.full(64, 0.6, dtype=np.float32), metric=metric, mode=mode)


def test_split_probes_per_query_radii():
    rng = np.random.default_rng(6)
    idx = _index(rng, 96, 48, 70, 200)
    q = (idx.centroids[rng.integers(0, 70, 300)] + 0.3 * rng.normal(size=(300, 96))).astype(np.float32)
    _check(idx, q, 32, 100, None, query_radii=rng.uniform(0.1, 0.9, size=(300, 48)).astype(np.float32))


# tiles of 64 lists x 16 queries, slices of 128 dimensions, 16-byte and scalar loads
@pytest.mark.parametrize("nlist,D,Q", [(1, 1, 1), (63, 3, 4), (64, 4, 5), (65, 127, 16), (700, 128, 17), (130, 129, 3),
                                       (257, 260, 33), (90, 520, 2), (4096, 64, 9)])
@pytest.mark.parametrize("metric", [0, 1])
def test_filtering_without_matrix_product(nlist, D, Q, metric):
    from paper_2312_01712_amd import binding as b
    rng = np.random.default_rng(nlist + D)
    c = rng.normal(size=(nlist, D)).astype(np.float32)
    q = np.ascontiguousarray(np.concatenate([c[rng.integers(0, nlist, Q - 1)], np.zeros((1, D), np.float32)]))
    cases = [c]
    if nlist > 300:   # masses of equal distances: more lists up to the cut than the selection collects
        few = c.copy()
        few[nlist // 8:] = few[0]
        cases.append(few)
    for cent in cases:
        gi = b.IvfPqIndex(cent, rng.normal(size=(1, 256, D)).astype(np.float32), np.arange(nlist + 1, dtype=np.int64),
                          np.zeros((nlist, 1), dtype=np.uint8), metric=metric)
        for nprobe in sorted({1, min(nlist, 7), min(nlist, 100)}):
            pid, pd = gi.coarse(torch.from_numpy(q).cuda(), nprobe)
            torch.cuda.synchronize()
            o_pid, o_pd = oracle.coarse(q, cent, nprobe, metric=metric)
            assert np.array_equal(pid.cpu().numpy(), o_pid)
            assert np.array_equal(pd.cpu().numpy().view(np.uint32), o_pd.view(np.uint32))
        gi.close()


# List-major main pass with byte tables: groups of eight queries (lists probed by 1, 7, 8, 9 and many
# queries), lists around a block and around sixteen blocks, ties at the k-th distance, radii that
# are infinite, zero in one subspace and small against the residuals, queries whose nearest list
# is shorter than k, more candidates than a task can hold.
@pytest.mark.parametrize("D,M", [(96, 48), (128, 64), (64, 16)])
@pytest.mark.parametrize("radius", ["mixed", "inf", "small"])
def test_byte_tables(D, M, radius):
    from paper_2312_01712_amd import binding as b
    rng = np.random.default_rng(M)
    sizes = np.array([1, 63, 64, 65, 1023, 1024, 1025, 2100, 0, 700, 40, 130, 900, 5000, 300, 1100])
    nlist, N = len(sizes), int(sizes.sum())
    offs = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
    idx = wl.Index(N=N, D=D, nlist=nlist, M=M, centroids=(0.2 * rng.normal(size=(nlist, D))).astype(np.float32),
                   codebooks=(0.3 * rng.normal(size=(M, 256, D // M))).astype(np.float32), list_offsets=offs,
                   codes=rng.integers(0, 256, size=(N, M), dtype=np.uint8), ids=rng.permutation(N).astype(np.int64))
    idx.codes[offs[13]:offs[13] + 4000] = idx.codes[offs[13]]      # 4000 equal points
    r = np.full(M, {"mixed": 0.45, "inf": np.inf, "small": 0.02}[radius], dtype=np.float32)
    if radius == "mixed":
        r *= rng.uniform(0.5, 1.5, M).astype(np.float32)
        r[3] = 0.0
    for Q, k in ((61, 10), (1, 128), (9, 100)):
        q = (idx.centroids[rng.integers(0, nlist, Q)] + 0.3 * rng.normal(size=(Q, D))).astype(np.float32)
        q[0] = idx.centroids[13]
        rq = (r[None, :] * rng.uniform(0.5, 1.5, (Q, M))).astype(np.float32) if radius == "mixed" else None
        for mode, radii in ((0, r), (1, r), (2, r)) + (((0, rq),) if rq is not None else ()):
            gi = b.IvfPqIndex.from_index(idx)
            kw = dict(mode=mode, strategy=b.SCAN_LIST_MAJOR)
            if radii is rq:
                ids, dist = gi.search(torch.from_numpy(q).cuda(), 12, k, None, query_radii=torch.from_numpy(rq).cuda(), **kw)
            else:
                ids, dist = gi.search(torch.from_numpy(q).cuda(), 12, k, radii, **kw)
            torch.cuda.synchronize()
            o_ids, o_dist = oracle.search(q, idx, 12, k, radii, threads=8, mode=mode)
            assert np.array_equal(ids.cpu().numpy(), o_ids), (Q, k, mode)
            assert np.array_equal(dist.cpu().numpy().view(np.uint32), o_dist.view(np.uint32)), (Q, k, mode)
            gi.close()


# Shapes without a specialised kernel: every number of code chunks, tails of 1 to 3 four-byte chunks,
# padding rows, each way of reading a codebook row (dsub 1, 2, 4, 8 and any other).
@pytest.mark.parametrize("M,dsub", [(1, 3), (3, 2), (4, 8), (5, 1), (15, 4), (16, 2), (17, 4), (20, 6), (31, 1), (33, 8),
                                    (47, 2), (64, 1), (65, 3), (80, 4), (81, 2), (97, 1), (112, 2), (113, 5), (128, 4)])
def test_shapes_without_a_specialised_kernel(M, dsub):
    from paper_2312_01712_amd import binding as b
    rng = np.random.default_rng(M * 10 + dsub)
    D = M * dsub
    idx = _index(rng, D, M, 30, 300, spread=0.3)
    q = (idx.centroids[rng.integers(0, 30, 21)] + 0.3 * rng.normal(size=(21, D))).astype(np.float32)
    radii = np.full(M, 0.5 * np.sqrt(dsub), dtype=np.float32)
    for Q, nprobe, k, mode in ((21, 12, 10, 0), (21, 3, 100, 0), (1, 1, 128, 0), (21, 12, 300, 0), (21, 12, 20, 1), (5, 12, 20, 2)):
        _check(idx, q[:Q], nprobe, k, radii, mode=mode)
    # more queries than probe groups are made for: one workgroup walks all of a query's lists
    big = np.ascontiguousarray(np.repeat(q, 100, axis=0)[:2050])
    gi = b.IvfPqIndex.from_index(idx)
    ids, dist = gi.search(torch.from_numpy(big).cuda(), 6, 10, radii)
    o_ids, o_dist = oracle.search(q, idx, 6, 10, radii)
    assert np.array_equal(ids.cpu().numpy(), np.repeat(o_ids, 100, axis=0)[:2050])
    assert np.array_equal(dist.cpu().numpy().view(np.uint32), np.repeat(o_dist, 100, axis=0)[:2050].view(np.uint32))
    pid, _ = gi.coarse(torch.from_numpy(q).cuda(), 4)
    o_offs, o_cd, o_ci = oracle.scan_all(q, idx, pid.cpu().numpy(), radii)
    cd, ci, err = gi.scan_all(torch.from_numpy(q).cuda(), pid, radii, torch.from_numpy(o_offs).cuda())
    assert int(err.item()) == 0 and np.array_equal(ci.cpu().numpy(), o_ci)
    assert np.array_equal(cd.cpu().numpy().view(np.uint32), o_cd.view(np.uint32))
    gi.close()


# The split (bf16 pair) product behind the keys: depths around its slices of 32 with 16-byte and scalar
# loads, a ragged last tile of lists and of queries, values that cancel (a large common offset), tiny
# and huge magnitudes (the reference-order path must take over, not a wrong list).
@pytest.mark.parametrize("nlist,D,Q", [(5000, 31, 130), (4000, 32, 257), (8193, 33, 1000), (6000, 100, 700), (3400, 260, 900)])
@pytest.mark.parametrize("what", ["plain", "offset", "tiny", "huge"])
@pytest.mark.parametrize("metric", [0, 1])
def test_split_product_proposals(nlist, D, Q, what, metric):
    from paper_2312_01712_amd import binding as b
    rng = np.random.default_rng(nlist + D)
    scale, offset = {"plain": (1.0, 0.0), "offset": (1.0, 300.0), "tiny": (1e-19, 0.0), "huge": (3e17, 0.0)}[what]
    c = (scale * rng.normal(size=(nlist, D)) + offset).astype(np.float32)
    q = (c[rng.integers(0, nlist, Q)] + 0.5 * scale * rng.normal(size=(Q, D))).astype(np.float32)
    gi = b.IvfPqIndex(c, rng.normal(size=(1, 256, D)).astype(np.float32), np.arange(nlist + 1, dtype=np.int64),
                      np.zeros((nlist, 1), dtype=np.uint8), metric=metric)
    b.coarse_fallbacks(reset=True)
    pid, pd = gi.coarse(torch.from_numpy(q).cuda(), 8)
    torch.cuda.synchronize()
    fb = b.coarse_fallbacks()
    o_pid, o_pd = oracle.coarse(q, c, 8, metric=metric)
    assert np.array_equal(pid.cpu().numpy(), o_pid)
    assert np.array_equal(pd.cpu().numpy().view(np.uint32), o_pd.view(np.uint32))
    if what == "plain" and metric == 0:
        assert fb <= Q // 20, f"{fb} of {Q} queries were not accepted from the proposal"
    gi.close()
