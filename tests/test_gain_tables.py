"""Byte tables that hold gains (lm_part_kernel), made from split factors: the bytes against exact values in 64 bits on the
CPU, and searches that take them, at the edges of segments, groups and parts, against the oracle bit for bit."""
import os
import re

import numpy as np
import pytest

import oracle
from paper_2312_01712_amd import workloads as wl

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SOURCE = open(os.path.join(ROOT, "paper_2312_01712_amd", "csrc", "scan_lm_parts.h")).read()
assert "LMP_RAISE = 1.0f / 1024.0f, LMP_REL = 1.0f / 32768.0f;" in SOURCE
assert "s = ((float)LMB_TOP - 0.6f) / fmaf(farthest, 2.0f * LMP_REL, cap);" in SOURCE
f32 = np.float32


def _bf16(x):
    u = np.ascontiguousarray(x, f32).view(np.uint32)
    return ((u + 0x7FFF + ((u >> 16) & 1)) & 0xFFFF0000).astype(np.uint32).view(f32)


def _split(x):
    hi = _bf16(x)
    return hi, _bf16(x - hi)


def _table(cb, res, r2, tau=np.inf, room=2.0):
    """A query's table as the kernel makes it from its residuals [M, 2], squared radii and k-th distance: the values before they
    become bytes (in 64 bits), what the fp32 sums of the products may lose of them, the raise, the exact gains, and what a
    point's bytes must add up to (-1: every point is a candidate)."""
    M = len(cb)
    nrm = (cb[..., 1].astype(np.float64) ** 2 + (cb[..., 0] * cb[..., 0])).astype(f32)
    rr = (res[:, 1].astype(np.float64) ** 2 + (res[:, 0] * res[:, 0])).astype(f32)
    far = (np.sqrt(rr) + np.sqrt(nrm.max(1))) ** 2
    cap = max(min(f32(r2.max()), f32(tau) * f32(4 / M)), f32(1e-30))
    s = f32((63 - 0.6) / (room * far.max() / 32768.0 + cap))
    most, err = np.minimum(r2, cap) * s, s * far / f32(32768) + f32(1 / 1024)
    con = (most - s * rr) + (f32(0.5) + err)
    a = [_split(f32(2) * s * res[:, j]) for j in range(2)] + [_split(np.full(M, -s, f32))]
    b = [_split(cb[..., j]) for j in range(2)] + [_split(nrm)]
    acc = con.astype(np.float64)[:, None] + sum((ah[:, None].astype(np.float64) + al[:, None]) * (bh.astype(np.float64) + bl)
                                                for (ah, al), (bh, bl) in zip(a, b))
    gain = float(s) * (np.minimum(r2, cap)[:, None].astype(np.float64) -
                       ((res[:, None, :].astype(np.float64) - cb) ** 2).sum(2))
    lost = f32(1.0e-5 if M <= 64 else 1.6e-5)
    with np.errstate(invalid="ignore"):
        least = (most - lost * (most + 1)).sum(dtype=f32) - f32(tau) * s * (1 + lost)
    start = int(least) - 1 if least > 1 else -1
    return acc, (far * s).astype(np.float64)[:, None] / 2 ** 19, err[:, None].astype(np.float64), gain, start


def _bytes(acc):
    return np.clip(np.rint(acc.astype(f32)), 0, 255)   # (the conversion saturates at 255, not at 63)


def _in_bounds(acc, sums, e, gain, what):
    byte = _bytes(acc)
    assert np.all(np.abs(acc - 0.5 - e - gain) <= 0.5 * e), what   # half of the raise is left to the products' sums
    assert np.all(byte >= gain) and np.all(byte <= np.maximum(gain, 0.0) + 1.0 + 2.0 * e), what
    assert _bytes(acc + sums).max() <= 63, what


@pytest.mark.parametrize("M", [48, 64, 100])
def test_bytes_are_no_less_than_what_an_entry_gains(M):
    """Rounded up by less than a unit and twice the error, never more than 63 (two of them add up within a signed byte),
    and 0 for what lies clearly outside; radii from nothing to far beyond the data, residuals near and far."""
    rng = np.random.default_rng(M)
    for spread in (0.01, 0.3, 3.0):
        for sigma in (0.1, 1.0, 30.0):
            for radius in (0.0, 1e-4, 0.02, 0.164, 0.6, 2.0, 50.0):
                cb = (spread * rng.normal(size=(M, 256, 2))).astype(f32)
                res = (sigma * spread * rng.normal(size=(M, 2))).astype(f32)
                r2 = (rng.uniform(0.5, 1.0, M).astype(f32) * f32(radius * spread)) ** 2
                _in_bounds(*_table(cb, res, r2)[:4], (spread, sigma, radius))


def _even_codebooks(rng, M, kind, spread):
    """Entries of one norm (on a circle, or with components of one size), or as they come."""
    if kind == "circle":
        at = 2 * np.pi * rng.random((M, 256))
        return (spread * np.stack([np.cos(at), np.sin(at)], 2)).astype(f32)
    if kind == "signs":
        return (spread * rng.choice([-1.0, 1.0], size=(M, 256, 2))).astype(f32)
    return (spread * rng.normal(size=(M, 256, 2))).astype(f32)


def _near_points(M, room):
    """Points that coincide with their query, or nearly, of tables that hold little but that: bytes at the top in all
    subspaces.  Yields (kind of point, the table, the point's codes, whether it is within tau and the radii)."""
    rng = np.random.default_rng(M)
    for kind in ("circle", "signs", "gauss"):
        for draw in range(4):
            spread = float(rng.choice([0.01, 0.3, 3.0]))
            cb = _even_codebooks(rng, M, kind, spread)
            code = rng.integers(0, 256, M) if draw % 2 else (cb.astype(np.float64) ** 2).sum(2).argmax(1)   # the farthest entries, too
            at = cb[np.arange(M), code]
            for off in (0.0, 2e-4, 1e-3, 1e-2):
                res = (at + spread * off * rng.normal(size=(M, 2))).astype(f32)
                apart = ((res.astype(np.float64) - at) ** 2).sum(1)
                dist = float(apart.sum())
                for tau in (0.0, dist * 1.001, 1.5 * dist, 100.0 * dist, 1e-4 * spread ** 2, 0.1 * spread ** 2 * M, np.inf):
                    for radius in (1e-3, 0.05, 0.6, np.inf):
                        r2 = np.full(M, (spread * radius) ** 2, f32)
                        if tau == radius == np.inf:
                            continue   # (no scale: every point is a candidate)
                        value = np.minimum(apart, r2.astype(np.float64)).sum()   # the point's distance: no entry counts more than r^2
                        yield (kind, draw, off, tau, radius), _table(cb, res, r2, tau, room), code, value * (1 + 1e-6) <= tau


@pytest.mark.parametrize("M", [48, 64, 100])
def test_points_on_their_query_are_found(M):
    """What two bytes add up to is taken for signed: with a byte above 63 a point that gains the most looks like one that
    gains nothing.  Room for the raise alone (1.0) did that."""
    missed, highest = {1.0: 0, 2.0: 0}, {1.0: 0, 2.0: 0}
    for room in missed:
        for what, (acc, sums, e, gain, start), code, within in _near_points(M, room):
            if room == 2.0:
                _in_bounds(acc, sums, e, gain, what)
            byte = _bytes(acc)
            highest[room] = max(highest[room], byte.max())
            pair = byte[np.arange(M), code].reshape(-1, 2).sum(1)
            total = np.where(pair >= 128, pair - 256, pair).sum()
            missed[room] += bool(within and start - total >= 0)
    assert highest[2.0] <= 63 and missed[2.0] == 0
    assert highest[1.0] > 63 and missed[1.0] > 0   # (these draws would have shown it)


def _index(rng, D, M, sizes, spread=0.3, centre=0.05):
    offs = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
    N, nlist = int(offs[-1]), len(sizes)
    return wl.Index(N=N, D=D, nlist=nlist, M=M, centroids=(centre * rng.normal(size=(nlist, D))).astype(np.float32),
                    codebooks=(spread * rng.normal(size=(M, 256, D // M))).astype(np.float32), list_offsets=offs,
                    codes=rng.integers(0, 256, size=(N, M), dtype=np.uint8), ids=rng.permutation(N).astype(np.int64))


@pytest.mark.gpu
@pytest.mark.parametrize("D,M", [(96, 48), (128, 64), (200, 100)])
@pytest.mark.parametrize("k,radius", [(1, 0.6), (10, 0.6), (10, 0.05), (10, np.inf)])
def test_segments_groups_and_parts(D, M, k, radius):
    """Lists of a block, of whole segments and one point more or less, of two segments and a bit; groups of one to eight
    queries; entries that are infinite, not a number or larger than the split holds; radii per query, some of them NaN."""
    import torch
    from paper_2312_01712_amd import binding as b
    rng = np.random.default_rng(M + k)
    sizes = np.array([2048, 2047, 2049, 4097, 64, 65, 1, 0, 300, 513, 511, 1100, 900, 700, 100, 1536, 1000, 800, 900, 1200])
    nprobe, distinct, reps = 16, 61, 17   # 1037 queries: groups of every size
    idx = _index(rng, D, M, sizes)
    q = (idx.centroids[rng.integers(0, len(sizes), distinct)] + 0.3 * rng.normal(size=(distinct, D))).astype(np.float32)
    radii = np.full(M, radius * np.sqrt(D / M), dtype=np.float32)
    for odd in (None, np.inf, np.nan, 3.0e19):
        if odd is not None:
            idx.codebooks[2, 5:40] = odd
            idx.codebooks[M - 1, 100, 0] = odd
        gi = b.IvfPqIndex.from_index(idx)
        dq = torch.from_numpy(q).cuda().repeat(reps, 1)
        if odd is None:
            want = oracle.search(q, idx, nprobe, k, radii, threads=8)
            want = (np.tile(want[0], (reps, 1)), np.tile(want[1], (reps, 1)))
        else:
            want = [x.cpu().numpy() for x in gi.search(dq, nprobe, k, radii, strategy=b.SCAN_QUERY_MAJOR)]
        got = [x.cpu().numpy() for x in gi.search(dq, nprobe, k, radii, strategy=b.SCAN_LIST_MAJOR)]
        assert np.array_equal(got[0], want[0]) and np.array_equal(got[1].view(np.uint32), want[1].view(np.uint32)), (odd, "shared radii")
        own = np.tile(radii, (distinct, 1)) * rng.uniform(0.7, 1.3, (distinct, M)).astype(np.float32)
        own[::2, 3] = np.nan
        rq = torch.from_numpy(own).cuda().repeat(reps, 1)
        want = [x.cpu().numpy() for x in gi.search(dq, nprobe, k, None, query_radii=rq, strategy=b.SCAN_QUERY_MAJOR)]
        got = [x.cpu().numpy() for x in gi.search(dq, nprobe, k, None, query_radii=rq, strategy=b.SCAN_LIST_MAJOR)]
        assert np.array_equal(got[0], want[0]) and np.array_equal(got[1].view(np.uint32), want[1].view(np.uint32)), (odd, "radii per query")
        gi.close()


@pytest.mark.gpu
@pytest.mark.parametrize("D,M", [(96, 48), (128, 64), (200, 100)])
@pytest.mark.parametrize("kind", ["circle", "signs"])
def test_points_on_their_query_behind_the_first_list(D, M, kind):
    """Codebooks of one norm, centroids that two lists share: copies of a query's point stand in both, with the smaller ids in
    the one that is scanned behind the other, at distance 0 or nearly; ordinary radii and very small ones."""
    import torch
    from paper_2312_01712_amd import binding as b
    rng = np.random.default_rng(M)
    pairs, nprobe, copies, per = 30, 8, 12, 10
    sizes = rng.integers(900, 1300, size=2 * pairs)
    idx = _index(rng, D, M, sizes)
    idx.codebooks[:] = np.round(_even_codebooks(rng, M, kind, 0.3) * 4096) / 4096   # (sums with the centroids are exact)
    idx.centroids[:] = np.repeat(np.round(np.linspace(-60, 60, pairs)[:, None] + 0.05 * rng.normal(size=(pairs, D)), 2), 2, axis=0)
    idx.centroids[:] = np.round(idx.centroids * 1024) / 1024
    at = rng.integers(0, pairs, pairs * per)
    ids = np.argsort(np.argsort(idx.ids + idx.N * (np.repeat(np.arange(2 * pairs), sizes) % 2 == 0)))   # smaller in the second of two lists
    idx.ids[:] = ids
    q = np.empty((len(at), D), np.float32)
    room = np.zeros(2 * pairs, np.int64)
    for i, p in enumerate(at):
        code = rng.integers(0, 256, M, dtype=np.uint8)
        for c in (2 * p, 2 * p + 1):
            lo = idx.list_offsets[c] + room[c]
            room[c] += copies
            assert lo + copies <= idx.list_offsets[c + 1]
            idx.codes[lo:lo + copies] = code
        q[i] = idx.centroids[2 * p] + idx.codebooks[np.arange(M), code].reshape(D)
    gi = b.IvfPqIndex.from_index(idx)
    try:
        for off in (0.0, 1e-4, 1e-3):
            qs = (q + off * 0.3 * rng.normal(size=q.shape)).astype(np.float32)
            for k in (1, 10):
                for radius in (0.6, 1e-3):
                    radii = np.full(M, 0.3 * radius, dtype=np.float32)
                    want = oracle.search(qs, idx, nprobe, k, radii, threads=8)
                    for reps in (1, 4):   # (whole tables, but with 100 subspaces; tables in parts)
                        got = [x.cpu().numpy() for x in gi.search(torch.from_numpy(qs).cuda().repeat(reps, 1), nprobe, k, radii, strategy=b.SCAN_LIST_MAJOR)]
                        wrong = int((got[0] != np.tile(want[0], (reps, 1))).any(1).sum())
                        assert wrong == 0, (off, k, radius, reps, f"{wrong} of {len(qs) * reps} queries")
                        assert np.array_equal(got[1].view(np.uint32), np.tile(want[1], (reps, 1)).view(np.uint32)), (off, k, radius, reps)
    finally:
        gi.close()
