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
assert "s = ((float)LMB_TOP - 0.6f) / fmaf(farthest, LMP_REL, cap);" in SOURCE
f32 = np.float32


def _bf16(x):
    u = np.ascontiguousarray(x, f32).view(np.uint32)
    return ((u + 0x7FFF + ((u >> 16) & 1)) & 0xFFFF0000).astype(np.uint32).view(f32)


def _split(x):
    hi = _bf16(x)
    return hi, _bf16(x - hi)


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
                nrm = (cb[..., 1].astype(np.float64) ** 2 + (cb[..., 0] * cb[..., 0])).astype(f32)
                rr = (res.astype(np.float64) ** 2).sum(1).astype(f32)
                far = (np.sqrt(rr) + np.sqrt(nrm.max(1))) ** 2
                cap = max(f32(r2.max()), f32(1e-30))
                s = f32((63 - 0.6) / (far.max() / 32768.0 + cap))
                most, err = np.minimum(r2, cap) * s, s * far / f32(32768) + f32(1 / 1024)
                con = (most - s * rr) + (f32(0.5) + err)
                a = [_split(f32(2) * s * res[:, j]) for j in range(2)] + [_split(np.full(M, -s, f32))]
                b = [_split(cb[..., j]) for j in range(2)] + [_split(nrm)]
                acc = con.astype(np.float64)[:, None] + sum((ah[:, None].astype(np.float64) + al[:, None]) * (bh.astype(np.float64) + bl)
                                                            for (ah, al), (bh, bl) in zip(a, b))
                byte = np.clip(np.rint(acc.astype(f32)), 0, 255)
                gain = float(s) * (np.minimum(r2, cap)[:, None].astype(np.float64) -
                                   ((res[:, None, :].astype(np.float64) - cb) ** 2).sum(2))
                e = err[:, None].astype(np.float64)
                assert np.all(np.abs(acc - 0.5 - e - gain) <= 0.5 * e), (spread, sigma, radius)   # half of the raise is left to the products' sums
                assert np.all(byte >= gain) and np.all(byte <= np.maximum(gain, 0.0) + 1.0 + 2.0 * e)
                assert byte.max() <= 63


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
