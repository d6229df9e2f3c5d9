"""The byte tables of the list-major scan on the CPU: a table's bytes in fp32, operation by operation as the kernel
forms them, against the exact table values in 64 bits."""
import os
import re

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SOURCE = open(os.path.join(ROOT, "paper_2312_01712_amd", "csrc", "scan_lm.hip")).read()
f32 = np.float32


def _constant(pattern):
    return float(re.search(pattern, SOURCE).group(1))


TOP = int(_constant(r"constexpr int LMB_TOP = ([0-9]+);"))
RANGE = _constant(r"constexpr float LMB_RANGE = ([0-9.e]+)f;")
assert "constexpr float RAISE = (DSUB + 3) / 512.0f, REL = (3 * DSUB + 8) / 16777216.0f;" in SOURCE
assert "const float err = fmaf(s * far, far * REL, RAISE);" in SOURCE


def _fma(a, b, c):
    return (np.float64(a) * np.float64(b) + np.float64(c)).astype(f32)


def _table(res, cb, r2, cap, cut=True):
    """Bytes [M][256], unit, offsets and errors of a query's table; res [M][dsub], cb [M][256][dsub], r2 [M]."""
    M, _, dsub = cb.shape
    rr, nrm = np.zeros(M, f32), np.zeros((M, 256), f32)
    for j in range(dsub):
        rr, nrm = _fma(res[:, j], res[:, j], rr), _fma(cb[:, :, j], cb[:, :, j], nrm)
    far = np.sqrt(rr) + np.sqrt(nrm.max(1))
    s = (f32(TOP) - f32(0.01)) / f32(max(cap, f32(1e-30)))
    x = np.minimum(r2, max(cap, f32(1e-30))) * s
    top = np.ceil(x)
    off = top - x
    err = _fma(s * far, far * f32((3 * dsub + 8) / 16777216.0), f32((dsub + 3) / 512.0))
    acc = np.repeat((_fma(rr, s, off + err) + f32(32768.0))[:, None], 256, 1)
    for j in range(dsub):
        acc = _fma((f32(-2.0) * s * res[:, j])[:, None], cb[:, :, j], acc)
    acc = _fma(s, nrm, acc)
    bits = acc.view(np.uint32)
    if cut and not np.all(s * far * far < f32(RANGE)):
        bits = np.minimum(bits, np.uint32(0x47C00000))
    byte = np.minimum((bits >> 8) & 0xFFFF, top.astype(np.uint32)[:, None]).astype(np.float64)
    return byte, float(s), off.astype(np.float64)[:, None], err.astype(np.float64)[:, None]


@pytest.mark.parametrize("M,dsub", [(16, 4), (48, 2), (64, 2)])
def test_bytes_bound_table_values_from_both_sides(M, dsub):
    """A byte is at most s v + offset + twice the raise, and more than s v + offset - 1 for every value that is not cut off:
    radii from nothing to far beyond the data, one for all subspaces or one each, subspaces of unequal spread."""
    rng = np.random.default_rng(M)
    wraps = 0
    for spread in (0.01, 0.3, 3.0):
        for sigma in (0.1, 1.0, 3.0):
            for radius in (0.0, 1e-4, 0.02, 0.05, 0.122, 0.164, 0.3, 0.6, 2.0, 50.0):
                for wide in (1.0, 35.0):
                    cb = (spread * rng.normal(size=(M, 256, dsub))).astype(f32)
                    cb[0] *= f32(wide)
                    res = (sigma * rng.normal(size=(M, dsub))).astype(f32)
                    res[1] = cb[1, 7]                      # on an entry
                    r = np.full(M, radius) if wide == 1.0 else radius * rng.uniform(0.5, 1.0, M)
                    r2 = (r.astype(f32) * r.astype(f32)).astype(f32)
                    d2 = ((res.astype(np.float64)[:, None, :] - cb.astype(np.float64)) ** 2).sum(2)
                    for cap in (r2.max(), f32(0.3) * r2.max()):
                        byte, s, off, err = _table(res, cb, r2, cap)
                        v = np.minimum(d2, r2[:, None].astype(np.float64))
                        assert byte.min() >= 0 and byte.max() <= TOP
                        assert np.all(byte <= s * v * (1 + 1e-6) + off + 2 * err)
                        kept = np.minimum(v, float(max(cap, f32(1e-30))))
                        assert np.all(byte > s * kept * (1 - 1e-6) + off - 1 - 1e-3)
                        bare = _table(res, cb, r2, cap, cut=False)[0]
                        wraps += int(np.any(bare != byte))
    assert wraps > 10   # the ranges reach values whose bits wrap


@pytest.mark.parametrize("M,dsub", [(16, 4), (48, 2), (64, 2)])
def test_head_pass_offers_every_nearest_point(M, dsub):
    """Where the head pass ranks a list by itself (units of the largest radius), the points up to the bin of the k-th byte sum
    and the slack behind it hold the k nearest."""
    rng = np.random.default_rng(M + 1)
    shift = 4 if M > 16 else 2
    assert "constexpr int lmb_shift(int mt) { return mt > 16 ? 4 : 2; }" in SOURCE
    assert "const float lim = HEAD ? add + (float)MT + 2.0f" in SOURCE and "add = HEAD ? 2.0f * err" in SOURCE
    rows = np.arange(M)[None, :]
    for sigma in (0.3, 1.0, 3.0):
        for radius in (0.02, 0.05, 0.1, 0.164, 0.3, 0.6):
            for wide in (1.0, 35.0):
                cb = (0.3 * rng.normal(size=(M, 256, dsub))).astype(f32)
                cb[0] *= f32(wide)
                res = (sigma * rng.normal(size=(M, dsub))).astype(f32)
                r2 = np.full(M, f32(radius) * f32(radius))
                codes = rng.integers(0, 256, size=(5000, M))
                byte, s, off, err = _table(res, cb, r2, r2.max())
                sums = byte[rows, codes].sum(1).astype(np.int64)
                d2 = ((res.astype(np.float64)[:, None, :] - cb.astype(np.float64)) ** 2).sum(2)
                dist = np.minimum(d2, r2[:, None].astype(np.float64))[rows, codes].sum(1)
                slack = int((2 * err).sum() + M + 2) + 1
                for k in (1, 10, 100):
                    kth = np.sort(sums >> shift)[k - 1]
                    limit = ((kth + 1) << shift) - 1 + slack
                    assert np.all(sums[dist <= np.sort(dist)[k - 1] * (1 + 1e-6)] < limit)
