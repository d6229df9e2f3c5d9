"""The error bound of the filtering stage's split (bf16 pair) product, on the CPU: what the three
products drop, evaluated over the mantissas of fp32, against the constant the selection counts."""
import os
import re

import numpy as np

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _constant(name):
    text = open(os.path.join(ROOT, "paper_2312_01712_amd", "csrc", "coarse.hip")).read()
    return float(re.search(r"constexpr float %s = ([0-9.e+-]+)f;" % name, text).group(1))


def _bf16(x):
    """Nearest bf16, ties to even."""
    u = x.astype(np.float32).view(np.uint32).astype(np.uint64)
    return ((u + 0x7FFF + ((u >> 16) & 1)) & 0xFFFF0000).astype(np.uint32).view(np.float32)


def _parts(x):
    hi = _bf16(x)
    lo = _bf16(x - hi)          # x - hi is exact
    return hi.astype(np.float64), lo.astype(np.float64)


def _dropped(q, c):
    """|q c - (qh ch + qh cl + ql ch)| / |q c|, exactly up to the roundings of 64 bits."""
    (qh, ql), (ch, cl) = _parts(q), _parts(c)
    q, c = q.astype(np.float64), c.astype(np.float64)
    return np.abs((q - qh) * c + qh * (c - ch) - qh * cl - ql * ch) / np.abs(q * c)


def test_dropped_part_is_counted():
    # in units of |q|^2 + |c|^2 >= 2 |q c|, the proposal's -2 q.c being off by twice the dropped part
    limit = _constant("SPLIT_ERR")
    worst = 0.0
    for first in range(0, 1 << 23, 1 << 20):
        x = ((0x3F800000 + first + np.arange(1 << 20)).astype(np.uint32)).view(np.float32)   # every mantissa
        worst = max(worst, _dropped(x, x).max())
        for y in (np.float32(1.0039136), np.float32(1.0039063), np.float32(1.9960938), x[::-1].copy()):
            worst = max(worst, _dropped(x, np.full_like(x, y) if np.ndim(y) == 0 else y).max())
    assert 2.9e-5 < worst <= limit, (worst, limit)


def test_truncated_keys_are_counted():
    # 6 low bits of a value of at most 2 (|q|^2 + |c|^2)
    assert 63 * 2.0 ** -23 * 2 <= _constant("KEY_ERR") < 1.6e-5
