"""The guard band of the prefill's projected signs (kSignBand): outside it the sign of a matrix-core sum
has to be the fixed-order binary32 chain's for any adder that the matrix cores may have. No GPU: models of
the adder that truncate, on rows whose sums cancel."""
import os
import re

import numpy as np

from paper_2603_26110_amd import synth

SOURCE = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2603_26110_amd", "csrc",
                      "tq_quantize.hip")


def _band():
    with open(SOURCE) as f:
        return float.fromhex(re.search(r"kSignBand = (0x1p-\d+)f", f.read()).group(1))


def _truncate(v):
    """fp64 to fp32 towards zero."""
    f = v.astype(np.float32)
    return np.where(np.abs(f.astype(np.float64)) > np.abs(v), np.nextafter(f, np.float32(0)), f).astype(np.float64)


def _parts(v):
    hi = v.astype(np.float16).astype(np.float64)
    return hi, (v - hi).astype(np.float16).astype(np.float64)


def _products(a, b):
    """hi hi, hi lo and lo hi of each step of 16, in the kernel's order: [3 x 4][rows][16]."""
    (ah, al), (bh, bl) = _parts(a), _parts(b)
    steps = [slice(16 * q, 16 * q + 16) for q in range(4)]
    return [x[:, s] * y[:, s] for s in steps for x, y in ((ah, bh), (ah, bl), (al, bh))]


def _one_by_one(parts):
    acc = np.zeros(len(parts[0]))
    for p in parts:
        for k in range(p.shape[1]):
            acc = _truncate(acc + p[:, k])
    return acc


def _aligned(parts):
    """Each instruction's 16 products and its addend cut to 24 bits below the largest of them, then summed."""
    acc = np.zeros(len(parts[0]))
    for p in parts:
        t = np.concatenate([acc[:, None], p], 1)
        unit = 2.0 ** (np.floor(np.log2(np.maximum(np.abs(t).max(1, keepdims=True), 1e-300))) - 23)
        acc = _truncate((np.trunc(t / unit) * unit).sum(1))
    return acc


def _chain(a, b):
    acc = np.zeros(len(a))
    for k in range(64):
        acc = (a[:, k] * b[:, k] + acc).astype(np.float32).astype(np.float64)
    return acc


def test_band_covers_every_order_of_truncated_additions():
    # units of ||S_i|| ||r||: 192 truncated additions to partial sums of at most 1/2, the split's products
    # and spacing, and the chain; twice over
    bound = 192 * 2.0 ** -24 + 2.0 ** -20.4 + 2.0 ** -21 + 64 * 2.0 ** -25
    assert _band() >= 2 * bound
    g = synth.rng(5)
    worst = 0.0
    for turn in range(4):
        r = g.standard_normal((2000, 64))
        S = g.standard_normal((2000, 64))
        if turn % 2:                                             # all of one sign, then all of the other
            S = np.abs(S) * np.sign(r) * np.where(np.arange(64) < 32, 1.0, -1.0)
        if turn >= 2:                                            # one large term, cancelled by the last
            r[:, 1:63] *= 0.05
            r[:, 0], r[:, 63], S[:, 0], S[:, 63] = 8.0, 8.0, 8.0, -8.0
        S -= (S * r).sum(1, keepdims=True) / (r * r).sum(1, keepdims=True) * r
        S = (S / 2.0 ** np.floor(np.log2(np.abs(S).max(1, keepdims=True)))).astype(np.float32).astype(np.float64)
        r = (r / 2.0 ** np.floor(np.log2(np.linalg.norm(r, axis=1, keepdims=True)))).astype(np.float32).astype(np.float64)
        norms = np.linalg.norm(S, axis=1) * np.linalg.norm(r, axis=1)
        chain = _chain(S, r)
        for adder in (_one_by_one, _aligned):
            worst = max(worst, np.max(np.abs(adder(_products(S, r)) - chain) / norms))
    assert worst <= bound, worst
