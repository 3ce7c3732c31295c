"""The calibration kernels at the sizes where they can go wrong: counts around
a wave's 16 vectors and the block's 128, the sampled walk (over 512 vectors),
coordinates that all fall into one bin, infinite inputs, and Gram matrices of
low rank.

Tolerances: the tables are fp64 inside and rounded to fp32 at the end, half an
ulp of a level below 8 (2.4e-7); ebar and sigma are relative fp32 roundings
(6e-8) of fp64 results."""
import numpy as np
import pytest
import torch

import paper_2603_26110_amd as tq
from oracle import oracle
from paper_2603_26110_amd import synth

pytestmark = pytest.mark.gpu
INIT = synth.GAUSS_LEVELS_MAX1960


def _keys(seed, H, n):
    g = synth.rng(seed)
    return np.ascontiguousarray(synth.keys(g, 1, 1, n, H, synth.outlier_channels(g, 1, H))[0, 0].transpose(1, 0, 2)), \
        synth.rotations(g, 1, H)[0]


def _d(a):
    return None if a is None else torch.from_numpy(np.ascontiguousarray(a)).cuda()


@pytest.mark.parametrize("rotate", [True, False])
@pytest.mark.parametrize("n", [1, 15, 16, 17, 127, 128, 129, 511, 1029])
def test_tables_and_ebar_at_every_remainder(n, rotate):
    x, pi = _keys(900 + n, 2, n)
    x[1, n // 2] = 0.0
    got = tq.calibrate_lut(_d(x), _d(pi) if rotate else None, INIT)
    eb = tq.calibrate_ebar(_d(x), got, _d(pi) if rotate else None).cpu().numpy()
    got = got.cpu().numpy()
    for h in range(2):
        p = pi[h] if rotate else None
        np.testing.assert_allclose(got[h], oracle.calibrate_lut(x[h], p, INIT), rtol=0, atol=5e-7)
        assert eb[h] == pytest.approx(oracle.calibrate_ebar(x[h], p, got[h]), rel=2e-7)


@pytest.mark.parametrize("n", [600, 2048])
def test_tables_of_equal_coordinates(n):
    # nine in ten coordinates are 0, the middle midpoint of the starting table:
    # a bin that no window holds
    g = synth.rng(31)
    x = (g.standard_normal((2, n, 64)) * (g.random((2, n, 64)) < 0.1)).astype(np.float32)
    x[1, :, 1:] = np.sign(x[1, :, 1:])                     # few values in all
    got = tq.calibrate_lut(_d(x), None, INIT).cpu().numpy()
    for h in range(2):
        np.testing.assert_allclose(got[h], oracle.calibrate_lut(x[h], None, INIT), rtol=0, atol=5e-7)


def _plain_lloyd(u, max_iter, tol):
    """The iteration as it is defined, over all coordinates (NaN compares false throughout)."""
    c = INIT.astype(np.float64)
    for _ in range(max_iter):
        t = 0.5 * (c[1:] + c[:-1])
        idx = (u[:, None] > t).sum(1)
        new = np.array([u[idx == k].mean() if np.any(idx == k) else c[k] for k in range(8)])
        delta = np.nanmax(np.abs(new - c))
        c = np.concatenate([[new[0]], np.sort(new[1:])]) if np.isnan(new[0]) else np.sort(new)
        if delta < tol:
            break
    return c


def test_tables_with_an_infinite_input():
    # its vector's norm is infinite: that coordinate is NaN, the others 0
    g = synth.rng(32)
    x = g.standard_normal((1, 200, 64)).astype(np.float32)
    x[0, 7, 3] = np.inf
    with np.errstate(invalid="ignore"):
        xd = x[0].astype(np.float64)
        u = xd * (8.0 / np.sqrt((xd * xd).sum(1, keepdims=True)))
        ref = _plain_lloyd(u.ravel(), 10, 1e-7)
    got = tq.calibrate_lut(_d(x), None, INIT, max_iter=10).cpu().numpy()[0]
    assert np.isnan(got[0]) and np.isnan(ref[0])
    np.testing.assert_allclose(got[1:], ref[1:], rtol=0, atol=5e-7)


@pytest.mark.parametrize("n", [1, 3, 4, 63, 65, 257, 1025])
def test_rotation_at_every_remainder_and_rank(n):
    x, _ = _keys(950 + n, 3, n)
    x[2] *= 1e-18                                          # (squares of fp64 entries far below fp32's range)
    pi, sg = (a.cpu().numpy().astype(np.float64) for a in tq.calibrate_rotation(_d(x)))
    for h in range(3):
        ref = np.zeros(64)
        s = np.linalg.svd(x[h].astype(np.float64), compute_uv=False)
        ref[:len(s)] = s
        np.testing.assert_allclose(pi[h] @ pi[h].T, np.eye(64), atol=5e-7)
        # singular values of the Gram matrix: its entries are exact to 2^-53 of sigma_0^2
        np.testing.assert_allclose(sg[h], ref, rtol=1e-6, atol=3e-7 * ref[0])
        y = x[h].astype(np.float64) @ pi[h].T
        gram = y.T @ y
        assert np.max(np.abs(gram - np.diag(np.diag(gram)))) <= 1e-6 * ref[0] ** 2
        assert np.all(np.take_along_axis(pi[h], np.abs(pi[h]).argmax(1)[:, None], 1) > 0)


def test_tables_of_more_equal_coordinates_than_32_bits_count():
    # 2^26 vectors of ones: all 2^32 coordinates are 1, in one bin
    x = torch.ones((1, 1 << 26, 64), device="cuda")
    init = np.array([-3, -2, -1, -0.5, 0.5, 1.25, 2, 3], np.float32)
    got = tq.calibrate_lut(x, None, init, max_iter=1).cpu().numpy()[0]
    np.testing.assert_array_equal(got, [-3, -2, -1, -0.5, 0.5, 1, 2, 3])


@pytest.mark.parametrize("n,rotate", [(600, False), (129, True), (5000, True)])
def test_tables_of_coordinates_far_below_the_largest(n, rotate):
    # one channel 1e15 times the others: levels of 1e-14 come from sums of such
    # coordinates, beside levels of 8 (two heads, the second without such)
    g = synth.rng(33)
    x = g.standard_normal((2, n, 64))
    x[0, :, 1:] *= 1e-15
    x = x.astype(np.float32)
    pi = np.zeros((2, 64, 64), np.float32)
    pi[:, 0, 0] = 1.0                                      # (the other channels among themselves)
    pi[:, 1:, 1:] = np.linalg.qr(g.standard_normal((63, 63)))[0]
    got = tq.calibrate_lut(_d(x), _d(pi) if rotate else None, INIT).cpu().numpy()
    for h in range(2):
        ref = oracle.calibrate_lut(x[h], pi[h] if rotate else None, INIT)
        np.testing.assert_allclose(got[h], ref, rtol=2.0 ** -22, atol=0)
        assert np.all(np.diff(got[h]) > 0)
