"""Several bands in segments: the launches of one call (3 and fewer bands of a solve,
2 and fewer of an adjoint) factor a series in the same segments, so they agree on
which series are singular to working precision; and two and four segments, where the
number of bands, the order and the weights decide between segments and one lane per
series."""

import numpy as np
import pytest
import torch

from paper_2604_00048_amd import synth, whs
from tests._cases import from_device_rows, from_device_series, random_case, to_device
from tests.test_gpu_seg import _check

pytestmark = pytest.mark.gpu


def nearly_singular(P, T, d, C, seed):
    """Between d and d + 3 observations and weights up to 1e10 (order 2) or of 1e10 to 1e14
    throughout (order 1): pivots around the rounding of larger terms, on either side of zero."""
    r = np.random.default_rng(seed)
    w = np.zeros((P, T), dtype=np.uint8)
    for p in range(P):
        w[p, r.choice(T, size=d + p % 4, replace=False)] = 1
    top = r.choice([6.0, 7.0, 8.0, 9.0, 10.0], size=(P, 1)) + 4.0 * (2 - d)
    lam = 10.0 ** (r.uniform(-1.0, 1.0, size=(P, T - d)) * (top - 1.0) / 2 + (top + 1.0) / 2)
    if d == 1:
        lam = 10.0 ** top * r.uniform(1.0, 2.0, size=lam.shape)
    x = 0.3 + 0.1 * r.normal(size=(P, T, C))
    return x, w, lam.astype(np.float32).astype(np.float64)


@pytest.mark.parametrize("P,T,d,C", [(1500, 3288, 2, 4), (1500, 1000, 2, 7), (1500, 3288, 1, 10), (1500, 3288, 2, 3),
                                     (3000, 1000, 2, 5)])
def test_bands_agree_on_singular_series(P, T, d, C):
    x, w, lam = nearly_singular(P, T, d, C, seed=P + T + C)
    xt, wt, lt = to_device(x, w, lam, 64, torch.float32)
    z, info = whs.whs_solve(xt, wt, lt, d, P)
    g = synth.pack_series(torch.randn((P, T, C), generator=torch.Generator().manual_seed(C)), 64).cuda()
    zin = synth.pack_series(torch.randn((P, T, C), generator=torch.Generator().manual_seed(d)), 64).cuda()
    gx, gl, jnfo = whs.whs_backward(wt, lt, zin, g, d, P)
    torch.cuda.synchronize()
    bad, gbad = info.cpu().numpy() != 0, jnfo.cpu().numpy() != 0
    assert 0 < bad.sum() < P and 0 < gbad.sum() < P   # series on either side
    for got, fail in ((from_device_series(z, P), bad), (from_device_series(gx, P), gbad)):
        nan = np.isnan(got)
        np.testing.assert_array_equal(nan.all(axis=(1, 2)), fail)
        np.testing.assert_array_equal(nan.any(axis=(1, 2)), fail)
    gl = np.isnan(from_device_rows(gl, P).reshape(P, -1))
    np.testing.assert_array_equal(gl.all(1), gbad)
    np.testing.assert_array_equal(gl.any(1), gbad)


@pytest.mark.parametrize("P,T,d,C,per_diff", [
    (16385, 131, 2, 2, True), (16451, 400, 1, 3, False), (20001, 100, 2, 4, False), (20001, 97, 1, 4, False),
    (32768, 97, 2, 7, True), (16400, 150, 1, 10, True), (16390, 96, 2, 5, True), (8193, 120, 2, 3, True), (16384, 113, 1, 4, True),
])
def test_bands_in_two_and_four_segments(P, T, d, C, per_diff):
    x, w, lam = random_case(P, T, d, C=C, per_diff=per_diff, seed=P + T + C, dtype=torch.float32, p_obs=0.1)
    _check(x, w, lam, d, P, rows=np.r_[0:3, P // 2:P // 2 + 3, P - 3:P])
