"""Series-contiguous batches of more than 32,768 series, which take one segment: the
recurrence that the interleaved call of that size runs, so the same results bit for
bit; and against the oracle, on the first, last and middle series."""

import numpy as np
import pytest
import torch

from oracle import whs_ref as R
from paper_2604_00048_amd import whs
from tests import test_gpu_seg as seg
from tests._cases import assert_solution, from_device_series, random_case, to_device

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("P,T,d,per_diff,k_x,k_w", [
    (32769, 96, 2, True, 0, 1), (32801, 131, 2, True, 1, 3), (32801, 131, 1, True, 3, 2), (40000, 96, 2, False, 0, 0),
    (33000, 530, 2, False, 1, 1), (33000, 515, 1, False, 2, 3), (65599, 121, 2, True, 0, 0),
])
def test_large_contiguous_batches_equal_interleaved_ones(P, T, d, per_diff, k_x, k_w):
    seg.test_contiguous_arrays_match_interleaved_bit_for_bit(P, T, d, per_diff, k_x, k_w)


@pytest.mark.parametrize("P,T,d", [(32801, 131, 2), (32833, 100, 1)])
def test_large_contiguous_batches_against_the_oracle(P, T, d):
    x, w, lam = random_case(P, T, d, per_diff=True, seed=P + T, dtype=torch.float32, p_obs=0.1)
    w[P - 2] = 0                       # singular
    lam[P // 2, T // 2] = -1e6         # indefinite
    x1, w1, l1 = to_device(x, w, lam, 1, torch.float32)
    z, info = whs.whs_solve(x1, w1, l1, d, P)
    torch.cuda.synchronize()
    rows = np.r_[0:3, P // 2 - 1:P // 2 + 2, P - 3:P]
    x, w, lam = x[rows], w[rows], lam[rows]
    zref, iref = R.solve_band(x, w, lam, d)
    assert (iref != 0).sum() == 2
    got = from_device_series(z, P)[rows]
    np.testing.assert_array_equal(info.cpu().numpy()[rows] != 0, iref != 0)
    assert np.isnan(got[iref != 0]).all()
    assert_solution(got, zref, x, w, lam, d, False, info=iref)
