"""The GCV kernel's forms (grid over lanes, over wavefronts, in one wavefront) give every
grid value the same score: large batches of repeated series against the small batch,
which is checked against the oracle."""

import numpy as np
import pytest
import torch

from oracle import whs_ref as R
from paper_2604_00048_amd import whs
from tests._cases import random_case, to_device

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dt", [torch.float64, torch.float32])
@pytest.mark.parametrize("d,T,n_grid", [(1, 41, 21), (2, 23, 21), (2, 9, 1), (2, 50, 40), (3, 37, 8), (4, 30, 21)])
def test_every_form_gives_the_same_scores(d, T, n_grid, dt):
    P0 = 64
    x, w, _ = random_case(P0, T, d, per_diff=False, seed=7 * d + T, p_obs=0.5, dtype=dt)
    w[5] = 0                                      # fails for every weight
    x[5] = 0
    grid = np.tile(R.gcv_grid(), 2)[:n_grid]      # equal values: the first minimum is kept
    xt, wt, _ = to_device(x, w, np.ones(P0), 64, dt)
    gt = torch.tensor(grid, device="cuda")
    lb0, sc0, in0 = whs.whs_gcv(xt, wt, gt, d, P0, want_scores=True)
    ref, _, _ = R.gcv_scores(x[:, :, 0], w, grid, d)
    ok = np.isfinite(ref)
    s0 = sc0.cpu().numpy()
    assert (np.abs(s0[ok] - ref[ok]) <= 1e-7 * np.abs(ref[ok])).all()
    # over lanes (two sizes, the second with a ragged end), over wavefronts, alone on a SIMD
    for P in (200, 8192 // (-(-n_grid // 8)) * 3 + 8, 16384 + 7, 49152 + 64, 65536):
        nb = -(-P // 64)
        lb, sc, info = whs.whs_gcv(xt.expand(nb, -1, -1, -1).contiguous(), wt.expand(nb, -1, -1).contiguous(), gt, d, P,
                                   want_scores=True)
        torch.cuda.synchronize()
        for got, one in ((lb, lb0), (sc, sc0), (info, in0)):
            want = one.repeat(nb, *([1] * (one.dim() - 1)))[:P]
            assert torch.equal(got.nan_to_num(nan=-1.0) if got.is_floating_point() else got,
                               want.nan_to_num(nan=-1.0) if want.is_floating_point() else want), (P, n_grid)
