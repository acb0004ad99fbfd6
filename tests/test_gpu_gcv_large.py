"""GCV of large batches: grids whose passes one wavefront takes for a block of 64 series at
sizes where the 21-value grid is spread over several; and more series than a launch has
work-items for with several wavefronts to a block (614,400,000 of 21 values at order 3)."""

import numpy as np
import pytest
import torch

from oracle import whs_ref as R
from paper_2604_00048_amd import whs
from tests import test_gpu_gcv_forms as forms

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dt", [torch.float64, torch.float32])
@pytest.mark.parametrize("d,T,n_grid", [(1, 33, 7), (2, 21, 14), (3, 22, 14), (4, 19, 10)])
def test_grids_of_other_sizes_in_every_form(d, T, n_grid, dt):
    forms.test_every_form_gives_the_same_scores(d, T, n_grid, dt)


def test_more_series_than_a_split_launch_holds():
    T, d, nb = 4, 3, 9_600_000
    r = np.random.default_rng(4)
    x = torch.tensor(r.normal(size=(1, T, 1, 64)), dtype=torch.float32, device="cuda")
    w = torch.ones((1, T, 64), dtype=torch.uint8, device="cuda")
    w[0, 1, ::5] = 0
    grid = torch.tensor(R.gcv_grid(), device="cuda")
    lb0, _, in0 = whs.whs_gcv(x, w, grid, d, 64)
    ref, _, _ = R.gcv_scores(x[0, :, 0].T.double().cpu().numpy(), w[0].T.cpu().numpy(), R.gcv_grid(), d)
    full = w[0].cpu().numpy().all(axis=0)          # with as many observations as the order a score is 0 / 0
    got = lb0.cpu().numpy()[full]
    best = np.array([row[np.argmin(np.abs(R.gcv_grid() - g))] for row, g in zip(ref[full], got)])
    assert (best <= ref[full].min(1) * (1 + 1e-7)).all()
    lb, _, info = whs.whs_gcv(x.expand(nb, -1, -1, -1).contiguous(), w.expand(nb, -1, -1).contiguous(), grid, d, 64 * nb)
    torch.cuda.synchronize()
    for got, one in ((lb.view(nb, 64), lb0), (info.view(nb, 64), in0)):
        for part in got.split(1_000_000):
            assert torch.equal(part.nan_to_num(nan=-1.0), one.nan_to_num(nan=-1.0).expand_as(part))
