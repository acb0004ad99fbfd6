"""A plan's groups against whs_solve on the same group: bit for bit where both run one
lane per series (float64; order 3 and 4; fewer than 96 steps, or 512 with one weight per
series; more than 32,768 series), and within the accuracy bar where whs_solve runs several
segments per series, which eliminate in another order."""

import numpy as np
import pytest
import torch

from oracle import whs_ref as R
from paper_2604_00048_amd import synth, whs
from tests._cases import assert_solution, random_case

pytestmark = pytest.mark.gpu

SAME = [  # dtype, per_diff, [(T, d, n)]
    (torch.float32, False, [(511, 2, 70), (511, 1, 65), (95, 2, 64), (730, 3, 33), (365, 4, 10)]),
    (torch.float32, True, [(95, 1, 70), (95, 2, 130), (600, 3, 20)]),
    (torch.float64, False, [(730, 2, 70), (1461, 1, 20)]),
    (torch.float64, True, [(512, 2, 70), (730, 1, 20)]),
    (torch.float32, False, [(520, 2, 32769)]),
    (torch.float32, True, [(100, 1, 32833)]),
]
CLOSE = [
    (torch.float32, False, [(512, 2, 70), (512, 1, 65), (730, 2, 2100), (1461, 1, 129), (3288, 2, 20)]),
    (torch.float32, True, [(96, 2, 70), (96, 1, 65), (365, 2, 130), (3288, 1, 20)]),
]


def solve_both(dtype, per_diff, shapes):
    """Per group: the batch, the plan's z and info, whs_solve's z and info."""
    groups = []
    for T, d, n in shapes:
        x, w, lam = random_case(n, T, d, per_diff=per_diff, seed=T + d + n, dtype=dtype, p_obs=0.1)
        groups.append(((T, d), synth.Batch(torch.tensor(x), torch.tensor(w), torch.tensor(lam), d)))
    x, w, lam, descs = synth.pack_groups(groups, dtype=dtype, device="cuda")
    plan = whs.Plan(descs, dtype, per_diff=per_diff)
    plan.set_config(1, 2, 1, 0)                     # one lane per series
    z = torch.zeros_like(x)
    info = torch.full((sum(g["n_series"] for g in descs),), -1, dtype=torch.int32, device="cuda")
    plan.solve(w, lam, x, z, info)
    for (_, b), desc in zip(groups, descs):
        lam1 = b.lam.to(dtype).cuda() if not per_diff else synth.pack_rows(b.lam.to(dtype), 64).cuda()
        z1, info1 = whs.whs_solve(synth.pack_series(b.x.to(dtype), 64).cuda(), synth.pack_rows(b.w, 64).cuda(), lam1,
                                  desc["d"], b.P)
        torch.cuda.synchronize()
        yield (b, synth.unpack_group(z, desc), info[desc["info_off"]:desc["info_off"] + b.P],
               synth.unpack_series(z1, b.P), info1)
    plan.close()


@pytest.mark.parametrize("dtype,per_diff,shapes", SAME)
def test_one_lane_both_ways_is_the_same_bit_for_bit(dtype, per_diff, shapes):
    for b, z, info, z1, info1 in solve_both(dtype, per_diff, shapes):
        assert torch.equal(info, info1), (b.x.shape, b.d)
        assert torch.equal(z.nan_to_num(nan=-1e30), z1.nan_to_num(nan=-1e30)), (b.x.shape, b.d)


@pytest.mark.parametrize("dtype,per_diff,shapes", CLOSE)
def test_segments_agree_with_the_plan_within_the_bar(dtype, per_diff, shapes):
    for b, z, info, z1, info1 in solve_both(dtype, per_diff, shapes):
        assert torch.equal(info, info1), (b.x.shape, b.d)
        k = np.r_[0:min(b.P, 40)]
        x, w, lam = b.x.numpy()[k], b.w.numpy()[k], b.lam.numpy()[k]
        ref, iref = R.solve_band(x, w, lam, b.d)
        for got in (z, z1):
            assert_solution(got[k].double().cpu().numpy(), ref, x, w, lam, b.d, False, info=iref)
