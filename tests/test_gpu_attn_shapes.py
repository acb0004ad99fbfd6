"""GPU parity of attention at the edges of its launch shapes (workgroups of 4,
8 and 12 wavefronts of 32 rows, staged 128, 288 or 384 rows at a time) and with
numbers of workgroups that do not divide by the eight XCDs, against the FP64
reference with the bars of the other attention tests."""

import pytest
import torch

from paper_2604_00048_amd import tf
from tests.test_gpu_tf import check_attention

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("P,T", [(5, 16), (3, 33), (7, 160), (2, 161), (1, 256), (3, 257), (2, 288), (1, 289), (1, 384),
                                 (3, 385), (1, 513)])
def test_attention_at_the_edges_of_its_shapes(P, T):
    check_attention(P, T)


@pytest.mark.parametrize("P,T", [(256, 97), (257, 129), (256, 280), (300, 289), (256, 384), (256, 385)])
def test_large_batches_equal_small_ones(P, T):
    """From 256 series on the backward takes a (series, head) in rounds of one
    workgroup; every block's arithmetic is that of the small batch."""
    g = torch.Generator(device="cuda").manual_seed(T)
    n = 5
    qkv = torch.randn((n, T, 192), generator=g, device="cuda").bfloat16().view(torch.int16)
    go = torch.randn((n, T, 64), generator=g, device="cuda").bfloat16().view(torch.int16)
    out = []
    for P1 in (n, P):
        rep = -(-P1 // n)
        q, d = (v.repeat(rep, 1, 1)[:P1].contiguous().reshape(P1 * T, -1) for v in (qkv, go))
        o = torch.full((P1 * T, 64), -1, dtype=torch.int16, device="cuda")
        lse = torch.full((P1, 2, T), float("nan"), device="cuda")
        dq = torch.full((P1 * T, 192), -1, dtype=torch.int16, device="cuda")
        tf.attn_fwd(q, P1, T, o, lse)
        tf.attn_bwd(q, o, d, lse, P1, T, dq)
        out.append([v.reshape(P1, -1) for v in (o, lse, dq)])
    torch.cuda.synchronize()
    for small, large in zip(*out):
        assert torch.equal(large, small.repeat(-(-P // n), 1)[:P])
