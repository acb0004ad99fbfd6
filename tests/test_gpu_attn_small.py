"""Attention on small batches takes workgroups of four wavefronts at every length; each
block's arithmetic is that of the large batch, which the reference covers."""

import pytest
import torch

from paper_2604_00048_amd import tf
from tests.test_gpu_tf import check_attention

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("P,T", [(1, 129), (1, 280), (2, 384), (1, 385), (2, 1000)])
def test_small_batches_against_the_reference(P, T):
    check_attention(P, T)


@pytest.mark.parametrize("n,P,T", [(85, 86, 280), (64, 65, 384), (64, 65, 400), (1, 65, 513), (2, 33, 1030)])
def test_batches_on_either_side_of_the_rule_agree(n, P, T):
    g = torch.Generator(device="cuda").manual_seed(T)
    qkv = torch.randn((P * T, 192), generator=g, device="cuda").bfloat16().view(torch.int16)
    go = torch.randn((P * T, 64), generator=g, device="cuda").bfloat16().view(torch.int16)
    out = []
    for P1 in (n, P):
        o = torch.full((P1 * T, 64), -1, dtype=torch.int16, device="cuda")
        lse = torch.full((P1, 2, T), float("nan"), device="cuda")
        dq = torch.full((P1 * T, 192), -1, dtype=torch.int16, device="cuda")
        tf.attn_fwd(qkv[:P1 * T], P1, T, o, lse)
        tf.attn_bwd(qkv[:P1 * T], o, go[:P1 * T], lse, P1, T, dq)
        out.append([v.reshape(P1, -1) for v in (o, lse, dq)])
    torch.cuda.synchronize()
    for small, large in zip(*out):
        assert torch.equal(large[:n], small)


@pytest.mark.parametrize("P,T,bound", [(64, 40, 1.92e-7), (40, 500, 2.82e-7), (8, 1000, 3.07e-7)])
def test_log_sum_exp_is_as_close_as_with_natural_exponents(P, T, bound):
    """The root mean square error of the log-sum-exps against 64 bits; the bounds are those of
    a kernel that keeps scores in units of e and rounds the scaled score once."""
    g = torch.Generator(device="cuda").manual_seed(T)
    qkv = torch.randn((P * T, 192), generator=g, device="cuda").bfloat16()
    o = torch.empty((P * T, 64), dtype=torch.int16, device="cuda")
    lse = torch.empty((P, 2, T), device="cuda")
    tf.attn_fwd(qkv.view(torch.int16), P, T, o, lse)
    q, k = (qkv[:, 64 * i:64 * i + 64].double().view(P, T, 2, 32).transpose(1, 2).contiguous() for i in (0, 1))
    ref = torch.logsumexp((q @ k.transpose(-1, -2).contiguous()) / 32 ** 0.5, -1)
    assert (lse.double() - ref).pow(2).mean().sqrt().item() <= bound
