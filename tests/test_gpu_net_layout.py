"""The network's input and head for layouts of whole groups of 64 series go through
LDS in tiles of 64 x 64; element for element they equal the series-contiguous form.
The weight gradient of a hidden layer takes items of 64 rows."""

import numpy as np
import pytest
import torch

from oracle import convnet_ref as N
from paper_2604_00048_amd import net
from tests.test_gpu_net import from_bf, rel, to_bf

pytestmark = pytest.mark.gpu
dev = "cuda"


@pytest.mark.parametrize("P,T,S,d", [(1, 5, 64, 1), (64, 64, 64, 2), (65, 67, 64, 2), (100, 131, 128, 3), (200, 3, 64, 2),
                                     (129, 127, 192, 1)])
def test_tiles_equal_the_contiguous_form(P, T, S, d):
    nb = -(-P // S)
    g = torch.Generator(device=dev).manual_seed(P + T)
    x1 = torch.randn((P, T), generator=g, device=dev)
    w1 = (torch.rand((P, T), generator=g, device=dev) < 0.5).to(torch.uint8)
    h = torch.randn((P, T), generator=g, device=dev) * 3
    x1[0, 1] = float("nan")
    h[0, T // 2] = float("nan")
    feat = torch.randn((T, 4), generator=g, device=dev)

    def blocks(v):                                    # (P, T) -> (nb, T, S), rows past the batch unused
        pad = torch.full((nb * S, T), 7, dtype=v.dtype, device=dev)
        pad[:P] = v
        return pad.view(nb, S, T).transpose(1, 2).contiguous()

    one = net.net_input(x1.view(P, T, 1, 1), w1.view(P, T, 1), P, T, 1, 0.3, 0.1, feat)
    got = net.net_input(blocks(x1).view(nb, T, 1, S), blocks(w1), P, T, S, 0.3, 0.1, feat)
    assert torch.equal(got.view(torch.int16), one.view(torch.int16))

    def lam(S, nb):
        out = torch.full((nb, T - d, S), -5.0, device=dev)
        assert net.lib().whs_net_head_fwd(net._p(h), P, T, S, d, -1.0, 5.0, net._p(out), net._s(out.device)) == 0
        return out

    rows = lam(1, P)[:, :, 0]
    tiles = lam(S, nb).transpose(1, 2).reshape(nb * S, T - d)
    assert torch.equal(tiles[:P].view(torch.int32), rows.view(torch.int32))
    assert (tiles[P:] == -5.0).all()                  # rows past the batch are not written


@pytest.mark.parametrize("P,T,parts", [(1, 1, 1), (3, 4, 2), (2, 59, 3), (5, 63, 4), (3, 64, 2), (4, 65, 9), (2, 128, 1),
                                       (7, 133, 5)])
def test_hidden_weight_gradient_at_the_edges_of_its_items(P, T, parts):
    """Ends of a series inside the halo, items cut short, more workgroups than items; the
    bar of the other shapes (FP32 sums of exact bfloat16 products)."""
    r = np.random.default_rng(P * T)
    x, gy = (N.bf16_round(r.normal(size=(P, T, 64))) for _ in range(2))
    grad = torch.empty(64 * 9 * 64 + 64, dtype=torch.float32, device=dev)
    net.conv_wgrad(to_bf(x), 64, to_bf(gy), 64, grad, P, T, parts=parts)
    gW, gb = N.conv1d_wgrad(x, gy)
    g = grad.cpu().double().numpy()
    assert rel(g[:64 * 9 * 64].reshape(64, 9, 64), gW) < 1e-5
    assert rel(g[64 * 9 * 64:], gb) < 1e-5
