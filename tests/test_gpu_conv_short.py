"""The 64-to-64 convolution layers on series shorter than their tile of 256 rows, and
on ones that end a few rows into a further tile: a tile's rows past its series are
neither read as data nor written, neither over the next series nor past the last
one, in the output and in its ReLU bits.  Outputs lie inside larger arrays whose other
values must stay.  Against the FP64 reference they may be off by one unit in the last
place of bfloat16 (2^-7) and the bound of an FP32 sum of 9 x 64 products and a bias,
577 x 2^-24 times the sum of their magnitudes."""

import numpy as np
import pytest
import torch

from oracle import convnet_ref as N
from paper_2604_00048_amd import net
from tests.test_gpu_net import from_bf, relu_bits, to_bf

pytestmark = pytest.mark.gpu
dev = "cuda"
ROOM = 300   # rows on either side: more than a tile


def inside(P, T, width, dtype, fill):
    """A (P, T, width) array inside a larger one, and the larger one."""
    buf = torch.full(((P * T + 2 * ROOM) * width,), fill, dtype=dtype, device=dev)
    return buf[ROOM * width:(ROOM + P * T) * width].view(P, T, width), buf.view(-1, width)


def untouched(buf, P, T, fill):
    return bool((buf[:ROOM] == fill).all()) and bool((buf[ROOM + P * T:] == fill).all())


def close(got, ref, size):
    return bool((np.abs(got - ref) <= 2.0 ** -7 * np.abs(ref) + 577 * 2.0 ** -24 * size).all())


@pytest.mark.parametrize("P,T", [(4, 1), (4, 5), (3, 31), (3, 32), (3, 100), (2, 223), (2, 224), (2, 225), (2, 255), (2, 257),
                                 (2, 285), (2, 289), (2, 480), (2, 513)])
def test_rows_past_a_series_are_left_alone(P, T):
    r = np.random.default_rng(1000 * P + T)
    x = N.bf16_round(np.abs(r.normal(size=(P, T, 64))))
    W = N.bf16_round(r.normal(size=(64, 9, 64)) * 0.2)
    b = r.normal(size=64).astype(np.float32).astype(np.float64)
    out, obuf = inside(P, T, 64, torch.int16, 0x3A5A)
    bits, bbuf = inside(P, T, 8, torch.uint8, 0xA5)
    net.conv_fwd(to_bf(x), 64, to_bf(W), torch.tensor(b, dtype=torch.float32, device=dev), 64, 0, None, out, P, T, bits=bits)
    got = from_bf(out)
    assert close(got, np.maximum(N.conv1d_same(x, W, b), 0.0), N.conv1d_same(np.abs(x), np.abs(W), np.abs(b)))
    np.testing.assert_array_equal(bits.cpu().numpy(), relu_bits(got))
    assert untouched(obuf, P, T, 0x3A5A) and untouched(bbuf, P, T, 0xA5)

    # input gradient, with the mask's bits next to bits that are all set
    act = N.bf16_round(np.maximum(r.normal(size=(P, T, 64)), 0.0))
    mask, mbuf = inside(P, T, 8, torch.uint8, 0xFF)
    mask.copy_(torch.tensor(relu_bits(act)))
    gx, gbuf = inside(P, T, 64, torch.int16, 0x3A5A)
    Wd = np.transpose(W[:, ::-1, :], (2, 1, 0)).copy()
    net.conv_fwd(to_bf(x), 64, to_bf(Wd), None, 64, 3, mask, gx, P, T)
    assert close(from_bf(gx), N.conv1d_dgrad(x, W) * (act > 0), N.conv1d_dgrad(np.abs(x), np.abs(W)))
    assert untouched(gbuf, P, T, 0x3A5A) and bool((mbuf[:ROOM] == 0xFF).all())
