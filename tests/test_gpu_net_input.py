"""The network's input through LDS tiles, which batches of two million series-days and more
take: element for element the series-contiguous form, on either side of the rule."""

import pytest

from tests import test_gpu_net_layout as layout

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("P,T,S,d", [(1001, 2100, 64, 2), (16500, 131, 128, 1), (4096, 512, 64, 2), (4096, 511, 64, 2),
                                     (65, 33000, 64, 3)])
def test_large_batches_equal_the_contiguous_form(P, T, S, d):
    layout.test_tiles_equal_the_contiguous_form(P, T, S, d)
