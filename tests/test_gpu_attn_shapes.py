"""GPU parity of attention at the edges of its launch shapes (workgroups of 4,
8 and 12 wavefronts of 32 rows, staged 128 or 288 rows at a time) and with
numbers of workgroups that do not divide by the eight XCDs, against the FP64
reference with the bars of the other attention tests."""

import pytest

from tests.test_gpu_tf import check_attention

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("P,T", [(5, 16), (3, 33), (7, 160), (2, 161), (1, 256), (3, 257), (2, 288), (1, 289), (1, 384),
                                 (3, 385), (1, 513)])
def test_attention_at_the_edges_of_its_shapes(P, T):
    check_attention(P, T)
