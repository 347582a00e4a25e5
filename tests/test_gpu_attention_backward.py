"""GPU parity of the one-launch attention backward at the edges of its blocks of 32 tokens, against the oracle."""
import pytest

import test_gpu_kernels
from test_gpu_kernels import env  # noqa: F401  (a fixture)

pytestmark = pytest.mark.gpu


# whole blocks, one token less and one more, up to its limit of 224 and the first length past it
@pytest.mark.parametrize("B,T,H", [(1, 2, 1), (2, 31, 1), (1, 32, 2), (2, 64, 1), (1, 65, 3), (2, 160, 2), (1, 161, 1), (1, 192, 2), (2, 223, 1), (1, 224, 2),
                                   (1, 225, 1)])
def test_attention_backward_at_block_edges(env, orc64, B, T, H):
    test_gpu_kernels.test_attention_backward(env, orc64, B, T, H)
