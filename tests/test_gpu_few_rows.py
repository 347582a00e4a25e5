"""GPU parity of the products of few rows (wavefronts of a workgroup share k, rings of their own in LDS) at the edges of
their tiles and k-groups, and the tiled kernels' own edges at row counts that stay with them."""
import numpy as np
import pytest

import test_gpu_kernels as K
from test_gpu_kernels import env  # noqa: F401  (a fixture)

pytestmark = pytest.mark.gpu


# one row; a tile and one row more or less; fewer k-groups than wavefronts (64, 128), a ring refilled with some wavefronts
# one group ahead (832 = 13 groups), the longest; columns ending inside a 32- and a 64-wide tile; 788, 1182: 64 x 64 tiles
@pytest.mark.parametrize("M,kin,out", [(1, 64, 8), (31, 128, 40), (33, 192, 72), (64, 832, 104), (65, 3072, 768), (197, 320, 392),
                                       (788, 768, 768), (1182, 3072, 776)])
def test_products_of_few_rows(env, orc64, M, kin, out):
    K.test_linear_forward(env, orc64, M, kin, out)
    if kin % 64 == 0 and out % 64 == 0:
        K.test_linear_dgrad(env, orc64, M, kin, out)
    K.test_layernorm_folded_into_linear(env, orc64, M, kin, out)


# row counts that stay with the tiled kernels whatever the tile shape: the same bits from every shape, ragged edges
@pytest.mark.parametrize("M,kin,out", [(2200, 64, 1544), (2300, 320, 1160), (2050, 832, 2312)])
def test_every_tile_shape_at_larger_row_counts(env, orc64, M, kin, out):
    K.test_every_tile_shape_gives_the_same_bits(env, orc64, M, kin, out)
