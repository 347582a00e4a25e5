"""GPU parity of the fp32 matrix-core kernels (products and attention) at the edges of their tiles, against the oracle."""
import pytest

import bsr_synth as S
from test_gpu_parity import TOL_FP32, check_step, hip  # noqa: F401  (hip is a fixture)

pytestmark = pytest.mark.gpu


# one block on tokens in fp32: 32-wide tiles with ragged edges everywhere; 64-wide ones; 128-wide ones (8192 rows)
@pytest.mark.parametrize("dim,hidden,tokens,batch", [(64, 72, 33, 1), (64, 8, 1, 3), (192, 776, 129, 3), (384, 1536, 197, 8),
                                                     (256, 1024, 1024, 8)])
def test_fp32_block_at_tile_edges(hip, orc64, dim, hidden, tokens, batch):
    cfg = S.get_config("c1_block_fp32", dim=dim, heads=dim // 64, mlp_hidden=hidden, tokens_in=tokens, batch=batch,
                       drop_blocks=[0] if tokens > 1 else [])
    p = S.make_params(cfg, std=0.05)
    x, y = S.make_inputs(cfg)
    check_step(hip, orc64, cfg, p, x, y, TOL_FP32, free_running=False)
