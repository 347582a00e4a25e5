"""GPU parity of the fp32 matrix-core kernels (products and attention) at the edges of their tiles, against the oracle."""
import re

import pytest

import bsr_synth as S
from gpu_common import product_kernels
from test_gpu_kernels import env  # noqa: F401  (a fixture)
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


# a 192-wide block: 32 x 32 tiles for 8 and 32 sequences, 64 x 64 ones for three products of 16
@pytest.mark.parametrize("batch,wider", [(8, 0), (16, 3), (32, 0)])
def test_no_product_takes_a_larger_tile_than_its_area_asks_for(env, batch, wider):
    """More k in one chain of additions: gradients of the step of 32 sequences are 1.35e-7 off their values in 64 bits with 32 x 32
    tiles, 1.44e-7 with 64 x 64 ones for the wider products."""
    torch, P = env
    cfg = S.get_config("c1_block_fp32", batch=batch)
    x, _ = S.make_inputs(cfg)
    ctx = P.Context(cfg, S.make_params(cfg), batch)
    xin = torch.as_tensor(x).cuda().to(ctx.act_dtype).contiguous()
    xf = torch.empty((batch, ctx.T_f, cfg["dim"]), dtype=ctx.act_dtype, device="cuda")
    loss, grads = torch.zeros(4, device="cuda"), ctx.new_grads()

    def step():
        ctx.bsr_forward_frozen(xin, x_out=xf)
        ctx.bsr_train_blocks_fwd_bwd(xf, None, grads, loss_out=loss)

    # (a launch of both gradients of a layer names the tile of each)
    edges = [int(e) for n in product_kernels(step) for e in re.findall(r"<(\d+),", n)]
    assert len(edges) == 12 and sorted(edges) == [32] * (12 - wider) + [64] * wider
