"""The two fp32 gradients of a layer in one launch: against the oracle, from one run to the next, and the input gradient bit for bit against
the launch of its own that it has in a block without weight gradients."""
import pytest

import bsr_synth as S
from gpu_common import product_kernels
from test_gpu_kernels import env  # noqa: F401  (a fixture)
from test_gpu_parity import TOL_FP32, check_step, hip  # noqa: F401  (hip is a fixture)

pytestmark = pytest.mark.gpu

# ragged edges of 32 x 32 tiles, few and many rows against the width (either product first), 64 x 64 tiles for one of the products or
# both, and one product too large for the joint launch; the last number: how many of the four layers have one
LAYERS = [(64, 72, 33, 1, 4), (64, 8, 1, 3, 4), (64, 72, 129, 5, 4), (192, 776, 65, 4, 4), (192, 768, 65, 16, 4), (384, 1544, 197, 1, 4),
          (384, 1536, 197, 8, 4), (256, 1024, 1024, 8, 3)]


def a_step(torch, P, cfg, p, x):
    """-> its kernels' names, its gradients (of a second run, on buffers that held none)"""
    ctx = P.Context(cfg, p, cfg["batch"])
    xin = torch.as_tensor(x).cuda().to(ctx.act_dtype).contiguous()
    xf = torch.empty((cfg["batch"], ctx.T_f, cfg["dim"]), dtype=ctx.act_dtype, device="cuda")
    loss, grads = torch.zeros(4, device="cuda"), ctx.new_grads()

    def step():
        ctx.bsr_forward_frozen(xin, x_out=xf)
        ctx.bsr_train_blocks_fwd_bwd(xf, None, grads, loss_out=loss)

    names = product_kernels(step)
    first = {n: g.clone() for n, g in grads.items()}
    for g in grads.values():
        g.fill_(float("nan"))
    step()
    assert all(torch.equal(first[n], g) for n, g in grads.items())
    return names, grads


@pytest.mark.parametrize("dim,hidden,tokens,batch,joint", LAYERS)
def test_joint_gradients_of_a_layer(hip, orc64, env, dim, hidden, tokens, batch, joint):
    torch, P = env
    cfg = S.get_config("c1_block_fp32", dim=dim, heads=dim // 64, mlp_hidden=hidden, tokens_in=tokens, batch=batch, drop_blocks=[])
    p = S.make_params(cfg, std=0.05)
    x, y = S.make_inputs(cfg)
    check_step(hip, orc64, cfg, p, x, y, TOL_FP32, free_running=False)
    names, _ = a_step(torch, P, cfg, p, x)
    assert sum("pair" in n for n in names) == joint


@pytest.mark.parametrize("dim,hidden,tokens,batch,joint", LAYERS)
def test_the_input_gradient_has_the_bits_of_a_launch_of_its_own(env, dim, hidden, tokens, batch, joint):
    torch, P = env
    cfg = S.get_config("c1_block_fp32", dim=dim, heads=dim // 64, mlp_hidden=hidden, tokens_in=tokens, batch=batch, depth=2, first_trainable=0,
                       drop_blocks=[])
    p = S.make_params(cfg, std=0.05)
    x, _ = S.make_inputs(cfg)
    both, grads = a_step(torch, P, cfg, p, x)
    first, passed = a_step(torch, P, dict(cfg, trainable_blocks=[0]), p, x)      # block 1 only passes the gradient on
    assert sum("pair" in n for n in both) == 2 * joint and sum("pair" in n for n in first) == joint
    assert len(passed) < len(grads) and all(torch.equal(grads[n], g) for n, g in passed.items())
