"""A layer's two gradients behind a GELU' at many rows: two launches, and the bits of the joint one."""
import re

import pytest

import bsr_synth as S
from gpu_common import families, product_kernels
from test_gpu_kernels import env  # noqa: F401  (a fixture)

pytestmark = pytest.mark.gpu

APART, JOINT = ["tiled", "wgrad"], ["joint"]


# either side of the lines of large and of smaller weight matrices, also where the rounds of tiles of one shape or another just end; matrices too
# small for it; without a GELU'
@pytest.mark.parametrize("rows,kin,out,gelu,kernels", [
    (9456, 3072, 768, True, JOINT), (10239, 3072, 768, True, JOINT), (10240, 3072, 768, True, APART), (11328, 3072, 768, True, APART),
    (12608, 3072, 768, True, APART), (14200, 3072, 768, True, APART), (16400, 3072, 768, True, APART), (17731, 3072, 768, True, APART),
    (17731, 3072, 768, False, JOINT), (19700, 3072, 768, True, APART), (10240, 1536, 384, True, JOINT), (13311, 1536, 384, True, JOINT),
    (13312, 1536, 384, True, APART), (20480, 1536, 384, True, APART), (20480, 384, 384, True, JOINT), (20480, 768, 192, True, JOINT)])
def test_gradients_behind_a_gelu_at_many_rows(env, rows, kin, out, gelu, kernels):
    torch, P = env
    g = torch.Generator(device="cuda").manual_seed(rows)
    rnd = lambda *s: torch.randn(s, generator=g, device="cuda").bfloat16()      # noqa: E731
    x, dy, w, u = rnd(rows, kin), rnd(rows, out), rnd(kin, out), rnd(rows, kin)
    ws = torch.empty(2 * (8 * kin * out + 16 * max(kin, out)), device="cuda")
    call = lambda tile=0: P.bsr_linear_backward(x, dy, w, u=u if gelu else None, workspace=ws, tile=tile)      # noqa: E731
    got, joint = call(), call(7128128)
    torch.cuda.synchronize()
    assert all(torch.equal(a, b) for a, b in zip(got, joint))
    assert families(n for n in product_kernels(call) if "gemm_" in n) == kernels


JOINT_TILES = [(128, 64), (128, 128), (192, 128), (256, 128)]      # of the input gradient, by the kernel's first number


def launches_of(choices):
    """[(family, rows, columns of the tile)] that the choices of a trained part name: the forward products, then a layer's gradients each"""
    out, layers = [], len(choices) // 2
    for i, (_, _, _, tile, _) in enumerate(choices):
        shape = (tile % 1000000 // 1000, tile % 1000)
        joint = i >= layers and tile < 9000000 and shape in JOINT_TILES
        out.append(("joint" if joint else "tiled", *shape))
        if i >= layers and not joint:
            out.append(("wgrad", 0, 0))
    return out


def launches_run(names):
    out = []
    for name, kind in zip(names, families(names)):
        a, b = (int(v) for v in re.search(r"<(\d+), (\d+)", name).groups()) if kind != "wgrad" else (0, 0)
        out.append((kind, *(JOINT_TILES[a] if kind == "joint" else (a, b))))
    return out


# past the line with either width, and before it
@pytest.mark.parametrize("dim,batch", [(768, 100), (384, 90), (384, 60)])
def test_a_tuned_step_runs_what_its_choices_name(env, dim, batch):
    torch, P = env
    cfg = S.get_config("c1_block_fp32", dtype="bf16", dim=dim, heads=dim // 64, mlp_hidden=4 * dim, tokens_in=197, batch=batch, depth=2, drop_blocks=[],
                       first_trainable=1)
    x, _ = S.make_inputs(cfg)
    ctx = P.Context(cfg, S.make_params(cfg), batch)
    xin = torch.as_tensor(x).cuda().to(ctx.act_dtype).contiguous()
    xf, xs = (torch.empty((batch, ctx.T_f, dim), dtype=ctx.act_dtype, device="cuda") for _ in range(2))
    loss, grads = torch.zeros(4, device="cuda"), ctx.new_grads()
    step = lambda: ctx.bsr_train_blocks_fwd_bwd(xf, None, grads, loss_out=loss)      # noqa: E731
    ctx.bsr_forward_frozen(xin, x_out=xf)
    step()
    first = {n: g.clone() for n, g in grads.items()}
    untuned = launches_run(product_kernels(step, "gemm_nt", "gemm_pair", "gemm_tn"))
    side = torch.cuda.Stream()
    torch.cuda.synchronize()
    for tune in (lambda: ctx.bsr_autotune(xin, None, xf, loss, grads),
                 lambda: ctx.bsr_autotune_overlapped(xin, None, xf, xs, loss, grads, side)):
        _, changed = tune()
        choices = ctx.bsr_tile_choices(1)
        assert len(choices) == 8
        ran = launches_run(product_kernels(step, "gemm_nt", "gemm_pair", "gemm_tn"))
        assert ran == launches_of(choices), (choices, untuned)
        assert all(torch.equal(first[n], g) for n, g in grads.items())
        if changed == 0:                      # every launch as it is without a choice
            assert ran == untuned, choices
