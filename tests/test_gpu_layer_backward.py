"""GPU parity of a layer's two gradients where the joint launch can go wrong: token counts around the k-tiles of the weight
gradient (64 tokens) and around its parts, both of its tiles, widths that end inside a tile, and scratch too small for the
parts.  And attention forward: a head by one workgroup or by two is the same bits."""
import re

import numpy as np
import pytest

import test_gpu_kernels as K
from gpu_common import families, product_kernels
from test_gpu_kernels import env  # noqa: F401  (a fixture)

pytestmark = pytest.mark.gpu


# the joint launch: one token .. a few k-tiles, on either side of a k-tile's 64 tokens; columns that end inside its tiles of 64 and 128;
# several parts, the last one ragged, in one workgroup (2111) or more (450 and above), the 256 x 128 tile (13000)
JOINT = [(1, 136, 64), (33, 264, 192), (63, 264, 128), (64, 392, 192), (65, 264, 192), (191, 264, 192), (320, 392, 448), (450, 392, 384), (520, 136, 64),
         (1000, 776, 320), (1337, 776, 704), (2111, 776, 2304), (6305, 776, 768), (13000, 1544, 768),
         (191, 768, 64), (2111, 768, 2304), (4416, 768, 3072), (6304, 3072, 768)]
# two launches, since the input gradient has no whole k-tiles
TWO = [(1, 64, 8), (63, 192, 136), (64, 136, 264), (65, 264, 72), (197, 768, 776), (1000, 264, 520)]


@pytest.mark.parametrize("M,kin,out,kernels", [s + (["joint"],) for s in JOINT] + [s + (["tiled", "wgrad"],) for s in TWO] +
                         [(788, 384, 1536, ["few", "wgrad"])])
def test_both_gradients_within_the_rounding_of_their_sums(env, M, kin, out, kernels):
    """Products of bf16 numbers are exact in fp32 and each of n additions errs by at most 2^-23 of what it adds up to, so an
    fp32 sum is within n 2^-23 of the sum of the terms' magnitudes; dX is then rounded to bf16 (2^-8 of its value)."""
    torch, P = env
    rng = np.random.default_rng(5 * M + kin + out)
    x, dy, w = (K.to_dev(torch, K.bf16_np(rng, s), torch.bfloat16) for s in ((M, kin), (M, out), (kin, out)))
    X, DY, W = x.double(), dy.double(), w.double()
    dx_ref, dw_ref, db_ref = DY @ W.t().contiguous(), X.t().contiguous() @ DY, DY.sum(0)
    dx_mag, dw_mag, db_mag = DY.abs() @ W.abs().t().contiguous(), X.abs().t().contiguous() @ DY.abs(), DY.abs().sum(0)
    per = (kin + 1) * out
    for floats in (0, 2 * per, 16 * per):                   # no room for a second part, for two, for all
        ws = torch.full((floats,), float("nan"), device="cuda") if floats else None
        names = product_kernels(lambda: P.bsr_linear_backward(x, dy, w, workspace=ws))
        assert families(names) == kernels
        if M == 13000 and floats == 16 * per:
            assert re.search(r"gemm_pair_kernel<\d, 1>", names[0]), names
        dx, dw, db = P.bsr_linear_backward(x, dy, w, workspace=ws)
        alone, _ = P.bsr_linear_wgrad(x, dy, workspace=ws)
        torch.cuda.synchronize()
        for name, got, ref, mag, n, rounding in (("dx", dx, dx_ref, dx_mag, out, 2.0 ** -8), ("dw", dw, dw_ref, dw_mag, M, 0.0),
                                                 ("db", db, db_ref, db_mag, M, 0.0), ("dw alone", alone, dw_ref, dw_mag, M, 0.0)):
            over = ((got.double() - ref).abs() - n * 2.0 ** -23 * mag * (1 + rounding) - rounding * ref.abs()).max().item()
            assert over <= 1e-30, f"{name}, scratch for {floats} numbers: {over:.3g} beyond the bound"
    for tile in (160256, 7320256):                          # shapes that the joint launch does not have: two launches, the same bits
        again = P.bsr_linear_backward(x, dy, w, workspace=ws, tile=tile)
        assert all(torch.equal(a, b) for a, b in zip((dx, dw, db), again)), f"tile {tile}"


def test_sums_added_up_by_the_next_launch_are_the_same_bits(env):
    """With one block trained, the partial sums of its last weight gradient are added up by a launch of their own; with two, by spare
    wavefronts of the next block's first joint launch."""
    import bsr_synth as S
    torch, P = env
    grads = []
    for first in (2, 1):
        cfg = S.get_config("c1_block_fp32", dtype="bf16", depth=3, first_trainable=first, drop_blocks=[], tokens_in=130, batch=8)
        x, _ = S.make_inputs(cfg)
        ctx = P.Context(cfg, S.make_params(cfg), 8)
        xf = torch.empty((8, ctx.T_f, cfg["dim"]), dtype=ctx.act_dtype, device="cuda")
        ctx.bsr_forward_frozen(torch.as_tensor(x).cuda().to(ctx.act_dtype).contiguous(), x_out=xf)
        loss, g = torch.zeros(4, device="cuda"), ctx.new_grads()
        names = product_kernels(lambda: ctx.bsr_train_blocks_fwd_bwd(xf, None, g, loss_out=loss), "splitk_reduce", "gemm_pair")
        # (the layer from 192 to 768 takes the kernel for few rows)
        assert ["splitk_reduce" in n for n in names] == [False] * 3 * (3 - first) + [True]
        grads.append({n: t.clone() for n, t in g.items() if n.startswith("blocks.2.")})
    assert len(grads[0]) == 12
    for n, t in grads[0].items():
        assert torch.equal(t, grads[1][n]), n


# parts of at least four k-tiles (64 tokens each), for 384 or, from 96 k-tiles on, 512 workgroups of 128 x 128, at most 16
def tokens_per_part(M, kin, out):
    nk, tiles = -(-M // 64), -(-kin // 128) * -(-out // 128)
    parts = max(1, min((512 if nk >= 96 else 384) // tiles, nk // 4, 16))
    return 64 * -(-nk // parts)


# a part a workgroup (1000, 4 parts), all of a tile's parts in one (2111: 3; 2144: 2), runs of 3, 2 (1337), 3, 3, 1 (2144) and 4, 4, 3
# (6305) parts, the 256 x 128 tile (13000: 6); ragged tokens and columns
@pytest.mark.parametrize("M,kin,out", [(255, 264, 192), (1000, 264, 192), (2111, 768, 2304), (2144, 3072, 768), (1337, 776, 704), (2144, 768, 768),
                                       (6305, 776, 768), (13000, 1544, 768)])
def test_weight_gradients_are_sums_of_parts(env, M, kin, out):
    """Which tokens are summed together depends on the sizes alone, and the parts are added up in order: the same bits as the parts on
    their own, added up one after the other."""
    torch, P = env
    rng = np.random.default_rng(M + kin + out)
    x, dy, w = (K.to_dev(torch, K.bf16_np(rng, s), torch.bfloat16) for s in ((M, kin), (M, out), (kin, out)))
    ws = torch.full((16 * (kin + 1) * out,), float("nan"), device="cuda")
    _, dw, db = P.bsr_linear_backward(x, dy, w, workspace=ws)
    alone, _ = P.bsr_linear_wgrad(x, dy, workspace=ws)
    step = tokens_per_part(M, kin, out)
    parts = [P.bsr_linear_backward(x[i:i + step], dy[i:i + step], w)[1:] for i in range(0, M, step)]
    dw_ref, db_ref = parts[0]
    for p in parts[1:]:
        dw_ref, db_ref = dw_ref + p[0], db_ref + p[1]
    torch.cuda.synchronize()
    assert torch.equal(dw, dw_ref) and torch.equal(db, db_ref), "with the input gradient"
    assert torch.equal(alone, dw_ref), "on its own"


@pytest.mark.parametrize("tile", [96128, 128256, 192256, 256064, 96256, 3064128, 2192128, 2256128, 2128128])
def test_ids_that_are_no_longer_shapes_run_what_no_id_runs(env, tile):
    torch, P = env
    x, dy, w = (torch.zeros(s, dtype=torch.bfloat16, device="cuda") for s in ((1000, 768), (1000, 768), (768, 768)))
    default = product_kernels(lambda: P.bsr_linear_backward(x, dy, w))
    assert len(default) == 1 and product_kernels(lambda: P.bsr_linear_backward(x, dy, w, tile=tile)) == default
    default = product_kernels(lambda: P.bsr_linear_forward(x, w, None))
    assert product_kernels(lambda: P.bsr_linear_forward(x, w, None, tile=tile)) == default


@pytest.mark.parametrize("T", [1, 33, 64, 65, 128, 197, 256])
def test_attention_of_few_heads_is_the_same_bits(env, T):
    """24 heads (two workgroups share a head) against the same heads among 132 (one workgroup each)."""
    torch, P = env
    rng = np.random.default_rng(T)
    qkv = K.to_dev(torch, K.bf16_np(rng, (11, T, 3 * 12 * 64), 1.5), torch.bfloat16)
    many = P.bsr_attention_forward(qkv, 12)
    few = P.bsr_attention_forward(qkv[:2].contiguous(), 12)
    torch.cuda.synchronize()
    for name, a, b in zip(("out", "lse", "CLS row"), many, few):
        assert torch.equal(a[:2], b), name
