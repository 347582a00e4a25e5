"""GPU parity of the products of few rows (wavefronts of a workgroup share k, rings of their own in LDS) at the edges of
their tiles and k-groups, and the tiled kernels' own edges at row counts that stay with them."""
import re

import numpy as np
import pytest

import test_gpu_kernels as K
from gpu_common import families, product_kernels
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


# The two families add over k in different orders, so the line between them is part of the results.  Products of a step (768 wide: class
# rows, half the tokens of 27 images; 384 wide) and ragged ones, on either side; a layer's two gradients likewise
@pytest.mark.parametrize("M,kin,out,kernel", [(128, 768, 3072, "few"), (300, 448, 392, "few"), (729, 3072, 768, "few"), (702, 768, 768, "tiled"),
                                              (729, 768, 768, "tiled"), (1300, 448, 584, "tiled"), (65, 192, 576, "tiled")])
def test_which_kernel_multiplies(env, M, kin, out, kernel):
    torch, P = env
    x, w = (torch.zeros(s, dtype=torch.bfloat16, device="cuda") for s in ((M, kin), (out, kin)))
    assert families(product_kernels(lambda: P.bsr_linear_forward(x, w, None))) == [kernel]


@pytest.mark.parametrize("M,kin,out,kernels", [(32, 768, 768, ["joint"]), (128, 768, 768, ["joint"]), (129, 3072, 768, ["joint"]), (67, 1536, 384, ["joint"]),
                                               (32, 768, 3072, ["few", "wgrad"]), (128, 768, 3072, ["few", "wgrad"])])
def test_which_kernel_takes_the_gradients_of_a_layer(env, M, kin, out, kernels):
    torch, P = env
    x, dy, w = (torch.zeros(s, dtype=torch.bfloat16, device="cuda") for s in ((M, kin), (M, out), (kin, out)))
    assert families(product_kernels(lambda: P.bsr_linear_backward(x, dy, w))) == kernels


# row counts that stay with the tiled kernels whatever the tile shape (of the sizes that test has, 300 x 448 x 392 and
# 333 x 1536 x 264 are products of few rows): the same bits from every shape, ragged edges, 1 .. 24 k-tiles
@pytest.mark.parametrize("M,kin,out", [(2200, 64, 1544), (2300, 320, 1160), (1300, 448, 584), (2050, 832, 2312), (1650, 1536, 1160)])
def test_every_tile_shape_at_larger_row_counts(env, orc64, M, kin, out):
    K.test_every_tile_shape_gives_the_same_bits(env, orc64, M, kin, out)


# a layer's two gradients together, at rows where a product on its own takes the kernel for few rows and one that can carry
# the weight gradient does not (768 x 768 up to 128 and at 321 .. 672 rows, 768 from 2304 at 673 .. 1024, 3072 from 768 at 65 .. 160,
# 384 x 384 up to 1344, 1536 from 384 up to 320), and where both take it: no tile changes a bit
@pytest.mark.parametrize("M,kin,out", [(32, 768, 768), (128, 768, 768), (400, 768, 768), (1000, 768, 2304), (129, 3072, 768), (536, 384, 384),
                                       (1343, 384, 384), (67, 1536, 384), (32, 768, 3072)])
def test_no_tile_changes_the_gradients_of_a_layer(env, orc64, M, kin, out):
    torch, P = env
    rng = np.random.default_rng(M + kin + out)
    dev = lambda a: K.to_dev(torch, a, torch.bfloat16)      # noqa: E731
    x, dy, u = K.bf16_np(rng, (M, kin)), K.bf16_np(rng, (M, out)), K.bf16_np(rng, (M, kin))
    w = K.bf16_np(rng, (kin, out), 0.05)
    xt, dyt, wt, ut = dev(x), dev(dy), dev(w), dev(u)

    ws = torch.full((16 * (kin + 1) * out,), float("nan"), device="cuda")

    def run(tile):
        got = P.bsr_linear_backward(xt, dyt, wt, u=ut, workspace=ws, tile=tile)
        torch.cuda.synchronize()
        return [t.float().cpu().numpy() for t in got]

    assert families(product_kernels(lambda: run(0))) == (["few", "wgrad"] if (M, out) == (32, 3072) else ["joint"])
    if (M, out) != (32, 3072):
        assert families(product_kernels(lambda: P.bsr_linear_dgrad(dyt, wt))) == ["few"]
    base = run(0)
    K.assert_close(base[0], orc64.gelu_bwd(orc64.linear_dgrad(dy, w), u), "dx")
    dw, db = orc64.linear_wgrad(x, dy)
    K.assert_close(base[1], dw, "dw")
    K.assert_close(base[2], db, "db")
    for tile in P.bsr_gemm_tile_shapes():
        for name, a, c in zip(("dx", "dw", "db"), base, run(tile)):
            assert np.array_equal(a, c), f"tile shape {tile}, {name}: {int(np.sum(a != c))} of {a.size} elements differ"


# an operand of more than 2^32 elements (8.6 GB): columns for the kernel for few rows, for the direct-to-LDS kernels, and a
# weight matrix of that size; only its last rows, beyond the 32-bit offsets, are not zero
@pytest.mark.parametrize("M,kin,out", [(1048600, 4096, 8), (1048600, 4096, 256), (320, 4096, 1048600)])
def test_operands_of_more_than_2_32_elements(env, M, kin, out):
    torch, P = env
    rng = np.random.default_rng(M + out)
    big, small = max(M, out), min(M, out)
    a = torch.zeros((big, kin), dtype=torch.bfloat16, device="cuda")
    tail, b = K.bf16_np(rng, (64, kin)), K.bf16_np(rng, (small, kin), 0.05)
    a[-64:] = K.to_dev(torch, tail, torch.bfloat16)
    bt = K.to_dev(torch, b, torch.bfloat16)
    y, used = P.bsr_linear_forward(*((a, bt) if M > out else (bt, a)), None)
    torch.cuda.synchronize()
    assert used == 1
    if M < out:
        y = y.T
    K.assert_close(y[-64:].float().cpu().numpy(), tail.astype(np.float64) @ b.astype(np.float64).T, "last rows")
    assert not bool(y[:-64].any())


def test_tuning_reports_what_products_of_few_rows_run(env):
    """They run one kernel whatever is asked for: no shape is listed for them and none counts as changed."""
    import bsr_synth as S
    torch, P = env
    cfg = S.get_config("c2_deit_s", dtype="bf16", batch=4)
    x, y = S.make_inputs(cfg)
    ctx = P.Context(cfg, S.make_params(cfg), 4)
    xf = torch.empty((4, ctx.T_f, cfg["dim"]), dtype=ctx.act_dtype, device="cuda")
    launches, changed = ctx.bsr_autotune(torch.as_tensor(x).cuda().to(ctx.act_dtype).contiguous(), torch.as_tensor(y, dtype=torch.int32).cuda(), xf,
                                         torch.zeros(1, device="cuda"), ctx.new_grads())
    picks = ctx.bsr_tile_choices(0) + ctx.bsr_tile_choices(1)
    few = [t for t in picks if t[3] >= 9000000]
    assert len(picks) == launches and 0 < len(few) < launches and changed <= launches - len(few)
    assert {t[3] for t in few} <= {9032032, 9064032, 9064064} and all(t[4] > 0 for t in few)
    assert {t[3] for t in picks} - {t[3] for t in few} <= set(P.bsr_gemm_tile_shapes())


def shape_id(name):
    """Shape id of a product kernel's instance, from its name; None for kernels that have none"""
    kind, args = re.match(r".*?(gemm_\w+)<([^>]*)>", name).groups() if "<" in name else ("", "")
    v = [{"true": 1, "false": 0}.get(a.strip(), a.strip()) for a in args.split(",")]
    if kind == "gemm_nt_few_kernel":
        return 9000000 + 32000 * int(v[0]) + 32 * int(v[1])
    if kind == "gemm_pair_kernel":
        return (7128064, 7128128, 7192128, 7256128)[int(v[0])]
    if kind == "gemm_ntd_kernel":
        deep = (v[0], v[1], v[4]) in (("192", "128", "3"), ("128", "128", "3"))
        return (8000000 if deep else 7000000) + 1000 * int(v[0]) + int(v[1])
    if kind == "gemm_nt_kernel":
        return (1000000 * int(v[5]) if int(v[5]) > 1 else 0) + 1000 * int(v[0]) + int(v[1])
    return None


@pytest.mark.parametrize("fold", [False, True])
@pytest.mark.parametrize("two_streams", [False, True])
def test_tuning_reports_the_shapes_that_run(env, two_streams, fold):
    """Several ids name one kernel in a backward launch, and some shapes cannot take some products: what is reported is what
    runs, and compared with the model's choice as such."""
    import bsr_synth as S
    torch, P = env
    cfg = S.get_config("c2_deit_s", dtype="bf16", batch=16, fold_frozen_layernorm=int(fold))
    x, y = S.make_inputs(cfg)
    ctx = P.Context(cfg, S.make_params(cfg), 16)
    xin, lab = torch.as_tensor(x).cuda().to(ctx.act_dtype).contiguous(), torch.as_tensor(y, dtype=torch.int32).cuda()
    xf, xs = (torch.empty((16, ctx.T_f, cfg["dim"]), dtype=ctx.act_dtype, device="cuda") for _ in range(2))
    loss, grads = torch.zeros(4, device="cuda"), ctx.new_grads()

    def step():
        ctx.bsr_forward_frozen(xin, x_out=xf)
        ctx.bsr_train_blocks_fwd_bwd(xf, lab, grads, loss_out=loss)

    model = [i for i in map(shape_id, product_kernels(step)) if i]
    if two_streams:
        frozen, train = torch.cuda.Stream(), torch.cuda.Stream()
        torch.cuda.synchronize()
        with torch.cuda.stream(frozen):
            launches, changed = ctx.bsr_autotune_overlapped(xin, lab, xf, xs, loss, grads, train)
        torch.cuda.synchronize()
    else:
        launches, changed = ctx.bsr_autotune(xin, lab, xf, loss, grads)
    reported = [t[3] for t in ctx.bsr_tile_choices(0) + ctx.bsr_tile_choices(1)]
    ran = [i for i in map(shape_id, product_kernels(step)) if i]
    assert len(ran) == launches and reported == ran
    assert changed == sum(a != b for a, b in zip(model, ran))
