"""GPU parity of a layer's two gradients where the joint launch can go wrong: token counts around the k-tiles of the weight
gradient (64 tokens) and around its splits, both of its tiles, widths that end inside a tile, and scratch too small for the
splits.  And attention forward: a head by one workgroup or by two is the same bits."""
import numpy as np
import pytest

import test_gpu_kernels as K
from gpu_common import product_kernels
from test_gpu_kernels import env  # noqa: F401  (a fixture)

pytestmark = pytest.mark.gpu


# one token .. a few k-tiles; 8 .. 264 columns; splits with a ragged last one (788, 1000, 2111); the 256 x 128 tile (4416 and
# 6304 tokens at 768 x 3072)
@pytest.mark.parametrize("M,kin,out", [(1, 64, 8), (63, 192, 136), (64, 136, 264), (65, 264, 72), (191, 768, 64), (197, 768, 776),
                                       (788, 384, 1536), (1000, 264, 520), (2111, 768, 2304), (4416, 768, 3072), (6304, 3072, 768)])
def test_both_gradients_within_the_rounding_of_their_sums(env, M, kin, out):
    """Products of bf16 numbers are exact in fp32 and each of n additions errs by at most 2^-23 of what it adds up to, so an
    fp32 sum is within n 2^-23 of the sum of the terms' magnitudes; dX is then rounded to bf16 (2^-8 of its value)."""
    torch, P = env
    rng = np.random.default_rng(5 * M + kin + out)
    x, dy, w = (K.to_dev(torch, K.bf16_np(rng, s), torch.bfloat16) for s in ((M, kin), (M, out), (kin, out)))
    X, DY, W = x.double(), dy.double(), w.double()
    dx_ref, dw_ref, db_ref = DY @ W.t().contiguous(), X.t().contiguous() @ DY, DY.sum(0)
    dx_mag, dw_mag, db_mag = DY.abs() @ W.abs().t().contiguous(), X.abs().t().contiguous() @ DY.abs(), DY.abs().sum(0)
    per = (kin + 1) * out
    for floats in (0, 2 * per, 16 * per):                   # no room for a split, for two, for all
        ws = torch.full((floats,), float("nan"), device="cuda") if floats else None
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
