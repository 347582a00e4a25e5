"""GPU parity of the row-wise kernels (selection, LayerNorm, head) at the edges of their ranges, against the oracle."""
import numpy as np
import pytest

import bsr_synth as S
from test_gpu_parity import TOL_BF16, TOL_FP32, check_step, hip  # noqa: F401  (hip is a fixture)

pytestmark = pytest.mark.gpu


# one score; a wavefront's worth and one more or less; the largest; nothing, one, all but one and everything kept
@pytest.mark.parametrize("n", [1, 63, 64, 65, 196, 577, 1023])
def test_selection_at_the_edges(hip, orc32, n):
    import torch
    import paper_2405_10951_amd as P
    cfg = S.get_config("c1_block_fp32", dim=64, heads=1)
    ctx = P.Context(cfg, S.make_params(cfg), 3)
    rng = np.random.default_rng(n)
    sc = rng.standard_normal((3, n)).astype(np.float32)
    sc[1] = np.round(sc[1])                                   # many ties
    sc[2, ::3] = 0.0                                          # -0 and +0 are one value
    sc[2, 1::3] = -0.0
    x = rng.standard_normal((3, n + 1, 64)).astype(np.float32)
    for k in sorted({0, 1, n // 2, n - 1, n}):
        idx, out = ctx.bsr_select_tokens(torch.as_tensor(sc).cuda(), torch.as_tensor(x).cuda(), k)
        torch.cuda.synchronize()
        for b in range(3):
            ref = orc32.topk(sc[b], k)
            assert np.array_equal(idx[b].cpu().numpy(), ref), (k, b)
            assert np.array_equal(out[b].cpu().numpy(), x[b][np.concatenate([[0], 1 + ref]).astype(int)]), (k, b)


# rows of 1 .. 8 sixteen-byte pieces per lane (2048: the longest a wavefront holds, 2056: past it), the dropped tokens
# fused; head: odd class counts, more classes than threads, one class per load and four
@pytest.mark.parametrize("dtype,tol", [("fp32", TOL_FP32), ("bf16", TOL_BF16)])
@pytest.mark.parametrize("dim,heads,classes,fuse", [(128, 2, 37, 1), (1032, 6, 101, 1), (2048, 8, 3, 1), (2056, 257, 6, 1),
                                                    (128, 2, 1100, 0), (128, 2, 1201, 0)])
def test_long_rows_and_odd_heads(hip, orc64, dtype, tol, dim, heads, classes, fuse):
    cfg = S.get_config("mini_4blk", dtype=dtype, dim=dim, heads=heads, mlp_hidden=128, depth=2, drop_blocks=[1], first_trainable=1,
                       num_classes=classes, batch=2, fuse_dropped=fuse)
    p = S.make_params(cfg, std=0.05 if dim < 1000 else 0.02)
    x, y = S.make_inputs(cfg)
    check_step(hip, orc64, cfg, p, x, y, tol, free_running=False)


# heads at the edges of their kernels: one class short of a wide head and the first (groups of four, and single classes),
# classes that do and do not fill the wavefronts' walk; the last that fit their LDS and the first that do not; the last under
# 300000 weights and the first that go to the general products, with and without groups of four; 41 images, from where
# single classes stay here while they fit
@pytest.mark.parametrize("dtype,tol", [("fp32", TOL_FP32), ("bf16", TOL_BF16)])
@pytest.mark.parametrize("dim,classes,batch", [(128, 127, 2), (128, 128, 2), (128, 129, 3), (128, 508, 2), (128, 512, 2), (128, 772, 1),
                                               (128, 1301, 2), (128, 1788, 2), (128, 1792, 2), (128, 1789, 2), (128, 1791, 2), (256, 1168, 2),
                                               (256, 1172, 2), (256, 1171, 2), (256, 1173, 40), (256, 1173, 41)])
def test_heads_of_many_classes(hip, orc64, dtype, tol, dim, classes, batch):
    cfg = S.get_config("mini_4blk", dtype=dtype, dim=dim, num_classes=classes, batch=batch)
    p = S.make_params(cfg, std=0.05)
    x, y = S.make_inputs(cfg)
    ref = orc64.step(cfg, p, x, y)
    got = hip.run_hip_step(cfg, p, x, y, forced_idx=ref["kept_idx"])
    assert abs(got["loss"] - ref["loss"]) <= tol * abs(ref["loss"])
    assert hip.rel(got["logits"], ref["logits"]) < tol
    for n, g in ref["grads"].items():
        assert hip.rel(got["grads"][n], g) < tol, n


# the largest count that takes two bits a step, one less and the first that takes one
@pytest.mark.parametrize("n", [255, 256, 257])
def test_selection_where_its_two_forms_meet(hip, orc32, n):
    test_selection_at_the_edges(hip, orc32, n)
