"""The head's walk over its weights, whose first rows per thread stay in registers from the logits to the gradient: at the edges of
what is held and of a chunk of rows, against the oracle."""
import numpy as np
import pytest

import bsr_synth as S
from test_gpu_parity import TOL_BF16, TOL_FP32, hip  # noqa: F401  (hip is a fixture)

pytestmark = pytest.mark.gpu


# rows per thread = ceil(dim / (1024 / groups of classes)).  Four classes a load (400: ten rows at a time): 5, 6, 20 (all held), 21, 26;
# 8 classes (two groups, even pitch) and 32 (eight, odd pitch); one class a load (102): 7, 8, 42 (all held), 43, 50; one class, with
# fewer rows than threads and with more
@pytest.mark.parametrize("dtype,tol", [("fp32", TOL_FP32), ("bf16", TOL_BF16)])
@pytest.mark.parametrize("dim,classes", [(48, 400), (56, 400), (200, 400), (208, 400), (256, 400), (64, 102), (72, 102), (416, 102), (424, 102),
                                         (504, 102), (64, 8), (64, 32), (64, 1), (1032, 1)])
def test_head_at_the_edges_of_held_rows(hip, orc64, dtype, tol, dim, classes):  # noqa: F811
    cfg = S.get_config("mini_4blk", dtype=dtype, dim=dim, heads=dim // 8, mlp_hidden=64, depth=1, drop_blocks=[], first_trainable=0,
                       num_classes=classes, batch=3)
    p = S.make_params(cfg, std=0.05)
    x, y = S.make_inputs(cfg)
    ref = orc64.step(cfg, p, x, y)
    out = hip.run_hip_step(cfg, p, x, y, forced_idx=ref["kept_idx"])
    # z has unit variance and W_h 0.05: a logit is of order 0.05 sqrt(dim), and so is what the rounding of z is a share of, also where
    # the three logits of one class all come out small
    assert np.abs(out["logits"] - ref["logits"]).max() < tol * max(np.abs(ref["logits"]).max(), 0.05 * dim ** 0.5)
    assert abs(out["loss"] - ref["loss"]) <= tol * abs(ref["loss"])
    for n in ("w_head", "b_head", "lnf_g", "lnf_b", "blocks.0.w_fc2"):
        if classes > 1:                                   # (one class: every gradient is zero)
            assert hip.rel(out["grads"][n], ref["grads"][n]) < tol, n
        else:
            assert abs(out["grads"][n]).max() == 0.0, n


# rows per thread around the eight that are added up together: four classes (400) 8, 9, 16, 17; one class (102) 8, 9, 40 (all held), 41, 48, 49; sums of as many
# values as threads share, fewer and one more (7, 8, 9 groups; 8 and 9 rows at a time); the largest scratch with an odd pitch (8 groups, two chunks)
@pytest.mark.parametrize("dtype,tol", [("fp32", TOL_FP32), ("bf16", TOL_BF16)])
@pytest.mark.parametrize("dim,classes", [(80, 400), (88, 400), (160, 400), (168, 400), (80, 102), (88, 102), (400, 102), (408, 102), (480, 102),
                                         (488, 102), (768, 28), (256, 36), (80, 127), (80, 508), (128, 113), (1032, 32)])
def test_head_at_the_edges_of_a_sum(hip, orc64, dtype, tol, dim, classes):  # noqa: F811
    test_head_at_the_edges_of_held_rows(hip, orc64, dtype, tol, dim, classes)


def test_the_widest_rows_take_more_than_64_kb_of_lds(hip, orc64):  # noqa: F811
    test_head_at_the_edges_of_held_rows(hip, orc64, "bf16", TOL_BF16, 3904, 10)
