"""Backward of a token drop: the LayerNorm's gradient goes to the kept tokens' places, the dropped ones get zero (against the oracle)."""
import numpy as np
import pytest

import bsr_synth as S
from test_gpu_parity import TOL_BF16, TOL_FP32, hip  # noqa: F401  (hip is a fixture)

pytestmark = pytest.mark.gpu


# one token kept, all but one, a few: the first ones, the last ones, every other one; a block that is trained and one that only passes the gradient on.
# In bf16 the one block: every product rounds by 2^-9, and with one token kept the three blocks' dozen roundings in a row leave more than the
# 2 % that gradients are held to.
@pytest.mark.parametrize("dtype,tol,dim,depth", [("fp32", TOL_FP32, 64, 3), ("bf16", TOL_BF16, 768, 1)])
@pytest.mark.parametrize("kept", [[0], [15], list(range(15)), list(range(1, 16)), [0, 1, 2, 3], [12, 13, 14, 15], [1, 3, 5, 7, 9, 11, 13, 15]])
def test_gradient_goes_to_the_kept_places(hip, orc64, dtype, tol, dim, depth, kept):
    k, batch = len(kept), 3
    cfg = S.get_config("c1_block_fp32", dtype=dtype, dim=dim, heads=dim // 64, mlp_hidden=128, tokens_in=17, batch=batch, depth=depth,
                       drop_blocks=[depth // 2], first_trainable=0, keep_ratio=k / 16)
    if depth == 3 and k % 2:
        cfg["trainable_blocks"] = [0, 2]
    p = S.make_params(cfg, std=0.05)
    x, y = S.make_inputs(cfg)
    idx = [np.stack([np.asarray(kept, np.int32), np.asarray(kept[::-1], np.int32)[::-1], np.asarray(kept, np.int32)])]
    ref = orc64.step(cfg, p, x, y, forced_idx=idx)
    got = hip.run_hip_step(cfg, p, x, y, forced_idx=idx)
    assert got["keep_k"] == ref["keep_k"] == [k]
    for n, g in ref["grads"].items():
        assert hip.rel(got["grads"][n], g) < tol, n
