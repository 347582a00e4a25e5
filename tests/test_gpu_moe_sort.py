"""The rows of each expert where the sort's wavefronts hold more pairs than stay in registers between its two walks
(more than 16384 pairs, here ragged), and the sixteen wavefronts where most hold none (fewer pairs than wavefronts
times lanes): the step against the CPU oracle with the oracle's choice forced, and the choice itself bit for bit."""
import numpy as np
import pytest

import bsr_synth as S

pytestmark = pytest.mark.gpu

TOL = 2e-2      # bf16, max|gpu-ref| / max|ref| per tensor, as for the other mixture-of-experts steps


@pytest.fixture(scope="module")
def hip():
    import torch
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a HIP device")
    import gpu_common
    return gpu_common


@pytest.mark.parametrize("over", [dict(batch=131, moe_top_k=3, n_experts=5), dict(batch=200, moe_top_k=2),
                                  dict(batch=3, moe_top_k=1)])
def test_rows_of_each_expert(hip, orc64, over):
    cfg = S.get_config("mini_moe", dtype="bf16", **over)
    p = S.make_params(cfg, std=0.05, bf16_exact=True)
    x, y = S.make_inputs(cfg, bf16_exact=True)
    ref = orc64.step(cfg, p, x, y)
    got = hip.run_hip_step(cfg, p, x, y, forced_idx=ref["kept_idx"], forced_experts=ref["experts"])
    for l, e in ref["experts"].items():
        assert np.array_equal(got["experts"][l], e), f"forced experts of block {l} not used"
    assert hip.rel(got["x_trainable"], ref["x_trainable"]) < TOL
    assert hip.rel_rms(got["x_final"], ref["x_final"]) < TOL
    for l in cfg["moe_blocks"]:
        if l < cfg["first_trainable"]:
            continue
        for n in ("w_fc1", "w_fc2", "b_fc1", "b_fc2"):
            g, r = got["grads"][f"blocks.{l}.{n}"], ref["grads"][f"blocks.{l}.{n}"]
            for e in range(cfg["n_experts"]):
                assert np.abs(g[e] - r[e]).max() <= TOL * np.abs(r).max(), (l, n, e)
