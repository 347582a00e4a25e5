"""Backward of a token drop: the LayerNorm's gradient goes to the kept tokens' places, the dropped ones get zero (against the oracle)."""
import numpy as np
import pytest

import bsr_synth as S
from test_gpu_parity import TOL_BF16, TOL_FP32, hip  # noqa: F401  (hip is a fixture)

pytestmark = pytest.mark.gpu

N = 16       # patch tokens before the drop


def ranked_inputs(cfg, wanted, seed=0):
    """Parameters and tokens with which the ranking itself keeps the tokens wanted[image]: queries and keys agree, and the wanted tokens
    resemble the class token where the others are its opposite."""
    p = S.make_params(cfg, std=0.05)
    D = cfg["dim"]
    for l in range(cfg["depth"]):
        w, b = p[f"blocks.{l}.w_qkv"], p[f"blocks.{l}.b_qkv"]
        w[:, :D] *= 8 / D ** 0.5                              # (scores of about +-1 at any width)
        w[:, D:2 * D] = w[:, :D]
        b[:2 * D] = 0
    x, y = S.make_inputs(cfg)
    rng = np.random.default_rng(seed)
    for image, kept in enumerate(wanted):
        toward = np.where(np.isin(np.arange(N), kept), 0.8, -0.8)[:, None]
        cls = rng.standard_normal(D)
        x[image, 0] = cls
        x[image, 1:] = toward * cls + 0.6 * rng.standard_normal((N, D))
    return p, x, y


def lists_of(kept):
    """a different list for each of three images: these, their mirror, as many others"""
    others = np.sort(np.random.default_rng(len(kept)).choice(N, len(kept), replace=False))
    return [np.asarray(v, np.int32) for v in (kept, sorted(N - 1 - i for i in kept), others)]


def config(dtype, dim, depth, k, batch=3):
    cfg = S.get_config("c1_block_fp32", dtype=dtype, dim=dim, heads=dim // 64, mlp_hidden=128, tokens_in=N + 1, batch=batch, depth=depth,
                       drop_blocks=[depth // 2], first_trainable=0, keep_ratio=k / N)
    if depth == 3 and k % 2:
        cfg["trainable_blocks"] = [0, 2]
    return cfg


# one token kept, all but one, a few: the first ones, the last ones, every other one; a block that is trained and one that only passes the gradient on.
# In bf16 the one block: every product rounds by 2^-9, and with one token kept the three blocks' dozen roundings in a row leave more than the
# 2 % that gradients are held to.
@pytest.mark.parametrize("dtype,tol,dim,depth", [("fp32", TOL_FP32, 64, 3), ("bf16", TOL_BF16, 768, 1)])
@pytest.mark.parametrize("kept", [[0], [15], list(range(15)), list(range(1, 16)), [0, 1, 2, 3], [12, 13, 14, 15], [1, 3, 5, 7, 9, 11, 13, 15]])
def test_gradient_goes_to_the_kept_places(hip, orc64, dtype, tol, dim, depth, kept):
    cfg, wanted = config(dtype, dim, depth, len(kept)), lists_of(kept)
    assert not np.array_equal(wanted[0], wanted[1])
    p, x, y = ranked_inputs(cfg, wanted)
    got = hip.run_hip_step(cfg, p, x, y)
    assert got["keep_k"] == [len(kept)] and np.array_equal(got["kept_idx"][0], np.stack(wanted))
    ref = orc64.step(cfg, p, x, y, forced_idx=[np.stack(wanted)])
    for n, g in ref["grads"].items():
        assert hip.rel(got["grads"][n], g) < tol, n


@pytest.mark.parametrize("dtype,dim,depth", [("fp32", 64, 3), ("bf16", 768, 1)])
def test_lists_of_the_caller(hip, dtype, dim, depth):
    """The ranked list handed back gives the bits of the ranking (its gradient takes another kernel to the same places), and with a list in
    any order, or with a token twice, every row of the gradient is written once: the same bits every time, whatever the buffers held before."""
    kept = [1, 3, 5, 7, 9, 11, 13, 15]
    cfg, wanted = config(dtype, dim, depth, len(kept)), lists_of(kept)
    p, x, y = ranked_inputs(cfg, wanted)
    free = hip.run_hip_step(cfg, p, x, y)
    ctx = free["ctx"]
    back = hip.run_hip_step(cfg, p, x, y, forced_idx=[np.stack(wanted)], ctx=ctx)
    assert all(np.array_equal(free["grads"][n], g) for n, g in back["grads"].items())
    rng = np.random.default_rng(1)
    for lists in (np.stack([v[::-1] for v in wanted]), np.stack([rng.permutation(v) for v in wanted]), rng.integers(0, N, (3, len(kept)))):
        seen = []
        for left in (0.0, 1e4):
            # other gradients left in the same workspace
            hip.run_hip_step(cfg, p, x + np.float32(left) * np.roll(x, 1, axis=1), y, ctx=ctx)
            seen.append(hip.run_hip_step(cfg, p, x, y, forced_idx=[lists], ctx=ctx)["grads"])
        assert all(np.isfinite(g).all() and np.array_equal(g, seen[1][n]) for n, g in seen[0].items())
