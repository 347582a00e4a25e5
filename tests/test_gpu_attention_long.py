"""GPU parity of the attention kernels beyond 256 tokens, at the edges of their chunks, against the oracle."""
import numpy as np
import pytest

from test_gpu_kernels import assert_close, bf16_np, env, to_dev  # noqa: F401  (env is a fixture)

pytestmark = pytest.mark.gpu


# 257: one key past the short kernel; 384 / 385: whole chunks and one row more; 577, 785: ragged; 1024: the limit
@pytest.mark.parametrize("B,T,H", [(2, 257, 2), (1, 384, 1), (1, 385, 2), (2, 577, 3), (1, 785, 1), (1, 1024, 1)])
def test_attention_beyond_256_tokens(env, orc64, B, T, H):
    torch, P = env
    rng = np.random.default_rng(T)
    # unit-variance q, k, v as in the test of the short backward kernels, whose bounds these are
    qkv = bf16_np(rng, (B, T, 3 * H * 64), 1.0)
    dout = bf16_np(rng, (B, T, H * 64), 1.0)
    qt = to_dev(torch, qkv, torch.bfloat16)
    out, lse, cls, used = P.bsr_attention_forward(qt, H)
    dqkv, used_bwd = P.bsr_attention_backward(qt, out, to_dev(torch, dout, torch.bfloat16), lse, H)
    torch.cuda.synchronize()
    assert used == 1 and used_bwd == 1
    Pm, o = orc64.attention(qkv, H)
    assert_close(out.float().cpu().numpy(), o, "attention output")                  # bounds: as up to 256 tokens
    assert_close(cls.cpu().numpy(), Pm[:, :, 0, :], "CLS softmax row", tol=2e-3)
    ref = orc64.attention_bwd(qkv, Pm, dout, H)
    got, D = dqkv.float().cpu().numpy(), H * 64
    for name, sl in (("dq", slice(0, D)), ("dk", slice(D, 2 * D)), ("dv", slice(2 * D, 3 * D))):
        assert_close(got[..., sl], ref[..., sl], name, tol=1.5e-2)


# In fp32 from the scores to the sums: what comes out is the exact value rounded to bf16, no further off (in rms) than that
# rounding by more than 1 in 50.  (With probabilities, score gradients or dO . O in bf16 dq and dk are 1.4 to 2.6 times as far.)
@pytest.mark.parametrize("B,T,H,std", [(2, 257, 2, 1.0), (1, 385, 2, 1.5), (2, 400, 3, 2.5), (1, 785, 1, 1.5), (1, 1024, 1, 1.5)])
def test_attention_beyond_256_tokens_rounds_only_its_results(env, orc64, B, T, H, std):
    torch, P = env
    rng = np.random.default_rng(T + 1)
    qkv, dout = bf16_np(rng, (B, T, 3 * H * 64), std), bf16_np(rng, (B, T, H * 64), 1.0)
    qt = to_dev(torch, qkv, torch.bfloat16)
    out, lse, _, _ = P.bsr_attention_forward(qt, H)
    dqkv, _ = P.bsr_attention_backward(qt, out, to_dev(torch, dout, torch.bfloat16), lse, H)
    torch.cuda.synchronize()
    Pm, o = orc64.attention(qkv, H)
    ref, got, D = orc64.attention_bwd(qkv, Pm, dout, H), dqkv.float().cpu().numpy(), H * 64
    rms = lambda a: float(np.sqrt(np.mean(np.square(a, dtype=np.float64))))      # noqa: E731
    for name, a, r in (("output", out.float().cpu().numpy(), o), ("dq", got[..., :D], ref[..., :D]), ("dk", got[..., D:2 * D], ref[..., D:2 * D]),
                       ("dv", got[..., 2 * D:], ref[..., 2 * D:])):
        rounding = rms(torch.from_numpy(np.ascontiguousarray(r, np.float32)).bfloat16().float().numpy() - r)
        assert rms(a - r) <= 1.02 * rounding, f"{name}: {rms(a - r) / rounding:.3f} of the rounding"
