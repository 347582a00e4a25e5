"""Attention at lengths around the rows it stages and the blocks of 32 it leaves out, with whatever LDS held before (NaN) behind the last token, against the oracle."""
import numpy as np
import pytest

from test_gpu_kernels import assert_close, bf16_np, env, to_dev  # noqa: F401  (env is a fixture)

pytestmark = pytest.mark.gpu


def fill_lds_with_nan(torch, P, T):
    """A head of NaN for every CU, twice over: its keys and values stay in LDS behind the kernel."""
    P.bsr_attention_forward(torch.full((43, T, 3 * 12 * 64), float("nan"), dtype=torch.bfloat16, device="cuda"), 12)


# one row of tokens more or less than whole groups of 8 staged rows, blocks of 32 and halves of a head; 1 token: the least
@pytest.mark.parametrize("T", [1, 7, 8, 9, 32, 33, 96, 127, 128, 129, 159, 160, 161, 167, 168, 192, 193, 199, 200, 201, 223, 224, 225, 255, 256])
def test_attention_forward_reads_no_row_past_the_tokens(env, orc64, T):
    torch, P = env
    rng = np.random.default_rng(T)
    qkv = bf16_np(rng, (2, T, 3 * 3 * 64), 1.5)
    fill_lds_with_nan(torch, P, 256)
    out, lse, cls, used = P.bsr_attention_forward(to_dev(torch, qkv, torch.bfloat16), 3)
    torch.cuda.synchronize()
    assert used == 1
    Pm, o = orc64.attention(qkv, 3)
    assert_close(out.float().cpu().numpy(), o, "attention output")                   # bounds: those of test_attention_forward
    assert_close(cls.cpu().numpy(), Pm[:, :, 0, :], "CLS softmax row", tol=2e-3)
    assert bool(torch.isfinite(lse).all())


# A head in one workgroup: 132 heads, and 516 where no three halves fit a CU (200 and up; 193 and 199: halves on the other side of that line)
@pytest.mark.parametrize("T,images", [(T, 11) for T in (1, 31, 32, 33, 63, 64, 65, 95, 96, 97, 127, 128, 129, 138, 159, 160, 161, 192, 193, 199, 223, 224, 225, 255, 256)] +
                         [(T, 43) for T in (193, 199, 200, 207, 208, 215, 216, 223, 224)])
def test_attention_of_many_heads_reads_no_row_past_the_tokens(env, orc64, T, images):
    torch, P = env
    rng = np.random.default_rng(T)
    qkv = bf16_np(rng, (images, T, 3 * 12 * 64), 1.5)
    fill_lds_with_nan(torch, P, 256)
    out, lse, cls, used = P.bsr_attention_forward(to_dev(torch, qkv, torch.bfloat16), 12)
    torch.cuda.synchronize()
    assert used == 1
    some = [0, images - 1]
    Pm, o = orc64.attention(qkv[some], 12)
    assert_close(out[some].float().cpu().numpy(), o, "attention output")              # bounds: those of test_attention_forward
    assert_close(cls[some].cpu().numpy(), Pm[:, :, 0, :], "CLS softmax row", tol=2e-3)
    assert bool(torch.isfinite(out).all()) and bool(torch.isfinite(lse).all()) and bool(torch.isfinite(cls).all())


# 11 images: whole heads; 22 (264 heads): halves of 161 .. 224 tokens; 43: whole heads again from 200 tokens on
@pytest.mark.parametrize("T,images", [(T, 11) for T in (129, 138, 159, 160, 161, 192, 193, 224)] + [(T, 22) for T in (160, 161, 224)] + [(T, 43) for T in (199, 200, 208, 211, 224)])
def test_attention_of_a_few_heads_is_the_same_bits_as_among_many(env, T, images):
    """24 heads (two workgroups share a head) against the same heads among 132, 264 or 516."""
    torch, P = env
    rng = np.random.default_rng(T)
    qkv = to_dev(torch, bf16_np(rng, (images, T, 3 * 12 * 64), 1.5), torch.bfloat16)
    many = P.bsr_attention_forward(qkv, 12)
    few = P.bsr_attention_forward(qkv[:2].contiguous(), 12)
    torch.cuda.synchronize()
    for name, a, b in zip(("out", "lse", "CLS row"), many, few):
        assert torch.equal(a[:2], b), name


# 257, 385: one key into a chunk of 128; 288 / 289, 416 / 417: a block of 32 full and one key more; 1023: one short of the limit
@pytest.mark.parametrize("T", [257, 288, 289, 385, 416, 417, 512, 1023])
def test_long_attention_leaves_out_blocks_past_the_tokens(env, orc64, T):
    torch, P = env
    rng = np.random.default_rng(T)
    qkv, dout = bf16_np(rng, (1, T, 3 * 2 * 64), 1.0), bf16_np(rng, (1, T, 2 * 64), 1.0)
    fill_lds_with_nan(torch, P, 512)
    qt = to_dev(torch, qkv, torch.bfloat16)
    out, lse, cls, _ = P.bsr_attention_forward(qt, 2)
    dqkv, _ = P.bsr_attention_backward(qt, out, to_dev(torch, dout, torch.bfloat16), lse, 2)
    torch.cuda.synchronize()
    Pm, o = orc64.attention(qkv, 2)
    assert_close(out.float().cpu().numpy(), o, "attention output")
    assert_close(cls.cpu().numpy(), Pm[:, :, 0, :], "CLS softmax row", tol=2e-3)
    assert_close(dqkv.float().cpu().numpy(), orc64.attention_bwd(qkv, Pm, dout, 2), "dq, dk, dv", tol=1.5e-2)
