"""GELU and its derivative as the bf16 products apply them, at every bf16 value, against 64 bits."""
import numpy as np
import pytest
import torch

import paper_2405_10951_amd as P

pytestmark = pytest.mark.gpu


def every_bf16():
    """[512, 128]: all bf16 values, infinities and NaN among them"""
    return torch.arange(65536, dtype=torch.int32).to(torch.int16).view(torch.bfloat16).view(512, 128)


def ulp(y):
    return 2.0 ** (np.floor(np.log2(np.maximum(np.abs(y), 2.0 ** -126))) - 7)


def check(got, want, x, slack):
    """Finite values: half a step of bf16 and what the fp32 arithmetic in front of the rounding may be off by; elsewhere what IEEE arithmetic gives."""
    fine = np.isfinite(x) & np.isfinite(want) & (np.abs(want) < 3.3e38)
    err = np.abs(got[fine] - want[fine])
    assert np.all(err <= 0.5 * ulp(want[fine]) * (1 + 1e-3) + slack), (x[fine][err.argmax()], err.max())
    assert np.all(np.isnan(got[np.isnan(x)]))


@pytest.mark.parametrize("tile", [0, 7192128, 7320256, 7256192, 256128])
def test_gelu_at_every_bf16_value(tile):
    """A unit product hands every finite value through unchanged; infinities and NaN, which would spread in it, come through the bias.
    The GELU is within 4.7e-7 of its value in 64 bits before it is rounded."""
    x = every_bf16()
    finite = torch.where(torch.isfinite(x.float()), x, torch.zeros_like(x))
    u = torch.empty((512, 128), dtype=torch.bfloat16, device="cuda")
    y, _ = P.bsr_linear_forward(finite.cuda(), torch.eye(128, dtype=torch.bfloat16, device="cuda"), None, act=1, u_out=u, tile=tile)
    assert torch.equal(u.cpu().view(torch.int16)[finite != 0], finite.view(torch.int16)[finite != 0])
    f = finite.float().double()
    want = (f * torch.special.ndtr(f)).numpy()
    check(y.float().cpu().numpy().astype(np.float64), want, finite.float().numpy(), 6e-7)
    bias = torch.tensor([float("inf"), float("-inf"), float("nan"), 1.0] * 32, device="cuda")
    z, _ = P.bsr_linear_forward(torch.zeros_like(finite).cuda(), torch.eye(128, dtype=torch.bfloat16, device="cuda"), bias, act=1, tile=tile)
    z = z.float().cpu()
    assert torch.all(torch.isposinf(z[:, 0::4])) and torch.all(torch.isnan(z[:, 1::4])) and torch.all(torch.isnan(z[:, 2::4]))


@pytest.mark.parametrize("tile", [0, 7192128, 7320256, 7256192, 256128])
def test_gelu_derivative_at_every_bf16_value(tile):
    """(within 2.9e-7 before the rounding)"""
    x = every_bf16()
    dx, _ = P.bsr_linear_dgrad(torch.ones((512, 128), dtype=torch.bfloat16, device="cuda"), torch.eye(128, dtype=torch.bfloat16, device="cuda"),
                               u=x.cuda(), tile=tile)
    f = x.float().double()
    want = (torch.special.ndtr(f) + f * torch.exp(-0.5 * f * f) * (2 * np.pi) ** -0.5).numpy()
    check(dx.float().cpu().numpy().astype(np.float64), want, x.float().numpy(), 4e-7)
