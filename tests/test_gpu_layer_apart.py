"""A layer's two gradients behind a GELU' at many rows: two launches, and the bits of the joint one."""
import pytest

from gpu_common import families, product_kernels
from test_gpu_kernels import env  # noqa: F401  (a fixture)

pytestmark = pytest.mark.gpu


# either side of the line (about 16000 rows of 768), and without a GELU' past it
@pytest.mark.parametrize("rows,gelu,kernels", [(12608, True, ["joint"]), (17731, True, ["tiled", "wgrad"]), (17731, False, ["joint"])])
def test_gradients_behind_a_gelu_at_many_rows(env, rows, gelu, kernels):
    torch, P = env
    g = torch.Generator(device="cuda").manual_seed(rows)
    rnd = lambda *s: torch.randn(s, generator=g, device="cuda").bfloat16()      # noqa: E731
    x, dy, w, u = rnd(rows, 3072), rnd(rows, 768), rnd(3072, 768), rnd(rows, 3072)
    ws = torch.empty(2 * (8 * 4 * 768 * 768 + 16 * 4 * 768), device="cuda")
    call = lambda tile=0: P.bsr_linear_backward(x, dy, w, u=u if gelu else None, workspace=ws, tile=tile)      # noqa: E731
    got, joint = call(), call(7128128)
    torch.cuda.synchronize()
    assert all(torch.equal(a, b) for a, b in zip(got, joint))
    assert families(n for n in product_kernels(call) if "gemm_" in n) == kernels
