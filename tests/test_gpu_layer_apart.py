"""A layer's two gradients behind a GELU' at many rows: two launches, and the bits of the joint one."""
import pytest

from gpu_common import families, product_kernels
from test_gpu_kernels import env  # noqa: F401  (a fixture)

pytestmark = pytest.mark.gpu

APART, JOINT = ["tiled", "wgrad"], ["joint"]


# either side of the line, also where the rounds of tiles of one shape or another just end; weight matrices too small for it; without a GELU'
@pytest.mark.parametrize("rows,kin,out,gelu,kernels", [
    (11328, 3072, 768, True, JOINT), (12608, 3072, 768, True, JOINT), (13311, 3072, 768, True, JOINT), (13312, 3072, 768, True, APART),
    (14200, 3072, 768, True, APART), (16400, 3072, 768, True, APART), (17731, 3072, 768, True, APART), (17731, 3072, 768, False, JOINT),
    (19700, 3072, 768, True, APART), (13311, 1536, 384, True, JOINT), (13312, 1536, 384, True, APART), (20480, 1536, 384, True, APART),
    (20480, 384, 384, True, JOINT), (20480, 768, 192, True, JOINT)])
def test_gradients_behind_a_gelu_at_many_rows(env, rows, kin, out, gelu, kernels):
    torch, P = env
    g = torch.Generator(device="cuda").manual_seed(rows)
    rnd = lambda *s: torch.randn(s, generator=g, device="cuda").bfloat16()      # noqa: E731
    x, dy, w, u = rnd(rows, kin), rnd(rows, out), rnd(kin, out), rnd(rows, kin)
    ws = torch.empty(2 * (8 * kin * out + 16 * max(kin, out)), device="cuda")
    call = lambda tile=0: P.bsr_linear_backward(x, dy, w, u=u if gelu else None, workspace=ws, tile=tile)      # noqa: E731
    got, joint = call(), call(7128128)
    torch.cuda.synchronize()
    assert all(torch.equal(a, b) for a, b in zip(got, joint))
    assert families(n for n in product_kernels(call) if "gemm_" in n) == kernels
