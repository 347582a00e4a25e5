"""The last block on its class rows alone (what the head reads): loss, logits and every gradient against the oracle, and
the same bits whether or not the block's whole output (or the routing of all its tokens) is asked for."""
import numpy as np
import pytest

import bsr_synth as S
from test_gpu_parity import TOL_BF16, TOL_FP32, hip  # noqa: F401  (hip is a fixture)

pytestmark = pytest.mark.gpu

# several blocks trained; only the last one; the last one frozen in the gradient path; one image; a head size of 16
# (fewer pieces per row than lanes on it); experts in the last block
CASES = [("mini_4blk", dict()), ("mini_4blk", dict(first_trainable=3)), ("mini_interleaved", dict(trainable_blocks=[1, 3])),
         ("mini_4blk", dict(batch=1, drop_blocks=[1], keep_k=[63])), ("mini_4blk", dict(heads=8)), ("mini_moe", dict(batch=16))]


@pytest.mark.parametrize("dtype,tol", [("fp32", TOL_FP32), ("bf16", TOL_BF16)])
@pytest.mark.parametrize("name,over", CASES, ids=lambda v: v if isinstance(v, str) else "-".join(map(str, v)) or "plain")
def test_last_block_on_class_rows(hip, orc64, name, over, dtype, tol):
    import torch
    if name == "mini_moe" and dtype == "fp32":
        pytest.skip("mixtures of experts exist in bf16 only")
    cfg = S.get_config(name, dtype=dtype, **over)
    p = S.make_params(cfg, std=0.05)
    x, y = S.make_inputs(cfg)
    ref = orc64.step(cfg, p, x, y)
    forced = ref.get("experts") if name == "mini_moe" else None
    full = hip.run_hip_step(cfg, p, x, y, forced_idx=ref["kept_idx"], forced_experts=forced)
    ctx, dev, B = full["ctx"], torch.device("cuda:0"), x.shape[0]
    if forced:
        fex = torch.as_tensor(np.concatenate([np.asarray(forced[l], np.int32).reshape(-1) for l in sorted(forced)]), dtype=torch.int32)
        ctx.bsr_moe_routing_io(fex.to(dev))
    cat = lambda which: (torch.as_tensor(np.concatenate([np.asarray(ref["kept_idx"][i], np.int32).reshape(-1) for i in which]),  # noqa: E731
                                         dtype=torch.int32).to(dev) if which else None)
    xf = ctx.bsr_forward_frozen(torch.as_tensor(x).to(dev).to(ctx.act_dtype).contiguous(), forced_idx=cat(ctx.frozen_drops))
    grads = ctx.new_grads()
    logits = torch.zeros((B, cfg["num_classes"]), dtype=torch.float32, device=dev)
    loss = ctx.bsr_train_blocks_fwd_bwd(xf, torch.as_tensor(y, dtype=torch.int32).to(dev), grads, logits_out=logits,
                                        forced_idx=cat(ctx.train_drops))
    torch.cuda.synchronize()
    assert hip.rel(logits.cpu().numpy(), ref["logits"]) < tol
    for n, g in ref["grads"].items():
        bar = 2 * tol if n.endswith("w_router") else tol          # (the router matrix is measured, not held to the bar: see smoke())
        assert hip.rel(grads[n].cpu().numpy(), g) < bar, n
        assert np.array_equal(grads[n].cpu().numpy(), full["grads"][n]), n
    assert float(loss[0]) == full["loss"] and np.array_equal(logits.cpu().numpy(), full["logits"])


@pytest.mark.parametrize("T", [65, 300])
def test_class_attention_does_not_see_the_rounding_of_its_output(hip, orc64, T):
    """Values of 32 +- 1/4, which bf16 holds and their means it does not: with delta = dO . O of the stored output the gradients
    of queries are 7 to 9 % off, with delta = sum P dP as close as elsewhere."""
    cfg = S.get_config("mini_4blk", dtype="bf16", image_size=0, patch_size=0, in_chans=0, tokens_in=T, dim=64, heads=2, mlp_hidden=64, depth=1,
                       drop_blocks=[], first_trainable=0, batch=4)
    p = S.make_params(cfg, std=0.05)
    rng = np.random.default_rng(T)
    x = np.where(rng.random((4, T, 64)).argsort(2) < 32, 1.0, -1.0).astype(np.float32)      # LayerNorm leaves these as they are
    p["blocks.0.ln1_g"][:], p["blocks.0.ln1_b"][:] = 1.0, 0.0
    wv = p["blocks.0.w_qkv"][:, 128:]
    wv[:] = 0.0
    wv[rng.permutation(64), np.arange(64)] = 0.25
    p["blocks.0.b_qkv"][128:] = 32.0
    w = p["blocks.0.w_proj"]
    w[:] = S.round_to_bf16(w - w.mean(0))                     # the 32 does not reach the residual row
    y = rng.integers(0, cfg["num_classes"], 4).astype(np.int32)
    ref = orc64.step(cfg, p, x, y)
    got = hip.run_hip_step(cfg, p, x, y)
    for name, cols in (("q", slice(0, 64)), ("k", slice(64, 128))):
        g = ref["grads"]["blocks.0.w_qkv"][:, cols]
        assert hip.rel(got["grads"]["blocks.0.w_qkv"][:, cols], g) < TOL_BF16, name


@pytest.mark.parametrize("dtype", ["bf16", "fp32"])
def test_reported_class_rows_are_those_the_loss_came_from(hip, dtype):
    """Logits from the reported output of the last block: the head's own, up to the order of fp32 sums."""
    cfg = S.get_config("mini_4blk", dtype=dtype, batch=8, heads=2)
    p = S.make_params(cfg, std=0.05, peaky=4.0)
    x, y = S.make_inputs(cfg)
    got = hip.run_hip_step(cfg, p, x, y)
    z = got["x_final"][:, 0].astype(np.float64)
    z = (z - z.mean(1, keepdims=True)) / np.sqrt(z.var(1, keepdims=True) + 1e-6) * p["lnf_g"] + p["lnf_b"]
    assert hip.rel(got["logits"], z @ p["w_head"].astype(np.float64) + p["b_head"]) < 1e-5


def test_recorded_routing_replays_to_the_same_bits(hip):
    """Among 4096 class tokens some sit on a near-tie of their experts: what a free step reports and a step given that choice
    have equal loss and gradients."""
    cfg = S.get_config("mini_moe", batch=4096, image_size=32, moe_top_k=1)
    p = S.make_params(cfg, std=0.05, peaky=4.0)
    x, y = S.make_inputs(cfg)
    free = hip.run_hip_step(cfg, p, x, y)
    again = hip.run_hip_step(cfg, p, x, y, forced_experts=free["experts"])
    assert again["loss"] == free["loss"]
    for n, g in free["grads"].items():
        assert np.array_equal(again["grads"][n], g), n


def products_after_class_attention(torch, call):
    """Names of the product kernels of a step, in order, from the class rows' attention on"""
    from torch.profiler import ProfilerActivity, profile
    call()
    torch.cuda.synchronize()
    with profile(activities=[ProfilerActivity.CUDA]) as prof:
        call()
        torch.cuda.synchronize()
    runs = sorted((e for e in prof.events() if e.device_type == torch.autograd.DeviceType.CUDA), key=lambda e: e.time_range.start)
    names = [e.name for e in runs]
    first = next(i for i, n in enumerate(names) if "attn_cls_fwd" in n)
    return [n for n in names[first:] if "gemm_" in n]


def test_asking_for_the_output_keeps_the_tuned_shapes(hip):
    """The last block's whole output takes products of its own; the others keep their measured shapes and bits."""
    import torch
    cfg = S.get_config("c2_deit_s", dtype="bf16", batch=8)
    p = S.make_params(cfg)
    x, y = S.make_inputs(cfg)
    import paper_2405_10951_amd as P
    ctx, dev = P.Context(cfg, p, 8), torch.device("cuda:0")
    xin, lab = torch.as_tensor(x).to(dev).to(ctx.act_dtype).contiguous(), torch.as_tensor(y, dtype=torch.int32).to(dev)
    xf = torch.empty((8, ctx.T_f, cfg["dim"]), dtype=ctx.act_dtype, device=dev)
    xo = torch.empty((8, ctx.T_last, cfg["dim"]), dtype=ctx.act_dtype, device=dev)
    loss = torch.zeros(4, dtype=torch.float32, device=dev)
    ctx.bsr_forward_frozen(xin, x_out=xf)
    grads = [ctx.new_grads() for _ in range(3)]
    ctx.bsr_train_blocks_fwd_bwd(xf, lab, grads[0], loss_out=loss)
    ctx.bsr_autotune(xin, lab, xf, loss, grads[1])
    plain = products_after_class_attention(torch, lambda: ctx.bsr_train_blocks_fwd_bwd(xf, lab, grads[1], loss_out=loss))
    asked = products_after_class_attention(torch, lambda: ctx.bsr_train_blocks_fwd_bwd(xf, lab, grads[2], loss_out=loss, x_final_out=xo))
    assert len(plain) > 10 and plain == asked
    for n in grads[0]:                                         # tuned or not, asked or not: the same bits
        assert torch.equal(grads[0][n], grads[1][n]) and torch.equal(grads[0][n], grads[2][n]), n
