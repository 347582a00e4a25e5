"""CPU-only checks of the C ABI: the built library loads, exports every function include/bsr.h
declares, and its host-only entry points (token schedule, workspace size, configuration checks)
behave as documented.  Nothing here launches a kernel."""
import ctypes as C
import os
import re

import pytest

import bsr_synth as S
import paper_2405_10951_amd as P
from oracle import token_schedule

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def declared_functions():
    text = open(os.path.join(ROOT, "include", "bsr.h")).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    return sorted(set(re.findall(r"\b(bsr_[a-z_0-9]+)\s*\(", text)))


def test_library_exports_every_declared_symbol():
    lib = P.load_library()
    names = declared_functions()
    assert {"bsr_init", "bsr_forward_frozen", "bsr_select_tokens", "bsr_train_blocks_fwd_bwd",
            "bsr_sgd_step"} <= set(names)
    for n in names:
        assert hasattr(lib, n), f"{n} is declared in include/bsr.h but not exported"


def test_python_binding_has_the_entry_points_names():
    for n in ("bsr_forward_frozen", "bsr_select_tokens", "bsr_train_blocks_fwd_bwd", "bsr_sgd_step",
              "bsr_refresh_weights", "bsr_profile_begin", "bsr_profile_end", "bsr_destroy"):
        assert hasattr(P.Context, n)
    for n in ("bsr_token_schedule", "bsr_workspace_bytes", "bsr_linear_forward", "bsr_linear_dgrad", "bsr_ln_linear_fold",
              "bsr_ln_linear_forward", "bsr_gemm_tile_shapes",
              "bsr_linear_wgrad", "bsr_attention_forward", "bsr_attention_backward"):
        assert hasattr(P, n)


@pytest.mark.parametrize("name,keep,expect", [("c3_vit_b", 0.7, [137, 95, 66]), ("c3_vit_b", 0.5, [98, 49, 24]),
                                              ("c3_vit_b", 1.0, [196, 196, 196]), ("c1_block_fp32", 0.7, [44])])
def test_token_schedule_matches_the_paper_and_the_oracle(name, keep, expect):
    cfg = S.get_config(name, keep_ratio=keep)
    kk, ta, tm = P.bsr_token_schedule(P.make_config(cfg, 4))
    assert kk == expect                                   # N/2, N/4, N/8 at drop rate 0.5 (Sec. 4.3)
    n0 = S.tokens_at_input(cfg) - 1
    assert kk == token_schedule(n0, keep, len(cfg["drop_blocks"]))
    for i, blk in enumerate(cfg["drop_blocks"]):
        assert tm[blk] == kk[i] + 1 and ta[blk] == (n0 + 1 if i == 0 else kk[i - 1] + 1)


def test_explicit_keep_k_wins_over_the_ratio():
    cfg = S.get_config("c2_deit_s", keep_k=[12, 8, 4])
    kk, _, tm = P.bsr_token_schedule(P.make_config(cfg, 2))
    assert kk == [12, 8, 4] and tm[-1] == 5


def test_workspace_grows_with_batch_and_trainable_blocks():
    cfg = S.get_config("c3_vit_b")
    a = P.bsr_workspace_bytes(P.make_config(cfg, 32))
    b = P.bsr_workspace_bytes(P.make_config(cfg, 64))
    c = P.bsr_workspace_bytes(P.make_config(dict(cfg, first_trainable=0), 32))
    assert 0 < a < b and a < c


@pytest.mark.parametrize("bad", [dict(dim=770), dict(heads=5), dict(depth=17), dict(drop_blocks=[6, 3, 9]),
                                 dict(drop_blocks=[3, 6, 12]), dict(keep_ratio=0.0), dict(keep_ratio=1.5),
                                 dict(first_trainable=13), dict(loss=S.LOSS_MEAN_SQ), dict(num_classes=0),
                                 dict(image_size=225), dict(keep_k=[300, 10, 5]), dict(mlp_hidden=3071)])
def test_bad_configurations_are_rejected_with_a_message(bad):
    cfg = S.get_config("c3_vit_b", **bad)
    with pytest.raises(P.BsrError) as e:
        P.bsr_workspace_bytes(P.make_config(cfg, 8))
    assert e.value.code == -2 and len(str(e.value)) > 20


def test_max_batch_must_be_positive_and_null_arguments_fail():
    cfg = S.get_config("c3_vit_b")
    with pytest.raises(P.BsrError):
        P.bsr_workspace_bytes(P.make_config(cfg, 0))
    lib = P.load_library()
    assert lib.bsr_workspace_bytes(None, None) == -1
    assert lib.bsr_token_schedule(None, None, None, None) == -1
    assert lib.bsr_destroy(None) == 0
    assert lib.bsr_last_error(None) is not None


def test_step_flop_count_matches_the_closed_form():
    # product-side counter used by the benchmark against the oracle-side MAC count (Table 4's 2249 GMacs)
    from paper_2405_10951_amd.flops import step_flops
    from oracle import accounting as acc
    tb = acc.tokens_per_block(197, 12, [], [])
    macs = acc.forward_macs(tb, 768, 3072, 196, 768, 100)
    fl = step_flops(768, 3072, 100, 768, 196, [197] * 12, [197] * 12, 12, 1)
    assert abs((fl["fwd_gemm"] + fl["fwd_attn"] + fl["head"] / 3) / (2 * macs) - 1) < 1e-9
    c3 = step_flops(768, 3072, 100, 768, 196, [197, 197, 197, 197, 138, 138, 138, 96, 96, 96, 67, 67],
                    [197, 197, 197, 138, 138, 138, 96, 96, 96, 67, 67, 67], 8, 32)
    assert abs(c3["total"] / 1e9 - 1012.8) < 0.5


# ---------------------------------------------------------------- saved-activation byte report (host only)

def _deit_s(**over):
    return dict(S.get_config("c2_deit_s", dtype="fp32", keep_ratio=1.0, drop_blocks=[], first_trainable=0), **over)


def test_saved_bytes_match_table_1_categories():
    # Table 1: DeiT-S, one image, fp32, 197 tokens: Q,K,V 0.87 MB, softmax input 0.89 MB, GELU input 1.15 MB
    from oracle import accounting as acc
    per, tot = P.bsr_saved_activation_bytes(P.make_config(_deit_s(), 4), 1)
    nl = acc.saved_bytes_nonlinear(T=197, D=384, H=6, F=1536)
    MB = 2.0 ** 20
    for r in per:
        assert r["qkv"] == nl["qkv"] and abs(r["qkv"] / MB - 0.87) < 0.005
        assert r["gelu_in"] == nl["gelu_in"] and abs(r["gelu_in"] / MB - 1.15) < 0.005
        # one log-sum-exp per row stands in for the row itself
        assert r["softmax"] * 197 == nl["softmax_in"] and abs(r["softmax"] * 197 / MB - 0.89) < 0.005
        # a trained block stays below the paper's 5.5 MB (it keeps no [H,T,T] tensor)
        assert r["total"] < acc.saved_bytes_trainable(197, 384, 6, 1536) and r["total"] / MB < 5.5
        assert r == dict(acc.saved_bytes_lse_design(197, 197, 384, 6, 1536, 4, trained=True, drop=False), moe=0)
    assert tot["total"] == sum(r["total"] for r in per) == 12 * per[0]["total"]


def test_saved_bytes_follow_the_token_schedule_and_the_trainable_set():
    from oracle import accounting as acc
    cfg = S.get_config("c6_vit_b_interleaved")          # bf16, trainable {3,7,11}, drops {3,6,9} at 0.5
    c = P.make_config(cfg, 8)
    _, ta, tm = P.bsr_token_schedule(c)
    per, tot = P.bsr_saved_activation_bytes(c, 1)
    for l, r in enumerate(per):
        if l < 3:
            assert all(v == 0 for v in r.values()), l    # the frozen prefix stores nothing
            continue
        want = acc.saved_bytes_lse_design(ta[l], tm[l], 768, 12, 3072, 2, trained=l in (3, 7, 11),
                                          drop=l in (3, 6, 9))
        assert r == dict(want, moe=0), l
    assert per[4]["linear_in"] == 0 and per[7]["linear_in"] > 0
    # frozen in the gradient path: below Table 1's three tensors at the same token count, fp32
    cfg32 = _deit_s(trainable_blocks=[11], first_trainable=0)
    per32, _ = P.bsr_saved_activation_bytes(P.make_config(cfg32, 2), 1)
    assert per32[5]["total"] <= sum(acc.saved_bytes_nonlinear(197, 384, 6, 1536).values())
    assert per32[5]["total"] < per32[11]["total"]


def test_saved_bytes_scale_with_batch_dtype_and_fit_the_workspace():
    cfg = S.get_config("c3_vit_b")
    c = P.make_config(cfg, 32)
    p1, t1 = P.bsr_saved_activation_bytes(c, 1)
    p32, t32 = P.bsr_saved_activation_bytes(c, 32)
    assert all(t32[k] == 32 * t1[k] for k in t1)
    assert 0 < t32["total"] < P.bsr_workspace_bytes(c)
    _, t1f = P.bsr_saved_activation_bytes(P.make_config(dict(cfg, dtype="fp32"), 32), 1)
    for k in ("qkv", "attn_out", "gelu_in", "linear_in", "residual"):
        assert t1f[k] == 2 * t1[k], k
    assert t1f["softmax"] == t1["softmax"] and t1f["stats"] == t1["stats"]
    # token dropping shrinks what the trained suffix keeps (Sec. 4.3 Discussion 2)
    _, full = P.bsr_saved_activation_bytes(P.make_config(dict(cfg, keep_ratio=1.0), 32), 1)
    assert t1["total"] < 0.5 * full["total"]
    # fused inattentive token: one more row per drop and the fusion weights
    _, fu = P.bsr_saved_activation_bytes(P.make_config(dict(cfg, fuse_dropped=True), 32), 1)
    assert fu["total"] > t1["total"] and fu["stats"] > t1["stats"]
    # mixture-of-experts blocks report their routing state
    pm, tmoe = P.bsr_saved_activation_bytes(P.make_config(S.get_config("c5_vit_s_moe"), 8), 1)
    assert tmoe["moe"] > 0 and all((r["moe"] > 0) == (l in (9, 11)) for l, r in enumerate(pm) if r["total"])


def test_workspace_holds_the_class_sums_of_a_wide_head():
    # beyond 8 x the widest layer, the 64 rows of partial class sums are the longest thing their buffer takes
    cfg = S.get_config("mini_4blk", num_classes=20000)
    more = P.bsr_workspace_bytes(P.make_config(dict(cfg, num_classes=40000), 64)) - P.bsr_workspace_bytes(P.make_config(cfg, 64))
    assert more >= 4 * 20000 * (64 + 2 * 64)               # partial sums, logits and their gradient


def test_saved_bytes_errors():
    c = P.make_config(S.get_config("mini_4blk"), 4)
    for bad in (0, 5):
        with pytest.raises(P.BsrError):
            P.bsr_saved_activation_bytes(c, bad)
    assert P.load_library().bsr_saved_activation_bytes(None, 1, None, None) == -1


def test_null_context_is_rejected_before_any_gpu_work():
    lib = P.load_library()
    assert lib.bsr_autotune(None, None, None, 1, None, None, None, None, None, None) == -1
    assert lib.bsr_autotune_overlapped(None, None, None, 1, None, None, None, None, None, None, None, None) == -1
    assert lib.bsr_pipeline_step(None, None, None, None, None, 1, None, None, None, 0.0, 0.0, 0.0, None, None) == -1
    assert lib.bsr_adamw_step(None, None, None, None, 0.0, 0.9, 0.999, 1e-8, 0.0, 1, None) == -1
    assert lib.bsr_sgd_step(None, None, None, 0.0, 0.0, 0.0, None) == -1


@pytest.mark.parametrize("call", [
    lambda t, w: P.bsr_linear_forward(t, w), lambda t, w: P.bsr_linear_dgrad(t, w), lambda t, w: P.bsr_linear_wgrad(t, t),
    lambda t, w: P.bsr_linear_wgrad_static(t, t), lambda t, w: P.bsr_linear_backward(t, t, w),
    lambda t, w: P.bsr_ln_linear_fold(w.float(), w[0].float(), w[0].float(), w[0].float()),
    lambda t, w: P.bsr_ln_linear_forward(t, w, w[0].float(), w[0].float()),
    lambda t, w: P.bsr_attention_forward(t[None], 1),
    lambda t, w: P.bsr_attention_backward(t[None], t[None, :, :64], t[None, :, :64], w.float(), 1),
    lambda t, w: P.Context(S.get_config("c1_block_fp32"), S.make_params(S.get_config("c1_block_fp32")), 1, device="cpu")])
def test_host_tensors_are_refused_before_the_library_sees_them(call, monkeypatch):
    import torch
    lib = P.load_library()

    class Closed:                     # whatever would launch is not to be reached
        def __getattr__(self, name):
            if name in ("bsr_token_schedule", "bsr_workspace_bytes", "bsr_last_error"):
                return getattr(lib, name)
            return lambda *a: pytest.fail(f"{name} was called with host memory")

    monkeypatch.setattr(P.binding, "_lib", Closed())
    with pytest.raises(ValueError):
        call(torch.zeros(8, 192, dtype=torch.bfloat16), torch.zeros(192, 192, dtype=torch.bfloat16))


def test_tensor_names_are_taken_and_refused_as_the_struct_takes_them():
    import torch
    from paper_2405_10951_amd import binding
    t = torch.zeros(1)
    table = binding._params_struct({"lnf_g": t, "blocks.15.w_router": t, "blocks.0.b_qkv": None, "ema": t, "blocks.0.ema": t})
    p = binding.bsr_params.from_buffer(table)
    assert p.lnf_g == p.blocks[15].w_router == t.data_ptr()
    assert sum(v != 0 for v in table) == 2
    known = len(binding._position)
    for i in range(100):                              # names that are none of the library's leave nothing behind
        binding._params_struct({f"ema.{i}": t})
    assert len(binding._position) == known
    for name, error in (("blocks", TypeError), ("blocks.16.w_qkv", IndexError), ("blocks.w_qkv", ValueError)):
        with pytest.raises(error):
            binding._params_struct({name: t})
