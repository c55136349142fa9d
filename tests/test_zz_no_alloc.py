"""The entry point that allocates nothing (workspace in a static device array) against
svf_verify_attn: the same bits, on two calls in a row, the second with a smaller input."""
import dataclasses

import numpy as np
import pytest
import torch

import paper_2512_21911_amd as S
import workloads as W
from svf_harness import DeviceRun, check_attn, oracle_attn, to_gpu
from test_gpu_parity import small as small_cfg

pytestmark = pytest.mark.gpu


def run_both(cfg):
    x = W.make_layer(cfg)
    run = DeviceRun(cfg, to_gpu(x))
    run.block_reps().score_select().verify_attn().sync()
    out0, lse0 = run.out.clone(), run.lse.clone()
    ref, lse_ref = oracle_attn(cfg, x, run.sel_idx.cpu(), run.sel_cnt.cpu())
    check_attn(cfg, out0, lse0, ref, lse_ref)
    run.out.fill_(float("nan"))
    run.lse.fill_(float("nan"))
    g = run.x
    before = torch.cuda.memory_allocated()
    S.svf_verify_attn_static_ws(run.shape, g["q"], g["k_pool"], g["v_pool"], g["block_table"], g["seq_lens"],
                                g["k_draft"], g["v_draft"], g["draft_mask"], run.sel_idx, run.sel_cnt, run.out, run.lse)
    torch.cuda.synchronize()
    assert torch.cuda.memory_allocated() == before
    assert torch.equal(run.out.view(torch.int16 if cfg.dtype == "bf16" else torch.int32),
                       out0.view(torch.int16 if cfg.dtype == "bf16" else torch.int32)), cfg.name
    assert torch.equal(run.lse.view(torch.int32), lse0.view(torch.int32)), cfg.name
    check_attn(cfg, run.out, run.lse, ref, lse_ref)
    return run


def test_static_workspace_entry_point_matches_on_two_calls_in_a_row():
    assert S.svf_static_workspace_bytes() == 16 << 20
    big = W.shrink(W.CONFIGS[3], 8192)                     # several splits per (sequence, KV head)
    small = W.shrink(W.CONFIGS[2], 2048)                   # a smaller input right behind it, another shape
    run_both(big)
    run_both(small)
    run_both(big)                                          # and back: the array is cleared per call
    run_both(W.CONFIGS[1])                                 # fp32: the vector-ALU kernels and their merge launch
    # a 24-node draft tree: the many-rows kernel, whose splits meet through the same words of the array
    run_both(dataclasses.replace(W.shrink(W.CONFIGS[3], 8192), name="cfg3_8k_tree24", gamma=24, tree_depth=4))
    run_both(small)


def test_static_workspace_entry_point_refuses_what_does_not_fit():
    cfg = W.shrink(W.CONFIGS[3], 4096)
    x = W.make_layer(cfg)
    run = DeviceRun(cfg, to_gpu(x))
    run.block_reps().score_select().sync()
    g = run.x
    huge = S.make_shape(B=cfg.B, gamma=64, Hq=cfg.Hq * 4, Hkv=cfg.Hkv, d=cfg.d, dtype="f32", block_size=cfg.block_size,
                        max_seq_len=cfg.T, k_blocks=cfg.k_blocks, k_pool=g["k_pool"], page_size=cfg.page_size,
                        max_pages_per_seq=g["block_table"].shape[1])
    assert S.svf_workspace_bytes(huge) > S.svf_static_workspace_bytes()
    with pytest.raises(S.SvfError) as e:
        S.svf_verify_attn_static_ws(huge, g["q"], g["k_pool"], g["v_pool"], g["block_table"], g["seq_lens"],
                                    g["k_draft"], g["v_draft"], g["draft_mask"], run.sel_idx, run.sel_cnt, run.out)
    assert e.value.code == -6


def test_static_workspace_entry_point_at_head_dimension_64():
    run_both(small_cfg(d=64, B=4, Hq=32, Hkv=16, gamma=7, T=8192, k_blocks=60, min_len=3000))      # matrix cores
    # 33 and more splits of many pairs do not fit the array: the vector-ALU kernel takes the call
    cfg = small_cfg(d=64, B=16, Hq=32, Hkv=32, gamma=2, T=4200, k_blocks=64, min_len=4150)
    run = DeviceRun(cfg, to_gpu(W.make_layer(cfg)))
    assert S.svf_workspace_bytes(run.shape) > S.svf_static_workspace_bytes()
    run.block_reps().score_select().sync()
    g = run.x
    args = (g["q"], g["k_pool"], g["v_pool"], g["block_table"], g["seq_lens"], g["k_draft"], g["v_draft"], g["draft_mask"],
            run.sel_idx, run.sel_cnt)
    ws = S.new_diag_workspace(run.shape, S.SVF_KERNEL_VECTOR_ALU)
    want, want_lse = torch.empty_like(run.out), torch.empty_like(run.lse)
    S.svf_diag_verify_attn(run.shape, S.SVF_KERNEL_VECTOR_ALU, *args, want, ws, want_lse)
    for _ in range(2):
        run.out.fill_(float("nan"))
        S.svf_verify_attn_static_ws(run.shape, *args, run.out, run.lse)
        torch.cuda.synchronize()
        assert torch.equal(run.out.view(torch.int16), want.view(torch.int16))
        assert torch.equal(run.lse.view(torch.int32), want_lse.view(torch.int32))


@pytest.mark.parametrize("kw", [dict(B=2, Hq=16, Hkv=4, gamma=5, T=16384, k_blocks=256, min_len=16100),
                                dict(B=8, Hq=16, Hkv=16, gamma=8, T=8192, block_size=16, k_blocks=128, min_len=8100)])
def test_static_workspace_entry_point_with_splits_shared_out(kw):
    """Counts that differ per pair: the same splits, hence the same bits."""
    cfg = small_cfg(**kw)
    run = DeviceRun(cfg, to_gpu(W.make_layer(cfg)))
    assert S.svf_workspace_bytes(run.shape) <= S.svf_static_workspace_bytes()
    run.block_reps().score_select().sync()
    for b in range(cfg.B):
        for h in range(cfg.Hkv):
            c = (0, 3, cfg.k_blocks // 2, cfg.k_blocks, 1)[(b + h) % 5]
            run.sel_idx[b, h, c:] = -1
            run.sel_cnt[b, h] = c
    run.verify_attn().sync()
    out, lse = run.out.clone(), run.lse.clone()
    g = run.x
    run.out.fill_(float("nan"))
    S.svf_verify_attn_static_ws(run.shape, g["q"], g["k_pool"], g["v_pool"], g["block_table"], g["seq_lens"], g["k_draft"],
                                g["v_draft"], g["draft_mask"], run.sel_idx, run.sel_cnt, run.out, run.lse)
    torch.cuda.synchronize()
    assert torch.equal(run.out.view(torch.int16), out.view(torch.int16)) and torch.equal(run.lse.view(torch.int32), lse.view(torch.int32))
