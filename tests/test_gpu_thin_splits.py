"""Attention whose tiles are spread over more workgroups than their wavefronts would need, against the CPU oracle:
one to three tiles per workgroup, splits without a tile, up to sixteen splits, two row groups, lists shorter than the
plan, with all step modes on one workspace (full_parity() asks for the same blocks and the same bits).  What one workgroup
can take is rounded once."""
import pytest
import torch

import workloads as W
from svf_harness import DeviceRun, full_parity, to_gpu
from test_gpu_parity import small

pytestmark = pytest.mark.gpu

CASES = {
    "one_tile_and_the_draft": small(B=1, Hq=8, Hkv=2, gamma=2, T=200, block_size=32, k_blocks=1, page_size=0),
    "draft_only_splits_empty": small(B=2, Hq=8, Hkv=2, gamma=3, T=300, k_blocks=4, min_len=1),
    "nine_tiles_one_split": small(B=1, Hq=8, Hkv=8, gamma=4, T=900, k_blocks=4),
    "seventeen_tiles_eight_splits": small(B=4, Hq=32, Hkv=8, gamma=8, T=1100, k_blocks=8),
    "eighteen_tiles_nine_to_eight": small(B=3, Hq=8, Hkv=8, gamma=3, T=1100, block_size=32, k_blocks=17),
    "33_tiles_sixteen_splits": small(B=1, Hq=32, Hkv=8, gamma=5, T=1500, k_blocks=16, page_size=0),
    "34_tiles_seventeenth_split_not_taken": small(B=1, Hq=32, Hkv=8, gamma=5, T=1500, block_size=32, k_blocks=33),
    "129_tiles_full_wavefronts": small(B=1, Hq=8, Hkv=2, gamma=3, T=4500, k_blocks=64),
    "131_tiles_seventeen_splits": small(B=1, Hq=8, Hkv=2, gamma=3, T=4500, k_blocks=65),
    "two_row_groups_sixteen_splits": small(B=1, Hq=32, Hkv=8, gamma=16, tree_depth=5, T=2000, k_blocks=17),
    "two_draft_tiles": small(B=1, Hq=2, Hkv=2, gamma=40, tree_depth=5, T=900, k_blocks=6),
    "ragged_lists_shorter_than_the_plan": small(B=4, Hq=8, Hkv=4, gamma=6, T=2500, k_blocks=20, min_len=40),
    "d64_one_tile_and_the_draft": small(B=1, Hq=8, Hkv=2, d=64, gamma=2, T=200, block_size=32, k_blocks=1, page_size=0),
    "d64_draft_only_splits_empty": small(B=2, Hq=8, Hkv=2, d=64, gamma=3, T=300, k_blocks=4, min_len=1),
    "d64_nine_tiles_eight_splits": small(B=1, Hq=8, Hkv=8, d=64, gamma=4, T=900, k_blocks=4),
    "d64_33_tiles": small(B=3, Hq=32, Hkv=8, d=64, gamma=7, T=1500, k_blocks=16, min_len=200),
    "d64_seventeen_tiles_two_row_groups": small(B=1, Hq=32, Hkv=8, d=64, gamma=10, T=1100, k_blocks=8),
}


@pytest.mark.parametrize("name", sorted(CASES))
def test_thin_splits(name):
    r = full_parity(CASES[name])
    print(f"[thin splits] {name}: max_abs_err={r['max_abs_err']:.3e} near_ties={r['near_ties']}", flush=True)


@pytest.mark.parametrize("d, k_blocks", [(128, 1), (128, 2), (128, 4), (64, 1), (64, 4), (64, 16)])
def test_short_lists_are_rounded_once(d, k_blocks):
    """A query of zeros weighs every key alike: weights and their sum are exact, the output is the mean of the values,
    and where nothing but the result is held in 16 bits it is off by half a bfloat16 step, plus n fp32 roundings."""
    T = 64 * k_blocks
    cfg = small(B=1, Hq=32, Hkv=8, d=d, gamma=4, T=T, k_blocks=k_blocks, page_size=0)
    x = W.make_layer(cfg)
    x["q"] = torch.zeros_like(x["q"])
    run = DeviceRun(cfg, to_gpu(x)).block_reps().score_select().verify_attn(mask=None).sync()
    length = int(x["seq_lens"][0])
    v, vd = x["v_pool"][0, :length].double(), x["v_draft"][0].double()          # [T][Hkv][d], [gamma][Hkv][d]
    for i in range(cfg.gamma):
        keys = torch.cat([v, vd[:i + 1]])
        mean = keys.mean(0)
        half = 2.0 ** (torch.frexp(mean.float())[1].double() - 9)
        bound = half + len(keys) * 2.0 ** -23 * keys.abs().mean(0)
        got = run.out[0, i].double().cpu().view(cfg.Hkv, cfg.Hq // cfg.Hkv, d)
        assert ((got - mean[:, None]).abs() <= bound[:, None]).all(), (i, d, k_blocks)


THIN = {                                                 # splits of the plan; lists of one to all of its tiles
    "sixteen_splits": small(B=2, Hq=32, Hkv=8, gamma=4, T=1100, k_blocks=17, page_size=0),
    "sixteen_splits_two_row_groups": small(B=2, Hq=16, Hkv=2, gamma=7, T=1100, block_size=32, k_blocks=33),
    "eight_splits": small(B=4, Hq=32, Hkv=8, gamma=5, T=2100, k_blocks=16),
    "four_splits": small(B=8, Hq=16, Hkv=8, gamma=3, T=600, k_blocks=8),
    "three_splits": small(B=10, Hq=8, Hkv=8, gamma=2, T=500, k_blocks=7),
    "d64_sixteen_splits": small(B=2, Hq=32, Hkv=8, d=64, gamma=4, T=1100, k_blocks=17),
}


@pytest.mark.parametrize("by", ["length", "count"])
@pytest.mark.parametrize("name", sorted(THIN))
def test_lists_shorter_than_the_plan_are_rounded_once(name, by):
    """The same for lists of one tile to all of the plan's, because a sequence is short or because few blocks are handed
    over: spread over the plan's splits, whose partials hold fp32."""
    cfg = THIN[name]
    x = W.make_layer(cfg)
    x["q"] = torch.zeros_like(x["q"])
    most = cfg.k_blocks * cfg.block_size
    pairs = cfg.B * cfg.Hkv
    tokens = [[1 + (most - 1) * ((b * cfg.Hkv + h) ** 2) // (pairs - 1) ** 2 for h in range(cfg.Hkv)] for b in range(cfg.B)]
    if by == "length":
        tokens = [[t[0]] * cfg.Hkv for t in tokens]
        x["seq_lens"] = torch.tensor([t[0] for t in tokens], dtype=torch.int32).minimum(x["seq_lens"])
    count = torch.tensor([[-(-n // cfg.block_size) for n in t] for t in tokens], dtype=torch.int32)
    idx = torch.arange(cfg.k_blocks, dtype=torch.int32).expand(cfg.B, cfg.Hkv, -1).contiguous()
    idx[idx >= count[..., None]] = -1
    run = DeviceRun(cfg, to_gpu(x)).verify_attn(mask=None, sel_idx=idx.cuda(), sel_cnt=count.cuda()).sync()
    got = run.out.double().cpu().view(cfg.B, cfg.gamma, cfg.Hkv, cfg.Hq // cfg.Hkv, cfg.d)
    for b in range(cfg.B):
        for h in range(cfg.Hkv):
            n = min(int(count[b, h]) * cfg.block_size, int(x["seq_lens"][b]))
            if x["block_table"] is None:
                v = x["v_pool"][b, :n, h]
            else:
                t = torch.arange(n)
                v = x["v_pool"][x["block_table"][b, t // cfg.page_size].long(), t % cfg.page_size, h]
            for i in range(cfg.gamma):
                keys = torch.cat([v, x["v_draft"][b, :i + 1, h]]).double()
                mean = keys.mean(0)
                half = 2.0 ** (torch.frexp(mean.float())[1].double() - 9)
                # (an addition for each key and split, products with a weight and a reciprocal in each of the two steps)
                bound = half + (len(keys) + 24) * 2.0 ** -23 * keys.abs().mean(0)
                assert ((got[b, i, h] - mean).abs() <= bound).all(), (b, h, i, n)
