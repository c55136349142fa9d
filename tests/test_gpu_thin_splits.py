"""Attention whose tiles are spread over more workgroups than their wavefronts would need, against the CPU oracle:
one to three tiles per workgroup, splits without a tile, up to sixteen splits, two row groups, lists shorter than the
plan, with all step modes on one workspace (full_parity() asks for the same blocks and the same bits).  What one workgroup
can take is rounded once."""
import pytest
import torch

import paper_2512_21911_amd as S
import workloads as W
from oracle import svf_oracle as O
from svf_harness import LSE_TOL, OUT_TOL, DeviceRun, full_parity, to_gpu
from test_gpu_parity import small

pytestmark = pytest.mark.gpu

CASES = {
    "one_tile_and_the_draft": small(B=1, Hq=8, Hkv=2, gamma=2, T=200, block_size=32, k_blocks=1, page_size=0),
    "draft_only_splits_empty": small(B=2, Hq=8, Hkv=2, gamma=3, T=300, k_blocks=4, min_len=1),
    "nine_tiles_one_split": small(B=1, Hq=8, Hkv=8, gamma=4, T=900, k_blocks=4),
    "seventeen_tiles_eight_splits": small(B=4, Hq=32, Hkv=8, gamma=8, T=1100, k_blocks=8),
    "eighteen_tiles_eight_splits": small(B=3, Hq=8, Hkv=8, gamma=3, T=1100, block_size=32, k_blocks=17),
    "33_tiles_ten_splits_cut_to_eight": small(B=3, Hq=32, Hkv=8, gamma=6, T=1500, k_blocks=16),
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


def limit_shape(d, nb):
    """Eight pairs with lists of 33 tiles and so many blocks that their scores fill most of the static array."""
    return S.make_shape(B=1, gamma=4, Hq=32, Hkv=8, d=d, dtype="bf16", block_size=64, max_seq_len=64 * nb, k_blocks=16, page_size=64,
                        max_pages_per_seq=nb, kv_strides=(64 * 8 * d, 8 * d, d))


# the last numbers of blocks (in steps of eight: 256 bytes of scores) whose sixteen splits, and whose four, fit the array
AT_THE_LIMIT = {128: (456168, 515048), 64: (489448, 515560)}


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


@pytest.mark.parametrize("by", [0, 1])
@pytest.mark.parametrize("d", [64, 128])
def test_plans_at_the_size_of_the_static_array(d, by):
    """On either side of the limit (test_split_plans.py): the entry point with the static array gives the bits of the one with a
    workspace, and what the oracle gives."""
    for nb in (AT_THE_LIMIT[d][by], AT_THE_LIMIT[d][by] + 8):
        shape = limit_shape(d, nb)
        g = torch.Generator().manual_seed(d + by)
        r = lambda *dims: torch.randn(*dims, generator=g).to(torch.bfloat16)
        x = dict(q=r(1, 4, 32, d), k=r(16, 64, 8, d), v=r(16, 64, 8, d), kd=r(1, 4, 8, d), vd=r(1, 4, 8, d),
                 lens=torch.tensor([1000], dtype=torch.int32), table=torch.zeros(1, nb, dtype=torch.int32),
                 idx=torch.arange(16, dtype=torch.int32).expand(1, 8, 16).contiguous(),
                 cnt=torch.tensor([[16, 15, 12, 8, 4, 2, 1, 0]], dtype=torch.int32))
        x["table"][0, :16] = torch.randperm(16, generator=g).to(torch.int32)
        c = {k: t.cuda() for k, t in x.items()}
        out = torch.full_like(c["q"], float("nan"))
        lse = torch.full((1, 4, 32), float("nan"), device="cuda")
        args = (shape, c["q"], c["k"], c["v"], c["table"], c["lens"], c["kd"], c["vd"], None, c["idx"], c["cnt"])
        S.svf_verify_attn(*args, out, S.new_workspace(shape), lse)
        ref, lref = O.verify_attn(x["q"], x["k"], x["v"], x["table"], x["lens"], x["kd"], x["vd"], None, x["idx"], x["cnt"], 64, None)
        assert abs(out.double().cpu().numpy() - ref).max() <= OUT_TOL["bf16"]
        assert abs(lse.double().cpu().numpy() - lref).max() <= LSE_TOL["bf16"]
        again, lagain = torch.full_like(out, float("nan")), torch.full_like(lse, float("nan"))
        if S.svf_workspace_bytes(shape) <= S.svf_static_workspace_bytes():
            S.svf_verify_attn_static_ws(*args, again, lagain)
            assert torch.equal(out.view(torch.int16), again.view(torch.int16)) and torch.equal(lse, lagain)
        elif d == 128:
            with pytest.raises(S.SvfError):
                S.svf_verify_attn_static_ws(*args, again, lagain)
