"""The fp32 attention kernel against the CPU oracle where its tiles of sixteen tokens, halves of sixteen rows,
splits and trips of eight splits have edges, and its own retrieval (up to 1024 blocks, page-table row in
LDS or not) against the stand-alone one: full_parity() asks for the same blocks and the same bits in all modes."""
import pytest
import torch

import paper_2512_21911_amd as S
import workloads as W
from svf_harness import DeviceRun, check_attn, full_parity, oracle_attn, shape_for, to_gpu
from test_gpu_parity import small

pytestmark = pytest.mark.gpu


def f32(**kw):
    return small(**dict(dict(dtype="f32", B=1, Hq=4, Hkv=1, planted=1), **kw))


CASES = {
    # rows around a half and a row group (4 query heads per KV head), two and four draft tiles
    "rows_16_17_drafts": f32(gamma=4, T=300),
    "rows_20": f32(gamma=5, T=300, d=64),
    "rows_32_block_16": f32(gamma=8, T=500, block_size=16, k_blocks=3),
    "rows_36_d64": f32(gamma=9, T=500, d=64),
    "drafts_17_mha": f32(Hq=2, Hkv=2, gamma=17, T=300),
    "drafts_64_mha_tree": f32(Hq=2, Hkv=2, gamma=64, T=300, tree_depth=6),
    # tokens around a tile; sequences shorter than a block
    "tokens_15_16_17": f32(B=3, T=17, min_len=15, block_size=32, k_blocks=1, gamma=1, page_size=0, planted=0),
    "block_1_page_1": f32(T=60, block_size=1, page_size=1, k_blocks=37, gamma=2, d=64),
    "block_21": f32(B=2, T=500, min_len=77, block_size=21, page_size=7, k_blocks=9),
    # two units and five; as many splits as tiles; one, two and three trips of eight splits, the last one also not full; many
    "two_units": f32(T=40, block_size=16, page_size=16, k_blocks=1, gamma=1, d=64),
    "five_units": f32(T=400, block_size=64, k_blocks=1, gamma=4),
    "splits_8": f32(T=2000, block_size=32, k_blocks=15, gamma=2),
    "splits_16": f32(T=2000, block_size=16, k_blocks=70, gamma=2, d=64),
    "splits_24_two_halves": f32(T=4000, block_size=32, k_blocks=65, gamma=8),
    "splits_12_of_20_groups": f32(B=5, Hq=16, Hkv=4, T=1500, min_len=900, block_size=32, k_blocks=42, gamma=4, d=64),
    "splits_21_of_12_groups": f32(B=3, Hq=16, Hkv=4, T=2400, block_size=32, k_blocks=70, gamma=6),
    "splits_64": f32(T=16000, block_size=32, k_blocks=470, gamma=6, d=64),
    "splits_8_of_16_row_groups": f32(Hq=8, gamma=64, T=900, block_size=32, k_blocks=14),
    "splits_cut_by_groups": f32(B=16, Hq=32, Hkv=16, T=600, block_size=32, k_blocks=9, gamma=3),
    # retrieval: a single block, one and two batches of passes, the most blocks and one more, forced blocks
    "blocks_1": f32(B=2, T=16, block_size=16, k_blocks=4, planted=0),
    "blocks_513": f32(T=8200, block_size=16, k_blocks=20, planted=5, n_sink=2, n_local=3),
    "blocks_1024_all_pages_in_lds": f32(T=16384, block_size=16, page_size=8, k_blocks=16, planted=5, d=64),
    "blocks_1024_table_too_long": f32(T=16384, block_size=16, page_size=4, k_blocks=16, planted=5, d=64),
    "blocks_1025": f32(T=16400, block_size=16, k_blocks=16, planted=5, d=64),
    "budget_above_blocks": f32(B=3, T=400, min_len=20, block_size=16, k_blocks=40),
    "many_heads_per_group": f32(Hq=40, gamma=1, T=600),
    "bf16_blocks_of_6_in_one_split": small(B=16, Hq=32, Hkv=16, T=120, block_size=6, page_size=6, k_blocks=2, min_len=50),
    "bf16_block_33_contiguous": small(d=64, T=900, block_size=33, page_size=0, k_blocks=11, min_len=300, gamma=6),
}


@pytest.mark.parametrize("name", sorted(CASES))
def test_f32(name):
    r = full_parity(CASES[name])
    print(f"[fp32] {name}: max_abs_err={r['max_abs_err']:.3e} near_ties={r['near_ties']}", flush=True)


@pytest.mark.parametrize("d", [64, 128])
def test_fewer_splits_where_the_static_workspace_is_full_of_scores(d):
    """A limit of some four million blocks: with eight splits the workspace is larger than the static array, with
    fewer it fits, and both entry points give the same bits."""
    cfg = f32(T=700, block_size=1, page_size=16, k_blocks=300, gamma=2, d=d)
    x = W.make_layer(cfg)
    idx = torch.arange(300, dtype=torch.int32).view(1, 1, 300) * 2
    cnt = torch.full((1, 1), 300, dtype=torch.int32)
    nb = (S.svf_static_workspace_bytes() - 40 * 1024) // 4 // 64 * 64
    table = torch.zeros(1, nb // 16, dtype=torch.int32)
    table[:, :x["block_table"].shape[1]] = x["block_table"]
    xg = to_gpu(dict(x, block_table=table))
    shape = shape_for(cfg, xg, max_seq_len=nb)
    assert S.svf_static_workspace_bytes() - 64 * 1024 < S.svf_workspace_bytes(shape) <= S.svf_static_workspace_bytes()
    shape_1k = shape_for(cfg, to_gpu(x))
    partials = S.svf_workspace_bytes(shape_1k)                # eight splits, hardly any scores
    assert partials + 4 * nb > S.svf_static_workspace_bytes()
    out, ws = torch.empty_like(xg["q"]), S.new_workspace(shape)
    lse = torch.empty(1, cfg.gamma, cfg.Hq, device="cuda")
    args = (shape, xg["q"], xg["k_pool"], xg["v_pool"], xg["block_table"], xg["seq_lens"], xg["k_draft"], xg["v_draft"], None,
            idx.cuda(), cnt.cuda(), out)
    S.svf_verify_attn(*args, ws, lse)
    check_attn(cfg, out, lse, *oracle_attn(cfg, x, idx, cnt, mask=None))
    first = out.clone()
    out.fill_(float("nan"))
    S.svf_verify_attn_static_ws(*args)
    torch.cuda.synchronize()
    assert torch.equal(out, first)
