"""One budget over all KV heads of a sequence: the selection against the variants oracle on the
library's own scores (no near-ties then: exact), at the edges of its keys-per-thread variants and with
equal scores; and the attention over lists of very different lengths per KV head."""
import numpy as np
import pytest
import torch

import paper_2512_21911_amd as S
import workloads as W
from oracle import svf_variants_oracle as V
from svf_harness import DeviceRun, check_attn, oracle_attn, to_gpu
from test_gpu_variants import F32, GLOBAL, GMAX, MEAN, small
from test_gpu_parity import small as small_bf16

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ties", [False, True])
@pytest.mark.parametrize("Hkv,nb,n_total", [(1, 1, 1), (2, 65, 1), (8, 512, 256), (8, 513, 300), (4, 2048, 100),
                                            (3, 2731, 500), (8, 4096, 2000), (16, 2049, 64), (300, 30, 700)])
def test_global_selection_is_exact(Hkv, nb, n_total, ties):
    # 1 .. 4, 5 .. 8 and 9 .. 32 keys per thread, one more than 32, more heads than the kernel's table
    cfg = small(B=2, Hq=Hkv, Hkv=Hkv, gamma=1, T=nb * 4, min_len=max(1, nb * 2), block_size=4, page_size=4,
                n_sink=int(nb > 8 and n_total >= 2 * Hkv), n_local=int(nb > 8 and n_total >= 2 * Hkv))
    gen = torch.Generator().manual_seed(nb)
    lens = torch.tensor([nb * 4, cfg.min_len], dtype=torch.int32)
    q = torch.randn(2, 1, Hkv, 64, generator=gen)
    shape = S.make_shape(B=2, gamma=1, Hq=Hkv, Hkv=Hkv, d=64, dtype="f32", block_size=4, max_seq_len=nb * 4,
                         k_blocks=min(nb, n_total), kv_strides=(nb * 4 * Hkv * 64, Hkv * 64, 64), n_sink=cfg.n_sink,
                         n_local=cfg.n_local)
    rt = S.SvfRetrieval(MEAN, F32, GMAX, GLOBAL, n_total)
    summ = torch.randn(2, Hkv, nb, 64, generator=gen)
    if ties:                       # runs of equal scores, the weakest kept one among them
        summ = summ[:, :, :3].repeat_interleave(-(-nb // 3), dim=2)[:, :, :nb].contiguous()
        q[:] = q[:, :, :1]
        summ[:] = summ[:, :1]
    scores = torch.full((2, Hkv, nb), float("nan"), device="cuda")
    idx = torch.full((2, Hkv, shape.k_blocks), -7, dtype=torch.int32, device="cuda")
    cnt = torch.full((2, Hkv), -7, dtype=torch.int32, device="cuda")
    for _ in range(2):
        S.svf_retrieve(shape, rt, q.cuda(), summ.cuda(), lens.cuda(), idx, cnt, S.new_workspace(shape), scores)
    torch.cuda.synchronize()
    ref_idx, ref_cnt = V.select_global(scores.double().cpu().numpy(), lens, 4, n_total, shape.k_blocks, cfg.n_sink, cfg.n_local)
    np.testing.assert_array_equal(cnt.cpu().numpy(), ref_cnt)
    np.testing.assert_array_equal(idx.cpu().numpy(), ref_idx)


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("counts", [(0, 1, 5, 60), (16, 4, 200, 3), (17, 16, 15, 256)])
def test_attention_over_lists_of_different_lengths(counts, d):
    """Splits follow each head's own count; counts of no, one, several and all planned splits."""
    cfg = small_bf16(B=2, Hq=16, Hkv=4, d=d, T=16384, gamma=5, k_blocks=256, min_len=16100)
    x = W.make_layer(cfg)
    run = DeviceRun(cfg, to_gpu(x))
    rng = np.random.default_rng(5)
    idx = np.full((2, 4, 256), -1, dtype=np.int32)
    for b in range(2):
        for h, c in enumerate(counts):
            idx[b, h, :min(c, 251)] = np.sort(rng.choice(251, min(c, 251), replace=False))
    cnt = (idx >= 0).sum(-1).astype(np.int32)
    idx, cnt = torch.from_numpy(idx), torch.from_numpy(cnt)
    out0 = None
    for polls in (-1, 0, 1):
        S.svf_workspace_set_wait_polls(run.shape, run.ws, polls)
        for _ in range(3):
            run.out.fill_(float("nan"))
            run.verify_attn(sel_idx=idx.cuda(), sel_cnt=cnt.cuda()).sync()
            out0 = run.out.clone() if out0 is None else out0
            assert torch.equal(run.out.view(torch.int16), out0.view(torch.int16)), f"polls={polls}"
    out_ref, lse_ref = oracle_attn(cfg, x, idx, cnt)
    check_attn(cfg, run.out, run.lse, out_ref, lse_ref)


@pytest.mark.parametrize("kw", [
    dict(B=3, Hq=6, Hkv=3, gamma=5, T=8192, k_blocks=250),                       # 9 pairs: no multiple of eight
    dict(B=5, Hq=40, Hkv=5, gamma=5, T=2400, k_blocks=70, d=64),                 # 40 rows: two row groups
    dict(B=13, Hq=10, Hkv=5, gamma=3, T=1600, k_blocks=50),                      # 65 pairs: the second chunk holds one
    dict(B=9, Hq=90, Hkv=15, gamma=6, T=1500, k_blocks=44, d=64),                # 135 pairs, two row groups
    dict(B=16, Hq=16, Hkv=16, gamma=4, T=1600, k_blocks=50, d=64),               # 256 pairs, all four chunks
], ids=lambda kw: f"{kw['B']}x{kw['Hkv']}")
def test_shared_out_splits_over_many_pairs(kw):
    """Counts drawn per pair (empty, short, all that fits): every chunk of 64 pairs, the padded pairs of the grid
    and both row groups, against the oracle; then every count the per-head rule's: the planned splits,
    the bits of the step that reuses the selection through its gather list."""
    cfg = small_bf16(block_size=32, page_size=16, min_len=kw["T"] - 200, **kw)
    x = W.make_layer(cfg)
    run = DeviceRun(cfg, to_gpu(x))
    rng = np.random.default_rng(cfg.B)
    idx = np.full((cfg.B, cfg.Hkv, cfg.k_blocks), -1, dtype=np.int32)
    lens = x["seq_lens"].tolist()
    for b in range(cfg.B):
        nb = min(-(-lens[b] // 32), cfg.k_blocks)
        for h in range(cfg.Hkv):
            c = int(rng.choice([0, 1, 3, 9, nb, rng.integers(1, nb + 1)]))
            idx[b, h, :c] = np.sort(rng.choice(nb, c, replace=False))
    cnt = (idx >= 0).sum(-1).astype(np.int32)
    idx, cnt = torch.from_numpy(idx), torch.from_numpy(cnt)
    for _ in range(2):
        run.out.fill_(float("nan"))
        run.verify_attn(sel_idx=idx.cuda(), sel_cnt=cnt.cuda()).sync()
    check_attn(cfg, run.out, run.lse, *oracle_attn(cfg, x, idx, cnt))
    run.block_reps().verify_step(S.SVF_STEP_ANCHOR).verify_step(S.SVF_STEP_REUSE_GATHER).sync()
    out = run.out.clone()
    run.out.fill_(float("nan"))
    run.verify_attn().sync()
    assert torch.equal(run.out.view(torch.int16), out.view(torch.int16))


def test_shared_out_splits_that_do_not_fit_at_once():
    """Many lists of one block beside a few full ones: a split for each of them is more than the grid holds beside the full
    lists' shares of all of it, so fewer are shared out."""
    cfg = small_bf16(B=12, Hq=32, Hkv=8, gamma=8, T=2100, k_blocks=32, block_size=32, page_size=16)
    x = W.make_layer(cfg)
    run = DeviceRun(cfg, to_gpu(x))
    rng = np.random.default_rng(3)
    idx = np.full((12, 8, 32), -1, dtype=np.int32)
    for b in range(12):
        for h in range(8):
            c = 32 if (8 * b + h) % 3 == 0 else int(rng.integers(0, 2))
            idx[b, h, :c] = np.sort(rng.choice(65, c, replace=False))
    cnt = (idx >= 0).sum(-1).astype(np.int32)
    idx, cnt = torch.from_numpy(idx), torch.from_numpy(cnt)
    for _ in range(2):
        run.out.fill_(float("nan"))
        run.verify_attn(sel_idx=idx.cuda(), sel_cnt=cnt.cuda()).sync()
    check_attn(cfg, run.out, run.lse, *oracle_attn(cfg, x, idx, cnt))
