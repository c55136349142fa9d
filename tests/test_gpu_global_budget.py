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
