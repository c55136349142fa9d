"""Representatives of a few blocks (one workgroup per head) give the bits of a launch over all blocks
(one workgroup per block): heads, channels, types, block sizes around the stage, partial last blocks."""
import pytest
import torch

import paper_2512_21911_amd as S

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,Hkv,d,block,page", [
    ("bf16", 8, 128, 64, 16), ("bf16", 4, 128, 128, 0), ("bf16", 1, 64, 32, 32), ("bf16", 3, 128, 16, 16), ("bf16", 16, 64, 7, 7),
    ("bf16", 1, 64, 256, 64), ("bf16", 2, 128, 129, 0), ("f32", 2, 64, 16, 0), ("f32", 1, 128, 64, 16), ("f32", 5, 64, 33, 0),
])
def test_few_blocks_same_bits(dtype, Hkv, d, block, page):
    dt = torch.float32 if dtype == "f32" else torch.bfloat16
    nb = 512 // Hkv + 3                                   # a launch over all of them is over the line
    T = nb * block - block // 3
    max_pages = -(-T // page) if page else 0
    g = torch.Generator(device="cuda").manual_seed(block)
    B, step = 2, max(1, 256 // Hkv - 5)                   # two sequences: below the line
    dims = (B * max_pages, page, Hkv, d) if page else (B, T, Hkv, d)
    K = torch.randn(*dims, generator=g, device="cuda").to(dt)
    table = torch.randperm(B * max_pages, generator=g, device="cuda").to(torch.int32).view(B, max_pages) if page else None
    lens = torch.tensor([T, T - 3 * block - 1], dtype=torch.int32, device="cuda")
    shape = S.make_shape(B=B, gamma=1, Hq=Hkv, Hkv=Hkv, d=d, dtype=dtype, block_size=block, max_seq_len=T, k_blocks=1, k_pool=K,
                         page_size=page, max_pages_per_seq=max_pages)
    for minmax, out in ((False, torch.float32), (True, torch.float32), (True, torch.bfloat16)):
        rule = S.SvfRetrieval(S.SVF_SUMMARY_MINMAX if minmax else S.SVF_SUMMARY_MEAN, S.SVF_BF16 if out == torch.bfloat16 else S.SVF_F32,
                              0, 0, 0)
        rows = (2,) if minmax else ()
        whole = torch.full((B, Hkv, nb, *rows, d), -7.0, device="cuda", dtype=out)
        few = whole.clone()
        S.svf_block_summaries(shape, rule, K, table, lens, whole)
        for first in range(0, nb, step):
            S.svf_block_summaries(shape, rule, K, table, lens, few, first, min(step, nb - first))
        torch.cuda.synchronize()
        assert torch.equal(whole.view(torch.uint8), few.view(torch.uint8)), (minmax, out)
        assert bool((few[1, :, nb - 2:].float() == -7.0).all())        # blocks that do not exist stay as they were
