"""Representatives of a few blocks (one workgroup per head) give the bits of a launch over all blocks
(one workgroup per block): heads, channels, types, block sizes around the stage, partial last blocks.
TAKES: shapes of which launches of two blocks take the kernel for few blocks, at the edges of what it is made
for (odd numbers of token lanes, blocks just past a whole trip, a full stage, the last that pays), also
against the oracle.  The other sets lie on either side of the rule that chooses it."""
import numpy as np
import pytest
import torch

import paper_2512_21911_amd as S
from oracle import svf_oracle as O

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,Hkv,d,block,page", [
    ("bf16", 8, 128, 64, 16), ("bf16", 4, 128, 128, 0), ("bf16", 1, 64, 32, 32), ("bf16", 3, 128, 16, 16), ("bf16", 16, 64, 7, 7),
    ("bf16", 1, 64, 256, 64), ("bf16", 2, 128, 129, 0), ("f32", 2, 64, 16, 0), ("f32", 1, 128, 64, 16), ("f32", 5, 64, 33, 0),
])
def test_few_blocks_same_bits(dtype, Hkv, d, block, page):
    few_against_all(dtype, Hkv, d, block, page, max(1, 256 // Hkv - 5))          # two sequences: below the line


TAKES = [("bf16", 3, 128, 33, 33), ("bf16", 3, 128, 32, 32), ("bf16", 16, 64, 23, 23), ("bf16", 8, 128, 127, 127),
         ("bf16", 8, 128, 128, 16), ("bf16", 16, 128, 31, 0), ("bf16", 5, 64, 96, 32), ("bf16", 32, 64, 13, 13),
         ("bf16", 12, 64, 255, 0), ("bf16", 6, 128, 40, 0), ("f32", 3, 64, 33, 33), ("f32", 8, 128, 64, 0),
         ("f32", 7, 64, 127, 0)]


@pytest.mark.parametrize("dtype,Hkv,d,block,page", TAKES)
def test_few_blocks_against_all_and_oracle(dtype, Hkv, d, block, page):
    few_against_all(dtype, Hkv, d, block, page, 2, oracle=True)


def few_against_all(dtype, Hkv, d, block, page, step, oracle=False):
    dt = torch.float32 if dtype == "f32" else torch.bfloat16
    nb = 512 // Hkv + 3                                   # a launch over all of them is over the line
    T = nb * block - block // 3
    max_pages = -(-T // page) if page else 0
    g = torch.Generator(device="cuda").manual_seed(block)
    B = 2
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
        if oracle and not minmax:
            ref = O.block_reps(K.cpu(), table.cpu() if page else None, lens.cpu(), block, nb)
            got = few.double().cpu().numpy()
            for b, n in ((0, nb), (1, nb - 3)):
                # n fp32 additions, each off by 2^-24 of a partial sum (below 80 here), divided by n: 5e-6
                assert np.abs(got[b, :, :n] - ref[b, :, :n]).max() <= 2e-5
