"""The selection inside the retrieval launch (svf_retrieve, svf_score_select with scores asked for) at the edges of
its key counts: one and several keys per thread, the most one workgroup holds and one more (the general path), many
equal scores on both sides of the threshold, forced blocks, empty and one-block sequences.  The query picks channel 0
of the representatives, whole numbers, so the scores are exact and the kept blocks are a stable sort's."""
import numpy as np
import pytest
import torch

import paper_2512_21911_amd as S

pytestmark = pytest.mark.gpu

BLOCK = 4


def run(lens, Hkv, nb_max, k, total, levels, n_sink=0, n_local=0, dtype="f32", d=64, G=2, seed=0):
    g = torch.Generator().manual_seed(seed)
    B = len(lens)
    values = torch.randint(-levels, levels + 1, (B, Hkv, nb_max), generator=g).float()
    reps = torch.zeros(B, Hkv, nb_max, d)
    reps[..., 0] = values
    reps[..., 1:] = torch.randint(-3, 4, (B, Hkv, nb_max, d - 1), generator=g).float()     # the query is zero there
    t = torch.float32 if dtype == "f32" else torch.bfloat16
    q = torch.zeros(B, 1, Hkv * G, d, dtype=t)
    q[..., 0] = 1
    K = torch.zeros(1, BLOCK, Hkv, d, dtype=t, device="cuda")
    k_blocks = min(nb_max, total) if total else k
    shape = S.make_shape(B=B, gamma=1, Hq=Hkv * G, Hkv=Hkv, d=d, dtype=dtype, block_size=BLOCK, max_seq_len=nb_max * BLOCK,
                         k_blocks=k_blocks, n_sink=n_sink, n_local=n_local, k_pool=K, page_size=BLOCK, max_pages_per_seq=nb_max)
    rule = S.SvfRetrieval(S.SVF_SUMMARY_MEAN, S.SVF_F32, S.SVF_GROUP_MEAN, S.SVF_BUDGET_GLOBAL if total else S.SVF_BUDGET_PER_HEAD, total)
    idx = torch.full((B, Hkv, k_blocks), -7, dtype=torch.int32, device="cuda")
    cnt = torch.full((B, Hkv), -7, dtype=torch.int32, device="cuda")
    scores = torch.full((B, Hkv, nb_max), float("nan"), device="cuda")
    ws = S.new_workspace(shape)
    sl = torch.tensor(lens, dtype=torch.int32, device="cuda")
    first = None
    for _ in range(2):                                    # (the second call finds the counters as the first left them)
        S.svf_retrieve(shape, rule, q.cuda(), reps.cuda(), sl, idx, cnt, ws, scores=scores)
        torch.cuda.synchronize()
        now = (idx.cpu().numpy().copy(), cnt.cpu().numpy().copy())
        assert first is None or all(np.array_equal(a, b) for a, b in zip(first, now))
        first = now
    idx, cnt = first
    scores = scores.cpu().numpy()
    for b, L in enumerate(lens):
        nb = -(-L // BLOCK)
        assert np.array_equal(scores[b, :, :nb], values[b, :, :nb].numpy())
        assert (scores[b, :, nb:] == 0).all()
        key = values[b, :, :nb].numpy().copy()
        key[:, :n_sink] = np.inf
        key[:, max(nb - n_local, 0):] = np.inf
        keep = np.zeros_like(key, dtype=bool)
        if total:
            keep.reshape(-1)[np.argsort(-key.reshape(-1), kind="stable")[:total]] = True
        else:
            for h in range(Hkv):
                keep[h, np.argsort(-key[h], kind="stable")[:k]] = True
        for h in range(Hkv):
            want = np.flatnonzero(keep[h])
            assert cnt[b, h] == len(want), (b, h)
            assert np.array_equal(idx[b, h, :len(want)], want), (b, h)
            assert (idx[b, h, len(want):] == -1).all()


@pytest.mark.parametrize("nb", [1, 63, 64, 65, 128, 129, 1023, 1024, 1025, 2048, 4100, 8192, 8193])
@pytest.mark.parametrize("levels", [2, 100000])
def test_per_head(nb, levels):
    for k in sorted({1, min(nb, 32), nb}):
        run([nb * BLOCK, 0, max(1, nb * BLOCK // 2 - 1)], 2, nb, k, 0, levels, seed=nb + k)


@pytest.mark.parametrize("Hkv,nb", [(1, 100), (8, 1), (3, 77), (8, 128), (5, 205), (16, 512), (2, 4096), (2, 4097), (256, 32), (257, 3)])
@pytest.mark.parametrize("levels", [1, 100000])
def test_all_heads(Hkv, nb, levels):
    for total in sorted({1, min(Hkv * nb, 250), Hkv * nb, Hkv * nb + 9}):
        run([nb * BLOCK, 0, max(1, nb * BLOCK // 3)], Hkv, nb, 0, total, levels, G=1, seed=nb + total)


@pytest.mark.parametrize("nb", [3, 40, 1030, 8200])
def test_forced_blocks(nb):
    run([nb * BLOCK, BLOCK, 2 * BLOCK], 2, nb, max(4, min(nb, 20)), 0, 3, n_sink=1, n_local=2, dtype="bf16", d=128)
    run([nb * BLOCK, BLOCK], 2, nb, 0, 50, 3, n_sink=2, n_local=1, d=128)
