"""The kept blocks of an anchor layer where the selection changes its ways: numbers of blocks around a wavefront's keys,
around the most that every workgroup scores for itself and every wavefront selects from (128), budgets from one
block to all, and scores that are exact, so that the expected set is (many ties, one value, neighbours in fp32, forced blocks)."""
import numpy as np
import pytest
import torch

import paper_2512_21911_amd as S

pytestmark = pytest.mark.gpu

BLOCK = 16


def scores_of(kind, rng, shape):
    if kind == "spread":
        return rng.permutation(int(np.prod(shape))).reshape(shape).astype(np.float32) - 300.0
    if kind == "few_values":
        return rng.integers(-2, 3, shape).astype(np.float32)
    if kind == "one_value":
        return np.full(shape, -3.0, np.float32)
    return (1.0 + rng.integers(0, 40, shape) * 2.0 ** -23).astype(np.float32)      # "neighbours": the same first bytes


@pytest.mark.parametrize("dtype,d", [("bf16", 128), ("bf16", 64), ("f32", 64), ("f32", 128)])
@pytest.mark.parametrize("nb", [1, 63, 64, 65, 127, 128, 129, 257, 513, 700])
def test_kept_blocks(nb, dtype, d):
    rng = np.random.default_rng(nb * 131 + d)
    B, Hkv, gamma = 2, 2, 2
    dt = torch.float32 if dtype == "f32" else torch.bfloat16
    T = nb * BLOCK
    K = torch.zeros(B, T, Hkv, d, device="cuda", dtype=dt)
    q = torch.zeros(B, gamma, Hkv, d, device="cuda", dtype=dt)
    q[:, 0, :, 5] = 1.0                                  # score = channel 5 of the representative
    kd = torch.zeros(B, gamma, Hkv, d, device="cuda", dtype=dt)
    lens = torch.tensor([T, max(1, T - 7 * BLOCK - 3)], dtype=torch.int32, device="cuda")
    for k in sorted({1, 2, max(1, nb // 3), max(1, nb - 1), nb}):
        for kind in ("spread", "few_values", "one_value", "neighbours"):
            n_sink, n_local = (1, 1) if k > 2 and kind != "spread" else (0, 0)
            shape = S.make_shape(B=B, gamma=gamma, Hq=Hkv, Hkv=Hkv, d=d, dtype=dtype, block_size=BLOCK, max_seq_len=T, k_blocks=k,
                                 k_pool=K, page_size=0, max_pages_per_seq=0, n_sink=n_sink, n_local=n_local)
            value = scores_of(kind, rng, (B, Hkv, nb))
            reps = torch.zeros(B, Hkv, nb, d, device="cuda")
            reps[..., 5] = torch.from_numpy(value).cuda()
            idx = torch.full((B, Hkv, k), -7, dtype=torch.int32, device="cuda")
            cnt = torch.full((B, Hkv), -7, dtype=torch.int32, device="cuda")
            out, ws = torch.empty_like(q), S.new_workspace(shape)
            for _ in range(2):                           # (the second call on a workspace that has been used)
                S.svf_verify_step(shape, S.SVF_STEP_ANCHOR, q, reps, K, K, None, lens, kd, kd, None, idx, cnt, out, ws)
            got, n = idx.cpu().numpy(), cnt.cpu().numpy()
            for b in range(B):
                own = -(-int(lens[b]) // BLOCK)
                for h in range(Hkv):
                    v = value[b, h, :own].astype(np.float64)
                    v[:n_sink] = np.inf
                    if n_local:
                        v[own - min(n_local, own):] = np.inf
                    want = np.sort(np.argsort(-v, kind="stable")[:min(k, own)])
                    assert n[b, h] == len(want), (k, kind, b, h)
                    assert np.array_equal(got[b, h, :len(want)], want), (k, kind, b, h)
                    assert (got[b, h, len(want):] == -1).all()
