"""Times of calls whose kernels are chosen by size, against each other: on either side of a choice more work must
not cost out of proportion.  Every bound lies well inside what separates the right choice from the wrong one."""
import pytest
import torch

import paper_2512_21911_amd as S

pytestmark = pytest.mark.gpu


def us_per_call(call, calls=20):
    """Best of several replays of a graph of `calls` calls."""
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        call()
    torch.cuda.current_stream().wait_stream(side)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        for _ in range(calls):
            call()
    graph.replay()
    times = []
    for _ in range(9):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        graph.replay()
        b.record()
        torch.cuda.synchronize()
        times.append(a.elapsed_time(b) * 1e3 / calls)
    return min(times)


def us_per_retrieval(B, Hkv, nb, total=0):
    g = torch.Generator(device="cuda").manual_seed(nb)
    summaries = torch.randn(B, Hkv, nb, 128, generator=g, device="cuda")
    q = torch.randn(B, 1, Hkv, 128, generator=g, device="cuda")
    k = min(nb, total) if total else 32
    shape = S.make_shape(B=B, gamma=1, Hq=Hkv, Hkv=Hkv, d=128, dtype="f32", block_size=16, max_seq_len=nb * 16, k_blocks=k,
                         kv_strides=(nb * 16 * Hkv * 128, Hkv * 128, 128))
    rule = S.SvfRetrieval(S.SVF_SUMMARY_MEAN, S.SVF_F32, S.SVF_GROUP_MEAN, S.SVF_BUDGET_GLOBAL if total else S.SVF_BUDGET_PER_HEAD, total)
    lens = torch.full((B,), nb * 16, dtype=torch.int32, device="cuda")
    idx = torch.zeros(B, Hkv, k, dtype=torch.int32, device="cuda")
    cnt = torch.zeros(B, Hkv, dtype=torch.int32, device="cuda")
    ws = S.new_workspace(shape)
    return us_per_call(lambda: S.svf_retrieve(shape, rule, q, summaries, lens, idx, cnt, ws))


def test_one_budget_over_an_eighth_more_pairs():
    """8192 pairs are selected from in the launch that scores, 9216 behind it.  (16 and 21 us a call; 37 where
    the scores are read again in every pass.)"""
    assert us_per_retrieval(1, 8, 1152, 256) < 1.7 * us_per_retrieval(1, 8, 1024, 256)


def test_retrieval_of_eight_times_the_heads():
    """256 workgroups score and select in one launch, 2048 only score.  (9 and 30 us a call; 57 in one launch.)"""
    assert us_per_retrieval(16, 8, 2048) < 4.5 * us_per_retrieval(2, 8, 2048)


def test_expert_skipping_of_one_expert_more():
    """16 lanes per token up to 16 experts, 32 behind that.  (65 536 tokens: 6.5 us a call and, with
    broadcasts through LDS, 24.)"""
    def us(k):
        w = torch.rand(65536, k, generator=torch.Generator().manual_seed(k)).cuda()
        beta = torch.full((k - 1,), 0.5, device="cuda")
        n, keep = (torch.zeros(65536, dtype=torch.int32, device="cuda") for _ in range(2))
        return us_per_call(lambda: S.svf_moe_skip(w, 3, beta, n, keep))
    assert us(17) < 2.5 * us(16)


class Attention:
    """Attention over lists of kept blocks, full ones or about half of that, unevenly."""

    def __init__(self, B, Hkv, G, gamma, d, k, T=16384, block=64):
        g = torch.Generator(device="cuda").manual_seed(1)
        self.K, self.V = (torch.randn(B, T, Hkv, d, generator=g, device="cuda", dtype=torch.bfloat16) for _ in range(2))
        self.q, self.kd, self.vd = (torch.randn(B, gamma, h, d, generator=g, device="cuda", dtype=torch.bfloat16)
                                    for h in (Hkv * G, Hkv, Hkv))
        self.lens = torch.full((B,), T, dtype=torch.int32, device="cuda")
        self.shape = S.make_shape(B=B, gamma=gamma, Hq=Hkv * G, Hkv=Hkv, d=d, dtype="bf16", block_size=block, max_seq_len=T,
                                  k_blocks=k, k_pool=self.K)
        self.out, self.ws = torch.empty_like(self.q), S.new_workspace(self.shape)
        self.size = B, Hkv, k, T // block

    def us(self, uneven=False):
        B, Hkv, k, nb = self.size
        r = torch.Generator().manual_seed(2)
        idx = torch.full((B, Hkv, k), -1, dtype=torch.int32)
        cnt = torch.full((B, Hkv), k, dtype=torch.int32)
        if uneven:
            w = torch.empty(B, Hkv).exponential_(1.0, generator=r) + 0.1
            cnt = (w / w.mean(dim=1, keepdim=True) * k / 2).round().clamp(1, k).to(torch.int32)
        for b in range(B):
            for h in range(Hkv):
                c = int(cnt[b, h])
                idx[b, h, :c] = torch.randperm(nb, generator=r)[:c].sort().values
        idx, cnt = idx.cuda(), cnt.cuda()
        return us_per_call(lambda: S.svf_verify_attn(self.shape, self.q, self.K, self.V, None, self.lens, self.kd, self.vd, None,
                                                     idx, cnt, self.out, self.ws))


def test_attention_over_half_of_what_was_planned():
    """Lists that hold half of the planned blocks, unevenly, take no longer than full ones.  (96 pairs of 1024 tokens: 18.4
    and 19.9 us a call; 21 to 22 with fewer shares than there are workgroups.)"""
    a = Attention(B=12, Hkv=8, G=4, gamma=8, d=128, k=16)
    assert a.us(uneven=True) < 1.02 * a.us()


@pytest.mark.parametrize("d", [64, 128])
def test_attention_of_half_as_many_pairs_more(d):
    """16 pairs are a workgroup for every compute unit, 24 are 11 splits each, of which an XCD holds 10.  (D = 64: 10.6 and
    13.2 us a call, 20.2 with 11 splits; D = 128: 13.1 and 17.9, 34.)"""
    assert Attention(B=3, Hkv=8, G=4, gamma=8, d=d, k=64).us() < 1.6 * Attention(B=2, Hkv=8, G=4, gamma=8, d=d, k=64).us()
