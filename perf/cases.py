"""Performance cases of libsvf: what a speculative-decoding server has the library do.

Kinds of pass (the field "kind" of a case):

  step      a slice of the layers of one verification step: svf_verify_step for every layer, with
            retrieval on anchor layers and the anchor's blocks on the layers behind it.  "graph":
            the server replays a captured HIP graph (as bench.py does), otherwise it makes the
            calls.  "append": before an anchor layer the representatives of the last blocks are
            brought up to date, as after the tokens of the step before were added to the cache.
  prefill   block representatives or summaries of whole caches, as after a prompt was read.
  variant   retrieval with another rule (svf_retrieve: min/max or bf16 summaries, maximum over the
            query heads, one budget over all KV heads) and attention over what it kept.
  ffn       the sparse feed-forward layer for the tokens of a step.
  rules     the per-token rules of a step: expert skipping in every mixture-of-experts layer, then
            acceptance and resampling of the drafts.

Offline calibration (analytics, threshold maps) runs once per model and is not among them.
"""
from __future__ import annotations

import math
import random

import torch

import paper_2512_21911_amd as S

DT = {"f32": torch.float32, "bf16": torch.bfloat16}
SHIFT = 1.5                 # length of the shift that makes a planted block's keys match the first query
PLANTED = 0.05              # share of a sequence's blocks that are planted
ACCEPT_RATE = 0.7           # share of draft tokens accepted, for the bytes of a rules pass


# ---- the cases -------------------------------------------------------------------------------------

def _step(name=None, *, dtype="bf16", B, Hq=32, Hkv=8, d=128, T, min_len=0, block=64, page=16, gamma, tree=False, k,
          layers, every, n_sink=0, n_local=0, graph=False, append=False, lse=False):
    c = dict(kind="step", dtype=dtype, B=B, Hq=Hq, Hkv=Hkv, d=d, T=T, min_len=min_len or T, block=block, page=page,
             gamma=gamma, tree=tree, k=k, layers=layers, every=every, n_sink=n_sink, n_local=n_local, graph=graph,
             append=append, lse=lse)
    return dict(c, name=name) if name else c


def _prefill(name=None, *, dtype="bf16", B, Hkv=8, d=128, T, min_len=0, block=64, page=16, minmax=False,
             out="f32", layers=1):
    c = dict(kind="prefill", dtype=dtype, B=B, Hkv=Hkv, d=d, T=T, min_len=min_len or T, block=block, page=page,
             minmax=minmax, out=out, layers=layers)
    return dict(c, name=name) if name else c


def _variant(name=None, *, B, Hq=32, Hkv=8, d=128, T, min_len=0, block=64, page=16, gamma, k, minmax, out, gmax,
             total=False, layers=2):
    c = dict(kind="variant", dtype="bf16", B=B, Hq=Hq, Hkv=Hkv, d=d, T=T, min_len=min_len or T, block=block, page=page,
             gamma=gamma, tree=False, k=k, minmax=minmax, out=out, gmax=gmax, total=total, layers=layers)
    return dict(c, name=name) if name else c


def _ffn(name=None, *, M, d_model, d_ff, tau, act="silu", bias=False, gate_first=False, active=False, layers=1):
    c = dict(kind="ffn", M=M, d_model=d_model, d_ff=d_ff, tau=tau, act=act, bias=bias, gate_first=gate_first,
             active=active, layers=layers)
    return dict(c, name=name) if name else c


def _rules(name=None, *, B, gamma, V, experts=8, skip=3, layers=4):
    c = dict(kind="rules", B=B, gamma=gamma, V=V, experts=experts, skip=skip, layers=layers)
    return dict(c, name=name) if name else c


def listed():
    return [
        # one short fp32 sequence, head dimension 64: what a correctness run or a tiny model asks for;
        # every launch and every microsecond of the host path shows
        _step("step_1k_f32", dtype="f32", B=1, Hq=8, Hkv=2, d=64, T=1024, block=16, page=0, gamma=4, k=8, layers=2,
              every=2),
        # one user with an 8k context, contiguous cache, calls made layer by layer
        _step("step_8k", B=1, T=8192, page=0, gamma=5, k=16, layers=4, every=2, append=True),
        # the headline: four users with 32k contexts, paged cache, 8 drafts, 2k-token budget
        _step("step_32k_b4", B=4, T=32768, gamma=8, k=32, layers=8, every=2, graph=True),
        # one user with a 128k context and a 16-node draft tree
        _step("step_128k_tree16", B=1, T=131072, block=128, page=64, gamma=16, tree=True, k=32, layers=4, every=2),
        # a batch of eight of different lengths over four KV heads, anchors every fourth layer
        _step("step_64k_varlen_b8", B=8, Hkv=4, T=65536, min_len=16384, gamma=6, k=32, layers=8, every=4, graph=True),
        # a 60-node draft tree over the headline's cache: 240 query rows per KV head
        _step("step_32k_tree60", B=4, T=32768, gamma=60, tree=True, k=32, layers=4, every=2, graph=True),
        # head dimension 64, ragged lengths, first and last blocks always kept, log-sum-exp asked for
        _step("step_16k_d64_ragged", B=3, d=64, T=15999, min_len=5000, gamma=7, k=24, n_sink=1, n_local=2, layers=4,
              every=2, lse=True),
        # a batch of 32k prompts has been read: mean keys of all their blocks, two anchor layers
        _prefill("prefill_32k_b4", B=4, T=32768, min_len=24000, layers=2),
        # min/max summaries in bf16, maximum over the query heads, one budget over all KV heads
        _variant("variant_global_32k", B=4, T=32768, gamma=8, k=32, minmax=True, out="bf16", gmax=True, total=True),
        # the feed-forward layer of an 8B model for 8 drafts
        _ffn("ffn_8b_m8", M=8, d_model=4096, d_ff=14336, tau=0.05),
        # the same under a 60-node draft tree, with biases and the active sets asked for
        _ffn("ffn_8b_m60", M=60, d_model=4096, d_ff=14336, tau=0.05, bias=True, active=True),
        # 64 sequences of four drafts over a 129 280-token vocabulary, 8 experts per token
        _rules("rules_b64", B=64, gamma=4, V=129280),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _draw_step(rng):
    if rng.random() < 0.15:                              # fp32: small models and correctness runs
        B, T, gamma = rng.choice((1, 2)), _log_int(rng, 700, 8000), rng.randint(1, 8)
        block = rng.choice((16, 32))
        Hq, Hkv = rng.choice(((8, 2), (4, 4), (16, 4)))
        return _step(dtype="f32", B=B, Hq=Hq, Hkv=Hkv, d=rng.choice((64, 128)), T=T, min_len=rng.choice((0, T // 2)),
                     block=block, page=rng.choice((0, 16)), gamma=gamma, k=rng.randint(4, 512 // block),
                     layers=rng.choice((1, 2)), every=2, graph=rng.random() < 0.3)
    B = _log_int(rng, 1, 8)
    T = _log_int(rng, 1500, min(131072, 400000 // B))
    d = 128 if rng.random() < 0.75 else 64
    Hq, Hkv = rng.choice(((32, 8), (32, 8), (32, 4), (40, 8), (28, 4), (64, 8), (16, 16)))
    block = rng.choice((32, 64, 64, 128))
    tree = rng.random() < 0.35
    gamma = _log_int(rng, 6, 64) if tree else _log_int(rng, 1, 12)
    ragged = B > 1 and rng.random() < 0.6
    n_sink, n_local = rng.choice(((0, 0), (0, 0), (1, 1), (1, 2)))
    page = rng.choice((0, 16, 16, 64)) if block != 32 else rng.choice((0, 16, 32))
    return _step(B=B, Hq=Hq, Hkv=Hkv, d=d, T=T, min_len=T // 4 if ragged else 0, block=block, page=page, gamma=gamma,
                 tree=tree, k=max(4, _log_int(rng, 256, 4096) // block),
                 layers=rng.choice((2, 4, 6, 8)), every=rng.choice((1, 2, 2, 4)), n_sink=n_sink, n_local=n_local,
                 graph=rng.random() < 0.5, append=not ragged and rng.random() < 0.4, lse=rng.random() < 0.25)


def _draw_prefill(rng):
    B = _log_int(rng, 1, 8)
    T = _log_int(rng, 2000, min(131072, 200000 // B))
    return _prefill(B=B, Hkv=rng.choice((4, 8, 8, 16)), d=rng.choice((128, 128, 64)), T=T, min_len=rng.choice((0, T // 3)),
                    block=rng.choice((32, 64, 64, 128)), page=rng.choice((0, 16, 32)), minmax=rng.random() < 0.4,
                    out=rng.choice(("f32", "bf16")), layers=rng.choice((1, 2)))


def _draw_variant(rng):
    B = _log_int(rng, 1, 4)
    T = _log_int(rng, 4000, 65536 // B * 2)
    minmax, out, gmax, total = rng.random() < 0.6, rng.choice(("f32", "bf16")), rng.random() < 0.5, rng.random() < 0.5
    Hq, Hkv = rng.choice(((32, 8), (32, 4), (64, 8)))
    return _variant(B=B, Hq=Hq, Hkv=Hkv, T=T, min_len=rng.choice((0, T // 2)), block=rng.choice((32, 64, 64, 128)),
                    page=rng.choice((0, 16)), gamma=rng.randint(1, 8), k=_log_int(rng, 8, 40), minmax=minmax, out=out,
                    gmax=gmax, total=total, layers=rng.choice((1, 2)))


def _draw_ffn(rng):
    d_model, d_ff = 128 * _log_int(rng, 8, 40), 32 * _log_int(rng, 16, 512)
    layers = rng.randint(1, 8)
    return _ffn(M=_log_int(rng, 1, 64), d_model=d_model, d_ff=d_ff, tau=rng.choice((0.0, 0.01, 0.05, 0.1)),
                act=rng.choice(("silu", "silu", "gelu")), bias=rng.random() < 0.3, gate_first=rng.random() < 0.15,
                active=rng.random() < 0.4, layers=layers)


def _draw_rules(rng):
    experts = rng.choice((2, 4, 8, 8))
    V = rng.choice((32000, 50257, 128256, 129280, 151936 - rng.randrange(999)))
    return _rules(B=_log_int(rng, 1, 64), gamma=rng.randint(1, 4), V=V,
                  experts=experts, skip=rng.randint(1, min(3, experts - 1)), layers=rng.randint(1, 4))


def _cost(case):
    w = work(case)
    return max(w["bytes"], w["flops"] / 50)


def draw(rng: random.Random):
    """One more case.  A draw that costs more than the largest listed case of its kind is drawn again."""
    make = rng.choices((_draw_step, _draw_prefill, _draw_variant, _draw_ffn, _draw_rules), (10, 2, 2, 4, 2))[0]
    most = None
    while True:
        c = make(rng)
        if most is None:
            most = max(_cost(x) for x in listed() if x["kind"] == c["kind"])
        if _cost(c) <= most and (c.get("d") != 64 or c["kind"] != "step" or _vector_cost(c) <= 1.0):
            return c


def _vector_cost(c):
    """Arithmetic of a step at head dimension 64, in units of the listed step of that head dimension."""
    def of(x):
        return x["layers"] * x["B"] * x["Hq"] * x["gamma"] * (x["k"] * x["block"] + x["gamma"])
    return of(c) / of(next(x for x in listed() if x["name"] == "step_16k_d64_ragged"))


# ---- inputs ----------------------------------------------------------------------------------------

def _lens(case, seed):
    r = random.Random(seed * 7919 + 11)
    return [r.randint(case["min_len"], case["T"]) for _ in range(case["B"])]


def _tree_masks(gamma, seed):
    """Ancestor-or-self masks of a random tree: a chain of up to six nodes, then random shallower parents."""
    r = random.Random(seed * 7919 + 13)
    depth, masks = [0], [1]
    for i in range(1, gamma):
        p = i - 1 if i <= 6 else r.choice([j for j in range(i) if depth[j] < 6])
        depth.append(depth[p] + 1)
        masks.append(masks[p] | (1 << i))
    return torch.tensor([m - (1 << 64) if m >> 63 else m for m in masks], dtype=torch.int64).cuda()


class _Cache:
    """Page table, pools of `layers` layers and the queries; keys of planted blocks lean towards the first query."""

    def __init__(self, case, seed, with_values):
        dev, dt = "cuda", DT[case["dtype"]]
        g = torch.Generator(device=dev).manual_seed(seed)
        B, Hkv, d, T, block, page = (case[x] for x in ("B", "Hkv", "d", "T", "block", "page"))
        lens = _lens(case, seed)
        self.lens = torch.tensor(lens, dtype=torch.int32).to(dev)
        self.nb_max = -(-T // block)
        r = random.Random(seed * 7919 + 19)
        if page:
            used = [-(-n // page) for n in lens]
            max_pages = -(-T // page)
            perm = torch.randperm(sum(used), generator=g, device=dev).to(torch.int32)
            self.table = torch.zeros(B, max_pages, dtype=torch.int32, device=dev)
            at = 0
            for b, u in enumerate(used):
                self.table[b, :u] = perm[at:at + u]
                at += u
            dims = (sum(used), page, Hkv, d)
        else:
            self.table, max_pages, dims = None, 0, (B, T, Hkv, d)
        self.max_pages = max_pages

        def randn(*shape):
            return torch.randn(*shape, generator=g, device=dev, dtype=torch.float32).to(dt)

        if "Hq" in case:
            Hq, gamma, G = case["Hq"], case["gamma"], case["Hq"] // Hkv
            # (b, h, planted block)
            planted = [(b, h, sorted(r.sample(range(-(-n // block)), int(PLANTED * -(-n // block))))) for b, n in enumerate(lens)
                       for h in range(Hkv)]
            tok = [[b, h, j] for b, h, js in planted for j in js]
            tok = torch.tensor(tok, dtype=torch.int64).to(dev).view(-1, 3)
        self.q, self.k_draft, self.v_draft, self.K, self.V = [], [], [], [], []
        for _ in range(case["layers"]):
            K = torch.randn(*dims, generator=g, device=dev, dtype=dt)
            self.K.append(K)
            if with_values:
                self.V.append(torch.randn(*dims, generator=g, device=dev, dtype=dt))
            if "Hq" not in case:
                continue
            q = randn(B, gamma, Hq, d)
            self.q.append(q)
            self.k_draft.append(randn(B, gamma, Hkv, d))
            self.v_draft.append(randn(B, gamma, Hkv, d))
            if tok.numel():
                q0 = q[:, 0].float().view(B, Hkv, G, d).mean(dim=2)
                u = (SHIFT * q0 / q0.norm(dim=-1, keepdim=True)).to(dt)
                t = tok[:, 2:] * block + torch.arange(block, device=dev)                     # [planted][block]
                b, h = (x.expand_as(t) for x in (tok[:, :1], tok[:, 1:2]))
                ok = t < self.lens.long()[b]
                b, h, t = b[ok], h[ok], t[ok]
                at = (self.table[b, t // page].long(), t % page, h) if page else (b, t, h)
                K[at] += u[b, h]

    def shape(self, case, k_blocks, **kw):
        return S.make_shape(B=case["B"], gamma=case.get("gamma", 1), Hq=case.get("Hq", case["Hkv"]), Hkv=case["Hkv"], d=case["d"],
                            dtype=case["dtype"], block_size=case["block"], max_seq_len=case["T"], k_blocks=k_blocks,
                            k_pool=self.K[0], page_size=case["page"], max_pages_per_seq=self.max_pages, **kw)


def _selection(case, k_blocks):
    return (torch.full((case["B"], case["Hkv"], k_blocks), -1, dtype=torch.int32, device="cuda"),
            torch.zeros(case["B"], case["Hkv"], dtype=torch.int32, device="cuda"))


def _prepare_step(case, seed):
    c = _Cache(case, seed, True)
    shape = c.shape(case, case["k"], n_sink=case["n_sink"], n_local=case["n_local"])
    s = dict(case=case, cache=c, shape=shape, ws=S.new_workspace(shape),
             mask=_tree_masks(case["gamma"], seed) if case["tree"] else None, reps=[], sel=[],
             out=[torch.empty_like(q) for q in c.q],
             lse=[torch.zeros(case["B"], case["gamma"], case["Hq"], device="cuda") if case["lse"] else None for _ in c.q])
    for layer in range(case["layers"]):
        anchor = layer % case["every"] == 0
        s["reps"].append(torch.zeros(case["B"], case["Hkv"], c.nb_max, case["d"], device="cuda") if anchor else None)
        s["sel"].append(_selection(case, case["k"]) if anchor else s["sel"][-1])
        if anchor:
            S.svf_block_reps(shape, c.K[layer], c.table, c.lens, s["reps"][layer])
    s["graph"] = None
    if case["graph"]:
        side = torch.cuda.Stream()
        side.wait_stream(torch.cuda.current_stream())
        with torch.cuda.stream(side):
            _run_step(s)
        torch.cuda.current_stream().wait_stream(side)
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            _run_step(s)
        s["graph"] = graph
    return s


def _tail(case):
    """First block and number of blocks that the tokens of one step can touch."""
    first = max(0, (case["T"] - case["gamma"]) // case["block"])
    return first, -(-case["T"] // case["block"]) - first


def _run_step(s):
    case, c = s["case"], s["cache"]
    for layer in range(case["layers"]):
        idx, cnt = s["sel"][layer]
        reps = s["reps"][layer]
        if reps is not None and case["append"]:
            S.svf_block_reps(s["shape"], c.K[layer], c.table, c.lens, reps, *_tail(case))
        S.svf_verify_step(s["shape"], S.SVF_STEP_ANCHOR if reps is not None else S.SVF_STEP_REUSE_GATHER, c.q[layer], reps,
                          c.K[layer], c.V[layer], c.table, c.lens, c.k_draft[layer], c.v_draft[layer], s["mask"], idx, cnt,
                          s["out"][layer], s["ws"], lse=s["lse"][layer])
    return None


def _prepare_prefill(case, seed):
    c = _Cache(case, seed, False)
    rows = (2,) if case["minmax"] else ()
    return dict(case=case, cache=c, shape=c.shape(case, 1),
                rule=S.SvfRetrieval(S.SVF_SUMMARY_MINMAX if case["minmax"] else S.SVF_SUMMARY_MEAN,
                                    S.SVF_BF16 if case["out"] == "bf16" else S.SVF_F32, 0, 0, 0),
                out=[torch.zeros(case["B"], case["Hkv"], c.nb_max, *rows, case["d"], device="cuda", dtype=DT[case["out"]])
                     for _ in c.K])


def _prepare_variant(case, seed):
    c = _Cache(case, seed, True)
    total = case["k"] * case["Hkv"]
    k_blocks = min(c.nb_max, total) if case["total"] else case["k"]
    rule = S.SvfRetrieval(S.SVF_SUMMARY_MINMAX if case["minmax"] else S.SVF_SUMMARY_MEAN,
                          S.SVF_BF16 if case["out"] == "bf16" else S.SVF_F32,
                          S.SVF_GROUP_MAX if case["gmax"] else S.SVF_GROUP_MEAN,
                          S.SVF_BUDGET_GLOBAL if case["total"] else S.SVF_BUDGET_PER_HEAD, total if case["total"] else 0)
    shape = c.shape(case, k_blocks)
    s = dict(case=case, cache=c, shape=shape, rule=rule, ws=S.new_workspace(shape), summaries=[],
             sel=[_selection(case, k_blocks) for _ in c.K], out=[torch.empty_like(q) for q in c.q])
    rows = (2,) if case["minmax"] else ()
    for K in c.K:
        sm = torch.zeros(case["B"], case["Hkv"], c.nb_max, *rows, case["d"], device="cuda", dtype=DT[case["out"]])
        S.svf_block_summaries(shape, rule, K, c.table, c.lens, sm)
        s["summaries"].append(sm)
    return s


def _prepare_ffn(case, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    dm, df, M = case["d_model"], case["d_ff"], case["M"]

    def randn(*shape, dtype=torch.float32):
        return torch.randn(*shape, generator=g, device="cuda", dtype=dtype)

    shape = S.make_ffn_shape(M=M, d_model=dm, d_ff=df, act=case["act"], tau=case["tau"],
                             walk=S.SVF_FFN_WALK_GATE_FIRST if case["gate_first"] else S.SVF_FFN_WALK_AUTO)
    s = dict(case=case, shape=shape, ws=S.new_ffn_workspace(shape), layers=[])
    for _ in range(case["layers"]):
        # a gate row's scale is log-normal: quiet channels are quiet for all tokens, and the thresholds leave
        # out 18 %, 47 % and 64 % of a token's channels at 0.01, 0.05 and 0.1
        scale = torch.exp(-1.6 + 1.5 * randn(df, 1))
        s["layers"].append(dict(
            x=randn(M, dm).to(torch.bfloat16),
            w_gate=(randn(df, dm, dtype=torch.bfloat16) * (scale / dm ** 0.5)).to(torch.bfloat16),
            w_up=randn(df, dm, dtype=torch.bfloat16) * dm ** -0.5, w_down_t=randn(df, dm, dtype=torch.bfloat16) * df ** -0.5,
            b_gate=randn(df) * 0.02 if case["bias"] else None, b_up=randn(df) * 0.1 if case["bias"] else None,
            b_down=randn(dm) * 0.1 if case["bias"] else None,
            y=torch.zeros(M, dm, device="cuda", dtype=torch.bfloat16),
            active=torch.zeros(df, dtype=torch.int64, device="cuda") if case["active"] else None))
    return s


def _prepare_rules(case, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    B, gamma, V, k = case["B"], case["gamma"], case["V"], case["experts"]

    def randn(*shape):
        return torch.randn(*shape, generator=g, device="cuda")

    def routing(T):
        logits = randn(T, 256) * torch.exp(0.5 * randn(T, 1))
        w = torch.softmax(torch.topk(logits, k, dim=1).values, dim=1)
        order = torch.argsort(torch.rand(T, k, generator=g, device="cuda"), dim=1)
        return torch.gather(w, 1, order).contiguous()

    lt = 3.0 * randn(B, gamma, V)
    pt, pd = torch.softmax(lt, -1), torch.softmax(lt + 0.7 * randn(B, gamma, V), -1)
    tok = torch.multinomial(pd.reshape(-1, V), 1, generator=g).reshape(B, gamma).to(torch.int32)
    s = dict(case=case, pt=pt, pd=pd, tok=tok, ua=torch.rand(B, gamma, generator=g, device="cuda"),
             ur=torch.rand(B, generator=g, device="cuda"), n=torch.zeros(B, dtype=torch.int32, device="cuda"),
             resampled=torch.zeros(B, dtype=torch.int32, device="cuda"), layers=[])
    for _ in range(case["layers"]):
        beta = torch.zeros(k - 1, device="cuda")
        S.svf_moe_calibrate(routing(1024), beta)
        T = B * gamma
        s["layers"].append((routing(T), beta, torch.zeros(T, dtype=torch.int32, device="cuda"),
                            torch.zeros(T, dtype=torch.int32, device="cuda")))
    return s


def prepare(case, seed):
    return {"step": _prepare_step, "prefill": _prepare_prefill, "variant": _prepare_variant, "ffn": _prepare_ffn,
            "rules": _prepare_rules}[case["kind"]](case, seed)


# ---- one pass --------------------------------------------------------------------------------------

def run(s):
    case = s["case"]
    kind = case["kind"]
    if kind == "step":
        if s["graph"] is not None:
            s["graph"].replay()
        else:
            _run_step(s)
        return [s["out"], s["sel"], s["lse"]]
    if kind == "prefill":
        c = s["cache"]
        for K, out in zip(c.K, s["out"]):
            if case["minmax"] or case["out"] != "f32":
                S.svf_block_summaries(s["shape"], s["rule"], K, c.table, c.lens, out)
            else:
                S.svf_block_reps(s["shape"], K, c.table, c.lens, out)
        return s["out"]
    if kind == "variant":
        c = s["cache"]
        for i, (idx, cnt) in enumerate(s["sel"]):
            S.svf_retrieve(s["shape"], s["rule"], c.q[i], s["summaries"][i], c.lens, idx, cnt, s["ws"])
            S.svf_verify_attn(s["shape"], c.q[i], c.K[i], c.V[i], c.table, c.lens, c.k_draft[i], c.v_draft[i], None, idx, cnt,
                              s["out"][i], s["ws"])
        return [s["out"], s["sel"]]
    if kind == "ffn":
        for x in s["layers"]:
            S.svf_sparse_ffn(s["shape"], x["x"], x["w_gate"], x["w_up"], x["w_down_t"], x["y"], s["ws"], b_gate=x["b_gate"],
                             b_up=x["b_up"], b_down=x["b_down"], active=x["active"])
        return [(x["y"], x["active"]) for x in s["layers"]]
    for w, beta, n_skip, keep in s["layers"]:
        S.svf_moe_skip(w, case["skip"], beta, n_skip, keep)
    S.svf_accept_resample(s["pt"], s["pd"], s["tok"], s["ua"], s["ur"], s["n"], s["resampled"])
    return [s["n"], s["resampled"]] + [(n, k) for _, _, n, k in s["layers"]]


# ---- what a pass cannot do without -----------------------------------------------------------------

def _attention_work(case, tokens):
    """One layer over `tokens` kept tokens per KV head and sequence (a mean)."""
    e = DT[case["dtype"]].itemsize
    B, Hq, Hkv, d, gamma = (case[x] for x in ("B", "Hq", "Hkv", "d", "gamma"))
    n = 2 * B * Hkv * tokens * d * e                                # selected keys and values
    n += 2 * B * gamma * (Hkv + Hq) * d * e                         # draft keys and values, queries, output
    n += B * Hkv * tokens / case["block"] * 4                       # block ids
    n += B * tokens / case["page"] * 4 if case["page"] else 0       # page table entries
    return n, 4.0 * B * gamma * Hq * (tokens + gamma / 2) * d


def work(case):
    kind = case["kind"]
    if kind in ("step", "prefill", "variant"):
        B, Hkv, d, block = (case[x] for x in ("B", "Hkv", "d", "block"))
        e = DT[case["dtype"]].itemsize
        mean_len = (case["min_len"] + case["T"]) / 2
        nb = mean_len / block
    if kind == "step":
        n, f = _attention_work(case, min(case["k"], nb) * block)
        anchors = -(-case["layers"] // case["every"])
        a = B * Hkv * nb * d * 4 + B * case["Hq"] * d * e           # representatives, the first draft's queries
        if case["append"]:
            a += B * Hkv * _tail(case)[1] * (block * d * e + d * 4)
        return {"bytes": case["layers"] * n + anchors * a, "flops": case["layers"] * f + anchors * 2.0 * B * Hkv * nb * d}
    if kind == "prefill":
        rows = 2 if case["minmax"] else 1
        return {"bytes": case["layers"] * B * Hkv * (mean_len * d * e + nb * rows * d * DT[case["out"]].itemsize),
                "flops": float(case["layers"] * B * Hkv * mean_len * d)}
    if kind == "variant":
        n, f = _attention_work(case, min(case["k"], nb) * block)
        rows = 2 if case["minmax"] else 1
        n += B * Hkv * nb * rows * d * DT[case["out"]].itemsize + B * case["Hq"] * d * e
        return {"bytes": case["layers"] * n, "flops": case["layers"] * (f + 2.0 * rows * B * case["Hq"] * nb * d)}
    if kind == "ffn":
        M, dm, df = case["M"], case["d_model"], case["d_ff"]
        # share of the channels that some token keeps (the scales above; more tokens keep more)
        kept = {0.0: 1.0, 0.01: 0.97, 0.05: 0.8, 0.1: 0.66}[case["tau"]]
        n = df * dm * 2 * (1 + 2 * kept) + 2 * M * dm * 2 + (df * 8 if case["active"] else 0)
        return {"bytes": case["layers"] * n, "flops": case["layers"] * 2.0 * M * df * dm * (1 + 2 * kept)}
    B, gamma, V, k = case["B"], case["gamma"], case["V"], case["experts"]
    # the rejected position's two distributions, for the sequences that have one
    n = B * (1 - ACCEPT_RATE ** gamma) * 2 * V * 4 + B * gamma * 16
    n += case["layers"] * B * gamma * (k * 4 + 8)
    return {"bytes": n, "flops": 2.0 * n / 4}


def tolerance(case):
    # whole numbers (kept blocks, skip masks, tokens): near-ties may fall either way
    if case["kind"] == "rules":
        return {"differ": 0.005}
    if case["kind"] == "prefill":
        return {"rel": 1e-5 if case["out"] == "f32" else 1e-2}      # fp32 sums of a bf16 cache
    if case["kind"] == "step" and case["dtype"] == "f32":
        return {"rel": 1e-5, "differ": 0.001}
    return {"rel": 1e-2, "differ": 0.001}
