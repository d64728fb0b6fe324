"""The work a rollout asks of this library, as cases that can be timed and compared.

A case is a dict: what is called (`kind`: a decode step, a prefill chunk, a scoring chunk), the policy's shape and how
many of its layers (a slice of `layers` layers with the whole vocabulary; the per-layer work is that of the full depth),
the 16-bit format, the number of sequences, how many of them share a prompt, the cached positions per sequence and the
new tokens per sequence.  Lengths are spread evenly from lo to hi over the sequences, in a shuffled order that the case
alone decides; weights, token ids and cache contents come from the seed.
"""
import math
import random

import torch

import paper_2604_11554_amd as pkg
import rollout_inputs as RI

DENSE, MOE, TINY = RI.QWEN3_4B.name, RI.QWEN3_30B_A3B.name, RI.TINY_DENSE.name
DTYPES = {"bf16": torch.bfloat16, "f16": torch.float16}
DEV = "cuda:0"


def _case(name, kind, shape, layers, seqs, ctx, new=(1, 1), group=1, fmt="bf16"):
    c = dict(kind=kind, shape=shape, layers=layers, fmt=fmt, seqs=seqs, group=group, ctx_lo=ctx[0], ctx_hi=ctx[1],
             new_lo=new[0], new_hi=new[1])
    return dict(c, name=name) if name else c


def listed():
    return [
        # the smallest call: four sequences of the two-layer policy, everything in caches, launches and latency
        _case("decode_tiny_b4", "decode", TINY, 2, 4, (17, 95)),
        # the tail of a rollout: one long response left, weights read for a single token
        _case("decode_4b_b1", "decode", DENSE, 8, 1, (3001, 3001)),
        # the dense batch at full depth, in the middle of its decode phase (prompts 256..1024, half of 1024 tokens out)
        _case("decode_4b_b64", "decode", DENSE, 36, 64, (769, 1535)),
        # the FP16 option on a batch that is no multiple of a tile
        _case("decode_4b_f16_b45", "decode", DENSE, 8, 45, (301, 2003), fmt="f16"),
        # sampling groups: 32 prompts x 8 responses that share the prompt's pages
        _case("decode_4b_group_b256", "decode", DENSE, 8, 256, (517, 2048), group=8),
        # the MoE batch in the middle of its decode phase: every expert is read
        _case("decode_30b_b128", "decode", MOE, 4, 128, (1530, 1530)),
        # a few agentic sessions with long contexts: a part of the experts is read
        _case("decode_30b_b12", "decode", MOE, 4, 12, (2900, 6900)),
        # prompt intake of the dense batch in one large call
        _case("prefill_4b_32k", "prefill", DENSE, 4, 51, (0, 0), new=(257, 1021)),
        # continuous refill: the prompts of three freed slots
        _case("prefill_4b_refill", "prefill", DENSE, 8, 3, (0, 0), new=(257, 701)),
        # prompt intake of the MoE batch
        _case("prefill_30b_16k", "prefill", MOE, 4, 32, (0, 0), new=(512, 512)),
        # a turn of agentic sessions: 128 tool tokens each on top of what is cached
        _case("turn_30b_b16", "prefill", MOE, 4, 16, (2900, 6900), new=(128, 128)),
        # log-probabilities of finished responses with their routing replayed
        _case("score_30b_4k", "score", MOE, 4, 8, (0, 0), new=(411, 637)),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["decode", "decode", "decode", "decode", "group", "prefill", "prefill", "prefill", "turn", "score"])
    shape = rng.choice([DENSE, DENSE, MOE])
    fmt = "f16" if rng.random() < 0.15 else "bf16"
    if kind == "decode":
        if rng.random() < 0.1:
            return _case(None, "decode", TINY, 2, _log(rng, 1, 8), (rng.randint(3, 40), rng.randint(41, 99)), fmt=fmt)
        seqs = _log(rng, 1, 256)
        hi = _log(rng, 64, min(8000, 400000 // seqs))
        return _case(None, "decode", shape, 8 if shape == DENSE else 4, seqs, (max(1, int(hi * rng.uniform(0.3, 1.0))), hi),
                     fmt=fmt)
    if kind == "group":
        group, hi = rng.choice([2, 4, 8]), rng.randint(600, 2048)
        return _case(None, "decode", DENSE, 8, group * _log(rng, 1, 256 // group), (rng.randint(200, 599), hi), group=group,
                     fmt=fmt)
    if kind == "turn":
        seqs, new, hi = _log(rng, 2, 48), rng.randint(33, 160), rng.randint(1000, 6900)
        return _case(None, "prefill", MOE, 4, seqs, (int(hi * rng.uniform(0.4, 1.0)), hi), new=(new, new), fmt=fmt)
    total = _log(rng, 100, 28000 if kind == "prefill" and shape == DENSE else (16000 if kind == "prefill" else 4500))
    seqs = max(1, min(64, total // rng.randint(100, 1000)))
    mean = max(2, total // seqs)
    lo = max(1, int(mean * rng.uniform(0.4, 1.0)))
    return _case(None, kind, shape, 4, seqs, (0, 0), new=(lo, 2 * mean - lo), fmt=fmt)


def _shape(case):
    return RI.SHAPES[case["shape"]].replace(n_layers=case["layers"])


def _spread(lo, hi, n, salt):
    v = [lo + (hi - lo) * i // max(1, n - 1) for i in range(n)]
    random.Random(n * 7919 + lo * 31 + hi + salt).shuffle(v)
    return v


def _lengths(case):
    """(shared prompt positions, cached positions, new tokens) of every sequence."""
    n, g = case["seqs"], case["group"]
    ctx = [c for c in _spread(case["ctx_lo"], case["ctx_hi"], n // g, 1) for _ in range(g)]
    own = _spread(1, 255, n, 3) if g > 1 else [0] * n      # response tokens a group's member has emitted
    return ctx, [c + o for c, o in zip(ctx, own)], _spread(case["new_lo"], case["new_hi"], n, 2)


def _tensor(s, seed, fmt):
    """tensor(layer, name) of the policy: matrices N(0, 0.02), gains 1 + N(0, 0.02), router rows N(0, 1/d)."""
    gen = torch.Generator(device=DEV)

    def tensor(layer, name):
        dims, kind = RI.tensor_names(s, layer)[name]
        gen.manual_seed((seed * 1000003 + (layer + 1) * 101 + sum(map(ord, name))) & 0x7FFFFFFF)
        t = torch.empty(dims, device=DEV, dtype=torch.float32)
        t.normal_(1.0 if kind == "gain" else 0.0, s.d_model ** -0.5 if kind == "router" else 0.02, generator=gen)
        return t.to(DTYPES[fmt])

    return tensor


def _inputs(case, seed):
    """Host token ids per sequence, the tokens that follow them, the experts to replay, and the generator of the cache."""
    s = _shape(case)
    gen = torch.Generator().manual_seed(seed + 1)
    _, _, new = _lengths(case)
    total = sum(new)
    ids = torch.randint(0, s.vocab - 2, (2, total), generator=gen, dtype=torch.int32)
    replay = None
    if case["kind"] == "score" and s.is_moe:
        replay = torch.rand((total, s.n_layers, s.n_experts), generator=gen).topk(s.top_k, dim=-1).indices.to(torch.int32)
    return ids[0], ids[1], replay, torch.Generator(device=DEV).manual_seed(seed + 2)


def _pages(case):
    """First page and number of pages of every sequence's own run (a group's members list the leader's full prompt pages
    and then their own), and the number of pages in all."""
    prompt, ctx, new = _lengths(case)
    first, count, at = [], [], 0
    for i in range(case["seqs"]):
        n = (ctx[i] + new[i] + 15) // 16 - (prompt[i] // 16 if i % case["group"] else 0)
        if i % case["group"] == 0 and case["group"] > 1:
            n = max(n, (prompt[i] + 16) // 16)
        first.append(at)
        count.append(n)
        at += n
    return first, count, at


def _fill(pool, s, n_blocks, fmt, gen):
    """Cached keys and values: unit-variance elements, as normalised keys and projected values have."""
    pool.view(DTYPES[fmt]).normal_(generator=gen)
    return pool.view(DTYPES[fmt]).view(s.n_layers, n_blocks, s.n_kv_heads, 2, 16 * s.head_dim)


def prepare(case, seed):
    s = _shape(case)
    model = pkg.RolloutModel(_config(s, case["fmt"]), _tensor(s, seed, case["fmt"]), DEV)
    prompt, ctx, new = _lengths(case)
    ids, target, replay, gen = _inputs(case, seed)
    n, g = case["seqs"], case["group"]
    first, count, n_blocks = _pages(case)
    widest = max(prompt[i] // 16 + count[i] if i % g else count[i] for i in range(n))
    eng = pkg.RolloutEngine(model, n_blocks=n_blocks, max_seqs=n, max_chunk_tokens=sum(new), max_blocks_per_seq=widest)
    for i in range(n):
        if i % g == 0:
            eng.add_sequence(2000 + i, reserve_tokens=16 * count[i])
            eng.ctx_lens[i] = prompt[i]
        else:
            eng.fork(i - i % g, 2000 + i, reserve_tokens=16 * (prompt[i] // 16 + count[i]))
    if max(ctx) > 0:
        _fill(eng.kv_pool, s, n_blocks, case["fmt"], gen)
    ctx_dev = torch.tensor(ctx, dtype=torch.int32, device=DEV)
    eng.ctx_lens.copy_(ctx_dev)
    st = dict(engine=eng, ctx=ctx_dev, kind=case["kind"], moe=s.is_moe, pool=eng.kv_pool.view(DTYPES[case["fmt"]]))
    if case["kind"] == "decode":
        # the step consumes `ids` and emits `target`: forcing the emitted token keeps its log-probability comparable
        st["tokens"], st["forced"] = ids.to(DEV), target.to(DEV)
        return st
    cuts = [0]
    for x in new:
        cuts.append(cuts[-1] + x)
    per = lambda t: [t[a:b].numpy() for a, b in zip(cuts, cuts[1:])]  # noqa: E731
    st["rows"], st["toks"], st["targets"] = list(range(n)), per(ids), per(target)
    st["forced"] = [int(t[-1]) for t in st["targets"]]
    st["replay"] = None if replay is None else per(replay)
    return st


def run(state):
    eng = state["engine"]
    eng.ctx_lens.copy_(state["ctx"])             # the step before this one, again
    if state["kind"] == "decode":
        eng.tokens.copy_(state["tokens"])
        out = eng.decode_step(forced=state["forced"], want_logits=True, want_routing=state["moe"])
        return dict(logits=out.logits, logprobs=out.logprobs, routing=out.routing, ctx_lens=eng.ctx_lens)
    if state["kind"] == "prefill":
        out = eng.prefill(state["rows"], state["toks"], forced=state["forced"], want_logits=True,
                          want_routing=state["moe"])
        return dict(logits=out.logits, logprobs=out.logprobs, routing=out.routing, kv=state["pool"])
    logprobs, _ = eng.score(state["rows"], state["toks"], state["targets"], replay_routing=state["replay"])
    return dict(logprobs=logprobs, kv=state["pool"])


def work(case):
    s = _shape(case)
    prompt, ctx, new = _lengths(case)
    T, g = sum(new), case["group"]
    proj = s.d_model * (2 * s.q_dim + 2 * s.kv_dim)
    expert = 3 * s.d_model * (s.d_ff_expert if s.is_moe else s.d_ff)
    read, used = expert, expert
    if s.is_moe:                                 # experts that T tokens with top_k distinct ones each reach
        reached = s.n_experts * (1 - (1 - s.top_k / s.n_experts) ** T)
        read, used = reached * expert + s.n_experts * s.d_model, s.top_k * expert + s.n_experts * s.d_model
    rows = T if case["kind"] == "score" else case["seqs"]
    kv_tok = 4 * s.n_layers * s.kv_dim
    cached = sum(ctx) - sum(p // 16 * 16 for i, p in enumerate(prompt) if i % g)     # shared pages are read once
    keys = sum(n * c + n * (n + 1) // 2 for n, c in zip(new, ctx))
    nbytes = 2 * (s.n_layers * (proj + read) + s.vocab * s.d_model) + kv_tok * (cached + T) + 2 * T * s.d_model
    nbytes += 4 * T if case["kind"] == "score" else 4 * rows * s.vocab
    flops = 2 * T * s.n_layers * (proj + used) + 2 * rows * s.vocab * s.d_model + 4 * s.n_layers * s.q_dim * keys
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    """About four times the distance to exact() of the library as it stood when the cases were written (relative 2-norm):
    dense decode 4e-5 (36 layers) with two bf16 terms per activation and 1.6e-3 with one fp16 term; cached keys and values
    1e-3, a 16-bit store being one unit off where a sum comes in another order, and the logits that read them 4.5e-4.
    Without a replayed routing a MoE token at a tie may take either of two experts: 4e-3 on the logits of a prefill,
    with single rows that differ by a sizeable part of their root mean square."""
    if _shape(case).is_moe and case["kind"] != "score":
        return {"rel": 1.5e-2 if case["fmt"] == "bf16" else 3e-2, "max": 0.9, "differ": 0.01}
    if case["fmt"] == "f16":
        return {"rel": 7e-3, "max": 0.1}
    return {"rel": 2e-4, "max": 5e-3} if case["kind"] == "decode" else {"rel": 5e-3, "max": 0.1}


def _config(s, fmt):
    # two 16-bit terms per activation with bf16, one with fp16: the library's two settings
    return dict(dtype=0 if fmt == "bf16" else 1, activation_split=1 if fmt == "bf16" else 0, n_layers=s.n_layers,
                d_model=s.d_model, n_q_heads=s.n_q_heads, n_kv_heads=s.n_kv_heads, head_dim=s.head_dim, d_ff=s.d_ff,
                n_experts=s.n_experts, top_k=s.top_k, d_ff_expert=s.d_ff_expert, vocab=s.vocab,
                kv_block_size=s.kv_block_size, rms_eps=s.rms_eps, rope_theta=s.rope_theta, qk_norm=int(s.qk_norm),
                eos_token_id=s.eos_token_id, pad_token_id=s.pad_token_id)


def exact(case, seed):
    """The same outputs in 64 bits.  Keys and values are rounded to 16 bits where the cache stores them, which is part of
    the computation; nothing else is.  Where a MoE policy routes by itself its cache has no exact value: a token at
    a tie may rightly take either expert, and its keys in the layers above follow."""
    s, fmt = _shape(case), case["fmt"]
    f64, dt = torch.float64, DTYPES[case["fmt"]]
    tensor = _tensor(s, seed, fmt)
    W = lambda l, n: tensor(l, n).to(f64)  # noqa: E731
    prompt, ctx, new = _lengths(case)
    ids, target, replay, gen = _inputs(case, seed)
    n, g, hd, H, KV = case["seqs"], case["group"], s.head_dim, s.n_q_heads, s.n_kv_heads
    first, count, n_blocks = _pages(case)
    pool = torch.zeros(s.n_layers * n_blocks * KV * 2 * 16 * hd * 2, dtype=torch.uint8, device=DEV)
    pages = pool.view(dt).view(s.n_layers, n_blocks, KV, 2, 16 * hd)
    if max(ctx) > 0:
        _fill(pool, s, n_blocks, fmt, gen)
    table = []                                   # pages of every sequence
    for i in range(n):
        shared = prompt[i] // 16 if i % g else 0
        lead = first[i - i % g]
        table.append(torch.tensor(list(range(lead, lead + shared)) + list(range(first[i], first[i] + count[i])),
                                  device=DEV))
    cuts = [0]
    for x in new:
        cuts.append(cuts[-1] + x)
    pos = torch.cat([torch.arange(c, c + m, device=DEV) for c, m in zip(ctx, new)]).to(f64)
    freq = s.rope_theta ** (-2.0 * torch.arange(hd // 2, device=DEV, dtype=f64) / hd)
    cos, sin = torch.cos(pos[:, None] * freq)[:, None], torch.sin(pos[:, None] * freq)[:, None]

    def norm(x, gain):
        return x / torch.sqrt((x * x).mean(-1, keepdim=True) + s.rms_eps) * gain

    def rope(x):
        a, b = x[..., :hd // 2], x[..., hd // 2:]
        return torch.cat([a * cos - b * sin, b * cos + a * sin], -1)

    h = tensor(-1, "embed")[ids.to(DEV).long()].to(f64)
    T = h.shape[0]
    for l in range(s.n_layers):
        x = norm(h, W(l, "attn_norm"))
        q, k, v = ((x @ W(l, w).t()).view(T, -1, hd) for w in ("wq", "wk", "wv"))
        if s.qk_norm:
            q, k = norm(q, W(l, "q_norm")), norm(k, W(l, "k_norm"))
        q, k, v = rope(q), rope(k).to(dt), v.to(dt)
        o = torch.empty(T, H, hd, device=DEV, dtype=f64)
        for i in range(n):
            a, b, end = cuts[i], cuts[i + 1], ctx[i] + new[i]
            at = torch.arange(ctx[i], end, device=DEV)
            pg, slot = table[i][at // 16], at % 16
            pages[l].view(n_blocks, KV, 2, 16, hd)[pg, :, 0, slot] = k[a:b]
            pages[l].view(n_blocks, KV, 2, hd, 16)[pg, :, 1, :, slot] = v[a:b]
            own = pages[l][table[i][:(end + 15) // 16]]
            K = own[:, :, 0].view(-1, KV, 16, hd).transpose(0, 1).reshape(KV, -1, hd)[:, :end].to(f64)
            V = own[:, :, 1].view(-1, KV, hd, 16).permute(1, 0, 3, 2).reshape(KV, -1, hd)[:, :end].to(f64).contiguous()
            Q = q[a:b].view(b - a, KV, H // KV, hd).permute(1, 2, 0, 3).reshape(KV, -1, hd)
            z = (Q @ K.transpose(1, 2).contiguous()).view(KV, H // KV, b - a, end) / math.sqrt(hd)
            z.masked_fill_(torch.arange(end, device=DEV) > at[:, None], float("-inf"))
            y = torch.softmax(z, -1).view(KV, -1, end) @ V
            o[a:b] = y.view(KV, H // KV, b - a, hd).permute(2, 0, 1, 3).reshape(b - a, H, hd)
        h = h + o.view(T, -1) @ W(l, "wo").t()
        x = norm(h, W(l, "ffn_norm"))
        if not s.is_moe:
            h = h + (torch.nn.functional.silu(x @ W(l, "w_gate").t()) * (x @ W(l, "w_up").t())) @ W(l, "w_down").t()
            continue
        z = x @ W(l, "w_router").t()
        pick = z.topk(s.top_k, -1).indices if replay is None else replay[:, l].to(DEV).long()
        weight = torch.softmax(z.gather(1, pick), -1)
        wg, wu, wd = tensor(l, "w_gate"), tensor(l, "w_up"), tensor(l, "w_down")
        for e in range(s.n_experts):
            t, j = (pick == e).nonzero(as_tuple=True)
            if t.numel():
                u = torch.nn.functional.silu(x[t] @ wg[e].to(f64).t()) * (x[t] @ wu[e].to(f64).t())
                h.index_add_(0, t, weight[t, j, None] * (u @ wd[e].to(f64).t()))
    x = norm(h, W(-1, "final_norm"))
    head = W(-1, "lm_head").t().contiguous()
    kv = None if s.is_moe and replay is None else pages.reshape(-1)
    wanted = target.to(DEV).long()
    if case["kind"] == "score":
        lp = []
        for a in range(0, T, 512):
            z = x[a:a + 512] @ head
            lp.append(z.gather(1, wanted[a:a + 512, None])[:, 0] - torch.logsumexp(z, -1))
        return dict(logprobs=torch.cat(lp), kv=kv)
    last = torch.tensor([c - 1 for c in cuts[1:]], device=DEV)
    z = x[last] @ head
    lp = z.gather(1, wanted[last][:, None])[:, 0] - torch.logsumexp(z, -1)
    out = dict(logits=z, logprobs=lp, routing=None)
    return dict(out, ctx_lens=None) if case["kind"] == "decode" else dict(out, kv=kv)
