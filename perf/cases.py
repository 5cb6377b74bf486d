"""Performance cases of the PEFT-BD speculative step on one GPU.

What a program does with this framework is decode with it: it builds a context
over a model's weights, prefills prompts, and then repeats draft, verify and
accept.  The cases are those calls, from one short sequence to a batch of long
ones.  Each runs at the layer shape of one of the two models of this repository
(the tiny fp32 decoder, Qwen3-0.6B in bf16), over the whole stack of layers or
over its first ``layers`` (one layer's kernels repeat down the stack, and the
largest batches then fit the time and memory of a measurement).

A case is a dict of
  model   "tiny" or "qwen"             layers  depth of the stack
  call    "round"      draft, verify, accept       (every output fp32-exact enough to return tokens)
          "denoise"    two-step draft               (as above)
          "draft"      adapter-on bidirectional block draft
          "verify"     adapter-off causal verify and greedy acceptance
          "unanchored" the unanchored draft and verify pair
          "prefill"    a prompt's prefill and the verify of the first block after it
  batch, lo, hi   sequences, and the range their prefix (prompt) lengths are drawn from
  block, rank     D and the LoRA rank (alpha = 2 rank)
  chunk           prompt rows per prefill pass ("prefill" only; 0: the library's default)
  graph           the call is replayed from a HIP graph, as a serving loop does

bf16 models return logits and not the token ids: random weights leave top-2
gaps of the order of the rounding, so that ids flip between two equally good
implementations.  For the same reason the verified block and its anchor are
given (drawn from the seed) instead of taken from the draft before.
"""
import math

import torch

import synth
from paper_2607_12422_amd import Engine

DEV = "cuda:0"
LINEARS = ("q", "k", "v", "o", "gate", "up", "down")


def listed():
    q = dict(model="qwen", layers=28, block=16, rank=16, chunk=0, graph=True)
    return [
        # smallest calls: the tiny decoder's whole round, launched call by call
        dict(name="tiny_round_b1_p128", model="tiny", layers=2, call="round", batch=1, lo=128, hi=128,
             block=16, rank=8, chunk=0, graph=False),
        # interactive decoding of one sequence, the benchmark's default workload (draft half)
        dict(q, name="draft_b1_p512", call="draft", batch=1, lo=512, hi=512),
        # the generation loop at a long prefix (verify half and the commit)
        dict(q, name="verify_b1_p4096", call="verify", batch=1, lo=4096, hi=4096),
        # the unanchored-drafting ablation, one sequence
        dict(q, name="unanchored_b1_p512", call="unanchored", batch=1, lo=512, hi=512, graph=False),
        # plain greedy decoding steps (block 0) of a batch: one row per sequence
        dict(q, name="greedy_b16_p256-1024", call="verify", batch=16, lo=256, hi=1024, block=0),
        # a small ragged batch
        dict(q, name="verify_b4_p256-2048", call="verify", batch=4, lo=256, hi=2048),
        # the ragged batch of 8 at rank 32, both halves of its step
        dict(q, name="draft_b8_p256-2048_r32", call="draft", batch=8, lo=256, hi=2048, rank=32),
        dict(q, name="verify_b8_p256-2048", call="verify", batch=8, lo=256, hi=2048, rank=32),
        # the largest batch: 32 long sequences, D = 32, rank 64, both halves of its step
        dict(q, name="draft_b32_p8192_r64", call="draft", batch=32, lo=8192, hi=8192, block=32, rank=64, layers=8),
        dict(q, name="verify_b32_p8192", call="verify", batch=32, lo=8192, hi=8192, block=32, rank=64, layers=8),
        # a prompt of ordinary length in one chunk, and a long one in several
        dict(q, name="prefill_b1_p512_c512", call="prefill", batch=1, lo=512, hi=512, chunk=512, graph=False),
        dict(q, name="prefill_b1_p4096_c1024", call="prefill", batch=1, lo=4096, hi=4096, chunk=1024, graph=False),
    ]


def _log(rng, lo, hi):
    """A whole number between lo and hi, uniform over its logarithm."""
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    if rng.random() < 0.15:
        hi = _log(rng, 4, 512)
        return dict(model="tiny", layers=2, call=rng.choice(["round", "denoise"]), batch=rng.randint(1, 4),
                    lo=rng.randint(max(1, hi // 2), hi), hi=hi, block=rng.randint(2, 24), rank=rng.choice([8, 16]),
                    chunk=0, graph=rng.random() < 0.5)
    call = rng.choice(["draft", "draft", "draft", "verify", "verify", "verify", "unanchored", "prefill"])
    if call == "prefill":
        batch = rng.choice([1, 1, 2, 4, 8])
        chunk = rng.choice([0, _log(rng, 24, 128), _log(rng, 128, 1024), _log(rng, 128, 1024)])
        chunk = min(chunk, 4096 // batch)
        hi = _log(rng, 32, 4096 // batch) if chunk >= 128 else _log(rng, 16, 128)
        return dict(model="qwen", layers=rng.choice([2, 4, 7, 14, 28]), call=call, batch=batch,
                    lo=rng.randint(max(1, hi // 2), hi), hi=hi, block=16, rank=16, chunk=chunk, graph=False)
    batch = _log(rng, 1, 32)
    hi = _log(rng, 16, 8192)
    layers = rng.choice([1, 2, 4, 7])
    if batch * hi <= 16384 and rng.random() < 0.4:
        layers = 28
    block = rng.choice([4, 7, 8, 15, 16, 16, 16, 24, 31, 32])
    if call == "verify" and rng.random() < 0.2:
        block = 0
    return dict(model="qwen", layers=layers, call=call, batch=batch, lo=rng.randint(max(1, hi // 4), hi), hi=hi,
                block=block, rank=rng.choice([8, 16, 16, 32, 64]), chunk=0, graph=rng.random() < 0.5)


def _config(case):
    base = synth.TINY if case["model"] == "tiny" else synth.QWEN3_0_6B
    return base.with_(n_layers=case["layers"], block=case["block"], lora_rank=case["rank"],
                      lora_alpha=2.0 * case["rank"])


def _generator(seed, stream):
    return torch.Generator(device=DEV).manual_seed(1000003 * int(seed) + stream)


def _weights(cfg, seed):
    """Random-init weights of the model's distributions (linears, embedding and
    LoRA N(0, 0.02), gains 1 + N(0, 0.02)) in its dtype, on the GPU."""
    g = _generator(seed, 0)
    dt = torch.bfloat16 if cfg.dtype == "bf16" else torch.float32

    def lin(o, i):
        return (torch.randn(o, i, generator=g, device=DEV) * 0.02).to(dt)

    def gain(n):
        return (1.0 + torch.randn(n, generator=g, device=DEV) * 0.02).to(dt)

    shapes = {n: (o, i) for n, o, i in cfg.linear_shapes()}
    layers = []
    for _ in range(cfg.n_layers):
        d = {n: lin(*shapes[n]) for n in LINEARS}
        d.update(attn_norm=gain(cfg.hidden), mlp_norm=gain(cfg.hidden), q_norm=gain(cfg.head_dim),
                 k_norm=gain(cfg.head_dim))
        d["lora"] = {n: (lin(cfg.lora_rank, shapes[n][1]), lin(shapes[n][0], cfg.lora_rank)) for n in LINEARS}
        layers.append(d)
    return {"embed": lin(cfg.vocab, cfg.hidden), "final_norm": gain(cfg.hidden), "layers": layers}


def _tokens(case, cfg, seed):
    """(lengths, prompts [B][hi], anchors [B], drafts [B][D], one unused column if D = 0): ids
    uniform below the mask id."""
    g = _generator(seed, 1)
    B = case["batch"]

    def ids(*shape):
        return torch.randint(0, cfg.vocab - 1, shape, generator=g, device=DEV, dtype=torch.int32)

    lengths = torch.randint(case["lo"], case["hi"] + 1, (B,), generator=g, device=DEV, dtype=torch.int32)
    return lengths, ids(B, case["hi"]), ids(B), ids(B, max(1, cfg.block))


def prepare(case, seed):
    cfg = _config(case)
    B, W, V = case["batch"], cfg.width, cfg.vocab
    lengths, prompts, anchor0, drafts = _tokens(case, cfg, seed)
    # room for 256 generated tokens; the prompt is prefilled in the largest chunks the batch allows
    chunk = case["chunk"] if case["call"] == "prefill" else min(1024, 4096 // B, max(W, case["hi"]))
    eng = Engine(cfg, _weights(cfg, seed), max_batch=B, max_seq=case["hi"] + 256 + 2 * W, device=DEV,
                 prefill_chunk=chunk)
    i32 = dict(dtype=torch.int32, device=DEV)
    f32 = dict(dtype=torch.float32, device=DEV)
    s = dict(case=case, cfg=cfg, eng=eng, lengths=lengths, prompts=prompts, anchor0=anchor0, drafts=drafts,
             seq=torch.zeros(B, **i32), anchor=torch.zeros(B, **i32), first=torch.zeros(B, **i32),
             draft=torch.zeros(B, cfg.block, **i32), verify=torch.zeros(B, W, **i32),
             n_acc=torch.zeros(B, **i32), out=torch.zeros(B, W, **i32), replay=None)
    call = case["call"]
    if call in ("round", "draft", "unanchored", "denoise"):
        s["dlog"] = torch.zeros(B, W, V, **f32)
    if call in ("round", "verify", "prefill"):
        s["vlog"] = torch.zeros(B, W, V, **f32)
    if call == "unanchored":
        s["vlog"] = torch.zeros(B, cfg.block, V, **f32)
    if call == "denoise":
        s["conf"] = torch.zeros(B, cfg.block, **f32)
        s["fixed"] = torch.zeros(B, cfg.block, **i32)
    if call != "prefill":
        eng.pbd_prefill(prompts, lengths, case["hi"], s["seq"], s["first"])
        s["anchor"].copy_(anchor0)
    if case["graph"]:
        torch.cuda.synchronize()
        side = torch.cuda.Stream()
        with torch.cuda.stream(side):
            _call(s)
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            s["outputs"] = _call(s)
        s["replay"] = graph
    return s


def _call(s):
    eng, call = s["eng"], s["case"]["call"]
    seq, anchor = s["seq"], s["anchor"]
    if call == "draft":
        eng.pbd_draft_block(seq, anchor, s["draft"], s["dlog"])
        return {"logits": s["dlog"]}
    if call == "denoise":
        eng.pbd_draft_block_denoise(seq, anchor, s["draft"], 2, s["conf"], s["fixed"], s["dlog"])
        return {"logits": s["dlog"], "draft": s["draft"], "conf": s["conf"], "fixed": s["fixed"]}
    if call == "unanchored":
        eng.pbd_draft_block_unanchored(seq, anchor, s["draft"], s["verify"], s["dlog"])
        eng.pbd_verify_block_unanchored(seq, s["drafts"], s["verify"], s["vlog"])
        return {"draft_logits": s["dlog"], "verify_logits": s["vlog"]}
    if call == "prefill":
        # the first block after the prompt reads every key and value the prefill wrote
        eng.pbd_prefill(s["prompts"], s["lengths"], s["case"]["hi"], seq, s["first"])
        eng.pbd_verify_block(seq, s["anchor0"], s["drafts"], s["verify"], s["vlog"])
        return {"logits": s["vlog"], "seq_len": seq}
    # a round or its verify half, then the commit; the state goes back to the
    # prefill's, so that every pass is the same step
    seq.copy_(s["lengths"])
    anchor.copy_(s["anchor0"])
    got = {"verify_logits": s["vlog"], "seq_len": seq, "n_accepted": s["n_acc"]}
    if call == "round":
        eng.pbd_draft_block(seq, anchor, s["draft"], s["dlog"])
        eng.pbd_verify_block(seq, anchor, s["draft"], s["verify"], s["vlog"])
        eng.pbd_accept_commit(s["draft"], s["verify"], seq, anchor, s["n_acc"], s["out"])
        got.update(draft_logits=s["dlog"], draft=s["draft"], verify=s["verify"], out_tokens=s["out"], anchor=anchor)
        return got
    eng.pbd_verify_block(seq, anchor, s["drafts"], s["verify"], s["vlog"])
    eng.pbd_accept_commit(s["drafts"], s["verify"], seq, anchor, s["n_acc"], s["out"])
    return got


def run(state):
    if state["replay"] is None:
        return _call(state)
    state["replay"].replay()
    return state["outputs"]


def work(case):
    cfg = _config(case)
    es = 2 if cfg.dtype == "bf16" else 4
    B, W, D, L = case["batch"], cfg.width, cfg.block, cfg.n_layers
    prefix = (case["lo"] + case["hi"]) / 2.0
    lin = L * sum(o * i for _, o, i in cfg.linear_shapes())
    lora = L * sum(cfg.lora_rank * (o + i) for _, o, i in cfg.linear_shapes())
    kv_row = L * 2 * cfg.n_kv_heads * cfg.head_dim * es
    att = 4 * L * cfg.n_q_heads * cfg.head_dim          # flops per (query row, key)
    head = cfg.vocab * cfg.hidden

    def block_pass(rows, adapter, keep):
        m = B * rows
        return (es * (lin + head + (lora if adapter else 0)) + B * prefix * kv_row + B * keep * kv_row + 4 * m * cfg.vocab,
                2 * m * (lin + head + (lora if adapter else 0)) + att * m * (prefix + rows / 2.0))

    call = case["call"]
    if call == "draft":
        parts = [block_pass(W, True, 0)]
    elif call == "denoise":
        parts = [block_pass(W, True, 0)] * 2
    elif call == "verify":
        parts = [block_pass(W, False, W)]
    elif call == "round":
        parts = [block_pass(W, True, 0), block_pass(W, False, W)]
    elif call == "unanchored":
        parts = [block_pass(W, True, 1), block_pass(D, False, D)]
    else:
        m = B * prefix
        parts = [(es * lin + m * kv_row, 2 * m * lin + att * m * prefix / 2.0), block_pass(W, False, W)]
    return {"bytes": float(sum(p[0] for p in parts)), "flops": float(sum(p[1] for p in parts))}


def tolerance(case):
    # measured against exact() over the listed and drawn cases: fp32 sums are
    # within 6e-7 (2-norm); bf16 passes round the cache, the attention weights
    # and their operands to 8 to 16 bits in every layer and are within 4e-3
    if case["model"] == "tiny":
        return {"rel": 3e-6, "max": 3e-5}
    return {"rel": 1.6e-2, "max": 1e-1}


# ---- the same calls in float64, plain torch ---------------------------------

def _rms(x, gain, eps):
    return x / torch.sqrt((x * x).mean(-1, keepdim=True) + eps) * gain


def _rope(v, pos, theta):
    half = v.shape[-1] // 2
    freq = theta ** (-(torch.arange(half, dtype=torch.float64, device=DEV) * 2.0) / v.shape[-1])
    ang = pos.double()[:, None] * freq[None, :]
    cos, sin = torch.cos(ang)[:, None, :], torch.sin(ang)[:, None, :]
    a, b = v[..., :half], v[..., half:]
    return torch.cat([a * cos - b * sin, b * cos + a * sin], -1)


class _Exact:
    """One sequence at a time; weights and cache in float64."""

    def __init__(self, cfg, w):
        self.cfg = cfg
        self.embed, self.final = w["embed"].double(), w["final_norm"].double()
        self.layers = []
        for lw in w["layers"]:
            d = {n: t.double() for n, t in lw.items() if n != "lora"}
            d["lora"] = {n: (a.double(), b.double()) for n, (a, b) in lw["lora"].items()}
            self.layers.append(d)

    def linear(self, lw, n, x, on):
        """on: rows [on:] take the adapter (None: none do)."""
        y = x @ lw[n].T
        if on is not None:
            a, b = lw["lora"][n]
            y[on:] += (self.cfg.lora_alpha / self.cfg.lora_rank) * ((x[on:] @ a.T) @ b.T)
        return y

    def block(self, tokens, pos0, cache, vis, on):
        """Hidden rows of a block at pos0.. over cache[l] = (K, V) [pos0][h][d]; vis[i]:
        the block rows row i sees are those below vis[i].  Returns (x, the block's K/V)."""
        cfg, n = self.cfg, tokens.shape[0]
        d, hq, hk = cfg.head_dim, cfg.n_q_heads, cfg.n_kv_heads
        pos = pos0 + torch.arange(n, device=DEV)
        x = self.embed[tokens.long()]
        new = []
        for li, lw in enumerate(self.layers):
            xn = _rms(x, lw["attn_norm"], cfg.rms_eps)
            q = self.linear(lw, "q", xn, on).view(n, hq, d)
            k = self.linear(lw, "k", xn, on).view(n, hk, d)
            v = self.linear(lw, "v", xn, on).view(n, hk, d)
            q = _rope(_rms(q, lw["q_norm"], cfg.rms_eps), pos, cfg.rope_theta)
            k = _rope(_rms(k, lw["k_norm"], cfg.rms_eps), pos, cfg.rope_theta)
            new.append((k, v))
            if cache is not None:
                k, v = torch.cat([cache[li][0], k]), torch.cat([cache[li][1], v])
            kt = k.permute(1, 2, 0).contiguous()
            vt = v.transpose(0, 1).contiguous()
            o = torch.empty(n, hq, d, dtype=torch.float64, device=DEV)
            col = torch.arange(n, device=DEV)
            for i in range(0, n, 512):
                qi = q[i:i + 512].reshape(-1, hk, hq // hk, d).permute(1, 2, 0, 3).reshape(hk, -1, d)
                sc = (qi @ kt).view(hk, hq // hk, -1, pos0 + n) / math.sqrt(d)
                sc[..., pos0:].masked_fill_(col[None, :] >= vis[i:i + 512, None], float("-inf"))
                p = torch.softmax(sc, -1).view(hk, -1, pos0 + n)
                o[i:i + 512] = (p @ vt).view(hk, hq // hk, -1, d).permute(2, 0, 1, 3).reshape(-1, hq, d)
            x = x + self.linear(lw, "o", o.reshape(n, hq * d), on)
            xm = _rms(x, lw["mlp_norm"], cfg.rms_eps)
            h = torch.nn.functional.silu(self.linear(lw, "gate", xm, on)) * self.linear(lw, "up", xm, on)
            x = x + self.linear(lw, "down", h, on)
        return x, new

    def logits(self, x):
        return _rms(x, self.final, self.cfg.rms_eps) @ self.embed.T

    def causal(self, n):
        return torch.arange(1, n + 1, device=DEV)


@torch.no_grad()
def exact(case, seed):
    cfg = _config(case)
    m = _Exact(cfg, _weights(cfg, seed))
    lengths, prompts, anchor0, drafts = _tokens(case, cfg, seed)
    B, W, D, mask = case["batch"], cfg.width, cfg.block, cfg.vocab - 1
    call = case["call"]
    rows = {}

    def keep(name, v):
        rows.setdefault(name, []).append(v)

    for b in range(B):
        t = int(lengths[b])
        _, cache = m.block(prompts[b, :t], 0, None, m.causal(t), None)
        anc = anchor0[b:b + 1]
        masks = torch.full((D,), mask, dtype=torch.int32, device=DEV)
        every = torch.full((W,), W, device=DEV)
        draft = drafts[b, :D]
        if call in ("round", "draft", "denoise"):
            y = torch.cat([anc, masks])
            lg = m.logits(m.block(y, t, cache, every, 0)[0])
            if call == "denoise":
                conf = torch.zeros(D, dtype=torch.float64, device=DEV)
                for step, n in ((1, D - D // 2), (2, D // 2)):
                    if step == 2:
                        lg = m.logits(m.block(y, t, cache, every, 0)[0])
                    lp = torch.log_softmax(lg[1:], -1)
                    lp[:, mask] = float("-inf")
                    c, tok = lp.max(-1)
                    c[y[1:] != mask] = float("-inf")
                    pick = torch.sort(c, descending=True, stable=True)[1][:n]
                    y[1 + pick], conf[pick] = tok[pick].int(), c[pick]
                keep("conf", conf)
            keep("draft_logits" if call == "round" else "logits", lg)
            if call == "round":
                lg = lg.clone()
                lg[:, mask] = float("-inf")
                draft = lg[1:].argmax(-1).int()
        if call in ("round", "verify", "prefill"):
            x, _ = m.block(torch.cat([anc, draft]), t, cache, m.causal(W), None)
            keep("logits" if call == "prefill" else "verify_logits", m.logits(x))
        if call == "unanchored":
            x0, kv0 = m.block(anc, t, cache, m.causal(1), None)
            after = [(torch.cat([c[0], n[0]]), torch.cat([c[1], n[1]])) for c, n in zip(cache, kv0)]
            x, _ = m.block(masks, t + 1, after, torch.full((D,), D, device=DEV), 0)
            keep("draft_logits", torch.cat([m.logits(x0), m.logits(x)]))
            x, _ = m.block(draft, t + 1, after, m.causal(D), None)
            keep("verify_logits", m.logits(x))
    return {k: torch.stack(v) for k, v in rows.items()}
