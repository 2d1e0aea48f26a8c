"""The work a user of this library has it do, as cases that can be timed and checked one by one.

A case is a dict of plain values.  `prepare` makes what a program has in hand before the call (weights and model, tables,
session, prompts), `run` is one pass through the public entry points, `exact` the same result in 64 bits by plain torch.

Kinds
  verify    one `tasc_verify_step` that returns the logits of every candidate row: the step the decode loop is made of.
            The sequences already hold the tokens they were asked for, so the step scores its rows, writes their keys and
            values and commits nothing: a pass leaves the session as it found it.
  generate  `tasc_generate` (prompt forward, then draft + verify until every sequence has its tokens), then the logits of
            the position after the last token.
  prefill   `tasc_session_prefill` of new prompts, then the logits of the first generated position.
  draft     `tasc_draft` over sequences of a given length.
  build     `tasc_ngram_build` of a task corpus, its statistics, its token counts and the drafts it gives.
  enrich    `tasc_tok_enrich`: some merges of the tokenizer enrichment over a corpus.

Models are the shapes of the workload configurations with fewer layers (every layer is alike) and, but for one case, the
vocabulary of the 135M-class one, so that the layers weigh about as much against the LM head as in the full models.
"""
import math
import types

import numpy as np
import torch

import paper_2602_24174_amd as T

# dtype, d_model, heads, KV heads, head_dim, d_ffn of the five configurations
SHAPES = {
    "tiny": ("f32", 128, 4, 4, 32, 512),
    "135m": ("bf16", 576, 9, 3, 64, 1536),
    "05b": ("bf16", 896, 14, 2, 64, 4864),
    "15b": ("bf16", 1536, 12, 2, 128, 8960),
    "3b": ("bf16", 2048, 16, 2, 128, 11008),
}
ALPHA = 8.0              # strength of the corpus bias on the LM head
POOL = 5000              # phrases of a task corpus
EPS, THETA = 1e-6, 10000.0
LAMBDA_Q16 = 49152       # 0.75
MAX_ORDER = 8            # longest n-gram of the library


def listed():
    return [
        # the smallest call: an fp32 model of two layers, one sequence; launches and host work are most of it
        {"name": "generate_tiny_f32", "kind": "generate", "model": "tiny", "layers": 2, "vocab": 512, "batch": 1, "prompt": 64, "gen": 64,
         "k": 4, "n_max": 3, "corpus": 128_000},
        # interactive decoding of one sequence on a small model, all 30 layers: 9 rows, bound by dependent latency
        {"name": "verify_135m_b1", "kind": "verify", "model": "135m", "layers": 30, "vocab": 49_152, "batch": 1, "prompt": 512, "k": 8,
         "corpus": 500_000},
        # the same user's whole call: prompt, drafts, verify steps
        {"name": "generate_135m_b1", "kind": "generate", "model": "135m", "layers": 30, "vocab": 49_152, "batch": 1, "prompt": 512, "gen": 64,
         "k": 8, "n_max": 4, "corpus": 1_000_000},
        # a small serving batch: 224 rows over ragged contexts of up to 1024 tokens
        {"name": "verify_05b_b32", "kind": "verify", "model": "05b", "layers": 6, "vocab": 49_152, "batch": 32, "prompt": 1024, "k": 6,
         "corpus": 500_000},
        # long contexts, 576 rows, the large vocabulary
        {"name": "verify_15b_b64", "kind": "verify", "model": "15b", "layers": 4, "vocab": 151_936, "batch": 64, "prompt": 2048, "k": 8,
         "corpus": 500_000},
        # high-volume batch: 1280 rows, bound by the matrix cores
        {"name": "verify_3b_b256", "kind": "verify", "model": "3b", "layers": 4, "vocab": 49_152, "batch": 256, "prompt": 256, "k": 4,
         "corpus": 500_000},
        # whole calls of a batch: many short steps after a prompt
        {"name": "generate_05b_b32", "kind": "generate", "model": "05b", "layers": 6, "vocab": 49_152, "batch": 32, "prompt": 256, "gen": 96,
         "k": 6, "n_max": 4, "corpus": 2_000_000},
        {"name": "generate_3b_b256", "kind": "generate", "model": "3b", "layers": 4, "vocab": 49_152, "batch": 256, "prompt": 128, "gen": 64,
         "k": 4, "n_max": 5, "corpus": 2_000_000},
        # long prompts: the prompt forward alone
        {"name": "prefill_15b_b16", "kind": "prefill", "model": "15b", "layers": 4, "vocab": 49_152, "batch": 16, "prompt": 2048,
         "corpus": 500_000},
        # drafting for a batch with long contexts
        {"name": "draft_b64", "kind": "draft", "vocab": 151_936, "batch": 64, "prompt": 2300, "k": 8, "n_max": 5, "corpus": 4_000_000},
        # the one-off table build of a mid-sized task corpus that is already on the GPU
        {"name": "build_32m", "kind": "build", "vocab": 151_936, "corpus": 32_000_000, "n_max": 5, "p_min": 5, "host": False, "batch": 64,
         "prompt": 200, "k": 8},
        # tokenizer enrichment: a table build per merge over a small corpus
        {"name": "enrich_1m", "kind": "enrich", "vocab": 49_152, "corpus": 1_000_000, "n_max": 4, "budget": 8, "host": False},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["verify", "verify", "generate", "generate", "prefill", "draft", "build", "enrich"])
    vocab = _log(rng, 4096, 49_152)
    if kind in ("verify", "generate", "prefill"):
        model = rng.choice(["135m", "05b", "15b", "3b"] + (["tiny"] if kind == "generate" else []))
        c = {"kind": kind, "model": model, "layers": rng.randint(2, 4), "vocab": 512 if model == "tiny" else vocab,
             "batch": 1 if model == "tiny" else _log(rng, 1, {"135m": 24, "05b": 64, "15b": 64, "3b": 256}[model]),
             "corpus": _log(rng, 200_000, 1_000_000)}
        if kind == "prefill":
            c["prompt"] = min(_log(rng, 16, 2048), 32_768 // c["batch"])
            return c
        c["prompt"] = min(_log(rng, 16, 1024 if kind == "verify" else 300), 65_536 // c["batch"])
        c["k"] = rng.randint(1, 10)
        while c["batch"] * (c["k"] + 1) > 1280:
            c["k"] -= 1
        if kind == "generate":
            c["gen"] = rng.randint(8, 64)
            c["n_max"] = rng.randint(2, 6)
        return c
    if kind == "draft":
        return {"kind": kind, "vocab": vocab, "batch": _log(rng, 1, 256), "prompt": _log(rng, 16, 3800), "k": rng.randint(1, 15),
                "n_max": rng.randint(2, 7), "corpus": _log(rng, 100_000, 4_000_000)}
    if kind == "build":
        return {"kind": kind, "vocab": vocab, "corpus": _log(rng, 20_000, 16_000_000), "n_max": rng.randint(2, 6), "p_min": rng.randint(1, 8),
                "host": rng.random() < 0.5, "batch": _log(rng, 1, 64), "prompt": _log(rng, 16, 400), "k": rng.randint(1, 10)}
    return {"kind": kind, "vocab": vocab, "corpus": _log(rng, 20_000, 1_000_000), "n_max": rng.randint(2, 6), "budget": rng.randint(1, 8),
            "host": rng.random() < 0.5}


# ---------------------------------------------------------------- inputs
def _gen(seed, purpose):
    return torch.Generator(device="cuda").manual_seed((seed * 64 + purpose) & 0x7FFFFFFFFFFF)


class Corpus:
    """Task outputs of 64 to 256 tokens: phrases drawn from a bounded Zipf(1.1) law over a pool, 10 % of the tokens replaced."""

    def __init__(self, seed, n_tokens, vocab):
        g = _gen(seed, 1)

        def rnd(lo, hi, *n):
            return torch.randint(lo, hi, n, generator=g, device="cuda")

        n_docs = max(1, n_tokens // 160)
        self.plen = rnd(2, 9, POOL)
        self.poff = torch.cumsum(self.plen, 0) - self.plen
        self.ptok = rnd(0, vocab, int(self.plen.sum())).int()
        w = torch.arange(1, POOL + 1, device="cuda", dtype=torch.float64) ** -1.1
        self.cdf = torch.cumsum(w / w.sum(), 0)
        ends = torch.cumsum(rnd(64, 257, n_docs), 0).double()
        ends = torch.round(ends * (n_tokens / ends[-1])).long()        # n_tokens in all, whatever the seed
        dlen = torch.diff(ends, prepend=ends[:1] * 0)
        self.tokens, self.offsets = self.text(g, dlen)
        hit = torch.rand(self.tokens.numel(), generator=g, device="cuda") < 0.1
        self.tokens = torch.where(hit, rnd(0, vocab, self.tokens.numel()).int(), self.tokens)

    def phrases(self, g, shape):
        u = torch.rand(shape, generator=g, device="cuda", dtype=torch.float64)
        return torch.searchsorted(self.cdf, u).clamp_(max=POOL - 1)

    def text(self, g, dlen):
        """Phrase text cut at the lengths `dlen`: tokens int32, offsets int64 (host)."""
        m = (int(dlen.max()) + 1) // 2
        ids = self.phrases(g, (dlen.numel(), m))
        lens = self.plen[ids]
        starts = torch.cumsum(lens, 1) - lens
        take = torch.minimum((dlen[:, None] - starts).clamp_(min=0), lens).reshape(-1)
        src = torch.repeat_interleave(self.poff[ids.reshape(-1)], take)
        first = torch.repeat_interleave(torch.cumsum(take, 0) - take, take)
        within = torch.arange(src.numel(), device="cuda") - first
        offs = np.zeros(dlen.numel() + 1, dtype=np.int64)
        np.cumsum(dlen.cpu().numpy(), out=offs[1:])
        return self.ptok[src + within], offs

    def prompts(self, seed, batch, longest, ragged=True):
        """Prompts of longest / 2 to longest tokens (one of `longest`) of the task's phrases, each ending inside a frequent phrase."""
        g = _gen(seed, 2)
        plen = torch.randint(max(1, longest // 2), longest + 1, (batch,), generator=g, device="cuda") if ragged else torch.full((batch,), longest, device="cuda")
        plen[0] = longest
        tok, offs = self.text(g, plen)
        rank = torch.randint(0, 64, (batch,), generator=g, device="cuda")
        tok[torch.from_numpy(offs[1:] - 1).cuda()] = self.ptok[self.poff[rank]]
        return tok.contiguous(), offs

    def bias(self, vocab):
        """LM-head bias ALPHA * log P_bigram with add-one smoothing, as sparse rows plus a value for the unseen pairs of a row."""
        a, b = self.tokens[:-1].long(), self.tokens[1:].long()
        keep = torch.ones(a.numel(), dtype=torch.bool, device="cuda")
        ends = torch.from_numpy(self.offsets[1:-1] - 1).cuda()
        keep[ends] = False
        key, cnt = torch.unique(a[keep] * vocab + b[keep], return_counts=True)
        row = key // vocab
        c1 = torch.zeros(vocab, dtype=torch.float64, device="cuda").index_add_(0, row, cnt.double())
        norm = torch.log(c1 + vocab)
        ptr = torch.zeros(vocab + 1, dtype=torch.int64, device="cuda")
        ptr[1:] = torch.cumsum(torch.bincount(row, minlength=vocab), 0)
        val = ALPHA * (torch.log(cnt.double() + 1.0) - norm[row])
        return {"rowptr": ptr, "col": (key % vocab).int(), "val": val.float(), "base": (-ALPHA * norm).float()}


def _weights(seed, case):
    """(config, names -> GPU tensors): N(0, 0.02^2) matrices (slices of one pool of random values), gains near 1."""
    dtype, d, h, hk, hd, f = SHAPES[case["model"]]
    v, layers = case["vocab"], case["layers"]
    cfg = types.SimpleNamespace(dtype=dtype, n_layers=layers, d_model=d, n_heads=h, n_kv_heads=hk, head_dim=hd, d_ffn=f, vocab=v,
                                rope_theta=THETA, rms_eps=EPS)
    shape = {"wq": (h * hd, d), "wk": (hk * hd, d), "wv": (hk * hd, d), "wo": (d, h * hd), "wg": (f, d), "wu": (f, d), "wd": (d, f)}
    slack = 1 << 20
    pool = torch.empty(max(v * d, f * d) + slack, dtype=torch.float32 if dtype == "f32" else torch.bfloat16, device="cuda")
    g = _gen(seed, 3)
    for i in range(0, pool.numel(), 1 << 26):
        n = min(1 << 26, pool.numel() - i)
        pool[i:i + n] = torch.randn(n, generator=g, device="cuda").mul_(0.02)
    at = torch.randint(0, slack // 8, (2 + 7 * layers,), generator=g, device="cuda").mul_(8).tolist()
    gains = 1.0 + 0.1 * torch.randn((2 * layers + 1, d), generator=g, device="cuda")
    mats = {"embed": (at[0], (v, d)), "lm_head": (at[1], (v, d))}
    for l in range(layers):
        for j, n in enumerate(shape):
            mats[n, l] = (at[2 + 7 * l + j], shape[n])
    return cfg, pool, mats, gains


def _view(pool, where):
    o, (r, c) = where
    return pool[o:o + r * c].reshape(r, c)


def _model(seed, case, corpus, max_len):
    cfg, pool, mats, gains = _weights(seed, case)
    raw = pool.view(torch.int16) if pool.dtype == torch.bfloat16 else pool
    host = torch.empty(raw.numel(), dtype=raw.dtype, pin_memory=True).copy_(raw).numpy()
    host = host.view(np.uint16) if host.dtype == np.int16 else host
    gn = gains.cpu().numpy()
    w = {"embed": _view(host, mats["embed"]), "lm_head": _view(host, mats["lm_head"]), "gf": gn[-1],
         "layers": [dict({n: _view(host, mats[n, l]) for n in ("wq", "wk", "wv", "wo", "wg", "wu", "wd")}, g1=gn[2 * l], g2=gn[2 * l + 1])
                    for l in range(cfg.n_layers)],
         "bias": {n: t.cpu().numpy() for n, t in corpus.bias(cfg.vocab).items()}}
    return T.tasc_model_create(cfg, w, max_len)


def _rows(batch, k):
    return max(k + 1, 512 if batch == 1 else 64)      # rows per sequence of a prompt chunk


def _drafts(seed, corpus, batch, k):
    at = torch.randint(0, corpus.tokens.numel(), (batch, k), generator=_gen(seed, 4), device="cuda")
    return corpus.tokens[at].contiguous()


def prepare(case, seed):
    kind, v = case["kind"], case["vocab"]
    corpus = Corpus(seed, case["corpus"], v)
    s = types.SimpleNamespace(case=case)
    if kind in ("build", "enrich"):
        s.tokens = corpus.tokens.cpu().numpy() if case["host"] else corpus.tokens
        s.offsets = corpus.offsets
        if kind == "enrich":
            s.text = torch.empty(case["corpus"], dtype=torch.int32, device="cpu" if case["host"] else "cuda")
            return s
    b, k = case["batch"], case.get("k", 0)
    s.prompts, s.poff = corpus.prompts(seed, b, case["prompt"])
    gen = case.get("gen", 2)
    rows = _rows(b, k)
    max_len = case["prompt"] + gen + 2 * rows
    if kind in ("draft", "build"):
        # a small model stands for the target: drafting only looks at the sequences' tokens
        target = {"model": "tiny", "layers": 1, "vocab": v}
        rows = k + 1 if b == 1 else 16
        max_len = case["prompt"] + gen + 2 * rows
    else:
        target = case
    s.model = _model(seed, target, corpus, max_len)
    s.session = T.tasc_session_create(s.model, b, max_len, rows)
    s.params = T.spec_params(k, LAMBDA_Q16)
    if kind == "verify":
        T.tasc_session_prefill(s.model, s.session, s.prompts, s.poff, 1)
    if kind in ("draft", "build"):
        T.tasc_session_prefill(s.model, s.session, s.prompts, s.poff, gen)
        s.drafts = torch.zeros((b, k), dtype=torch.int32, device="cuda")
        if kind == "draft":
            s.ng = T.tasc_ngram_build(corpus.tokens, corpus.offsets, v, case["n_max"], 5)
    if kind == "generate":
        s.ng = T.tasc_ngram_build(corpus.tokens, corpus.offsets, v, case["n_max"], 5)
        s.out = torch.zeros((b, gen), dtype=torch.int32, device="cuda")
    if kind == "verify":
        s.drafts = _drafts(seed, corpus, b, k)
        s.accept = torch.zeros(b, dtype=torch.int32, device="cuda")
    if kind in ("verify", "generate", "prefill"):
        nq = k + 1 if kind == "verify" else 1
        s.emitted = torch.zeros((b, nq), dtype=torch.int32, device="cuda")
        s.logits = torch.zeros((b, nq, v), dtype=torch.float32, device="cuda")
    return s


def run(s):
    c = s.case
    kind = c["kind"]
    if kind == "verify":
        T.tasc_verify_step(s.model, s.session, s.drafts, c["k"], s.accept, s.emitted, s.logits)
        return {"logits": s.logits, "emitted": s.emitted, "accept_len": s.accept}
    if kind == "generate":
        T.tasc_generate(s.model, s.ng, s.session, s.prompts, s.poff, c["gen"], s.params, s.out)
        T.tasc_verify_step(s.model, s.session, None, 0, None, s.emitted, s.logits)
        return {"logits": s.logits, "tokens": s.out}
    if kind == "prefill":
        T.tasc_session_prefill(s.model, s.session, s.prompts, s.poff, 2)
        T.tasc_verify_step(s.model, s.session, None, 0, None, s.emitted, s.logits)
        return {"logits": s.logits, "emitted": s.emitted}
    if kind == "draft":
        T.tasc_draft(s.ng, s.session, s.params, s.drafts)
        return {"drafts": s.drafts}
    if kind == "build":
        ng = T.tasc_ngram_build(s.tokens, s.offsets, c["vocab"], c["n_max"], c["p_min"])
        st = T.tasc_ngram_get_stats(ng)
        fallback, counts = T.tasc_ngram_unigram(ng, c["vocab"])
        T.tasc_draft(ng, s.session, s.params, s.drafts)
        out = {"drafts": s.drafts, "counts": counts.astype(np.int64), "fallback": fallback}
        for name in ("windows", "distinct", "kept", "contexts"):
            out[name] = np.array(getattr(st, name)[:], dtype=np.int64)
        ng.close()
        return out
    merges, tokens, offsets, lens = T.tasc_tok_enrich(s.tokens, s.offsets, c["vocab"], c["n_max"], c["budget"])
    grams = np.full((len(merges), MAX_ORDER), -1, dtype=np.int64)
    for i, (gram, _, _) in enumerate(merges):
        grams[i, :len(gram)] = gram
    s.text.fill_(-1)[:len(tokens)] = torch.from_numpy(tokens) if c["host"] else tokens
    return {"merges": grams, "freq": np.array([m[1] for m in merges], dtype=np.int64), "text": s.text, "offsets": offsets, "lengths": lens}


# ---------------------------------------------------------------- what a pass cannot do without
def work(case):
    kind = case["kind"]
    if kind == "draft":
        b, k = case["batch"], case["k"]      # the context once, two table rows per proposal, the proposals
        return {"bytes": 3.0 * b * case["prompt"] + b * k * (64 + 4), "flops": 0.0}
    if kind == "build":
        return {"bytes": 4.0 * case["corpus"] + 4.0 * case["vocab"], "flops": 0.0}
    if kind == "enrich":
        return {"bytes": 8.0 * case["corpus"], "flops": 0.0}
    dtype, d, h, hk, hd, f = SHAPES[case["model"]]
    es = 4 if dtype == "f32" else 2
    b, v, n, prompt = case["batch"], case["vocab"], case["layers"], 0.75 * case["prompt"]
    layer = d * (2 * h * hd + 2 * hk * hd) + 3 * d * f

    def forward(rows, sel, context):         # one forward of `rows` rows per sequence, `sel` of them through the LM head
        fl = 2.0 * b * (rows * n * layer + sel * v * d) + 4.0 * b * rows * n * h * hd * (context + rows / 2)
        by = es * (n * layer + v * d + n * b * 2 * hk * hd * (context + rows))
        return np.array([by, fl])

    if kind == "verify":
        total = forward(case["k"] + 1, case["k"] + 1, prompt) + np.array([4.0 * b * (case["k"] + 1) * v, 0])
    else:
        total = forward(prompt, 1, 0) + forward(1, 1, prompt) + np.array([4.0 * b * v, 0])
        if kind == "generate":
            steps = -(-(case["gen"] - 1) // (case["k"] + 1))
            total = total + steps * forward(case["k"] + 1, case["k"] + 1, prompt + case["gen"] / 2)
    return {"bytes": float(total[0]), "flops": float(total[1])}


def tolerance(case):
    if case["kind"] in ("draft", "build", "enrich"):
        return "exact"
    if case["model"] == "tiny":
        return {"rel": 1e-6, "max": 1e-5}
    # logits are around -90 (the bias of an unseen successor) and the model's own part is of order one, computed with bf16
    # matrix operands
    return {"rel": 4e-4, "max": 4e-3, "differ": 0.005}


# ---------------------------------------------------------------- 64-bit results
class Exact:
    """The target model in float64 on the rounded weights, with a plain key / value cache."""

    def __init__(self, seed, case, corpus, max_len):
        self.cfg, pool, mats, gains = _weights(seed, case)
        self.w = {n: _view(pool, where).double() for n, where in mats.items()}
        self.gains = gains.double()
        self.bias = corpus.bias(case["vocab"])
        c = self.cfg
        inv = THETA ** (-2.0 * torch.arange(c.head_dim // 2, device="cuda", dtype=torch.float64) / c.head_dim)
        ang = torch.arange(max_len, device="cuda", dtype=torch.float64)[:, None] * inv
        self.cos, self.sin = ang.cos().float().double(), ang.sin().float().double()     # the model's table is fp32
        shape = (c.n_layers, case["batch"], c.n_kv_heads, max_len, c.head_dim)
        self.k, self.v = torch.zeros(shape, device="cuda", dtype=torch.float64), torch.zeros(shape, device="cuda", dtype=torch.float64)

    def norm(self, x, g):
        return x * torch.rsqrt(x.square().mean(-1, keepdim=True) + EPS) * g

    def rope(self, x, pos):          # x [b, t, heads, hd], pos [b, t]
        half = x.shape[-1] // 2
        cs, sn = self.cos[pos][:, :, None], self.sin[pos][:, :, None]
        a, b = x[..., :half], x[..., half:]
        return torch.cat([a * cs - b * sn, b * cs + a * sn], -1)

    def rows(self, tok, pos0):
        """Final hidden rows of tokens [B, t] at positions pos0[b] + i; their keys and values go to the cache."""
        out = []
        step = max(1, (1 << 14) // tok.shape[1])
        for b0 in range(0, tok.shape[0], step):
            out.append(self.some_rows(slice(b0, min(tok.shape[0], b0 + step)), tok[b0:b0 + step], pos0[b0:b0 + step]))
        return torch.cat(out)

    def some_rows(self, seqs, tok, pos0):
        c, w = self.cfg, self.w
        b, t = tok.shape
        pos = pos0[:, None] + torch.arange(t, device="cuda")
        n_keys = int(pos.max()) + 1
        at = torch.arange(b, device="cuda")[:, None]
        x = w["embed"][tok.long()]
        for l in range(c.n_layers):
            h = self.norm(x, self.gains[2 * l])
            q = self.rope((h @ w["wq", l].T).reshape(b, t, c.n_heads, c.head_dim), pos)
            kk = self.rope((h @ w["wk", l].T).reshape(b, t, c.n_kv_heads, c.head_dim), pos)
            vv = (h @ w["wv", l].T).reshape(b, t, c.n_kv_heads, c.head_dim)
            ck, cv = self.k[l, seqs], self.v[l, seqs]
            ck[at, :, pos] = kk
            cv[at, :, pos] = vv
            group = c.n_heads // c.n_kv_heads
            # one product per (sequence, KV head): the group's heads side by side as rows
            qh = q.reshape(b, t, c.n_kv_heads, group, c.head_dim).permute(0, 2, 3, 1, 4).reshape(b * c.n_kv_heads, group * t, c.head_dim).contiguous()
            kh = ck[:, :, :n_keys].reshape(b * c.n_kv_heads, n_keys, c.head_dim).transpose(1, 2).contiguous()
            vh = cv[:, :, :n_keys].reshape(b * c.n_kv_heads, n_keys, c.head_dim).contiguous()
            seen = torch.arange(n_keys, device="cuda")[None, None] <= pos[:, :, None]           # [b, t, keys]
            att = torch.empty_like(qh)
            few = max(1, (1 << 27) // (c.n_heads * t * n_keys))
            for i in range(0, b, few):
                g, j = slice(i * c.n_kv_heads, min(b, i + few) * c.n_kv_heads), slice(i, min(b, i + few))
                sc = torch.bmm(qh[g], kh[g]).mul_(c.head_dim ** -0.5).reshape(-1, c.n_kv_heads, group, t, n_keys)
                sc = sc.masked_fill_(~seen[j][:, None, None], -math.inf).softmax(-1)
                att[g] = torch.bmm(sc.reshape(-1, group * t, n_keys), vh[g])
            att = att.reshape(b, c.n_kv_heads, group, t, c.head_dim).permute(0, 3, 1, 2, 4).reshape(b, t, c.n_heads * c.head_dim)
            x = x + att @ w["wo", l].T
            h = self.norm(x, self.gains[2 * l + 1])
            gate = h @ w["wg", l].T
            x = x + (gate * torch.sigmoid(gate) * (h @ w["wu", l].T)) @ w["wd", l].T
        return self.norm(x, self.gains[-1])

    def logits(self, h, tok):
        """h [n, d], tok [n]: the input token of every row."""
        z = h @ self.w["lm_head"].T + self.bias["base"].double()[tok.long()][:, None]
        ptr, tok = self.bias["rowptr"], tok.long()
        n = ptr[tok + 1] - ptr[tok]
        row = torch.repeat_interleave(torch.arange(tok.numel(), device="cuda"), n)
        p = torch.arange(row.numel(), device="cuda") - torch.repeat_interleave(torch.cumsum(n, 0) - n - ptr[tok], n)
        z[row, self.bias["col"][p].long()] += self.bias["val"][p].double() - self.bias["base"].double()[tok][row]
        return z


def greedy(case, seed, steps):
    """The target's greedy tokens [batch, steps + 1] after the prompts, the logits of the last one's row, and the model."""
    b, longest = case["batch"], case["prompt"]
    corpus = Corpus(seed, case["corpus"], case["vocab"])
    prompts, offs = corpus.prompts(seed, b, longest)
    plen = torch.from_numpy(np.diff(offs)).cuda()
    m = Exact(seed, case, corpus, longest + steps + case.get("k", 0) + 2)
    at = torch.from_numpy(offs[:-1]).cuda()[:, None] + torch.minimum(torch.arange(longest, device="cuda")[None], plen[:, None] - 1)
    h = m.rows(prompts[at], torch.zeros(b, dtype=torch.int64, device="cuda"))     # rows past a prompt's end are overwritten later
    z = m.logits(h[torch.arange(b, device="cuda"), plen - 1], prompts[at[:, -1]])
    got = [z.argmax(-1).int()]
    for i in range(steps):
        z = m.logits(m.rows(got[-1][:, None], plen + i)[:, 0], got[-1])
        got.append(z.argmax(-1).int())
    return torch.stack(got, 1), z, m, corpus, plen


def exact(case, seed):
    kind = case["kind"]
    if kind not in ("verify", "prefill"):
        # whole numbers; and a generate stops at a position of its own, up to k tokens past the ones asked for
        return None
    if kind == "prefill":
        tok, z = greedy(case, seed, 1)[:2]
        return {"logits": z[:, None], "emitted": tok[:, 1:]}
    b, k = case["batch"], case["k"]
    tok, _, m, corpus, plen = greedy(case, seed, 0)
    rows = torch.cat([tok, _drafts(seed, corpus, b, k)], 1)
    z = m.logits(m.rows(rows, plen).reshape(b * (k + 1), -1), rows.reshape(-1))
    return {"logits": z.reshape(b, k + 1, -1), "emitted": None, "accept_len": None}
