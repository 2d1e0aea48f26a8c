"""Prompt chunks without padding rows: prompts of very different lengths (one token to many chunks) lie one behind the other in
a forward, on the type-generic kernels and on every head size of the tiled ones; more rows than one chunk holds; then a verify
step over the cache they filled, against the oracle."""
import numpy as np
import pytest

import workload as W
from oracle import model as OM

pytestmark = pytest.mark.gpu

BF16 = dict(dtype="bf16", d_model=128, d_ffn=192)
CASES = {
    # fp32, chunks of 24 positions: the last one holds a single position of a single sequence
    "f32": (dict(n_heads=4, n_kv_heads=2, head_dim=32), [73, 1, 24, 25, 3], 24, 1e-3),
    # head sizes and a vocabulary that only the type-generic kernels take: several dimensions per lane, odd columns
    "f32_hd200": (dict(n_heads=2, n_kv_heads=1, head_dim=200, d_model=136, vocab=701), [70, 1, 130, 65], 24, 1e-3),
    "bf16_hd96": (dict(BF16, n_heads=2, n_kv_heads=2, head_dim=96, vocab=1003), [40, 17, 3], 24, 5e-2),
    # one chunk (5 to 37 rows of head_dim 32: the unstaged attention), tail sequences of one token
    "hd32": (dict(BF16, n_heads=6, n_kv_heads=2, head_dim=32, d_model=192), [37, 1, 5, 30], 32, 5e-2),
    "hd64": (dict(BF16, n_heads=4, n_kv_heads=2, head_dim=64), [300, 1, 2, 77, 150, 16], 40, 5e-2),
    "hd128": (dict(BF16, n_heads=4, n_kv_heads=1, head_dim=128), [260, 64, 65, 1], 17, 5e-2),
    # 21,000 rows: three chunks of about 7,000 whose sequences end in different ones
    "many": (dict(BF16, n_heads=2, n_kv_heads=1, head_dim=64), [640 - (b * 53) % 600 for b in range(64)], 20, 5e-2),
}


@pytest.mark.parametrize("name", list(CASES))
def test_packed_prompts(name):
    import torch
    import paper_2602_24174_amd as T
    shape, lens, max_rows, tol = CASES[name]
    k, B = 3, len(lens)
    cfg = W.get_config("cfg1").scaled(**dict(dict(n_layers=2, vocab=700, batch=B, n_docs=800), **shape))
    weights = W.make_model(cfg, W.make_corpus(cfg))
    rng = np.random.default_rng(3)
    prompts = [rng.integers(0, cfg.vocab, n).astype(np.int32) for n in lens]
    max_len = max(lens) + 1 + 2 * max_rows
    model = T.tasc_model_create(cfg, weights, max_len)
    sess = T.tasc_session_create(model, B, max_len, max_rows)
    drafts = rng.integers(0, cfg.vocab, (B, k)).astype(np.int32)
    z = torch.zeros((B, k + 1, cfg.vocab), dtype=torch.float32, device="cuda")
    for again in range(2):       # the second prefill finds the first one's rows in every buffer
        print(f"{name} prefill {again}", flush=True)
        T.tasc_session_prefill(model, sess, np.concatenate(prompts), np.cumsum([0] + lens).astype(np.int64), 1)
        T.tasc_verify_step(model, sess, torch.from_numpy(drafts).cuda(), k, None, None, z)
        torch.cuda.synchronize()
        if again == 0:
            first = z.cpu().numpy()
    assert (z.cpu().numpy() == first).all()
    om = OM.OracleModel(cfg, weights)
    for b in sorted({0, 1, B // 2, B - 1}):
        c = om.new_cache(max_len)
        zp = om.forward(prompts[b].tolist(), c, last_only=True)[0]
        c.length = lens[b]
        tok = T.tasc_session_get_tokens(sess, b)
        assert tok[:-1].tolist() == prompts[b].tolist()
        assert zp[int(tok[-1])] >= zp.max() - 2 * tol, "the committed token is not the target's argmax"
        want = om.forward([int(tok[-1])] + drafts[b].tolist(), c)
        worst = float(np.abs(first[b].astype(np.float64) - want).max())
        print(f"{name} sequence {b} ({lens[b]} tokens): max |logit - oracle| = {worst:.3e}", flush=True)
        assert worst <= tol


@pytest.mark.parametrize("chains", [2, 4])
def test_chains_of_equal_prompts(chains):
    """Prompts of one length make chunks in which every sequence has as many rows as the next, the only ones the forward could cut
    into chains; these hold more rows (32 x 250) than a chain's share of the partial sums.  The same bits as one chain, then and
    in the verify step over the cache, which does run as chains."""
    import torch
    import paper_2602_24174_amd as T
    B, P, k, max_rows = 32, 250, 3, 20
    cfg = W.get_config("cfg1").scaled(**dict(BF16, n_layers=2, vocab=700, batch=B, n_docs=800, n_heads=4, n_kv_heads=2, head_dim=64, d_ffn=3072))
    rng = np.random.default_rng(9)
    prompts = rng.integers(0, cfg.vocab, B * P).astype(np.int32)
    max_len = P + 1 + 2 * max_rows
    model = T.tasc_model_create(cfg, W.make_model(cfg, W.make_corpus(cfg)), max_len)
    sess = T.tasc_session_create(model, B, max_len, max_rows)
    drafts = torch.from_numpy(rng.integers(0, cfg.vocab, (B, k)).astype(np.int32)).cuda()
    z = torch.zeros((B, k + 1, cfg.vocab), dtype=torch.float32, device="cuda")
    got = []
    try:
        for c in (1, chains):
            print(f"chains {c}", flush=True)
            T.tasc_config_set(T.TASC_CFG_CHAINS, c)
            T.tasc_session_prefill(model, sess, prompts, np.arange(B + 1, dtype=np.int64) * P, 1)
            T.tasc_verify_step(model, sess, drafts, k, None, None, z)
            torch.cuda.synchronize()
            got.append((z.cpu().numpy(), [T.tasc_session_get_tokens(sess, b).tolist() for b in range(B)]))
    finally:
        T.tasc_config_set(T.TASC_CFG_CHAINS, 0)
    assert (got[0][0] == got[1][0]).all() and got[0][1] == got[1][1]


@pytest.mark.parametrize("heads", [(4, 2, 64), (4, 1, 128), (6, 2, 32)])
def test_prompt_does_not_depend_on_its_neighbours(heads):
    """One prompt among short, long and ragged others, so that a chunk holds from 250 to several thousand rows, split over one or
    more chunks: its cached keys and values, its first token and the logits of the next step are the same bits."""
    import torch
    import paper_2602_24174_amd as T
    H, Hkv, hd = heads
    B, k, max_rows, longest = 16, 3, 20, 900
    cfg = W.get_config("cfg1").scaled(**dict(BF16, n_layers=2, d_model=192, d_ffn=3072, vocab=700, batch=B, n_docs=800, n_heads=H,
                                             n_kv_heads=Hkv, head_dim=hd))
    rng = np.random.default_rng(13)
    mine = rng.integers(0, cfg.vocab, 230).astype(np.int32)
    max_len = longest + 1 + 2 * max_rows
    model = T.tasc_model_create(cfg, W.make_model(cfg, W.make_corpus(cfg)), max_len)
    sess = T.tasc_session_create(model, B, max_len, max_rows)
    drafts = torch.from_numpy(rng.integers(0, cfg.vocab, (B, k)).astype(np.int32)).cuda()
    z = torch.zeros((B, k + 1, cfg.vocab), dtype=torch.float32, device="cuda")
    blocks = (max_len + 15) // 16
    got = []
    for others in ([1] * 15, [230] * 15, [longest] * 15, [longest - 55 * i for i in range(15)]):
        print(f"heads {heads} others {others}", flush=True)
        lens = others[:5] + [len(mine)] + others[5:]
        prompts = [mine if b == 5 else rng.integers(0, cfg.vocab, n).astype(np.int32) for b, n in enumerate(lens)]
        T.tasc_session_prefill(model, sess, np.concatenate(prompts), np.cumsum([0] + lens).astype(np.int64), 1)
        pool = sess._kv_pool.view(torch.int16).view(cfg.n_layers, blocks, B, -1)     # block j of sequence b: page j B + b
        kv = pool[:, :len(mine) // 16, 5].clone()                                    # those the prompt fills
        assert bool((kv != 0).any())
        T.tasc_verify_step(model, sess, drafts, k, None, None, z)
        torch.cuda.synchronize()
        got.append((kv, z[5].clone(), T.tasc_session_get_tokens(sess, 5).tolist()))
    for kv, logits, tokens in got[1:]:
        assert torch.equal(kv, got[0][0]) and torch.equal(logits, got[0][1]) and tokens == got[0][2]


def test_smaller_workspaces():
    """A session in less memory than tasc_session_workspace_bytes asks for takes shorter prompt chunks, down to batch x max_rows
    rows; below that it is refused.  Logits of every size against the oracle, and nothing past the workspace is written."""
    import ctypes as C
    import re
    import torch
    import paper_2602_24174_amd as T
    from paper_2602_24174_amd.binding import Session
    shape, lens, _, tol = CASES["hd64"]
    B, max_rows, k = len(lens), 20, 3
    cfg = W.get_config("cfg1").scaled(**dict(dict(n_layers=2, vocab=700, batch=B, n_docs=800), **shape))
    weights = W.make_model(cfg, W.make_corpus(cfg))
    rng = np.random.default_rng(3)
    prompts = [rng.integers(0, cfg.vocab, n).astype(np.int32) for n in lens]
    drafts = rng.integers(0, cfg.vocab, (B, k)).astype(np.int32)
    max_len = max(lens) + 1 + 2 * max_rows
    model = T.tasc_model_create(cfg, weights, max_len)
    kvb, full = T.tasc_session_kv_bytes(model, B, max_len), T.tasc_session_workspace_bytes(model, B, max_len, max_rows)
    kv = torch.empty(kvb, dtype=torch.uint8, device="cuda")
    ws = torch.empty(full + 4096, dtype=torch.uint8, device="cuda")

    def create(nbytes):
        out = C.c_void_p()
        rc = T.lib().tasc_session_create(model.handle, B, max_len, max_rows, kv.data_ptr(), kvb, ws.data_ptr(), nbytes, C.byref(out))
        return rc, Session(out.value, model, B, max_len, max_rows, kv, ws) if rc == 0 else None

    rc, _ = create(16)
    assert rc == -2
    least = int(re.search(rb"workspace 16 of (\d+) bytes", T.lib().tasc_last_error()).group(1))
    assert least < full // 2 and create(least - 1)[0] == -2
    om = OM.OracleModel(cfg, weights)
    for nbytes in (least, least + (full - least) // 3, full - 1, full):
        print(f"workspace {nbytes} of {full}", flush=True)
        ws.fill_(0x5A)
        rc, sess = create(nbytes)
        assert rc == 0
        T.tasc_session_prefill(model, sess, np.concatenate(prompts), np.cumsum([0] + lens).astype(np.int64), 1)
        z = torch.zeros((B, k + 1, cfg.vocab), dtype=torch.float32, device="cuda")
        T.tasc_verify_step(model, sess, torch.from_numpy(drafts).cuda(), k, None, None, z)
        torch.cuda.synchronize()
        assert bool((ws[nbytes:] == 0x5A).all())
        for b in (0, 3, B - 1):
            c = om.new_cache(max_len)
            om.forward(prompts[b].tolist(), c, last_only=True)
            c.length = lens[b]
            first = int(T.tasc_session_get_tokens(sess, b)[-1])
            want = om.forward([first] + drafts[b].tolist(), c)
            assert float(np.abs(z[b].cpu().numpy().astype(np.float64) - want).max()) <= tol
        sess.close()


def test_tail_of_a_prompt_stays_with_its_kernels():
    """One sequence of a model that the persistent kernels serve and the tiled ones do not, in prompt chunks of more than 16 rows: the
    few rows that the last chunk has left run on the kernels of the chunks before, so the cache and the first token are, bit for bit,
    those of a session that may not use the persistent kernels at all."""
    import torch
    import paper_2602_24174_amd as T
    cfg = W.get_config("cfg1").scaled(dtype="bf16", n_layers=2, d_model=96, n_heads=3, n_kv_heads=3, head_dim=32, d_ffn=160, vocab=700,
                                      batch=1, n_docs=800)
    rng = np.random.default_rng(17)
    model = T.tasc_model_create(cfg, W.make_model(cfg, W.make_corpus(cfg)), 208)
    try:
        for n in (5, 17, 70, 73):
            prompt, got = rng.integers(0, cfg.vocab, n).astype(np.int32), []
            for small in (2, 0):
                print(f"prompt of {n}, small path {small}", flush=True)
                T.tasc_config_set(T.TASC_CFG_SMALL_PATH, small)
                sess = T.tasc_session_create(model, 1, 208, 64)
                T.tasc_session_prefill(model, sess, prompt, np.array([0, n], dtype=np.int64), 1)
                torch.cuda.synchronize()
                got.append((sess._kv_pool.clone(), T.tasc_session_get_tokens(sess, 0).tolist()))
            assert torch.equal(got[0][0], got[1][0]) and got[0][1] == got[1][1], f"prompt of {n}"
    finally:
        T.tasc_config_set(T.TASC_CFG_SMALL_PATH, 2)
