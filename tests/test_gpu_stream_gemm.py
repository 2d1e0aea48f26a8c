"""Launches of more large GEMM tiles than the device has compute units (the streaming kernel): rotation epilogue at every head
size, gate/up and LM head at 192- and 256-row tiles, one to three stages of k, ragged feature and row edges, an odd vocabulary
(logit rows at any 4-byte address), bias lists that are empty, short, and longer than the ones a lane fetches ahead."""
import numpy as np
import pytest

import workload as W
from oracle import model as OM

pytestmark = pytest.mark.gpu


def _bias(vocab, rng):
    """Sparse rows: none, up to three scattered entries, or (every seventh token) a run of 150 neighbouring columns."""
    rows = []
    for u in range(vocab):
        if u % 7 == 0:
            first = int(rng.integers(0, vocab - 150))
            rows.append(np.arange(first, first + 150))
        else:
            rows.append(np.unique(rng.integers(0, vocab, u % 4)))
    col = np.concatenate(rows).astype(np.int32)
    ptr = np.cumsum([0] + [len(r) for r in rows]).astype(np.int64)
    return {"rowptr": ptr, "col": col, "val": rng.normal(0, 2, col.size).astype(np.float32),
            "base": rng.normal(-3, 0.5, vocab).astype(np.float32)}


@pytest.mark.parametrize("heads,d_model", [((120, 4, 32), 64), ((60, 2, 64), 128), ((28, 2, 128), 192)])
def test_streaming_gemm(heads, d_model):
    import torch
    import paper_2602_24174_amd as T
    H, Hkv, hd = heads
    B, max_rows, V = 288, 16, 22_101
    cfg = W.get_config("cfg1").scaled(dtype="bf16", n_layers=1, d_model=d_model, n_heads=H, n_kv_heads=Hkv, head_dim=hd, d_ffn=11_072,
                                      vocab=V, batch=B)
    rng = np.random.default_rng(5)
    weights = W.make_model(cfg)
    weights["bias"] = _bias(V, rng)
    lens = [int(n) for n in rng.integers(3, 30, B)]
    prompts = [rng.integers(0, V, n).astype(np.int32) for n in lens]
    max_len = 30 + 1 + 2 * max_rows
    model = T.tasc_model_create(cfg, weights, max_len)
    sess = T.tasc_session_create(model, B, max_len, max_rows)
    # prompt chunks: 288 x 16 = 4608 rows (18 row tiles x 16 column tiles of q/k/v, x 87 of gate/up); one token asked for, so
    # the sequences are finished and every verify step below sees the same state
    T.tasc_session_prefill(model, sess, np.concatenate(prompts), np.cumsum([0] + lens).astype(np.int64), 1)
    got = {}
    drafts = rng.integers(0, V, (B, 2)).astype(np.int32)
    for k in (0, 1, 2):          # 288 rows (small tiles), 576 rows (192-row tiles: 3 x 87), 864 rows (256-row tiles: 4 x 87)
        print(f"heads {heads} k {k}", flush=True)
        z = torch.full((B, k + 1, V), -7.0, dtype=torch.float32, device="cuda")
        em = torch.zeros((B, k + 1), dtype=torch.int32, device="cuda")
        d = torch.from_numpy(np.ascontiguousarray(drafts[:, :k])).cuda() if k else None
        T.tasc_verify_step(model, sess, d, k, None, em, z)
        torch.cuda.synchronize()
        got[k] = z.cpu().numpy()
    # a row's result does not depend on the tile shape or on the kernel: the same bits from all three launches
    assert (got[1][:, 0] == got[0][:, 0]).all() and (got[2][:, 0] == got[0][:, 0]).all()
    assert (got[2][:, 1] == got[1][:, 1]).all()
    om = OM.OracleModel(cfg, weights)
    for b in (0, 100, B - 1):
        c = om.new_cache(max_len)
        om.forward(prompts[b].tolist(), c, last_only=True)
        c.length = lens[b]
        first = int(T.tasc_session_get_tokens(sess, b)[-1])
        z = om.forward([first] + drafts[b].tolist(), c)
        worst = float(np.abs(got[2][b].astype(np.float64) - z).max())
        print(f"heads {heads} sequence {b}: max |logit - oracle| = {worst:.3e}", flush=True)
        assert worst <= 5e-2     # bf16 matrix operands, one layer: the bound of the other bf16 parity tests


@pytest.mark.parametrize("B,V,ks,d_model", [(33, 22_101, (0, 2, 3, 5), 128), (14, 33_000, (1, 2, 9, 15), 128), (14, 3001, (1, 15), 2048),
                                            (14, 3001, (1, 15), 2112)])
def test_lm_head_tile_edges(B, V, ks, d_model):
    """The LM head on both sides of its line (more 128 x 128 tiles than compute units, more than 32 rows): 33 and 99 rows on
    small tiles, 132 and 198 on the streaming kernel with fewer tiles than workgroups; 28 rows small, 42, 140 and 224
    streaming.  Embedding, first norm and bias cursors in one launch, also without a spare thread per row, and (2112) apart."""
    import torch
    import paper_2602_24174_amd as T
    max_rows = max(ks) + 1
    cfg = W.get_config("cfg1").scaled(dtype="bf16", n_layers=1, d_model=d_model, n_heads=2, n_kv_heads=2, head_dim=64, d_ffn=192, vocab=V,
                                      batch=B)
    rng = np.random.default_rng(V)
    weights = W.make_model(cfg)
    weights["bias"] = _bias(V, rng)
    prompts = [rng.integers(0, V, 3 + b % 5).astype(np.int32) for b in range(B)]
    lens = [len(p) for p in prompts]
    max_len = 8 + 1 + 2 * max_rows
    model = T.tasc_model_create(cfg, weights, max_len)
    sess = T.tasc_session_create(model, B, max_len, max_rows)
    T.tasc_session_prefill(model, sess, np.concatenate(prompts), np.cumsum([0] + lens).astype(np.int64), 1)
    drafts = rng.integers(0, V, (B, max(ks))).astype(np.int32)
    got = {}
    for k in ks:
        print(f"batch {B} vocab {V} k {k}", flush=True)
        z = torch.full((B, k + 1, V), -7.0, dtype=torch.float32, device="cuda")
        d = torch.from_numpy(np.ascontiguousarray(drafts[:, :k])).cuda() if k else None
        T.tasc_verify_step(model, sess, d, k, None, None, z)
        torch.cuda.synchronize()
        got[k] = z.cpu().numpy()
        assert (got[k] != -7.0).all()
    for k in ks[1:]:             # the same bits whatever the tile shape
        n = ks[0] + 1
        assert (got[k][:, :n] == got[ks[0]][:, :n]).all()
    om = OM.OracleModel(cfg, weights)
    for b in (0, B - 1):
        c = om.new_cache(max_len)
        om.forward(prompts[b].tolist(), c, last_only=True)
        c.length = lens[b]
        first = int(T.tasc_session_get_tokens(sess, b)[-1])
        z = om.forward([first] + drafts[b].tolist(), c)
        assert float(np.abs(got[ks[-1]][b].astype(np.float64) - z).max()) <= 5e-2    # one bf16 layer: the bound of the other parity tests


LENGTHS = (0, 1, 4, 5, 8, 9, 16, 17, 63, 64, 65, 104)


def _bias_by_strip(vocab, rng, strips):
    """Rows that hold up to 104 successors in each of the given strips of 128 columns, and none elsewhere: lists that end on
    both sides of the ones the streaming LM head takes four entries a lane, and two; the last strip ends the whole table."""
    rows = []
    for u in range(vocab):
        n = rng.permutation(LENGTHS)[:len(strips)]
        if u % 3 == 0:
            n = np.minimum(n, 9)             # rows, and by chance groups of rows, without a long list
        rows.append(np.concatenate([128 * s + np.sort(rng.permutation(min(128, vocab - 128 * s))[:m]) for s, m in zip(strips, n)]))
    rows[-1] = np.arange(128 * strips[-1], vocab)
    col = np.concatenate(rows).astype(np.int32)
    ptr = np.cumsum([0] + [len(r) for r in rows]).astype(np.int64)
    return {"rowptr": ptr, "col": col, "val": rng.normal(0, 2, col.size).astype(np.float32),
            "base": rng.normal(-3, 0.5, vocab).astype(np.float32)}


@pytest.mark.parametrize("B,V", [(24, 16_488), (30, 33_000)])
def test_lm_head_bias_lists(B, V):
    """Bias lists of every length class, mixed within a block of 32 rows: 24 or 30 rows on small tiles, then the same rows in steps
    of more rows on the streaming kernel's 192- and 256-row tiles, bit for bit, and against the oracle."""
    import torch
    import paper_2602_24174_amd as T
    ks, max_rows, d_model = (0, 3, 8, 15), 16, 128
    cfg = W.get_config("cfg1").scaled(dtype="bf16", n_layers=1, d_model=d_model, n_heads=2, n_kv_heads=2, head_dim=64, d_ffn=192, vocab=V,
                                      batch=B)
    rng = np.random.default_rng(V)
    weights = W.make_model(cfg)
    weights["bias"] = _bias_by_strip(V, rng, (0, 1, 6, 77, V // 128))
    prompts = [rng.integers(0, V, 3 + b % 5).astype(np.int32) for b in range(B)]
    lens = [len(p) for p in prompts]
    max_len = 8 + 1 + 2 * max_rows
    model = T.tasc_model_create(cfg, weights, max_len)
    sess = T.tasc_session_create(model, B, max_len, max_rows)
    T.tasc_session_prefill(model, sess, np.concatenate(prompts), np.cumsum([0] + lens).astype(np.int64), 1)
    drafts = rng.integers(0, V, (B, max(ks))).astype(np.int32)
    drafts[::4, 2] = V - 1                   # the row whose list ends the table
    got = {}
    for k in ks:
        print(f"batch {B} vocab {V} k {k}", flush=True)
        z = torch.full((B, k + 1, V), -7.0, dtype=torch.float32, device="cuda")
        em = torch.zeros((B, k + 1), dtype=torch.int32, device="cuda")
        d = torch.from_numpy(np.ascontiguousarray(drafts[:, :k])).cuda() if k else None
        T.tasc_verify_step(model, sess, d, k, None, em, z)
        torch.cuda.synchronize()
        got[k] = z.cpu().numpy()
    for a, b in zip(ks, ks[1:]):             # the same bits whatever the kernel and the tile shape
        assert (got[b][:, :a + 1] == got[a]).all()
    om = OM.OracleModel(cfg, weights)
    for b in (0, 4, B - 1):
        c = om.new_cache(max_len)
        om.forward(prompts[b].tolist(), c, last_only=True)
        c.length = lens[b]
        first = int(T.tasc_session_get_tokens(sess, b)[-1])
        z = om.forward([first] + drafts[b].tolist(), c)
        assert float(np.abs(got[ks[-1]][b].astype(np.float64) - z).max()) <= 5e-2    # one bf16 layer: the bound of the other parity tests
