"""Attention of long prompt chunks where its shape changes: prompts that end around a key tile, a wave's 32 and a workgroup's 128 (row, head)
pairs, group sizes of 1 to 7, both head sizes, in one chunk and in several: the second layer's keys and values, which hold every row's
attention of the first, against the float64 oracle, and a prompt's cache bit for bit the same beside other prompts."""
import numpy as np
import pytest

import workload as W
from oracle import model as OM

pytestmark = pytest.mark.gpu

EDGES = [1, 2, 16, 17, 31, 32, 33, 63, 64, 65, 95, 96, 97, 127, 128, 129, 191, 192, 193, 255, 256, 257, 300, 319, 320, 321, 383, 384, 385, 400, 18, 19]


@pytest.mark.parametrize("heads", [(4, 4, 64), (8, 4, 128), (6, 2, 64), (7, 1, 128), (14, 2, 64)])
@pytest.mark.parametrize("longer", [0, 420])
def test_second_layer_cache(heads, longer):
    import torch
    import paper_2602_24174_amd as T
    h, hk, hd = heads
    B, max_rows = 32, 20
    lens = [n + (longer if b % 2 else 0) for b, n in enumerate(EDGES)]
    max_len = max(lens) + 1 + 2 * max_rows
    # the rule: 128 pairs a workgroup are one workgroup per compute unit, and 64 pairs need no split of the keys
    ref = min(8192, B * (max_len - 2 * max_rows) * 3 // 4)
    assert B * hk * -(-(ref // B * h // hk) // 128) >= 256
    cfg = W.get_config("cfg1").scaled(dtype="bf16", n_layers=2, d_model=128, d_ffn=192, n_heads=h, n_kv_heads=hk, head_dim=hd, vocab=700,
                                      batch=B, n_docs=800)
    weights = W.make_model(cfg, W.make_corpus(cfg))
    rng = np.random.default_rng(h)
    model = T.tasc_model_create(cfg, weights, max_len)
    sess = T.tasc_session_create(model, B, max_len, max_rows)
    blocks, page = (max_len + 15) // 16, 2 * hk * 16 * hd
    om = OM.OracleModel(cfg, weights)
    prompts = [rng.integers(0, cfg.vocab, n).astype(np.int32) for n in lens]

    def cache(ps):
        T.tasc_session_prefill(model, sess, np.concatenate(ps), np.cumsum([0] + [len(p) for p in ps]).astype(np.int64), 1)
        torch.cuda.synchronize()
        return sess._kv_pool.view(torch.bfloat16).view(2, blocks, B, page)       # block j of sequence b: page j B + b
    pool = cache(prompts).clone()
    for b in (0, 5, 9, 14, 15, 21, 28, 29):
        n = lens[b]
        pages = pool[1, :-(-n // 16), b].float().cpu().numpy()
        k = pages[:, :page // 2].reshape(-1, hk, 16, hd).transpose(0, 2, 1, 3).reshape(-1, hk, hd)[:n]
        v = pages[:, page // 2:].reshape(-1, hk, hd, 16).transpose(0, 3, 1, 2).reshape(-1, hk, hd)[:n]
        c = om.new_cache(max_len)
        om.forward(prompts[b].tolist(), c, last_only=True)
        for name, got, want in (("keys", k, c.k[1, :n]), ("values", v, c.v[1, :n])):
            # bf16 activations through one layer and a projection: a few roundings of 2^-9 of the row's size
            err, size = np.abs(got - want).max(), np.abs(want).max()
            print(f"heads {heads} sequence {b} ({n} tokens) {name}: largest error {err:.2e} of {size:.2e}", flush=True)
            assert err <= 2.0 ** -6 * size
    mine = (3, 8, 15, 29)
    others = [p if b in mine else rng.integers(0, cfg.vocab, int(rng.integers(1, max_len - 2 * max_rows))).astype(np.int32) for b, p in enumerate(prompts)]
    again = cache(others)
    for b in mine:
        full = lens[b] // 16
        assert torch.equal(again[:, :full, b].view(torch.int16), pool[:, :full, b].view(torch.int16))
