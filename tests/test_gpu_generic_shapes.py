"""Verify steps of the type-generic kernels beyond the tiny model: norms along with the products and in launches of their own, lanes of 4 and
of 8 columns, vocabularies whose strips are cut and not, and attention of rows that leave waves idle over more (row, tile) pairs than meet
in LDS at a time, both types: logits against the float64 oracle, and a row scored alone bit for bit the same row of a step of many."""
import numpy as np
import pytest

import workload as W
from oracle import model as OM

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,d,heads,vocab,prompt,k,batch", [
    ("f32", 256, (4, 2, 32), 16_385, 40, 4, 2), ("f32", 264, (4, 4, 32), 700, 600, 4, 1), ("f32", 520, (2, 1, 256), 8200, 700, 8, 1),
    ("f32", 1032, (3, 1, 64), 8193, 200, 11, 2), ("f32", 512, (8, 4, 64), 20_000, 129, 15, 3), ("f32", 96, (4, 4, 32), 300, 1100, 2, 1),
    ("f32", 96, (2, 2, 128), 300, 1100, 5, 1), ("f32", 96, (2, 2, 72), 300, 1100, 9, 2), ("f32", 96, (2, 2, 32), 300, 1100, 15, 1),
    ("bf16", 200, (4, 2, 32), 900, 600, 4, 1), ("bf16", 328, (4, 2, 64), 17_000, 300, 8, 2), ("bf16", 584, (3, 3, 72), 1000, 700, 10, 3)])
def test_logits_and_bits(dtype, d, heads, vocab, prompt, k, batch):
    import torch
    import paper_2602_24174_amd as T
    from gpu_util import Rig
    h, hk, hd = heads
    cfg = W.get_config("cfg1").scaled(dtype=dtype, n_layers=2, d_model=d, n_heads=h, n_kv_heads=hk, head_dim=hd, d_ffn=528, vocab=vocab,
                                      prompt_len=prompt, gen_len=1, k=k, batch=batch, n_docs=300)
    rig = Rig(cfg, with_ngram=False)
    T.tasc_session_prefill(rig.model, rig.session, rig.prompts, rig.prompt_off, 1)      # one token: the steps below commit nothing
    rng = np.random.default_rng(prompt)
    drafts = rng.integers(0, vocab, (batch, k)).astype(np.int32)

    def step(n):
        z = torch.full((batch, n + 1, vocab), float("nan"), dtype=torch.float32, device="cuda")
        T.tasc_verify_step(rig.model, rig.session, torch.from_numpy(drafts[:, :n].copy()).cuda() if n else None, n, None, None, z)
        return z.cpu().numpy()
    many, few, alone = step(k), step(1), step(0)
    assert (alone[:, 0] == many[:, 0]).all() and (few == many[:, :2]).all()
    om = OM.OracleModel(cfg, rig.weights)
    for b in range(batch):
        cache = om.new_cache(rig.max_len)
        seq = T.tasc_session_get_tokens(rig.session, b)
        om.forward(seq[:prompt].tolist(), cache)
        cache.length = prompt
        want = om.forward([int(seq[prompt])] + drafts[b].tolist(), cache)
        err = np.abs(many[b] - want).max()
        print(f"{dtype} d {d} heads {heads} vocab {vocab} prompt {prompt} k {k}: largest error {err:.2e}", flush=True)
        assert err <= (1e-3 if dtype == "f32" else 5e-2)   # the workloads' bounds
