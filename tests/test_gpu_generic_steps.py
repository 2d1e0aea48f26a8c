"""Verify steps of the type-generic kernels where their shape changes: positions around a key tile's end, (row, tile) pairs that meet in
LDS and rows that go through their tiles one by one, positions past the page ids a wave holds, head sizes from 8 to 256,
vocabularies split finely and not, rows past a chunk of 8: logits against the float64 oracle, and a row scored alone (k = 0) bit for
bit the same row of a step of many."""
import numpy as np
import pytest

import workload as W
from oracle import model as OM

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("heads,vocab,prompt,k,batch", [
    ((4, 4, 32), 512, 63, 4, 1), ((4, 2, 8), 130, 64, 4, 3), ((2, 1, 256), 900, 65, 8, 2), ((6, 3, 72), 5000, 130, 15, 1),
    ((4, 4, 32), 512, 500, 4, 1), ((2, 2, 64), 300, 1030, 2, 2), ((2, 2, 64), 2000, 1030, 9, 1)])
def test_logits_and_bits(heads, vocab, prompt, k, batch):
    import torch
    import paper_2602_24174_amd as T
    from gpu_util import Rig
    h, hk, hd = heads
    cfg = W.get_config("cfg1").scaled(n_layers=2, d_model=96, n_heads=h, n_kv_heads=hk, head_dim=hd, d_ffn=176, vocab=vocab, prompt_len=prompt,
                                      gen_len=1, k=k, batch=batch, n_docs=300)
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
        print(f"heads {heads} vocab {vocab} prompt {prompt} k {k}: largest error {err:.2e}", flush=True)
        assert err <= 1e-3                  # the fp32 bound of the workload; fp32 sums of at most 1024 terms leave about 1e-5
