"""Drafts where a proposal reads all positions of the sequence instead of the bucket of its last token: few proposals over short
sequences, up to the line (one proposal, room for 512 tokens) and beyond it; and lambda 1, where the context has no part."""
import numpy as np
import pytest

import workload as W
from oracle import ngram as ON

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("room,k,lam", [(120, 4, 300), (120, 5, 300), (512, 1, 300), (513, 1, 300), (512, 1, 0),
                                        (512, 8, 65536), (2000, 1, 65536)])
def test_drafts_without_buckets(room, k, lam):
    import torch
    import paper_2602_24174_amd as T
    from gpu_util import Rig
    V = 512
    probe = W.get_config("cfg1").scaled(vocab=V, n_max=4, gen_len=8, prompt_len=room - 40)
    ref = ON.build_tables_flat(*W.make_corpus(probe), V, 4, probe.p_min)
    rng = np.random.default_rng(room + k)
    few = rng.integers(0, V, 4)
    lengths = [n for n in (1, 2, 3, 63, 64, 65, 66, 400, room - 40) if n <= room - 40]
    prompts = [few[rng.integers(0, 4, n)] for n in lengths]                      # many places of the last token, a few successors
    prompts += [rng.integers(0, V, n) for n in lengths]                          # few or none
    prompts += [np.full(n, few[0]) for n in lengths]                             # every place
    prompts = [np.asarray(p, dtype=np.int32) for p in prompts]
    cfg = probe.scaled(batch=len(prompts))
    rig = Rig(cfg, max_rows=16)
    assert rig.max_len == room
    T.tasc_session_prefill(rig.model, rig.session, np.concatenate(prompts), np.cumsum([0] + [len(p) for p in prompts]).astype(np.int64),
                           cfg.gen_len)
    for p_min_ctx in (1, 2):
        drafts = torch.zeros((cfg.batch, k), dtype=torch.int32, device="cuda")
        T.tasc_draft(rig.ng, rig.session, T.spec_params(k, lam, p_min_ctx, 1), drafts)
        got = drafts.cpu().numpy()
        for b in range(cfg.batch):
            want = ON.draft(ref, T.tasc_session_get_tokens(rig.session, b), k, lam, p_min_ctx)
            assert got[b].tolist() == want, f"p_min_ctx {p_min_ctx} sequence {b}: {got[b].tolist()} vs oracle {want}"
