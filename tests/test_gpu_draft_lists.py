"""Drafts where the context source changes its way of counting: the last token occurs 62 to 67 times before the end (up to 64
occurrences are counted in the wave's lanes, more in the hash table), with few successors and with as many as occurrences;
sequences shorter than the longest context; 128-bit keys of 8 tokens."""
import numpy as np
import pytest

import workload as W
from oracle import ngram as ON

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("vocab,n_max", [(512, 2), (512, 4), (65536, 8)])
def test_drafts_at_list_edges(vocab, n_max):
    import torch
    import paper_2602_24174_amd as T
    from gpu_util import Rig
    probe = W.get_config("cfg1").scaled(vocab=vocab, n_max=n_max, gen_len=8, prompt_len=300)
    corpus = W.make_corpus(probe)
    ref = ON.build_tables_flat(*corpus, vocab, n_max, probe.p_min)
    rng = np.random.default_rng(vocab + n_max)
    A = ref.fallback                                    # what a context without a match proposes: the next proposal's last token
    others = np.setdiff1d(np.arange(vocab), [A])
    prompts = [[A], [int(others[3])], [A, A], [A, int(others[0]), A]]
    for times in (62, 63, 64, 65, 67):
        few = np.concatenate([[A], others[:3]])
        prompts.append(np.concatenate([rng.permutation(few) for _ in range(times)]))             # A: `times` times, 4 successors
        prompts.append(np.stack([np.full(times, A), rng.permutation(others)[:times]], 1).ravel())  # A: `times` successors
    prompts = [np.asarray(p, dtype=np.int32) for p in prompts]
    cfg = probe.scaled(batch=len(prompts))
    rig = Rig(cfg, max_rows=16)
    T.tasc_session_prefill(rig.model, rig.session, np.concatenate(prompts), np.cumsum([0] + [len(p) for p in prompts]).astype(np.int64),
                           cfg.gen_len)
    edges = set()
    for lam, p_min_ctx in ((0, 1), (0, 2), (49152, 1), (300, 2)):
        drafts = torch.zeros((cfg.batch, 8), dtype=torch.int32, device="cuda")
        T.tasc_draft(rig.ng, rig.session, T.spec_params(8, lam, p_min_ctx, 1), drafts)
        got = drafts.cpu().numpy()
        for b in range(cfg.batch):
            committed = T.tasc_session_get_tokens(rig.session, b)
            want = ON.draft(ref, committed, 8, lam, p_min_ctx)
            assert got[b].tolist() == want, f"lambda {lam} p_min_ctx {p_min_ctx} sequence {b}: {got[b].tolist()} vs oracle {want}"
            edges |= {int((np.asarray(committed)[:-1] == t).sum()) for t in [committed[-1], *want[:-1]]}
    assert {63, 64, 65} <= edges, f"list lengths met: {sorted(edges)}"
