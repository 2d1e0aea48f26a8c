"""Recorded verify steps against plain launches: what may change between two steps of one session without changing the step's
buffers must not be remembered by the recording."""
import numpy as np
import pytest

import workload as W

pytestmark = pytest.mark.gpu

MODELS = {
    "f32": dict(),                                                                     # the type-generic kernels
    "bf16": dict(dtype="bf16", n_layers=2, d_model=256, n_heads=4, n_kv_heads=2, head_dim=64, d_ffn=448, vocab=1000, batch=28,
                 prompt_len=40, n_docs=1500, n_max=4),                                 # the tiled ones
}


@pytest.mark.parametrize("name", list(MODELS))
def test_generate_lengths_on_one_session(name):
    """The number of tokens to generate changes from call to call, up and down; every call records or replays the same steps (the
    first one is long enough to record both kinds).  Tokens, steps and counters of plain launches."""
    import paper_2602_24174_amd as T
    from gpu_util import Rig
    cfg = W.get_config("cfg1").scaled(**dict(MODELS[name], gen_len=64))
    rig = Rig(cfg, max_rows=16)
    runs = {}
    try:
        for graph in (0, 1):
            T.tasc_config_set(T.TASC_CFG_STEP_GRAPH, graph)
            for i, (n, k) in enumerate([(6, None), (6, 0), (64, None), (3, 0), (40, 0), (9, None), (64, 0)]):
                print(f"{name} graph {graph}: {n} tokens, k {k}", flush=True)
                out, st, _ = rig.generate(k=k, max_new=n)
                runs[graph, i] = (out.copy(), st.steps, st.accepted, st.proposed, tuple(st.accept_hist),
                                  [len(T.tasc_session_get_tokens(rig.session, b)) for b in range(rig.batch)])
    finally:
        T.tasc_config_set(T.TASC_CFG_STEP_GRAPH, 1)
    for (graph, i), run in runs.items():
        assert (run[0] == runs[0, i][0]).all() and run[1:] == runs[0, i][1:], f"call {i}"
    assert (runs[1, 2][0][:, :40] == runs[1, 4][0]).all() and (runs[1, 2][0] == runs[1, 6][0]).all()


def test_kernel_family_changes_on_one_session():
    """TASC_CFG_TILED_PATH is switched between steps of one session: what a step wrote into the cache, bit for bit, says which
    kernels ran it, and it is what plain launches of the family then selected write."""
    import torch
    import paper_2602_24174_amd as T
    from gpu_util import Rig
    cfg = W.get_config("cfg1").scaled(**dict(MODELS["bf16"], gen_len=40, k=4))
    rig = Rig(cfg, max_rows=16)
    drafts = torch.zeros((cfg.batch, cfg.k), dtype=torch.int32, device="cuda")

    def cache_after_steps(graph, tiled):
        print(f"graph {graph} tiled {tiled}", flush=True)
        T.tasc_config_set(T.TASC_CFG_STEP_GRAPH, graph)
        T.tasc_config_set(T.TASC_CFG_TILED_PATH, 1)
        T.tasc_session_prefill(rig.model, rig.session, rig.prompts, rig.prompt_off, cfg.gen_len)
        T.tasc_config_set(T.TASC_CFG_TILED_PATH, tiled)
        for _ in range(4):
            T.tasc_draft(rig.ng, rig.session, rig.params(), drafts)
            T.tasc_verify_step(rig.model, rig.session, drafts, cfg.k)
        torch.cuda.synchronize()
        return rig.session._kv_pool.clone()

    try:
        plain = {t: cache_after_steps(0, t) for t in (1, 0)}
        assert not torch.equal(plain[0], plain[1]), "both families write the same bits: the test would compare nothing"
        for tiled in (1, 0, 1, 0):
            assert torch.equal(cache_after_steps(1, tiled), plain[tiled]), f"tiled {tiled}"
    finally:
        T.tasc_config_set(T.TASC_CFG_STEP_GRAPH, 1)
        T.tasc_config_set(T.TASC_CFG_TILED_PATH, 1)
