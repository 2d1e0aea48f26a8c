"""Attention of the type-generic kernels where every product of a key tile overflows to -inf: such a tile weighs nothing, between
others and as the first one, for (row, tile) pairs that meet in LDS and for rows that go through their tiles one by one."""
import numpy as np
import pytest

import workload as W
from oracle import model as OM

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("k", [4, 15])                    # 5 x 3 (row, tile) pairs of at most 32 in LDS, 16 x 3
@pytest.mark.parametrize("first", [0, 64])
def test_tile_of_minus_infinity(k, first):
    import torch
    import paper_2602_24174_amd as T
    cfg = W.get_config("cfg1").scaled(n_layers=1, prompt_len=130, k=k, n_docs=300)
    hd, far, max_len = cfg.head_dim, cfg.vocab - 1, 200
    # token `far` and the others differ in the embedding's first two dimensions; in the pair of head dimensions that turns slowest (by at
    # most 0.03 here) the others' queries are 3e20, the keys of `far` -3e20 and the others' keys 0
    weights = W.make_model(cfg, W.make_corpus(cfg))
    weights["embed"][:, :2] = (0.0, 1.0)
    weights["embed"][far] = 0.0
    weights["embed"][far, 0] = 1.0
    for name, dim, size in (("wq", 1, 3e19), ("wk", 0, -3e19)):
        m = weights["layers"][0][name].reshape(-1, hd, cfg.d_model)
        m[:, [hd // 2 - 1, hd - 1]] = 0.0
        m[:, hd // 2 - 1, dim] = size
    model = T.tasc_model_create(cfg, weights, max_len)
    sess = T.tasc_session_create(model, 1, max_len, 16)
    rng = np.random.default_rng(k)
    prompt = rng.integers(0, far, cfg.prompt_len).astype(np.int32)
    prompt[first:first + 64] = far
    drafts = rng.integers(0, far, (1, k)).astype(np.int32)
    T.tasc_session_prefill(model, sess, prompt, np.array([0, prompt.size], dtype=np.int64), 1)
    z = torch.full((1, k + 1, cfg.vocab), float("nan"), dtype=torch.float32, device="cuda")
    T.tasc_verify_step(model, sess, torch.from_numpy(drafts).cuda(), k, None, None, z)
    om = OM.OracleModel(cfg, weights)
    cache = om.new_cache(max_len)
    om.forward(prompt.tolist(), cache)
    cache.length = prompt.size
    seq = T.tasc_session_get_tokens(sess, 0)
    want = om.forward([int(seq[prompt.size])] + drafts[0].tolist(), cache)
    err = np.abs(z[0].cpu().numpy() - want).max()
    print(f"k {k}, keys of -inf from {first}: largest error {err:.2e}", flush=True)
    assert err <= 1e-3                                    # the fp32 bound of the workload
