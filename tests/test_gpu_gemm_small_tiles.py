"""Products on 128 x 128 tiles, more of them than the device has compute units: rotation at every head size (also with rows that begin at any
slot of a page, on both sides of a page's end), SwiGLU, residual and k-slices, against the same rows on 256-row tiles and against the oracle."""
import numpy as np
import pytest

import workload as W
from oracle import model as OM

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("heads,d_model", [((345, 4, 32), 128), ((174, 1, 64), 128), ((84, 2, 128), 1536)])
def test_more_small_tiles_than_compute_units(heads, d_model):
    import torch
    import paper_2602_24174_amd as T
    H, Hkv, hd = heads
    B, max_rows, V = 290, 17, 1000
    cfg = W.get_config("cfg1").scaled(dtype="bf16", n_layers=1, d_model=d_model, n_heads=H - H % Hkv, n_kv_heads=Hkv, head_dim=hd, d_ffn=5632, vocab=V, batch=B)
    rng = np.random.default_rng(11)
    weights = W.make_model(cfg)
    lens = [int(n) for n in rng.integers(3, 40, B)]
    prompts = [rng.integers(0, V, n).astype(np.int32) for n in lens]
    max_len = 40 + 1 + 2 * max_rows
    model = T.tasc_model_create(cfg, weights, max_len)
    sess = T.tasc_session_create(model, B, max_len, max_rows)
    T.tasc_session_prefill(model, sess, np.concatenate(prompts), np.cumsum([0] + lens).astype(np.int64), 1)
    drafts = rng.integers(0, V, (B, 6)).astype(np.int32)
    got = {}
    for k in (0, 1, 6):          # 290 rows (3 row tiles x 88 column tiles), 580 and 2030 (larger tiles)
        print(f"heads {heads} k {k}", flush=True)
        z = torch.full((B, k + 1, V), -7.0, dtype=torch.float32, device="cuda")
        d = torch.from_numpy(np.ascontiguousarray(drafts[:, :k])).cuda() if k else None
        T.tasc_verify_step(model, sess, d, k, None, None, z)
        torch.cuda.synchronize()
        got[k] = z.cpu().numpy()
    assert (got[1][:, 0] == got[0][:, 0]).all() and (got[6][:, :2] == got[1]).all()
    om = OM.OracleModel(cfg, weights)
    for b in (0, 100, B - 1):
        c = om.new_cache(max_len)
        om.forward(prompts[b].tolist(), c, last_only=True)
        c.length = lens[b]
        first = int(T.tasc_session_get_tokens(sess, b)[-1])
        z = om.forward([first] + drafts[b].tolist(), c)
        worst = float(np.abs(got[6][b].astype(np.float64) - z).max())
        print(f"heads {heads} sequence {b}: max |logit - oracle| = {worst:.3e}", flush=True)
        assert worst <= 5e-2     # bf16 matrix operands, one layer: the bound of the other bf16 parity tests
