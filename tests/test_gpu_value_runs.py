"""Values that the rotation's epilogue stores for rows of several sequences at once: the first sequence owns page 0, its last row sits at an even slot
and the second sequence's first row at the slot behind that, in a page of its own, the row after it not.  Every sequence's logits are those of
a step of another row count (whose rows meet elsewhere) bit for bit, and the first sequences' those of the oracle."""
import numpy as np
import pytest

import workload as W
from oracle import model as OM

pytestmark = pytest.mark.gpu

SERVING = ((16, 2, 128), 2048, 256)        # more 128 x 128 tiles of q/k/v than compute units from 1665 rows on
WIDE32, WIDE64, WIDE128 = ((344, 4, 32), 128, 290), ((174, 1, 64), 128, 290), ((84, 2, 128), 1536, 290)       # ... from 257 rows on; 256 x 256 tiles at 2320


@pytest.mark.parametrize("shape,k,other,first", [
    (SERVING, 7, 6, (7, 15, 30)), (SERVING, 6, 5, (8, 31, 15)),
    (WIDE128, 0, 1, (4, 5, 9)), (WIDE128, 0, 1, (14, 31, 2)), (WIDE64, 0, 1, (4, 5, 9)), (WIDE32, 0, 1, (10, 27, 3)),
    (WIDE128, 7, 6, (7, 15, 31)), (WIDE64, 7, 6, (7, 15, 47)), (WIDE32, 7, 6, (7, 31, 2))])
def test_rows_of_two_sequences(shape, k, other, first):
    import torch
    import paper_2602_24174_amd as T
    (H, Hkv, hd), d_model, B = shape
    max_rows, V = 8, 1000
    cfg = W.get_config("cfg1").scaled(dtype="bf16", n_layers=1, d_model=d_model, n_heads=H, n_kv_heads=Hkv, head_dim=hd, d_ffn=1024, vocab=V, batch=B)
    rng = np.random.default_rng(k)
    weights = W.make_model(cfg)
    lens = list(first) + [int(n) for n in rng.integers(3, 48, B - len(first))]
    prompts = [rng.integers(0, V, n).astype(np.int32) for n in lens]
    max_len = 48 + 1 + 2 * max_rows
    model = T.tasc_model_create(cfg, weights, max_len)
    sess = T.tasc_session_create(model, B, max_len, max_rows)
    T.tasc_session_prefill(model, sess, np.concatenate(prompts), np.cumsum([0] + lens).astype(np.int64), 1)
    drafts = rng.integers(0, V, (B, max(k, other))).astype(np.int32)
    got = {}
    for n in (k, other):         # (the step under test first: its slots hold nothing yet)
        print(f"heads {shape[0]} k {n} lengths {first}", flush=True)
        z = torch.full((B, n + 1, V), -7.0, dtype=torch.float32, device="cuda")
        d = torch.from_numpy(np.ascontiguousarray(drafts[:, :n])).cuda() if n else None
        T.tasc_verify_step(model, sess, d, n, None, None, z)
        torch.cuda.synchronize()
        got[n] = z.cpu().numpy()
    rows = min(k, other) + 1
    wrong = np.nonzero((got[k][:, :rows] != got[other][:, :rows]).any(axis=(1, 2)))[0]
    om = OM.OracleModel(cfg, weights)
    far = []
    for b in range(len(first)):
        c = om.new_cache(max_len)
        om.forward(prompts[b].tolist(), c, last_only=True)
        c.length = lens[b]
        z = om.forward([int(T.tasc_session_get_tokens(sess, b)[-1])] + drafts[b, :k].tolist(), c)
        far.append(float(np.abs(got[k][b].astype(np.float64) - z).max()))
    print(f"sequences that differ: {wrong.tolist()}; max |logit - oracle| of the first: {far}", flush=True)
    assert wrong.size == 0
    assert max(far) <= 5e-2      # bf16 matrix operands, one layer: the bound of the other bf16 parity tests
