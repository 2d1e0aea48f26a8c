"""Packing of the weights: the same model from host memory, from device memory, and once more after the others have run and gone."""
import ctypes as C

import numpy as np
import pytest

import workload as W
from oracle import model as OM

pytestmark = pytest.mark.gpu

SHAPES = {
    "f32": dict(d_model=72, n_heads=3, n_kv_heads=1, head_dim=24, d_ffn=176),      # 11 blocks of 16 gate rows
    "bf16_small": dict(dtype="bf16", d_model=96, n_heads=3, n_kv_heads=3, head_dim=32, d_ffn=160),
    "bf16_tiled": dict(dtype="bf16", d_model=192, n_heads=4, n_kv_heads=2, head_dim=64, d_ffn=448, batch=20),
}


def _from_device(T, torch, cfg, weights, max_pos):
    from paper_2602_24174_amd import binding as B
    alive = []

    def dev(a):
        alive.append(torch.from_numpy(np.ascontiguousarray(a).view(np.uint8).reshape(-1)).cuda())
        return alive[-1].data_ptr()

    def layers(name):
        a = (C.c_void_p * cfg.n_layers)(*[dev(y[name]) for y in weights["layers"]])
        alive.append(a)
        return C.cast(a, C.POINTER(C.c_void_p))

    b = weights["bias"]
    w = B.WeightPtrs(B.TASC_MEM_DEVICE, dev(weights["embed"]), dev(weights["lm_head"]), dev(weights["gf"]),
                     *[layers(n) for n in ("wq", "wk", "wv", "wo", "wg", "wu", "wd", "g1", "g2")],
                     dev(b["rowptr"]), dev(b["col"]), dev(b["val"]), dev(b["base"]))
    desc = B.ModelDesc(B.TASC_BF16 if cfg.dtype == "bf16" else B.TASC_F32, cfg.n_layers, cfg.d_model, cfg.n_heads, cfg.n_kv_heads,
                       cfg.head_dim, cfg.d_ffn, cfg.vocab, max_pos, cfg.rope_theta, cfg.rms_eps)
    out = C.c_void_p()
    torch.cuda.synchronize()
    assert T.lib().tasc_model_create(C.byref(desc), C.byref(w), C.byref(out)) == 0
    return B.Model(out.value, desc)


@pytest.mark.parametrize("name", list(SHAPES))
def test_same_model_three_times(name):
    import torch
    import paper_2602_24174_amd as T
    cfg = W.get_config("cfg1").scaled(**dict(dict(n_layers=3, vocab=300, batch=2, n_docs=400, prompt_len=20, gen_len=24, k=3), **SHAPES[name]))
    weights = W.make_model(cfg, W.make_corpus(cfg))
    prompts, off = W.make_prompts(cfg)
    max_len = cfg.prompt_len + cfg.gen_len + 32
    drafts = torch.from_numpy(np.random.default_rng(5).integers(0, cfg.vocab, (cfg.batch, cfg.k)).astype(np.int32)).cuda()
    got = []
    for where in ("host", "device", "host again"):
        print(f"{name}: {where}", flush=True)
        model = _from_device(T, torch, cfg, weights, max_len) if where == "device" else T.tasc_model_create(cfg, weights, max_len)
        sess = T.tasc_session_create(model, cfg.batch, max_len, 16)
        z = torch.zeros((cfg.batch, cfg.k + 1, cfg.vocab), dtype=torch.float32, device="cuda")
        T.tasc_session_prefill(model, sess, prompts, off, 1)
        T.tasc_verify_step(model, sess, drafts, cfg.k, None, None, z)
        torch.cuda.synchronize()
        got.append((z.cpu().numpy(), [int(T.tasc_session_get_tokens(sess, b)[-1]) for b in range(cfg.batch)]))
        out = torch.zeros((cfg.batch, cfg.gen_len), dtype=torch.int32, device="cuda")
        T.tasc_generate(model, None, sess, prompts, off, cfg.gen_len, T.spec_params(0), out)
        del sess, model
    for z, first in got[1:]:
        assert (z == got[0][0]).all() and first == got[0][1]
    om = OM.OracleModel(cfg, weights)
    for b in range(2):
        c = om.new_cache(max_len)
        p = prompts[off[b]:off[b + 1]].tolist()
        om.forward(p, c, last_only=True)
        c.length = len(p)
        want = om.forward([got[0][1][b]] + drafts[b].tolist(), c)
        err = float(np.abs(got[0][0][b].astype(np.float64) - want).max())
        assert err <= (1e-3 if cfg.dtype == "f32" else 5e-2)        # the bounds of the other parity tests
