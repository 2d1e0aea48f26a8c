"""The scratch that builds and enrichments leave to each other: several threads on streams of their own at a time, given back to the
library's other allocations on a full card, and given back on demand."""
import threading

import numpy as np
import pytest

import workload as W

pytestmark = pytest.mark.gpu


def _corpus(seed, length, vocab):
    import torch
    g = torch.Generator(device="cuda").manual_seed(seed)
    tok = (torch.rand(length, generator=g, device="cuda") ** 3 * vocab).int()
    off = np.arange(0, length + 200, 200, dtype=np.int64)
    off[-1] = length
    return tok, off


def _tables(T, ng, n_max):
    return [x.tobytes() for n in range(2, n_max + 1) for x in T.tasc_ngram_export(ng, n)]


def test_threads_and_streams():
    import torch
    import paper_2602_24174_amd as T
    jobs = [_corpus(s, length, vocab) + (vocab,) for s, (length, vocab) in enumerate([(300_000, 5000), (40_000, 200_000), (1_100_000, 900), (9000, 50)])]
    want = []
    for tok, off, vocab in jobs:
        m, text, o, _ = T.tasc_tok_enrich(tok, off, vocab, 3, 3)
        want.append((_tables(T, T.tasc_ngram_build(tok, off, vocab, 4, 3), 4), m, text.cpu().numpy().tobytes(), o.tobytes()))
    torch.cuda.synchronize()
    wrong = []

    def work(i):
        stream = torch.cuda.Stream()
        for r in range(6):
            j = (i + r) % len(jobs)
            tok, off, vocab = jobs[j]
            with torch.cuda.stream(stream):
                m, text, o, _ = T.tasc_tok_enrich(tok, off, vocab, 3, 3)
                got = (_tables(T, T.tasc_ngram_build(tok, off, vocab, 4, 3), 4), m, text.cpu().numpy().tobytes(), o.tobytes())
            if got != want[j]:
                wrong.append((i, r, j))
    threads = [threading.Thread(target=work, args=(i,)) for i in range(4)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not wrong, wrong


def test_given_back():
    """A model that needs more than is left on the card beside the kept block, its first allocations small and the third large."""
    import torch
    import paper_2602_24174_amd as T
    small = T.tasc_ngram_build(np.arange(100, dtype=np.int32), np.array([0, 100]), 100, 2, 1)       # (a table: scratch is kept)

    def keep():
        tok, off = _corpus(7, 60_000_000, 100_000)
        torch.cuda.empty_cache()
        T.tasc_ngram_build(tok, off, 100_000, 5, 8)
        del tok
        torch.cuda.empty_cache()
    T.tasc_config_set(T.TASC_CFG_KEEP_SCRATCH_KIB, 0)
    torch.cuda.empty_cache()
    before = torch.cuda.mem_get_info()[0]
    try:
        keep()
        assert before - torch.cuda.mem_get_info()[0] < 100 << 20                  # nothing stays
        T.tasc_config_set(T.TASC_CFG_KEEP_SCRATCH_KIB, 2 << 20)
        keep()
        kept = before - torch.cuda.mem_get_info()[0]
        print(f"{kept >> 20} MiB kept", flush=True)
        assert 1500 << 20 < kept <= 2100 << 20
        T.tasc_config_set(T.TASC_CFG_KEEP_SCRATCH_KIB, 1 << 20)
        assert before - torch.cuda.mem_get_info()[0] < 100 << 20
        T.tasc_config_set(T.TASC_CFG_KEEP_SCRATCH_KIB, 2 << 20)
        keep()
        # the card filled up but for one or two blocks of 256 MiB
        hog = []
        try:
            while True:
                hog.append(torch.empty(256 << 20, dtype=torch.uint8, device="cuda"))
        except torch.OutOfMemoryError:
            pass
        hog.pop()
        torch.cuda.empty_cache()
        cfg = W.get_config("cfg1").scaled(dtype="bf16", d_ffn=70_000, d_model=2048, n_heads=16, n_kv_heads=2, head_dim=128, n_layers=1, vocab=64)
        z = np.zeros((70_000, 2048), dtype=np.uint16)
        weights = {"embed": z[:64], "lm_head": z[:64], "gf": np.ones(2048, dtype=np.float32), "bias": None,
                   "layers": [{"wq": z[:2048], "wk": z[:256], "wv": z[:256], "wo": z[:2048], "wg": z, "wu": z, "wd": z.reshape(2048, 70_000),
                               "g1": np.ones(2048, dtype=np.float32), "g2": np.ones(2048, dtype=np.float32)}]}
        model = T.tasc_model_create(cfg, weights, 64)
        model.close()
    finally:
        hog = None
        torch.cuda.empty_cache()
        T.tasc_config_set(T.TASC_CFG_KEEP_SCRATCH_KIB, 2 << 20)
        small.close()
