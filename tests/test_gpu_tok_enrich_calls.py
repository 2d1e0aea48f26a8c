"""tasc_tok_enrich called in ways the binding does not: results written over the corpus."""
import ctypes as C

import numpy as np
import pytest

from oracle import tok_enrich as OT

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("docs", [[[], [1, 2, 1, 2, 3], [], [], [1, 2], [5], []], [[1, 2, 1, 2, 1, 2], [4], [1, 2]]])
def test_in_place(docs):
    import paper_2602_24174_amd as T
    from paper_2602_24174_amd import binding as B
    vocab, n_max, budget = 8, 3, 2
    tok = np.array([t for d in docs for t in d], dtype=np.int32)
    off = np.cumsum([0] + [len(d) for d in docs]).astype(np.int64)
    rows, freq = np.zeros((budget, 1 + B.TASC_MAX_ORDER), np.int32), np.zeros(budget, np.int64)
    lens, n = np.zeros(budget + 1, np.int64), C.c_int32(0)
    B._check(B.lib().tasc_tok_enrich(B._ptr(tok), B._ptr(off), len(docs), vocab, n_max, budget, B.TASC_MEM_HOST, B._stream(None), B._ptr(rows),
                                     B._ptr(freq), B._ptr(lens), B._ptr(tok), B._ptr(off), C.byref(n)))
    want_m, want_docs, want_l = OT.enrich(docs, vocab, n_max, budget)
    assert n.value == len(want_m) and lens[:n.value + 1].tolist() == want_l
    assert off.tolist() == np.cumsum([0] + [len(d) for d in want_docs]).tolist()
    assert tok[:off[-1]].tolist() == [t for d in want_docs for t in d]


@pytest.mark.parametrize("n_max", [2, 3, 5, 8])
@pytest.mark.parametrize("period", [1, 2, 3])
def test_long_runs_of_overlapping_occurrences(period, n_max):
    """Runs that end around the 64 positions a wave takes at a time, inside one output and over several, with a break now and then."""
    import paper_2602_24174_amd as T
    from test_gpu_tok_enrich import _run_and_compare
    rng = np.random.default_rng(10 * period + n_max)
    docs = [[int(t) for t in np.arange(n + 1) % period] for n in (0, 62, 63, 64, 65, 130, 700)]
    noisy = np.arange(1500) % period
    noisy[rng.integers(0, 1500, 8)] = 5
    docs += [noisy.tolist(), [7] * 300, [3, 4]]
    _run_and_compare(T, docs, 9, n_max, 6, device=True)


@pytest.mark.parametrize("n_max", [2, 5, 8])
def test_orders_in_groups(n_max):
    """Orders counted all together, in groups of some and one by one: the same merges, texts and boundaries."""
    import paper_2602_24174_amd as T
    from test_gpu_tok_enrich import _run_and_compare
    rng = np.random.default_rng(n_max)
    phrases = [rng.integers(0, 300, rng.integers(2, 9)).tolist() for _ in range(40)]
    docs = [sum((phrases[i] for i in rng.zipf(1.3, 60) % 40), []) for _ in range(40)]
    # 4 to 8 chunks of 2048 positions and 256 partitions: 8 or 16 bytes a position and 640 a chunk
    order = -(-sum(map(len, docs)) // 2048) * (2048 * (16 if n_max == 8 else 8) + 640)
    try:
        for orders in (1, 2, 3, 7):
            T.tasc_config_set(T.TASC_CFG_BUILD_LIST_KIB, 0 if orders == 1 else (orders * order + order // 2) // 1024)
            _run_and_compare(T, docs, 300, n_max, 5)
    finally:
        T.tasc_config_set(T.TASC_CFG_BUILD_LIST_KIB, 8 << 20)


def test_memory_does_not_grow_with_the_orders():
    """24 M tokens, orders 2 to 8: records of every order at once would be 3.3 GB; the result is the same on a card with 2.4 GiB left."""
    import torch
    import paper_2602_24174_amd as T
    g = torch.Generator(device="cuda").manual_seed(5)
    tok = (torch.rand(24_000_000, generator=g, device="cuda") ** 4 * 40_000).int()
    off = np.arange(0, tok.numel() + 1, 240, dtype=np.int64)
    torch.cuda.empty_cache()
    want = T.tasc_tok_enrich(tok, off, 40_000, 8, 2)
    free = torch.cuda.mem_get_info()[0]
    hog = torch.empty(free - (2400 << 20) - 4 * tok.numel(), dtype=torch.uint8, device="cuda")      # (the result's text is allocated too)
    try:
        got = T.tasc_tok_enrich(tok, off, 40_000, 8, 2)
    finally:
        del hog
        torch.cuda.empty_cache()
    assert got[0] == want[0] and (got[2] == want[2]).all() and torch.equal(got[1], want[1])
