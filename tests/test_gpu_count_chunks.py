"""The counting stage at the edges of its 2048-position chunks: corpora of one chunk more or less, windows that span two chunks,
chunks whose n-grams are all distinct (more kept ones than a workgroup collects before it appends), one n-gram for the whole
corpus, and counts that reach p_min in a chunk of their own or only over several: tables bit-exact against the oracle."""
import numpy as np
import pytest

from oracle import ngram as ON

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("length", [2047, 2048, 2049, 6145, 40_000])
@pytest.mark.parametrize("kind", ["distinct", "constant", "mixed"])
def test_chunk_edges(length, kind):
    import paper_2602_24174_amd as T
    from test_gpu_ngram import _compare_tables
    vocab, n_max = 50_000, 4
    rng = np.random.default_rng(length)
    if kind == "distinct":
        tok = rng.permutation(vocab)[:length]
    elif kind == "constant":
        tok = np.full(length, 7)
    else:                        # a few phrases over and over, every tenth token random
        phrases = [rng.integers(0, 300, rng.integers(2, 8)) for _ in range(40)]
        tok = np.concatenate([phrases[i] for i in rng.zipf(1.3, length) % 40])[:length]
        hit = rng.random(length) < 0.1
        tok[hit] = rng.integers(0, vocab, int(hit.sum()))
    tok = tok.astype(np.int32)
    cuts = np.sort(rng.integers(0, length, 5))
    off = np.concatenate([[0], cuts, [length]]).astype(np.int64)
    docs = [tok[a:b].tolist() for a, b in zip(off[:-1], off[1:])]
    for p_min in (1, 2, 5):
        print(f"{kind} {length} p_min {p_min}", flush=True)
        ng = T.tasc_ngram_build(tok, off, vocab, n_max, p_min)
        ref = ON.build_tables(docs, vocab, n_max, p_min)
        _compare_tables(T, ng, ref, n_max, vocab)
        st = T.tasc_ngram_get_stats(ng)
        for n in range(2, n_max + 1):
            grams = [tuple(d[i:i + n]) for d in docs for i in range(len(d) - n + 1)]
            assert st.windows[n] == len(grams) and st.distinct[n] == len(set(grams))


@pytest.mark.parametrize("p_min,kib", [(1, 0), (2, 240), (1, 710), (30, 0), (300, 0), (10_000, 0)])
def test_orders_in_groups(p_min, kib):
    """The orders of a build in several groups, whose lists share their memory and whose context tables share the counting table's:
    one order a group, two and three, orders without kept n-grams, builds without any; tables bit-exact against the oracle."""
    import paper_2602_24174_amd as T
    from test_gpu_ngram import _compare_tables
    vocab, n_max, length = 3000, 6, 30_000
    rng = np.random.default_rng(21)
    phrases = [rng.integers(0, vocab, rng.integers(2, 6)) for _ in range(60)]
    tok = np.concatenate([phrases[i] for i in rng.zipf(1.2, length) % 60])[:length].astype(np.int32)
    hit = rng.random(length) < 0.2
    tok[hit] = rng.integers(0, vocab, int(hit.sum()))
    off = np.array([0, 9000, 9001, 20_000, length], dtype=np.int64)
    ref = ON.build_tables([tok[a:b].tolist() for a, b in zip(off[:-1], off[1:])], vocab, n_max, p_min)
    kept = []
    try:
        for k in (kib, 8 << 20):
            print(f"p_min {p_min}: {k} KiB", flush=True)
            T.tasc_config_set(T.TASC_CFG_BUILD_LIST_KIB, k)
            ng = T.tasc_ngram_build(tok, off, vocab, n_max, p_min)
            _compare_tables(T, ng, ref, n_max, vocab)
            st = T.tasc_ngram_get_stats(ng)
            kept.append([(st.windows[n], st.distinct[n], st.kept[n], st.contexts[n]) for n in range(2, n_max + 1)])
    finally:
        T.tasc_config_set(T.TASC_CFG_BUILD_LIST_KIB, 8 << 20)
    assert kept[0] == kept[1]
    if p_min == 300:
        assert kept[0][0][2] > 0 and kept[0][-1][2] == 0, "an order with kept n-grams and one without"
