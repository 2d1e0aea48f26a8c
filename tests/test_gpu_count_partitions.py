"""The counting stage where its shape changes: chunks of 8192 positions and turned offsets (2 M tokens on), partitions with more
distinct n-grams than LDS slots, keys of exactly and of more than 64 bits and of all 128, token histograms of one and several ranges
of the vocabulary and of one too large for them, and the enrichment of a corpus long enough for all of it: bit-exact."""
import numpy as np
import pytest

from oracle import ngram as ON

pytestmark = pytest.mark.gpu


def _corpus(kind, length, vocab):
    rng = np.random.default_rng(length)
    if kind == "random":
        tok = rng.integers(0, vocab, length)
    elif kind == "top":                     # the largest ids only: keys whose bits are all set
        tok = vocab - 1 - (rng.random(length) < 0.3)
    else:
        phrases = [rng.integers(0, vocab, rng.integers(2, 9)) for _ in range(3000)]
        tok = np.concatenate([phrases[i] for i in np.minimum(rng.zipf(1.2, length // 2), 3000) - 1])[:length]
        hit = rng.random(tok.size) < 0.1
        tok[hit] = rng.integers(0, vocab, int(hit.sum()))
    cuts = np.sort(rng.integers(0, tok.size, 40))
    return tok.astype(np.int32), np.concatenate([[0], cuts, [tok.size]]).astype(np.int64)


@pytest.mark.parametrize("kind,length,vocab,n_max,p_min", [
    ("phrases", 256 * 8192 - 1, 30_000, 3, 3), ("phrases", 256 * 8192 + 1, 30_000, 3, 3), ("phrases", 2_300_000, 151_936, 5, 4),
    ("random", 1_500_000, 1_000_000, 2, 1), ("random", 1_000_000, 140_000, 4, 1), ("random", 2_200_000, 3, 8, 5),
    ("phrases", 60_000, 65_536, 8, 2), ("top", 50_000, 65_536, 8, 1), ("top", 9000, 2, 8, 1)])
def test_counts(kind, length, vocab, n_max, p_min):
    import paper_2602_24174_amd as T
    tok, off = _corpus(kind, length, vocab)
    ng = T.tasc_ngram_build(tok, off, vocab, n_max, p_min)
    st = T.tasc_ngram_get_stats(ng)
    for n in range(2, n_max + 1):
        grams, counts = ON.count_windows_sorted(tok, off, n)
        rows, got = T.tasc_ngram_export(ng, n)
        keep = counts >= p_min
        print(f"order {n}: {len(counts)} distinct, {int(keep.sum())} kept", flush=True)
        assert st.distinct[n] == len(counts) and st.windows[n] == counts.sum()
        assert (rows == np.asarray(grams)[keep]).all() and (got == counts[keep]).all()
        # contexts: total and most frequent successor (smallest among equals) of every run of equal heads
        g, c = np.asarray(grams)[keep].astype(np.int64), counts[keep].astype(np.int64)
        ctx, total, top, topc = T.tasc_ngram_export_contexts(ng, n)
        if len(g) == 0:
            assert len(ctx) == 0
            continue
        head = np.concatenate([[True], (g[1:, :-1] != g[:-1, :-1]).any(1)])
        first = np.flatnonzero(head)
        run = np.cumsum(head) - 1
        best = np.maximum.reduceat(c, first)
        succ = np.where(c == best[run], g[:, -1], np.iinfo(np.int64).max)
        assert (ctx == g[first, :-1]).all() and (total == np.add.reduceat(c, first)).all()
        assert (topc == best).all() and (top == np.minimum.reduceat(succ, first)).all()


@pytest.mark.parametrize("vocab", [36_864, 36_865, 151_936, 32 * 36_864, 32 * 36_864 + 1])
def test_token_counts(vocab):
    import paper_2602_24174_amd as T
    rng = np.random.default_rng(vocab)
    tok = rng.integers(0, vocab, 300_000)
    tok[::3] = rng.integers(vocab - 5, vocab, tok[::3].size)
    ng = T.tasc_ngram_build(tok.astype(np.int32), np.array([0, tok.size], dtype=np.int64), vocab, 2, 2)
    fallback, counts = T.tasc_ngram_unigram(ng, vocab)
    want = np.bincount(tok, minlength=vocab)
    assert (counts == want).all() and fallback == int(np.argmax(want))
    bad = tok.astype(np.int32)
    for v in (vocab, -1):
        bad[-1] = v
        with pytest.raises(T.TascError):
            T.tasc_ngram_build(bad, np.array([0, tok.size], dtype=np.int64), vocab, 2, 2)


def test_enrichment_of_a_long_corpus():
    """More blocks than their sums are added up without a scan, an n-gram that overlaps itself among the merges, more merges than the
    host waits for at a time."""
    import paper_2602_24174_amd as T
    from test_gpu_tok_enrich import _run_and_compare
    tok, off = _corpus("phrases", 4_300_000, 500)
    tok[1_000_000:1_200_001] = 9
    docs = [tok[a:b].tolist() for a, b in zip(off[:-1], off[1:])]
    merges = _run_and_compare(T, docs, 500, 2, 2, device=True)
    assert merges[0][0] == (9, 9), merges
    tok, off = _corpus("phrases", 6000, 50)
    _run_and_compare(T, [tok[a:b].tolist() for a, b in zip(off[:-1], off[1:])], 50, 3, 40)


@pytest.mark.parametrize("length", [8191, 8192, 8256, 70_001])
def test_unique_grams_leave_no_record(length):
    """p_min 1 keeps every n-gram, p_min 2 counts the unique ones of the higher orders without looking at them: the same distinct
    n-grams, the same counts, whatever lies across a wave's 64 positions or a chunk's end."""
    import paper_2602_24174_amd as T
    rng = np.random.default_rng(length)
    tok = rng.integers(0, 40, length)
    tok[rng.random(length) < 0.3] = rng.integers(0, 100_000)
    hit = rng.random(length) < 0.1
    tok[hit] = rng.integers(0, 100_000, int(hit.sum()))
    off = np.concatenate([[0], np.sort(rng.integers(0, length, 30)), [length]]).astype(np.int64)
    tok = tok.astype(np.int32)
    a, b = (T.tasc_ngram_build(tok, off, 100_000, 7, p) for p in (1, 2))
    sa, sb = T.tasc_ngram_get_stats(a), T.tasc_ngram_get_stats(b)
    for n in range(2, 8):
        ra, ca = T.tasc_ngram_export(a, n)
        rb, cb = T.tasc_ngram_export(b, n)
        assert sa.distinct[n] == sb.distinct[n] == len(ca) and (ra[ca > 1] == rb).all() and (ca[ca > 1] == cb).all()
