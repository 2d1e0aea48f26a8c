"""What an order of the counting stage leaves beside its positions for the order above: documents that end at and around the multiples of 8, of a
wave's 64 positions and of a chunk, windows that recur in their chunk, in another one only, and never, and a last chunk of a few positions;
tables bit-exact against the oracle, up to the longest order."""
import numpy as np
import pytest

from oracle import ngram as ON

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("length,vocab,n_max", [(7, 20, 4), (2048 + 3, 40_000, 8), (3 * 2048, 60_000, 8), (256 * 8192 + 5, 40_000, 5), (257 * 8192, 150_000, 7)])
def test_marks(length, vocab, n_max):
    import paper_2602_24174_amd as T
    rng = np.random.default_rng(length)
    phrases = [rng.integers(0, vocab, rng.integers(2, 12)) for _ in range(max(2, length // 40))]        # most of them twice or so
    tok = np.concatenate([phrases[i] for i in rng.integers(0, len(phrases), length)])[:length]
    hit = rng.random(length) < 0.05
    tok[hit] = rng.integers(0, vocab, int(hit.sum()))
    near = np.concatenate([m * rng.integers(1, length // m + 1, 1 + length // m // 4) for m in (8, 64, 2048, 8192) if length >= m] or [[3]])
    cuts = np.unique(np.clip(near + rng.integers(-7, 8, near.size), 0, length))
    off = np.concatenate([[0], cuts, [length]]).astype(np.int64)
    tok = tok.astype(np.int32)
    for p_min in (2, 3):
        ng = T.tasc_ngram_build(tok, off, vocab, n_max, p_min)
        st = T.tasc_ngram_get_stats(ng)
        for n in range(2, n_max + 1):
            grams, counts = ON.count_windows_sorted(tok, off, n)
            rows, got = T.tasc_ngram_export(ng, n)
            keep = counts >= p_min
            print(f"{length} order {n} p_min {p_min}: {len(counts)} distinct, {int(keep.sum())} kept", flush=True)
            assert st.distinct[n] == len(counts) and st.windows[n] == counts.sum()
            assert (rows == np.asarray(grams).reshape(-1, n)[keep]).all() and (got == counts[keep]).all()
