"""Corpora made against the counting stage's hash: more n-grams of one hash than a probe sequence is long (keys of more than 64 bits), more
n-grams that share the half of the hash that ranges are cut by than a table has slots (keys of 64 bits): counted like any other."""
import numpy as np
import pytest

from oracle import ngram as ON

pytestmark = pytest.mark.gpu
M64 = (1 << 64) - 1


def _lo_of(h, hi):                                # the key's lower half, given its hash and its upper half
    x = h * 0x319642B2D24D8EC3 & M64
    x ^= (x >> 29) ^ (x >> 58)
    x = x * 0x96DE1B173F119089 & M64
    x ^= x >> 32
    return (x - hi * 0x9E3779B97F4A7C15) & M64


def _corpus(kind, rng):
    """Documents of one 8-gram each, some of them more than once."""
    if kind == "wide":                            # 200 keys of 128 bits, one hash
        bits, h = 16, int(rng.integers(0, 1 << 63))
        keys = []
        for _ in range(200):
            hi = int(rng.integers(0, 1 << 63))
            keys.append(hi << 64 | _lo_of(h, hi))
    else:                                         # 6000 keys of 64 bits, one upper half of the hash
        bits, top = 8, int(rng.integers(0, 1 << 31))
        keys = [_lo_of(top << 32 | int(low), 0) for low in rng.choice(1 << 32, 6000, replace=False)]
    docs = np.array([[k >> (bits * j) & ((1 << bits) - 1) for j in range(8)] for k in keys], dtype=np.int32)
    assert len(np.unique(docs, axis=0)) == len(keys)
    docs = docs[rng.permutation(np.repeat(np.arange(len(keys)), rng.integers(1, 4, len(keys))))]
    other = rng.integers(0, 1 << bits, (500, 8)).astype(np.int32)
    return np.concatenate([other[:250], docs, other[250:]]), bits


@pytest.mark.parametrize("kind,seed", [("wide", 1), ("wide", 2), ("narrow", 3)])
def test_equal_hashes(kind, seed):
    import paper_2602_24174_amd as T
    docs, bits = _corpus(kind, np.random.default_rng(seed))
    tok, off = docs.reshape(-1), np.arange(0, docs.size + 1, 8, dtype=np.int64)
    for p_min in (1, 2):
        ng = T.tasc_ngram_build(tok, off, 1 << bits, 8, p_min)
        st = T.tasc_ngram_get_stats(ng)
        for n in range(2, 9):
            grams, counts = ON.count_windows_sorted(tok, off, n)
            rows, got = T.tasc_ngram_export(ng, n)
            keep = counts >= p_min
            print(f"{kind} p_min {p_min} order {n}: {len(counts)} distinct", flush=True)
            assert st.distinct[n] == len(counts)
            assert (rows == np.asarray(grams)[keep]).all() and (got == counts[keep]).all()
    # the most frequent one, found by the enrichment (keys of one more bit there: other hashes, unless the vocabulary leaves room)
    if kind == "wide":
        docs = docs[(docs < (1 << bits) - 2).all(1)]
        docs = np.concatenate([docs, docs[300:301], docs[300:301], docs[300:301]])
        uniq, counts = np.unique(docs, axis=0, return_counts=True)
        merges = T.tasc_tok_enrich(docs.reshape(-1), np.arange(0, docs.size + 1, 8, dtype=np.int64), (1 << bits) - 1, 8, 1)[0]
        top = counts.max()
        assert merges[0][1] == top and len(merges[0][0]) == 8 and merges[0][0] == min(tuple(int(t) for t in u) for u in uniq[counts == top])
