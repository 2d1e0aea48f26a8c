"""Merges found without counting every n-gram, against the oracle: several looks of the host, blocks of 4096 positions and their edges, rewards that
fall slowly and at once, buckets and lists that are all full (the n-grams are counted in full then), tokens that have a new id already."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _docs(kind, rng):
    if kind == "phrases":            # 13,000 tokens in outputs of 1 to 300, phrases by a power law, a tenth of the tokens replaced
        phrases = [rng.integers(0, 900, rng.integers(2, 9)) for _ in range(300)]
        text = np.concatenate([phrases[i] for i in np.minimum(rng.zipf(1.4, 4000) - 1, 299)])[:13_000]
        text = np.where(rng.random(text.size) < 0.1, rng.integers(0, 900, text.size), text)
    elif kind == "one phrase":       # the best n-gram is worth many times the second
        text = np.concatenate([np.r_[np.arange(20, 28), rng.integers(100, 900, 2)] for _ in range(900)])
    elif kind == "few":              # every pair is frequent
        text = rng.integers(0, 5, 9000)
    elif kind == "flat":             # none is
        text = rng.integers(0, 900, 9000)
    else:                            # "new ids": tokens that the merges are going to have
        text = np.concatenate([np.r_[1, 2, 900, 3, 901, 902, 4] for _ in range(600)])
    cuts = np.unique(np.r_[0, np.cumsum(rng.integers(1, 300, 400)), text.size])
    cuts = cuts[cuts <= text.size]
    return [text[a:b].tolist() for a, b in zip(cuts, cuts[1:])]


@pytest.mark.parametrize("kind,n_max,budget", [("phrases", 2, 40), ("phrases", 4, 30), ("phrases", 8, 9), ("one phrase", 5, 20), ("few", 3, 20), ("few", 7, 6),
                                               ("flat", 4, 6), ("new ids", 3, 12)])
def test_sieve(kind, n_max, budget):
    import paper_2602_24174_amd as T
    from test_gpu_tok_enrich import _run_and_compare
    merges = _run_and_compare(T, _docs(kind, np.random.default_rng(n_max)), 900, n_max, budget, device=True)
    assert len(merges) == budget
