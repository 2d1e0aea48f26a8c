"""Merges that have to be taken back: of an n-gram that was counted wrong, and ones whose workgroups did not hear from each other."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

ONE, OTHER = (5, 9, 5), (411932615, 873892672, 411932615)


def _hash(gram):
    h0, h1 = len(gram), 0x1234567
    for v in gram:
        h0 = (h0 ^ v) * 0x9E3779B1 & 0xFFFFFFFF
        h0 ^= h0 >> 15
        h1 = (h1 + v) * 0x85EBCA77 & 0xFFFFFFFF
        h1 ^= h1 >> 13
    return h0, h1 & ~15


@pytest.mark.parametrize("budget", [1, 6])
@pytest.mark.parametrize("apart", [0, 4096])         # (the n-grams in one block of positions, and in several)
def test_two_ngrams_of_one_hash(budget, apart):
    """Two n-grams of one hash, each less frequent than a third, together more.  All three overlap themselves, so the wrong merge has marked
    its occurrences before its windows are found to be fewer than counted."""
    import paper_2602_24174_amd as T
    from test_gpu_tok_enrich import _run_and_compare
    assert _hash(ONE) == _hash(OTHER)                # (the hash of the kernel that counts windows)
    rng = np.random.default_rng(3)
    between = [rng.integers(1000, 1000 + 50 * apart, apart).tolist()] if apart else []

    def runs(g, times):
        return [[g[0], g[1], g[0], g[1], g[0]]] * times
    docs = runs(ONE, 50) + between + runs(OTHER, 45) + between + runs((6, 7, 6), 60)
    merges = _run_and_compare(T, docs, 900_000_000, 3, budget, device=True)
    assert merges[0][:2] == ((6, 7, 6), 120)


@pytest.mark.parametrize("kind,n_max,budget", [("phrases", 4, 30), ("few", 3, 12), ("flat", 4, 6), ("new ids", 3, 5), ("phrases", 2, 1)])
def test_workgroups_that_do_not_hear_from_each_other(kind, n_max, budget):
    """Every wait given up at once: the merge is made again without one, in the sieve's merges and in those that are counted in full."""
    import paper_2602_24174_amd as T
    from test_gpu_tok_enrich import _run_and_compare
    from test_gpu_tok_enrich_sieve import _docs
    try:
        T.tasc_config_set(T.TASC_CFG_ENRICH_WAIT, 0)
        for device in (False, True):
            _run_and_compare(T, _docs(kind, np.random.default_rng(n_max)), 900, n_max, budget, device=device)
    finally:
        T.tasc_config_set(T.TASC_CFG_ENRICH_WAIT, 1 << 20)
