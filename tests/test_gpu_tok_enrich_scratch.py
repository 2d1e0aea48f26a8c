"""Where an enrichment that counts in full has its records: in a block of their own, in one that an earlier call left and that holds everything, in one
that only holds the corpus; and nothing kept at all."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def test_records_in_kept_and_other_blocks():
    import paper_2602_24174_amd as T
    from test_gpu_tok_enrich import _run_and_compare
    rng = np.random.default_rng(8)
    flat = [rng.integers(0, 900, 300).tolist() for _ in range(30)]
    longer = [rng.integers(0, 900, 300).tolist() for _ in range(60)]
    table = T.tasc_ngram_build(np.arange(100, dtype=np.int32), np.array([0, 100]), 100, 2, 1)       # (scratch is kept while there is one)
    try:
        for docs in (flat, flat, longer, flat, longer):
            _run_and_compare(T, docs, 900, 4, 3, device=True)
        T.tasc_config_set(T.TASC_CFG_KEEP_SCRATCH_KIB, 0)
        _run_and_compare(T, flat, 900, 4, 3, device=True)
        T.tasc_config_set(T.TASC_CFG_KEEP_SCRATCH_KIB, 512)          # the corpus' block fits, the records' does not
        for _ in range(2):
            _run_and_compare(T, flat, 900, 4, 3, device=True)
    finally:
        T.tasc_config_set(T.TASC_CFG_KEEP_SCRATCH_KIB, 2 << 20)
        table.close()
    _run_and_compare(T, longer, 900, 4, 3)
