"""The largest vocabulary a table can be built for: 31 bits a token."""
import ctypes as C

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def test_tables():
    import torch
    import paper_2602_24174_amd as T
    from paper_2602_24174_amd import binding as B
    vocab = 0x7FFFFFFF
    torch.cuda.empty_cache()
    if torch.cuda.mem_get_info()[0] < 90 << 30:
        pytest.skip("eight token histograms of 8 GiB")
    tok = np.array([vocab - 1, 0, vocab - 1, 0, 7, vocab - 1, 0, vocab - 2], dtype=np.int32)
    ng = T.tasc_ngram_build(tok, np.array([0, 5, 8]), vocab, 4, 2)
    for n, want in ((2, [([vocab - 1, 0], 3)]), (3, []), (4, [])):
        rows, counts = T.tasc_ngram_export(ng, n)
        assert [(r.tolist(), int(c)) for r, c in zip(rows, counts)] == want
    fallback = C.c_int32(-1)
    B._check(B.lib().tasc_ngram_unigram(ng.handle, C.byref(fallback), None))
    assert fallback.value == 0                                     # three times, as vocab - 1 is: the smaller id
    with pytest.raises(T.TascError):
        tok[3] = vocab
        T.tasc_ngram_build(tok, np.array([0, 5, 8]), vocab, 4, 2)
    ng.close()
