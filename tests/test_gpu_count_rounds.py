"""Corpora whose partitions are counted in two rounds, or in several with the records laid out round by round, keys of up to 64 bits and more, for the
tables and for the enrichment: bit-exact against sorted keys.  Half of the tokens are of a few: their n-grams leave a record in nearly every
chunk, so that some partitions, and some rounds, hold more records than a workgroup has room for; of four tokens alone all do."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _corpus(length, vocab):
    import torch
    g = torch.Generator(device="cuda").manual_seed(length)
    tok = torch.randint(0, vocab, (length,), generator=g, device="cuda", dtype=torch.int32)
    few = torch.rand(length, generator=g, device="cuda") < 0.5
    tok = torch.where(few, tok % 24 * (vocab // 24), tok)
    off = np.arange(0, length + 240, 240, dtype=np.int64)
    off[-1] = length
    return tok, off


class Counts:
    """Every n-gram's key (ascending, as its tokens are) and count for n of 2, 3 and 4; a pair of tokens counts as its rank beyond 2."""

    def __init__(self, tok, off, vocab):
        import torch
        self.tok, self.vocab = tok.long(), vocab
        self.ends = torch.from_numpy(off[1:]).cuda()
        self.pairs, self.rank = torch.unique(self.tok[:-1] * vocab + self.tok[1:], return_inverse=True)

    def of(self, n):
        import torch
        t, r, size = self.tok, self.rank, self.pairs.numel()
        assert size * max(size, self.vocab) < 1 << 62
        key = r if n == 2 else r[:-1] * self.vocab + t[2:] if n == 3 else r[:-2] * size + r[2:]
        inside = torch.ones(key.numel(), dtype=torch.bool, device="cuda")
        for j in range(1, n):
            at = self.ends - j                             # an n-gram that begins here goes past the document
            inside[at[at < key.numel()]] = False
        return torch.unique(key[inside], return_counts=True)

    def key_of(self, rows):
        import torch
        rows = torch.from_numpy(rows.astype(np.int64)).cuda()
        first = torch.searchsorted(self.pairs, rows[:, 0] * self.vocab + rows[:, 1])
        if rows.shape[1] == 2:
            return first
        if rows.shape[1] == 3:
            return first * self.vocab + rows[:, 2]
        return first * self.pairs.numel() + torch.searchsorted(self.pairs, rows[:, 2] * self.vocab + rows[:, 3])

    def tokens_of(self, key, n):
        a = [int(key) if n == 2 else int(key) // (self.vocab if n == 3 else self.pairs.numel())]
        if n == 4:
            a.append(int(key) % self.pairs.numel())
        out = [t for r in a for t in divmod(int(self.pairs[r]), self.vocab)]
        return tuple(out + ([int(key) % self.vocab] if n == 3 else []))


@pytest.mark.parametrize("vocab,length,n_max,p_min", [(50_000, 140_000_000, 2, 40), (50_000, 250_000_000, 2, 60), (131_072, 290_000_000, 4, 3), (4, 200_000_000, 3, 1)])
def test_tables(vocab, length, n_max, p_min):
    import torch
    import paper_2602_24174_amd as T
    tok, off = _corpus(length, vocab)
    ng = T.tasc_ngram_build(tok, off, vocab, n_max, p_min)
    st = T.tasc_ngram_get_stats(ng)
    ref = Counts(tok, off, vocab)
    for n in range(2, n_max + 1):
        keys, counts = ref.of(n)
        keep = counts >= p_min
        rows, got = T.tasc_ngram_export(ng, n)
        print(f"{length} tokens, order {n}: {counts.numel()} distinct, {len(got)} kept, build {st.build_ms:.1f} ms", flush=True)
        assert st.distinct[n] == counts.numel() and len(got) == int(keep.sum())
        assert torch.equal(ref.key_of(rows), keys[keep]) and (counts[keep].cpu().numpy() == got).all()


@pytest.mark.parametrize("vocab,length", [(3000, 2_300_000), (90_000, 2_100_000), (100_000, 150_000_000)])
def test_enrichment(vocab, length):
    """From 2 M tokens on chunks are long and their offsets turned, of all orders at once (keys of 48 and of 68 bits); the longest corpus goes order
    by order, in rounds."""
    import torch
    import paper_2602_24174_amd as T
    tok, off = _corpus(length, vocab)
    docs = length // 240
    at = torch.from_numpy(240 * np.random.default_rng(1).permutation(docs)[:max(docs * 2 // 3, 60_000 if docs > 100_000 else 0)] + 100).cuda()
    for j, t in enumerate((1, vocab - 1, vocab // 2, 1)):     # one 4-gram often, and one of three in every output but the last
        tok[at + j] = t
    for j, t in enumerate((5, 6, vocab - 2)):
        tok[240 * torch.arange(docs, device="cuda") + 7 + j] = t
    merges, _, _, lens = T.tasc_tok_enrich(tok, off, vocab, 4, 2)
    text, bounds = tok, off
    for i in range(2):
        ref = Counts(text, bounds, vocab + 2)
        best = []
        for n in (2, 3, 4):
            keys, counts = ref.of(n)
            first = int(torch.nonzero(counts == counts.max())[0])      # (the smallest)
            best.append((-int(counts[first]) * (n - 1), n, ref.tokens_of(keys[first], n), int(counts[first])))
            del keys, counts
        _, n, gram, freq = min(best)
        print(f"{length} tokens, merge {i}: {gram} {freq} times", flush=True)
        assert merges[i][:2] == (gram, freq) and lens[i] == text.numel()
        del ref
        done, text, bounds, _ = T.tasc_tok_enrich(tok, off, vocab, 4, i + 1)
        assert done == merges[:i + 1]
    assert lens[2] == text.numel() == bounds[-1]
