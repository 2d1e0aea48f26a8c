"""Enrichments of more blocks of positions than the device has compute units, than one launch's blocks tell each other their sums, and than those sums
are added up without a scan of their own; phrases, and corpora whose pairs are all alike, where the sieve gives up in some blocks while others have not
begun.  Against counts by sorting the packed windows, and replacement left to right."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _reference(tok, off, vocab, n_max, budget):
    """tok: int64 on the GPU; off: numpy.  Windows as big-endian integers, so equal rewards go to the smallest tuple by the smallest key."""
    import torch
    bits = (vocab + budget - 1).bit_length()
    assert bits * n_max < 63
    ends = torch.zeros(tok.numel(), dtype=torch.bool, device="cuda")      # the output's last token
    filled = off[1:][np.diff(off) > 0]
    ends[torch.from_numpy(filled - 1).cuda()] = True
    merges, lens = [], [tok.numel()]
    for m in range(budget):
        best = None
        for n in range(2, n_max + 1):
            W = tok.numel() - n + 1
            if W <= 0:
                continue
            key, inside = torch.zeros(W, dtype=torch.int64, device="cuda"), torch.ones(W, dtype=torch.bool, device="cuda")
            for j in range(n):
                key = (key << bits) | tok[j:j + W]
                if j < n - 1:
                    inside &= ~ends[j:j + W]
            keys, counts = torch.unique(key[inside], return_counts=True)
            if not counts.numel():
                continue
            f = int(counts.max())
            k = int(keys[counts == f].min())
            if best is None or f * (n - 1) > best[0]:
                best = (f * (n - 1), n, k, f, torch.nonzero((key == k) & inside).flatten())
        if best is None:
            break
        _, n, k, f, at = best
        gram = tuple((k >> (bits * (n - 1 - j))) & ((1 << bits) - 1) for j in range(n))
        if at.numel() > 1 and int((at[1:] - at[:-1]).min()) < n:          # occurrences overlap: the first, then the next one past its end
            taken, free = [], 0
            for p in at.tolist():
                if p >= free:
                    taken.append(p)
                    free = p + n
            at = torch.tensor(taken, device="cuda")
        keep = torch.ones(tok.numel(), dtype=torch.bool, device="cuda")
        for j in range(1, n):
            keep[at + j] = False
        ends = ends.clone()
        ends[at] = ends[at + n - 1]
        tok = tok.clone()
        tok[at] = vocab + m
        tok, ends = tok[keep], ends[keep]
        merges.append((gram, f, vocab + m))
        lens.append(tok.numel())
    out = torch.nonzero(ends).flatten().cpu().numpy() + 1
    off_out = np.zeros_like(off)
    off_out[1:][np.diff(off) > 0] = out
    return merges, tok, np.maximum.accumulate(off_out), lens


@pytest.mark.parametrize("kind,length,n_max,budget", [("phrases", 2_500_000, 3, 6), ("flat", 2_500_000, 3, 3), ("few", 1_300_000, 2, 3), ("phrases", 5_000_000, 2, 3),
                                                      ("flat", 5_000_000, 2, 2), ("phrases", 18_000_001, 2, 2), ("flat", 18_000_001, 2, 2)])
def test_large_corpora(kind, length, n_max, budget):
    import torch
    import paper_2602_24174_amd as T
    rng = np.random.default_rng(length % 1000 + n_max)
    vocab = {"phrases": 30_000, "flat": 20_000, "few": 60}[kind]
    if kind == "phrases":
        phrases = rng.integers(0, vocab, (3000, 6))
        cut = rng.integers(2, 7, 3000)
        pick = np.minimum(rng.zipf(1.2, length // 2) - 1, 2999)
        tok = phrases[pick][np.arange(6) < cut[pick][:, None]][:length]
        hit = rng.random(tok.size) < 0.1
        tok[hit] = rng.integers(0, vocab, int(hit.sum()))
    else:
        tok = rng.integers(0, vocab, length)
    off = np.unique(np.r_[0, np.cumsum(rng.integers(1, 300, tok.size // 100)), tok.size])
    off = off[off <= tok.size].astype(np.int64)
    print(f"{kind} {tok.size} tokens, n_max {n_max}", flush=True)
    src = torch.from_numpy(tok.astype(np.int32)).cuda()
    merges, out, out_off, lens = T.tasc_tok_enrich(src, off, vocab, n_max, budget)
    want_m, want, want_off, want_l = _reference(src.long(), off, vocab, n_max, budget)
    assert merges == want_m
    assert lens.tolist() == want_l and (out_off == want_off).all() and torch.equal(out, want.int())
