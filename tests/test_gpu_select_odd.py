"""The target argmax over vocabularies that are no multiple of eight (nodes'
logits start off the 16-byte boundaries): the maximum at a node's edges and
around its chunks' ends, larger logits and NaNs of the neighbouring nodes just
outside, ties, rows of -inf, against numpy."""
import numpy as np
import pytest
import torch

import synth
from oracle import tv_oracle as O

pytestmark = pytest.mark.gpu

BIG, NAN, NEG_INF = 0x7F00, 0x7FC0, 0xFF80


@pytest.mark.parametrize("vocab", [1, 2, 5, 7, 9, 15, 1001, 8185, 8187, 8191, 8193, 8199, 16381, 24577, 129283])
def test_odd_vocab(vocab):
    from paper_2609_24698_amd import DeviceRound

    B, D = (3, 7) if vocab < 20000 else (2, 5)
    w = synth.make_workload("C0", seed=900, B=B, D=D, lens=[200 + b for b in range(B)], tree="random", topk=16)
    sel = synth.make_selection(w, vocab=vocab)
    rng = np.random.default_rng(vocab)
    bits = np.asarray(rng.integers(0x3C00, 0x4000, size=(B * D, vocab)), dtype=np.uint16)
    edges = {0, 1, 7, 8185, 8191, 8192, 8199, 16376, 16384, vocab - 8, vocab - 2, vocab - 1}
    spots = sorted(e for e in edges if 0 <= e < vocab)
    for n in range(B * D):
        if n % 5 == 4:
            bits[n] = NEG_INF  # no logit above the masks
        else:
            bits[n, spots[n % len(spots)]] = 0x4100 + (n % 2)
            bits[n, spots[(n + 3) % len(spots)]] = 0x4100  # a tie, or the runner-up
        if n % 7 == 3:  # large at both ends: the neighbours must not take it
            bits[n, 0], bits[n, -1] = BIG, BIG
        if n % 11 == 6:
            bits[n, -1] = NAN
    f = (bits.astype(np.uint32) << 16).view(np.float32)
    want = np.where(np.isnan(f).any(1), np.isnan(f).argmax(1), f.argmax(1)).astype(np.int32)
    r = DeviceRound(w, "cuda:0")
    sel.target_logits = bits.reshape(B, D, vocab)
    r.attach_selection(sel)
    r.mask()
    r.select()
    torch.cuda.synchronize()
    print("vocab", vocab, flush=True)
    assert np.array_equal(r.host("target_tokens").reshape(-1), want)
    tgt, acc, _ = O.select_accepted_path(w.parents, sel.draft_tokens, sel.target_logits, r.host("row_status"))
    assert np.array_equal(r.host("target_tokens"), tgt) and np.array_equal(r.host("accepted_last"), acc)
