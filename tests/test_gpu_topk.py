"""GPU top-k at the edges of its dispatch: candidate counts around a slot, the
few-slot and sixteen-slot bodies and a whole segment, a last segment of one
entry, survivors fewer than topk in one segment, odd topk and topk 1, against
the oracle."""
import numpy as np
import pytest
import torch

import synth
from oracle import tv_oracle as O

from .test_gpu_parity import _check_stages

pytestmark = pytest.mark.gpu

N4 = {  # committed CSA entries of each row
    "few": [0, 1, 40, 511, 512, 513, 2047, 2048, 2049],
    "many": [2560, 8191, 8192, 8193, 16895, 16896],
    "segments": [16897, 33792, 33793, 40],
}


@pytest.mark.parametrize("topk", [1, 33, 512, 2047])
@pytest.mark.parametrize("kind", list(N4))
def test_topk_edges(kind, topk):
    from paper_2609_24698_amd import DeviceRound

    # lengths 3 and 0 short of a block's end: the root closes one or opens one
    lens = [max(4 * n + 3 * (k % 2), 1) for k, n in enumerate(N4[kind])]
    D = 10 if kind == "few" else 4
    w = synth.make_workload("C0", seed=310 + topk, B=len(lens), D=D, lens=lens, tree="random", topk=topk)
    print("topk", topk, "n4", N4[kind], flush=True)
    nodes = [(b, i) for b in range(w.B) for i in range(w.D)]
    ref = O.run_round(w, nodes)

    def rerun(b, i, chosen):
        return O.verify_node(w, b, i, ref["anc"], ref["depth"], ref["scr_c4"], ref["scr_c128"], chosen=chosen)

    r = DeviceRound(w, "cuda:0")
    _check_stages(w, ref, r, nodes, rerun=rerun)
    # the same selection from the one-call step
    sel = r.host("sel").copy()
    r2 = DeviceRound(w, "cuda:0")
    r2.verify_round()
    torch.cuda.synchronize()
    s2 = r2.host("sel")
    assert np.mean(sel != s2) < 0.01  # its own scratch: near ties only


SEG = 512 * 33


def _committed_scores(w, b, i):
    """Node i's scores of the committed entries of row b, in float64."""
    n = w.lens[b] // w.dims["ratio_csa"]
    k = O.bf16_to_f64(w.c4_idx[w.c4_base[b]:w.c4_base[b] + n])
    q, wgt = O.bf16_to_f64(w.q_idx[b, i]), O.bf16_to_f64(w.w_idx[b, i])
    return (wgt[:, None] * np.maximum(q @ k.T, 0)).sum(0)


def _span_bits(scores, topk):
    """At least this many bits has the merge's largest distance: from the best
    key to the topk-th of the full segment that ends best."""
    u = (scores.astype(np.float32) + np.float32(0)).view(np.uint32).astype(np.int64)
    keys = np.where(u >> 31, u, u ^ 0x7FFFFFFF)
    ends = [np.partition(keys[s:s + SEG], topk - 1)[topk - 1] for s in range(0, len(keys), SEG)
            if len(keys[s:s + SEG]) > topk]
    return int(min(ends) - keys.min() + 1).bit_length()


@pytest.mark.parametrize("topk", [33, 2047])
def test_merge_across_zero(topk):
    """Segmented nodes whose scores straddle zero: with a topk past the positive
    ones the survivors' distances span more than 26 bits (the merge's wide first
    digit), with a small one those of some nodes do."""
    from paper_2609_24698_amd import DeviceRound

    w = synth.make_workload("C0", seed=340 + topk, B=2, D=3, lens=[4 * 33800 + 1, 4 * 17000], tree="random", topk=topk)
    w.w_idx[:, :, 1:] |= 0x8000  # head 0 alone can raise a score
    w.w_idx[:, :, 0] &= 0x7FFF
    nodes = [(b, i) for b in range(w.B) for i in range(w.D)]
    wide = [_span_bits(_committed_scores(w, b, i), topk) > 26 for b, i in nodes]
    assert all(wide) if topk == 2047 else any(wide) and not all(wide)
    ref = O.run_round(w, nodes)

    def rerun(b, i, chosen):
        return O.verify_node(w, b, i, ref["anc"], ref["depth"], ref["scr_c4"], ref["scr_c128"], chosen=chosen)

    print("topk", topk, flush=True)
    _check_stages(w, ref, DeviceRound(w, "cuda:0"), nodes, rerun=rerun)


@pytest.mark.parametrize("topk", [33, 2047])
def test_merge_of_equal_keys(topk):
    """Half of the scores are zero and none is above: every survivor has the same
    key, and the node keeps the first topk of them."""
    from paper_2609_24698_amd import DeviceRound

    w = synth.make_workload("C0", seed=360 + topk, B=2, D=3, lens=[4 * 33800, 4 * 17000], tree="random", topk=topk)
    w.w_idx[:, :, 1:] = 0
    w.w_idx[:, :, 0] |= 0x8000
    print("topk", topk, flush=True)
    r = DeviceRound(w, "cuda:0")
    r.mask(), r.compress(), r.verify()
    torch.cuda.synchronize()
    sel = r.host("sel")
    for b in range(w.B):
        for i in range(w.D):
            zeros = np.nonzero(_committed_scores(w, b, i) == 0)[0]
            assert len(zeros) > SEG // 3 and np.array_equal(sel[b, i], zeros[:topk]), (b, i)
