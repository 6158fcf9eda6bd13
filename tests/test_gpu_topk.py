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


@pytest.mark.parametrize("topk", [33, 2047])
def test_merge_across_zero(topk):
    """Segmented nodes whose scores straddle zero, many of them exactly zero:
    the survivors' distances span most of the 32 bits (the merge's wide first
    digit) and the threshold is a tie."""
    from paper_2609_24698_amd import DeviceRound

    w = synth.make_workload("C0", seed=340 + topk, B=2, D=3, lens=[4 * 33800 + 1, 4 * 17000], tree="random", topk=topk)
    w.w_idx[:, :, 1:] |= 0x8000  # head 0 alone can raise a score
    w.w_idx[:, :, 0] &= 0x7FFF
    nodes = [(b, i) for b in range(w.B) for i in range(w.D)]
    ref = O.run_round(w, nodes)

    def rerun(b, i, chosen):
        return O.verify_node(w, b, i, ref["anc"], ref["depth"], ref["scr_c4"], ref["scr_c128"], chosen=chosen)

    print("topk", topk, flush=True)
    _check_stages(w, ref, DeviceRound(w, "cuda:0"), nodes, rerun=rerun)
