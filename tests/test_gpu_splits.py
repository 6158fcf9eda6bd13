"""GPU parity over the attention's split plans: one to 32 splits a node, on
few rows (splits dealt over the XCDs, padded to a multiple of 8) and on 8 rows
or more (whole rows on an XCD), rows that use all of their splits, some or
one, against the oracle."""
import numpy as np
import pytest
import torch

import synth
from oracle import tv_oracle as O

from .test_gpu_parity import _check_stages

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("name", ["C0", "C1"])
@pytest.mark.parametrize("B,D,lens,topk,max_len", [
    (1, 8, [8191], 512, 8200),
    (1, 3, [700], 512, 8200),
    (2, 4, [9003, 127], 1024, 100000),
    (4, 8, [2001, 5999, 1, 640], 512, 6100),
    (3, 6, [4099, 255, 1500], 64, 300000),
    (8, 5, [4095, 90, 700, 2048, 3333, 1, 129, 512], 512, 8192),
    (9, 2, [4095, 90, 700, 2048, 3333, 1, 129, 512, 1023], 300, 8192),
])
def test_splits(name, B, D, lens, topk, max_len):
    from paper_2609_24698_amd import DeviceRound

    w = synth.make_workload(name, seed=800 + 10 * B + D, B=B, D=D, lens=lens, tree="random", topk=topk)
    w.dims["max_len"] = max_len
    nodes = [(b, i) for b in range(B) for i in sorted({0, D // 2, D - 1})]
    ref = O.run_round(w, nodes)

    def rerun(b, i, chosen):
        return O.verify_node(w, b, i, ref["anc"], ref["depth"], ref["scr_c4"], ref["scr_c128"], chosen=chosen)

    print(name, B, D, lens, topk, max_len, flush=True)
    _check_stages(w, ref, DeviceRound(w, "cuda:0"), nodes, rerun=rerun)


@pytest.mark.parametrize("name,D", [("C1", 4), ("C1", 40), ("C0", 4)], ids=["halves", "64 heads", "8 heads"])
def test_first_tile_maximum_has_probability_one(name, D):
    """One key of the first 32 outweighs the rest of the node by about e^6.  The
    reference of a split is its first tile's maximum, so that key's bfloat16
    probability is exactly 1 and lse keeps float32 precision: the other keys,
    0.3 % of the sum, add 2^-8 of that (1.2e-5) to the 1e-4 of the logits.  From
    a smaller reference the probability would be rounded, up to 3.9e-3 off."""
    from paper_2609_24698_amd import DeviceRound

    w = synth.make_workload(name, seed=840 + D, B=8, D=D, lens=803, tree="random", topk=300)  # keys 0..199: entries
    d = w.dims
    at = [3, 15, 16, 20, 31]
    for b in range(w.B):
        for i in range(D):
            for h in range(d["H"]):
                k = O.bf16_to_f64(w.c4[w.c4_base[b] + at[(h + i) % 5], :d["d_k"]])
                w.q[b, i, h] = O.f64_to_bf16(k * (12.0 / (d["scale"] * (k @ k))))
    nodes = [(b, i) for b in range(0, 8, 3) for i in (0, D - 1)]
    ref = O.run_round(w, nodes)
    r = DeviceRound(w, "cuda:0")
    r.mask(), r.compress(), r.verify()
    torch.cuda.synchronize()
    lse = r.host("lse").astype(np.float64)
    for b, i in nodes:
        assert np.abs(lse[b, i] - ref["detail"][(b, i)]["lse"]).max() <= 1.12e-4, (b, i)
