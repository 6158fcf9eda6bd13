"""GPU parity over the attention's split plans: one to 32 splits a node, on
few rows (splits dealt over the XCDs, padded to a multiple of 8) and on 8 rows
or more (whole rows on an XCD), rows that use all of their splits, some or
one, against the oracle."""
import pytest

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
