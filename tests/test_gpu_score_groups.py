"""GPU indexer scoring of trees of more than eight nodes (groups of eight
nodes, one or all groups a workgroup) at the edges of the groups and of the
256-entry chunks: against the oracle, and both splits of the groups against
each other bit for bit."""
import numpy as np
import pytest
import torch

import synth
from oracle import tv_oracle as O

from .test_gpu_parity import _check_stages

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("over", [{}, dict(idx_fmt=1), dict(page_size=256)], ids=["bf16", "fp8", "paged"])
@pytest.mark.parametrize("D", [9, 16, 17, 31, 40, 64])
def test_score_groups(D, over):
    from paper_2609_24698_amd import DeviceRound

    lens = [1, 1023, 1027, 2052, 4 * 769 + 3]  # 0, 255, 256, 513 and 769 committed entries
    w = synth.make_workload("C0", seed=700 + D, B=len(lens), D=D, lens=lens, tree="random", topk=48, **over)
    nodes = [(b, i) for b in range(w.B) for i in sorted({0, 7, 8, D // 2, D - 1})]
    ref = O.run_round(w, nodes)

    def rerun(b, i, chosen):
        return O.verify_node(w, b, i, ref["anc"], ref["depth"], ref["scr_c4"], ref["scr_c128"], chosen=chosen)

    print("D", D, over, flush=True)
    _check_stages(w, ref, DeviceRound(w, "cuda:0"), nodes, rerun=rerun)


@pytest.mark.parametrize("D", [12, 32])
def test_group_splits_agree(D):
    """With a larger max_len the grid has 1,024 chunks or more, so that one
    workgroup takes all groups of its chunk."""
    from paper_2609_24698_amd import DeviceRound

    got = []
    for max_len in (0, 1 << 19):
        w = synth.make_workload("C0", seed=720 + D, B=2, D=D, lens=[3001, 7777], tree="random", topk=100)
        if max_len:
            w.dims["max_len"] = max_len
        r = DeviceRound(w, "cuda:0")
        r.mask(), r.compress(), r.verify()
        torch.cuda.synchronize()
        got.append({k: r.host(k).copy() for k in ("sel", "row_status")})
    assert np.array_equal(got[0]["row_status"], got[1]["row_status"])
    assert np.array_equal(got[0]["sel"], got[1]["sel"])
