"""GPU indexer scoring of trees of more than eight nodes (groups of eight
nodes, one or all groups a workgroup) at the edges of the groups and of the
256-entry chunks: against the oracle, and the scores of both splits of the
groups against each other bit for bit."""
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


def _scores(r):
    """The score area of the workspace, [B, D, stride] float32."""
    d = r.host_dims
    stride = max((d["max_len"] // d["ratio_csa"] + 63) // 64 * 64, 1)
    n = d["B"] * d["D"] * stride
    return r.t["workspace"][:4 * n].view(torch.float32).view(d["B"], d["D"], stride).cpu().numpy()


def _keys(w, b, n4):
    """The committed indexer keys of row b in float64."""
    s = np.arange(n4)
    if w.dims["page_size"]:
        per = w.dims["page_size"] // w.dims["ratio_csa"]
        at = w.page_table[b, s // per].astype(np.int64) * per + s % per
    else:
        at = w.c4_base[b] + s
    k = w.c4_idx[at]
    if w.dims["idx_fmt"]:
        return torch.from_numpy(k).view(torch.float8_e4m3fn).to(torch.float64).numpy()
    return O.bf16_to_f64(k)


@pytest.mark.parametrize("D,over", [(9, {}), (9, dict(idx_fmt=1)), (12, dict(idx_fmt=1, page_size=256)),
                                    (17, dict(page_size=256)), (32, {}), (64, dict(idx_fmt=1)),
                                    (64, dict(page_size=256))])
def test_group_splits_agree(D, over):
    """72 rows, a workgroup per group of a chunk, and the same rows eight times
    over, 1,024 chunks or more, a workgroup for all groups of a chunk: the same
    score bits, which are the float64 sums as far as float32 goes.  Rows of no
    entry and of a bad length lie between the others."""
    from paper_2609_24698_amd import DeviceRound

    n4 = [257, 512, 0, 300, 513, 511, 600, 769]
    lens = [max(4 * n4[b % 8] + b % 4, 1) for b in range(72)]
    w = synth.make_workload("C0", seed=720 + D, B=72, D=D, lens=lens, tree="random", topk=48, **over)
    bad = [7, 63, 64]
    w.lens[bad] = [-1, w.dims["max_len"] + 1, -5]
    got = []
    for times in (1, 8):
        if times > 1:
            per_row = ["lens", "parents", "accepted_last", "c4_base", "c4_cap", "c128_base", "c128_cap", "tree_u",
                       "q", "q_idx", "w_idx"] + (["page_table"] if w.dims["page_size"] else ["ring"])
            for k in per_row:
                x = getattr(w, k)
                setattr(w, k, np.tile(x, (times,) + (1,) * (x.ndim - 1)))
            w.dims["B"] = 72 * times
        print("D", D, over, "rows", w.dims["B"], flush=True)
        r = DeviceRound(w, "cuda:0")
        r.mask(), r.compress(), r.verify()
        torch.cuda.synchronize()
        status = r.host("row_status")
        assert [b for b in range(72 * times) if status[b]] == [72 * t + b for t in range(times) for b in bad]
        got.append((_scores(r), r.host("sel").copy()))
    small, many = got
    live = [b for b in range(72) if b not in bad]
    assert 8 * sum(-(-(lens[b] // 4) // 256) for b in live) >= 1024
    for b in live:
        n = lens[b] // 4
        for t in range(8):
            assert np.array_equal(many[0][72 * t + b, :, :n].view(np.uint32), small[0][b, :, :n].view(np.uint32)), (b, t)
            assert np.array_equal(many[1][72 * t + b], small[1][b]), (b, t)
        # 64 products and 8 weighted terms summed in float32: each addition is off by at most 2^-23 of the terms' sum
        k, q = _keys(w, b, n), O.bf16_to_f64(w.q_idx[b])
        wgt = O.bf16_to_f64(w.w_idx[b])[..., None]
        ref = (wgt * np.maximum(q @ k.T, 0)).sum(1)
        size = (np.abs(wgt) * (np.abs(q) @ np.abs(k).T)).sum(1)
        assert (np.abs(small[0][b, :, :n] - ref) <= 80 * 2.0 ** -23 * size).all(), b
