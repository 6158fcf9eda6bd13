"""The one-call layer step on a paged pool (its compression shares the mask's
and the top-k's launches) against the separate calls: rows that lack the page
of an open CSA block, of an open HCA block, of a page that only the new tokens
need, rows with bad parents or lengths, on the first and on a later layer,
with bfloat16 and FP8 keys and a designated chain."""
import numpy as np
import pytest
import torch

import synth
from oracle import tv_oracle as O

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("with_mask", [True, False], ids=["first", "later"])
@pytest.mark.parametrize("fp8", [0, 1])
@pytest.mark.parametrize("chain", [False, True])
def test_paged_step_equals_calls(with_mask, fp8, chain):
    from paper_2609_24698_amd import DeviceRound

    # 0: whole; 1: lacks the page its open CSA block began in; 2: the same, for an HCA block only;
    # 3: lacks a page that only new tokens need; 4: bad parents; 5: bad length; 6: whole, closes an HCA block
    lens = [2041, 1010, 1020, 2048, 900, 700, 383]
    w = synth.make_workload("C1", seed=61, B=len(lens), D=6, chain=True, lens=lens, topk=64, idx_fmt=fp8,
                            page_size=256, max_len_margin=64)
    w.parents[4, 2] = 5
    rounds = [DeviceRound(w, "cuda:0") for _ in range(2)]
    for r in rounds:
        if chain:
            r.t["primary_last"] = torch.full((w.B,), w.D - 1, dtype=torch.int32, device="cuda:0")
        for row in (1, 2, 3):
            r.t["page_table"][row, lens[row] // 256] = -1
        r.t["len"][5] = -3
    a, b = rounds
    print("with_mask", with_mask, "fp8", fp8, "chain", chain, flush=True)
    a.mask(), a.compress(), a.verify()
    if not with_mask:
        b.mask()
    b.verify_round(with_mask=with_mask)
    torch.cuda.synchronize()
    st = a.host("row_status")
    assert list(st) == [O.ROW_OK, O.ROW_CAPACITY, O.ROW_CAPACITY, O.ROW_OK, O.ROW_BAD_PARENT, O.ROW_BAD_LEN, O.ROW_OK]
    assert np.array_equal(st, b.host("row_status"))
    ok = np.flatnonzero(st == O.ROW_OK)
    for k in ("out", "lse", "sel", "scr_c4", "scr_c128"):
        assert np.array_equal(a.host(k)[ok].view(np.uint8), b.host(k)[ok].view(np.uint8)), k
    for k in ("anc", "depth"):
        assert np.array_equal(a.host(k), b.host(k)), k
    if not chain:
        return
    for k in ("c4", "c4_idx"):  # the whole rows' designated chains, in the pool
        x, y = a.host(k), b.host(k)
        P = 256 // 4
        for row in ok:
            for pg in a.host("page_table")[row]:
                if pg >= 0:
                    assert np.array_equal(x[pg * P:(pg + 1) * P].view(np.uint8), y[pg * P:(pg + 1) * P].view(np.uint8))
