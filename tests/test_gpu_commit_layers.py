"""The commits of a captured round with every way its layers share out a
workgroup's wavefronts (1 to 32 layers a launch), against the commits issued
one by one: full rows, rows that fail in the first, a middle and the last
layer, and FP8 and paged pools."""
import pytest
import torch

from .test_gpu_graph import _layers, _same

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 2, 5, 8, 16, 17, 32])
@pytest.mark.parametrize("over", [{}, dict(idx_fmt=1), dict(page_size=256)], ids=["flat", "fp8", "paged"])
def test_commit_layers(n, over):
    from paper_2609_24698_amd import LayeredRound

    lens = [2043, 1021, 3071, 126, 380]
    if "page_size" in over:
        lens[:3] = [2048, 1024, 3072]  # the round opens a page
    sides = []
    for _ in range(2):
        ws, rounds = _layers("C0", n, False, B=5, D=7, chain=True, lens=lens, topk=16, **over)
        for k, row in ((0, 0), (n // 2, 1), (n - 1, 2)):  # the row closes an entry this layer has no place for
            t = rounds[k].t
            if "page_size" in over:
                t["page_table"][row, int(ws[0].lens[row]) // 256] = -1
            else:
                t["c4_cap"][row] = int(ws[0].lens[row]) // 4
        rounds[n - 1].t["len"][3] = -5  # a length out of range
        rounds[0].t["accepted_last"].fill_(6)
        rounds[0].t["accepted_last"][4] = 2
        sides.append(LayeredRound(rounds))
    print("layers", n, over, flush=True)
    eager, graph = sides
    graph.capture()
    for rnd in range(2):
        eager.eager(fused=False)
        graph.replay()
        torch.cuda.synchronize()
        _same(eager, graph, rnd)
    graph.release()
