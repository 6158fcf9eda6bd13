"""The attention's split plan through the workspace size: whatever fits the
no-alloc entry's array with the fewest splits fits it with the plan's own, and
the plan is the cheapest of all split counts, found for every size."""
import json
import os
import random
import subprocess
import sys

import numpy as np

from paper_2609_24698_amd import binding

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

MAX_CHUNK, SEG = 1280, 512 * 33


def _max_keys(d):
    return d["topk"] + d["max_len"] // d["ratio_hca"] + d["D"] + d["window"]


def _least_total(d):
    """Workspace bytes with the fewest splits the pointer table allows."""
    mk = _max_keys(d)
    least = -(-mk // MAX_CHUNK)
    chunk = (-(-mk // least) + 31) // 32 * 32
    return _total(d, -(-mk // chunk))


def _total(d, splits):
    nodes = d["B"] * d["D"]
    mk = _max_keys(d)
    stride = (d["max_len"] // d["ratio_csa"] + 63) // 64 * 64
    seg = max(1, -(-(d["max_len"] // d["ratio_csa"]) // SEG))
    parts = [4 * nodes * max(stride, 1), 4 * nodes * d["topk"]]
    if splits > 1:
        parts += [4 * nodes * splits * d["H"] * d["d_v"], 8 * nodes * splits * d["H"]]
    parts += [4 * d["B"]] * 2 + [8 * nodes * mk] + [4 * nodes] * 2
    if seg > 1:
        parts += [4 * nodes * seg * d["topk"]] * 2 + [4 * nodes * seg]
    return sum((p + 255) // 256 * 256 for p in parts)


def test_plan_keeps_the_noalloc_limit():
    rng = random.Random(5)
    limit = binding.NOALLOC_SCRATCH_BYTES
    near = exact = 0
    shapes = [dict(H=64, d_row=576, d_k=576, v_off=0, d_v=512), dict(H=8, d_row=256, d_k=128, v_off=128, d_v=128)]
    for _ in range(6000):
        D = rng.randint(1, 64)
        B = max(1, min(64, int(2 ** rng.uniform(0, 6)), 512 // D))
        max_len = int(2 ** rng.uniform(6, 21))
        d = dict(B=B, D=D, topk=rng.choice([16, 64, 512, 2048]), d_idx=64, H_idx=8, ratio_csa=4, ratio_hca=128,
                 window=128, ring_cap=256, idx_fmt=0, page_size=0, page_stride=0, max_len=max_len,
                 **rng.choice(shapes))
        d["scale"] = 0.1
        got = binding.tv_verify_workspace_bytes(binding.make_dims(d))
        if got == 0:  # more survivors than the merge holds: refused
            continue
        least = _least_total(d)
        exact += got == least
        if least <= limit:
            assert got <= limit, d
            near += got > limit // 2
        else:
            assert got > limit, d
    assert near > 100 and exact > 100


# The plan's costs: microseconds of a workgroup's prologue and epilogue and of
# a 32-key tile (all heads, half of them), of the combine, of one partial; and
# the workgroups an XCD holds.
COST = {64: ((8.0, 7.0), (0.8, 0.55), 5.0, 0.03, 32), 8: ((6.0, 6.0), (0.65, 0.65), 4.0, 0.002, 64)}


def _cheapest_splits(d):
    """The cheapest plan's splits, over every split count and both head splits."""
    f = np.float32
    fixed, tile, combine, partial, slots = COST[d["H"]]
    tiles = -(-_max_keys(d) // 32)
    least = -(-_max_keys(d) // MAX_CHUNK)
    nodes = d["B"] * d["D"]
    best = None
    for halves in (1, 2) if d["H"] == 64 else (1,):
        for s in range(least, tiles + 1):
            ct = -(-tiles // s)
            splits = -(-tiles // ct)
            padded = (splits + 7) // 8 * 8 if d["B"] < 8 and splits >= 8 else splits
            wgs = (d["B"] + 7) // 8 * d["D"] * halves * splits if d["B"] >= 8 else (nodes * halves * padded + 7) // 8
            if s > least and (_max_keys(d) < 512 or nodes >= 256):
                break  # too few keys, or enough workgroups without a split
            if wgs > slots and not (halves == 1 and s == least):
                break  # one round of workgroups, or the fewest splits in as many as they take
            c = f(-(-wgs // slots)) * (f(fixed[halves - 1]) + f(tile[halves - 1]) * f(ct))
            c += f(combine) + f(partial) * f(nodes * splits) if splits > 1 else f(0)
            if best is None or c < best[0]:
                best = (c, splits)
    return best[1]


def _sizes_of(dims):
    """The library's workspace sizes, from a process of its own: a search that
    does not end would stop this one for good."""
    child = ("import json, sys; from paper_2609_24698_amd import binding as b; "
             "print(json.dumps([b.tv_verify_workspace_bytes(b.make_dims(d)) for d in json.load(sys.stdin)]))")
    r = subprocess.run([sys.executable, "-c", child], input=json.dumps(dims), cwd=ROOT, text=True,
                       capture_output=True, timeout=120)
    assert r.returncode == 0, r.stderr
    return json.loads(r.stdout)


def _dims(H, B, D, topk, max_len, **over):
    shape = dict(d_row=576, d_k=576, v_off=0, d_v=512) if H == 64 else dict(d_row=256, d_k=128, v_off=128, d_v=128)
    return {**dict(H=H, B=B, D=D, topk=topk, max_len=max_len, d_idx=64, H_idx=8, ratio_csa=4, ratio_hca=128,
                   window=128, ring_cap=256, scale=0.1, idx_fmt=0, page_size=0, page_stride=0), **shape, **over}


def test_plan_is_the_cheapest():
    """Every tile count of the smallest batches, and random sizes."""
    rng = random.Random(11)
    dims = [_dims(H, B, D, 32 * t, 64) for H in (64, 8) for B, D in ((1, 1), (1, 8), (3, 5), (8, 3)) for t in range(1, 65)]
    for _ in range(3000):
        D = rng.randint(1, 64)
        dims.append(_dims(rng.choice((64, 8)), max(1, min(64, int(2 ** rng.uniform(0, 6)), 512 // D)), D,
                          rng.choice([16, 64, 300, 512, 2047, 2048]), int(2 ** rng.uniform(6, 21)),
                          ratio_hca=rng.choice([16, 128])))
    seen = set()
    for d, got in zip(dims, _sizes_of(dims)):
        splits = _cheapest_splits(d)
        want = _total(d, splits)
        if got == 0 or want > binding.NOALLOC_SCRATCH_BYTES:  # refused, or planned for that entry's limit
            continue
        assert got == want, (d, splits)
        seen.add(splits)
    assert len(seen) > 20


def test_noalloc_limit_to_the_byte():
    """Dims whose workspace ends within a few bytes per top-k segment of that
    entry's array: one word a segment beside its survivors is all that fits."""
    limit, rng, dims = binding.NOALLOC_SCRATCH_BYTES, random.Random(23), []
    while len(dims) < 12:
        B, D, topk = rng.randint(8, 40), rng.randint(1, 16), rng.choice([300, 512, 777, 2048])
        max_len = rng.randint(4 * (SEG + 1), 1 << 20)
        d = _dims(rng.choice((64, 8)), B, D, topk, max_len)
        seg = -(-(max_len // 4) // SEG)
        if seg * topk <= 34816 and limit - 4 * B * D * seg < _least_total(d) <= limit:
            dims.append(d)
    for d, got in zip(dims, _sizes_of(dims)):
        assert 0 < got <= limit, (d, got)


def test_no_split_where_short_rows_would_pay_for_it():
    """Up to 511 keys a node, or 256 nodes or more: one split, whatever the rest."""
    dims = [_dims(H, B, D, mk - D - 128 - 3, 399)  # 3 HCA entries
            for H in (8, 64) for B, D in ((1, 1), (4, 8), (30, 8), (255, 1)) for mk in (300, 459, 511)]
    dims += [_dims(8, B, D, 512, 8192) for B, D in ((16, 16), (32, 8), (64, 4), (128, 2), (64, 8))]
    for d, got in zip(dims, _sizes_of(dims)):
        assert got == _total(d, 1), d
    more = [_dims(8, 4, 8, 512 - 139, 399), _dims(8, 255, 1, 512, 8192), _dims(64, 4, 4, 512, 8192)]
    for d, got in zip(more, _sizes_of(more)):
        assert got > _total(d, 1), d
