"""The attention's split plan through the workspace size: whatever fits the
no-alloc entry's array with the fewest splits fits it with the plan's own."""
import random

from paper_2609_24698_amd import binding

MAX_CHUNK, SEG = 1280, 512 * 33


def _least_total(d):
    """Workspace bytes with the fewest splits the pointer table allows."""
    nodes = d["B"] * d["D"]
    mk = d["topk"] + d["max_len"] // d["ratio_hca"] + d["D"] + d["window"]
    least = -(-mk // MAX_CHUNK)
    chunk = (-(-mk // least) + 31) // 32 * 32
    splits = -(-mk // chunk)
    stride = (d["max_len"] // d["ratio_csa"] + 63) // 64 * 64
    seg = max(1, -(-(d["max_len"] // d["ratio_csa"]) // SEG))
    parts = [4 * nodes * max(stride, 1), 4 * nodes * d["topk"]]
    if splits > 1:
        parts += [4 * nodes * splits * d["H"] * d["d_v"], 8 * nodes * splits * d["H"]]
    parts += [4 * d["B"]] * 2 + [8 * nodes * mk] + [4 * nodes] * 2
    if seg > 1:
        parts += [4 * nodes * seg * d["topk"]] * 2 + [8 * nodes * seg]
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
