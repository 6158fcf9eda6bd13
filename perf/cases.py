"""Performance cases of the tree-verify library, through its public entry points.

A case is one call pattern of a serving program on one GPU: the verify step of
one layer (mask, compression, attention in one call or as separate calls), the
greedy path selection, a whole round with its commit, or a captured
multi-layer round.  Sizes follow the workloads of the benchmark and the tests:
draft trees of 1 to 32 nodes, contexts from a few hundred tokens to 1M, batches
of 1 to 64 rows, both head shapes, bfloat16 and FP8 indexer keys, flat and
paged pools.

``listed`` names the fixed cases, ``draw`` gives another one of the same
ranges, ``prepare`` makes the device state of a case from a seed, ``run`` is
one pass, ``work`` the bytes and operations a pass needs, ``tolerance`` how far
two correct implementations may differ, and ``exact`` the result in float64.
"""
from __future__ import annotations

import math
from types import SimpleNamespace

import numpy as np
import torch

import paper_2609_24698_amd as tv

RATIO4, RATIO128, WINDOW, RING, D_IDX, H_IDX = 4, 128, 128, 256, 64, 8
SHAPES = {
    "mla": dict(H=64, d_row=576, d_k=576, v_off=0, d_v=512),
    "mha128": dict(H=8, d_row=256, d_k=128, v_off=128, d_v=128),
}
SPARE4, SPARE128 = 32, 4  # pool slots of a row past its committed entries


def _case(name, path, B, D, lo, hi, *, shape="mla", topk=512, tree="random", fp8=False, page=0, layers=1, vocab=0):
    """path: "step" (one-call layer step), "calls" (mask, compress, verify as
    separate calls), "select", "round" (step, selection, commit) or "graph"
    (captured round over ``layers`` layers).  Committed lengths are spread
    log-uniformly over [lo, hi]; page > 0 lays the cache out in pages."""
    c = dict(path=path, shape=shape, B=B, D=D, lo=lo, hi=hi, topk=topk, tree=tree, fp8=fp8, page=page,
             layers=layers, vocab=vocab)
    if name:
        c["name"] = name
    return c


def listed():
    return [
        _case("step_8head_b1_2k", "step", 1, 5, 2048, 2048, shape="mha128", topk=64),
        _case("step_b1_8k", "step", 1, 8, 8192, 8192),
        _case("step_b8_8k", "step", 8, 6, 8192, 8192),
        _case("step_b32_32k", "step", 32, 8, 32768, 32768),
        _case("step_b64_ragged", "step", 64, 8, 1024, 65536),
        _case("step_b1_1m", "step", 1, 8, 1 << 20, 1 << 20, topk=2048),
        _case("step_b12_fp8_paged", "step", 12, 7, 700, 14000, fp8=True, page=256),
        _case("calls_8head_b37_chain", "calls", 37, 6, 300, 9000, shape="mha128", topk=200, tree="chain"),
        _case("calls_b6_d32", "calls", 6, 32, 3000, 24000),
        _case("select_b64", "select", 64, 8, 1024, 65536, vocab=129280),
        _case("round_b4_4k", "round", 4, 8, 2000, 6000, vocab=129280),
        _case("graph_b16_6layers", "graph", 16, 8, 1024, 16384, layers=6),
    ]


def draw(rng):
    """One more case: sizes log-uniform over the ranges, none costlier than
    the largest listed ones (at most 512 nodes, 2^20 committed tokens)."""
    def log_int(a, b):
        return max(a, min(b, int(round(math.exp(rng.uniform(math.log(a), math.log(b)))))))

    path = rng.choice(["step"] * 5 + ["calls"] * 3 + ["select", "round", "graph"])
    B = log_int(1, 64)
    D = rng.randint(1, 8) if path != "calls" or rng.random() < 0.5 else rng.randint(9, 32)
    B = max(1, min(B, 512 // D))
    shape = "mha128" if rng.random() < 0.25 else "mla"
    page = rng.choice([128, 256, 512]) if rng.random() < 0.25 else 0
    layers = rng.randint(2, 8) if path == "graph" else 1
    budget = (1 << 17 if page else 1 << 20) // layers
    hi = log_int(300, max(301, min(1 << 20, budget // B)))
    lo = hi if rng.random() < 0.3 else log_int(64, hi)
    segments = -(-(hi // RATIO4) // 16896)
    topk = log_int(32, min(2048, 34816 // segments))
    vocab = log_int(3000, 160000) if path in ("select", "round") else 0
    return _case("", path, B, D, lo, hi, shape=shape, topk=topk, tree=rng.choice(["random", "random", "chain"]),
                 fp8=rng.random() < 0.3, page=page, layers=layers, vocab=vocab)


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------
def _device():
    return torch.device("cuda:0" if torch.cuda.is_available() else "cpu")


def _lens(case, rng):
    B, lo, hi = case["B"], case["lo"], case["hi"]
    at = (rng.permutation(B) + 0.5) / B
    room = np.floor(np.exp(math.log(lo) + at * (math.log(hi) - math.log(lo))) + 1e-6).astype(np.int64)
    return np.maximum(room - rng.integers(0, 128, size=B), 1), room  # any place in the open blocks


def _dims(case):
    d = dict(B=case["B"], D=case["D"], topk=case["topk"], d_idx=D_IDX, H_idx=H_IDX, ratio_csa=RATIO4,
             ratio_hca=RATIO128, window=WINDOW, ring_cap=RING, idx_fmt=int(case["fp8"]), page_size=case["page"],
             page_stride=0, max_len=case["hi"], **SHAPES[case["shape"]])
    d["scale"] = 1.0 / math.sqrt(d["d_k"])
    if case["page"]:
        d["page_stride"] = -(-(case["hi"] + 64) // case["page"])
    return d


def _bits(gen, shape, std=1.0):
    """N(0, std) bfloat16 values as host bit patterns."""
    x = torch.randn(shape, generator=gen, device=gen.device, dtype=torch.float32)
    return (x * std if std != 1.0 else x).to(torch.bfloat16).view(torch.int16).cpu().numpy().view(np.uint16)


def _keys(gen, rows, fp8):
    if not fp8:
        return _bits(gen, (rows, D_IDX))
    x = torch.randn((rows, D_IDX), generator=gen, device=gen.device, dtype=torch.float32)
    return x.to(torch.bfloat16).float().to(torch.float8_e4m3fn).view(torch.uint8).cpu().numpy()


def _trees(case, rng):
    B, D = case["B"], case["D"]
    par = np.full((B, D), -1, dtype=np.int32)
    for i in range(1, D):
        par[:, i] = i - 1 if case["tree"] == "chain" else rng.integers(0, i, size=B)
    return par


def _depths(par):
    dep = np.zeros_like(par)
    for i in range(1, par.shape[1]):
        dep[:, i] = dep[np.arange(par.shape[0]), par[:, i]] + 1
    return dep


def _path(par_row, node):
    p = [int(node)]
    while par_row[p[-1]] >= 0:
        p.append(int(par_row[p[-1]]))
    return p[::-1]


def _layer(case, dims, gen, rng, lens, room, parents, accepted):
    """The host arrays of one layer (what DeviceRound takes); a row's pools
    hold ``room`` committed tokens and some spare entries."""
    B, D = dims["B"], dims["D"]
    d_u = dims["d_row"] + D_IDX
    P = case["page"]
    w = SimpleNamespace(dims=dims, lens=lens.astype(np.int32), parents=parents, accepted_last=accepted)
    w.c4_cap = (room // RATIO4 + SPARE4).astype(np.int32)
    w.c128_cap = (room // RATIO128 + SPARE128).astype(np.int32)
    if P:
        owned = -(-(room + D + 1) // P)
        table = np.full((B, dims["page_stride"]), -1, dtype=np.int32)
        ids = rng.permutation(int(owned.sum())).astype(np.int32)
        at = np.concatenate([[0], np.cumsum(owned)])
        for b in range(B):
            table[b, :owned[b]] = ids[at[b]:at[b + 1]]
        w.page_table = table
        w.ring = _bits(gen, (len(ids), P, d_u))
        t4, t128 = len(ids) * (P // RATIO4), len(ids) * (P // RATIO128)
    else:
        w.ring = _bits(gen, (B, RING, d_u))
        t4, t128 = int(w.c4_cap.sum()), int(w.c128_cap.sum())
    w.c4_base = np.concatenate([[0], np.cumsum(w.c4_cap)[:-1]]).astype(np.int64)
    w.c128_base = np.concatenate([[0], np.cumsum(w.c128_cap)[:-1]]).astype(np.int64)
    w.c4 = _bits(gen, (t4, dims["d_row"]))
    w.c4_idx = _keys(gen, t4, case["fp8"])
    w.c128 = _bits(gen, (t128, dims["d_row"]))
    w.tree_u = _bits(gen, (B, D, d_u))
    w.q = _bits(gen, (B, D, dims["H"], dims["d_k"]))
    w.q_idx = _bits(gen, (B, D, H_IDX, D_IDX))
    w.w_idx = _bits(gen, (B, D, H_IDX))
    w.gate_w = _bits(gen, (2, d_u), 0.02)
    return w


def _selection(case, gen, rng, parents, accepted):
    """Draft tokens and target logits that accept the root path of ``accepted``."""
    B, D, V = case["B"], case["D"], case["vocab"]
    draft = np.stack([rng.permutation(V)[:D] for _ in range(B)]).astype(np.int32)  # distinct within a row
    x = torch.randn((B, D, V), generator=gen, device=gen.device, dtype=torch.float32).to(torch.bfloat16)
    bs, ns, ts = [], [], []
    for b in range(B):
        p = _path(parents[b], accepted[b])
        for a, n in zip(p, p[1:]):
            bs.append(b), ns.append(a), ts.append(int(draft[b, n]))
    if bs:
        x[torch.tensor(bs), torch.tensor(ns), torch.tensor(ts)] = 16.0
    return SimpleNamespace(vocab=V, draft_tokens=draft, target_logits=x.view(torch.int16).cpu().numpy().view(np.uint16))


def _inputs(case, seed):
    rng = np.random.Generator(np.random.PCG64(seed))
    gen = torch.Generator(device=_device())
    gen.manual_seed(int(seed))
    dims = _dims(case)
    (lens, room), parents = _lens(case, rng), _trees(case, rng)
    accepted = rng.integers(0, case["D"], size=case["B"]).astype(np.int32)
    sel = _selection(case, gen, rng, parents, accepted) if case["vocab"] else None
    layers = [] if case["path"] == "select" else [_layer(case, dims, gen, rng, lens, room, parents, accepted)
                                                   for _ in range(case["layers"])]
    return SimpleNamespace(dims=dims, lens=lens, parents=parents, accepted=accepted, sel=sel, layers=layers)


def prepare(case, seed):
    x = _inputs(case, seed)
    if case["path"] == "select":  # the selection alone: trees, masks, draft tokens, logits
        dev = _device()
        B, D, V = case["B"], case["D"], case["vocab"]
        dims = tv.make_dims(x.dims)
        i32 = dict(dtype=torch.int32, device=dev)
        s = SimpleNamespace(path="select", dims=dims, vocab=V, parents=torch.from_numpy(x.parents).to(dev),
                            anc=torch.zeros((B, D), dtype=torch.int64, device=dev), depth=torch.zeros((B, D), **i32),
                            status=torch.zeros(B, **i32), draft=torch.from_numpy(x.sel.draft_tokens).to(dev),
                            logits=torch.from_numpy(x.sel.target_logits.view(np.int16)).to(dev),
                            target=torch.zeros((B, D), **i32), accepted=torch.zeros(B, **i32),
                            next=torch.zeros(B, **i32),
                            ws=torch.empty(tv.tv_select_workspace_bytes(dims, V), dtype=torch.uint8, device=dev))
        tv.tv_build_tree_mask(dims, s.parents, s.anc, s.depth, s.status)
        return s
    rounds = [tv.DeviceRound(w, poison_outputs=False) for w in x.layers]
    r = rounds[0]
    if x.sel is not None:
        r.attach_selection(x.sel)
    s = SimpleNamespace(path=case["path"], rounds=rounds, r=r, layered=None)
    if case["path"] in ("round", "graph"):
        # The layers' lengths side by side, so that one copy takes a round's commits back.
        stride = (case["B"] + 3) // 4 * 4
        s.lens = torch.zeros((len(rounds), stride), dtype=torch.int32, device=r.t["len"].device)
        for k, q in enumerate(rounds):
            s.lens[k, :case["B"]] = q.t["len"]
            q.t["len"] = s.lens[k, :case["B"]]
            t = q.t
            q.cache = tv.make_cache(t["ring"], t["c4"], t["c4_idx"], t["c128"], t["c4_base"], t["c4_cap"],
                                    t["c128_base"], t["c128_cap"], t["len"], t["page_table"])
        s.start = s.lens.clone()
    if case["path"] == "graph":
        s.layered = tv.LayeredRound(rounds)
        s.layered.capture()
    return s


def _bf(t):
    return t.view(torch.bfloat16)


def _verify_outputs(t):
    return dict(out=_bf(t["out"]), lse=t["lse"], sel=t["sel"], scr_c4=_bf(t["scr_c4"]), scr_c128=_bf(t["scr_c128"]))


def _commit_outputs(t):
    return dict(len=t["len"], ring=_bf(t["ring"]), c4=_bf(t["c4"]),
                c4_idx=_bf(t["c4_idx"]) if t["c4_idx"].dtype == torch.int16 else t["c4_idx"], c128=_bf(t["c128"]),
                accept_nodes=t["accept_nodes"], accept_len=t["accept_len"])


def run(s):
    if s.path == "select":
        tv.tv_select_accepted_path(s.dims, s.parents, s.anc, s.depth, s.draft, s.logits, s.vocab, s.target,
                                   s.accepted, s.next, s.status, s.ws)
        return dict(target=s.target, accepted=s.accepted, next=s.next)
    r = s.r
    if s.path == "step":
        r.verify_round()
        return _verify_outputs(r.t)
    if s.path == "calls":
        r.mask()
        r.compress()
        r.verify()
        return _verify_outputs(r.t)
    s.lens.copy_(s.start)  # the same round again: the last commit is taken back
    if s.path == "round":
        r.round()
        return dict(_verify_outputs(r.t), **_commit_outputs(r.t), accepted=r.t["accepted_last"],
                    next=r.t["next_token"], target=r.t["target_tokens"])
    s.layered.replay()
    shared = r.t
    return [dict(out=_bf(q.t["out"]), lse=q.t["lse"], sel=q.t["sel"], scr_c4=_bf(q.t["scr_c4"]), len=q.t["len"],
                 c4=_bf(q.t["c4"]), **({} if k else dict(accept_len=shared["accept_len"])))
            for k, q in enumerate(s.rounds)]


# ---------------------------------------------------------------------------
# work and tolerances
# ---------------------------------------------------------------------------
def work(case):
    """Bytes read once and written once, and operations, of one pass."""
    B, D, V = case["B"], case["D"], case["vocab"]
    n_bytes, flops = 0.0, 0.0
    if V:
        n_bytes += B * D * V * 2.0 + B * (D * 28.0 + 8)
    if case["path"] == "select":
        return dict(bytes=n_bytes, flops=float(B * D * V))
    d = _dims(case)
    H, row, d_u = d["H"], d["d_row"] * 2.0, (d["d_row"] + D_IDX) * 2.0
    step_b = step_f = 0.0
    at = (np.arange(B) + 0.5) / B
    for L in np.exp(math.log(case["lo"]) + at * (math.log(case["hi"]) - math.log(case["lo"]))):
        L = max(1.0, L - 63.5)
        n4, n128 = L // RATIO4, L // RATIO128
        k = min(float(case["topk"]), n4)
        union = n4 * (1.0 - (1.0 - k / n4) ** D) if n4 else 0.0  # CSA rows at least one node selects
        keys = k + n128 + min(L + 1, WINDOW)
        step_b += n4 * D_IDX * (1 if case["fp8"] else 2)                       # indexer keys
        step_b += (union + n128 + min(L, WINDOW)) * row + D * d_u              # attended rows, tree rows
        step_b += D * (H * (d["d_k"] + d["d_v"]) * 2.0 + H * 4 + case["topk"] * 4 + H_IDX * (D_IDX + 1) * 2 + 16)
        closed = D / RATIO4                                                    # CSA blocks the tree closes
        step_b += closed * (RATIO4 + 1) * d_u
        step_f += 2.0 * D * H_IDX * D_IDX * n4 + 2.0 * D * H * (d["d_k"] + d["d_v"]) * keys
        if case["path"] in ("round", "graph"):
            step_b += 2.0 * (D / 4 + 1) * d_u * 1.25
    return dict(bytes=float(n_bytes + case["layers"] * step_b), flops=float(flops + case["layers"] * step_f))


def tolerance(case):
    """bfloat16 outputs of float32 sums: half a unit in the last place of the
    result (2^-9) and of the probabilities; "differ" covers near ties of the
    indexer scores, which move entries of an ascending selection list."""
    if case["path"] == "select":
        return "exact"
    return dict(rel=1e-2, max=0.25, differ=0.01)


# ---------------------------------------------------------------------------
# the result in float64
# ---------------------------------------------------------------------------
def _f64(bits, dev):
    return torch.from_numpy(np.ascontiguousarray(bits).view(np.int16)).to(dev).view(torch.bfloat16).double()


def _codes64(codes, dev):
    return torch.from_numpy(codes).to(dev).view(torch.float8_e4m3fn).double()


def _store(x):
    return x.to(torch.bfloat16).double()  # a value the cache stores


def _exact_layer(case, w, parents, lens):
    dev = _device()
    d = w.dims
    B, D, P, k = d["B"], d["D"], case["page"], d["topk"]
    d_row, d_v, v_off = d["d_row"], d["d_v"], d["v_off"]
    dep = _depths(parents)
    out = torch.zeros((B, D, d["H"], d_v), dtype=torch.float64, device=dev)
    lse = torch.zeros((B, D, d["H"]), dtype=torch.float64, device=dev)
    scr4 = torch.zeros((B, D, d_row + D_IDX), dtype=torch.float64, device=dev)
    scr128 = torch.zeros((B, D, d_row), dtype=torch.float64, device=dev)
    gate = _f64(w.gate_w, dev)
    for b in range(B):
        L = int(lens[b])
        n4, n128 = L // RATIO4, L // RATIO128
        q_lo = max(0, L - RATIO128)
        pos = np.arange(q_lo, L)
        s4, s128 = np.arange(n4), np.arange(n128)
        if P:
            t = w.page_table[b].astype(np.int64)
            raw = w.ring.reshape(-1, d_row + D_IDX)[t[pos // P] * P + pos % P]
            s4 = t[s4 // (P // RATIO4)] * (P // RATIO4) + s4 % (P // RATIO4)
            s128 = t[s128 // (P // RATIO128)] * (P // RATIO128) + s128 % (P // RATIO128)
        else:
            raw = w.ring[b][pos % RING]
            s4, s128 = s4 + int(w.c4_base[b]), s128 + int(w.c128_base[b])
        raw = _f64(raw, dev)
        tree = _f64(w.tree_u[b], dev)
        keys = _codes64(w.c4_idx[s4], dev) if case["fp8"] else _f64(w.c4_idx[s4], dev)
        rows4 = torch.from_numpy(np.ascontiguousarray(w.c4[s4]).view(np.int16)).to(dev).view(torch.bfloat16)
        rows128 = _f64(w.c128[s128], dev)
        qi, wi = _f64(w.q_idx[b], dev), _f64(w.w_idx[b], dev)
        q = _f64(w.q[b], dev)
        entries = {}
        for i in range(D):
            p = L + int(dep[b, i])
            seq = torch.cat([raw, tree[_path(parents[b], i)]])  # positions q_lo .. p
            for ri, r in enumerate((RATIO4, RATIO128)):
                if (p + 1) % r:
                    continue
                toks = seq[len(seq) - r:]
                e = torch.softmax(toks @ gate[ri], 0) @ toks
                if ri == 0:
                    e = _store(e) if not case["fp8"] else torch.cat(
                        [_store(e[:d_row]), e[d_row:].float().clamp(-448, 448).to(torch.float8_e4m3fn).double()])
                    scr4[b, i] = e
                else:
                    e = _store(e[:d_row])
                    scr128[b, i] = e
                entries[(i, ri)] = e
        for i in range(D):
            p = L + int(dep[b, i])
            nodes = _path(parents[b], i)
            on4 = [entries[(j, 0)] for j in nodes if (j, 0) in entries]
            on128 = [entries[(j, 1)] for j in nodes if (j, 1) in entries]
            kk = torch.cat([keys] + [e[None, d_row:] for e in on4])
            cand = torch.cat([rows4.double() if len(kk) <= k else rows4[:0].double()] + [e[None, :d_row] for e in on4])
            if len(kk) > k:
                score = torch.relu(kk @ qi[i].T) @ wi[i]
                top = torch.sort(torch.sort(score, descending=True, stable=True).indices[:k]).values
                mine = top[top < n4]
                cand = torch.cat([rows4[mine].double()] + [on4[int(s) - n4][None, :d_row] for s in top[top >= n4]])
            lo = max(0, p - WINDOW + 1)
            window = torch.cat([raw[max(0, lo - q_lo):, :d_row], tree[nodes][max(0, lo - L):, :d_row]])
            R = torch.cat([cand, rows128] + [e[None] for e in on128] + [window])
            logits = (q[i] @ R[:, :d["d_k"]].T) * float(np.float32(d["scale"]))
            lse[b, i] = torch.logsumexp(logits, 1)
            out[b, i] = torch.softmax(logits, 1) @ R[:, v_off:v_off + d_v]
    return out, lse, scr4, scr128


def exact(case, seed):
    """Float64 results of the computed outputs (None for whole numbers and for
    state that is copied)."""
    if case["path"] == "select":
        return None
    x = _inputs(case, seed)
    if case["path"] == "graph":
        got = []
        for k, w in enumerate(x.layers):
            out, lse, scr4, _ = _exact_layer(case, w, x.parents, x.lens)
            got.append(dict(out=out, lse=lse, sel=None, scr_c4=scr4, len=None, c4=None,
                            **({} if k else dict(accept_len=None))))
        return got
    out, lse, scr4, scr128 = _exact_layer(case, x.layers[0], x.parents, x.lens)
    res = dict(out=out, lse=lse, sel=None, scr_c4=scr4, scr_c128=scr128)
    if case["path"] == "round":
        res.update(len=None, ring=None, c4=None, c4_idx=None, c128=None, accept_nodes=None, accept_len=None,
                   accepted=None, next=None, target=None)
    return res
