"""A CPU model of the device top-k's threshold search, checked against a sort.

Keys are complements of order-preserving score bits: the best candidates have
the smallest keys, padding is all ones.  Up to three digits are counted (11,
11 and 10 bits; 13, 11 and 8 for many keys), each pass over the keys sharing
the digits found so far, until the bin of the k-th key holds exactly the keys
still needed; padding is counted like any key.  The merge of a segmented node
first bounds the keys (no segment's k best exceed its own threshold bin) and
takes the digits of the distance to the best key, the wide first digit where
the distances have more than 26 bits.  Both must give exactly the k smallest
keys, ties to the lower index.
"""
import numpy as np
import pytest

PAD = 0xFFFFFFFF


def _threshold(keys, k, widths, bits=32):
    keys = keys.astype(np.int64)
    prefix, pmask, rem, left, all_eq = 0, 0, k, bits, False
    for w in widths:
        nb = min(w, left)
        sft = left - nb
        m = (keys & pmask) == prefix
        h = np.bincount((keys[m] >> sft) & ((1 << nb) - 1), minlength=1 << nb)
        run = np.cumsum(h)
        dig = int(np.argmax(run >= rem))
        prefix |= dig << sft
        pmask |= ((1 << nb) - 1) << sft
        rem -= int(run[dig] - h[dig])
        left = sft
        all_eq = int(h[dig]) == rem
        if all_eq or left == 0:
            break
    return prefix, pmask, rem, all_eq


def _taken(keys, t, pad=PAD):
    prefix, pmask, rem, all_eq = t
    km = keys.astype(np.int64) & pmask
    if all_eq:
        return np.nonzero(km <= prefix)[0]
    eq = np.nonzero((km == prefix) & (keys != pad))[0][:rem]
    return np.sort(np.concatenate([np.nonzero(km < prefix)[0], eq]))


def _by_sort(keys, k):
    return np.sort(np.argsort(keys, kind="stable")[:k])


def _draw(kind, n, rng):
    if kind == "uniform":
        return rng.integers(0, PAD, size=n)
    if kind == "last_bin":  # every key shares its leading digits with the padding
        return PAD - rng.integers(1, 200, size=n)
    if kind == "ties":
        return rng.integers(5, 40, size=n)
    if kind == "scores":  # the keys of ordinary scores
        u = rng.normal(0, 16, size=n).astype(np.float32).view(np.uint32).astype(np.int64)
        return np.where(u >> 31, u, u ^ 0x7FFFFFFF)
    return np.full(n, int(rng.integers(0, PAD)))


KINDS = ["uniform", "last_bin", "ties", "scores", "all_equal"]


@pytest.mark.parametrize("widths", [(11, 11, 10), (13, 11, 8)], ids=["narrow", "wide"])
@pytest.mark.parametrize("kind", KINDS)
def test_threshold_equals_sort(kind, widths):
    rng = np.random.default_rng(KINDS.index(kind) + 3)
    for _ in range(80):
        n = int(rng.integers(2, 3000))
        k = int(rng.integers(1, n))
        keys = np.full(n + int(rng.integers(0, 600)), PAD)
        keys[:n] = _draw(kind, n, rng)
        assert np.array_equal(_taken(keys, _threshold(keys, k, widths)), _by_sort(keys, k))


def _merge_draw(kind, n, rng):
    if kind.startswith("span"):  # distances of a given number of bits, the best key anywhere
        bits = int(kind[4:])
        lo = int(rng.integers(0, PAD - (1 << bits) + 1))
        return lo + rng.integers(0, (1 << bits) - 1, size=n)
    return _draw(kind, n, rng)


MERGE_KINDS = KINDS + ["span26", "span27", "span30", "span31"]


@pytest.mark.parametrize("kind", MERGE_KINDS)
def test_merge_equals_sort(kind):
    rng = np.random.default_rng(MERGE_KINDS.index(kind) + 23)
    seen = set()
    for _ in range(60):
        seg, nseg, k = int(rng.integers(40, 400)), int(rng.integers(2, 9)), int(rng.integers(1, 300))
        n = seg * (nseg - 1) + int(rng.integers(1, seg + 1))
        k = min(k, seg - 1)  # a full segment has more candidates than a node keeps
        keys = _merge_draw(kind, n, rng)
        slots, index, bound = [], [], PAD - 1
        for s in range(nseg):
            part = keys[s * seg:(s + 1) * seg]
            if len(part) <= k:
                got = np.arange(len(part))
            else:
                t = _threshold(part, k, (13, 11, 8))
                got = _taken(part, t)
                assert len(got) == k
                bound = min(bound, t[0] | (~t[1] & PAD))
            row = np.full(k, PAD)
            row[:len(got)] = part[got]
            slots.append(row)
            index.append(np.concatenate([got + s * seg, np.full(k - len(got), -1)]))
        slots, index = np.concatenate(slots), np.concatenate(index)
        best = int(slots.min())
        worst = max(min(bound, PAD - 1), best)
        bits = (worst - best + 1).bit_length()
        pad = (1 << bits) - 1
        dist = np.where(slots <= worst, slots - best, pad)
        assert dist[slots <= worst].max() < pad
        seen.add(bits)
        t = _threshold(dist, k, (13, 11, 8) if bits > 26 else (11, 11, 10), bits)
        assert np.array_equal(index[_taken(dist, t, pad)], _by_sort(keys, k))
    wide = {"uniform": True, "scores": True, "last_bin": False, "ties": False, "all_equal": False, "span26": False,
            "span27": True, "span30": True, "span31": True}[kind]
    assert any(b > 26 for b in seen) if wide else all(b <= 26 for b in seen), seen
