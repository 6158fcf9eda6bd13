"""The CPU model of the device top-k's threshold search (test_topk_model) on
keys that float32 scores cannot be made to have.

The kernels select the k best keys with digits of 13, 11 and 8 or of 11, 11 and
10 bits, padding counted like any key (its key is the worst one); an ordered
compaction then takes the keys better than the threshold and the lowest-index
keys equal to it.  The GPU parity tests cannot put the threshold among the worst
keys, beside the padding: only -inf and NaN scores have such keys, and float32
scoring and the float64 oracle do not produce them alike.  The model covers it
(keys concentrated in the last bin, ties, padding between real keys) and must
give exactly the k best keys, ties to the lower index.  Keys here grow with the
score and 0 is padding; the model takes their complements.
"""
import numpy as np
import pytest

from .test_topk_model import PAD, _taken, _threshold


def _by_sort(keys, n, k):
    real = [e for e in range(n) if keys[e] != 0]
    return np.array(sorted(sorted(real, key=lambda e: (-int(keys[e]), e))[:k]))


@pytest.mark.parametrize("widths", [(11, 11, 10), (13, 11, 8)], ids=["narrow", "wide"])
@pytest.mark.parametrize("kind", ["uniform", "bin0", "tiny_ties", "mixed", "all_equal"])
def test_radix_select_model_equals_sort(kind, widths):
    rng = np.random.default_rng(["uniform", "bin0", "tiny_ties", "mixed", "all_equal"].index(kind) + 11)
    cases = 0
    for trial in range(160):
        nt = int(rng.choice([64, 128, 512]))
        kpt = int(rng.integers(1, 5))
        k = int(rng.choice([1, 3, 16, 50, 200]))
        n = int(rng.integers(1, nt * kpt + 1))
        if kind == "uniform":
            v = rng.integers(1, 2**32, size=n)
        elif kind == "bin0":  # every key below 2**19: the threshold lies in the padding's bin of the first pass
            v = rng.integers(1, 1 << 19, size=n)
        elif kind == "tiny_ties":
            v = rng.integers(1, 40, size=n)
        elif kind == "mixed":
            v = np.where(rng.random(n) < 0.5, rng.integers(1, 5, size=n), rng.integers(1, 2**32, size=n))
        else:
            v = np.ones(n, dtype=np.int64)
        keys = np.zeros(nt * kpt, dtype=np.uint32)
        keys[:n] = v.astype(np.uint32)
        if trial % 2:  # merge-like: padding slots between the real keys
            keys[:n][rng.random(n) < 0.3] = 0
        n_real = int((keys[:n] != 0).sum())
        if n_real <= k:
            continue
        cases += 1
        inv = PAD - keys[:-(-n // nt) * nt].astype(np.int64)  # whole slots of nt threads
        assert np.array_equal(_taken(inv, _threshold(inv, k, widths)), _by_sort(keys, n, k)), (kind, trial)
    assert cases > 50
