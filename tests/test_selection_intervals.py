"""The top-k of a step's candidates cuts the range of their scores into intervals: score sets that crowd into one interval, at several
levels, and what is left of it at the edges of a wave, against the oracle."""
import numpy as np
import pytest
import torch

from gpu_util import dev, host


def _scores(kind, n, rng):
    s = np.abs(rng.standard_normal(n)).astype(np.float32) + np.float32(0.5)
    if kind == "outlier":  # one score far away: all others in one of the first intervals
        s[rng.integers(n)] = np.float32(3e38)
    elif kind == "zero":  # the keys' range ends at zero
        s[rng.integers(n)] = 0.0
    elif kind == "levels":  # neighbours in the last bits, beside a wide range
        s[: n // 2] = (np.float32(1.0).view(np.uint32) + rng.integers(0, 200, n // 2).astype(np.uint32)).view(np.float32)
        s[n - 1] = np.float32(1e-30)
    elif kind == "few":  # a handful of values, hundreds of equal keys each
        s = rng.choice(np.array([0.25, 0.5, 0.5000001, 7.0], np.float32), n)
    elif kind == "inf":
        s[rng.integers(0, n, max(n // 8, 1))] = np.inf
    elif kind == "adjacent":  # keys in a range below 1024
        s = (np.float32(2.0).view(np.uint32) + rng.integers(0, 900, n).astype(np.uint32)).view(np.float32)
    return s


@pytest.fixture(scope="module")
def modules():
    from oracle import pop_oracle
    from paper_2602_06822_amd import binding
    return binding, pop_oracle


@pytest.mark.gpu
@pytest.mark.parametrize("kind", ["plain", "outlier", "zero", "levels", "few", "inf", "adjacent"])
@pytest.mark.parametrize("n", [1, 2, 63, 64, 65, 130, 1000, 4095, 4096, 4097, 16000])
def test_topk_of_crowded_scores(modules, kind, n):
    pop, oracle = modules
    rng = np.random.default_rng(n * 7 + len(kind))
    m = n + 37
    cand = np.sort(rng.choice(m, n, replace=False)).astype(np.int32)
    region = np.full(m, 2, np.uint8)
    region[cand] = 1
    cs = _scores(kind, n, rng)
    for k in sorted({0, 1, n // 3, n // 2, n - 1, n}):
        mask = torch.full((m,), 9, dtype=torch.uint8, device="cuda")
        sel = torch.full((max(k, 1),), -1, dtype=torch.int32, device="cuda")
        pop.pop_topk_from_scores(dev(cs), dev(cand), n, k, dev(region), m, mask, sel)
        mask0, sel0, _ = oracle.select(region, cs, cand, k)
        assert np.array_equal(host(mask), mask0), (n, k)
        assert np.array_equal(host(sel)[:k], sel0), (n, k)
