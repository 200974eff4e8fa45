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


def _crowded(kind, n, rng):
    s = np.abs(rng.standard_normal(n)).astype(np.float32) + np.float32(0.5)
    if kind == "dead":  # nine tenths of the channels score zero
        s[rng.permutation(n)[: 9 * n // 10]] = 0.0
    elif kind == "dead_first":  # zeros where a wave looks first, or only where it does not
        s[: n // 2] = 0.0
    elif kind == "dead_last":
        s[n // 2:] = 0.0
    elif kind == "two_crowds":  # neighbours in the last bits at both ends of all numbers
        s = np.where(rng.random(n) < 0.5, np.float32(3.4e38), np.float32(-3.4e38)).astype(np.float32)
        s = (s.view(np.uint32) - rng.integers(0, 3, n).astype(np.uint32)).view(np.float32)
    elif kind == "crowd_within":  # a third of the keys in one interval, spread over some 40 values in the middle of it
        s[: n // 3] = (np.float32(1.25).view(np.uint32) + rng.integers(0, 40, n // 3).astype(np.uint32)).view(np.float32)
        s[n - 1] = 0.0
    return s


@pytest.mark.gpu
@pytest.mark.parametrize("kind", ["dead", "dead_first", "dead_last", "two_crowds", "crowd_within"])
@pytest.mark.parametrize("n", [65, 513, 2048, 2049, 2113, 4096])
def test_topk_of_equal_scores(modules, kind, n):
    pop, oracle = modules
    rng = np.random.default_rng(n * 5 + len(kind))
    m = n + 41
    cand = np.sort(rng.choice(m, n, replace=False)).astype(np.int32)
    region = np.full(m, 2, np.uint8)
    region[cand] = 1
    cs = _crowded(kind, n, rng)
    for k in sorted({1, n // 20, n // 10, n // 10 + 1, n // 3, n // 2, n // 2 + 1, 9 * n // 10, n - 1}):
        mask = torch.full((m,), 9, dtype=torch.uint8, device="cuda")
        sel = torch.full((k,), -1, dtype=torch.int32, device="cuda")
        pop.pop_topk_from_scores(dev(cs), dev(cand), n, k, dev(region), m, mask, sel)
        mask0, sel0, _ = oracle.select(region, cs, cand, k)
        assert np.array_equal(host(mask), mask0), (n, k)
        assert np.array_equal(host(sel), sel0), (n, k)


@pytest.mark.gpu
def test_dead_channels_take_no_longer(modules):
    """4096 candidates, nine tenths of them zero, half selected: no longer than spread scores (counted one lane at a time they took 2.2 times
    as long as those, counted by the wave .9 times)."""
    pop, _ = modules
    n = 4096
    cand, region = torch.arange(n, dtype=torch.int32, device="cuda"), torch.ones(n, dtype=torch.uint8, device="cuda")
    mask = torch.empty(n, dtype=torch.uint8, device="cuda")
    sel = torch.empty(n // 2, dtype=torch.int32, device="cuda")
    spread = torch.rand(n, device="cuda")
    dead = torch.where(torch.rand(n, device="cuda") < 0.9, torch.zeros_like(spread), spread)

    def best(scores):
        times = []
        for _ in range(7):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            for _ in range(200):
                pop.pop_topk_from_scores(scores, cand, n, n // 2, region, n, mask, sel)
            b.record()
            torch.cuda.synchronize()
            times.append(a.elapsed_time(b))
        return min(times)

    best(spread)
    assert best(dead) < 1.5 * best(spread)
