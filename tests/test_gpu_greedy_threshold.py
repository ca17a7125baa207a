"""Where the candidate greedy decides every step itself and where it gives up (the profile counts one index build and
greedy then, and a second one over all nodes otherwise): equal counts, small counts whose threshold falls between nodes of
one count, counts that differ little, hubs that come first or last by id.  Seeds and gains equal the oracle's."""
import sys

import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def eng():
    import paper_1404_0900_amd as tim
    e = tim.Engine(0)
    yield e
    e.close()


def _check(eng, n, off, nodes, k, runs, tag):
    import torch
    print(f"{tag}: n={n} sets={len(off) - 1} entries={len(nodes)} k={k}", file=sys.stderr, flush=True)
    off, nodes = np.asarray(off, dtype=np.int64), np.asarray(nodes, dtype=np.int32)
    eng.profile(True)
    seeds, gains = eng.max_coverage(n, torch.from_numpy(off).cuda(), torch.from_numpy(nodes).cuda(), k)
    calls = eng.read_profile().index_calls
    eng.profile(False)
    ws, wg = oracle.greedy(n, off, nodes, k)
    assert np.array_equal(seeds, ws) and np.array_equal(gains, wg)
    if runs:
        assert calls == runs


def _of_size(x):
    return np.arange(len(x) + 1, dtype=np.int64) * x.shape[1], x.ravel()


@pytest.mark.parametrize("k", [2, 8, 9, 50, 256])
@pytest.mark.parametrize("n", [2048, 2049, 2304, 2305, 9000, 65536, 65537, 300001])
def test_equal_counts(eng, n, k):
    b = np.arange(n)
    _check(eng, n, *_of_size(np.stack([b, (b + 1) % n], 1)), k, 1, "ring")
    _check(eng, n, *_of_size(b[:, None]), k, 1, "one each")


@pytest.mark.parametrize("mean", [1, 3, 31, 32, 33, 40])
def test_threshold_among_small_counts(eng, mean):
    """Counts of mean to mean + 3, most of them mean: the threshold lies between nodes of one count (below 32 of them)."""
    n = 30000
    r = np.random.default_rng(mean)
    cnt = mean + r.choice(4, size=n, p=[0.9, 0.08, 0.015, 0.005])
    nodes = r.permutation(np.repeat(np.arange(n), cnt))
    off = np.concatenate([np.arange(0, len(nodes), 3), [len(nodes)]])
    sets = np.repeat(np.arange(len(off) - 1), np.diff(off))
    keep = np.unique(sets.astype(np.int64) * n + nodes)
    off = np.concatenate([[0], np.cumsum(np.bincount(keep // n, minlength=len(off) - 1))])
    for k in (5, 30, 100):
        _check(eng, n, off, keep % n, k, 1, "small counts")


def test_counts_that_differ_little(eng):
    """Counts of 16000 +- 126, well inside one sixteenth of their power of two."""
    n = 4000
    r = np.random.default_rng(1)
    x = (r.integers(0, n, 2_000_000)[:, None] * 7 + np.arange(32)[None] * r.integers(1, n // 32, 2_000_000)[:, None]) % n
    for k in (4, 8):
        _check(eng, n, *_of_size(x), k, 1, "alike")


@pytest.mark.parametrize("first", [True, False])
@pytest.mark.parametrize("n", [700, 8000, 100000])
def test_hubs_in_order_of_their_ids(eng, n, first):
    r = np.random.default_rng(n)
    ln = 1 + r.poisson(3, size=20000)
    u = np.minimum((r.pareto(0.8, int(ln.sum())) * 5).astype(np.int64), n - 1)
    sid = np.repeat(np.arange(20000, dtype=np.int64), ln)
    key = np.unique(sid * n + (u if first else n - 1 - u))
    off = np.concatenate([[0], np.cumsum(np.bincount(key // n, minlength=20000))])
    for k in (3, 20, 200):
        _check(eng, n, off, key % n, k, 0, "hubs in order")


def test_steps_that_the_candidates_do_not_decide(eng):
    """One node covers every set of the 9000 next ones, so that the second step needs a node below all of those."""
    n = 20000
    r = np.random.default_rng(3)
    sets = [np.concatenate([[0], r.choice(np.arange(1, 9001), size=1500, replace=False)]) for _ in range(300)]
    sets += [[10000 + int(x)] for x in r.integers(0, 10000, size=400)]
    off = np.concatenate([[0], np.cumsum([len(s) for s in sets])])
    for k in (2, 25):
        _check(eng, n, off, np.concatenate(sets), k, 2, "overlap")
