"""tim_max_coverage where the candidate greedy meets its edges: few and many nodes against its candidate limits, sets
that span windows and 128-byte lines of its stream, ties, collections its candidates cannot decide (the greedy over
all nodes takes over), and every count of steps around its limit.  Seeds and gains equal the oracle's."""
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


def _check(eng, n, sets, k, tag):
    import torch
    print(f"{tag}: n={n} sets={len(sets)} k={k}", file=sys.stderr, flush=True)
    off = np.zeros(len(sets) + 1, dtype=np.int64)
    off[1:] = np.cumsum([len(x) for x in sets])
    nodes = np.concatenate([np.asarray(x, dtype=np.int32) for x in sets]) if len(sets) else np.zeros(0, np.int32)
    seeds, gains = eng.max_coverage(n, torch.from_numpy(off).cuda(), torch.from_numpy(nodes).cuda(), k)
    ws, wg = oracle.greedy(n, off, nodes, k)
    assert np.array_equal(seeds, ws) and np.array_equal(gains, wg)


def _zipf_sets(r, n, count, mean, a=1.0):
    p = (np.arange(n) + 3.0) ** -a
    perm = r.permutation(n)
    ln = np.maximum(1, r.poisson(mean, size=count))
    flat = r.choice(n, size=int(ln.sum()), p=p / p.sum())
    out, at = [], 0
    for l in ln:
        out.append(perm[np.unique(flat[at:at + l])])
        at += l
    return out


@pytest.mark.parametrize("n,count,mean,k", [(2, 1, 1, 2), (64, 200, 3, 10), (2048, 5000, 4, 50), (2049, 5000, 4, 50),
                                            (8192, 20000, 5, 40), (8193, 20000, 5, 40), (70000, 60000, 8, 30),
                                            (300, 900, 90, 20), (70000, 300000, 2, 256), (70000, 30000, 8, 257)])
def test_heavy_tailed_collections(eng, n, count, mean, k):
    r = np.random.default_rng(n + count)
    _check(eng, n, _zipf_sets(r, n, count, mean), min(k, n), "zipf")


def test_sets_longer_than_windows(eng):
    """Sets of 1 to 30000 nodes side by side: entries of one set in many windows, lines and chunks."""
    r = np.random.default_rng(5)
    n = 40000
    sets = [r.choice(n, size=s, replace=False) for s in (1, 30000, 1, 1, 63, 64, 65, 5000, 2, 4096, 4097, 127, 129, 1, 9999)]
    sets += [r.choice(n, size=int(s), replace=False) for s in r.integers(1, 40, size=3000)]
    r.shuffle(sets)
    _check(eng, n, sets, 60, "long sets")
    _check(eng, 8000, [x % 8000 for x in [np.unique(y % 8000) for y in sets]], 60, "long sets, all nodes candidates")


@pytest.mark.parametrize("n", [5000, 50000])
def test_ties_and_exhausted_collections(eng, n):
    """Equal counts everywhere (one bin above the limit of candidates), disjoint sets, and more steps than coverable sets."""
    _check(eng, n, [[i] for i in range(n)], 20, "one node each")
    _check(eng, n, [[i, (i + 1) % n] for i in range(0, n, 2)], 20, "pairs")
    _check(eng, n, [[7, 3], [7, 9], [n - 1]], 10, "three sets")
    r = np.random.default_rng(n)
    _check(eng, n, [r.choice(n, size=3, replace=False) for _ in range(200)], 100, "uniform")
    _check(eng, n, [np.arange(n // 2)] * 3 + [[n - 1, n - 2]] * 5, 30, "one giant set")


def test_overlapping_hubs_fall_below_the_threshold(eng):
    """One node covers every set that holds the 9000 next ones, so the second step needs a node below all of those."""
    n = 20000
    r = np.random.default_rng(3)
    sets = [np.concatenate([[0], r.choice(np.arange(1, 9001), size=1500, replace=False)]) for _ in range(300)]
    sets += [[10000 + int(x)] for x in r.integers(0, 10000, size=400)]
    _check(eng, n, sets, 25, "overlap")


@pytest.mark.parametrize("hubs,noise", [(8, 0), (9, 30), (12, 400), (40, 20)])
def test_hubs_chosen_together(eng, hubs, noise):
    """Sets of every mix of a few hubs, whose counts one launch follows over several steps, with other nodes' counts
    in between."""
    n, count, k = 30000, 20000, 30
    r = np.random.default_rng(hubs + noise)
    sets = []
    for _ in range(count):
        s = np.concatenate([np.flatnonzero(r.random(hubs) < 0.3), hubs + r.integers(0, noise, 2) if noise else [],
                            1000 + r.choice(n - 1000, size=int(r.integers(1, 4)), replace=False)]).astype(np.int32)
        sets.append(np.unique(s))
    _check(eng, n, sets, k, "hubs")


def test_parts_of_several_tiles(eng):
    """More candidate entries per block than it holds at once, with long sets over the edges of its tiles."""
    n = 8192
    r = np.random.default_rng(0)
    sets = [r.permutation(n)[:int(s)] for s in r.integers(1, 8000, size=2600)]
    _check(eng, n, sets, 12, "tiles")
    _check(eng, n, [x[x % 97 == 0] if len(x) < 4000 else x for x in sets] + [[i] for i in range(900)], 40, "tiles, mixed")


@pytest.mark.parametrize("k", [2, 3, 4, 9])
def test_the_last_step_falls_below_the_threshold(eng, k):
    """k - 1 hubs that the candidates decide, the first of which covers all sets of the other candidates: only the last
    step needs a node outside them."""
    n = 20000
    r = np.random.default_rng(k)
    sets = [np.concatenate([[0], r.choice(np.arange(100, 9100), size=1500, replace=False)]) for _ in range(300)]
    sets += [[i] for i in range(1, k - 1) for _ in range(250 - 10 * i)]
    sets += [[10000 + int(x)] for x in r.integers(0, 10000, size=400)]
    _check(eng, n, sets, k, "last step")
