"""Maximum coverage on a slice of a collection: the offsets of sets [a, b) of a larger CSR, so that the first set does not
start at entry 0.  Seeds and gains equal the oracle's on those sets alone, for every way the sets are counted (few and many
entries, one step and several, with and without allocations)."""
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


@pytest.mark.parametrize("n,count,mean", [(300, 400, 3), (5000, 6000, 20), (60000, 400000, 5)])
def test_offsets_that_start_past_zero(eng, n, count, mean):
    import torch
    r = np.random.default_rng(n)
    ln = 1 + r.poisson(mean, size=count)
    sid = np.repeat(np.arange(count, dtype=np.int64), ln)
    flat = np.unique(sid * n + (n * r.random(int(ln.sum())) ** 3).astype(np.int64))
    # the sets before the slice hold the last nodes, which the slice hardly has
    first = count // 3
    nodes = np.where(flat // n < first, n - 1 - flat % n, flat % n).astype(np.int32)
    off = np.zeros(count + 1, dtype=np.int64)
    off[1:] = np.cumsum(np.bincount(flat // n, minlength=count))
    d_off, d_nodes = torch.from_numpy(off).cuda(), torch.from_numpy(nodes).cuda()
    for a, b in ((first, count), (first, count - count // 4), (1, count), (count - 1, count)):
        for k in (1, 2, 20, 60, 257):
            print(f"n={n} sets [{a}, {b}) k={k}", file=sys.stderr, flush=True)
            ws, wg = oracle.greedy(n, off[a:b + 1] - off[a], nodes[off[a]:off[b]], k)
            for fn in (eng.max_coverage, eng.max_coverage_noalloc):
                seeds, gains = fn(n, d_off[a:b + 1], d_nodes, k)
                assert np.array_equal(seeds, ws) and np.array_equal(gains, wg), (a, b, k, fn.__name__)
