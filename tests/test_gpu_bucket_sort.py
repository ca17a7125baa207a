"""The counting sort behind greedy coverage: sets around its tiles (512 sets), windows (4096 entries) and 64-entry chunks,
empty sets, one and several buckets of 8192 nodes, with the set ids (k above the candidate greedy's limit) and without."""
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


@pytest.mark.parametrize("k", [3, 260])
@pytest.mark.parametrize("n,lens", [
    (8192, [4096] * 260),
    (8193, [4095, 1, 4097, 0, 63, 64, 65] * 130),
    (300, [0, 1, 2, 300] * 3600),
    (50000, [50000, 0, 0, 1] * 22),
    (200000, "mixed"),
])
def test_sort_of_the_entries(eng, n, lens, k):
    import torch
    r = np.random.default_rng(n + k)
    if lens == "mixed":
        lens = np.where(r.random(400000) < 0.001, 700, r.integers(0, 6, size=400000))
    print(f"n={n} sets={len(lens)} k={k}", file=sys.stderr, flush=True)
    lens = np.asarray(lens, dtype=np.int64)
    off = np.zeros(len(lens) + 1, dtype=np.int64)
    off[1:] = np.cumsum(lens)
    # distinct nodes per set: consecutive ones from a skewed start, modulo n
    first = (n * r.random(len(lens)) ** 3).astype(np.int64)
    step = np.arange(off[-1]) - np.repeat(off[:-1], lens)
    nodes = ((np.repeat(first, lens) + step) % n).astype(np.int32)
    seeds, gains = eng.max_coverage(n, torch.from_numpy(off).cuda(), torch.from_numpy(nodes).cuda(), k)
    ws, wg = oracle.greedy(n, off, nodes, k)
    assert np.array_equal(seeds, ws) and np.array_equal(gains, wg)
