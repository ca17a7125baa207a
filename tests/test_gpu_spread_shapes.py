"""tim_spread_mc at the edges of its kernel variants (LDS bitmaps of 2^16, 2^18, 2^19 and 1212416 nodes, device
stamps above), with hubs whose out-lists span several edge windows, against the CPU oracle run by run (equal)."""
import sys

import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu
IC, LT, TRIGGER = 0, 1, 2


@pytest.fixture(scope="module")
def eng():
    import paper_1404_0900_amd as tim
    e = tim.Engine(0)
    yield e
    e.close()


def _hub_graph(n, seed):
    """Node 0 has an edge to most nodes, node n-1 to a quarter, the rest a few random ones: out-lists from 0 to n-2."""
    r = np.random.default_rng(seed)
    v = np.arange(1, n - 1)
    a = np.stack([np.zeros(n - 2, dtype=np.int64), v], axis=1)[r.random(n - 2) < 0.9]
    b = np.stack([np.full(n - 2, n - 1, dtype=np.int64), v], axis=1)[r.random(n - 2) < 0.25]
    c = r.integers(0, n, size=(n, 2))
    e = np.unique(np.concatenate([a, b, c[c[:, 0] != c[:, 1]]]), axis=0)
    order = np.lexsort((e[:, 0], e[:, 1]))
    e = e[order]
    off = np.zeros(n + 1, dtype=np.int64)
    off[1:] = np.cumsum(np.bincount(e[:, 1], minlength=n))
    return synth.Graph(n, len(e), off, e[:, 0].astype(np.int32).copy(), f"hub{n}")


@pytest.mark.parametrize("n", [2, 33, 65_536, 65_537, 262_144, 262_145, 524_289, 1_212_416, 1_212_417])
@pytest.mark.parametrize("case", ["ic", "ic-thr", "lt", "lt-weighted"])
def test_spread_variants_equal_oracle(eng, n, case):
    g = _hub_graph(n, n) if n > 100 else synth.from_edges(n, [(0, n - 1), (n - 1, 0)])
    thr = None
    model = IC if case.startswith("ic") else LT
    if case == "ic-thr":
        thr = synth.random_thresholds(g.m, 3)
    elif case == "lt-weighted":
        thr = synth.random_lt_thresholds(g, 4, total=0.9)
    dg = eng.upload(g, thr=thr if model == IC else None)
    if case == "lt-weighted":
        eng.set_lt_weights(dg, g, thr)
    S = np.array([0, n - 1, 0, n // 2], dtype=np.int32)  # a repeat among them
    runs = 5 if n > 100_000 else 40
    print(f"{case} n={n} m={g.m}", file=sys.stderr, flush=True)
    for _ in range(2):  # the second call finds the lists the first one built
        _, total, counts = eng.spread(dg, model, 64, S, runs, first=(1 << 33) + 7, per_run=True)
        want = oracle.forward_spread(g, model, 64, (1 << 33) + 7, runs, S, thr=thr)
        assert np.array_equal(counts.cpu().numpy().astype(np.uint64), want)
        assert total == int(want.sum())
    eng.free(dg)
