"""tim_spread_mc where runs start with device stamps and large ones go on to the LDS bitmap (262145 to 1212416 nodes, more
runs than the bitmap's blocks): runs around the 64 visited nodes and 1024 edges of the hand-over, more large runs than its
list takes (65536), and a mix against the oracle, run by run."""
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


def _graph(n, e):
    e = np.asarray(e, dtype=np.int64)
    order = np.lexsort((e[:, 0], e[:, 1]))
    e = e[order]
    off = np.zeros(n + 1, dtype=np.int64)
    off[1:] = np.cumsum(np.bincount(e[:, 1], minlength=n))
    return synth.Graph(n, len(e), off, e[:, 0].astype(np.int32).copy(), f"passes{n}")


@pytest.mark.parametrize("n", [262_145, 600_000])
@pytest.mark.parametrize("runs", [100, 3000, 70_000])
def test_certain_runs_around_the_limits(eng, n, runs):
    """Every edge live.  Stars of 63 to 1100 leaves and chains of stars, side by side: the spread is the nodes reached."""
    e, at, want = [], 0, {}
    for size in (0, 62, 63, 64, 65, 66, 1023, 1024, 1025, 1100):
        want[at] = size + 1
        e.append(np.stack([np.full(size, at), at + 1 + np.arange(size)], 1))
        at += size + 1
    for leaves in (30, 40, 1020):  # a star whose leaves have a leaf each
        want[at] = 2 * leaves + 1
        e.append(np.stack([np.full(leaves, at), at + 1 + np.arange(leaves)], 1))
        e.append(np.stack([at + 1 + np.arange(leaves), at + 1 + leaves + np.arange(leaves)], 1))
        at += 2 * leaves + 1
    g = _graph(n, np.concatenate(e))
    dg = eng.upload(g, thr=np.full(g.m, 0xFFFFFFFF, dtype=np.uint32))
    for seeds in [[s] for s in want] + [list(want)[1:6], list(want)]:
        if runs == 70_000 and len(seeds) > 1:
            continue
        print(f"n={n} runs={runs} seeds={seeds}", file=sys.stderr, flush=True)
        mean, total, per = eng.spread(dg, IC, 3, seeds, runs, per_run=True)
        w = sum(want[s] for s in seeds)
        assert total == w * runs and mean == w
        assert int(per.min()) == int(per.max()) == w
    eng.free(dg)


@pytest.mark.parametrize("n", [262_145, 1_000_003])
@pytest.mark.parametrize("model", [IC, LT])
def test_mixed_runs_equal_oracle(eng, n, model):
    g = synth.chung_lu(n, 4 * n, 2.1, 7)
    dg = eng.upload(g)
    hub = int(np.argsort(-np.bincount(g.src, minlength=n))[500])
    for seeds, runs in (([5], 2000), ([hub], 600), ([5, 77, 1234, n - 1], 1500)):
        print(f"n={n} model={model} seeds={seeds}", file=sys.stderr, flush=True)
        _, total, per = eng.spread(dg, model, 11, seeds, runs, first=(1 << 32) - 50, per_run=True)
        want = oracle.forward_spread(g, model, 11, (1 << 32) - 50, runs, seeds)
        assert np.array_equal(per.cpu().numpy().astype(np.int64), np.asarray(want, dtype=np.int64))
        assert total == int(np.sum(want))
    eng.free(dg)


def test_triggering_runs_equal_oracle(eng):
    n = 262_145
    g = synth.chung_lu(n, 3 * n, 2.1, 5)
    trig = synth.random_triggering(g, 6)
    dg = eng.upload(g)
    eng.set_triggering(dg, g, trig)
    hub = int(np.argsort(-np.bincount(g.src, minlength=n))[200])
    for seeds in ([hub], [5, 77, hub]):
        print(f"triggering seeds={seeds}", file=sys.stderr, flush=True)
        _, total, per = eng.spread(dg, TRIGGER, 11, seeds, 1500, per_run=True)
        want = oracle.forward_spread(g, TRIGGER, 11, 0, 1500, seeds, thr=trig)
        assert np.array_equal(per.cpu().numpy().astype(np.int64), np.asarray(want, dtype=np.int64))
    eng.free(dg)
