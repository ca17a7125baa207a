"""LT chains around the sizes where they change hands: 64 nodes (the first tier's), 192 (the table walk's) and lists of more
chains than the table walk takes (32768).  Sets (sorted), sizes, widths and coverage equal the oracle's."""
import sys

import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu
LT = 1


@pytest.fixture(scope="module")
def eng():
    import paper_1404_0900_amd as tim
    e = tim.Engine(0)
    yield e
    e.close()


def _chains(size, copies, cycle):
    """Disjoint chains or cycles of `size` nodes: every node has one in-edge, or none at a chain's start."""
    e = []
    for c in range(copies):
        b = c * size
        e += [(b + i, b + i + 1) for i in range(size - 1)] + ([(b + size - 1, b)] if cycle else [])
    return synth.from_edges(size * copies, e)


@pytest.mark.parametrize("size", [64, 65, 66, 128, 191, 192, 193, 194, 256, 400])
@pytest.mark.parametrize("kind", ["cycle", "chain", "weighted"])
def test_chains_of_one_size(eng, size, kind):
    g = _chains(size, 30, kind != "chain")
    thr = None
    if kind == "weighted":  # stops with probability 2^-12 at every node
        thr = np.full(g.m, 0xFFFFFFFF - (1 << 20), dtype=np.uint32)
    dg = eng.upload(g)
    if thr is not None:
        eng.set_lt_weights(dg, g, thr)
    for count in (1, 700, 3000):
        print(f"{kind} {size} sets={count}", file=sys.stderr, flush=True)
        off, nodes, widths, _ = eng.sample_rr(dg, LT, 3, 2, 11, count)
        ws, sizes, _ = eng.sample_widths(dg, LT, 3, 2, 11, count, 5)
        wo, wn, ww = oracle.sample_sets(g, LT, 3, 2, 11, count, thr=thr)
        assert np.array_equal(off.cpu().numpy(), wo) and np.array_equal(sizes.cpu().numpy(), np.diff(wo))
        assert np.array_equal(widths.cpu().numpy().astype(np.uint64), ww)
        assert np.array_equal(ws.cpu().numpy().astype(np.uint64), ww)
        sid = np.repeat(np.arange(count, dtype=np.int64), np.diff(wo))
        assert np.array_equal(np.sort(sid * g.n + nodes.cpu().numpy()), np.sort(sid * g.n + wn))
        seeds = [0, g.n // 2]
        assert eng.sample_cover(dg, LT, 3, 2, 11, count, seeds).covered == len(np.unique(sid[np.isin(wn, seeds)]))
    eng.free(dg)


@pytest.mark.parametrize("count", [32768, 32769, 40000])
def test_lists_around_the_table_walks_limit(eng, count):
    g = _chains(70, 50, True)
    dg = eng.upload(g)
    ws, sizes, st = eng.sample_widths(dg, LT, 4, 2, 0, count, 5)
    assert st.deferred == count
    assert int(sizes.min()) == int(sizes.max()) == 70 and int(ws.min()) == int(ws.max()) == 70
    off, nodes, _, _ = eng.sample_rr(dg, LT, 4, 2, 0, count)
    x = nodes.cpu().numpy().reshape(count, 70)
    assert np.array_equal(np.sort(x, axis=1) % 70, np.tile(np.arange(70), (count, 1)))
    eng.free(dg)


@pytest.mark.parametrize("d", [1, 2, 3, 4, 5, 7, 8, 9, 64, 1000, 20000])
@pytest.mark.parametrize("kind", ["random", "half", "steps", "one", "equal"])
def test_weighted_pick_at_hubs(eng, d, kind):
    """Hubs of in-degree d over leaves whose only in-neighbour is a hub; cumulative thresholds from even to extreme."""
    hubs, leaves = 4, max(d, 8)
    e = [(hubs + (i * 7 + h) % leaves, h) for h in range(hubs) for i in range(d)]
    e += [(x % hubs, hubs + x) for x in range(leaves)]
    g = synth.from_edges(hubs + leaves, sorted(set(e)))
    r = np.random.default_rng(d)
    thr = np.empty(g.m, dtype=np.uint32)
    for v in range(g.n):
        k = int(g.off[v + 1] - g.off[v])
        w = {"random": r.random(k) + 1e-3, "half": r.random(k) + 1e-3, "steps": np.where(r.random(k) < 0.05, 1.0, 1e-12),
             "one": np.eye(1, k, k // 2)[0] + 1e-15, "equal": np.ones(k)}[kind]
        c = np.cumsum(w) / w.sum() * (0.5 if kind == "half" else 1.0)
        thr[g.off[v]:g.off[v + 1]] = np.maximum(np.floor(c * 2.0**32) - 1, 0).clip(0, 2**32 - 1).astype(np.uint64)
    dg = eng.upload(g)
    eng.set_lt_weights(dg, g, thr)
    print(f"pick {kind} d={d} m={g.m}", file=sys.stderr, flush=True)
    count = 3000
    off, nodes, widths, _ = eng.sample_rr(dg, LT, 5, 3, 0, count)
    wo, wn, ww = oracle.sample_sets(g, LT, 5, 3, 0, count, thr=thr)
    assert np.array_equal(off.cpu().numpy(), wo) and np.array_equal(widths.cpu().numpy().astype(np.uint64), ww)
    sid = np.repeat(np.arange(count, dtype=np.int64), np.diff(wo))
    assert np.array_equal(np.sort(sid * g.n + nodes.cpu().numpy()), np.sort(sid * g.n + wn))
    eng.free(dg)
