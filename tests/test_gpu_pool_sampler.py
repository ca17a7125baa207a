"""The IC first tier that deals the groups of sixteen sets over a wavefront, at the edges of its structures: sets around
its blocks of 32 nodes and its limit of 160, hubs around its limit for whole-wavefront nodes and its most groups, in-lists
at every alignment, and set ids across 2^32.  Sets (sorted), widths and coverage equal the oracle's."""
import sys

import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu
IC = 0


@pytest.fixture(scope="module")
def eng():
    import paper_1404_0900_amd as tim
    e = tim.Engine(0)
    yield e
    e.close()


def _check(eng, g, thr, first, count, tag):
    print(f"{tag}: n={g.n} m={g.m} sets={count}", file=sys.stderr, flush=True)
    dg = eng.upload(g, thr=thr)
    off, nodes, widths, _ = eng.sample_rr(dg, IC, 9, 5, first, count)
    off, nodes = off.cpu().numpy(), nodes.cpu().numpy()
    ws, sizes, _ = eng.sample_widths(dg, IC, 9, 5, first, count, 7)
    wo, wn, ww = oracle.sample_sets(g, IC, 9, 5, first, count, thr=thr)[:3]
    assert np.array_equal(off, wo)
    assert np.array_equal(widths.cpu().numpy().astype(np.uint64), np.asarray(ww, dtype=np.uint64))
    assert np.array_equal(ws.cpu().numpy().astype(np.uint64), np.asarray(ww, dtype=np.uint64))
    assert np.array_equal(sizes.cpu().numpy(), np.diff(wo))
    sid = np.repeat(np.arange(count, dtype=np.int64), np.diff(wo))
    assert np.array_equal(np.sort(sid * g.n + nodes), np.sort(sid * g.n + wn))
    seeds = np.unique(nodes[:3])
    got = eng.sample_cover(dg, IC, 9, 5, first, count, seeds).covered
    assert got == len(np.unique(sid[np.isin(wn, seeds)]))
    eng.free(dg)


@pytest.mark.parametrize("size", [1, 2, 31, 32, 33, 64, 65, 128, 159, 160, 161, 300])
@pytest.mark.parametrize("kind", ["cycle", "tree"])
def test_certain_sets_of_one_size(eng, size, kind):
    """Every edge live: disjoint cycles (one node per level) or two-level trees (every node at once) of `size` nodes."""
    copies = 40
    e = []
    for c in range(copies):
        b = c * size
        if size > 1 and kind == "cycle":
            e += [(b + i, b + (i + 1) % size) for i in range(size)]
        elif size > 1:
            e += [(b + 1 + i, b) for i in range(size - 1)] + [(b, b + 1 + i) for i in range(size - 1)]
    e.append((copies * size, copies * size + 1))
    g = synth.from_edges(copies * size + 2, e)
    _check(eng, g, np.full(g.m, 0xFFFFFFFF, dtype=np.uint32), (1 << 32) - 700, 1500, f"{kind} {size}")


@pytest.mark.parametrize("deg", [1, 3, 4, 5, 121, 122, 123, 124, 125, 126, 128, 129, 250, 16381, 16390])
def test_hub_in_lists_at_every_alignment(eng, deg):
    """Four hubs of in-degree `deg`, one-edge lists between them so that theirs start at different positions of a group;
    every other node has a hub as its only in-neighbour, so every set reaches one (31, 32 and 4096 groups among them)."""
    n = deg + 7
    e = [((2 * i) % 8, x) for i, x in enumerate([1, 3, 5] + list(range(7, n)))]
    for h in (0, 2, 4, 6):
        e += [(7 + i, h) for i in range(deg)]
    g = synth.from_edges(n, e)
    count = 2000 if deg < 1000 else 900
    _check(eng, g, None, 0, count, f"hub {deg} weighted cascade")
    thr = np.random.default_rng(deg).integers(0, 2**32, size=g.m, dtype=np.uint64).astype(np.uint32) // np.uint32(16 + deg)
    _check(eng, g, thr, 5, count, f"hub {deg} thresholds")
