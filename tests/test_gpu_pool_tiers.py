"""The default IC first tier in launches large enough for it (2048 sets).  Which sets it keeps, by the number it defers: all of up to 32 nodes, none beyond its largest
(160 nodes, or 128 when sets are stored under a device-memory budget) or with over 4096 groups, some of the sizes between
(as far as the wavefront's shared blocks go).  In-lists around 32 and 4096 groups at every alignment, set ids across 2^32.
Sets, widths and coverage equal the oracle's, stored sets with and without a budget."""
import sys

import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu
IC = 0


@pytest.mark.parametrize("budget", [0, 256 << 20])
@pytest.mark.parametrize("size", [1, 32, 33, 128, 129, 160, 161, 300])
def test_sets_of_one_size(size, budget):
    import paper_1404_0900_amd as tim
    copies, count = 40, 2500
    b = np.arange(size * copies)
    e = np.stack([b, b // size * size + (b % size + 1) % size], 1) if size > 1 else np.zeros((0, 2), dtype=np.int64)
    g = synth.from_edges(copies * size + 2, np.concatenate([e, [[copies * size, copies * size + 1]]]))
    thr = np.full(g.m, 0xFFFFFFFF, dtype=np.uint32)
    print(f"size={size} budget={budget}", file=sys.stderr, flush=True)
    with tim.Engine(0, budget_bytes=budget) as eng:
        dg = eng.upload(g, thr=thr)
        wo, wn, ww = oracle.sample_sets(g, IC, 9, 5, 0, count, thr=thr)[:3]
        big = int(np.sum(np.diff(wo) == size))  # all but the few sets rooted at the two last nodes
        off, nodes, widths, rr = eng.sample_rr(dg, IC, 9, 5, 0, count)
        assert np.array_equal(off.cpu().numpy(), wo)
        assert np.array_equal(widths.cpu().numpy().astype(np.uint64), np.asarray(ww, dtype=np.uint64))
        sid = np.repeat(np.arange(count, dtype=np.int64), np.diff(wo))
        assert np.array_equal(np.sort(sid * g.n + nodes.cpu().numpy()), np.sort(sid * g.n + wn))
        w = eng.sample_widths(dg, IC, 9, 5, 0, count, 7)[2]
        for deferred, most in ((w.deferred, 160), (rr.deferred, 128 if budget else 160)):
            if size <= 32:
                assert deferred == 0
            elif size > most:
                assert deferred == big
            else:
                assert deferred < big


@pytest.mark.parametrize("deg,deferred_all", [(16300, False), (16400, True)])
def test_sets_around_the_most_groups(deg, deferred_all):
    """A hub that takes in `deg` leaves nobody else reaches: 4096 groups hold 16384 edges."""
    import paper_1404_0900_amd as tim
    count = 3000
    # a thousand nodes have the hub as their only in-neighbour
    e = np.concatenate([np.stack([1 + np.arange(deg), np.zeros(deg, dtype=np.int64)], 1),
                        np.stack([np.zeros(1000, dtype=np.int64), deg + 1 + np.arange(1000)], 1)])
    g = synth.from_edges(deg + 1001, e)
    thr = np.where(np.repeat(np.arange(g.n), np.diff(g.off)) == 0, 0, 0xFFFFFFFF).astype(np.uint32)
    with tim.Engine(0) as eng:
        dg = eng.upload(g, thr=thr)
        wo, _, ww = oracle.sample_sets(g, IC, 9, 5, 0, count, thr=thr)[:3]
        ws, sizes, st = eng.sample_widths(dg, IC, 9, 5, 0, count, 7)
        assert np.array_equal(ws.cpu().numpy().astype(np.uint64), np.asarray(ww, dtype=np.uint64))
        assert np.array_equal(sizes.cpu().numpy(), np.diff(wo))
        hub = int(np.sum(np.asarray(ww) >= deg))
        assert hub > 50 and st.deferred == (hub if deferred_all else 0)


@pytest.mark.parametrize("deg", [1, 3, 4, 5, 121, 122, 123, 124, 125, 126, 128, 129, 250, 16381, 16390])
@pytest.mark.parametrize("kind", ["weighted cascade", "thresholds"])
def test_hub_in_lists_at_every_alignment(deg, kind):
    """Four hubs of in-degree `deg`, one-edge lists between them so that theirs start at different positions of a group;
    every other node has a hub as its only in-neighbour, so every set reaches one."""
    import paper_1404_0900_amd as tim
    n, count, first = deg + 7, 2100, (1 << 32) - 1000
    e = [((2 * i) % 8, x) for i, x in enumerate([1, 3, 5] + list(range(7, n)))]
    for h in (0, 2, 4, 6):
        e += [(7 + i, h) for i in range(deg)]
    g = synth.from_edges(n, e)
    thr = None
    if kind == "thresholds":
        thr = np.random.default_rng(deg).integers(0, 2**32, size=g.m, dtype=np.uint64).astype(np.uint32) // np.uint32(16 + deg)
    print(f"hub {deg} {kind}", file=sys.stderr, flush=True)
    with tim.Engine(0) as eng:
        dg = eng.upload(g, thr=thr)
        wo, wn, ww = oracle.sample_sets(g, IC, 9, 5, first, count, thr=thr)[:3]
        off, nodes, widths, _ = eng.sample_rr(dg, IC, 9, 5, first, count)
        eng.profile(True)
        ws, sizes, _ = eng.sample_widths(dg, IC, 9, 5, first, count, 7)
        assert eng.read_profile().sampler[0][0].launches == 1
        assert np.array_equal(off.cpu().numpy(), wo) and np.array_equal(sizes.cpu().numpy(), np.diff(wo))
        assert np.array_equal(widths.cpu().numpy().astype(np.uint64), np.asarray(ww, dtype=np.uint64))
        assert np.array_equal(ws.cpu().numpy().astype(np.uint64), np.asarray(ww, dtype=np.uint64))
        sid = np.repeat(np.arange(count, dtype=np.int64), np.diff(wo))
        assert np.array_equal(np.sort(sid * g.n + nodes.cpu().numpy()), np.sort(sid * g.n + wn))
        seeds = np.unique(wn[:3])
        assert eng.sample_cover(dg, IC, 9, 5, first, count, seeds).covered == len(np.unique(sid[np.isin(wn, seeds)]))
