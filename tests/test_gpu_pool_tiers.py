"""Which sets the default IC first tier keeps, by the number it defers: all of up to 32 nodes, none beyond its largest
(160 nodes, or 128 when sets are stored under a device-memory budget) or with over 4096 groups, some of the sizes between
(as far as the wavefront's shared blocks go).  Stored sets equal the oracle's with and without a budget."""
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
    copies, count = 40, 1500
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
