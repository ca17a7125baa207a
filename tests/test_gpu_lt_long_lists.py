"""LT launches with more long chains than the table walk takes (32768), so that the blocks of the cycle search share them:
the launch's totals (kappa sum, widths, nodes, coverage), which its blocks add up, equal the oracle's, and so do those of
lists just below."""
import sys

import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu
LT = 1


@pytest.mark.parametrize("count", [32767, 32768, 32769, 33000, 50000, 150000])
def test_totals_of_long_lists(count):
    import paper_1404_0900_amd as tim
    size, copies, k = 90, 60, 7
    b = np.arange(size * copies)
    edges = np.stack([b, b // size * size + (b + 1 - b // size * size) % size], 1)
    # every other cycle takes in a leaf at each node, so that walks end early there and widths differ
    leaf = b[(b // size) % 2 == 1]
    n = size * copies + len(leaf)
    g = synth.from_edges(n, np.concatenate([edges, np.stack([size * copies + np.arange(len(leaf)), leaf], 1)]))
    with tim.Engine(0) as eng:
        dg = eng.upload(g)
        first = 0
        wo, wn, ww = oracle.sample_sets(g, LT, 4, 2, first, 4 * count)
        long_ = np.flatnonzero(np.diff(wo) > 64)
        total = int(long_[count - 1]) + 1  # this many sets hold `count` long chains
        print(f"long chains={count} sets={total}", file=sys.stderr, flush=True)
        wo, ww = wo[:total + 1], ww[:total]
        for _ in range(3):
            _, _, st = eng.sample_widths(dg, LT, 4, 2, first, total, k, per_set=False)
            assert st.deferred == count
            assert st.kappa_sum == oracle.round_sum(g, LT, 4, 2, first, total, k)["sum"]
            assert st.width_sum == int(ww.sum()) and st.node_sum == int(wo[-1])
            off, _, _, st = eng.sample_rr(dg, LT, 4, 2, first, total)
            assert st.width_sum == int(ww.sum()) and st.node_sum == int(wo[-1]) and st.deferred == count
            assert np.array_equal(off.cpu().numpy(), wo)
            seeds = [0, size + 3, n - 1]
            sid = np.repeat(np.arange(total), np.diff(wo))
            assert eng.sample_cover(dg, LT, 4, 2, first, total, seeds).covered == len(
                np.unique(sid[np.isin(wn[:wo[-1]], seeds)]))
