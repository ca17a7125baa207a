"""LT walks that run along a tail into a cycle, with both around the sizes where the table walk (192 nodes) hands over to
the cycle search, which goes on from the table's last node: stored sets, sizes, widths and coverage equal the oracle's."""
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


@pytest.mark.parametrize("tail", [0, 1, 100, 190, 191, 192, 193, 400])
@pytest.mark.parametrize("cycle", [2, 3, 91, 191, 192, 193, 256, 447, 448, 449, 700])
def test_tails_into_cycles(eng, tail, cycle):
    size, copies, count = tail + cycle, 24, 900
    b = np.arange(size * copies)
    i, base = b % size, b // size * size
    # a walk goes from node i to i + 1, from the cycle's last node back to its first
    to = base + np.where(i + 1 < size, i + 1, tail)
    g = synth.from_edges(size * copies, np.stack([to, b], 1))
    dg = eng.upload(g)
    print(f"tail={tail} cycle={cycle}", file=sys.stderr, flush=True)
    off, nodes, widths, _ = eng.sample_rr(dg, LT, 3, 2, 11, count)
    ws, sizes, st = eng.sample_widths(dg, LT, 3, 2, 11, count, 5)
    wo, wn, ww = oracle.sample_sets(g, LT, 3, 2, 11, count)
    assert np.array_equal(off.cpu().numpy(), wo) and np.array_equal(sizes.cpu().numpy(), np.diff(wo))
    assert np.array_equal(widths.cpu().numpy().astype(np.uint64), ww)
    assert np.array_equal(ws.cpu().numpy().astype(np.uint64), ww)
    assert st.kappa_sum == oracle.round_sum(g, LT, 3, 2, 11, count, 5)["sum"]
    sid = np.repeat(np.arange(count, dtype=np.int64), np.diff(wo))
    assert np.array_equal(np.sort(sid * g.n + nodes.cpu().numpy()), np.sort(sid * g.n + wn))
    for seeds in ([0, size - 1], [tail], [size + tail + cycle // 2]):
        assert eng.sample_cover(dg, LT, 3, 2, 11, count, seeds).covered == len(np.unique(sid[np.isin(wn, seeds)]))
    eng.free(dg)
