"""Which first-tier shape an IC launch of few sets takes (by the profile's ic_wide entries): below one set per twenty nodes
or 2048 sets the 64-lane shape on sparse graphs, below 65536 sets on graphs of ten edges per node or more.  Widths, sizes and
the kappa sum equal the oracle's on both sides of the line."""
import sys

import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu
IC = 0


@pytest.mark.parametrize("n,m,line", [(3000, 12000, 2048), (40001, 160004, 2048), (100001, 400004, 5000),
                                      (3000, 29999, 2048), (3000, 30000, 65536),
                                      (1_400_000, 14_000_000, 70000)])
def test_lines_between_the_shapes(n, m, line):
    import paper_1404_0900_amd as tim
    g = synth.chung_lu(n, m, 2.1, 3)
    with tim.Engine(0) as eng:
        dg = eng.upload(g)
        for count in (line - 1, line):
            print(f"n={n} m={m} sets={count}", file=sys.stderr, flush=True)
            eng.profile(True)
            ws, sizes, st = eng.sample_widths(dg, IC, 3, 2, 0, count, 9)
            p = eng.read_profile()
            assert (p.ic_wide[0].launches, p.sampler[0][0].launches) == ((1, 0) if count < line else (0, 1))
            wo, _, ww = oracle.sample_sets(g, IC, 3, 2, 0, count)[:3]
            assert np.array_equal(ws.cpu().numpy().astype(np.uint64), np.asarray(ww, dtype=np.uint64))
            assert np.array_equal(sizes.cpu().numpy(), np.diff(wo))
            assert st.kappa_sum == oracle.round_sum(g, IC, 3, 2, 0, count, 9)["sum"]
