"""Step graphs over a growing tree: the lists of the stage fills pass through every size class
(24, 96, 384 and 1440 items on the finest level) under one finest level, and each tree is stepped
by graphs of its own or of an earlier tree of the same class.  Bitwise the eager launches' run."""
import itertools

import numpy as np
import pytest

from paper_2012_04385_amd import workloads as W

pytestmark = pytest.mark.gpu


def test_growing_tree_graph_equals_eager():
    from paper_2012_04385_amd.mrfv import Solver
    pb = W.sod_single_level()
    pb.n0, pb.lmax, pb.dx0, pb.eps = (4, 4, 4), 2, 1.0 / 64, 1e9      # starts without level 2
    graph, eager = (Solver([pb], dtype="f32", batched=m, adapt=0).init() for m in (2, 1))
    cells = list(itertools.product(range(0, 8, 2), repeat=3))
    at = 0
    for upto in (1, 2, 4, 16, 17, 60):
        for s in (graph, eager):
            for c in cells[at:upto]:
                s.refine(0, 1, *c)
            s.run(3)
            s.check()
        at = upto
        a, b = graph.leaf_states(), eager.leaf_states()
        assert set(a) == set(b) and len(a) == 512 + 7 * upto
        for k in a:
            assert np.array_equal(a[k], b[k]), (upto, k)
