"""Exit counters at the most that a block's LDS takes, beside the FP64 tables and
the snapshot counts of streaming sets, and one slot pair beyond: pools, lanes and
batches count the same."""
import numpy as np
import pytest

import workloads

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec,edges", [(0, 5376), (0, 5377), (1, 5632), (0, 8192), (0, 8193)])
def test_counters_at_the_limit(prec, edges):
    import torch  # noqa: F401
    from paper_2512_02175_amd import binding as B
    w = np.where(np.arange(edges) % 1000 == 7, 1.0, 1e-4)
    G = B.mg_graph_create(workloads.star_graph(edges, 0.2, b_center=w / w.sum()))
    out = []
    for sched, batch in ((B.MG_SCHED_LANES, False), (B.MG_SCHED_POOLS_W8, False),
                         (B.MG_SCHED_LANES, True), (B.MG_SCHED_POOLS_W8, True)):
        p = B.mg_particles_init(G, 20_011, B.MG_INIT_AT_VERTEX, vertex=0, init_seed=3,
                                precision=prec, schedule=sched)
        B.mg_observe_histogram(p, 3, 4)
        if batch:
            B.mg_batch_simulate(B.mg_batch_create([p]), 30, 1e-3, 11)
        else:
            B.mg_simulate(p, 30, 1e-3, 11)
        r = B.mg_particles_read(p)
        out.append([r[f] for f in ("edge", "x", "alive")] + list(B.mg_exit_counts(p)) +
                   list(B.mg_observed_histogram(p)))
    for other in out[1:]:
        for x, y in zip(out[0], other):
            assert np.array_equal(x, y)
