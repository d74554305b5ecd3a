"""The untuned automatic schedule on both sides of the drift at which it takes
one particle per lane (0.85 of a step's noise towards an end on every edge):
the same bits as the pools."""
import numpy as np
import pytest

import workloads

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("length", [2.0, np.inf])
@pytest.mark.parametrize("dt", [7.2e-3, 7.3e-3, 1e-2])
def test_auto_equals_pools(length, dt):
    from paper_2512_02175_amd import binding as B
    G = B.mg_graph_create(workloads.paper_star5("linear", length))
    out = []
    for sched in (B.MG_SCHED_AUTO, B.MG_SCHED_POOLS_W8):
        p = B.mg_particles_init(G, 10_001, B.MG_INIT_AT_VERTEX, vertex=0, init_seed=3,
                                precision=1, schedule=sched)
        B.mg_observe_histogram(p, 16, 7)
        for k in (1, 40):
            B.mg_simulate(p, k, dt, 11)
        r = B.mg_particles_read(p)
        out.append([r[f] for f in ("edge", "x", "alive")] + list(B.mg_exit_counts(p)) +
                   list(B.mg_observed_histogram(p)))
    for x, y in zip(*out):
        assert np.array_equal(x, y)
