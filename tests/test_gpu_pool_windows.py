"""Wave-pool windows at their edges, against the lane schedule bit for bit:
launches that start and end at every step of a four-step random-number group,
sets on both sides of each pool size (16, 32, 64 and 128 particles a wave),
and snapshots that fall on every step of a group, more than one per group."""
import numpy as np
import pytest

import workloads

pytestmark = pytest.mark.gpu

CALLS = (1, 2, 3, 4, 5, 7, 9, 1, 6)   # starts and ends at all offsets mod 4


@pytest.fixture(scope="module")
def B():
    from paper_2512_02175_amd import binding
    binding.lib()
    return binding


def _run(B, G, g, n, prec, sched, every, calls=CALLS, dt=1e-2):
    p = B.mg_particles_init(G, n, B.MG_INIT_AT_VERTEX, vertex=0, init_seed=3, precision=prec,
                            schedule=sched, trace=True)
    if every:
        B.mg_observe_histogram(p, 16, every)
    for k in calls:
        B.mg_simulate(p, k, dt, 11)
    r = B.mg_particles_read(p, trace=True)
    out = [r[k] for k in ("edge", "x", "alive", "seqhash", "hits")]
    out += list(B.mg_exit_counts(p))
    if every:
        out += list(B.mg_observed_histogram(p))
    return out


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("n,every", [(1, 1), (15, 2), (16, 3), (17, 0), (16384, 5), (16385, 4),
                                     (32769, 0), (131072, 3), (131073, 0)])
def test_pools_equal_lanes_at_window_edges(B, prec, n, every):
    g = workloads.config2()[0] if n % 2 else workloads.star_graph(5, 0.4, -3.0, None, 1.0)
    G = B.mg_graph_create(g)
    a = _run(B, G, g, n, prec, B.MG_SCHED_LANES, every)
    b = _run(B, G, g, n, prec, B.MG_SCHED_POOLS_W8, every)
    for x, y in zip(a, b):
        assert np.array_equal(x, y)


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("name", ["cubic", "tables", "wentzell"])
def test_general_coefficients_at_window_edges(B, prec, name):
    g = {"cubic": lambda: workloads.double_well_star(7, 2),
         "tables": lambda: workloads.periodic_star(5, 4),
         "wentzell": lambda: workloads.wentzell_star(5, 7)}[name]()
    G = B.mg_graph_create(g)
    if name == "wentzell":   # start away from the sticky centre as well as near it
        kw = dict(dt=3e-3)
    else:
        kw = {}
    def run(sched):
        p = B.mg_particles_init(G, 1000, B.MG_INIT_UNIFORM_LENGTH, init_seed=3, precision=prec,
                                schedule=sched, trace=True)
        B.mg_observe_histogram(p, 16, 3)
        for k in CALLS * 3:
            B.mg_simulate(p, k, kw.get("dt", 1e-2), 11)
        r = B.mg_particles_read(p, trace=True)
        return [r[k] for k in ("edge", "x", "alive", "seqhash", "hits")] + \
            list(B.mg_exit_counts(p)) + list(B.mg_observed_histogram(p))
    for x, y in zip(run(B.MG_SCHED_LANES), run(B.MG_SCHED_POOLS_W8)):
        assert np.array_equal(x, y)
