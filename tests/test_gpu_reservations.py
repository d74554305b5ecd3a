"""Reservations and pool sizes by launch length: launches on both sides of 32
steps, of sets about the sizes where a wave's pool and its reservations grow
(2 and 6 waves of 64 particles a SIMD, eight full pools a SIMD), against the
lane schedule bit for bit."""
import numpy as np
import pytest

import workloads

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("n", [131_073, 393_216, 393_217, 1_048_577, 1_200_003])
def test_reservations_equal_lanes(prec, n):
    from paper_2512_02175_amd import binding as B
    G = B.mg_graph_create(workloads.star_graph(5, 0.4, -3.0, None, 1.0))
    out = []
    for sched in (B.MG_SCHED_LANES, B.MG_SCHED_POOLS_W8):
        p = B.mg_particles_init(G, n, B.MG_INIT_AT_VERTEX, vertex=0, init_seed=3,
                                precision=prec, schedule=sched)
        for k in (31, 32, 33):
            B.mg_simulate(p, k, 1e-2, 11)
        r = B.mg_particles_read(p)
        out.append([r[f] for f in ("edge", "x", "alive")] + list(B.mg_exit_counts(p)))
    for x, y in zip(*out):
        assert np.array_equal(x, y)
