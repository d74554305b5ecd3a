"""First reservations by a wave's place in the grid: every particle is taken once
by launches of one and a few steps, at set sizes about one particle, one claim,
one wave, one block, and the sizes where the particles per wave grow and where
the counter begins to hand out ids."""
import numpy as np
import pytest

import workloads

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec,sched", [(0, "POOLS_W8"), (1, "POOLS_W8"), (1, "POOLS"), (1, "POOLS256")])
def test_every_particle_steps_once(prec, sched):
    import torch  # noqa: F401
    from paper_2512_02175_amd import binding as B
    G = B.mg_graph_create(workloads.star_graph(5, 0.4, -3.0, None, 1.0))
    for n in (1, 15, 16, 17, 63, 64, 65, 255, 257, 1023, 16_383, 16_385, 32_767, 32_769, 131_071,
              131_073, 393_217, 524_289, 786_433, 1_572_865):
        out = []
        for s in (B.MG_SCHED_LANES, getattr(B, "MG_SCHED_" + sched)):
            p = B.mg_particles_init(G, n, B.MG_INIT_UNIFORM_LENGTH, init_seed=n, precision=prec,
                                    schedule=s)
            for k in (1, 1, 3, 40):
                B.mg_simulate(p, k, 1e-2, 11)
            r = B.mg_particles_read(p)
            out.append([r[f] for f in ("edge", "x", "alive")] + list(B.mg_exit_counts(p)))
        assert int(out[1][-1][3]) == 45 * n, n
        for x, y in zip(*out):
            assert np.array_equal(x, y), n
