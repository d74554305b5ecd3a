"""A batch runs its sets on the first set's stream: a set of another stream whose
streaming was switched on just before gives the counts of the set alone."""
import numpy as np
import pytest

import workloads

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", [0, 1])
def test_streaming_switched_on_just_before_a_batch(prec):
    import ctypes as C

    import torch
    from paper_2512_02175_amd import binding as B
    streams = [torch.cuda.Stream() for _ in range(2)]
    G = [B.mg_graph_create(workloads.star_graph(E, 0.5)) for E in (3, 4000)]

    def make(on):
        return [B.mg_particles_init(g, 5001, 2, init_seed=i, graph_tag=i, precision=prec,
                                    schedule=B.MG_SCHED_POOLS_W8,
                                    stream=C.c_void_p(s.cuda_stream))
                for i, (g, s) in enumerate(zip(G, on))]
    alone = make([streams[0]] * 2)
    for p in alone:
        B.mg_observe_histogram(p, 64, 1)
        B.mg_simulate(p, 5, 1e-2, 7)
    sets = make(streams)
    b = B.mg_batch_create(sets)
    for _ in range(2):                      # the second time replaces the first
        for p in sets:
            B.mg_observe_histogram(p, 64, 1)
        B.mg_batch_simulate(b, 5, 1e-2, 7)
        torch.cuda.synchronize()
        for p, q in zip(sets, alone):
            h, k = B.mg_observed_histogram(p)
            assert k == 5 and int(h.sum()) == 5 * 5001
            if B.mg_particles_step(p) == 5:
                assert np.array_equal(h, B.mg_observed_histogram(q)[0])
