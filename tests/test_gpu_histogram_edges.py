"""Histogram kernels at the edges of their ranges, against the same binning of
the particles read back: bins just within and beyond one LDS copy, more edges
than the LDS keeps the binning of, and sets whose size is no multiple of the
four particles that a thread takes."""
import numpy as np
import pytest

import workloads

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def B():
    from paper_2512_02175_amd import binding
    binding.lib()
    return binding


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("edges,nb,n", [(3, 1, 1), (3, 7, 2), (64, 256, 3), (64, 256, 100_003),
                                        (512, 64, 4097), (513, 63, 50_001), (1024, 32, 70_002),
                                        (1025, 32, 70_002), (2000, 64, 200_001), (1, 32769, 5)])
def test_histogram_equals_binned_positions(B, prec, edges, nb, n):
    rng = np.random.default_rng(edges + n)
    g = workloads.star_graph(edges, rng.uniform(0.3, 2.0, size=edges))
    g.vtx_kind[1] = 1 if edges > 1 else 0   # some particles are removed
    G = B.mg_graph_create(g)
    p = B.mg_particles_init(G, n, B.MG_INIT_UNIFORM_LENGTH, init_seed=2, precision=prec)
    B.mg_simulate(p, 5, 1e-2, 7)
    r = B.mg_particles_read(p)
    live = r["alive"] == 1
    e, x = r["edge"][live], r["x"][live]
    b = np.clip(np.floor(x * (nb / g.length[e])), 0, nb - 1).astype(np.int64)
    want = np.bincount(e.astype(np.int64) * nb + b, minlength=edges * nb)
    assert np.array_equal(B.mg_histogram(p, nb).ravel().astype(np.int64), want)
    off, up, _ = workloads.csr_bins(g, 0.01, min(nb, 60))
    pos = np.searchsorted(up + np.repeat(np.arange(edges) * 1e3, np.diff(off)), x + e * 1e3)
    want = np.bincount(np.clip(pos, off[e], off[e + 1] - 1), minlength=int(off[-1]))
    got = B.mg_histogram_csr(p, off, up).astype(np.int64)
    # (the shifted search may round a position within 1e-10 of a boundary)
    assert got.sum() == live.sum() and np.abs(got - want).sum() <= 2 * (n > 1e5)
