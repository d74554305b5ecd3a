"""The uniform placement finds each draw's edge inside the bucket that a guide
table gives for the draw's top bits: the oracle's edges, at edge numbers about
the powers of two where the guide grows, with even lengths, with one edge that
fills nearly every bucket, and with runs of edges too short to own a draw."""
import numpy as np
import pytest

import workloads

pytestmark = pytest.mark.gpu


def _lengths(kind, E):
    L = np.ones(E)
    if kind == "one_long":
        L[E // 2] = 1e6
    elif kind == "tiny_runs":
        L[np.arange(E) % 3 != 0] = 1e-12
    return L


@pytest.mark.parametrize("kind", ["even", "one_long", "tiny_runs"])
@pytest.mark.parametrize("E", [1, 2, 3, 4, 5, 31, 32, 33, 1000, 4097])
def test_uniform_placement_equals_oracle(orc, kind, E):
    from paper_2512_02175_amd import binding as B
    g = workloads.star_graph(E, _lengths(kind, E))
    n = 20_001
    st = orc.init(g, n, orc.INIT_UNIFORM_LENGTH, seed=9)
    p = B.mg_particles_init(B.mg_graph_create(g), n, 2, init_seed=9)
    r = B.mg_particles_read(p)
    assert np.array_equal(r["edge"], st.edge)
    # one product of the drawn fraction with the length: a rounding or two
    assert np.allclose(r["x"], st.x, rtol=4.5e-16, atol=0.0)
