"""Host paths of the C ABI that a GPU test cannot force: failing allocations and
launches, captures, other devices and streams, and which kernel a set runs.
They run over the HIP stand-in, without a GPU."""
import os

import pytest

import host_stub

ROOT = host_stub.ROOT


@pytest.fixture(scope="module")
def stub(tmp_path_factory):
    if not os.path.exists(os.path.join(ROOT, "paper_2512_02175_amd", "libmetricgraph.so")):
        pytest.skip("the library is not built")
    so = host_stub.build(tmp_path_factory.mktemp("stub"))
    return lambda code, **env: host_stub.run(so, code, **env)


def test_streaming_is_set_up_when_the_call_returns(stub):
    """A batch may run the set on another stream than its own: the cleared
    counters and the table of edges are in place when the call returns."""
    stub("""
G = B.mg_graph_create(workloads.star_graph(5))
st = C.c_void_p(0x77)
p = B.mg_particles_init(G, 100, 2, precision=1, stream=st)
log()
B.mg_observe_histogram(p, 8, 2)
l = log()
last = max(i for i, x in enumerate(l) if "k_obs_edges" in x or x.startswith("memset"))
assert any(x == "sync stream=0x77" or x == "sync_device" for x in l[last + 1:]), l
""")
