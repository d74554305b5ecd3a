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


@pytest.mark.parametrize("name", ["hipHostMalloc", "hipMalloc"])
def test_readback_without_staging_memory(stub, name):
    """No pinned (or no device) memory for a staging block: every call that read
    its results without allocating any still returns them."""
    stub(f"name = {name!r}" + """
def results(p, trace):
    r = B.mg_particles_read(p, 3, 9000, trace=trace)
    return ([r[k] for k in r] + [B.mg_particles_read(p)["x"]] + list(B.mg_exit_counts(p))
            + list(B.mg_observed_histogram(p)))
G = B.mg_graph_create(workloads.star_graph(5, [0.5, 1.0, 1.5, 2.0, 2.5]))
for prec in (0, 1):
    for trace in (False, True):
        p = B.mg_particles_init(G, 10_001, 2, precision=prec, trace=trace)
        img = B.mg_particles_save(p)
        # states of every kind: edges, both reference ends, removed particles
        i = np.arange(10_001)
        ef = (i % 5).astype(np.uint32)
        if prec:
            ef |= ((i // 5) % 2).astype(np.uint32) << 30
        ef |= (i % 7 == 0).astype(np.uint32) << 31
        img[96:96 + 4 * i.size] = ef.view(np.uint8)
        at = 96 + -(-4 * i.size // 8) * 8
        x = (0.4 * i / i.size)
        x = x.astype(np.float32) if prec else x
        img[at:at + 8 * i.size] = (np.stack([x, x * np.float32(1e-9)], 1).copy().view(np.uint8).ravel()
                                   if prec else x.view(np.uint8))
        p = B.mg_particles_load(G, img)
        B.mg_observe_histogram(p, 7, 3)
        want = results(p, trace)
        for q in (p, None):
            if q is None:                     # and with no block kept from before
                del p
                G2 = G; B.mg_graph_destroy(G)
                G = B.mg_graph_create(workloads.star_graph(5, [0.5, 1.0, 1.5, 2.0, 2.5]))
                q = B.mg_particles_load(G, img)
                B.mg_observe_histogram(q, 7, 3)
            fail(name)
            got = results(q, trace)
            fail("")
            assert all(np.array_equal(a, b) for a, b in zip(want, got)), (prec, trace)
        del q
""")


def test_a_readback_takes_no_device_memory(stub):
    stub("""
G = B.mg_graph_create(workloads.star_graph(5))
p = B.mg_particles_init(G, 100_001, 2, precision=1)
B.mg_observe_histogram(p, 7, 3)
log()
B.mg_particles_read(p), B.mg_exit_counts(p), B.mg_observed_histogram(p)
out = C.c_void_p(S.stub_device_block(8 * 50))
assert L.mg_histogram(p.handle, 10, out, 50) == 0
assert not [x for x in log() if x.startswith("malloc")]
B.mg_histogram(p, 10)                       # its counters
assert len([x for x in log() if x.startswith("malloc")]) == 1
B.mg_histogram(p, 10)                       # kept
assert not [x for x in log() if "malloc" in x]
""")


@pytest.mark.parametrize("call", ["histogram", "csr", "exits", "observed", "read"])
def test_a_block_is_given_back_without_work_on_it(stub, call):
    """After a failed launch the call waits for what it had queued before its
    staging blocks go back to the pool."""
    stub(f"call = {call!r}" + """
E = 5000
G = B.mg_graph_create(workloads.star_graph(E))
st = C.c_void_p(0x77)
p = B.mg_particles_init(G, 700_001, 2, stream=st)
B.mg_observe_histogram(p, 300, 3)           # 12 MB of counters: several pieces
off = (np.arange(E + 1) * 4).astype(np.int32)
up = np.tile([0.25, 0.5, 0.75, 1.0], E)
f = {"histogram": lambda: B.mg_histogram(p, 100), "csr": lambda: B.mg_histogram_csr(p, off, up),
     "exits": lambda: B.mg_exit_counts(p), "observed": lambda: B.mg_observed_histogram(p),
     "read": lambda: B.mg_particles_read(p)}[call]
log()
f()
n = len([x for x in log() if x.startswith("launch")])
for k in range(n):
    fail("hipLaunchKernel", skip=k, count=1)
    try:
        f()
        assert False
    except B.MgError as e:
        assert e.status == B.MG_EDEVICE
    l = log()
    last = max([i for i, x in enumerate(l) if x.startswith(("launch ", "copy "))], default=-1)
    assert last < 0 or "sync stream=0x77" in l[last + 1:], (k, l)
""")


def test_readback_on_the_sets_device(stub):
    """With another device current, the results of a set come through kernels,
    blocks and events of its own device, and the current one is restored."""
    stub("""
E = 5000
S.stub_device(1)
g = workloads.star_graph(E)
G = B.mg_graph_create(g)
p = B.mg_particles_init(G, 700_001, 2)
B.mg_observe_histogram(p, 300, 3)
S.stub_device(0)
off = (np.arange(E + 1) * 4).astype(np.int32)
up = np.tile([0.25, 0.5, 0.75, 1.0], E)
log()
for f in (lambda: B.mg_particles_read(p), lambda: B.mg_exit_counts(p),
          lambda: B.mg_observed_histogram(p), lambda: B.mg_histogram(p, 100),
          lambda: B.mg_histogram_csr(p, off, up)):
    f()
    l = log()
    seen = [x for x in l if "device=" in x]
    assert seen and all("device=1" in x for x in seen), l
    q = B.mg_particles_init(G, 10, 2)       # still the caller's
    assert any(x.startswith("malloc") and "device=0" in x for x in log())
""")


def test_no_probe_inside_a_capture(stub):
    """A set that has run may be captured: the call only launches, also where its
    graph has become due for tuning or a tuning file is named."""
    code = """
G = B.mg_graph_create(workloads.star_graph(5))
p = B.mg_particles_init(G, 100, 2, precision=1)
%s
S.stub_capture(1)
log()
for dt in (1e-2, 1e-2, 1e-3):
    B.mg_simulate(p, 10, dt, 1)
    l = log()
    assert all(x.startswith("launch") for x in l) and steps(l) and not any("probe" in x for x in l), l
S.stub_capture(0)
B.mg_simulate(p, 10, 1e-2, 1)
assert any("probe" in x for x in log())
S.stub_capture(1)                           # a known result is taken
q = B.mg_particles_init(G, 100, 2, precision=1)
log()
B.mg_simulate(q, 10, 1e-2, 1)
assert steps(log())[0][2]["kernel"] == 0    # (the first of equal probes)
"""
    stub(code % f"B.mg_simulate(p, {20 * 14336 - 1}, 1e-2, 1)")
    stub(code % "", MG_TUNE_CACHE="/nonexistent/tune")


def test_a_tuned_choice_holds_at_its_time_step(stub):
    """A set tuned at one dt runs the default at another (one particle per lane
    where nearly every step is spent at vertices), not the tuned choice, until
    it is tuned there; and the tuned choice again at its own."""
    stub("""
def ran(p, dt):
    log()
    B.mg_simulate(p, 5, dt, 1)
    a = steps(log())[-1][2]
    return a["kernel"], a["idle"]
n = 1_000_000                               # full pools: idle as chosen
G = B.mg_graph_create(workloads.star_graph(5))
p = B.mg_particles_init(G, n, 2, precision=1)
assert ran(p, 1e-2) == (3, 16)
S.stub_fast(0)                              # lanes
B.mg_autotune(p, 1e-2)
assert ran(p, 1e-2)[0] == 0
assert ran(p, 1e-3) == (3, 16)
assert ran(p, 1e-2)[0] == 0
S.stub_fast(5)                              # pools of 256 at 8 idle lanes
B.mg_autotune(p, 1e-3)
assert ran(p, 1e-3) == (2, 8)
assert ran(p, 2e-3) == (3, 16)
assert ran(p, 1e-2)[0] == 0                 # (known from the graph)
# strong drift to the centre
G = B.mg_graph_create(workloads.paper_star5("linear", np.inf))
p = B.mg_particles_init(G, n, 1, vertex=0, precision=1)
S.stub_fast(7)                              # MG_SCHED_POOLS_W8 at 8 idle lanes
B.mg_autotune(p, 1e-4)
assert ran(p, 1e-4) == (3, 8)
assert ran(p, 2e-2)[0] == 0
assert ran(p, 1e-3) == (3, 16)
""")


def test_batches_of_tuned_and_untuned_sets(stub):
    """Sets that ran on the automatic schedule share a batch whether or not each
    has run far enough to be tuned; what differed in schedule still does."""
    stub("""
G = [B.mg_graph_create(workloads.star_graph(5 + i)) for i in range(2)]
def make(i, **kw):
    return B.mg_particles_init(G[i], 1000, 2, precision=1, **kw)
far, near, new = make(0), make(1), make(1)
lanes, pools = make(1, schedule=B.MG_SCHED_LANES), make(1, schedule=B.MG_SCHED_POOLS)
B.mg_simulate(near, 3, 1e-2, 1)
B.mg_simulate(far, 3, 1e-2, 1)
B.mg_batch_create([near, far, new])         # none tuned: one default
S.stub_fast(5)                              # pools of 256 at 8 idle lanes
B.mg_autotune(far, 1e-2)
def refused(*sets):
    try:
        B.mg_batch_create(list(sets))
    except B.MgError as e:
        return e.status == B.MG_EINVAL and "schedule" in str(e)
    return False
for sets in ([near, far], [far, near]):
    b = B.mg_batch_create(sets)
    log()
    B.mg_batch_simulate(b, 4, 1e-2, 1)
    (k, _, a), = steps(log())
    assert "k_pool32_batch" in k and "Li256E" in k and a["kernel"] == 2 and a["idle"] == 8, (k, a)
B.mg_autotune(lanes, 1e-2)                  # a fixed schedule stays what it is
assert refused(far, new) and refused(far, lanes) and refused(near, lanes) and refused(lanes, near)
assert refused(far, pools) and refused(near, pools, far)
B.mg_batch_create([lanes, make(0, schedule=B.MG_SCHED_LANES)])
""")


def test_when_an_automatic_set_is_tuned(stub):
    """By the call that brings the work of a graph's untuned sets at a dt to 20
    times the probes' particle-steps: short calls together, or one long one."""
    stub("""
def probed(p, k, dt=1e-2):
    log()
    B.mg_simulate(p, k, dt, 1)
    return any("probe" in x for x in log())
due = 20 * (10 * 1024 + 2 * 2048)
def new(n=100, G=None, **kw):
    return B.mg_particles_init(G or B.mg_graph_create(workloads.star_graph(5)), n, 2,
                               precision=1, **kw)
p = new()
assert not probed(p, due - 1) and probed(p, 1) and not probed(p, due)
assert probed(new(), due)                   # one call
p = new()                                   # each dt by itself
assert not probed(p, due - 1, 1e-2) and not probed(p, due - 1, 1e-3)
assert probed(p, 1, 1e-3) and probed(p, 1, 1e-2)
G = B.mg_graph_create(workloads.star_graph(5))
p, q = new(100, G), new(50, G)              # the sets of a graph together
assert not probed(p, due // 4) and not probed(q, 1) and probed(q, due // 2)
assert not probed(p, 1)                     # known
assert not probed(new(schedule=B.MG_SCHED_POOLS_W8), due)
assert not probed(new(100, B.mg_graph_create(workloads.double_well_star(3))), due)
""")


def test_untuned_kernel_by_expected_hits(stub):
    """Lanes where a step is expected to make 0.45 of its hits, pools below: the
    sides that were measured faster, for drifts on every edge, drifts on some,
    short edges, one long edge among short ones, and other split caps."""
    stub("""
def kernel(g, dt=1e-2, M=8):
    G = B.mg_graph_create(g)
    p = B.mg_particles_init(G, 1000, 1, vertex=0, precision=1, max_splits=M)
    out = []
    for d in (dt, 1e-9, dt):
        log()
        B.mg_simulate(p, 5, d, 1)
        out.append(steps(log())[-1][2]["kernel"])
    assert out[0] == out[2] and out[1] == 3
    return out[0]
star = workloads.star_graph
for E in (3, 64):
    for r, k in ((0.85, 3), (1.0, 3), (1.5, 3), (2.1, 0), (3.0, 0), (6.0, 0)):
        assert kernel(star(E, 2.0, -10 * r)) == k, r
        g = star(E, 0.5, 10 * r)                     # towards the leaves
        assert kernel(g) == k, r
    for q, k in ((1, 3), (3, 3), (5, 0), (16, 0)):
        assert kernel(star(E, 0.1 / q)) == k, q
for q in (2, 4, 8):
    assert kernel(star(5, np.where(np.arange(5) == 0, 1.0, 0.1 / q))) == 3
assert kernel(star(64, 0.1 / 4 * np.random.default_rng(3).uniform(0.3, 1.0, 64))) == 0
lin = workloads.paper_star5("linear", np.inf)
assert [kernel(lin, d) for d in (1e-3, 5e-3, 7.3e-3, 2e-2)] == [3, 3, 0, 0]
assert kernel(star(5, 0.1 / 8), M=32) == 3 and kernel(star(5, 2.0, -60.0), M=32) == 0
assert kernel(star(5, 0.1), M=1) == 0 and kernel(star(5, 1.0), M=1) == 3
# a semi-infinite edge without a drift back, and general coefficients
assert kernel(star(3, [np.inf, 0.001, 0.001], bin_span=[1.0, 0.001, 0.001])) == 3
assert kernel(workloads.double_well_star(3), 1.0) == 3
""")


def test_refill_follows_the_launch_plan(stub):
    """Lanes that end a window: 16 of MG_SCHED_POOLS_W8 where the launch stages
    the graph's tables in LDS or diffusion makes a hit in every hundred steps,
    else 8 in FP32; 16 in every group of a batch."""
    stub("""
small, large = (B.mg_graph_create(workloads.star_graph(E)) for E in (20, 2000))
longer = B.mg_graph_create(workloads.star_graph(2000, np.linspace(2.0, 6.0, 2000), sigma=0.5))
endless = B.mg_graph_create(workloads.star_graph(2000, np.inf, bin_span=1.0))
def staged(kernel):                         # <trace, exits in LDS, tables in LDS, ...>
    return re.search(r"(?:k_pool|k_step)\\w*?I((?:Lb[01]E)+)", kernel)[1][10] == "1"
n = 1_000_000
# 0.8 sigma sqrt(dt) / L hits: at 1.5e-4 of the unit star 0.98 %, at 1.6e-4 1.01 %
for prec, sched, G, dt, want in (
        (1, 4, small, 1e-5, 16), (1, 4, large, 1e-5, 8), (1, 4, large, 1.5e-4, 8),
        (1, 4, large, 1.6e-4, 16), (1, 4, large, 1e-2, 16), (1, 4, longer, 9.8e-3, 8),
        (1, 4, longer, 1.02e-2, 16), (1, 4, endless, 1.0, 8), (1, 2, small, 1e-2, 8),
        (1, 2, large, 1e-2, 8), (0, 4, small, 1e-5, 16), (0, 4, large, 1e-5, 16)):
    p = B.mg_particles_init(G, n, 1 if G is endless else 2, precision=prec,
                            schedule=sched)
    log()
    B.mg_simulate(p, 5, dt, 1)
    (k, _, a), = steps(log())
    assert a["refill"] == want and staged(k) == (G is small), (k, a)
for prec in (1, 0):
    sets = [B.mg_particles_init(G, n, 2, precision=prec, schedule=4, graph_tag=i)
            for i, G in enumerate((small, large))]
    S.stub_blocks_per_cu(8)
    b = B.mg_batch_create(sets)
    log()
    B.mg_batch_simulate(b, 5, 1e-2, 1)
    l = steps(log())
    assert len({staged(k) for k, _, _ in l}) == 2, l
    for k, _, a in l:
        assert a["refill"] == 16, (k, a)
""")


def test_reservations_leave_every_simd_several(stub):
    """Ids that a wave reserves at a time: at most an eighth of a SIMD's share of
    the set (1024 SIMDs here), a sixteenth from 96 steps on, or a pool's worth."""
    stub("""
G = B.mg_graph_create(workloads.star_graph(20))
W = B.mg_graph_create(workloads.wentzell_star())
for prec, n, k, cap, want in ((1, 2_000_000, 95, 128, 240), (1, 2_000_000, 96, 128, 128),
                              (1, 3_000_000, 60, 128, 352), (1, 3_000_000, 100, 128, 176),
                              (1, 1_000_000, 60, 128, 128), (1, 300_000, 400, 64, 64),
                              (1, 10_000, 400, 16, 16), (1, 20_000_000, 4000, 128, 64),
                              (0, 2_000_000, 60, 128, 240), (0, 2_000_000, 400, 128, 128)):
    p = B.mg_particles_init(G, n, 2, precision=prec)
    log()
    B.mg_simulate(p, k, 1e-3, 1)
    (_, _, a), = steps(log())
    assert a["pool_cap"] == cap and a["claim"] == want, (n, k, a)
for g, n, cap in ((G, 393_216, 64), (G, 393_217, 128), (W, 262_144, 64), (W, 262_145, 128)):
    p = B.mg_particles_init(g, n, 2, precision=1)   # (waves that are resident)
    log()
    B.mg_simulate(p, 100, 1e-3, 1)
    (_, _, a), = steps(log())
    assert a["pool_cap"] == cap and a["claim"] == cap, (n, a)
""")


def test_equal_candidates_are_probed_once(stub):
    """On a graph whose tables are not staged and whose hits are few
    MG_SCHED_POOLS_W8 launches what MG_SCHED_POOLS launches: seven probes, and
    the times of the other three are those of their equals."""
    stub("""
for E, dt, launches in ((20, 1e-5, 10), (2000, 1e-5, 7), (2000, 1e-2, 10)):
    p = B.mg_particles_init(B.mg_graph_create(workloads.star_graph(E)), 1_000_000, 2, precision=1)
    log()
    S.stub_fast(3)                          # pools of 128 at 16 idle lanes
    t = B.mg_autotune(p, dt)
    l = [(re.search(r"I.*E", k)[0], a["idle"], a["refill"], a["nsteps"]) for k, _, a in steps(log())
         if a["kernel"]]
    assert len([x for x in l if x[3] == 1024]) - 2 == launches - 1, l   # (2: the launch length)
    assert t["schedule"] == B.MG_SCHED_POOLS and t["idle_trigger"] == 16 and t["n_probes"] == 10
    assert t["probe_ms"][3] == 0.5 and (t["probe_ms"][8] == 0.5) == (launches == 7)
    fail("hipMemcpyAsync")                  # a probe that cannot run
    p = B.mg_particles_init(B.mg_graph_create(workloads.star_graph(E)), 100, 2, precision=1)
    try:
        B.mg_autotune(p, 1e-2)
        assert False
    except B.MgError as e:
        assert e.status == B.MG_EDEVICE
    fail("")
""")


def test_exit_counters_stay_in_lds(stub):
    """The most exit slots counted in LDS are those that fit in 64 KiB beside the
    four pools of a block (44 bytes a particle in FP64, 40 in FP32), whatever the
    FP64 tables and the snapshot counts of a streaming set need beside them; the
    lane schedule counts 16384."""
    stub("""
def exits_in_lds(kernel):   # <trace, exits, ...>; the lane kernels <fp64, trace, exits, ...>
    f = re.findall(r"Lb([01])E", re.search(r"I((?:Lb[01]E)+)", kernel)[1])
    return f[2 if "k_step" in kernel or "7k_batch" in kernel else 1] == "1"
def counted(edges, prec, sched, obs, batch):
    p = B.mg_particles_init(B.mg_graph_create(workloads.star_graph(edges)), 1000, 2,
                            precision=prec, schedule=sched)
    if obs:
        B.mg_observe_histogram(p, 4, 5)
    log()
    if batch:
        B.mg_batch_simulate(B.mg_batch_create([p]), 5, 1e-2, 1)
    else:
        B.mg_simulate(p, 5, 1e-2, 1)
    (k, _, _), = steps(log())
    return exits_in_lds(k)
KB64 = 65536
for prec, sched, most in ((0, 1, 16384), (1, 1, 16384), (0, 4, (KB64 - 4 * 128 * 44) // 4),
                          (1, 4, (KB64 - 4 * 128 * 40) // 4), (1, 2, (KB64 - 4 * 128 * 40) // 4),
                          (1, 3, (KB64 - 4 * 256 * 40) // 4)):
    for obs in (False, True):
        for batch in (False, True):
            at = [counted(most // 2 + d, prec, sched, obs, batch) for d in (0, 1)]
            assert at == [True, False], (prec, sched, obs, batch, at)
""")


def test_blocks_of_a_csr_histogram(stub):
    """At least a block per CU (or a turn of four particles per thread) where each
    block counts in LDS; never more than the uniform histogram's 512."""
    stub("""
for E, nb, n, want in ((64, 256, 1_000_000, 256), (64, 256, 10_000_000, 256), (5, 100, 10_000_000, 512),
                       (64, 256, 30_000, 30), (5, 2, 1, 1), (64, 512, 300_000, 256)):
    p = B.mg_particles_init(B.mg_graph_create(workloads.star_graph(E)), n, 2, precision=1)
    log()
    B.mg_histogram_csr(p, (np.arange(E + 1) * nb).astype(np.int32),
                       np.tile(np.arange(1, nb + 1) / nb, E))
    (grid,) = [int(re.search(r"grid=(\\d+)", x)[1]) for x in log() if "k_hist_csr" in x]
    assert grid == want, (E, nb, n, grid)
""")


def test_no_exception_leaves_a_step_call(stub):
    """Host memory that runs out inside mg_simulate or mg_batch_simulate is an
    error code or costs nothing, not an exception through the C entry."""
    out = stub("""
G = B.mg_graph_create(workloads.star_graph(5))
p = B.mg_particles_init(G, 100, 2, precision=1)
fail("new", 0, 1)
for dt in (1e-2, 1e-3, 1e-4):
    assert L.mg_simulate(p.handle, 5, C.c_double(dt), C.c_uint64(1)) == B.MG_OK
fail("")
sets = [B.mg_particles_init(B.mg_graph_create(workloads.star_graph(E)), 1000, 2, precision=1)
        for E in (5, 2000)]
S.stub_blocks_per_cu(8)
b = B.mg_batch_create(sets)
k = 0
while True:
    fail("new", k, 1)
    r = L.mg_batch_simulate(b.handle, 5, C.c_double(1e-2), C.c_uint64(1))
    if r == B.MG_OK:
        break
    assert r == B.MG_ENOMEM and B.mg_particles_step(sets[0]) == 0, r
    k += 1
fail("")
assert B.mg_particles_step(sets[0]) == 5
print(k)
""")
    assert int(out) > 0
