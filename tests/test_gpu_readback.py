"""Readback through staged pieces: ranges that start and end anywhere, sets of
several pieces, and several threads reading their own sets at once."""
import threading

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
@pytest.mark.parametrize("trace", [False, True])
def test_pieces_equal_the_image(B, prec, trace):
    g, _ = workloads.config2()
    G = B.mg_graph_create(g)
    n = 700_001
    p = B.mg_particles_init(G, n, B.MG_INIT_UNIFORM_LENGTH, init_seed=4, precision=prec,
                            trace=trace)
    B.mg_simulate(p, 6, 1e-2, 5)
    whole = B.mg_particles_read(p, trace=trace)
    # the state as the checkpoint image holds it
    img = B.mg_particles_save(p)
    at = 96
    ef = img[at:at + 4 * n].view(np.uint32)
    at += -(-4 * n // 8) * 8
    pos = img[at:at + 8 * n]
    assert np.array_equal(whole["edge"], (ef & 0x3FFFFFFF).astype(np.int32))
    if prec == 0:
        x = pos.view(np.float64)
    else:
        y = pos.view(np.float32).reshape(n, 2).astype(np.float64).sum(axis=1)
        x = np.where(ef & 0x40000000, g.length[whole["edge"]] - y, y)
    assert np.array_equal(whole["x"], x)
    for first, count in ((0, 1), (699_999, 2), (1, 163_841), (12_345, 650_001)):
        part = B.mg_particles_read(p, first, count, trace=trace)
        for k, v in part.items():
            assert np.array_equal(v, whole[k][first:first + count]), (k, first, count)


def test_threads_read_their_own_sets(B):
    g = workloads.star_graph(300)
    G = B.mg_graph_create(g)
    sets = [B.mg_particles_init(G, 50_000 + i, B.MG_INIT_UNIFORM_LENGTH, init_seed=i,
                                precision=i % 2) for i in range(6)]
    want = [(B.mg_histogram(p, 64), B.mg_exit_counts(p), B.mg_particles_read(p)) for p in sets]
    bad = []

    def work(i):
        for _ in range(20):
            h, ex, r = (B.mg_histogram(sets[i], 64), B.mg_exit_counts(sets[i]),
                        B.mg_particles_read(sets[i]))
            same = np.array_equal(h, want[i][0]) and all(
                np.array_equal(a, b) for a, b in zip(ex, want[i][1])) and all(
                np.array_equal(r[k], want[i][2][k]) for k in r)
            if not same:
                bad.append(i)
    ts = [threading.Thread(target=work, args=(i,)) for i in range(len(sets))]
    for t in ts:
        t.start()
    for t in ts:
        t.join()
    assert not bad
