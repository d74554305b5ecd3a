"""Histograms of more bins than LDS holds where many particles share a few bins:
all in one, in several of one bucket of the kernel's table (more than its two
entries), in a later part of the set, among even ones; counts beyond a staging
block (16 MiB) in host memory.  The counts are those of the positions."""
import numpy as np
import pytest

import workloads

pytestmark = pytest.mark.gpu

EDGES, NB = 300, 200


def _bins(mode, n, rng):
    bins = EDGES * NB
    bucket = (np.arange(bins, dtype=np.uint64) * 2654435769 % 2**32) >> 22
    one = np.flatnonzero(bucket == bucket[12_345])          # about 58 bins of one bucket
    b = rng.integers(0, bins, n)
    if mode == "one":
        b[:] = 12_345
    elif mode == "bucket":
        b = rng.choice(one[:6], n)
    elif mode == "late":
        b[n // 2:] = 777
    elif mode == "mixed":
        hot = rng.random(n) < 0.7
        b[hot] = rng.choice(one[:40], hot.sum())
    return b


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("mode", ["even", "one", "bucket", "late", "mixed"])
@pytest.mark.parametrize("n", [1, 3, 1027, 70_001, 1_200_003])
def test_gathered_particles(prec, mode, n):
    import torch
    from paper_2512_02175_amd import binding as B
    rng = np.random.default_rng(n)
    g = workloads.star_graph(EDGES)
    G = B.mg_graph_create(g)
    b = _bins(mode, n, rng)
    p = B.mg_particles_init(G, n, B.MG_INIT_EXPLICIT, edge=(b // NB).astype(np.int32),
                            pos=(b % NB + 0.5) / NB, precision=prec)
    if n > 3:                                   # remove every fifth particle
        img = B.mg_particles_save(p)
        ef = img[96:96 + 4 * n].view(np.uint32)
        ef[::5] |= np.uint32(1 << 31)
        p = B.mg_particles_load(G, img)
        b = b[np.arange(n) % 5 != 0]
    want = np.bincount(b, minlength=EDGES * NB)
    assert np.array_equal(B.mg_histogram(p, NB).ravel().astype(np.int64), want)
    out = torch.full((EDGES * NB,), 5, dtype=torch.int64, device="cuda")
    B.mg_histogram(p, NB, out)
    assert np.array_equal(out.cpu().numpy(), want)


def test_more_counters_than_a_staging_block():
    import torch  # noqa: F401
    from paper_2512_02175_amd import binding as B
    nb = 7001
    assert EDGES * nb * 8 > 16 << 20
    G = B.mg_graph_create(workloads.star_graph(EDGES))
    p = B.mg_particles_init(G, 300_007, B.MG_INIT_UNIFORM_LENGTH, init_seed=1)
    r = B.mg_particles_read(p)
    b = np.minimum(np.floor(r["x"] * (nb / 1.0)), nb - 1).astype(np.int64)
    want = np.bincount(r["edge"].astype(np.int64) * nb + b, minlength=EDGES * nb)
    assert np.array_equal(B.mg_histogram(p, nb).ravel().astype(np.int64), want)
    off = (np.arange(EDGES + 1) * nb).astype(np.int32)
    edge_up = np.arange(1, nb + 1) / nb
    got = B.mg_histogram_csr(p, off, np.tile(edge_up, EDGES))
    k = np.minimum(np.searchsorted(edge_up, r["x"]), nb - 1)
    want = np.bincount(r["edge"].astype(np.int64) * nb + k, minlength=EDGES * nb)
    assert np.array_equal(got.astype(np.int64), want)
