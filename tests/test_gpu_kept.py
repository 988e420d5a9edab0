"""Device blocks that a handle keeps for its next requests: given back once they are more than
its present graph goes on to take, never more than its peak in all, and given up for another
handle that finds no room."""
import sys

import numpy as np
import pytest

import graphgen as G

pytestmark = pytest.mark.gpu

MB = 1 << 20


@pytest.fixture(scope="module")
def lf():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2210_03211_amd as lfmod
    lfmod.load_library()
    return lfmod


@pytest.fixture(scope="module")
def orc():
    import oracle
    oracle.build(force=False)
    return oracle


def say(*a):
    print("[case]", *a, flush=True)
    sys.stdout.flush()


def ring(n, d=6):
    a = np.repeat(np.arange(n, dtype=np.int64), d)
    return G.Graph(n, a, (a + np.tile(np.arange(1, d + 1), n)) % n)


def load(h, g):
    import torch
    return h.load_graph(g.n, torch.from_numpy(g.src).cuda(), torch.from_numpy(g.dst).cuda())


def same_run(lf, orc, h, g, q):
    o = orc.Oracle().load_graph(g.n, g.src, g.dst).init_communities()
    a, b = h.run_iterations(q, 0.0, 2), o.run_iterations(q, 0.0, 2)
    assert np.array_equal(a["wtilde_hist"].view(np.int64), b["wtilde_hist"].view(np.int64))
    for u, v in zip(h.memberships(), o.memberships()):
        assert np.array_equal(u, v)
    o.close()


def test_small_graph_after_a_large_one(lf, orc):
    """A handle that goes on to a small graph holds its scratch and that graph, not the arrays
    of the large one before."""
    large, small = ring(600_000), ring(5_000)
    h = lf.Handle(0)
    load(h, large)
    loaded = h.lf_get_memory()[0]           # scratch and CSR
    h.init_communities().run_iterations(4096, 0.0, 2)
    ran = h.lf_get_memory()[0]
    load(h, small)
    say("load", loaded, "run", ran, "small", h.lf_get_memory())
    assert h.lf_get_memory()[0] < loaded + 64 * MB + 16 * MB
    assert ran > loaded + 200 * MB          # (else there is nothing to give back)
    h.init_communities()
    assert h.lf_get_memory()[0] < loaded + 64 * MB + 16 * MB
    same_run(lf, orc, h, small, 64)
    h.close()


def test_holds_no_more_than_its_peak(lf):
    h = lf.Handle(0)
    for n in (40, 90_000, 70, 30_000, 3, 120_000, 2_000, 50_000):
        load(h, ring(n)).init_communities()
        h.run_iterations(256, 0.0, 1)
        now, peak = h.lf_get_memory()
        say("nodes", n, "now", now, "peak", peak)
        assert now <= peak
    h.close()


def test_another_handle_gets_kept_blocks(lf, orc):
    """An allocation that finds no room takes back what idle handles keep, and both go on."""
    a, b, g = lf.Handle(0), lf.Handle(0), ring(200_000)
    load(a, g).init_communities().run_iterations(4096, 0.0, 1)
    load(a, g)                              # keeps what the set-up and the run took before
    held = a.lf_get_memory()[0]
    b.lf_debug_fail_alloc(-3)
    small = ring(3_000)
    load(b, small).init_communities()
    say("kept by the other handle", held, a.lf_get_memory()[0])
    assert a.lf_get_memory()[0] < held - 50 * MB
    same_run(lf, orc, b, small, 64)
    a.init_communities()
    same_run(lf, orc, a, g, 4096)
    a.close()
    b.close()
