"""Queues of very many nodes: the lists that they go through are sized by the nodes that use
them, and workgroup-path nodes beyond one slice are taken in further ones, alone and in a
batch, with the oracle's bits."""
import sys

import numpy as np
import pytest

import graphgen as G

pytestmark = pytest.mark.gpu

ENTRY, SMALL, GROUP = 12, 64, 1024     # bytes of a list entry, entries per node of two paths
SLICE = 65536                          # workgroup-path nodes per slice


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


def bits(v):
    return np.asarray(v, np.float64).view(np.int64)


def same(h, o):
    for u, v in zip(h.memberships() + (h.in_counts(),), o.memberships() + (o.in_counts(),)):
        assert np.array_equal(u, v)


def near_graph(n, d, seed):
    rng = np.random.default_rng(seed)
    a = np.repeat(np.arange(n), d // 2)
    return G.Graph(n, a.astype(np.int64), ((a + rng.integers(1, 3 * d, a.size)) % n).astype(np.int64))


def loaded(lf, g, opts):
    import torch
    h = lf.Handle(0)
    for k, v in opts.items():
        h.lf_set_option(k, v)
    return h.load_graph(g.n, torch.from_numpy(g.src).cuda(), torch.from_numpy(g.dst).cuda()).init_communities()


def test_one_queue_reserves_no_unused_lists(lf):
    """Small nodes of a queue that is scored without lists take no list memory."""
    g = near_graph(140_000, 8, 1)
    peak = {}
    for q in (64, g.n):
        h = loaded(lf, g, {})
        h.run_iterations(q, 0.0, 2)
        peak[q] = h.lf_get_memory()[1]
        h.close()
    say("peaks", peak)
    assert peak[g.n] - peak[64] < g.n * SMALL * ENTRY


@pytest.mark.parametrize("n", [SLICE, SLICE + 1, 2 * SLICE + 5000])
def test_workgroup_path_in_slices(lf, orc, n):
    """Nearly all nodes of one queue on the workgroup path: exactly a slice of them at most, one
    more, three slices; the lists stay those of one slice."""
    g = near_graph(n, 8, n)
    say("slices", n)
    h = loaded(lf, g, {"wave_table": 16, "med_table": 16})
    o = orc.Oracle().load_graph(g.n, g.src, g.dst).init_communities()
    ref = o.run_iterations(n, 0.0, 2)
    assert np.array_equal(bits(h.run_iterations(n, 0.0, 2)["wtilde_hist"]), bits(ref["wtilde_hist"]))
    same(h, o)
    lists = SLICE * GROUP * ENTRY
    assert h.lf_get_memory()[1] < 1.25 * lists + n * 4096
    h.close()
    h = loaded(lf, g, {"wave_table": 16, "med_table": 16})
    b = lf.Batch(0)
    m = b.add(h, n, 0.0, 2)
    while b.step() > 0:
        pass
    assert np.array_equal(bits(b.member_info(m)["wtilde_hist"]), bits(ref["wtilde_hist"]))
    b.remove(m)
    same(h, o)
    b.close()
    h.close()
    o.close()


def jobs():
    big = [j for j in G.serving_mix(n_jobs=400, seed=9) if j["n"] > 30000][0]
    return [("near", near_graph(40_000, 40, 1)), ("served", G.serving_job_graph(big)),
            ("dense", G.named_config("dense", scale=0.01)), ("small", G.named_config("tiny_sbm"))]


@pytest.mark.parametrize("which", range(4))
def test_server_reserves_for_long_queues(lf, which):
    """What the server reserves covers the peak of the same job as a member of a batch, with a
    queue of a share of the nodes and of all of them; one that only fits the budget by
    itself is still admitted."""
    name, g = jobs()[which]
    for q in (g.n // 32, g.n):
        h = loaded(lf, g, {})
        b = lf.Batch(0)
        m = b.add(h, q, 0.01, 50)
        while b.step() > 0:
            pass
        assert b.member_info(m) is not None
        b.remove(m)
        peak = h.lf_get_memory()[1]
        h.close()
        b.close()
        srv = lf.Server(0, hbm_budget=64 << 30, max_batch=4)
        srv.submit(g.n, g.src, g.dst, q, 0.01, 1)
        srv.tick()
        reserved = srv.stats()["used"]
        while srv.tick() > 0:
            pass
        srv.close()
        say(name, "queue", q, "peak", peak, "reserved", reserved)
        assert reserved >= peak
        nn = 48 * 2**20 + g.n * 768 + g.src.size * 64 + q * 256
        srv = lf.Server(0, hbm_budget=nn + nn // 8, max_batch=4)
        jid = srv.submit(g.n, g.src, g.dst, q, 0.01, 1)
        while srv.tick() > 0:
            assert srv.stats()["used"] <= srv.stats()["budget"]
        assert srv.fetch(jid) is not None
        srv.close()


@pytest.mark.parametrize("n,opts", [(16384, {}), (16385, {}), (40_001, {}), (4096, {"wave_table": 16}),
                                    (9001, {"wave_table": 16}), (21_000, {"wave_table": 32}),
                                    (9001, {"wave_table": 16, "med_table": 32})])
def test_lists_of_a_batch_in_slices(lf, orc, n, opts):
    """All nodes of a batch member in one queue, up to 4,096 blocks of small and medium nodes and
    past it, of one path or both, with workgroup nodes beside them; another member beside it."""
    say("batch slices", n, opts)
    g, g2 = near_graph(n, 8, n), near_graph(500, 8, 3)
    o = orc.Oracle().load_graph(g.n, g.src, g.dst).init_communities()
    o2 = orc.Oracle().load_graph(g2.n, g2.src, g2.dst).init_communities()
    for replay in (False, True):
        h, h2 = loaded(lf, g, opts), loaded(lf, g2, opts)
        b = lf.Batch(0)
        b.set_graph(replay)
        m, m2 = b.add(h, n, 0.0, 3), b.add(h2, 50, 0.0, 3)
        while b.step() > 0:
            pass
        if not replay:
            ref, ref2 = o.run_iterations(n, 0.0, 3), o2.run_iterations(50, 0.0, 3)
        assert np.array_equal(bits(b.member_info(m)["wtilde_hist"]), bits(ref["wtilde_hist"]))
        assert np.array_equal(bits(b.member_info(m2)["wtilde_hist"]), bits(ref2["wtilde_hist"]))
        b.close()
        same(h, o)
        same(h2, o2)
        h.close()
        h2.close()
    o.close()
    o2.close()
