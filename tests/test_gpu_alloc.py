"""Allocations that fail (forced one after the other on the host): the call reports LF_ENOMEM,
and the handle goes on, at another queue size too, from the partition it still has or from a
new clustering, with the oracle's bits."""
import sys

import numpy as np
import pytest

import graphgen as G

pytestmark = pytest.mark.gpu

TABLES = {"wave_table": 16, "med_table": 16, "grp_table": 64}   # many nodes on the larger paths


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


def graph():
    """3,000 nodes of some 60 neighbours: more table-path chunks and buckets, slots and list
    entries than the first buffers hold."""
    rng = np.random.default_rng(4)
    n = 3000
    a = np.repeat(np.arange(n), 30)
    b = (a + rng.integers(1, 100, a.size)) % n
    return G.Graph(n, a.astype(np.int64), b.astype(np.int64))


def bits(v):
    return np.asarray(v, np.float64).view(np.int64)


def same(h, o):
    for u, v in zip(h.memberships() + (h.in_counts(),), o.memberships() + (o.in_counts(),)):
        assert np.array_equal(u, v)


def run_both(h, o, q, iters):
    assert np.array_equal(bits(h.run_iterations(q, 0.0, iters)["wtilde_hist"]),
                          bits(o.run_iterations(q, 0.0, iters)["wtilde_hist"]))
    same(h, o)


def loaded(lf, g):
    import torch
    h = lf.Handle(0)
    for k, v in TABLES.items():
        h.lf_set_option(k, v)
    return h.load_graph(g.n, torch.from_numpy(g.src).cuda(), torch.from_numpy(g.dst).cuda()).init_communities()


def oracle_of(lf, orc, g, h):
    """The oracle in the handle's state; the handle gets a new clustering if it has none."""
    o = orc.Oracle().load_graph(g.n, g.src, g.dst)
    try:
        off, ids = h.memberships()
    except lf.LazyFoxError as e:
        assert e.code == lf.LF_ESTATE
        h.init_communities()
        return o.init_communities(), False
    return o.init_from_memberships(off, ids, h.lf_get_graph_info()[2]), True


def failing(lf, h, nth, call):
    """Whether the nth allocation of the call failed (False: it makes fewer)."""
    h.lf_debug_fail_alloc(nth)
    try:
        call()
    except lf.LazyFoxError as e:
        assert e.code == lf.LF_ENOMEM
        return True
    finally:
        h.lf_debug_fail_alloc(0)
    return False


def test_run_after_a_failed_long_queue(lf, orc):
    g = graph()
    kept = 0
    for nth in range(1, 100):
        say("run, allocation", nth)
        h = loaded(lf, g)
        h.run_iterations(16, 0.0, 1)
        if not failing(lf, h, nth, lambda: h.run_iterations(g.n, 0.0, 2)):
            h.close()
            break
        o, has = oracle_of(lf, orc, g, h)
        kept += has
        run_both(h, o, 16, 1)
        run_both(h, o, g.n, 1)
        h.close()
        o.close()
    assert 5 < nth < 99 and kept > 5


def test_first_run_and_post_processing(lf, orc):
    g = graph()
    for nth in range(1, 100):
        say("first run, allocation", nth)
        h = loaded(lf, g)
        if not failing(lf, h, nth, lambda: h.run_iterations(64, 0.0, 2)):
            h.close()
            break
        o, _ = oracle_of(lf, orc, g, h)
        assert np.array_equal(h.postprocess()[0], o.postprocess()[0])
        run_both(h, o, 64, 2)
        h.close()
        o.close()
    assert 5 < nth < 99


def test_load_and_set_up(lf, orc):
    import torch
    g = graph()
    src, dst = torch.from_numpy(g.src).cuda(), torch.from_numpy(g.dst).cuda()
    o = orc.Oracle().load_graph(g.n, g.src, g.dst).init_communities()
    off, ids = o.memberships()
    wcc, f1 = o.exact_wcc()["wcc"], o.cover_f1(off, ids)[0]
    stages = {"load": lambda h: h.load_graph(g.n, src, dst),
              "init": lambda h: h.init_communities(),
              "warm": lambda h: h.init_from_memberships(off, ids, h.lf_get_graph_info()[2]),
              "wcc": lambda h: h.exact_wcc(),
              "f1": lambda h: h.cover_f1(off, ids)}
    for name in stages:
        for nth in range(1, 100):
            h = lf.Handle(0)
            for before in list(stages)[:list(stages).index(name)]:
                stages[before](h)
            say(name, "allocation", nth)
            fired = failing(lf, h, nth, lambda: stages[name](h))
            if name in ("load", "init", "warm"):
                for again in list(stages)[list(stages).index(name):3]:
                    stages[again](h)
            same(h, o)
            assert h.exact_wcc()["wcc"] == wcc and h.cover_f1(off, ids)[0] == f1
            h.close()
            if not fired:
                break
        assert nth < 99
    o.close()


def test_member_of_a_batch(lf, orc):
    """A member that fails leaves the others alone, and runs on once it has left the batch."""
    g, g2 = graph(), G.random_gnp(300, 0.1, 5)
    o2 = orc.Oracle().load_graph(g2.n, g2.src, g2.dst).init_communities()
    want = bits(o2.run_iterations(16, 0.0, 3)["wtilde_hist"])
    o2.close()
    for nth in range(1, 100):
        say("batch, allocation", nth)
        h, h2 = loaded(lf, g), loaded(lf, g2)
        b = lf.Batch(0)
        m, m2 = b.add(h, 600, 0.0, 3), b.add(h2, 16, 0.0, 3)
        h.lf_debug_fail_alloc(nth)
        while b.step() > 0:
            pass
        h.lf_debug_fail_alloc(0)
        assert np.array_equal(bits(b.member_info(m2)["wtilde_hist"]), want)
        try:
            info = b.member_info(m)
        except lf.LazyFoxError as e:
            assert e.code == lf.LF_ENOMEM
            info = None
        b.remove(m)
        b.close()
        if info is None:
            o, _ = oracle_of(lf, orc, g, h)
            run_both(h, o, 600, 1)
            o.close()
        h.close()
        h2.close()
        if info is not None:
            break
    assert 5 < nth < 99
