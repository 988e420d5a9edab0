"""Queue kernels at the sizes where their forms change: batches with 1 to 130 members (the
first-block entries are searched 64 at a time); queues scored in one launch without lists; parts
of communities at one wave, one part and past it, with joiners beyond the plan; nodes with more
memberships than a line and than a byte hold.  Runs equal the oracle's bit for bit."""
import sys

import numpy as np
import pytest

import graphgen as G

pytestmark = pytest.mark.gpu


def say(*a):
    print("[case]", *a, flush=True)
    sys.stdout.flush()


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


def loaded(lf, g):
    import torch
    h = lf.Handle(0)
    h.load_graph(g.n, torch.from_numpy(g.src).cuda(), torch.from_numpy(g.dst).cuda())
    return h


def same_state(h, o):
    for u, v in zip(h.memberships() + (h.in_counts(),), o.memberships() + (o.in_counts(),)):
        assert np.array_equal(u, v)


def same_hist(a, b):
    assert np.array_equal(np.asarray(a["wtilde_hist"]).view(np.int64), np.asarray(b["wtilde_hist"]).view(np.int64))


@pytest.mark.parametrize("members,replay", [(1, None), (61, None), (62, None), (63, None), (64, None), (65, True),
                                            (130, None)])
def test_batch_sizes(lf, orc, members, replay):
    say("batch of", members, "replay", replay)
    b = lf.Batch(0)
    if replay is not None:
        b.set_graph(replay)
    gs = [G.random_gnp(20 + 3 * (i % 17), 0.3, i) for i in range(members)]
    hs = [loaded(lf, g).init_communities() for g in gs]
    ids = [b.add(h, 8, 0.0, 3) for h in hs]
    while b.step() > 0:
        pass
    for g, h, m in zip(gs, hs, ids):
        info = b.member_info(m)
        b.remove(m)
        o = orc.Oracle()
        o.load_graph(g.n, g.src, g.dst)
        o.init_communities()
        same_hist(info, o.run_iterations(8, 0.0, 3))
        same_state(h, o)
        h.close()
        o.close()
    b.close()


def cover(lists):
    off = np.zeros(len(lists) + 1, np.int64)
    off[1:] = np.cumsum([len(p) for p in lists])
    return off, np.concatenate([np.asarray(p, np.int32) for p in lists]).astype(np.int32)


def warm_run(lf, orc, g, lists, K, q, iters, opts=None):
    off, ids = cover(lists)
    h = lf.Handle(0)
    for k, v in (opts or {}).items():
        h.lf_set_option(k, v)
    import torch
    h.load_graph(g.n, torch.from_numpy(g.src).cuda(), torch.from_numpy(g.dst).cuda())
    h.init_from_memberships(off, ids, K)
    o = orc.Oracle()
    o.load_graph(g.n, g.src, g.dst)
    o.init_from_memberships(off, ids, K)
    same_hist(h.run_iterations(q, 0.0, iters), o.run_iterations(q, 0.0, iters))
    same_state(h, o)
    o.close()
    h.close()


@pytest.mark.parametrize("size,q", [(64, 16), (65, 16), (511, 7), (512, 64), (513, 64), (1100, 300), (1100, 1600)])
def test_community_parts(lf, orc, size, q):
    """Communities of one size, dense enough inside that members stay and others join."""
    say("parts", size, q)
    rng = np.random.default_rng(size)
    n = 3 * size if size > 200 else 20 * size
    home = np.arange(n) // size
    a = rng.integers(0, n, 12 * n)
    inside = home[a] * size + rng.integers(0, size, a.size)
    b = np.where(rng.random(a.size) < 0.8, np.minimum(inside, n - 1), rng.integers(0, n, a.size))
    g = G.Graph(n, a.astype(np.int64), b.astype(np.int64))
    K = int(home.max()) + 2
    lists = [[int(home[x])] if rng.random() < 0.9 else [K - 1] for x in range(n)]
    warm_run(lf, orc, g, lists, K, q, 3)
    warm_run(lf, orc, g, lists, K, q, 2, {"refresh_blocks": 1})


@pytest.mark.parametrize("most", [5, 6, 7, 13, 254, 255, 300])
def test_many_memberships(lf, orc, most):
    """Nodes with up to `most` memberships, inline and beyond the line, some of which they
    leave while their neighbours read them, over several iterations."""
    say("memberships", most)
    rng = np.random.default_rng(most)
    g = G.random_gnp(300, 0.08, most)
    K = 2 * most + 20
    count = np.where(rng.random(g.n) < 0.1, most, rng.integers(1, 4, g.n))
    count[rng.random(g.n) < 0.1] = max(1, most - 1)
    lists = [rng.choice(K, c, replace=False) for c in count]
    warm_run(lf, orc, g, lists, K, 32, 4)


@pytest.mark.parametrize("n,d", [(17000, 5), (9000, 60)])
def test_one_queue_without_lists(lf, orc, n, d):
    """All nodes in one queue, enough blocks that it is gathered and scored in one launch."""
    say("whole", n, d)
    rng = np.random.default_rng(n)
    a = np.repeat(np.arange(n), d // 2 + 1)
    b = (a + rng.integers(1, 3 * d, a.size)) % n
    g = G.Graph(n, a.astype(np.int64), b.astype(np.int64))
    h = loaded(lf, g).init_communities()
    o = orc.Oracle()
    o.load_graph(g.n, g.src, g.dst)
    o.init_communities()
    same_hist(h.run_iterations(n, 0.0, 3), o.run_iterations(n, 0.0, 3))
    same_state(h, o)
    h.close()
    o.close()


@pytest.mark.parametrize("n,opts", [(9000, {"wave_table": 16, "med_table": 16, "grp_table": 16}),
                                    (7000, {"wave_table": 16, "med_table": 64, "grp_table": 256})])
def test_split_launch_of_larger_nodes(lf, orc, n, opts):
    """More buckets in a queue than one launch for all larger nodes takes, without and with
    workgroup-path nodes beside them."""
    import torch
    say("split", n, opts)
    rng = np.random.default_rng(n)
    a = np.repeat(np.arange(n), rng.integers(30, 90, n))
    b = (a + rng.integers(1, 200, a.size)) % n
    g = G.Graph(n, a.astype(np.int64), b.astype(np.int64))
    h = lf.Handle(0)
    for k, v in opts.items():
        h.lf_set_option(k, v)
    h.load_graph(g.n, torch.from_numpy(g.src).cuda(), torch.from_numpy(g.dst).cuda()).init_communities()
    o = orc.Oracle()
    o.load_graph(g.n, g.src, g.dst)
    o.init_communities()
    same_hist(h.run_iterations(n, 0.0, 2), o.run_iterations(n, 0.0, 2))
    same_state(h, o)
    h.close()
    o.close()


@pytest.mark.parametrize("refs", [1, 2, 7, 300])
def test_f1_run_lengths(lf, orc, refs):
    """Detected communities that share 1 to 4,000 nodes with a reference one (runs whose end is
    found by doubling), one that meets hundreds of them (whole waves of runs), nodes with more
    ids than one thread checks, and id counts at which the keys gain a bit."""
    say("f1 runs", refs)
    sizes = [1, 2, 3, 4, 63, 64, 65, 127, 128, 129, 1023, 4000]
    n = sum(sizes)
    g = G.Graph(n, np.arange(n, dtype=np.int64), np.roll(np.arange(n, dtype=np.int64), -1))
    off, ids = cover([[c] for c, s in enumerate(sizes) for _ in range(s)])
    rng = np.random.default_rng(refs)
    few = [[int(rng.integers(0, refs))] for _ in range(n)]
    for x in (5, 700, n - 1):
        few[x] = rng.choice(refs, min(refs, 40), replace=False)
    roff, rids = cover(few)
    h = loaded(lf, g)
    h.init_from_memberships(off, ids, len(sizes))
    o = orc.Oracle()
    o.load_graph(g.n, g.src, g.dst)
    o.init_from_memberships(off, ids, len(sizes))
    a, b = h.cover_f1(roff, rids), o.cover_f1(roff, rids)
    assert a[0] == b[0]
    assert np.array_equal(np.asarray(a[1]).view(np.int64), np.asarray(b[1]).view(np.int64))
    assert np.array_equal(a[2], b[2])
    h.close()
    o.close()
