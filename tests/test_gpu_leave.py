"""A batch member that leaves within an iteration (between two queues, with an iteration start
or end queued): its handle holds a partition like a warm start from the memberships that it
then has, and runs on from there like the oracle."""
import sys

import numpy as np
import pytest

import graphgen as G

pytestmark = pytest.mark.gpu


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


def bits(v):
    return np.asarray(v, np.float64).view(np.int64)


def same(h, o):
    for u, v in zip(h.memberships() + (h.in_counts(),), o.memberships() + (o.in_counts(),)):
        assert np.array_equal(u, v)


# steps taken before the member leaves: an iteration start queued (1), 1 .. 11 of 12 queues
# applied, an iteration end queued (13), then the same in the second and third iteration
@pytest.mark.parametrize("steps", [0, 1, 2, 5, 9, 12, 13, 14, 17, 22, 26, 27, 28, 33, 38, 42])
@pytest.mark.parametrize("most", [1, 7])
def test_leaves_within_an_iteration(lf, orc, most, steps):
    import torch
    print("[case] leaves after", steps, "steps, up to", most, "memberships", flush=True)
    sys.stdout.flush()
    rng = np.random.default_rng(most)
    g = G.random_gnp(180, 0.1, 11)
    K = 40
    lists = [rng.choice(K, rng.integers(1, most + 1), replace=False) for _ in range(g.n)]
    off = np.concatenate([[0], np.cumsum([len(c) for c in lists])]).astype(np.int64)
    ids = np.concatenate(lists).astype(np.int32)
    h, other = lf.Handle(0), lf.Handle(0)
    for x in (h, other):
        x.load_graph(g.n, torch.from_numpy(g.src).cuda(), torch.from_numpy(g.dst).cuda())
        x.init_from_memberships(off, ids, K)
    b = lf.Batch(0)
    m, m2 = b.add(h, 15, 0.0, 9), b.add(other, 16, 0.0, 3)
    for _ in range(steps):
        b.step()
    b.remove(m)
    if 1 < steps < 12:                       # some of the first iteration's queues applied, no more
        applied = []
        for k in range(1, 12):
            p = orc.Oracle().load_graph(g.n, g.src, g.dst)
            p.init_from_memberships(off, ids, K)
            assert p.run_queue_prefix(15, k) == k
            applied.append(all(np.array_equal(u, v) for u, v in zip(h.memberships(), p.memberships())))
            p.close()
        assert any(applied)
    o = orc.Oracle().load_graph(g.n, g.src, g.dst)
    o.init_from_memberships(*h.memberships(), K)
    same(h, o)
    assert np.array_equal(bits(h.scores()["wtilde"]), bits(o.scores()["wtilde"]))
    for u, v in zip(h.communities(), o.communities()):
        assert np.array_equal(bits(u) if u.dtype == np.float64 else u, bits(v) if v.dtype == np.float64 else v)
    # the rest of the batch is unaffected, and the member runs on: alone, then in a batch again
    while b.step() > 0:
        pass
    o2 = orc.Oracle().load_graph(g.n, g.src, g.dst)
    o2.init_from_memberships(off, ids, K)
    assert np.array_equal(bits(b.member_info(m2)["wtilde_hist"]), bits(o2.run_iterations(16, 0.0, 3)["wtilde_hist"]))
    assert np.array_equal(bits(h.run_iterations(15, 0.0, 2)["wtilde_hist"]),
                          bits(o.run_iterations(15, 0.0, 2)["wtilde_hist"]))
    same(h, o)
    m = b.add(h, 15, 0.0, 2)
    while b.step() > 0:
        pass
    assert np.array_equal(bits(b.member_info(m)["wtilde_hist"]), bits(o.run_iterations(15, 0.0, 2)["wtilde_hist"]))
    b.remove(m)
    same(h, o)
    b.close()
    for x in (h, other, o, o2):
        x.close()
