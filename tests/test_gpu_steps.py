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
