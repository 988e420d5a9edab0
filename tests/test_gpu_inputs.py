"""Device inputs still being written when a call is made: work on the default stream is waited
for by every call that takes device arrays, other streams' work is not by a new handle's load."""
import sys

import numpy as np
import pytest

import graphgen as G

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def env():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import oracle
    import paper_2210_03211_amd as lf
    lf.load_library()
    oracle.build(force=False)
    g = G.random_gnp(400, 0.05, 3)
    return torch, lf, oracle.Oracle().load_graph(g.n, g.src, g.dst).init_communities(), g


def busy(torch, n):
    """Queue some n / 2 ms of work on the current stream."""
    a = torch.ones(8192, 8192, device="cuda", dtype=torch.bfloat16)
    b = torch.empty_like(a)
    for _ in range(n):
        torch.mm(a, a, out=b)


def late(torch, v):
    """A device array whose values arrive behind work queued on the default stream."""
    src = torch.from_numpy(np.ascontiguousarray(v)).cuda()
    out = torch.zeros_like(src)
    torch.cuda.synchronize()
    busy(torch, 100)
    out.copy_(src)
    return out


def say(*a):
    print("[case]", *a, flush=True)
    sys.stdout.flush()


def test_inputs_behind_work_on_the_default_stream(env):
    torch, lf, o, g = env
    off, ids = o.memberships()
    for again in (False, True):             # onto a new handle, and onto one that has a graph
        say("late inputs, again", again)
        h = lf.Handle(0)
        if again:
            h.load_graph(3, np.array([0], np.int64), np.array([1], np.int64))
        src, dst = torch.from_numpy(g.src).cuda(), late(torch, g.dst)
        h.load_graph(g.n, src, dst)
        for u, v in zip(h.csr(), o.csr()):
            assert np.array_equal(u, v)
        h.init_communities()
        ids_dev = torch.from_numpy(ids).cuda()
        h.init_from_memberships(late(torch, off), ids_dev, int(ids.max()) + 1)
        for u, v in zip(h.memberships(), o.memberships()):
            assert np.array_equal(u, v)
        assert h.cover_f1(late(torch, off), ids_dev)[0] == o.cover_f1(off, ids)[0]
        h.close()


def test_new_handle_does_not_wait_for_other_streams(env):
    torch, lf, o, g = env
    src, dst = torch.from_numpy(g.src).cuda(), torch.from_numpy(g.dst).cuda()
    lf.Handle(0).load_graph(g.n, src, dst).close()      # kernels loaded, blocks in the cache
    h, s, done = lf.Handle(0), torch.cuda.Stream(), torch.cuda.Event()
    torch.cuda.synchronize()
    with torch.cuda.stream(s):
        busy(torch, 2000)
        done.record()
    say("load beside another stream's work")
    h.load_graph(g.n, src, dst)
    assert not done.query()
    for u, v in zip(h.csr(), o.csr()):
        assert np.array_equal(u, v)
    torch.cuda.synchronize()
    h.close()
