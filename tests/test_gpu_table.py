"""The table path (largest nodes): hash buckets whose entries fit one per thread, that hold
more visits or more distinct communities than that, nodes with more memberships of their own
than a block has threads, and with more chunks of neighbours; runs equal the oracle's bit for
bit."""
import sys

import numpy as np
import pytest

import graphgen as G

pytestmark = pytest.mark.gpu

CHUNK, AVG, FIT = 256, 192, 256      # neighbours per chunk, bound per bucket, entries per block


def bucket(ids, P):
    return ((ids.astype(np.uint64) * np.uint64(0x85EBCA6B)) & np.uint64(0xFFFFFFFF)) * np.uint64(P) >> np.uint64(32)


def hub_graph(n, extra, seed):
    """Node 0 joined to every other node; `extra` random pairs and a ring close triangles."""
    rng = np.random.default_rng(seed)
    o = np.arange(1, n, dtype=np.int64)
    a, b = rng.integers(1, n, extra), rng.integers(1, n, extra)
    src = np.concatenate([np.zeros(n - 1, np.int64), o, a])
    dst = np.concatenate([o, np.roll(o, -1), b])
    return G.Graph(n, src, dst)


def cover(lists):
    off = np.zeros(len(lists) + 1, np.int64)
    off[1:] = np.cumsum([len(p) for p in lists])
    return off, np.concatenate([np.asarray(p, np.int32) for p in lists]).astype(np.int32)


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


def bound_of_hub(h, g, lists):
    order = h.node_stats()[2]
    rank = np.empty(g.n, np.int64)
    rank[order] = np.arange(g.n)
    nb = np.arange(1, g.n)
    return int(sum(len(lists[y]) for y in nb) + (rank[nb] < rank[0]).sum() + len(lists[0]) + 1)


@pytest.mark.parametrize("case", ["spread", "shared", "colliding", "many_own", "wide"])
def test_bucket_shapes(lf, orc, case):
    rng = np.random.default_rng(7)
    q, iters, K = 64, 2, -1
    if case == "wide":
        g, q, iters = hub_graph(CHUNK * 256 + 300, 60_000, 1), 16384, 1
        lists = [[3000]] + [[int(c)] for c in rng.integers(0, 3000, g.n - 1)]
    else:
        g = hub_graph(701, 2500, 2)
        if case == "spread":             # about 2,100 visits of 900 communities
            lists = [[1, 2]] + [rng.choice(900, 3, replace=False) for _ in range(g.n - 1)]
        elif case == "shared":           # 2,100 visits of 6 communities: 350 in a bucket
            lists = [[1, 2]] + [rng.choice(6, 3, replace=False) for _ in range(g.n - 1)]
        elif case == "many_own":         # 300 of the hub's own, and a node with 40
            lists = [rng.choice(700, 300, replace=False), rng.choice(700, 40, replace=False)]
            lists += [rng.choice(700, 2, replace=False) for _ in range(g.n - 2)]
        else:
            lists = [[0]] + [[0, 1]] * (g.n - 1)     # replaced below, the same counts
    import torch
    h = lf.Handle(0)
    h.load_graph(g.n, torch.from_numpy(g.src).cuda(), torch.from_numpy(g.dst).cuda()).init_communities()
    P = -(-bound_of_hub(h, g, lists) // AVG)
    if case == "colliding":              # every community in the hub's first bucket, 600 of them
        K = 600 * P * 2
        ids = np.arange(K)
        same = ids[bucket(ids, P) == 0][:600]
        assert same.size == 600 > FIT
        lists = [[int(same[0])]] + [rng.choice(same, 2, replace=False) for _ in range(g.n - 1)]
    off, ids = cover(lists)
    size = np.bincount(bucket(ids[off[1]:], P).astype(np.int64), minlength=P)
    print("[case]", case, "buckets", P, "visits", size.sum(), "largest", size.max(), flush=True)
    sys.stdout.flush()
    assert P > 1 and (size.max() > FIT) == (case in ("shared", "colliding"))
    h.init_from_memberships(off, ids, K)
    o = orc.Oracle()
    o.load_graph(g.n, g.src, g.dst)
    o.init_from_memberships(off, ids, K)
    a, b = h.run_iterations(q, 0.0, iters), o.run_iterations(q, 0.0, iters)
    assert np.array_equal(np.asarray(a["wtilde_hist"]).view(np.int64), np.asarray(b["wtilde_hist"]).view(np.int64))
    for u, v in zip(h.memberships() + (h.in_counts(),), o.memberships() + (o.in_counts(),)):
        assert np.array_equal(u, v)
    h.close()
    o.close()
