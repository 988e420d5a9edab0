"""Hubs of the table path around 256 chunks of 256 neighbours (from there on a chunk is several
rounds), whose buckets hold more than a block takes at once: runs equal the oracle's."""
import sys

import numpy as np
import pytest

import graphgen as G

pytestmark = pytest.mark.gpu

MOST = 256 * 256                       # neighbours of 256 chunks of one round


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


def hub_graph(d, rest, seed):
    """Node 0 joined to d others; a ring and random pairs among all but it."""
    rng = np.random.default_rng(seed)
    o = np.arange(1, d + 1, dtype=np.int64)
    a, b = rng.integers(1, d + 1, rest), rng.integers(1, d + 1, rest)
    return G.Graph(d + 1, np.concatenate([np.zeros(d, np.int64), o, a]), np.concatenate([o, np.roll(o, -1), b]))


# communities: many more than a bucket holds, so that its hash range is cut; few, each in very
# many visits; and (with `one`) a node's own and nothing else
@pytest.mark.parametrize("d,K,per", [(MOST - 1, 40_000, 2), (MOST, 5, 2), (MOST + 1, 40_000, 2), (MOST + 257, 3, 1),
                                     (2 * MOST, 900, 1), (2 * MOST + 1, 60_000, 2)])
def test_hubs(lf, orc, d, K, per):
    import torch
    print("[case] hub of", d, "neighbours,", K, "communities", flush=True)
    sys.stdout.flush()
    rng = np.random.default_rng(d)
    g = hub_graph(d, 20_000, d)
    ids = rng.integers(0, K, (g.n, 2), dtype=np.int32)
    ids[:, 1] = (ids[:, 0] + 1 + ids[:, 1] % (K - 1)) % K
    ids = np.ascontiguousarray(ids[:, :per])
    off = np.arange(g.n + 1, dtype=np.int64) * per
    h = lf.Handle(0)
    h.load_graph(g.n, torch.from_numpy(g.src).cuda(), torch.from_numpy(g.dst).cuda())
    h.init_from_memberships(off, ids.ravel(), K)
    o = orc.Oracle().load_graph(g.n, g.src, g.dst)
    o.init_from_memberships(off, ids.ravel(), K)
    a, b = h.run_iterations(16384, 0.0, 2), o.run_iterations(16384, 0.0, 2)
    assert np.array_equal(np.asarray(a["wtilde_hist"]).view(np.int64), np.asarray(b["wtilde_hist"]).view(np.int64))
    for u, v in zip(h.memberships() + (h.in_counts(),), o.memberships() + (o.in_counts(),)):
        assert np.array_equal(u, v)
    h.close()
    o.close()
