"""Graph set-up: the symmetric CSR from the two edge orders (isolated nodes, repeated and
reversed edges, self-loops, the first and last node without neighbours) and the triangle
passes at out-lists of exactly one and four waves, one more and one less, with empty lists
between them; adjacency, triangles and per-community weights equal the oracle's."""
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


def clique_graph(m, gap, seed):
    """A clique of m + 1 nodes, its lowest in (degree, id) order with m out-neighbours; `gap`
    nodes of degree 1 hang on random members; a tenth of the ids have no edge, the first and the
    last among them; a third of the edges come twice, some reversed, with self-loops between."""
    rng = np.random.default_rng(seed)
    a, b = np.triu_indices(m + 1, 1)
    a, b = np.concatenate([a, rng.integers(0, m + 1, gap)]), np.concatenate([b, m + 1 + np.arange(gap)])
    used = m + 1 + gap
    n = used + used // 10 + 2
    ids = np.sort(rng.choice(np.arange(1, n - 1), used, replace=False))
    ids = rng.permutation(ids)
    a, b = ids[a], ids[b]
    again = rng.random(a.size) < 1 / 3
    loops = rng.choice(ids, 5)
    src, dst = np.concatenate([a, b[again], loops]), np.concatenate([b, a[again], loops])
    p = rng.permutation(src.size)
    return G.Graph(n, src[p].astype(np.int64), dst[p].astype(np.int64))


@pytest.mark.parametrize("m,cap", [(1, 0), (2, 0), (63, 0), (64, 0), (65, 0), (256, 0), (257, 0), (257, 16), (400, 300)])
def test_csr_and_triangles(lf, orc, m, cap):
    import torch
    g = clique_graph(m, 40 if m > 2 else 3, m)
    print("[case]", m, cap, "n", g.n, "edges", g.src.size, flush=True)
    sys.stdout.flush()
    h = lf.Handle(0)
    h.lf_set_option("tri_lds_cap", cap)
    o = orc.Oracle()
    h.load_graph(g.n, torch.from_numpy(g.src).cuda(), torch.from_numpy(g.dst).cuda())
    o.load_graph(g.n, g.src, g.dst)
    for u, v in zip(h.csr(), o.csr()):
        assert np.array_equal(u, v)
    h.init_communities()
    o.init_communities()
    for u, v in zip(h.node_stats(), o.node_stats()):
        assert np.array_equal(np.asarray(u).view(np.int64) if u.dtype == np.float64 else u,
                              np.asarray(v).view(np.int64) if v.dtype == np.float64 else v)
    a, b = h.exact_wcc(), o.exact_wcc()
    for k in ("wcc_comm", "wcc_node", "t", "vt_out", "vt"):
        assert np.array_equal(np.asarray(a[k]), np.asarray(b[k])), k
    assert a["wcc"] == b["wcc"]
    h.close()
    o.close()


def test_one_handle_many_graphs(lf, orc):
    """Device blocks that a handle gave up serve its later requests: larger, smaller and again
    larger graphs on one handle leave what a new handle leaves."""
    import torch
    h = lf.Handle(0)
    for n, p, seed in ((40, 0.3, 1), (900, 0.02, 2), (7, 0.9, 3), (300, 0.2, 4), (900, 0.05, 5), (2, 1.0, 6)):
        g = G.random_gnp(n, p, seed)
        print("[case] reload", n, flush=True)
        o = orc.Oracle()
        o.load_graph(g.n, g.src, g.dst)
        o.init_communities()
        h.load_graph(g.n, torch.from_numpy(g.src).cuda(), torch.from_numpy(g.dst).cuda()).init_communities()
        a, b = h.run_iterations(8, 0.0, 3), o.run_iterations(8, 0.0, 3)
        assert np.array_equal(np.asarray(a["wtilde_hist"]), np.asarray(b["wtilde_hist"]))
        for u, v in zip(h.memberships() + (h.in_counts(),), o.memberships() + (o.in_counts(),)):
            assert np.array_equal(u, v)
        o.close()
    h.close()


@pytest.mark.parametrize("shape", ["even", "clustered", "narrow", "signed"])
def test_relabelled_ids(lf, orc, shape):
    """Ids found through a table of their leading bits: spread evenly, nearly all in one entry,
    closer together than the table is fine; negative ids are refused."""
    import torch
    rng = np.random.default_rng(5)
    n = 70_000
    if shape == "even":
        ids = np.sort(rng.choice(1 << 40, n, replace=False))
    elif shape == "clustered":
        ids = np.concatenate([[0, 3], 5_000_000_000 + np.arange(n - 4), [1 << 61, (1 << 62) - 1]])
    elif shape == "narrow":
        ids = 77 + np.arange(n)
    else:
        ids = np.concatenate([np.arange(n // 2) * 9, -1 - np.arange(n - n // 2) * 1_000_000_007])
    a = np.concatenate([np.arange(n), rng.integers(0, n, 3 * n)])
    b = np.concatenate([(np.arange(n) + 1) % n, rng.integers(0, n, 3 * n)])
    src, dst = ids[a].astype(np.int64), ids[b].astype(np.int64)
    print("[case] ids", shape, flush=True)
    h, o = lf.Handle(0), orc.Oracle()
    if shape == "signed":
        with pytest.raises(lf.LazyFoxError) as e:
            h.load_graph(0, torch.from_numpy(src).cuda(), torch.from_numpy(dst).cuda(), relabel=True)
        assert e.value.code == lf.LF_EINVAL
        return
    h.load_graph(0, torch.from_numpy(src).cuda(), torch.from_numpy(dst).cuda(), relabel=True)
    o.load_graph(0, src, dst, relabel=True)
    assert h.n == o.n == n
    for u, v in zip(h.csr() + (h.orig_ids(),), o.csr() + (o.orig_ids(),)):
        assert np.array_equal(u, v)
    h.close()
    o.close()
