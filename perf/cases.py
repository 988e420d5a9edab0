"""The work that users have this library do, as measured cases.

A case is one call or one short program through the package's public entry points, on
seeded synthetic graphs of the shapes that the repository's own workloads use (overlapping
block model, co-purchase-shaped, social-shaped, dense heavy-tailed and the serving mix).

* ``path``    raw edge list -> graph, node statistics, initial clustering, iterations until
              the stopping rule (or max_iters) -> memberships in host memory;
* ``init``    graph load and node statistics alone (the pre-processing of a graph);
* ``warm``    a saved cover taken up again: warm start, scores, some iterations;
* ``wcc``     the exact WCC of the current cover;
* ``cover``   F1 against a reference cover and the duplicate/contained check;
* ``batch``   several graphs of uneven size advanced together;
* ``serve``   a server that is handed a burst of jobs and run until all are done.
"""
import math

import numpy as np
import torch

import paper_2210_03211_amd as lf

# graph shapes: degree exponent, largest degree, memberships per node, community sizes
# (power law 1.5 on [lo, hi]) and the share of edges that leave the communities
SHAPES = {
    "sbm": dict(expo=0.0, dmax=64, mem=2, lo=50, hi=200, mu=0.2),
    "copurchase": dict(expo=2.5, dmax=550, mem=3, lo=5, hi=500, mu=0.3),
    "social": dict(expo=2.3, dmax=15_000, mem=4, lo=10, hi=3_000, mu=0.4),
    "dense": dict(expo=2.1, dmax=33_000, mem=5, lo=10, hi=3_000, mu=0.5),
    "job": dict(expo=2.5, dmax=1_000, mem=3, lo=5, hi=500, mu=0.3),
}


def listed():
    return [
        # the smallest whole job: a few hundred nodes, a handle of its own, launches and latency only
        dict(name="path_job_300", kind="path", shape="job", n=300, pairs=2_400, queue=16, iters=50,
             edges="host", relabel=False, own=True),
        # the small parity-sized graph (2,000 nodes, about 30,000 edges, queue 64)
        dict(name="path_sbm_2k", kind="path", shape="sbm", n=2_000, pairs=30_000, queue=64, iters=50,
             edges="device", relabel=False, own=False),
        # co-purchase-shaped graph with the small queue that keeps the order of changes fine
        dict(name="path_copurchase_335k", kind="path", shape="copurchase", n=335_000, pairs=926_000, queue=256,
             iters=50, edges="device", relabel=True, own=False),
        # the headline: social-shaped, 4 million nodes, from pinned host memory
        dict(name="path_social_4m", kind="path", shape="social", n=4_000_000, pairs=35_000_000, queue=4096,
             iters=50, edges="pinned", relabel=False, own=False),
        # the same shape at the largest queue of the sweep, where throughput counts
        dict(name="path_social_1m_q64k", kind="path", shape="social", n=1_000_003, pairs=8_750_000, queue=65536,
             iters=50, edges="device", relabel=False, own=False),
        # dense heavy-tailed graph whose hubs see most of the communities; the first iterations
        dict(name="path_dense_1m", kind="path", shape="dense", n=1_000_001, pairs=39_000_000, queue=16384,
             iters=6, edges="device", relabel=False, own=False),
        # pre-processing alone, ids to be compacted
        dict(name="init_social_1m", kind="init", shape="social", n=1_000_000, pairs=8_750_000, edges="host",
             relabel=True),
        # resume from a saved cover for three iterations
        dict(name="warm_social_700k", kind="warm", shape="social", n=700_001, pairs=6_125_000, queue=4096, iters=3,
             edges="device"),
        # the triangle score of a finished cover
        dict(name="wcc_social_1m", kind="wcc", shape="social", n=1_000_000, pairs=8_750_000),
        # evaluation of a cover against a known one, and its duplicates
        dict(name="cover_social_1m", kind="cover", shape="social", n=1_000_000, pairs=8_750_000),
        # graphs of uneven size advanced by one batch
        dict(name="batch_32_jobs", kind="batch", jobs=32, nodes=4_000, queue=64, iters=50),
        # a burst of serving jobs
        dict(name="serve_120_jobs", kind="serve", jobs=120, nodes=2_000, queue=0, iters=50),
    ]


def _logint(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["path", "path", "path", "path", "init", "warm", "wcc", "cover", "batch", "serve"])
    if kind == "path":
        shape = rng.choice(["job", "sbm", "copurchase", "social", "dense"])
        if shape == "job":
            n, deg = _logint(rng, 50, 20_000), rng.uniform(8, 40)
            q = min(4096, max(16, 2 ** round(math.log2(n / 32.0))))
        elif shape == "sbm":
            n, deg = _logint(rng, 500, 8_000), rng.uniform(20, 40)
            q = rng.choice([16, 33, 64, 128])
        elif shape == "copurchase":
            n, deg = _logint(rng, 10_000, 300_000), 5.5
            q = max(256, 2 ** round(math.log2(n / 1000.0)))
        elif shape == "social":
            n, deg = _logint(rng, 100_000, 1_500_000), 17.5
            q = max(1024 if n < 400_000 else 4096, rng.choice([1024, 3000, 4096, 16384, 65536]))
        else:
            n, deg = _logint(rng, 30_000, 350_000), 78.0
            q = rng.choice([4096, 10_007, 16384, 32768])
        return dict(kind=kind, shape=shape, n=n, pairs=int(n * deg / 2), queue=q, iters=6 if shape == "dense" else 50,
                    edges=rng.choice(["host", "pinned", "device"]), relabel=rng.random() < 0.3,
                    own=rng.random() < 0.5)
    if kind in ("init", "warm", "wcc", "cover"):
        shape = rng.choice(["social", "social", "copurchase"])
        n = _logint(rng, 20_000, 900_000)
        c = dict(kind=kind, shape=shape, n=n, pairs=int(n * (8.75 if shape == "social" else 2.76)))
        if kind == "init":
            c.update(edges=rng.choice(["host", "device"]), relabel=rng.random() < 0.5)
        if kind == "warm":
            c.update(queue=rng.choice([1024, 4096, 10_000, 16384]), iters=rng.randint(1, 3), edges="device")
        return c
    jobs = rng.randint(8, 32) if kind == "batch" else rng.randint(20, 100)
    return dict(kind=kind, jobs=jobs, nodes=_logint(rng, 500, 4_000), queue=rng.choice([0, 0, 64]), iters=50)


# ---------------------------------------------------------------- inputs
def _device():
    return "cuda" if torch.cuda.is_available() else "cpu"


def _cutoff(expo, dmax, mean):
    """Lower end c of a power law x^-expo on [c, dmax + 1) whose mean is `mean`."""
    def mean_of(c):
        a, b, hi = 1.0 - expo, 2.0 - expo, dmax + 1.0
        return (a / b) * (hi ** b - c ** b) / (hi ** a - c ** a)
    lo, hi = 0.5, float(dmax)
    for _ in range(60):
        mid = 0.5 * (lo + hi)
        lo, hi = (mid, hi) if mean_of(mid) < mean else (lo, mid)
    return 0.5 * (lo + hi)


def _power(gen, size, expo, lo, hi, dev):
    u = torch.rand(size, generator=gen, device=dev, dtype=torch.float64)
    a = 1.0 - expo
    x = (lo ** a + u * ((hi + 1.0) ** a - lo ** a)) ** (1.0 / a)
    return x.floor().clamp(max=hi).to(torch.int64)


def _shuffled(gen, x):
    key = torch.randint(0, 1 << 62, (x.numel(),), generator=gen, device=x.device)
    return x[torch.sort(key, stable=True).indices]


def _pairs(gen, owner, group):
    """Random perfect matching of the stubs within each group (an odd one out is dropped)."""
    bits = 32
    rnd = torch.randint(0, 1 << bits, (owner.numel(),), generator=gen, device=owner.device)
    key, idx = torch.sort((group << bits) | rnd, stable=True)
    owner, g = owner[idx], key >> bits
    m = owner.numel()
    if m < 2:
        return owner[:0], owner[:0]
    pos = torch.arange(m, device=owner.device)
    first = torch.searchsorted(g, g)
    left = ((pos - first) % 2 == 0)[:-1] & (g[:-1] == g[1:])
    at = left.nonzero().flatten()
    return owner[at], owner[at + 1]


def graph(shape, n, pairs, seed):
    """(src, dst, cover offsets, cover ids) on the device: planted overlapping communities,
    power-law degrees; raw pairs with repeats and both directions."""
    s, dev = SHAPES[shape], _device()
    gen = torch.Generator(device=dev).manual_seed(int(seed) * 7919 + n)
    dmax = max(4, min(s["dmax"], n - 1))
    mean = min(2.0 * pairs / n, 0.5 * dmax)
    if s["expo"]:
        deg = _power(gen, n, s["expo"], _cutoff(s["expo"], dmax, mean + 0.5), dmax, dev)
    else:
        deg = torch.randint(int(0.6 * mean), int(1.4 * mean) + 1, (n,), generator=gen, device=dev)
    # memberships: 1 .. mem with geometrically falling shares, placed on communities of power-law sizes
    share = 0.5 ** torch.arange(s["mem"], dtype=torch.float64, device=dev)
    cum = torch.cumsum(share / share.sum(), 0)
    u = torch.rand(n, generator=gen, device=dev, dtype=torch.float64)
    count = torch.searchsorted(cum[:-1].contiguous(), u, right=True) + 1
    total = int(count.sum())
    hi = min(s["hi"], max(5, n // 2))
    lo = min(s["lo"], hi)
    sizes = _power(gen, 2 * total // lo + 8, 1.5, float(lo), hi, dev)
    keep = int(torch.searchsorted(torch.cumsum(sizes, 0), total)) + 1
    sizes = sizes[:keep]
    k = sizes.numel()
    node = _shuffled(gen, torch.repeat_interleave(torch.arange(n, device=dev), count))
    comm = torch.repeat_interleave(torch.arange(k, device=dev), sizes)[:total]
    key = torch.unique(node[:comm.numel()] * k + comm)
    node, comm = key // k, key % k
    count = torch.bincount(node, minlength=n)
    off = torch.zeros(n + 1, dtype=torch.int64, device=dev)
    torch.cumsum(count, 0, out=off[1:])
    # (1 - mu) of a node's edges inside its communities (at most size - 1 in each), the rest anywhere
    intra = torch.where(count > 0, ((1.0 - s["mu"]) * deg.double()).round().to(torch.int64), 0)
    at = torch.arange(node.numel(), device=dev) - off[node]
    each = intra[node] // count[node] + (at < intra[node] % count[node])
    each = torch.minimum(each, (torch.bincount(comm, minlength=k) - 1)[comm])
    used = torch.zeros(n, dtype=torch.int64, device=dev).index_add_(0, node, each)
    a1, b1 = _pairs(gen, torch.repeat_interleave(node, each), torch.repeat_interleave(comm, each))
    stubs = _shuffled(gen, torch.repeat_interleave(torch.arange(n, device=dev), deg - used))
    half = stubs.numel() // 2
    a = torch.cat([a1, stubs[:half]])
    b = torch.cat([b1, stubs[half:2 * half]])
    order = _shuffled(gen, torch.arange(a.numel(), device=dev))
    a, b = a[order], b[order]
    flip = torch.rand(a.numel(), generator=gen, device=dev) < 0.5
    return torch.where(flip, b, a), torch.where(flip, a, b), off, comm.to(torch.int32)


def _placed(x, where):
    """An edge array where the user's program holds it: numpy, pinned host or device memory."""
    if where == "device":
        return x
    if where == "pinned" and torch.cuda.is_available():
        return torch.empty(x.shape, dtype=x.dtype, pin_memory=True).copy_(x)
    return x.cpu().numpy()


def _spread(x):
    """Ids as a user's file may hold them: not dense, order kept."""
    return 3 * x + 1_000


def _disturbed(off, ids, seed):
    """The planted cover as an earlier run may have left it: about a tenth of the
    memberships missing, another twentieth under ids of their own."""
    gen = torch.Generator(device=ids.device).manual_seed(int(seed) + 17)
    n = off.numel() - 1
    node = torch.repeat_interleave(torch.arange(n, device=ids.device), off[1:] - off[:-1])
    u = torch.rand(ids.numel(), generator=gen, device=ids.device)
    keep = u >= 0.1
    top = int(ids.max()) + 1 if ids.numel() else 0
    ids = torch.where(u > 0.95, top + (ids * 31 + node % 7) % max(1, top), ids.to(torch.int64))
    node, ids = node[keep], ids[keep]
    key = torch.unique(node * (2 * top + 1) + ids)
    node, ids = key // (2 * top + 1), key % (2 * top + 1)
    out = torch.zeros(n + 1, dtype=torch.int64, device=ids.device)
    torch.cumsum(torch.bincount(node, minlength=n), 0, out=out[1:])
    return out, ids.to(torch.int32)


def _job_sizes(case):
    """(nodes, queue, pairs) of each job: lognormal node counts (median `nodes`), mean degree 8 to 40."""
    r = np.random.default_rng(case["jobs"] * 1009 + case["nodes"])
    sizes = []
    for _ in range(case["jobs"]):
        n = int(np.clip(case["nodes"] * math.exp(r.normal(0.0, 1.0)), 50, 40_000))
        q = case["queue"] or int(min(4096, max(16, 2 ** round(math.log2(n / 32.0)))))
        sizes.append((n, q, int(n * r.uniform(8, 40) / 2)))
    return sizes


def _jobs(case, seed):
    r = np.random.default_rng(int(seed) * 31 + case["jobs"])
    jobs = []
    for n, q, pairs in _job_sizes(case):
        src, dst, _, _ = graph("job", n, pairs, int(r.integers(1 << 30)))
        jobs.append((n, q, src, dst))
    return jobs


# The program's result buffers, kept from one run to the next: what comes back is as long as the
# graph makes it, so each buffer has room for more and says with -1 (0 for values) where it ends.
ROOM = {"sbm": 16, "job": 16, "copurchase": 4, "social": 4, "dense": 8}


class Buffers:
    def __init__(self):
        self.have, self.used = {}, {}

    def put(self, name, values, room):
        b = self.have.get(name)
        if b is None:
            b = self.have[name] = np.full(room, 0 if values.dtype.kind == "f" else -1, values.dtype)
            self.used[name] = 0
        m = values.size
        if m > room:
            raise ValueError("%s: %d values, room for %d" % (name, m, room))
        b[:m] = values
        b[m:self.used[name]] = 0 if values.dtype.kind == "f" else -1
        self.used[name] = m
        return b


def prepare(case, seed):
    st = _prepare(case, seed)
    st["case"], st["buf"] = case, Buffers()
    if torch.cuda.is_available():
        torch.cuda.synchronize()
    return st


def _prepare(case, seed):
    kind = case["kind"]
    if kind in ("batch", "serve"):
        jobs = _jobs(case, seed)
        if kind == "serve":
            jobs = [(n, q, s.cpu().numpy(), d.cpu().numpy()) for n, q, s, d in jobs]
            return dict(jobs=jobs, server=lf.Server(0))
        return dict(jobs=jobs, batch=lf.Batch(0))
    src, dst, off, ids = graph(case["shape"], case["n"], case["pairs"], seed)
    st = {}
    if kind in ("path", "init"):
        if case["relabel"]:
            src, dst = _spread(src), _spread(dst)
        st["src"], st["dst"] = _placed(src, case["edges"]), _placed(dst, case["edges"])
        st["h"] = None if case.get("own") else lf.Handle(0)
        return st
    st["h"] = lf.Handle(0)
    st["off"], st["ids"] = _disturbed(off, ids, seed)
    torch.cuda.synchronize()                # the library works on a stream of its own
    st["h"].load_graph(case["n"], src, dst)
    if kind == "warm":
        st["h"].init_communities()          # node statistics, as the run that saved the cover had them
        return st
    st["h"].init_from_memberships(st["off"], st["ids"])
    st["roff"], st["rids"] = off, ids
    return st


# ---------------------------------------------------------------- one pass
def _result(put, case, n, shape, info, off, ids, tag=""):
    it = case["iters"]
    return dict(offsets=put("off" + tag, off, n + 1), ids=put("ids" + tag, ids, ROOM[shape] * n + 64),
                scores=put("scores" + tag, info["wtilde_hist"], it + 1), joins=put("joins" + tag, info["joins"], it),
                leaves=put("leaves" + tag, info["leaves"], it),
                communities=put("communities" + tag, info["communities"], it))


def run(state):
    case, put = state["case"], state["buf"].put
    kind, n = case["kind"], case.get("n")
    if kind == "path":
        h = state["h"] or lf.Handle(0)
        h.load_graph(case["n"], state["src"], state["dst"], relabel=case["relabel"])
        h.init_communities()
        info = h.run_iterations(case["queue"], 0.01, case["iters"])
        off, ids = h.memberships()
        if state["h"] is None:
            h.close()
        return _result(put, case, n, case["shape"], info, off, ids)
    if kind == "init":
        h = state["h"]
        h.load_graph(case["n"], state["src"], state["dst"], relabel=case["relabel"])
        h.init_communities()
        tri, ccl, order = h.node_stats()
        off, ids = h.memberships()
        return dict(triangles=put("tri", tri, n), cc_local=put("ccl", ccl, n), order=put("order", order, n),
                    cc=h.scores()["cc"], offsets=put("off", off, n + 1), ids=put("ids", ids, n))
    if kind == "warm":
        h = state["h"]
        h.init_from_memberships(state["off"], state["ids"])
        size, edges, score = h.communities()
        info = h.run_iterations(case["queue"], 0.0, case["iters"])
        off, ids = h.memberships()
        return dict(size=put("size", size, n), edges=put("edges", edges, n), score=put("score", score, n),
                    **_result(put, case, n, case["shape"], info, off, ids))
    if kind == "wcc":
        r = state["h"].exact_wcc()
        return dict(wcc=r["wcc"], wcc_comm=put("comm", r["wcc_comm"], n), wcc_node=put("node", r["wcc_node"], 4 * n),
                    t=put("t", r["t"], 4 * n), vt_out=put("out", r["vt_out"], 4 * n), vt=put("vt", r["vt"], n))
    if kind == "cover":
        f1, best, match = state["h"].cover_f1(state["roff"], state["rids"])
        keep, removed = state["h"].postprocess()
        return dict(f1=f1, best=put("best", best, n), match=put("match", match, n),
                    keep=put("keep", keep.astype(np.int8), n), duplicates=removed[0], contained=removed[1])
    if kind == "batch":
        b, hs, ms = state["batch"], [], []
        for m, q, src, dst in state["jobs"]:
            h = lf.Handle(0)
            h.load_graph(m, src, dst).init_communities()
            hs.append(h)
            ms.append(b.add(h, q, 0.01, case["iters"]))
        while b.step():
            pass
        out = []
        for i, (h, m) in enumerate(zip(hs, ms)):
            info = b.member_info(m)
            b.remove(m)
            out.append(_result(put, case, state["jobs"][i][0], "job", info, *h.memberships(), tag=str(i)))
            h.close()
        return _joined(out)
    srv, out = state["server"], {}
    at = {srv.submit(m, src, dst, q, 0.01, case["iters"]): i for i, (m, q, src, dst) in enumerate(state["jobs"])}
    pending = 1
    while pending or len(out) < len(at):
        pending = srv.tick()
        for j in srv.take_done():
            off, ids, info = srv.fetch(j)
            out[at[j]] = _result(put, case, state["jobs"][at[j]][0], "job", info, off, ids, tag=str(at[j]))
    return _joined([out[i] for i in range(len(at))])


def _joined(results):
    return {k: np.concatenate([r[k] for r in results]) for k in results[0]}


# ---------------------------------------------------------------- what a pass cannot do without
def work(case):
    kind = case["kind"]
    if kind in ("batch", "serve"):
        nodes = case["jobs"] * case["nodes"] * 1.6
        pairs, iters = nodes * 12.0, 8
    else:
        nodes, pairs, iters = float(case["n"]), float(case["pairs"]), min(case.get("iters", 0), 10)
    mem = 1.8 * nodes
    edges_in, csr = 16.0 * pairs, 8.0 * nodes + 8.0 * pairs
    cover = 8.0 * nodes + 4.0 * mem
    # an iteration reads every node's neighbours and their memberships (community, in-count) and
    # writes the memberships again; a candidate community's record is 44 bytes
    step = csr + 8.0 * 2.0 * pairs + 16.0 * mem + 44.0 * mem
    # an evaluated neighbour membership is two divisions and a sum
    ops = 2.0 * 2.0 * pairs * 1.8 * 8.0
    if kind == "path" or kind in ("batch", "serve"):
        return dict(bytes=edges_in + 2.0 * csr + iters * step + cover, flops=iters * ops)
    if kind == "init":
        return dict(bytes=edges_in + 2.0 * csr + 20.0 * nodes + cover, flops=10.0 * pairs)
    if kind == "warm":
        return dict(bytes=cover + iters * step + cover, flops=iters * ops)
    if kind == "wcc":
        return dict(bytes=csr + cover + 20.0 * mem + 4.0 * nodes, flops=20.0 * pairs)
    return dict(bytes=2.0 * cover + 20.0 * mem, flops=10.0 * mem)


# ---------------------------------------------------------------- the same in plain 64-bit torch
def _simple(n, src, dst):
    """Both directions of every simple edge, sorted: (row, column)."""
    keep = src != dst
    a, b = torch.minimum(src, dst)[keep], torch.maximum(src, dst)[keep]
    key = torch.unique(a * n + b)
    a, b = key // n, key % n
    key = torch.sort(torch.cat([a * n + b, b * n + a])).values
    return key // n, key % n, key


def _has(table, key):
    """Membership of `key` in the sorted `table`."""
    if table.numel() == 0:
        return torch.zeros_like(key, dtype=torch.bool)
    at = torch.searchsorted(table, key).clamp(max=table.numel() - 1)
    return table[at] == key


def _triangles(n, row, col, deg):
    """Every triangle once, as three node arrays, in chunks."""
    fwd = (deg[row] < deg[col]) | ((deg[row] == deg[col]) & (row < col))
    u, v = row[fwd], col[fwd]
    edge = u * n + v                         # sorted: rows ascend, columns ascend within a row
    start = torch.searchsorted(u, torch.arange(n + 1, device=u.device))
    length = (start[1:] - start[:-1])[v]
    cum = torch.cumsum(length, 0)
    lo, step = 0, 1 << 26
    while lo < u.numel():
        before = int(cum[lo - 1]) if lo else 0
        hi = max(lo + 1, int(torch.searchsorted(cum, before + step)))
        ln = length[lo:hi]
        e = torch.repeat_interleave(torch.arange(lo, hi, device=u.device), ln)
        pos = torch.arange(e.numel(), device=u.device) - torch.repeat_interleave(torch.cumsum(ln, 0) - ln, ln)
        w = v[start[v[e]] + pos]
        hit = _has(edge, u[e] * n + w)
        yield u[e[hit]], v[e[hit]], w[hit]
        lo = hi


def _padded(x, room):
    return torch.cat([x, torch.zeros(room - x.numel(), dtype=x.dtype, device=x.device)])


def exact(case, seed):
    kind = case["kind"]
    if kind in ("batch", "serve", "path"):
        # a run's scores follow from every one of its moves, and which of two nearly equal moves
        # is taken is part of the method's own exact arithmetic: plain floats walk elsewhere
        return None
    n = room = case["n"]
    src, dst, roff, rids = graph(case["shape"], n, case["pairs"], seed)
    dev = src.device
    off, ids = _disturbed(roff, rids, seed)
    node = torch.repeat_interleave(torch.arange(n, device=dev), off[1:] - off[:-1])
    comm = ids.to(torch.int64)
    k = int(comm.max()) + 1 if comm.numel() else 0
    size = torch.bincount(comm, minlength=k)
    if kind == "cover":
        rnode = torch.repeat_interleave(torch.arange(n, device=dev), roff[1:] - roff[:-1])
        refs = int(rids.max()) + 1
        rsize = torch.bincount(rids.to(torch.int64), minlength=refs)
        cnt = (roff[1:] - roff[:-1])[node]
        mine = torch.repeat_interleave(torch.arange(node.numel(), device=dev), cnt)
        pos = torch.arange(mine.numel(), device=dev) - torch.repeat_interleave(torch.cumsum(cnt, 0) - cnt, cnt)
        key, num = torch.unique(comm[mine] * refs + rids[roff[node[mine]] + pos].to(torch.int64), return_counts=True)
        f = 2.0 * num.double() / (size[key // refs] + rsize[key % refs]).double()
        best = torch.zeros(k, dtype=torch.float64, device=dev).scatter_reduce_(0, key // refs, f, "amax")
        return dict(f1=float(best.sum() / int((size > 0).sum())), best=_padded(best, room), match=None, keep=None,
                    duplicates=None, contained=None)
    if kind == "init" and case["relabel"]:
        n = int(torch.unique(torch.cat([src[src != dst], dst[src != dst]])).numel())
        keep = src != dst
        flat = torch.unique(torch.cat([src[keep], dst[keep]]), return_inverse=True)[1]
        src, dst = flat[:flat.numel() // 2], flat[flat.numel() // 2:]
    row, col, key = _simple(n, src, dst)
    deg = torch.bincount(row, minlength=n)
    if kind == "warm":
        member = torch.sort(comm * n + node).values
        cnt = deg[node]
        first = torch.searchsorted(row, torch.arange(n, device=dev))
        mine = torch.repeat_interleave(torch.arange(node.numel(), device=dev), cnt)
        pos = torch.arange(mine.numel(), device=dev) - torch.repeat_interleave(torch.cumsum(cnt, 0) - cnt, cnt)
        inside = _has(member, comm[mine] * n + col[first[node[mine]] + pos])
        i = torch.bincount(mine[inside], minlength=node.numel()).double()
        d, s = deg[node].double(), size[comm].double()
        g = torch.where((i >= 2) & (d >= 2), i * (i - 1) / ((d - 1) * (s - 1 + d - i)), 0.0)
        total = torch.zeros(k, dtype=torch.float64, device=dev).index_add_(0, comm, g)
        edges = torch.zeros(k, dtype=torch.float64, device=dev).index_add_(0, comm, i) / 2
        s = size.double()
        score = torch.where(s >= 2, 2 * edges / (s * (s - 1)), 0.0) * total
        return dict(size=None, edges=None, score=_padded(score, room), offsets=None, ids=None, scores=None, joins=None,
                    leaves=None, communities=None)
    tri = torch.zeros(n, dtype=torch.int64, device=dev)
    if kind == "init":
        for corners in _triangles(n, row, col, deg):
            for x in corners:
                tri += torch.bincount(x, minlength=n)
        d = deg.double()
        ccl = torch.where(deg > 1, tri.double() / (d * (d - 1) / 2), 0.0)
        return dict(triangles=None, cc_local=_padded(ccl, room), order=None, cc=float(ccl.sum() / n), offsets=None,
                    ids=None)
    # exact WCC of the disturbed cover
    member = node * k + comm                 # sorted: nodes ascend, ids ascend within a node
    t = torch.zeros(member.numel(), dtype=torch.int64, device=dev)
    closing = torch.zeros(key.numel(), dtype=torch.bool, device=dev)
    for corners in _triangles(n, row, col, deg):
        for a in range(3):
            x, y, z = corners[a], corners[(a + 1) % 3], corners[(a + 2) % 3]
            tri += torch.bincount(x, minlength=n)
            closing[torch.searchsorted(key, x * n + y)] = True
            closing[torch.searchsorted(key, y * n + x)] = True
            cnt = (off[1:] - off[:-1])[x]
            e = torch.repeat_interleave(torch.arange(x.numel(), device=dev), cnt)
            m = off[x[e]] + torch.arange(e.numel(), device=dev) - torch.repeat_interleave(
                torch.cumsum(cnt, 0) - cnt, cnt)
            both = _has(member, y[e] * k + comm[m]) & _has(member, z[e] * k + comm[m])
            t += torch.bincount(m[both], minlength=t.numel())
    crow, ccol = row[closing], col[closing]
    vt = torch.bincount(crow, minlength=n)
    first = torch.searchsorted(crow, torch.arange(n, device=dev))
    cnt = vt[node]
    mine = torch.repeat_interleave(torch.arange(node.numel(), device=dev), cnt)
    pos = torch.arange(mine.numel(), device=dev) - torch.repeat_interleave(torch.cumsum(cnt, 0) - cnt, cnt)
    away = ~_has(member, ccol[first[node[mine]] + pos] * k + comm[mine])
    out = torch.bincount(mine[away], minlength=node.numel())
    w = torch.where(tri[node] > 0, t.double() / tri[node].clamp(min=1).double()
                    * (vt[node].double() / (size[comm] - 1 + out).clamp(min=1).double()), 0.0)
    per = torch.zeros(k, dtype=torch.float64, device=dev).index_add_(0, comm, w)
    return dict(wcc=float(w.sum()), wcc_comm=_padded(per, room), wcc_node=_padded(w, 4 * room), t=None, vt_out=None,
                vt=None)
