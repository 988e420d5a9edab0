// iterate.hip -- one LazyFox iteration on the GPU: queues of q nodes in node order, each
// evaluated on the state at the start of the queue and then applied together
// (Methods, "Node Changes", Algorithm 2, "Stopping Criteria").
//
// At the start of an iteration every node is given an evaluation path from a bound on
// its visits that holds for the whole iteration (k_node_bounds), and each path gets the
// list of its nodes in order.  Per queue (all launches on the handle's stream, no host
// synchronisation):
//   k_refresh        the exact re-sums of the communities that the queue before touched, a
//                    wave per part (a community's parts leave their sums side by side and the
//                    last one adds them up); beside them, by block role, the gather of this
//                    queue's nodes: own and neighbours' memberships flattened into a list per
//                    node, and the table path's visits (largest nodes) grouped by hash bucket
//                    of their communities
//   k_eval           scores the lists in an LDS hash table: the small path, one wave per node
//                    with <= 64 entries, and the medium path, one 256-thread block per node
//                    with <= 256 (k_eval_whole gathers and scores, in very long queues)
//   k_eval_big       in queues with larger nodes: the workgroup path (one workgroup per node
//                    with <= 1024 entries), the table path's buckets (one block each), and the
//                    small and medium paths (k_eval_mid takes the latter two in long queues);
//                    block 0 of the scoring resets the queue's counters
//   k_big_tie        table path: the best of each node's buckets
//   k_apply          the bulk apply: membership edits, sizes, member-list appends and
//                    re-sum planning (a thread per queued node) beside the in-count
//                    changes around the moved nodes (a wave per in-count unit)
// After the last queue k_refresh runs once more, for the re-sums alone.
//
// Every sum is exact (fixed point), so none of the launch shapes above can change a bit
// of the result.
#include "method.h"

#define EW 4            // waves per block in the wave evaluation path
#define MXCAP 32        // own memberships kept in LDS (wave path)
#define INB 64          // neighbours per in-count unit (one per lane)
#define HOLE (-2)       // a membership left in the current iteration (removed at its end)
#define RB_MORE 3       // re-sum blocks of a queue per block of the option: 1,536 by default, six
                        // per CU (warm start, 700,000 nodes, queue 4096: 2 per CU 25.0 ms, 6 23.9)
#define PART 512        // members per re-sum part
#define EDITS 64        // queued nodes of an edit block of k_apply

static inline unsigned grid_for(long long n, int block) { return (unsigned)((n + block - 1) / block); }

// ------------------------------------------------------------------------------------
// evaluation, wave path
// ------------------------------------------------------------------------------------
// entry of C in the open-addressing table of T = 2^lg keys (-1: empty), claimed if absent
__device__ __forceinline__ int lds_insert(int *key, int T, int lg, int C, bool &claimed)
{
    unsigned hsh = hash_tab(C) >> (32 - lg);
    while (true) {
        int old = atomicCAS(&key[hsh], -1, C);
        if (old == -1 || old == C) {
            claimed = old == -1;
            return (int)hsh;
        }
        hsh = (hsh + 1) & (T - 1);
    }
}

// LDS of one node evaluation, 36 bytes per visit: the visit list (own memberships first,
// then the neighbours'), a hash table of 2*VCAP entries (community, count, the list entry
// that claimed it) and, in the list's storage once it is read, 128-bit sums for the few
// visits whose community another entry claimed first.  The last fields exchange values
// between the waves of a workgroup evaluation.
#define OWN_BIT 0x10000u    // kk: the community is one of the node's own (neighbours count below)
template <int VCAP>
struct NodeLds {
    int key[2 * VCAP];
    unsigned kk[2 * VCAP];
    unsigned short ow[2 * VCAP];
    union {
        struct {
            long long vslot[VCAP];
            int vdeg[VCAP];
        };
        unsigned long long acc[2][VCAP];
    };
    int wtot[4];
    double bjd[4], bld[4];
    int bj[4], bl[4];
};

#define VSMALL 64       // visits of the small wave path
#define VMED 256        // visits of the medium wave path
#define VGRP 1024       // visits of the workgroup path
#define GT 256          // threads of the workgroup path
// Small and medium blocks of a queue up to which its nodes go through lists in memory: their
// gather rides along in k_refresh and their scoring in k_eval_big (where there are larger
// nodes).  Beyond, both launches are bound by throughput, the lists are only traffic, and one
// light kernel does both.  Whole paths of social-shaped graphs: 1M nodes, queue 65,536 (over
// 10,000 blocks) 62 ms through lists, 56 without; 4M nodes, queue 4096 (about 1,500 blocks) 404
// through lists, 433 without; co-purchase shape, queue 256 (some 70 blocks) 88 to 92 against 100.
#define LIST_BLOCKS 4096
// Workgroup-path nodes of a queue that go through lists at once, 12 KB of list each: what is
// beyond is gathered and scored in further pairs of launches (slices of the queue), so that the
// lists of a queue of millions of nodes take 0.8 GB.  Slices this long cost nothing: three
// iterations of 262,144 such nodes in one queue spend 5.98 ms in the two kernels in one slice,
// 6.04 ms in four.  A batch holds the lists of all its members, so there a slice is shorter, and
// the small and medium nodes, which always go through lists, are also taken LIST_BLOCKS blocks
// at a time: a member's lists take 25 MB at most.
#define GROUP_SLICE 65536
#define BATCH_GROUP_SLICE 1024
#define SPARE_BYTES (4 << 20)   // most a batch member's buffer takes beyond a quarter more than it needs

// Every kernel of a queue is a chain of dependent reads, some 0.7 us each, so the kernels keep
// to three rules.  What does not depend on each other is read in one go: a read under a lane
// condition makes the compiler wait before the next one, so such reads take a clamped index
// and their value is dropped afterwards, and `arrived` keeps them from being moved behind a
// branch.  What is the same for a wave is made so for the compiler (uni).  And all of the
// arguments are read at once instead of a line at a time where each is first used.  (k_apply's
// in-count units had six round trips in a row where three depend on each other; 4M
// social-shaped nodes, queue 4096: k_apply 7.5 -> 6.5 us, k_refresh 10.8 -> 10.1, whole run 462 ->
// 437 ms.)

__device__ __forceinline__ int uni(int v) { return __builtin_amdgcn_readfirstlane(v); }
__device__ __forceinline__ long long uni(long long v)
{
    return ((long long)uni((int)(v >> 32)) << 32) | (unsigned)uni((int)v);
}

// one word of every 64-byte line of the arguments, so that they are all under way together
// and the scalar cache holds them afterwards
__device__ __forceinline__ void touch_args(const Ctx &cx, const QStep &qs)
{
    static_assert(sizeof(Ctx) > 320 && sizeof(Ctx) <= 384 && sizeof(QStep) > 64 && sizeof(QStep) <= 128,
                  "lines of the arguments");
    const int *a = (const int *)&cx, *b = (const int *)&qs;
    asm volatile("" ::"s"(a[0]), "s"(a[16]), "s"(a[32]), "s"(a[48]), "s"(a[64]), "s"(a[80]), "s"(b[0]), "s"(b[16]),
                 "s"(b[sizeof(QStep) / 4 - 2]));
}

// Member owning block b of a multi-graph launch, its blocks [b0, b1); -1 past the last one's.
// boff: n (a multiple of 64) entries, the first block of each member, ascending, then the
// number of blocks and BOFF_END to the end.  The wave reads 64 entries at a time.
__device__ __forceinline__ int find_member(const int *boff, int n, int b, int &b0, int &b1)
{
    const int lane = threadIdx.x & (WAVE - 1);
    int m = -1;
    b0 = b1 = 0;
    for (int i = 0; i < n; i += WAVE) {
        const int v = boff[i + lane];
        const unsigned long long at = __ballot(v <= b);
        m += __popcll(at);
        if (at) b0 = __builtin_amdgcn_readlane(v, 63 - __clzll((long long)at));
        if (~at) {                           // the first entry past b ends the search
            b1 = __builtin_amdgcn_readlane(v, __ffsll((long long)~at) - 1);
            break;
        }
    }
    return b1 != BOFF_END ? m : -1;
}

// Descriptors are constant during a launch.  Read as such, a line at a time ahead, they stay
// scalar; and every pointer is declared a global one, which those loaded from memory are not
// by themselves (a flat access also waits for the LDS).
template <class T>
__device__ __forceinline__ void as_global(T *&p)
{
    unsigned long long v;
    __builtin_memcpy(&v, &p, sizeof v);
    p = (T *)(__attribute__((address_space(1))) T *)v;
}

__device__ __forceinline__ void read_member(const Member *mem, Ctx &cx, QStep &qs)
{
    static_assert(sizeof(Ctx) % 8 == 0 && sizeof(QStep) % 8 == 0 && sizeof(Member) == sizeof(Ctx) + sizeof(QStep),
                  "read as 64-bit words");
    const __attribute__((address_space(4))) long long *w = (const __attribute__((address_space(4))) long long *)mem;
    long long a[sizeof(Ctx) / 8], b[sizeof(QStep) / 8];
#pragma unroll
    for (unsigned k = 0; k < sizeof(Ctx) / 8; k++) a[k] = w[k];
#pragma unroll
    for (unsigned k = 0; k < sizeof(QStep) / 8; k++) b[k] = w[sizeof(Ctx) / 8 + k];
    __builtin_memcpy(&cx, a, sizeof(Ctx));
    __builtin_memcpy(&qs, b, sizeof(QStep));
    as_global(cx.rowptr);
    as_global(cx.col);
    as_global(cx.deg);
    as_global(cx.order);
    as_global(cx.nh);
    as_global(cx.slot);
    as_global(cx.ln);
    as_global(cx.cr);
    as_global(cx.cm_off);
    as_global(cx.cm_len);
    as_global(cx.cm_node);
    as_global(cx.tflag);
    as_global(cx.ovf_node);
    as_global(cx.ovf_comm);
    as_global(cx.ovf_flag);
    as_global(cx.dec);
    as_global(cx.ctr);
#pragma unroll
    for (int k = 0; k < LF_PATH_COUNT; k++) {
        as_global(cx.plist[k]);
        as_global(cx.prec[k]);
    }
    as_global(cx.col_rank);
    as_global(cx.tpos);
    as_global(cx.tchunk);
    as_global(cx.tbuck);
    as_global(cx.tcur);
    as_global(cx.tvis);
    as_global(cx.trow);
    as_global(cx.tres);
    as_global(cx.lhdr);
    as_global(cx.lpair);
    as_global(cx.ldeg);
    as_global(cx.unit);
    as_global(cx.part_rec);
    as_global(cx.part_done);
    as_global(cx.psum);
    touch_args(cx, qs);
}

// Single-graph kernel K(Ctx, QStep) and multi-graph kernel K_multi over Member descriptors, both
// running BODY(cx, qs, block, blocks, lds).  k_refresh, k_eval and k_apply, which every queue
// launches, also take what their first reads need as leading scalar arguments: the dispatch
// puts those into registers (amdgpu-kernarg-preload-count), so the first round trip runs beside
// the argument read instead of behind it.  4M social-shaped nodes, queue 4096: 434 -> 423 ms;
// 335k co-purchase, queue 256: 93.3 -> 92.4.
#define SINGLE_KERNEL(K, BOUNDS, LDS_T, BODY)                                                 \
    __global__ void __launch_bounds__(BOUNDS) K(Ctx cx, QStep qs)                             \
    {                                                                                         \
        __shared__ LDS_T lds;                                                                 \
        touch_args(cx, qs);                                                                   \
        BODY(cx, qs, (int)blockIdx.x, (int)gridDim.x, lds);                                   \
    }
#define MULTI_KERNEL(K, BOUNDS, LDS_T, BODY)                                                  \
    __global__ void __launch_bounds__(BOUNDS) K##_multi(const Member *mem, const int *boff, int n) \
    {                                                                                         \
        __shared__ LDS_T lds;                                                                 \
        int b0, b1;                                                                           \
        const int m = find_member(boff, n, (int)blockIdx.x, b0, b1);                          \
        if (m < 0) return;                                                                    \
        Ctx cx;                                                                               \
        QStep qs;                                                                             \
        read_member(mem + m, cx, qs);                                                         \
        BODY(cx, qs, (int)blockIdx.x - b0, b1 - b0, lds);                                     \
    }

struct NoLds {
    int unused;
};

// barrier over the NT threads that evaluate one node (one wave or the whole workgroup)
template <int NT>
__device__ __forceinline__ void node_sync()
{
    if constexpr (NT == WAVE) WAVE_SYNC();
    else __syncthreads();
}

// inclusive prefix sum of v over the NT threads (within each wave, then the waves' totals
// through LDS); *total receives the sum over all NT threads
template <int NT>
__device__ __forceinline__ int node_incl_scan(int v, int tid, int *wtot, int *total)
{
    const int lane = tid & (WAVE - 1);
    int wsum;
    const int incl = wave_incl_scan(v, &wsum);
    if constexpr (NT == WAVE) {
        *total = wsum;
        return incl;
    } else {
        const int wv = tid / WAVE;
        if (lane == 0) wtot[wv] = wsum;
        __syncthreads();
        int off = 0, tot = 0;
        for (int w = 0; w < NT / WAVE; w++) {
            int t = wtot[w];
            if (w < wv) off += t;
            tot += t;
        }
        __syncthreads();
        *total = tot;
        return incl + off;
    }
}

// A node of degree d, evaluated from its list entries (entry b * NT + tid in sv[b]; a
// community below 0 is no entry; dg < 0: an own membership, else the neighbour's degree) in
// the cleared table of T = 2^lg entries.  Best join and leave on thread 0.
//
// Some 95 % of the visits are their community's only one, so the list entry that claims a
// community's table entry also scores it: it gathers the record and keeps its own
// correction in registers.  Only the other visits of a claimed community add theirs
// through LDS (two 64-bit atomics, the first one's carry taken into the second).  This
// needs no list of candidates, no record exchange and half the LDS of a table with digit
// counters, so eight 256-thread blocks share a CU instead of seven and the chain between
// the gathers is shorter: k_eval 16.2 -> 13.1 us per launch (4M-node social-shaped graph,
// queue 4096), 116 -> 86 us (1M nodes, queue 65,536).
struct Best {
    double jd, ld;
    int j, l;
    int ncand;                              // candidates this thread scored
};

template <int NT, int NB, int VCAP>
__device__ __forceinline__ Best score_list(const Ctx &cx, int d, const Slot (&sv)[NB], const int (&dg)[NB], int tid,
                                           NodeLds<VCAP> &L, int T, int lg)
{
    const int lane = tid & (WAVE - 1);
    int hs[NB];                             // table entry, or -1
    bool mine[NB];                          // this entry claimed it
#pragma unroll
    for (int b = 0; b < NB; b++) {
        hs[b] = -1;
        mine[b] = false;
        if (sv[b].comm >= 0) {
            hs[b] = lds_insert(L.key, T, lg, sv[b].comm, mine[b]);
            if (mine[b]) L.ow[hs[b]] = (unsigned short)(b * NT + tid);
            atomicAdd(&L.kk[hs[b]], dg[b] < 0 ? OWN_BIT : 1u);
        }
    }
    node_sync<NT>();
    // 2. one record gather per candidate (the other visits need its size only); the list is
    //    read, its storage becomes the sums
    CandRec rc[NB];
    unsigned kk[NB];
#pragma unroll
    for (int b = 0; b < NB; b++) {
        kk[b] = 0;
        if (hs[b] >= 0) {
            kk[b] = L.kk[hs[b]];
            if (mine[b]) load_cand(cx, sv[b].comm, kk[b] >= OWN_BIT, rc[b]);
            else rc[b].s = cx.cr[sv[b].comm].s;
            L.acc[0][b * NT + tid] = 0;
            L.acc[1][b * NT + tid] = 0;
        }
    }
    // 3. exact correction of every visit; those of a community another entry claimed are
    //    summed at that entry
    int bad = 0;
    u128 term[NB];
#pragma unroll
    for (int b = 0; b < NB; b++) {
        term[b] = 0;
        if (hs[b] >= 0 && dg[b] >= 0) term[b] = visit_term(kk[b] >= OWN_BIT, sv[b].in, dg[b], rc[b].s, bad);
    }
    node_sync<NT>();
#pragma unroll
    for (int b = 0; b < NB; b++) {
        if (hs[b] >= 0) {
            if (dg[b] < 0) {
                if ((unsigned)sv[b].in != (kk[b] & (OWN_BIT - 1))) atomicOr(&cx.ctr->error, LF_DEVERR_INCOUNT);
            } else if (!mine[b]) {
                const int o = L.ow[hs[b]];
                const unsigned long long lo = (unsigned long long)term[b];
                const unsigned long long was = atomicAdd(&L.acc[0][o], lo);
                atomicAdd(&L.acc[1][o], (unsigned long long)(term[b] >> 64) + (was + lo < lo ? 1ull : 0ull));
            }
        }
    }
    node_sync<NT>();
    // 4. change of every candidate's score, best join and best leave
    double bjd = 0.0, bld = 0.0;
    int bj = -1, bl = -1;
    int ncand = 0;
#pragma unroll
    for (int b = 0; b < NB; b++) {
        if (!mine[b]) continue;
        ncand++;
        const bool leave = kk[b] >= OWN_BIT;
        const int k = (int)(kk[b] & (OWN_BIT - 1));
        u128 corr = term[b];
        if (k > (dg[b] >= 0 ? 1 : 0)) {
            const int v = b * NT + tid;
            corr += ((u128)L.acc[1][v] << 64) | L.acc[0][v];
        }
        const double dl = cand_delta(rc[b], leave, k, d, corr, bad);
        if (leave) better(dl, sv[b].comm, bld, bl);
        else better(dl, sv[b].comm, bjd, bj);
    }
    wave_best(bjd, bj);
    wave_best(bld, bl);
    if constexpr (NT > WAVE) {
        const int wv = tid / WAVE;
        if (lane == 0) {
            L.bjd[wv] = bjd; L.bj[wv] = bj;
            L.bld[wv] = bld; L.bl[wv] = bl;
        }
        __syncthreads();
        if (tid == 0) {
            for (int w = 1; w < NT / WAVE; w++) {
                int oc = L.bj[w];
                double od = L.bjd[w];
                if (oc >= 0 && (bj < 0 || od > bjd || (od == bjd && oc < bj))) { bjd = od; bj = oc; }
                oc = L.bl[w];
                od = L.bld[w];
                if (oc >= 0 && (bl < 0 || od > bld || (od == bld && oc < bl))) { bld = od; bl = oc; }
            }
        }
    }
    if (bad) atomicOr(&cx.ctr->error, LF_DEVERR_INEXACT);
    Best r;
    r.jd = bjd;
    r.ld = bld;
    r.j = bj;
    r.l = bl;
    r.ncand = ncand;
    return r;
}

// The LDS evaluation takes two launches.  The gather (a role of k_refresh) flattens a node's
// own memberships and its neighbours' into a list in memory; the scoring (k_eval, k_eval_big)
// reads that list and needs the communities' records.  The gather reads nothing that the
// re-sums of the queue before write, so the two share a launch, and of a node's chain of
// dependent reads (column indices, neighbour lines, slots, records) only the last is left
// beside the scoring's own.  Each path's lists lie at a fixed stride per node.  Per queue of
// the 4M-node social-shaped graph: scoring 9.0 us instead of 13.1 for both, k_refresh 13.0
// instead of 10.7, and the larger nodes' launch is one instead of two.
struct NodeList {
    ListHdr *hdr;
    long long *pair;         // community | in-count << 32
    int *deg;                // neighbour's degree; -1: an own membership
};

// lists of the queue's small, medium and workgroup paths (path-list position i of each)
__device__ __forceinline__ NodeList list_at(const Ctx &cx, long long node, long long entry)
{
    return NodeList{cx.lhdr + node, cx.lpair + entry, cx.ldeg + entry};
}
__device__ __forceinline__ NodeList small_list(const Ctx &cx, const QStep &, int i)
{
    return list_at(cx, i, (long long)i * VSMALL);
}
__device__ __forceinline__ NodeList med_list(const Ctx &cx, const QStep &qs, int i)
{
    return list_at(cx, qs.ln + i, (long long)qs.ln * VSMALL + (long long)i * VMED);
}
__device__ __forceinline__ NodeList group_list(const Ctx &cx, const QStep &qs, int i)
{
    const int ln = qs.lists ? qs.ln : 0, em = qs.lists ? qs.em : 0;   // (the others have no lists)
    return list_at(cx, ln + em + i, (long long)ln * VSMALL + (long long)em * VMED + (long long)i * VGRP);
}

template <int VCAP>
struct GathLds {
    long long vslot[VCAP];
    int vdeg[VCAP];
    int wtot[4];
};

// node at position p of a path list, and its queue position
__device__ __forceinline__ NodeRec node_rec(const Ctx &cx, const QStep &qs, int path, int p, int &j)
{
    v4i r = *(const v4i *)&cx.prec[path][p];
    int pos = cx.plist[path][p];
    arrived(r, pos);
    j = uni(pos) - qs.cstart;
    return NodeRec{((long long)uni(r.y) << 32) | (unsigned)uni(r.x), uni(r.z), uni(r.w)};
}

// Flatten queued node j with NT threads (one wave, or a workgroup of GT threads) if its
// neighbours (<= VCAP), visits and own memberships fit (2 * (visits + own) <= table,
// <= VCAP of them, <= MXCAP own).  Returns false otherwise, the same for all NT threads.
// Every phase issues all of a thread's global gathers before it uses any: own slots +
// column indices, neighbour lines, neighbour slots.  With several neighbours per thread the
// lines' memberships are read a second time (from the cache) instead of held in registers.
// Thread tid receives list entries b * NT + tid (those below N) in e[b] and dg[b].
template <int NT, int VCAP>
__device__ __forceinline__ bool gather_node(const Ctx &cx, const NodeRec nr, int tid, GathLds<VCAP> &L, int wcap,
                                            int path, long long (&e)[VCAP / NT], int (&dg)[VCAP / NT], int &N,
                                            int &mcnt)
{
    constexpr int NB = VCAP / NT;
    const int x = nr.x, d = nr.d;
    const long long rb = nr.rb;
    if (d > VCAP) return false;
    // the adjacency gathers need only the node record; the own line (count, placement and
    // inline memberships) is fetched beside them
    const NodeLine *lxp = cx.ln + x;
    int yv[NB];
#pragma unroll
    for (int b = 0; b < NB; b++) {
        const int q = b * NT + tid;
        yv[b] = x;
        if (d > 0) yv[b] = cx.col[rb + (q < d ? q : d - 1)];
    }
    v4i hx = *(const v4i *)lxp;
    long long ownw = *(const long long *)&lxp->s[tid < LINE_SLOTS ? tid : LINE_SLOTS - 1];
    arrived(hx, ownw);
#pragma unroll
    for (int b = 0; b < NB; b++) arrived(yv[b]);
    // one line per neighbour: its count, degree and memberships in one gather
    constexpr int NL = NB == 1 ? 1 : 0;     // lines held
    NodeLine held;
    int yc[NB], yd[NB];
    long long yo[NB];
    if constexpr (NL == 1) {
        RawLine r = read_line(cx.ln + yv[0]);
        arrived(r.q[0], r.q[1], r.q[2], r.q[3]);
        held = as_line(r);
        yc[0] = held.cnt;
        yd[0] = held.deg;
        yo[0] = held.off;
    } else {
        v4i hy[NB];
#pragma unroll
        for (int b = 0; b < NB; b++) hy[b] = *(const v4i *)(cx.ln + yv[b]);
#pragma unroll
        for (int b = 0; b < NB; b++) {
            arrived(hy[b]);
            yc[b] = hy[b].x;
            yd[b] = hy[b].y;
            yo[b] = ((long long)hy[b].w << 32) | (unsigned)hy[b].z;
        }
    }
#pragma unroll
    for (int b = 0; b < NB; b++)
        if (b * NT + tid >= d) {
            yc[b] = 0;
            yo[b] = -1;
        }
    Slot own = {(int)ownw, (int)(ownw >> 32)};
    mcnt = uni(hx.x);
    const long long xoff = ((long long)uni(hx.w) << 32) | (unsigned)uni(hx.z);
    if (mcnt > MXCAP) return false;
    if (xoff >= 0 && tid < mcnt) own = cx.slot[xoff + tid];
    // neighbour memberships flattened into the list behind the own ones: an inline
    // membership is kept as its (community, in-count) pair, one in the slot array as the
    // complement of its slot index
    N = mcnt;
    int p0[NB];
#pragma unroll
    for (int b = 0; b < NB; b++) {
        p0[b] = 0;
        if (b * NT < d) {                   // uniform over the NT threads
            int tot;
            const int incl = node_incl_scan<NT>(yc[b], tid, L.wtot, &tot);
            p0[b] = N + incl - yc[b];
            N += tot;
            if (N > VCAP || 2 * N > wcap) return false;   // uniform
        }
    }
#pragma unroll
    for (int b = 0; b < NB; b++) {
        if (yo[b] < 0) {
            if constexpr (NL == 0)
                if (yc[b] > 0) held = cx.ln[yv[b]];
#pragma unroll
            for (int t = 0; t < LINE_SLOTS; t++)
                if (t < yc[b]) {
                    L.vslot[p0[b] + t] = ((long long)held.s[t].in << 32) | (unsigned)held.s[t].comm;
                    L.vdeg[p0[b] + t] = yd[b];
                }
        } else {
            for (int t = 0; t < yc[b]; t++) {
                L.vslot[p0[b] + t] = ~(yo[b] + t);
                L.vdeg[p0[b] + t] = yd[b];
            }
        }
    }
    if (tid < mcnt) {
        L.vslot[tid] = ((long long)own.in << 32) | (unsigned)own.comm;
        L.vdeg[tid] = -1;                   // an own membership, not a visit
    }
    node_sync<NT>();
#pragma unroll
    for (int b = 0; b < NB; b++) {
        const int v = b * NT + tid;
        e[b] = -1;
        dg[b] = 0;
        if (v < N) {
            e[b] = L.vslot[v];
            dg[b] = L.vdeg[v];
            if (e[b] < 0 && dg[b] >= 0) {
                const Slot sl = cx.slot[~e[b]];
                e[b] = ((long long)sl.in << 32) | (unsigned)sl.comm;
            }
        }
    }
    if (cx.stats && tid == 0) {
        unsigned long long *w = cx.ctr->work[path];
        atomicAdd(&w[0], 1ull);
        atomicAdd(&w[1], (unsigned long long)d);
        atomicAdd(&w[2], (unsigned long long)(N - mcnt));
        atomicAdd(&w[4], (unsigned long long)mcnt);
    }
    return true;
}

// Score a flattened node (entry b * NT + tid in e[b], dg[b]; those past its length are
// ignored); a membership its neighbour left earlier in this iteration (a hole) is no entry.
template <int NT, int VCAP>
__device__ __forceinline__ void score_entries(const Ctx &cx, const ListHdr h, const long long (&e)[VCAP / NT],
                                              const int (&dg)[VCAP / NT], int tid, NodeLds<VCAP> &L, int path)
{
    constexpr int NB = VCAP / NT;
    const int N = h.N;
    const int lg = N <= 4 ? 3 : 32 - __clz(2 * N - 1);    // T = 2^lg >= 2 N
    const int T = 1 << lg;
    for (int t = tid; t < T; t += NT) {
        L.key[t] = -1;
        L.kk[t] = 0;
    }
    Slot sv[NB];
#pragma unroll
    for (int b = 0; b < NB; b++) {
        sv[b].comm = b * NT + tid < N ? (int)(unsigned)e[b] : -1;
        sv[b].in = (int)(e[b] >> 32);
    }
    node_sync<NT>();
    const Best r = score_list<NT, NB, VCAP>(cx, h.d, sv, dg, tid, L, T, lg);
    if (tid == 0) cx.dec[h.j] = Decision{r.j, r.l, h.m, 0};
    if (cx.stats && r.ncand) atomicAdd(&cx.ctr->work[path][3], (unsigned long long)r.ncand);
}

// the list is read beside its length
template <int NT, int VCAP>
__device__ __forceinline__ void score_node(const Ctx &cx, const NodeList in, int tid, NodeLds<VCAP> &L, int path)
{
    constexpr int NB = VCAP / NT;
    const ListHdr h = *in.hdr;
    long long e[NB];
    int dg[NB];
#pragma unroll
    for (int b = 0; b < NB; b++) {
        e[b] = in.pair[b * NT + tid];
        dg[b] = in.deg[b * NT + tid];
    }
    score_entries<NT, VCAP>(cx, h, e, dg, tid, L, path);
}

// The gather roles take their queue's nodes from their path lists; the path was chosen so
// that the node fits, and a node that does not is an internal error (it is left without a
// move).
template <int NT, int VCAP>
__device__ __forceinline__ void gather_path(const Ctx &cx, const QStep &qs, int path, int p, int tid,
                                            GathLds<VCAP> &L, int wcap, const NodeList out)
{
    constexpr int NB = VCAP / NT;
    int j;
    const NodeRec nr = node_rec(cx, qs, path, p, j);
    long long e[NB];
    int dg[NB], N, mcnt;
    if (!gather_node<NT, VCAP>(cx, nr, tid, L, wcap, path, e, dg, N, mcnt)) {
        if (tid == 0) {
            *out.hdr = ListHdr{0, 0, nr.d, j};
            atomicOr(&cx.ctr->error, LF_DEVERR_CAP);
        }
        return;
    }
#pragma unroll
    for (int b = 0; b < NB; b++) {
        const int v = b * NT + tid;
        if (v < N) {
            out.pair[v] = e[b];
            out.deg[v] = dg[b];
        }
    }
    if (tid == 0) *out.hdr = ListHdr{N, mcnt, nr.d, j};
}

// both in one: gathered and scored by the same threads, no list in memory
template <int VCAP>
struct WholeLds {
    GathLds<VCAP> g;
    NodeLds<VCAP> n;
};

template <int NT, int VCAP>
__device__ __forceinline__ void whole_path(const Ctx &cx, const QStep &qs, int path, int p, int tid,
                                           WholeLds<VCAP> &L, int wcap)
{
    constexpr int NB = VCAP / NT;
    int j;
    const NodeRec nr = node_rec(cx, qs, path, p, j);
    long long e[NB];
    int dg[NB], N, mcnt;
    if (!gather_node<NT, VCAP>(cx, nr, tid, L.g, wcap, path, e, dg, N, mcnt)) {
        if (tid == 0) {
            cx.dec[j] = Decision{-1, -1, 0, 0};
            atomicOr(&cx.ctr->error, LF_DEVERR_CAP);
        }
        return;
    }
    score_entries<NT, VCAP>(cx, ListHdr{N, mcnt, nr.d, j}, e, dg, tid, L.n, path);
}

// The small and medium paths, in 256-thread blocks: the first es blocks score four
// small-path nodes each, one per wave; the next em blocks one medium-path node each, one
// list entry per thread.  These are all of k_eval (10 KB of LDS, eight blocks per CU), and
// block roles of k_eval_big where a launch of their own does not pay.
union EvalLds {
    NodeLds<VSMALL> w[EW];
    NodeLds<VMED> m;
};

__device__ __forceinline__ void eval_small_med(const Ctx &cx, const QStep &qs, int blk, EvalLds &L)
{
    const int wv = uni((int)threadIdx.x / WAVE), lane = threadIdx.x & (WAVE - 1);
    if (blk < qs.es) {
        const int i = blk * EW + wv;        // small blocks have no block barriers
        if (i < qs.ln) score_node<WAVE, VSMALL>(cx, small_list(cx, qs, i), lane, L.w[wv], LF_PATH_SMALL);
        return;
    }
    const int i = blk - qs.es;              // a medium block: every thread takes part
    if (i < qs.em) score_node<EW * WAVE, VMED>(cx, med_list(cx, qs, i), threadIdx.x, L.m, LF_PATH_MED);
}

// block 0 of a queue's scoring resets its apply counters (the launch before, which re-sums
// the communities of the queue before, is the last to use them)
__device__ __forceinline__ void reset_apply_counters(const Ctx &cx, int blk)
{
    if (blk == 0 && threadIdx.x == 0) {
        DevCounters *c = cx.ctr;
        c->parts_total = 0;
    }
}

__global__ void __launch_bounds__(EW * WAVE) k_eval(int es, int ln, int em, ListHdr *lhdr, long long *lpair, int *ldeg,
                                                    Ctx cx, QStep qs)
{
    __shared__ EvalLds lds;
    qs.es = es;
    qs.ln = ln;
    qs.em = em;
    cx.lhdr = lhdr;
    cx.lpair = lpair;
    cx.ldeg = ldeg;
    reset_apply_counters(cx, (int)blockIdx.x);
    eval_small_med(cx, qs, (int)blockIdx.x, lds);
}

// the same nodes gathered and scored in one launch (very long queues)
__global__ void __launch_bounds__(EW * WAVE) k_eval_whole(Ctx cx, QStep qs)
{
    __shared__ union {
        WholeLds<VSMALL> w[EW];
        WholeLds<VMED> m;
    } lds;
    const int blk = (int)blockIdx.x, wv = uni((int)threadIdx.x / WAVE), lane = threadIdx.x & (WAVE - 1);
    touch_args(cx, qs);
    reset_apply_counters(cx, blk);
    if (blk < qs.es) {
        const int i = blk * EW + wv;        // small blocks have no block barriers
        if (i < qs.ln) whole_path<WAVE, VSMALL>(cx, qs, LF_PATH_SMALL, qs.ls + i, lane, lds.w[wv], qs.wcap);
        return;
    }
    const int i = blk - qs.es;
    if (i < qs.em) whole_path<EW * WAVE, VMED>(cx, qs, LF_PATH_MED, qs.lm + i, threadIdx.x, lds.m, qs.mcap);
}

// ------------------------------------------------------------------------------------
// evaluation, table path
// ------------------------------------------------------------------------------------
// The largest nodes are gathered and scored without global atomics per visit.  First (a role
// of k_refresh) one block per chunk of TAB_CHUNK neighbours gathers their lines, counts their
// memberships per hash bucket of the communities, and writes them to the node's visit
// region grouped by bucket, with a row of the buckets' positions.  Then (in k_eval_big) one
// block per bucket collects its piece of every chunk and evaluates it like a medium-path
// node: all visits of a community meet in one bucket.  k_big_tie folds a node's buckets.
// A node has one bucket per BUCK_AVG visits of its bound, so a bucket's entries nearly
// always fit one per thread.
// The path is bound by its gathers (64-byte lines of the neighbours, 64-byte records of the
// candidates).  The former global hash table moved a 64-byte entry four to five times per
// visit besides: on a dense-shaped graph (1M nodes, 39M pairs, queue 16,384) its three launches
// took 201 + 146 + 19 us per queue, these roles as launches of their own 56 + 74 + 6; on the
// social-shaped one (4M nodes, queue 4096) 54 + 61 + 10 against 25 + 35 + 6.
#define TAB_CHUNK 256
#define TAB_MAXP 4096
#define VBUCK 256           // entries of a bucket evaluated one per thread
#define BUCK_AVG 192        // bound on visits per bucket aimed at

// Neighbours of a chunk of a node of degree d: TAB_CHUNK (one per thread), or, of a node with
// more than GT such chunks, as many rounds of them as leave it GT chunks, so that a bucket
// finds its piece of every chunk with one thread each.
__host__ __device__ __forceinline__ int chunk_span(int d)
{
    return d <= TAB_CHUNK * GT ? TAB_CHUNK : TAB_CHUNK * ((d - 1) / (TAB_CHUNK * GT) + 1);
}

// hash of a community: the top of h * P is its bucket of P, the rest orders it within
__device__ __forceinline__ unsigned long long bucket_hash(int C, int P)
{
    return (unsigned long long)((unsigned)C * 0x85EBCA6Bu) * (unsigned)P;
}

__device__ __forceinline__ int bucket_of(int C, int P) { return (int)(bucket_hash(C, P) >> 32); }

struct PartLds {
    int hist[TAB_MAXP];      // per bucket: visits, then the next position
    int wtot[GT / WAVE];
    int base;
};

// the line of neighbour i of a chunk (one without memberships past its last)
__device__ __forceinline__ NodeLine chunk_line(const Ctx &cx, const ChunkRec &cr, int i)
{
    const int y = cx.col[cr.rb + (i < cr.cnt ? i : cr.cnt - 1)];   // (a chunk is never empty)
    RawLine rl = read_line(cx.ln + y);
    arrived(rl.q[0], rl.q[1], rl.q[2], rl.q[3]);
    NodeLine ly = as_line(rl);
    if (i >= cr.cnt) {
        ly.cnt = 0;
        ly.off = -1;
    }
    return ly;
}

// the chunk k (thread per neighbour, TAB_CHUNK of them a round)
__device__ __forceinline__ void table_chunk(const Ctx &cx, const QStep &qs, int k, PartLds &S)
{
    const int tid = threadIdx.x;
    const ChunkRec cr = cx.tchunk[k];
    const int P = cr.P, cnt = uni(cr.cnt);
    for (int t = tid; t < P; t += GT) S.hist[t] = 0;
    NodeLine ly = chunk_line(cx, cr, tid);
    __syncthreads();
    int mine = 0;                            // memberships (holes left out)
    int r0 = 0;                              // the round held in ly
    while (true) {
        if (ly.off < 0) {
#pragma unroll
            for (int t = 0; t < LINE_SLOTS; t++)
                if (t < ly.cnt && ly.s[t].comm >= 0) {
                    atomicAdd(&S.hist[bucket_of(ly.s[t].comm, P)], 1);
                    mine++;
                }
        } else {
            for (int t0 = 0; t0 < ly.cnt; t0 += 4) {   // four slot loads per round trip
                int c[4];
#pragma unroll
                for (int q = 0; q < 4; q++) c[q] = cx.slot[ly.off + (t0 + q < ly.cnt ? t0 + q : t0)].comm;
                arrived(c[0], c[1], c[2], c[3]);
#pragma unroll
                for (int q = 0; q < 4; q++)
                    if (t0 + q < ly.cnt && c[q] >= 0) {
                        atomicAdd(&S.hist[bucket_of(c[q], P)], 1);
                        mine++;
                    }
            }
        }
        if (r0 + TAB_CHUNK >= cnt) break;
        r0 += TAB_CHUNK;
        ly = chunk_line(cx, cr, r0 + tid);
    }
    int total;
    (void)wave_incl_scan(mine, &total);
    if ((tid & (WAVE - 1)) == 0) S.wtot[tid / WAVE] = total;
    __syncthreads();
    if (tid == 0) {
        int all = 0;
        for (int w = 0; w < GT / WAVE; w++) all += S.wtot[w];
        S.base = atomicAdd(&cx.tcur[cr.p], all);   // this chunk's place in the node's region
        if (cx.stats) {
            atomicAdd(&cx.ctr->work[LF_PATH_TABLE][1], (unsigned long long)cr.cnt);
            atomicAdd(&cx.ctr->work[LF_PATH_TABLE][2], (unsigned long long)all);
        }
    }
    __syncthreads();
    // positions of the buckets: exclusive sums of the counts, GT buckets at a time
    int *row = cx.trow + (cr.row - qs.br.row0);
    int run = S.base;
    for (int t0 = 0; t0 < P; t0 += GT) {
        const int t = t0 + tid;
        const int v = t < P ? S.hist[t] : 0;
        int wsum;
        const int incl = wave_incl_scan(v, &wsum);
        __syncthreads();                     // the previous round's totals are read
        if ((tid & (WAVE - 1)) == 0) S.wtot[tid / WAVE] = wsum;
        __syncthreads();
        int off = run, all = 0;
        for (int w = 0; w < GT / WAVE; w++) {
            if (w < tid / WAVE) off += S.wtot[w];
            all += S.wtot[w];
        }
        if (t < P) {
            S.hist[t] = off + incl - v;
            row[t] = off + incl - v;
        }
        run += all;
    }
    if (tid == 0) row[P] = run;
    __syncthreads();
    TabVisit *out = cx.tvis + (cr.vis - qs.br.vis0);
    while (true) {                           // (from the last round, which is held, to the first)
        if (ly.off < 0) {
#pragma unroll
            for (int t = 0; t < LINE_SLOTS; t++)
                if (t < ly.cnt && ly.s[t].comm >= 0)
                    out[atomicAdd(&S.hist[bucket_of(ly.s[t].comm, P)], 1)] = TabVisit{ly.s[t].comm, ly.s[t].in, ly.deg, 0};
        } else {
            for (int t0 = 0; t0 < ly.cnt; t0 += 4) {
                long long sl[4];
#pragma unroll
                for (int q = 0; q < 4; q++)
                    sl[q] = *(const long long *)&cx.slot[ly.off + (t0 + q < ly.cnt ? t0 + q : t0)];
                arrived(sl[0], sl[1], sl[2], sl[3]);
#pragma unroll
                for (int q = 0; q < 4; q++) {
                    const int c = (int)sl[q];
                    if (t0 + q < ly.cnt && c >= 0)
                        out[atomicAdd(&S.hist[bucket_of(c, P)], 1)] = TabVisit{c, (int)(sl[q] >> 32), ly.deg, 0};
                }
            }
        }
        if (r0 == 0) break;
        r0 -= TAB_CHUNK;
        ly = chunk_line(cx, cr, r0 + tid);
    }
}

// A bucket whose entries do not fit one per thread (a community that many of the node's
// neighbours share, a node with more visits than TAB_MAXP buckets hold): the visits are
// streamed from memory, twice, and the distinct communities kept in the table.  The threads
// take the visits in turn and find each by the first positions of the chunks' pieces: with a
// walk over the chunks, all threads on one piece of a few visits, the buckets of a hub with a
// million neighbours took 7.9 ms, 60,000 0.36, now 0.55 and 0.14.  If the communities are more
// than VBUCK the bucket is cut into R slices of its hash range, R doubling until every slice
// fits; communities scored before a cut are scored again, which changes nothing.
struct GenLds {
    int key[2 * VBUCK];
    unsigned kk[2 * VBUCK];
    unsigned short ow[2 * VBUCK];   // candidate index
    int cl[VBUCK];                  // table entry of each candidate
    int sz[VBUCK];
    unsigned long long acc[2][VBUCK];
    int first[GT], lo[GT];          // per chunk: visits before its piece, where that starts
    int n, over;
};

// position of the bucket's visit i
__device__ __forceinline__ int gen_visit(const GenLds &G, int i)
{
    int c = 0;                      // the last chunk whose piece starts at or before i
#pragma unroll 1                    // (unrolled, the whole kernel spills more: dense graph 1.5 % slower)
    for (int s = GT / 2; s > 0; s /= 2)
        if (G.first[c + s] <= i) c += s;
    return G.lo[c] + (i - G.first[c]);
}

__device__ __forceinline__ int gen_find(const GenLds &G, int C)
{
    unsigned h = hash_tab(C) >> (32 - 9);
    while (G.key[h] != C) h = (h + 1) & (2 * VBUCK - 1);
    return (int)h;
}

__device__ __forceinline__ void gen_insert(GenLds &G, int C, unsigned add)
{
    static_assert(2 * VBUCK == 1 << 9, "table size of gen_find and gen_insert");
    if (*(volatile int *)&G.over) return;
    unsigned h = hash_tab(C) >> (32 - 9);
    for (int probe = 0; probe < 2 * VBUCK; probe++) {
        const int old = atomicCAS(&G.key[h], -1, C);
        if (old == -1) {
            const int i = atomicAdd(&G.n, 1);
            if (i >= VBUCK) {
                G.over = 1;
                return;
            }
            G.ow[h] = (unsigned short)i;
            G.cl[i] = (int)h;
        }
        if (old == -1 || old == C) {
            atomicAdd(&G.kk[h], add);
            return;
        }
        h = (h + 1) & (2 * VBUCK - 1);
    }
    G.over = 1;                              // the table is full
}

// whether C belongs to slice r of R of bucket b
__device__ __forceinline__ bool in_slice(int C, int P, int b, unsigned r, unsigned R)
{
    const unsigned long long h = bucket_hash(C, P);
    return (int)(h >> 32) == b && (unsigned)(((h & 0xffffffffull) * R) >> 32) == r;
}

__device__ __forceinline__ Best bucket_general(const Ctx &cx, const BuckRec &br, const TabVisit *vis, int nvis,
                                               const Slot *xs, int mcnt, GenLds &G)
{
    const int tid = threadIdx.x;
    Best r = {0.0, 0.0, -1, -1, 0};
    int bad = 0;
    for (unsigned R = 1;; R *= 2) {
        bool fits = true;
        for (unsigned sl = 0; sl < R && fits; sl++) {
            for (int t = tid; t < 2 * VBUCK; t += GT) {
                G.key[t] = -1;
                G.kk[t] = 0;
            }
            if (tid == 0) {
                G.n = 0;
                G.over = 0;
            }
            __syncthreads();
            for (int t = tid; t < mcnt; t += GT) {
                const int C = xs[t].comm;
                if (C >= 0 && in_slice(C, br.P, br.b, sl, R)) gen_insert(G, C, 0x80000000u);
            }
            for (int i = tid; i < nvis; i += GT) {
                const int C = vis[gen_visit(G, i)].comm;
                if (in_slice(C, br.P, br.b, sl, R)) gen_insert(G, C, 1u);
            }
            __syncthreads();
            if (G.over) {                    // uniform
                fits = false;
                __syncthreads();
                break;
            }
            const int nc = G.n;
            if (tid < nc) {
                G.sz[tid] = cx.cr[G.key[G.cl[tid]]].s;
                G.acc[0][tid] = 0;
                G.acc[1][tid] = 0;
            }
            __syncthreads();
            for (int t = tid; t < mcnt; t += GT) {
                const Slot o = xs[t];
                if (o.comm >= 0 && in_slice(o.comm, br.P, br.b, sl, R) &&
                    (unsigned)o.in != (G.kk[gen_find(G, o.comm)] & 0x7fffffffu))
                    atomicOr(&cx.ctr->error, LF_DEVERR_INCOUNT);
            }
            for (int i = tid; i < nvis; i += GT) {
                const TabVisit v = vis[gen_visit(G, i)];
                if (!in_slice(v.comm, br.P, br.b, sl, R)) continue;
                const int h = gen_find(G, v.comm);
                const int o = G.ow[h];
                const u128 term = visit_term(G.kk[h] >> 31, v.in, v.deg, G.sz[o], bad);
                const unsigned long long lw = (unsigned long long)term;
                const unsigned long long was = atomicAdd(&G.acc[0][o], lw);
                atomicAdd(&G.acc[1][o], (unsigned long long)(term >> 64) + (was + lw < lw ? 1ull : 0ull));
            }
            __syncthreads();
            if (tid < nc) {
                const int C = G.key[G.cl[tid]];
                const unsigned kk = G.kk[G.cl[tid]];
                CandRec rc;
                load_cand(cx, C, kk >> 31, rc);
                const u128 corr = ((u128)G.acc[1][tid] << 64) | G.acc[0][tid];
                const double dl = cand_delta(rc, kk >> 31, (int)(kk & 0x7fffffffu), br.d, corr, bad);
                if (kk >> 31) better(dl, C, r.ld, r.l);
                else better(dl, C, r.jd, r.j);
                r.ncand++;
            }
            __syncthreads();
        }
        if (fits) break;
        r.ncand = 0;
    }
    if (bad) atomicOr(&cx.ctr->error, LF_DEVERR_INEXACT);
    return r;
}

struct BuckLds {
    union {
        NodeLds<VBUCK> n;
        GenLds g;
    };
    double jd[GT / WAVE], ld[GT / WAVE];
    int j[GT / WAVE], l[GT / WAVE];
};

__device__ __forceinline__ void eval_bucket(const Ctx &cx, const QStep &qs, int k, BuckLds &S)
{
    const int tid = threadIdx.x;
    const BuckRec br = cx.tbuck[qs.br.b0 + k];
    const int *rows = cx.trow + (br.row - qs.br.row0);
    const TabVisit *vis = cx.tvis + (br.vis - qs.br.vis0);
    int lo = 0, len = 0;
    if (tid < br.nch) {                      // (a node has GT chunks at most)
        const int *rp = rows + (long long)tid * (br.P + 1) + br.b;
        lo = rp[0];
        len = rp[1] - lo;
    }
    const NodeLine *lxp = cx.ln + br.x;
    const int mcnt = lxp->cnt;
    const long long xoff = lxp->off;
    const Slot *xs = xoff < 0 ? lxp->s : cx.slot + xoff;
    Slot own = {-1, 0};
    if (tid < mcnt) own = xs[tid];
    const bool ownb = own.comm >= 0 && bucket_of(own.comm, br.P) == br.b;
    NodeLds<VBUCK> &L = S.n;
    // own memberships of this bucket, then its piece of every chunk
    int m, N;
    const int pm = node_incl_scan<GT>(ownb ? 1 : 0, tid, L.wtot, &m);
    const int pl = node_incl_scan<GT>(len, tid, L.wtot, &N);
    const int nvis = N;
    N += m;
    Best r;
    if (N <= VBUCK && mcnt <= GT) {          // uniform
        if (ownb) {
            L.vslot[pm - 1] = ((long long)own.in << 32) | (unsigned)own.comm;
            L.vdeg[pm - 1] = -1;
        }
        for (int i = 0; i < len; i++) {
            L.vslot[m + pl - len + i] = lo + i;
            L.vdeg[m + pl - len + i] = 0;
        }
        const int lg = N <= 4 ? 3 : 32 - __clz(2 * N - 1);    // T = 2^lg >= 2 N
        const int T = 1 << lg;
        for (int t = tid; t < T; t += GT) {
            L.key[t] = -1;
            L.kk[t] = 0;
        }
        __syncthreads();
        Slot sv[1] = {{-1, 0}};
        int dg[1] = {0};
        if (tid < N) {
            const long long e = L.vslot[tid];
            dg[0] = L.vdeg[tid];
            if (dg[0] < 0) {
                sv[0].comm = (int)(unsigned)e;
                sv[0].in = (int)(e >> 32);
            } else {
                const TabVisit v = vis[e];
                sv[0].comm = v.comm;
                sv[0].in = v.in;
                dg[0] = v.deg;
            }
        }
        r = score_list<GT, 1, VBUCK>(cx, br.d, sv, dg, tid, L, T, lg);
    } else {
        __syncthreads();                     // the scans' LDS is read
        S.g.first[tid] = pl - len;
        S.g.lo[tid] = lo;
        r = bucket_general(cx, br, vis, nvis, xs, mcnt, S.g);   // (its first barrier is before their use)
        wave_best(r.jd, r.j);
        wave_best(r.ld, r.l);
        const int wv = tid / WAVE;
        if ((tid & (WAVE - 1)) == 0) {
            S.jd[wv] = r.jd;
            S.ld[wv] = r.ld;
            S.j[wv] = r.j;
            S.l[wv] = r.l;
        }
        __syncthreads();
        if (tid == 0)
            for (int w = 1; w < GT / WAVE; w++) {
                better(S.jd[w], S.j[w], r.jd, r.j);
                better(S.ld[w], S.l[w], r.ld, r.l);
            }
    }
    if (tid == 0) {
        BuckRes q;
        q.jd = r.jd;
        q.ld = r.ld;
        q.j = r.j;
        q.l = r.l;
        cx.tres[k] = q;
    }
    if (cx.stats && r.ncand) atomicAdd(&cx.ctr->work[LF_PATH_TABLE][3], (unsigned long long)r.ncand);
}

// Queues with larger nodes, by block role: the workgroup path (one node per block at a time),
// the table path's buckets, and with fuse the small and medium paths.
union BigLds {
    BuckLds b;
    NodeLds<VGRP> g;
    EvalLds e;
};

__device__ __forceinline__ void body_eval_big(const Ctx &cx, const QStep &qs, int blk, int nblk, BigLds &L)
{
    (void)nblk;
    const BigRoles &r = qs.br;
    reset_apply_counters(cx, blk);
    int b = blk;
    if (b < r.bg) {
        for (int i = b; i < r.ng; i += r.bg) {
            score_node<GT, VGRP>(cx, group_list(cx, qs, i), threadIdx.x, L.g, LF_PATH_GROUP);
            __syncthreads();                // the next node reuses the LDS
        }
        return;
    }
    b -= r.bg;
    if (b < r.nb) {
        eval_bucket(cx, qs, b, L.b);
        return;
    }
    if (qs.lists) eval_small_med(cx, qs, b - r.nb, L.e);
}
#define BIG_BOUNDS GT, 4
#define MID_BOUNDS GT, 8
SINGLE_KERNEL(k_eval_big, BIG_BOUNDS, BigLds, body_eval_big)

// The same without the workgroup path, whose LDS (37 KB) and registers (112) leave four blocks
// to a CU where buckets and light nodes alone have eight.  The vector units are 43 % busy with
// four (dense graph), so for long launches the workgroup path gets a launch of its own: from
// SPLIT_BLOCKS blocks of the rest on, below which the launch costs more.  1M nodes, dense, queue
// 16,384: 101.8 ms in one launch, 97.3 split with six blocks to a CU, 95.5 with eight; 1M nodes,
// queue 65,536: 60.4, 58.9, 58.3.  4M nodes, queue 4096, one launch or split from 4096 / 2048 / 1024
// blocks on: 412.5, 411, 418.5, 420.5 ms.
#define SPLIT_BLOCKS 4096
union MidLds {
    BuckLds b;
    EvalLds e;
};
__global__ void __launch_bounds__(MID_BOUNDS) k_eval_mid(Ctx cx, QStep qs)
{
    __shared__ MidLds lds;
    touch_args(cx, qs);
    const int b = (int)blockIdx.x;
    reset_apply_counters(cx, b);
    if (b < qs.br.nb) {
        eval_bucket(cx, qs, b, lds.b);
        return;
    }
    if (qs.lists) eval_small_med(cx, qs, b - qs.br.nb, lds.e);
}
MULTI_KERNEL(k_eval_big, BIG_BOUNDS, BigLds, body_eval_big)

// the decision of every table-path node of the queue: the best of its buckets (one wave per
// node); communities in different buckets differ, so equal changes go to the lower id
__device__ __forceinline__ void body_big_tie(const Ctx &cx, const QStep &qs, int blk, int nblk, NoLds &)
{
    const int lane = threadIdx.x & (WAVE - 1), wv = threadIdx.x / WAVE;
    for (int i = blk * (GT / WAVE) + wv; i < qs.br.nt; i += nblk * (GT / WAVE)) {
        const int p = qs.br.lt + i;
        const int b0 = cx.tpos[p].bucket - qs.br.b0, b1 = cx.tpos[p + 1].bucket - qs.br.b0;
        const int x = cx.prec[LF_PATH_TABLE][p].x, j = cx.plist[LF_PATH_TABLE][p] - qs.cstart;
        const int mcnt = cx.ln[x].cnt;
        double bjd = 0.0, bld = 0.0;
        int bj = -1, bl = -1;
        for (int b = b0 + lane; b < b1; b += WAVE) {
            const BuckRes q = cx.tres[b];
            better(q.jd, q.j, bjd, bj);
            better(q.ld, q.l, bld, bl);
        }
        WAVE_SYNC();
        wave_best(bjd, bj);
        wave_best(bld, bl);
        if (lane == 0) {
            Decision dc;
            dc.J = bj;
            dc.L = bl;
            dc.pos = mcnt;
            dc.pad = 0;
            cx.dec[j] = dc;
            if (cx.stats) {
                atomicAdd(&cx.ctr->work[LF_PATH_TABLE][0], 1ull);
                atomicAdd(&cx.ctr->work[LF_PATH_TABLE][4], (unsigned long long)mcnt);
            }
        }
    }
}
SINGLE_KERNEL(k_big_tie, GT, NoLds, body_big_tie)
MULTI_KERNEL(k_big_tie, GT, NoLds, body_big_tie)

// ------------------------------------------------------------------------------------
// bulk apply
// ------------------------------------------------------------------------------------

// A queue's decisions are applied by one launch: the membership edits (one thread per
// queued node) and the in-count changes around the moved nodes (one wave per in-count
// unit of the queue) run side by side.  Slot positions stay put within an iteration: a
// leave turns its slot's community into HOLE, a join writes its community into the
// node's free slot (position dpos, in-count 0 from the iteration start).  So the in-count
// updates can target slots while the edits run, and they take each neighbour's
// membership after the queue from the neighbour's own decision rather than from its
// slots: the result is a from-scratch recount of every in-count on the new partition.

// Re-sum parts of a community at its first touch in the queue, planned from its member
// list's length then (joiners of the same queue that come later are the last part's).
__device__ __forceinline__ int part_count(long long cap, long long len)
{
    const int parts = (int)(((len < cap ? len : cap) + PART - 1) / PART);
    return parts < 1 ? 1 : parts;
}

// records of community C's parts from p0 on
__device__ __forceinline__ void plan_parts(const Ctx &cx, int C, long long base, long long cap, int parts, int p0)
{
    PartRec pr;
    pr.base = base;
    pr.C = C;
    pr.parts = parts;
    pr.cap = (int)cap;
    pr.pad[0] = pr.pad[1] = 0;
    if (p0 + parts > cx.part_cap) {
        atomicOr(&cx.ctr->error, LF_DEVERR_CAP);     // the run fails with this error
        pr.C = -1;                                    // the records that exist stay empty
    } else if (parts > 1) {
        cx.part_done[C] = 0;
    }
    for (int k = 0; k < parts && p0 + k < cx.part_cap; k++) {
        pr.k = k;
        cx.part_rec[p0 + k] = pr;
    }
}

struct EditLds {
    int sum[3][256 / WAVE];  // per wave: parts, joins, leaves
    int base;                // the block's first part
};

// Membership edits of queue position j; every thread of the block calls this (those past the
// queue take part in the counting only).  The queue's counters are one line of memory,
// whose atomics are served one after the other, so a block counts in LDS and adds once per
// counter, and a block has few enough nodes that their counters' atomics (six per node, each its
// own line) spread over the chip.  With three per wave the edits of a queue took 9.3 us where the
// in-counts beside them took 4.0 (1M nodes, dense, queue 16,384).  Whole runs, 32 / 64 / 128 / 256
// nodes to a block: 4M social-shaped nodes 437 / 434 / 433 / 436 ms, 32 graphs in a batch 312 /
// 293 / 297 / 307.
__device__ __forceinline__ void apply_edit(const Ctx &cx, const QStep &qs, int j, const int *order,
                                           EditLds &S)
{
    const int clen = qs.clen;
    const int lane = threadIdx.x & (WAVE - 1);
    const bool inq = j < clen;
    const int jc = inq ? j : clen - 1;      // (a queue is never empty)
    v4i dc = *(const v4i *)&cx.dec[jc];
    int x = order[jc];
    arrived(dc, x);
    const int J = inq ? dc.x : -1, L = inq ? dc.y : -1;
    const bool act = J >= 0 || L >= 0;
    bool firstL = false, firstJ = false, joined = false;
    long long cmoL = 0, capL = 0, cmoJ = 0, capJ = 0;
    int lenL = 0, lenJ = 0;
    int own_scanned = 0;
    if (act) {
        // everything that depends on x, J and L alone in one round trip: the node's line and
        // slot capacity, both member-list ranges, and the counters of both communities
        const int Lc = L >= 0 ? L : J, Jc = J >= 0 ? J : L;
        RawLine rx = read_line(cx.ln + x);
        long long nxt = cx.nh[x + 1].off;
        cmoL = cx.cm_off[Lc];
        capL = cx.cm_off[Lc + 1];
        cmoJ = cx.cm_off[Jc];
        capJ = cx.cm_off[Jc + 1];
        lenL = cx.cm_len[Lc];
        int oldL = 1, oldJ = 1, p = 0;
        if (L >= 0) {
            oldL = atomicExch(&cx.tflag[L], 1);
            atomicSub(&cx.cr[L].s, 1);
        }
        if (J >= 0) {
            p = atomicAdd(&cx.cm_len[J], 1);
            oldJ = atomicExch(&cx.tflag[J], 1);
            atomicAdd(&cx.cr[J].s, 1);
        }
        arrived(rx.q[0], rx.q[1], rx.q[2], rx.q[3], nxt);
        arrived(cmoL, capL, cmoJ, capJ);
        arrived(lenL, p, oldL, oldJ);
        const NodeLine hx = as_line(rx);
        capL -= cmoL;
        capJ -= cmoJ;
        lenJ = p + 1;
        firstL = oldL == 0;                 // first touch of the community in this queue
        firstJ = oldJ == 0;
        // a node's slots change only in its own queue, so they hold no hole yet and its
        // free slot is at cnt
        const int cnt = hx.cnt;
        const long long capx = hx.off < 0 ? LINE_SLOTS : nxt - hx.off;
        Slot *xs = hx.off < 0 ? cx.ln[x].s : cx.slot + hx.off;
        own_scanned = L >= 0 ? cnt : 0;
        if (L >= 0) {
            int tin = 0;
            const int t = line_find(cx, hx, L, &tin);
            if (t >= 0) xs[t].comm = HOLE;  // only the community word: in-counts are updated beside
        }
        if (J >= 0) {
            if (cnt < capx) {
                xs[cnt].comm = J;           // the free slot; its in-count is counted by the units
                cx.ln[x].cnt = cnt + 1;
                joined = true;
            } else {
                atomicOr(&cx.ctr->error, LF_DEVERR_SLOTS);   // the run fails; the lists stay whole
            }
            if (p < capJ) {
                cx.cm_node[cmoJ + p] = x;
            } else {
                int e = atomicAdd(&cx.ctr->ovf_cnt, 1);
                cx.ovf_node[e] = x;
                cx.ovf_comm[e] = J;
                cx.ovf_flag[J] = 1;
            }
        }
    }
    if (cx.stats) {
        const long long mv = wave_sum_i64(act ? 1 : 0), os = wave_sum_i64(own_scanned);
        if (lane == 0 && mv) {
            atomicAdd(&cx.ctr->apply[LF_APPLY_MOVES], (unsigned long long)mv);
            atomicAdd(&cx.ctr->apply[LF_APPLY_OWN_SLOTS], (unsigned long long)os);
        }
    }
    // one reservation per block for the parts of all its communities
    const int nL = firstL ? part_count(capL, lenL) : 0, nJ = firstJ ? part_count(capJ, lenJ) : 0;
    int tot;
    const int at = wave_incl_scan(nL + nJ, &tot) - (nL + nJ);
    const int wv = uni((int)threadIdx.x / WAVE);
    const int nj = __popcll(__ballot(joined)), nl = __popcll(__ballot(L >= 0));
    if (lane < 3) S.sum[lane][wv] = lane == 0 ? tot : lane == 1 ? nj : nl;
    __syncthreads();
    if (threadIdx.x < 3) {
        int v = 0;
        for (int w = 0; w < 256 / WAVE; w++) v += S.sum[lane][w];
        if (lane == 0) S.base = v ? atomicAdd(&cx.ctr->parts_total, v) : 0;
        else if (v) atomicAdd(lane == 1 ? &cx.ctr->joins : &cx.ctr->leaves, (unsigned long long)v);
    }
    __syncthreads();
    int p0 = S.base + at;
    for (int w = 0; w < wv; w++) p0 += S.sum[0][w];
    if (nL) plan_parts(cx, L, cmoL, capL, nL, p0);
    if (nJ) plan_parts(cx, J, cmoJ, capJ, nJ, p0 + nL);
}

// in-count changes of the neighbours in unit u (one wave): a neighbour y that holds J
// (L) from before this queue and keeps it gains (loses) one; the node's new J slot counts
// its neighbours in J after the queue (those that keep J and those that join it)
__device__ __forceinline__ void apply_unit(const Ctx &cx, const QStep &qs, long long u)
{
    const int lane = threadIdx.x & (WAVE - 1);
    const UnitRec ur = cx.unit[u];
    const int cnt = uni(ur.cnt), x = uni(ur.x);
    const long long e = uni(ur.rb) + (lane < cnt ? lane : cnt - 1);
    // the unit's neighbours, the node's decision, join position and line placement
    int y = cx.col[e];
    int ry = cx.col_rank[e];
    v4i dc = *(const v4i *)&cx.dec[uni(ur.r) - qs.cstart];
    long long xo = cx.ln[x].off;
    arrived(y, ry, dc, xo);
    const int J = uni(dc.x), L = uni(dc.y), pos = uni(dc.z);
    const long long xoff = uni(xo);
    if (J < 0 && L < 0) return;
    const int jy = ry - qs.cstart;
    const bool queued = jy >= 0 && jy < qs.clen;
    RawLine r = read_line(cx.ln + y);
    v4i dy = *(const v4i *)&cx.dec[queued ? jy : 0];
    arrived(r.q[0], r.q[1], r.q[2], r.q[3], dy);
    const NodeLine ly = as_line(r);
    const int Jy = queued ? dy.x : -1, Ly = queued ? dy.y : -1;
    if (lane >= cnt) y = -1;
    bool inJ = false;
    if (y >= 0) {
        if (ly.off < 0) {
#pragma unroll
            for (int t = 0; t < LINE_SLOTS; t++) {
                const int c = t < ly.cnt ? ly.s[t].comm : -1;
                if (J >= 0 && c == J) {
                    inJ = true;
                    if (Jy != J && Ly != J) atomicAdd(&cx.ln[y].s[t].in, 1);
                } else if (L >= 0 && c == L) {
                    if (Ly != L && Jy != L) atomicSub(&cx.ln[y].s[t].in, 1);
                }
            }
        } else {
            Slot *ys = cx.slot + ly.off;
            for (int t0 = 0; t0 < ly.cnt; t0 += 4) {   // four slot loads per round trip
                int cc[4];
#pragma unroll
                for (int q = 0; q < 4; q++) cc[q] = ys[t0 + q < ly.cnt ? t0 + q : t0].comm;
                arrived(cc[0], cc[1], cc[2], cc[3]);
#pragma unroll
                for (int q = 0; q < 4; q++) {
                    const int c = t0 + q < ly.cnt ? cc[q] : -1;
                    if (J >= 0 && c == J) {
                        inJ = true;
                        if (Jy != J && Ly != J) atomicAdd(&ys[t0 + q].in, 1);
                    } else if (L >= 0 && c == L) {
                        if (Ly != L && Jy != L) atomicSub(&ys[t0 + q].in, 1);
                    }
                }
            }
        }
    }
    const int fresh = __popcll(__ballot(J >= 0 && y >= 0 && (Jy == J || (inJ && Ly != J))));
    if (lane == 0 && fresh) {
        Slot *xs = xoff < 0 ? cx.ln[x].s : cx.slot + xoff;
        if (xoff >= 0 || pos < LINE_SLOTS) atomicAdd(&xs[pos].in, fresh);
    }
    if (cx.stats) {
        const long long sc = wave_sum_i64(y >= 0 ? ly.cnt : 0);
        if (lane == 0) {
            atomicAdd(&cx.ctr->apply[LF_APPLY_IN_ITEMS], 1ull);
            atomicAdd(&cx.ctr->apply[LF_APPLY_IN_NEIGHBOURS], (unsigned long long)cnt);
            atomicAdd(&cx.ctr->apply[LF_APPLY_IN_SLOTS], (unsigned long long)sc);
        }
    }
}

// blocks [0, eb) edit (a thread per queued node), the rest take one in-count unit per wave
__device__ __forceinline__ void body_apply(const Ctx &cx, const QStep &qs, int blk, const int *order, EditLds &S)
{
    const int eb = (qs.clen + EDITS - 1) / EDITS;
    if (blk < eb) {
        const int lane = threadIdx.x & (WAVE - 1), wv = uni((int)threadIdx.x / WAVE);
        constexpr int PER = EDITS / (256 / WAVE);
        apply_edit(cx, qs, lane < PER ? blk * EDITS + wv * PER + lane : qs.clen, order, S);
        return;
    }
    const long long w = (long long)(blk - eb) * (256 / WAVE) + uni((int)threadIdx.x / WAVE);
    if (w < qs.un) apply_unit(cx, qs, qs.ub + w);
}
__device__ __forceinline__ void multi_apply(const Ctx &cx, const QStep &qs, int blk, int nblk, EditLds &S)
{
    (void)nblk;
    body_apply(cx, qs, blk, cx.order + qs.cstart, S);
}

__global__ void __launch_bounds__(256) k_apply(const UnitRec *unit, int un, int clen, Decision *dec, const int *order,
                                               Ctx cx, QStep qs)
{
    __shared__ EditLds lds;
    cx.unit = unit;                          // the queue's
    qs.ub = 0;
    qs.un = un;
    qs.clen = clen;
    cx.dec = dec;
    body_apply(cx, qs, (int)blockIdx.x, order, lds);
}
MULTI_KERNEL(k_apply, 256, EditLds, multi_apply)

// ------------------------------------------------------------------------------------
// exact re-sum of the touched communities
// ------------------------------------------------------------------------------------
#define FOLD 64         // members per lane between two folds of its 128-bit sums
static_assert(FOLD < TERMS_U128, "a lane's sums hold that many terms");

// Exact re-sum of one part (one wave): the members' terms at sizes s, s+1 and s-1, and the
// sum of their in-counts.
__device__ __forceinline__ void refresh_part(const Ctx &cx, const PartRec &pr, long long p, int lane, int &bad)
{
    const int C = pr.C;
    const int k = pr.k;
    const long long base = pr.base, cap = pr.cap;
    const long long lo = (long long)k * PART;
    // size, list length and overflow after the edits, beside the part's first members (below
    // the list's capacity; those past its length are dropped)
    int s = cx.cr[C].s, ovf = cx.ovf_flag[C], fill = cx.cm_len[C];
    int y = 0;
    if (cap > 0) y = cx.cm_node[base + (lo + lane < cap ? lo + lane : cap - 1)];
    arrived(s, ovf, fill);
    s = uni(s);
    ovf = uni(ovf);
    const long long len = uni(fill) < cap ? uni(fill) : cap;
    // the plan is from the list's length at the community's first touch; the parts that hold
    // members after the edits (the same count for every part of C: the length is final here)
    // do the re-sum, the last one with whatever joined beyond the plan
    int parts = (int)((len + PART - 1) / PART);
    if (parts < 1) parts = 1;
    if (parts > pr.parts) parts = pr.parts;
    if (k >= parts) return;
    const long long hi = k == parts - 1 ? len : lo + PART;
    X192 S0 = x192_zero(), Sp = x192_zero(), Sm = x192_zero();
    long long ins = 0, mslots = 0;
    long long q = lo;
    while (q < hi) {
        const long long end = hi - q < FOLD * WAVE ? hi : q + FOLD * WAVE;
        u128 a0 = 0, ap = 0, am = 0;
        long long sumi = 0;
#pragma unroll 1
        for (; q < end; q += WAVE) {         // one member per lane in a round trip (two or four: slower)
            const bool in = q + lane < hi;
            const long long i = q + WAVE + lane;
            RawLine r = read_line(cx.ln + (in ? y : 0));
            int next = cx.cm_node[base + (i < hi ? i : hi - 1)];
            arrived(r.q[0], r.q[1], r.q[2], r.q[3], next);
            y = next;
            const NodeLine ly = as_line(r);
            if (in) {
                member_terms_of(cx, ly, C, s, a0, ap, am, sumi, bad);
                if (cx.stats) mslots += ly.cnt;
            }
        }
        WAVE_SYNC();
        x192_add(S0, wave_sum_u128(a0));
        x192_add(Sp, wave_sum_u128(ap));
        x192_add(Sm, wave_sum_u128(am));
        ins += (long long)wave_sum_u32((unsigned)sumi & 0xffffffu) +
               ((long long)wave_sum_u32((unsigned)(sumi >> 24)) << 24);
    }
    if (cx.stats) {
        mslots = wave_sum_i64(mslots);
        if (lane == 0) {
            atomicAdd(&cx.ctr->apply[LF_APPLY_PARTS], 1ull);
            if (k == 0) atomicAdd(&cx.ctr->apply[LF_APPLY_TOUCHED], 1ull);
            atomicAdd(&cx.ctr->apply[LF_APPLY_MEMBERS], (unsigned long long)(hi > lo ? hi - lo : 0));
            atomicAdd(&cx.ctr->apply[LF_APPLY_MEMBER_SLOTS], (unsigned long long)mslots);
        }
    }
    if (k == 0 && ovf) {                     // rare: joiners that did not fit the list
        const int no = __atomic_load_n(&cx.ctr->ovf_cnt, __ATOMIC_RELAXED);
        for (int e0 = 0; e0 < no; e0 += WAVE) {
            const int e = e0 + lane;
            u128 a0 = 0, ap = 0, am = 0;
            long long sumi = 0;
            if (e < no && cx.ovf_comm[e] == C) member_terms_line(cx, cx.ovf_node[e], C, s, a0, ap, am, sumi, bad);
            WAVE_SYNC();
            x192_add(S0, wave_sum_u128(a0));
            x192_add(Sp, wave_sum_u128(ap));
            x192_add(Sm, wave_sum_u128(am));
            ins += wave_sum_i64(sumi);
        }
    }
    if (parts == 1) {
        if (lane == 0) store_comm(cx, C, s, S0, Sp, Sm, ins, bad);
        return;
    }
    // A community's parts leave their sums beside each other (their records are consecutive),
    // and the last one to finish adds them up.  The sums are written and read past the caches
    // (device scope), so that waiting for the writes before the part is counted is enough; a
    // device-scope fence would also write the whole L2 back (212 us per queue with fences where
    // planted communities of up to 3,000 members are re-summed on a 700,000-node graph at
    // queue 4096, 82 with the wait).  One write by ten lanes instead of 19 atomics in a row on the
    // community's digit counters: a whole warm start of those nodes 28.7 -> 25.0 ms.  With parts
    // of 256 members instead of 512 it takes 23.6 (24.0 here), but small graphs with communities
    // of some 300 lose 2 %.
    u64 word = lane == 0 ? S0.w0 : lane == 1 ? S0.w1 : lane == 2 ? S0.w2 : lane == 3 ? Sp.w0 : lane == 4 ? Sp.w1
             : lane == 5 ? Sp.w2 : lane == 6 ? Sm.w0 : lane == 7 ? Sm.w1 : lane == 8 ? Sm.w2 : (u64)ins;
    if (lane < PSUM) __hip_atomic_store(&cx.psum[p * PSUM + lane], word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    int done = 0;
    if (lane == 0) done = atomicAdd(&cx.part_done[C], 1);
    if (uni(done) != parts - 1) return;
    S0 = Sp = Sm = x192_zero();
    ins = 0;
    for (int i0 = 0; i0 < parts; i0 += WAVE) {
        X192 t[3] = {x192_zero(), x192_zero(), x192_zero()};
        long long ti = 0;
        if (i0 + lane < parts) {
            unsigned long long *w = cx.psum + (p - k + i0 + lane) * PSUM;
#pragma unroll
            for (int v = 0; v < 3; v++) {
                t[v].w0 = __hip_atomic_load(w + 3 * v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                t[v].w1 = __hip_atomic_load(w + 3 * v + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                t[v].w2 = __hip_atomic_load(w + 3 * v + 2, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
            ti = (long long)__hip_atomic_load(w + 9, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        WAVE_SYNC();
        x192_add(S0, wave_sum_x192(t[0]));
        x192_add(Sp, wave_sum_x192(t[1]));
        x192_add(Sm, wave_sum_x192(t[2]));
        ins += wave_sum_i64(ti);
    }
    if (lane == 0) store_comm(cx, C, s, S0, Sp, Sm, ins, bad);
}

// Between two queues: the re-sums of the communities that the queue before touched (rb blocks,
// a wave per part), beside the gather of the next queue's nodes.  The two are independent:
// the re-sums write community records, the gather reads membership lines and slots, which
// nothing here writes.  The last queue of an iteration is followed by the re-sums alone.
union StepLds {
    PartLds t;
    GathLds<VGRP> g;
    GathLds<VMED> m;
    GathLds<VSMALL> w[EW];
};

__device__ __forceinline__ void body_refresh(const Ctx &cx, const QStep &qs, int blk, int nblk, StepLds &L)
{
    (void)nblk;
    const int wv = uni((int)threadIdx.x / WAVE), lane = threadIdx.x & (WAVE - 1);
    int b = blk;
    if (b < qs.rb) {
        const long long nw = (long long)qs.rb * (GT / WAVE);
        int bad = 0;
        long long p = (long long)b * (GT / WAVE) + wv;
        // the wave's first part is read beside the count (the buffer holds part_cap records)
        int count = cx.ctr->parts_total;
        v4i a0 = {0, 0, -1, 0}, a1 = {0, 0, 0, 0};
        if (p < cx.part_cap) {
            const v4i *q = (const v4i *)&cx.part_rec[p];
            a0 = q[0];
            a1 = q[1];
        }
        arrived(count, a0, a1);
        count = uni(count);
        if (count > cx.part_cap) count = cx.part_cap;
        while (p < count) {
            PartRec pr;
            pr.base = ((long long)uni(a0.y) << 32) | (unsigned)uni(a0.x);
            pr.C = uni(a0.z);
            pr.k = uni(a0.w);
            pr.parts = uni(a1.x);
            pr.cap = uni(a1.y);
            if (pr.C >= 0 && pr.C < cx.K) refresh_part(cx, pr, p, lane, bad);   // else: after a flagged overflow
            WAVE_SYNC();
            p += nw;
            if (p < count) {
                const v4i *q = (const v4i *)&cx.part_rec[p];
                a0 = q[0];
                a1 = q[1];
            }
        }
        if (bad) atomicOr(&cx.ctr->error, LF_DEVERR_INEXACT);
        return;
    }
    b -= qs.rb;
    const BigRoles &r = qs.br;
    if (b < r.bt) {
        for (int k = b; k < r.nc; k += r.bt) {
            table_chunk(cx, qs, r.c0 + k, L.t);
            __syncthreads();                // the next chunk reuses the LDS
        }
        return;
    }
    b -= r.bt;
    if (b < r.bg) {
        for (int i = b; i < r.ng; i += r.bg) {
            gather_path<GT, VGRP>(cx, qs, LF_PATH_GROUP, r.lg + i, threadIdx.x, L.g, qs.gcap, group_list(cx, qs, i));
            __syncthreads();                // the next node reuses the LDS
        }
        return;
    }
    b -= r.bg;
    if (!qs.lists) return;
    if (b < qs.em) {
        gather_path<GT, VMED>(cx, qs, LF_PATH_MED, qs.lm + b, threadIdx.x, L.m, qs.mcap, med_list(cx, qs, b));
        return;
    }
    const int i = (b - qs.em) * EW + wv;    // small blocks have no block barriers
    if (i < qs.ln)
        gather_path<WAVE, VSMALL>(cx, qs, LF_PATH_SMALL, qs.ls + i, lane, L.w[wv], qs.wcap, small_list(cx, qs, i));
}
__global__ void __launch_bounds__(GT) k_refresh(int rb, int bt, int bg, int em, PartRec *parts, DevCounters *ctr,
                                                const NodeRec *srec, const int *slist, Ctx cx, QStep qs)
{
    __shared__ StepLds lds;
    qs.rb = rb;
    qs.br.bt = bt;
    qs.br.bg = bg;
    qs.em = em;
    cx.part_rec = parts;
    cx.ctr = ctr;
    cx.prec[LF_PATH_SMALL] = srec;           // the queue's
    cx.plist[LF_PATH_SMALL] = (int *)slist;
    qs.ls = 0;
    body_refresh(cx, qs, (int)blockIdx.x, (int)gridDim.x, lds);
}
MULTI_KERNEL(k_refresh, GT, StepLds, body_refresh)

// ------------------------------------------------------------------------------------
// per-iteration sizing of the queue buffers
// ------------------------------------------------------------------------------------
// Evaluation path of every node for this iteration.  A node's own memberships do not
// change before it is evaluated, and each neighbour gains at most one membership per
// iteration, only if it is evaluated earlier (a smaller order position: the neighbours
// in the same queue are read at the queue's start).  So visits at evaluation <=
// B = visits at the iteration start + neighbours earlier in the order, and the path
// chosen from B always fits.  vbound = B + own + 1, at a table-path node's order position,
// bounds its distinct communities.
// Eight lanes per node (a wave for the longest), four neighbours per lane at a time: one read of
// columns, then four gathers under way.  A neighbour's membership count comes from one byte per
// node (mc8, 255: look in the node's header), an array that the caches hold where the headers do
// not, and the neighbours earlier in the order are counted once per clustering (FIRST) and
// kept.  70M gathers on the 4M-node social-shaped graph: 1,360 us a pass from the headers, 643
// from mc8 with a search for each neighbour's node, 551 now (8.7M gathers of 700,000 nodes 166 -> 90).
#define NB_LANES 8
#define NB_WAVE 512             // neighbours from which the whole wave takes the node
template <bool FIRST>
__global__ void __launch_bounds__(256) k_node_bounds(Ctx cx, const unsigned char *mc8, int *pre, long long *vbound,
                                                     int *cls, int wcap, int mcap, int gcap)
{
    if (blockIdx.x == 0 && threadIdx.x == 0) {          // the iteration's counters
        DevCounters *c = cx.ctr;
        c->joins = 0;
        c->leaves = 0;
        c->parts_total = 0;
        c->ovf_cnt = 0;
        c->live = 0;
    }
    const int lane = threadIdx.x & (WAVE - 1), sub = lane & (NB_LANES - 1);
    const long long x = (blockIdx.x * (long long)blockDim.x + threadIdx.x) / NB_LANES;
    if (x - lane / NB_LANES >= cx.n) return;            // uniform over the wave
    const bool in = x < cx.n;
    const long long xc = in ? x : cx.n - 1;
    const long long rb = cx.rowptr[xc], r1 = cx.rowptr[xc + 1];
    const int rx = cx.rank[xc];
    const NodeHdr hx = cx.nh[xc];
    const bool longer = in && r1 - rb > NB_WAVE;
    // visits and earlier neighbours among entries [e, e1) from e on in steps of `step`
    auto count = [&](long long e, long long e1, int step, int rank, long long &v, unsigned &b) {
        for (; e < e1; e += step) {
            const v4i y = read_entries(cx.col + e);
            v4i ry = {0, 0, 0, 0};
            if (FIRST) ry = read_entries(cx.col_rank + e);
            unsigned c[4];
#pragma unroll
            for (int t = 0; t < 4; t++) c[t] = mc8[e + t < e1 ? y[t] : y[0]];
#pragma unroll
            for (int t = 0; t < 4; t++)
                if (e + t < e1) {
                    v += c[t] == 255 ? cx.nh[y[t]].cnt : (int)c[t];
                    if (FIRST) b += ry[t] < rank;
                }
        }
    };
    long long v = 0;
    unsigned b = 0;
    count(rb + 4 * sub, in && !longer ? r1 : 0, 4 * NB_LANES, rx, v, b);
    WAVE_SYNC();
    long long V = (long long)oct_sum_u32((unsigned)v & 0xffffffu) + ((long long)oct_sum_u32((unsigned)(v >> 24)) << 24);
    unsigned P = FIRST ? oct_sum_u32(b) : 0;
    for (unsigned long long rest = __ballot(longer && sub == 0); rest; rest &= rest - 1) {
        const int src = __ffsll((long long)rest) - 1;
        long long vw = 0;
        unsigned bw = 0;
        count(__shfl(rb, src, WAVE) + 4 * lane, __shfl(r1, src, WAVE), 4 * WAVE, __shfl(rx, src, WAVE), vw, bw);
        WAVE_SYNC();
        vw = (long long)wave_sum_u32((unsigned)vw & 0xffffffu) + ((long long)wave_sum_u32((unsigned)(vw >> 24)) << 24);
        if (FIRST) bw = wave_sum_u32(bw);
        if (lane / NB_LANES == src / NB_LANES) {
            V = vw;
            P = bw;
        }
        WAVE_SYNC();
    }
    if (!in || sub != NB_LANES - 1) return;
    int before;
    if (FIRST) pre[x] = before = (int)P;
    else before = pre[x];
    const long long B = V + before, M = hx.cnt, dd = hx.deg;
    int c = LF_PATH_TABLE;
    if (M <= MXCAP) {
        if (dd <= VSMALL && B + M <= VSMALL && 2 * (B + M) <= wcap) c = LF_PATH_SMALL;
        else if (dd <= VMED && B + M <= VMED && 2 * (B + M) <= mcap) c = LF_PATH_MED;
        else if (dd <= VGRP && B + M <= VGRP && 2 * (B + M) <= gcap) c = LF_PATH_GROUP;
    }
    cls[rx] = c;
    if (c == LF_PATH_TABLE) vbound[rx] = B + M + 1;
}

// The path lists (ascending order positions, path after path): every tile of CLS_TILE positions
// counts its nodes per path (cnt[path][tile], a last entry of 0), one scan of those counts
// gives each tile's first list position per path, and the tiles place their nodes with their
// records and write the queues' first list positions.
#define CLS_ITEMS 4         // small tiles, so that small graphs spread over several blocks too
#define CLS_TILE (256 * CLS_ITEMS)

// a tile's counts per path, packed 16 bits each, before this thread's CLS_ITEMS positions
__device__ __forceinline__ unsigned long long class_prefix(unsigned long long v, unsigned long long *s_w,
                                                           unsigned long long *total)
{
    const int lane = threadIdx.x & (WAVE - 1), wv = threadIdx.x / WAVE;
    unsigned long long incl = v;
    for (int o = 1; o < WAVE; o <<= 1) {
        const unsigned long long t = (unsigned long long)__shfl_up((long long)incl, o, WAVE);
        if (lane >= o) incl += t;
    }
    if (lane == WAVE - 1) s_w[wv] = incl;
    __syncthreads();
    unsigned long long off = 0, tot = 0;
    for (int w = 0; w < 256 / WAVE; w++) {
        const unsigned long long t = s_w[w];
        if (w < wv) off += t;
        tot += t;
    }
    *total = tot;
    return off + incl - v;
}

__global__ void __launch_bounds__(256) k_class_count(const int *cls, long long n, long long ntiles, int *cnt)
{
    __shared__ unsigned long long s_w[256 / WAVE];
    const long long r0 = (long long)blockIdx.x * CLS_TILE + threadIdx.x * CLS_ITEMS;
    unsigned long long v = 0;
#pragma unroll
    for (int i = 0; i < CLS_ITEMS; i++)
        if (r0 + i < n) v += 1ull << (16 * cls[r0 + i]);
    unsigned long long tot;
    (void)class_prefix(v, s_w, &tot);
    if (threadIdx.x < LF_PATH_COUNT)
        cnt[threadIdx.x * ntiles + blockIdx.x] = (int)((tot >> (16 * threadIdx.x)) & 0xffff);
    if (blockIdx.x == 0 && threadIdx.x == 0) cnt[LF_PATH_COUNT * ntiles] = 0;
}

__global__ void __launch_bounds__(256) k_class_place(const int *cls, long long n, long long ntiles,
                                                     const long long *base, int *list, NodeRec *prec, int q,
                                                     long long nq, long long *qoff, const int *order,
                                                     const long long *rowptr, const int *deg)
{
    __shared__ unsigned long long s_w[256 / WAVE];
    const long long r0 = (long long)blockIdx.x * CLS_TILE + threadIdx.x * CLS_ITEMS;
    int cl[CLS_ITEMS];
    unsigned long long v = 0;
#pragma unroll
    for (int i = 0; i < CLS_ITEMS; i++) {
        cl[i] = r0 + i < n ? cls[r0 + i] : -1;
        if (cl[i] >= 0) v += 1ull << (16 * cl[i]);
    }
    unsigned long long tot;
    unsigned long long at = class_prefix(v, s_w, &tot);
#pragma unroll
    for (int i = 0; i < CLS_ITEMS; i++) {
        const long long r = r0 + i;
        if (r <= n && (r % q == 0 || r == n))          // a queue starts here (the end: after the last)
            for (int c = 0; c < LF_PATH_COUNT; c++)
                qoff[c * (nq + 1) + (r == n ? nq : r / q)] =
                    base[c * ntiles + blockIdx.x] + (long long)((at >> (16 * c)) & 0xffff) - base[c * ntiles];
        if (cl[i] < 0) continue;
        const long long p = base[cl[i] * ntiles + blockIdx.x] + (long long)((at >> (16 * cl[i])) & 0xffff);
        at += 1ull << (16 * cl[i]);
        const int x = order[r];
        list[p] = (int)r;
        prec[p] = NodeRec{rowptr[x], x, deg[x]};
    }
}

// Layout of the table path: for each of its nodes (their list starts at lbase[0] and ends at
// lbase[ntiles]) the exclusive sums of visit bounds, row entries, chunks and buckets, and the
// visits placed so far cleared.  One block: what it reads per node lies in list order (the
// bounds nearly so), LAYOUT_PER nodes per thread at a time, and the four sums share two barriers.
// With gathers by node and a scan of its own for each sum an iteration of the dense graph's 3M
// nodes spent 4.0 ms here, now 1.2, and one of 4M social-shaped nodes 194 us, now 60; 1M dense
// nodes take 97 us, and 266 with these sums but the gathers by node.
#define LAYOUT_PER 4
__global__ void __launch_bounds__(1024) k_table_layout(const int *list, const NodeRec *prec, const long long *lbase,
                                                       long long ntiles, const long long *vbound, TabPos *tpos,
                                                       int *tcur)
{
    __shared__ long long s_w[4][1024 / WAVE];
    const int lane = threadIdx.x & (WAVE - 1), wv = threadIdx.x / WAVE;
    list += lbase[0];
    prec += lbase[0];
    const long long nt = lbase[ntiles] - lbase[0];
    long long at[4] = {0, 0, 0, 0};          // visits, rows, chunks, buckets before this round
    for (long long p0 = 0; p0 < nt; p0 += 1024 * LAYOUT_PER) {
        const long long p = p0 + (long long)threadIdx.x * LAYOUT_PER;
        int r[LAYOUT_PER], d[LAYOUT_PER];
        long long vb[LAYOUT_PER];
#pragma unroll
        for (int i = 0; i < LAYOUT_PER; i++) {
            const long long pc = p + i < nt ? p + i : nt - 1;
            r[i] = list[pc];
            d[i] = prec[pc].d;
        }
#pragma unroll
        for (int i = 0; i < LAYOUT_PER; i++) vb[i] = vbound[r[i]];   // visits + own memberships + 1
        // row entries, chunks and buckets of node i
        auto parts = [&](int i, long long (&q)[4]) {
            const bool in = p + i < nt;
            const long long P = (vb[i] + BUCK_AVG - 1) / BUCK_AVG;
            q[0] = in ? vb[i] : 0;
            q[3] = !in ? 0 : P < TAB_MAXP ? P : TAB_MAXP;
            q[2] = in ? (d[i] - 1) / chunk_span(d[i]) + (d[i] > 0) : 0;
            q[1] = q[2] * (q[3] + 1);
        };
        long long sum[4] = {0, 0, 0, 0}, pos[4];
#pragma unroll
        for (int i = 0; i < LAYOUT_PER; i++) {
            long long q[4];
            parts(i, q);
#pragma unroll
            for (int k = 0; k < 4; k++) sum[k] += q[k];
            if (p + i < nt) tcur[p + i] = 0;
        }
#pragma unroll
        for (int k = 0; k < 4; k++) {
            pos[k] = sum[k];
#pragma unroll 1
            for (int o = 1; o < WAVE; o <<= 1) {
                const long long t = __shfl_up(pos[k], o, WAVE);
                if (lane >= o) pos[k] += t;
            }
        }
        __syncthreads();                                 // the round before has read s_w
        if (lane == WAVE - 1)
#pragma unroll
            for (int k = 0; k < 4; k++) s_w[k][wv] = pos[k];
        __syncthreads();
#pragma unroll
        for (int k = 0; k < 4; k++) pos[k] += at[k] - sum[k];
#pragma unroll 1
        for (int w = 0; w < 1024 / WAVE; w++)
#pragma unroll
            for (int k = 0; k < 4; k++) {
                const long long t = s_w[k][w];
                if (w < wv) pos[k] += t;
                at[k] += t;
            }
#pragma unroll
        for (int i = 0; i < LAYOUT_PER; i++) {
            if (p + i < nt) tpos[p + i] = TabPos{pos[0], pos[1], (int)pos[2], (int)pos[3]};
            long long q[4];
            parts(i, q);
#pragma unroll
            for (int k = 0; k < 4; k++) pos[k] += q[k];
        }
    }
    if (threadIdx.x == 0) tpos[nt] = TabPos{at[0], at[1], (int)at[2], (int)at[3]};
}

// the chunks and buckets of every table-path node (waves stride over the nodes; not written
// if they exceed the buffers: the host then grows them and runs this again), and the queues'
// first chunk, bucket, visit, row entry (out: four arrays of nq + 1) and in-count unit
__global__ void __launch_bounds__(256) k_table_fill(const int *list, const long long *lbase, long long ntiles,
                                                    const int *order, const long long *rowptr, const int *deg,
                                                    const TabPos *tpos, ChunkRec *chunk, long long chunk_cap,
                                                    BuckRec *buck, long long buck_cap, const long long *qoff_t,
                                                    long long nq, long long *out, const long long *ubase,
                                                    long long n, int q, long long *out_units)
{
    for (long long k = blockIdx.x * (long long)blockDim.x + threadIdx.x; k <= nq;
         k += (long long)gridDim.x * blockDim.x) {
        const TabPos t = tpos[qoff_t[k]];
        out[k] = t.chunk;
        out[nq + 1 + k] = t.bucket;
        out[2 * (nq + 1) + k] = t.vis;
        out[3 * (nq + 1) + k] = t.row;
        out_units[k] = ubase[k * q < n ? k * q : n];
    }
    const int *plist = list + lbase[0];
    const long long nt = lbase[ntiles] - lbase[0];
    if (tpos[nt].chunk > chunk_cap || tpos[nt].bucket > buck_cap) return;
    const int lane = threadIdx.x & (WAVE - 1);
    const long long nw = (long long)gridDim.x * (blockDim.x / WAVE);
    for (long long p = (blockIdx.x * (long long)blockDim.x + threadIdx.x) / WAVE; p < nt; p += nw) {
        const TabPos t0 = tpos[p], t1 = tpos[p + 1];
        const int r = plist[p], x = order[r], d = deg[x];
        const int nch = t1.chunk - t0.chunk, P = t1.bucket - t0.bucket;
        const long long rb = rowptr[x];
        const int span = chunk_span(d);
        for (int c = lane; c < nch; c += WAVE) {
            ChunkRec cr;
            cr.rb = rb + (long long)c * span;
            cr.vis = t0.vis;
            cr.row = t0.row + (long long)c * (P + 1);
            cr.cnt = d - c * span < span ? d - c * span : span;
            cr.p = (int)p;
            cr.P = P;
            cr.pad = 0;
            chunk[t0.chunk + c] = cr;
        }
        for (int b = lane; b < P; b += WAVE) {
            BuckRec br;
            br.vis = t0.vis;
            br.row = t0.row;
            br.x = x;
            br.d = d;
            br.nch = nch;
            br.P = P;
            br.b = b;
            br.pad = 0;
            buck[t0.bucket + b] = br;
        }
    }
}

// the membership lines of an iteration, from the slot layout (nodes whose capacity fits a
// line keep their memberships inline, the others point into the slot array)
__global__ void __launch_bounds__(256) k_line_build(Ctx cx, unsigned char *mc8)
{
    const long long x = blockIdx.x * (long long)blockDim.x + threadIdx.x;
    if (x >= cx.n) return;
    const NodeHdr hx = cx.nh[x];
    const long long cap = cx.nh[x + 1].off - hx.off;
    NodeLine l;
    l.cnt = hx.cnt;
    l.deg = hx.deg;
    l.off = cap <= LINE_SLOTS ? -1 : hx.off;
#pragma unroll
    for (int t = 0; t < LINE_SLOTS; t++) {
        Slot sl = {-1, 0};
        if (l.off < 0 && t < hx.cnt) sl = cx.slot[hx.off + t];
        l.s[t] = sl;
    }
    cx.ln[x] = l;
    mc8[x] = hx.cnt < 255 ? (unsigned char)hx.cnt : 255;
}

// in-count units of every node in node order (one per INB neighbours; ubase = their
// exclusive scan), and the first unit of every queue
__global__ void k_unit_counts(const int *order, const int *deg, long long n, long long *cnt)
{
    const long long r = blockIdx.x * (long long)blockDim.x + threadIdx.x;
    if (r < n) cnt[r] = (deg[order[r]] + INB - 1) / INB;
    else if (r == n) cnt[n] = 0;
}

__global__ void k_unit_fill(const int *order, const long long *rowptr, const int *deg, const long long *ubase,
                            long long n, UnitRec *unit, long long cap)
{
    const long long r = blockIdx.x * (long long)blockDim.x + threadIdx.x;
    if (r >= n) return;
    const int x = order[r], d = deg[x];
    const long long rb = rowptr[x], b = ubase[r];
    for (int k = 0; k * INB < d; k++) {
        if (b + k >= cap) break;            // cannot happen: cap bounds the total
        UnitRec u;
        u.rb = rb + (long long)k * INB;
        u.x = x;
        u.r = (int)r;
        u.cnt = d - k * INB < INB ? d - k * INB : INB;
        u.pad = 0;
        unit[b + k] = u;
    }
}

// ------------------------------------------------------------------------------------
// host side
// ------------------------------------------------------------------------------------
void lf_free_iteration_buffers(lf_handle *h)
{
    void **ptrs[] = {(void **)&h->dec, (void **)&h->unit, (void **)&h->part_rec, (void **)&h->psum,
                     (void **)&h->ubase, (void **)&h->tpos, (void **)&h->tcur, (void **)&h->tchunk,
                     (void **)&h->tbuck, (void **)&h->tvis, (void **)&h->trow, (void **)&h->tres,
                     (void **)&h->lhdr, (void **)&h->lpair, (void **)&h->ldeg};
    for (void **p : ptrs) {
        lf_dev_free(h, *p);
        *p = nullptr;
    }
    h->q_cap = 0;
    h->unit_cap = 0;
    h->static_ready = false;
    h->lines_ready = false;
    h->part_cap = 0;
    h->tchunk_cap = 0;
    h->tbuck_cap = 0;
    h->tvis_cap = 0;
    h->trow_cap = 0;
    h->tres_cap = 0;
    h->lhdr_cap = 0;
    h->lpair_cap = 0;
    h->ldeg_cap = 0;
}

// The iteration start's report (device dq, copied to the pinned host hqoff), for nq
// queues: per path the first list position of every queue ([LF_PATH_COUNT][nq + 1]), the
// first table-path chunk, bucket, visit and row entry of every queue, and the first
// in-count unit of every queue.
#define REP_TABLE(nq) ((long long)LF_PATH_COUNT * ((nq) + 1))
#define REP_UNITS(nq) ((long long)(LF_PATH_COUNT + 4) * ((nq) + 1))
#define REP_LEN(nq) ((long long)(LF_PATH_COUNT + 5) * ((nq) + 1))

static long long class_tiles(long long n) { return (n + CLS_TILE) / CLS_TILE; }   // covers position n

static void table_fill(lf_handle *h, long long q, long long nq)
{
    const long long nt = class_tiles(h->n);
    const long long *lbase = h->clsbase + LF_PATH_TABLE * nt;
    hipLaunchKernelGGL(k_table_fill, dim3(h->fill_grid), dim3(256), 0, h->stream, (const int *)h->plist_all, lbase, nt,
                       (const int *)h->order, (const long long *)h->rowptr, (const int *)h->deg,
                       (const TabPos *)h->tpos, h->tchunk, h->tchunk_cap, h->tbuck, h->tbuck_cap,
                       (const long long *)(h->dq + LF_PATH_TABLE * (nq + 1)), nq, h->dq + REP_TABLE(nq),
                       (const long long *)h->ubase, h->n, (int)q, h->dq + REP_UNITS(nq));
}

// Start of an iteration, first half: everything the host does not need to see, queued on
// the stream, ending with one copy of the queue offsets and bounds to pinned host memory.
// The second half (size_queue_complete) runs once that copy has landed.
static int size_queue_enqueue(lf_handle *h, long long q)
{
    TmpScope tmp_scope(h);
    hipStream_t st = h->stream;
    const int BS = 256;
    long long n = h->n;
    bool moved = false;
    if (!h->lists_ready) LF_TRY(lf_rebuild_member_lists(h));   // they did not fit at the last iteration end
    if (q > h->q_cap) {
        LF_TRY(lf_dev_regrow(h, (void **)&h->dec, &h->q_cap, q, sizeof(Decision)));
        moved = true;
    }
    const long long nq = (n + q - 1) / q;
    if (h->hqoff_cap < nq + 1) {            // pinned, so the one copy below is truly asynchronous
        // (the last copy into the old buffer was read by the previous iteration start)
        if (h->hqoff) lf_host_release(h->hqoff, sizeof(long long) * h->hqoff_len);
        h->hqoff = nullptr;
        h->hqoff_cap = 0;
        if (lf_host_alloc((void **)&h->hqoff, sizeof(long long) * REP_LEN(nq)) != LF_OK)
            return lf_set_error(h, LF_ENOMEM, "host queue offsets");
        h->hqoff_cap = nq + 1;
        h->hqoff_len = REP_LEN(nq);
    }
    const long long nrep = REP_LEN(nq);    // list offsets, table path, queue units
    if (nrep > h->dq_cap)                   // kept across the two halves (and iterations)
        LF_TRY(lf_dev_regrow(h, (void **)&h->dq, &h->dq_cap, nrep + nrep / 4 + 64, sizeof(long long)));
    long long *dq = h->dq;
    if (!h->ubase || !h->tpos || !h->tcur) {
        if (!h->ubase) LF_TRY(lf_dev_alloc(h, (void **)&h->ubase, sizeof(long long) * (n + 1)));
        if (!h->tpos) LF_TRY(lf_dev_alloc(h, (void **)&h->tpos, sizeof(TabPos) * (n + 1)));
        if (!h->tcur) LF_TRY(lf_dev_alloc(h, (void **)&h->tcur, sizeof(int) * (n + 1)));
        moved = true;
    }
    if (!h->tchunk) {
        LF_TRY(lf_dev_regrow(h, (void **)&h->tchunk, &h->tchunk_cap, 1024 + n / 16, sizeof(ChunkRec)));
        moved = true;
    }
    if (!h->tbuck) {
        LF_TRY(lf_dev_regrow(h, (void **)&h->tbuck, &h->tbuck_cap, 1024 + n / 8, sizeof(BuckRec)));
        moved = true;
    }
    const long long ucap = n + 2 * h->ne / INB + 1;   // >= sum of ceil(degree / INB)
    if (ucap > h->unit_cap) {
        h->static_ready = false;
        LF_TRY(lf_dev_regrow(h, (void **)&h->unit, &h->unit_cap, ucap, sizeof(UnitRec)));
        moved = true;
    }
    if (!h->lines) {
        LF_TRY(lf_dev_alloc(h, (void **)&h->lines, sizeof(NodeLine) * n));
        h->lines_ready = false;
        moved = true;
    }
    // the lines follow from the iteration end before; only a fresh partition builds them here
    if (!h->lines_ready)
        hipLaunchKernelGGL(k_line_build, dim3(grid_for(n, BS)), dim3(BS), 0, st, lf_ctx(h), h->mc8);
    h->lines_ready = true;
    // paths of this iteration
    const bool first = !h->static_ready;
    const dim3 bg(grid_for(n * NB_LANES, BS));
    const int wcap = h->eval_wave_cap < 2 * VSMALL ? h->eval_wave_cap : 2 * VSMALL;
    if (first)
        hipLaunchKernelGGL(k_node_bounds<true>, bg, dim3(BS), 0, st, lf_ctx(h), (const unsigned char *)h->mc8, h->pre,
                           h->vbound, h->cls, wcap, h->eval_med_cap, h->eval_grp_cap);
    else
        hipLaunchKernelGGL(k_node_bounds<false>, bg, dim3(BS), 0, st, lf_ctx(h), (const unsigned char *)h->mc8, h->pre,
                           h->vbound, h->cls, wcap, h->eval_med_cap, h->eval_grp_cap);
    const long long nt = class_tiles(n);
    hipLaunchKernelGGL(k_class_count, dim3((unsigned)nt), dim3(BS), 0, st, (const int *)h->cls, n, nt, h->clscnt);
    LF_TRY(lf_exclusive_scan_i32_to_i64(h, h->clscnt, h->clsbase, LF_PATH_COUNT * nt + 1));
    hipLaunchKernelGGL(k_class_place, dim3((unsigned)nt), dim3(BS), 0, st, (const int *)h->cls, n, nt,
                       (const long long *)h->clsbase, h->plist_all, h->prec_all, (int)q, nq, dq,
                       (const int *)h->order, (const long long *)h->rowptr, (const int *)h->deg);
    if (first) {                             // in-count units of every node in node order: they never change
        long long *ucnt = nullptr;
        LF_TRY(lf_tmp_alloc(h, (void **)&ucnt, sizeof(long long) * (n + 1)));
        hipLaunchKernelGGL(k_unit_counts, dim3(grid_for(n + 1, BS)), dim3(BS), 0, st, (const int *)h->order,
                           (const int *)h->deg, n, ucnt);
        LF_TRY(lf_exclusive_scan_i64(h, ucnt, h->ubase, n + 1));
        hipLaunchKernelGGL(k_unit_fill, dim3(grid_for(n, BS)), dim3(BS), 0, st, (const int *)h->order,
                           (const long long *)h->rowptr, (const int *)h->deg, (const long long *)h->ubase, n, h->unit,
                           h->unit_cap);
        h->static_ready = true;
    }
    // chunks and buckets of the table-path nodes, all on the device, and the queues' positions
    hipLaunchKernelGGL(k_table_layout, dim3(1), dim3(1024), 0, st, (const int *)h->plist_all,
                       (const NodeRec *)h->prec_all, (const long long *)(h->clsbase + LF_PATH_TABLE * nt), nt,
                       (const long long *)h->vbound, h->tpos, h->tcur);
    unsigned fill_grid = grid_for(n * WAVE, BS);
    if (fill_grid > 2048) fill_grid = 2048;
    h->fill_grid = fill_grid;
    table_fill(h, q, nq);
    // the host's one wait of the iteration start: list offsets per queue and path, the
    // queues' table-path and unit positions
    LF_HIP(h, hipMemcpyAsync(h->hqoff, dq, sizeof(long long) * nrep, hipMemcpyDeviceToHost, st));
    LF_HIP(h, hipGetLastError());
    h->pending_moved = moved;
    return LF_OK;
}

// whether a queue's small and medium nodes go through lists (the buffers are sized by this too)
static bool light_lists(bool batch, long long small, long long med)
{
    return batch || (small + EW - 1) / EW + med <= LIST_BLOCKS;
}

static int group_slice(bool batch) { return batch ? BATCH_GROUP_SLICE : GROUP_SLICE; }

// Entries of a batch member's lists at most, for queues of q nodes (the server reserves them).
long long lf_batch_list_bytes(long long q)
{
    const long long light = q < LIST_BLOCKS ? q : LIST_BLOCKS, group = q < BATCH_GROUP_SLICE ? q : BATCH_GROUP_SLICE;
    const long long entries = light * VMED + group * VGRP;
    return entries * (long long)(sizeof(long long) + sizeof(int)) + q * (long long)sizeof(ListHdr);
}

// second half: the host reads what the first half copied (the caller has waited for it)
// and grows whatever it found too small
static int size_queue_complete(lf_handle *h, long long q)
{
    hipStream_t st = h->stream;
    const int BS = 256;
    const long long n = h->n;
    const long long nq = (n + q - 1) / q;
    bool moved = h->pending_moved;
    h->second_half_work = false;
    {   // the records of path c start after those of the paths before it
        long long base = 0;
        for (int c = 0; c < LF_PATH_COUNT; c++) {
            h->prec[c] = h->prec_all + base;
            h->plist[c] = h->plist_all + base;
            base += h->hqoff[c * (nq + 1) + nq];
        }
    }
    // the queue with the largest table path sizes its buffers
    const long long *tb = h->hqoff + REP_TABLE(nq);
    long long most[4] = {0, 0, 0, 0};        // chunks, buckets, visits, row entries
    for (int a = 0; a < 4; a++)
        for (long long k = 0; k < nq; k++) {
            const long long v = tb[a * (nq + 1) + k + 1] - tb[a * (nq + 1) + k];
            if (v > most[a]) most[a] = v;
        }
    if (most[2] + 64 >= (1ll << 30))
        return lf_set_error(h, LF_EOVERFLOW, "queue of %lld nodes too large for the table path", q);
    const long long chunks = tb[nq], bucks = tb[2 * nq + 1];
    if (chunks > h->tchunk_cap || bucks > h->tbuck_cap) {   // rare: grow and lay them out again
        const long long f = h->phase_graphs ? 4 : 2;        // a batch member's graphs survive more growth
        if (chunks > h->tchunk_cap)
            LF_TRY(lf_dev_regrow(h, (void **)&h->tchunk, &h->tchunk_cap, f * chunks + 1024, sizeof(ChunkRec)));
        if (bucks > h->tbuck_cap)
            LF_TRY(lf_dev_regrow(h, (void **)&h->tbuck, &h->tbuck_cap, f * bucks + 1024, sizeof(BuckRec)));
        moved = true;
        table_fill(h, q, nq);
        LF_HIP(h, hipGetLastError());
        h->second_half_work = true;
    }
    // flattened lists of the queue with the most entries (its first slice has the most)
    long long lnodes = 0, lentries = 0;
    for (long long k = 0; k < nq; k++) {
        long long m[LF_PATH_COUNT];
        for (int c = 0; c < LF_PATH_COUNT; c++) m[c] = h->hqoff[c * (nq + 1) + k + 1] - h->hqoff[c * (nq + 1) + k];
        const bool lists = light_lists(h->phase_graphs, m[LF_PATH_SMALL], m[LF_PATH_MED]);
        long long light = lists ? m[LF_PATH_SMALL] + m[LF_PATH_MED] : 0;
        long long elight = lists ? m[LF_PATH_SMALL] * VSMALL + m[LF_PATH_MED] * VMED : 0;
        if (light > LIST_BLOCKS * EW) light = LIST_BLOCKS * EW;      // a slice's: a block has 256 entries,
        if (elight > LIST_BLOCKS * VMED) elight = LIST_BLOCKS * VMED;   // of four nodes or one
        const long long most = group_slice(h->phase_graphs);
        const long long group = m[LF_PATH_GROUP] < most ? m[LF_PATH_GROUP] : most;
        const long long nodes = light + group, entries = elight + group * VGRP;
        if (nodes > lnodes) lnodes = nodes;
        if (entries > lentries) lentries = entries;
    }
    struct { void **p; long long *cap; long long need; size_t each; } bufs[6] = {
        {(void **)&h->lhdr, &h->lhdr_cap, lnodes, sizeof(ListHdr)},
        {(void **)&h->lpair, &h->lpair_cap, lentries, sizeof(long long)},
        {(void **)&h->ldeg, &h->ldeg_cap, lentries, sizeof(int)},
        {(void **)&h->tres, &h->tres_cap, most[1], sizeof(BuckRes)},
        {(void **)&h->tvis, &h->tvis_cap, most[2], sizeof(TabVisit)},
        {(void **)&h->trow, &h->trow_cap, most[3], sizeof(int)}};
    for (auto &bf : bufs) {
        if (bf.need <= *bf.cap) continue;
        // a batch member's graphs survive more growth, while that is cheap
        long long spare = h->phase_graphs ? 3 * bf.need : 0;
        if (spare > SPARE_BYTES / (long long)bf.each) spare = SPARE_BYTES / (long long)bf.each;
        LF_TRY(lf_dev_regrow(h, bf.p, bf.cap, bf.need + bf.need / 4 + spare + 256, bf.each));
        moved = true;
    }
    long long pcap = 2 * q + (h->cm_cap + n) / PART + 64;
    if (pcap > h->part_cap) {
        if (h->phase_graphs) pcap *= 2;
        long long sums = 0;
        h->part_cap = 0;
        LF_TRY(lf_dev_regrow(h, (void **)&h->psum, &sums, pcap, sizeof(unsigned long long) * PSUM));
        LF_TRY(lf_dev_regrow(h, (void **)&h->part_rec, &h->part_cap, pcap, sizeof(PartRec)));
        moved = true;
    }
    if (moved) h->graph_version++;
    return LF_OK;
}

// Start of an iteration: buffers and path lists for queues of qq nodes, counters reset.
// lf_iter_begin_enqueue queues the work; lf_iter_begin_complete must follow once it is done
// (after a stream sync or a completed event recorded behind it).
static int begin_enqueue_plain(lf_handle *h, long long qq)
{
    return size_queue_enqueue(h, qq);
}

// ---- iteration starts and ends replayed from graphs --------------------------------
// A member of a batch repeats the same launch sequence at every iteration start (and end):
// the same buffers, sizes and temporaries, with only the slot buffer alternating.  A run
// that will allocate nothing (the host makes the run's own size checks first) is captured
// and later runs in the same state replay the graph: one host call for some thirty
// launches and copies.  The key covers whatever the launches bake in (the Ctx, every
// allocation, the temporaries' position, the options the start reads, the queue size and
// the slot parity); after a change the next run is captured again (the graph is updated
// in place).
static int finish_enqueue_plain(lf_handle *h);

static unsigned long long fnv_add(unsigned long long k, const void *p, size_t n)
{
    const unsigned char *b = (const unsigned char *)p;
    for (size_t i = 0; i < n; i++) k = (k ^ b[i]) * 1099511628211ull;
    return k;
}

static unsigned long long phase_key(lf_handle *h, long long qq, int which)
{
    unsigned long long k = 14695981039346656037ull;
    Ctx cx = lf_ctx(h);
    // the path lists' pointers move with the path counts at every start and are read only by
    // the queue kernels
    for (int c = 0; c < LF_PATH_COUNT; c++) {
        cx.prec[c] = nullptr;
        cx.plist[c] = nullptr;
    }
    k = fnv_add(k, &cx, sizeof cx);
    const long long v[] = {which, qq, h->cur, h->profiling, h->tmp_chunk, (long long)h->tmp_off,
                           h->eval_wave_cap, h->eval_med_cap, h->eval_grp_cap,
                           h->refresh_blocks, h->static_ready, h->lines_ready, (long long)h->allocs->size(), (long long)h->tmp_chunks->size()};
    k = fnv_add(k, v, sizeof v);
    k = fnv_add(k, h->allocs->data(), sizeof(void *) * h->allocs->size());
    k = fnv_add(k, h->alloc_sizes->data(), sizeof(size_t) * h->alloc_sizes->size());
    for (const TmpChunk &c : *h->tmp_chunks) k = fnv_add(k, &c, sizeof c);
    const void *hp[] = {h->hqoff, h->hrep};
    k = fnv_add(k, hp, sizeof hp);
    return k;
}

void lf_phase_graphs_drop(lf_handle *h)
{
    for (int a = 0; a < 2; a++)
        for (int b = 0; b < 2; b++) {
            if (h->pg[a][b].exec) (void)hipGraphExecDestroy(h->pg[a][b].exec);
            h->pg[a][b].exec = nullptr;
            h->pg[a][b].key = 0;
        }
}

// capture one plain run of the start (which = 0) or end (1) on the capture stream; the
// host-side effects of the run (slot parity, start bookkeeping) happen as in a plain run.
// *exec, if set, is updated in place when the new graph has its shape (a moved buffer
// changes only kernel arguments), else replaced.
static int capture_phase(lf_handle *h, int which, long long qq, hipGraphExec_t *exec)
{
    if (!h->cap_stream) LF_HIP(h, hipStreamCreateWithFlags(&h->cap_stream, hipStreamNonBlocking));
    hipStream_t saved = h->stream;
    LF_HIP(h, hipStreamBeginCapture(h->cap_stream, hipStreamCaptureModeThreadLocal));
    h->stream = h->cap_stream;
    int rc = which == 0 ? begin_enqueue_plain(h, qq) : finish_enqueue_plain(h);
    h->stream = saved;
    hipGraph_t g = nullptr;
    hipError_t e = hipStreamEndCapture(h->cap_stream, &g);
    if (rc == LF_OK && (e != hipSuccess || !g)) rc = lf_set_error(h, LF_EDEVICE, "iteration phase capture failed");
    if (rc == LF_OK && *exec) {
        hipGraphNode_t err_node = nullptr;
        hipGraphExecUpdateResult res;
        if (hipGraphExecUpdate(*exec, g, &err_node, &res) != hipSuccess || res != hipGraphExecUpdateSuccess) {
            (void)hipGetLastError();
            (void)hipGraphExecDestroy(*exec);
            *exec = nullptr;
        }
    }
    if (rc == LF_OK && !*exec && hipGraphInstantiate(exec, g, nullptr, nullptr, 0) != hipSuccess) {
        *exec = nullptr;
        rc = lf_set_error(h, LF_EDEVICE, "iteration phase graph instantiation failed");
    }
    if (g) (void)hipGraphDestroy(g);
    (void)hipGetLastError();
    return rc;
}

// whether a start (0) or end (1) would allocate: its size checks, made on the host
// beforehand (the temporaries it takes exist once it has run plainly)
static bool phase_allocates(lf_handle *h, int which, long long qq)
{
    if (!h->phase_ran[which]) return true;
    const long long n = h->n;
    if (which == 1) return !h->cm_node || h->slot_used + n + 1 > h->slot_capb[1 - h->cur];
    const long long nq = (n + qq - 1) / qq;
    const long long nrep = REP_LEN(nq);
    const long long ucap = n + 2 * h->ne / INB + 1;
    return !h->lists_ready || qq > h->q_cap || h->hqoff_cap < nq + 1 || nrep > h->dq_cap || !h->ubase || !h->tpos ||
           !h->tcur || !h->tchunk || !h->tbuck || ucap > h->unit_cap || (n > 0 && !h->lines);
}

static int run_plain(lf_handle *h, int which, long long qq)
{
    h->phase_runs[0]++;
    h->phase_ran[which] = 0;                 // (all of its temporaries exist only if it ran through)
    LF_TRY(which == 0 ? begin_enqueue_plain(h, qq) : finish_enqueue_plain(h));
    h->phase_ran[which] = 1;
    return LF_OK;
}

// one iteration start (0) or end (1), from a graph where the state allows
static int run_phase(lf_handle *h, int which, long long qq)
{
    if (!h->phase_graphs || h->profiling) return run_plain(h, which, qq);
    PhaseGraph &pg = h->pg[which][h->cur];
    const unsigned long long key = phase_key(h, qq, which);
    const bool allocates = phase_allocates(h, which, qq);
    if (!allocates && pg.exec && pg.key == key) {
        LF_HIP(h, hipGraphLaunch(pg.exec, h->stream));
        h->phase_runs[2]++;
        if (which == 0) {
            h->pending_moved = false;
            h->fill_grid = pg.fill_grid;
        } else {
            h->cur = 1 - h->cur;
        }
        return LF_OK;
    }
    if (!allocates) {
        LF_TRY(capture_phase(h, which, qq, &pg.exec));
        pg.key = key;
        pg.fill_grid = h->fill_grid;
        LF_HIP(h, hipGraphLaunch(pg.exec, h->stream));
        h->phase_runs[1]++;
        return LF_OK;
    }
    return run_plain(h, which, qq);
}

int lf_iter_begin_enqueue(lf_handle *h, long long qq) { return run_phase(h, 0, qq); }

// a failure here leaves the queues' changes without an iteration end: no partition to go on from
int lf_iter_finish_enqueue(lf_handle *h)
{
    const int rc = run_phase(h, 1, 0);
    if (rc != LF_OK) h->state = 1;
    return rc;
}

int lf_iter_begin_complete(lf_handle *h, long long qq, long long *nq)
{
    LF_TRY(size_queue_complete(h, qq));
    *nq = (h->n + qq - 1) / qq;
    return LF_OK;
}

int lf_iter_begin(lf_handle *h, long long qq, long long *nq)
{
    LF_TRY(lf_iter_begin_enqueue(h, qq));
    LF_HIP(h, hipStreamSynchronize(h->stream));
    return lf_iter_begin_complete(h, qq, nq);
}

// Parameters and grids of slice `slice` of queue k (of nq); returns the queue's slices.  The
// first one re-sums the queue before and takes all nodes but the workgroup path's beyond
// one slice of it (in a batch also the small and medium blocks beyond LIST_BLOCKS), the last
// one applies the queue.  compact_grids sizes the grid-stride kernels by
// the queue instead of by the whole device (for many graphs sharing one launch).
int lf_queue_params(lf_handle *h, long long k, long long nq, long long qq, bool compact_grids, int slice, QStep *qs,
                    QGrids *g)
{
    const long long *qo = h->hqoff;                                // [path][nq + 1]
    const long long *tb = h->hqoff + REP_TABLE(nq);    // [4][nq + 1]
    const long long *hu = h->hqoff + REP_UNITS(nq);    // first in-count unit per queue
    const long long start = k * qq;
    const int clen = (int)((h->n - start) < qq ? (h->n - start) : qq);
    int ls[LF_PATH_COUNT], ln[LF_PATH_COUNT];
    for (int c = 0; c < LF_PATH_COUNT; c++) {
        ls[c] = (int)qo[c * (nq + 1) + k];
        ln[c] = (int)(qo[c * (nq + 1) + k + 1] - ls[c]);
    }
    const bool lists = light_lists(compact_grids, ln[LF_PATH_SMALL], ln[LF_PATH_MED]);
    const int gs = group_slice(compact_grids), es = (int)grid_for(ln[LF_PATH_SMALL], EW), em = ln[LF_PATH_MED];
    int slices = ln[LF_PATH_GROUP] > gs ? (ln[LF_PATH_GROUP] - 1) / gs + 1 : 1;
    if (compact_grids && es + em > slices * LIST_BLOCKS) slices = (es + em - 1) / LIST_BLOCKS + 1;
    if (slices > 1) {
        // the slice's part [lo, hi) of `units` units of `per` nodes of a path
        auto cut = [&](int c, int lo, int hi, int units, int per) {
            lo = lo < 0 ? 0 : lo < units ? lo : units;
            hi = hi < 0 ? 0 : hi < units ? hi : units;
            const int end = hi * per < ln[c] ? hi * per : ln[c];
            ls[c] += lo * per;
            ln[c] = end > lo * per ? end - lo * per : 0;
        };
        cut(LF_PATH_GROUP, slice * gs, (slice + 1) * gs, ln[LF_PATH_GROUP], 1);
        if (compact_grids) {
            cut(LF_PATH_SMALL, slice * LIST_BLOCKS, (slice + 1) * LIST_BLOCKS, es, EW);
            cut(LF_PATH_MED, slice * LIST_BLOCKS - es, (slice + 1) * LIST_BLOCKS - es, em, 1);
        } else if (slice > 0) {
            ln[LF_PATH_SMALL] = ln[LF_PATH_MED] = 0;
        }
    }
    const int gb = h->hub_blocks;
    int rbk = RB_MORE * h->refresh_blocks;
    if (compact_grids) {
        int want = (int)grid_for(clen, 8);
        if (want < rbk) rbk = want;
    }
    if (slice > 0) rbk = 0;
    qs->cstart = (int)start;
    qs->clen = clen;
    qs->wcap = h->eval_wave_cap < 2 * VSMALL ? h->eval_wave_cap : 2 * VSMALL;
    qs->mcap = h->eval_med_cap;
    qs->gcap = h->eval_grp_cap;
    qs->ls = ls[LF_PATH_SMALL];
    qs->ln = ln[LF_PATH_SMALL];
    BigRoles &br = qs->br;
    br.c0 = (int)tb[k];
    br.nc = slice > 0 ? 0 : (int)(tb[k + 1] - tb[k]);
    br.b0 = (int)tb[nq + 1 + k];
    br.nb = slice > 0 ? 0 : (int)(tb[nq + 2 + k] - tb[nq + 1 + k]);
    br.vis0 = tb[2 * (nq + 1) + k];
    br.row0 = tb[3 * (nq + 1) + k];
    br.bt = br.nc < 4 * gb ? br.nc : 4 * gb;
    br.bg = ln[LF_PATH_GROUP] < 4 * gb ? ln[LF_PATH_GROUP] : 4 * gb;
    qs->es = (int)grid_for(ln[LF_PATH_SMALL], EW);
    qs->em = ln[LF_PATH_MED];
    qs->lm = ls[LF_PATH_MED];
    br.lt = ls[LF_PATH_TABLE];
    br.nt = ln[LF_PATH_TABLE];
    br.lg = ls[LF_PATH_GROUP];
    br.ng = ln[LF_PATH_GROUP];
    qs->ub = hu[k];
    qs->un = (int)(hu[k + 1] - hu[k]);
    qs->rb = rbk;
    const int light = qs->es + qs->em, heavy = br.bg + br.nb;
    qs->lists = lists;
    const bool fuse = compact_grids || (heavy > 0 && qs->lists);
    g->refresh = rbk + br.bt + br.bg + (qs->lists ? light : 0);
    g->eval = fuse ? 0 : light;
    g->big = heavy + (fuse ? light : 0);
    if (g->big < 1 && g->eval == 0) g->big = 1;   // block 0 resets the queue's counters
    const bool last = slice == slices - 1;
    g->tie = last ? (int)grid_for(br.nt, GT / WAVE) : 0;
    g->apply = last ? (int)grid_for(clen, EDITS) + (int)grid_for(qs->un, 256 / WAVE) : 0;
    return slices;
}

// the kernels of one slice of a queue of one graph, in order, on the handle's stream
static void launch_refresh(int grid, hipStream_t st, const Ctx &cx, const QStep &qs)
{
    hipLaunchKernelGGL(k_refresh, dim3(grid), dim3(GT), 0, st, qs.rb, qs.br.bt, qs.br.bg, qs.em, cx.part_rec, cx.ctr,
                       cx.prec[LF_PATH_SMALL] + qs.ls, cx.plist[LF_PATH_SMALL] + qs.ls, cx, qs);
}

int lf_launch_queue(lf_handle *h, Ctx &cx, const QStep &qs, const QGrids &g)
{
    hipStream_t st = h->stream;
    LF_TRY(lf_prof_begin(h, LF_K_REFRESH));
    launch_refresh(g.refresh, st, cx, qs);
    LF_TRY(lf_prof_end(h, LF_K_REFRESH, 1));
    if (g.eval > 0) {
        LF_TRY(lf_prof_begin(h, LF_K_EVAL));
        if (qs.lists) hipLaunchKernelGGL(k_eval, dim3(g.eval), dim3(EW * WAVE), 0, st, qs.es, qs.ln, qs.em,
                                         cx.lhdr, cx.lpair, cx.ldeg, cx, qs);
        else hipLaunchKernelGGL(k_eval_whole, dim3(g.eval), dim3(EW * WAVE), 0, st, cx, qs);
        LF_TRY(lf_prof_end(h, LF_K_EVAL, 1));
    }
    if (g.big > 0) {
        LF_TRY(lf_prof_begin(h, LF_K_EVAL_BIG));
        const int bg = qs.br.bg, mid = g.big - bg;
        const bool split = mid > SPLIT_BLOCKS;
        if (!split || bg > 0) hipLaunchKernelGGL(k_eval_big, dim3(split ? bg : g.big), dim3(GT), 0, st, cx, qs);
        if (split) hipLaunchKernelGGL(k_eval_mid, dim3(mid), dim3(GT), 0, st, cx, qs);
        LF_TRY(lf_prof_end(h, LF_K_EVAL_BIG, split && bg > 0 ? 2 : 1));
    }
    if (g.tie > 0) {
        LF_TRY(lf_prof_begin(h, LF_K_TAB_TIE));
        hipLaunchKernelGGL(k_big_tie, dim3(g.tie), dim3(GT), 0, st, cx, qs);
        LF_TRY(lf_prof_end(h, LF_K_TAB_TIE, 1));
    }
    if (g.apply == 0) return LF_OK;
    LF_TRY(lf_prof_begin(h, LF_K_APPLY_EDIT));
    hipLaunchKernelGGL(k_apply, dim3(g.apply), dim3(256), 0, st, cx.unit + qs.ub, qs.un, qs.clen, cx.dec,
                       cx.order + qs.cstart, cx, qs);
    LF_TRY(lf_prof_end(h, LF_K_APPLY_EDIT, 1));
    h->prof.chunks++;
    h->prof.node_evals += qs.clen;
    return LF_OK;
}

// One queue of each of several graphs: four grids, each block finding its graph from dboff
// (LF_MULTI_GRIDS arrays of n first-block offsets); total[i] = blocks of grid i.
int lf_launch_multi(hipStream_t st, const Member *dmem, const int *dboff, int n, const int *total)
{
    const int *o = dboff;
    if (total[0] > 0) hipLaunchKernelGGL(k_refresh_multi, dim3(total[0]), dim3(GT), 0, st, dmem, o, n);
    o += n;
    if (total[1] > 0) hipLaunchKernelGGL(k_eval_big_multi, dim3(total[1]), dim3(GT), 0, st, dmem, o, n);
    o += n;
    if (total[2] > 0) hipLaunchKernelGGL(k_big_tie_multi, dim3(total[2]), dim3(GT), 0, st, dmem, o, n);
    o += n;
    if (total[3] > 0) hipLaunchKernelGGL(k_apply_multi, dim3(total[3]), dim3(256), 0, st, dmem, o, n);
    return hipGetLastError() == hipSuccess ? LF_OK : LF_EDEVICE;
}

// The multi-graph kernels in launch order, the grid each uses and its block size, for
// building a graph of one batch step.
void lf_multi_kernels(const void **fn, int *grid, int *block)
{
    const void *f[LF_MULTI_KERNELS] = {(const void *)k_refresh_multi, (const void *)k_eval_big_multi,
                                       (const void *)k_big_tie_multi, (const void *)k_apply_multi};
    const int b[LF_MULTI_KERNELS] = {GT, GT, GT, 256};
    for (int i = 0; i < LF_MULTI_KERNELS; i++) {
        fn[i] = f[i];
        grid[i] = i;
        block[i] = b[i];
    }
}

// the re-sums of the last queue applied (no next queue to gather)
static void refresh_alone(lf_handle *h)
{
    QStep qs;
    memset(&qs, 0, sizeof qs);
    qs.rb = RB_MORE * h->refresh_blocks;
    launch_refresh(qs.rb, h->stream, lf_ctx(h), qs);
}

// End of an iteration: counters reset, degenerate communities removed, exact score.
// End of an iteration, in the same two halves as its start.
// A batch member leaves within an iteration, first half (queued): the queues applied so far
// stand, and what an iteration end leaves is made from them, but for the removal of small
// communities (a warm start may have them too): slots without holes and with one cleared free
// slot per node, member lists without those who left and with those who did not fit, scores.
// lf_iter_finish_complete is the second half.
int lf_iter_leave_enqueue(lf_handle *h)
{
    refresh_alone(h);
    int rc = lf_iteration_end_enqueue(h, 0);
    if (rc != LF_OK) h->state = 1;
    return rc;
}

static int finish_enqueue_plain(lf_handle *h)
{
    refresh_alone(h);
    LF_HIP(h, hipGetLastError());
    LF_TRY(lf_prof_begin(h, LF_K_ITEREND));
    LF_TRY(lf_iteration_end_enqueue(h, 2));
    LF_TRY(lf_prof_end(h, LF_K_ITEREND, 8));
    return LF_OK;
}

int lf_iter_finish_complete(lf_handle *h, long long *joins, long long *leaves, long long *live)
{
    LF_TRY(lf_iteration_end_complete(h, joins, leaves, live));
    return lf_dev_error_status(h, h->last_dev_error);   // the flags came with the iteration-end report
}

int lf_iter_finish(lf_handle *h, long long *joins, long long *leaves, long long *live)
{
    LF_TRY(lf_iter_finish_enqueue(h));
    LF_HIP(h, hipStreamSynchronize(h->stream));
    return lf_iter_finish_complete(h, joins, leaves, live);
}

int lf_iterate(lf_handle *h, int q, double theta, int max_iters, lf_run_info *out)
{
    long long n = h->n;
    lf_run_info dummy;
    memset(&dummy, 0, sizeof dummy);
    if (!out) out = &dummy;
    out->iterations = 0;
    out->converged = 0;
    out->hit_max = 0;
    if (out->wtilde_hist) out->wtilde_hist[0] = h->Wt;
    if (h->cc == 0.0) {
        out->converged = 1;
        out->wtilde = h->Wt;
        out->wcc_hat = 0.0;
        return LF_OK;
    }
    long long qq = q < n ? q : (n > 0 ? n : 1);
    double prev = h->Wt;
    for (int it = 0; it < max_iters; it++) {
        long long nq = 0;
        LF_TRY(lf_iter_begin(h, qq, &nq));
        Ctx cx = lf_ctx(h);
        for (long long k = 0; k < nq; k++) {
            QStep qs;
            QGrids g;
            for (int slice = 0, slices = 1; slice < slices; slice++) {
                slices = lf_queue_params(h, k, nq, qq, false, slice, &qs, &g);
                const int rc = lf_launch_queue(h, cx, qs, g);
                if (rc != LF_OK) {               // queues applied in part: no partition to go on from
                    h->state = 1;
                    return rc;
                }
            }
        }
        long long joins = 0, leaves = 0, live = 0;
        LF_TRY(lf_iter_finish(h, &joins, &leaves, &live));
        out->iterations = it + 1;
        if (out->wtilde_hist) out->wtilde_hist[it + 1] = h->Wt;
        if (out->joins) out->joins[it] = joins;
        if (out->leaves) out->leaves[it] = leaves;
        if (out->communities) out->communities[it] = live;
        bool stop = (prev == 0.0) || ((h->Wt - prev) / prev < theta);
        prev = h->Wt;
        if (stop) {
            out->converged = 1;
            break;
        }
    }
    if (!out->converged && out->iterations == max_iters) out->hit_max = 1;
    LF_TRY(lf_prof_flush(h));
    {
        unsigned long long w[LF_PATH_COUNT][5], aw[LF_APPLY_COUNT];
        LF_HIP(h, hipMemcpy(w, h->ctr->work, sizeof(w), hipMemcpyDeviceToHost));
        LF_HIP(h, hipMemcpy(aw, h->ctr->apply, sizeof(aw), hipMemcpyDeviceToHost));
        for (int k = 0; k < LF_APPLY_COUNT; k++) h->prof.apply_work[k] = (long long)aw[k];
        h->prof.visits = 0;
        h->prof.candidates = 0;
        for (int p = 0; p < LF_PATH_COUNT; p++) {
            h->prof.path_nodes[p] = (long long)w[p][0];
            h->prof.path_neighbours[p] = (long long)w[p][1];
            h->prof.path_visits[p] = (long long)w[p][2];
            h->prof.path_candidates[p] = (long long)w[p][3];
            h->prof.path_own[p] = (long long)w[p][4];
            h->prof.visits += (long long)w[p][2];
            h->prof.candidates += (long long)w[p][3];
        }
    }
    out->wtilde = h->Wt;
    out->wcc_hat = h->Wt / h->cc;
    lf_trim_kept(h);
    return LF_OK;
}
