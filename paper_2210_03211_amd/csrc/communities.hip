// communities.hip -- initial clustering and LazyFox iterations on the GPU.
//
// Method (Garrels et al., arXiv 2210.03211, Methods):
//  * Initial clustering: in node order, a node without a community opens a new one and its
//    unassigned neighbours join it.  Equivalently, the openers are the lexicographically
//    first maximal independent set in rank order, and every other node joins the
//    lowest-ranked opener among its neighbours; community ids number the openers by rank.
//    The GPU decides openers in rounds (a node is decided once all lower-ranked neighbours
//    are), resuming each node's neighbour scan where it stopped.
//  * WCC-hat (WCC-hat subsection): for a member x of C with d = deg(x,V), i = deg(x,C),
//    s = |C| and community density p, WCC-hat(x,C) = p * g(i,d,s) / cc with
//    g = i(i-1) / ((d-1)(s-1+d-i)) (0 if i < 2 or d < 2).  cc > 0 scales every term alike,
//    so all decisions use the cc-free community score W(C) = fl(p * R(sum_y g)), R = exact
//    sum rounded once.
//  * Node changes (Algorithm 2): for every node x of a queue, on the state at the start of
//    the queue, the change of W(C) when x joins a community C of a neighbour (or leaves one
//    of its own).  With stored exact sums S+ = sum g(i_y, d_y, s+1) and
//    S- = sum g(i_y, d_y, s-1) over C's members, only x's neighbours in C change their in-
//    count, so
//      join:  W' = p(s+1, m+k) * R(S+ + sum_{y in N(x)∩C} [g(i_y+1,..,s+1) - g(i_y,..,s+1)]
//                                     + g(k, d_x, s+1))
//      leave: W' = p(s-1, m-k) * R(S- + sum_{y in N(x)∩C} [g(i_y-1,..,s-1) - g(i_y,..,s-1)]
//                                     - g(k, d_x, s-1))
//    with k = |N(x) ∩ C|.  A move is taken if W' - W(C) > 0, the largest wins, ties go to
//    the lowest community id; the best join and the best leave are both applied.
//  * Bulk apply: membership edits, community sizes, in-counts of the affected neighbours
//    (integer atomics; a node that joined in this queue is counted afresh), then an exact
//    re-sum of every touched community (size changes alter every member's term).
//  * Iteration end: communities with < 2 members are removed, membership slots compacted
//    (+1 free slot per node: a node gains at most one community per iteration), member
//    lists rebuilt and the exact partition score reduced.
//
// Layout in HBM: CSR (rowptr int64, col int32); per node a 16-byte header {slot offset,
// count, degree} and, within an iteration, a 64-byte line with up to six memberships;
// membership slots {community, in-count} (8 bytes); per community one 64-byte record (size,
// internal edges, score, S+ and S- as 160-bit fixed point); member lists with per-community
// capacity for the iteration's joiners (overflow goes to a global list).
#include "method.h"

static inline unsigned grid_for(long long n, int block) { return (unsigned)((n + block - 1) / block); }

// ------------------------------------------------------------------------------------
// A3: initial clustering
// ------------------------------------------------------------------------------------
// state: 0 undecided, 1 opener, 2 joins an opener.  An undecided node looks at its neighbours
// earlier in the order from where it stopped last: an opener among them decides it, the first
// undecided one ends the round for it, and when none is left it opens.  A thread looks at
// LFMIS_OWN neighbours, four per round trip; the wave takes over the nodes that have more, 256
// neighbours per round trip.  A state read from the cache may be older than the round, which
// only delays the node.  Whether any node is left is a plain store: counted with an atomic per
// wave on one address, a round took as long as 15,600 of them in a row.  1M nodes, 8M edges:
// 195 us for each of 15 rounds -> 81 us for the first and less for each after it, all of
// them 2.8 -> 0.44 ms; 4M nodes, 35M edges 5.0 -> 1.4 ms.
#define LFMIS_OWN 16
__device__ __forceinline__ int lfmis_state(const int *state, int y)
{
    return __hip_atomic_load(&state[y], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

__global__ void __launch_bounds__(256) k_lfmis_round(const long long *rowptr, const int *col, const int *col_rank,
                                                     const int *rank, long long n, int *state, int *cursor,
                                                     int *undecided)
{
    const int lane = threadIdx.x & (WAVE - 1);
    bool left = false;
    for (long long x0 = blockIdx.x * (long long)blockDim.x + (threadIdx.x - lane); x0 < n;
         x0 += (long long)gridDim.x * blockDim.x) {
        const long long x = x0 + lane;
        const bool open = x < n && lfmis_state(state, (int)x) == 0;
        if (!__ballot(open)) continue;
        int rx = 0, mine = 0;
        long long b = 0, c = 0, e = 0;
        bool pending = false;
        if (open) {
            rx = rank[x];
            b = rowptr[x];
            e = rowptr[x + 1];
            c = b + cursor[x];
        }
        const long long own = c + LFMIS_OWN < e ? c + LFMIS_OWN : e;
        while (c < own && mine == 0 && !pending) {
            int ry[4], sy[4];
#pragma unroll
            for (int k = 0; k < 4; k++) {
                const long long q = c + k < own ? c + k : own - 1;
                ry[k] = col_rank[q];
                sy[k] = lfmis_state(state, col[q]);
            }
            long long next = c + 4 < own ? c + 4 : own;
#pragma unroll
            for (int k = 3; k >= 0; k--) {       // the first undecided one, unless an opener is among them
                if (c + k >= own || ry[k] >= rx) continue;
                if (sy[k] == 1) mine = 2;
                if (sy[k] == 0) {
                    pending = true;
                    next = c + k;
                }
            }
            if (mine) pending = false;
            c = next;
        }
        WAVE_SYNC();
        unsigned long long more = __ballot(open && mine == 0 && !pending && c < e);
        while (more) {
            const int src = __ffsll((long long)more) - 1;
            more &= more - 1;
            const int rs = __shfl(rx, src, WAVE);
            const long long es = __shfl(e, src, WAVE);
            long long q = __shfl(c, src, WAVE);
            int got = 0;
            bool wait = false;
            for (; q < es && got == 0 && !wait; q += 4 * WAVE) {
                int ry[4], sy[4];
#pragma unroll
                for (int k = 0; k < 4; k++) {
                    const long long p = q + k * WAVE + lane < es ? q + k * WAVE + lane : es - 1;
                    ry[k] = col_rank[p];
                    sy[k] = lfmis_state(state, col[p]);
                }
                long long stop = -1;
#pragma unroll
                for (int k = 3; k >= 0; k--) {   // (the clamped last entry changes nothing)
                    const unsigned long long o = __ballot(ry[k] < rs && sy[k] == 1);
                    const unsigned long long u = __ballot(ry[k] < rs && sy[k] == 0);
                    if (o) got = 2;
                    if (u) stop = q + k * WAVE + __ffsll((long long)u) - 1;
                }
                if (got == 0 && stop >= 0) {
                    wait = true;
                    q = (stop < es ? stop : es - 1) - 4 * WAVE;
                }
            }
            if (lane == src) {
                c = q < es ? q : es;
                mine = got;
                pending = wait;
            }
            WAVE_SYNC();
        }
        if (open) {
            cursor[x] = (int)(c - b);
            if (mine == 0 && !pending) mine = 1;
            if (mine) __hip_atomic_store(&state[x], mine, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            else left = true;
        }
        WAVE_SYNC();
    }
    if (__ballot(left) && lane == 0) *undecided = 1;
}

__global__ void k_opener_flags(const int *order, const int *state, long long n, int *flag)
{
    long long r = blockIdx.x * (long long)blockDim.x + threadIdx.x;
    if (r >= n) return;
    flag[r] = state[order[r]] == 1;
}

__global__ void k_opener_ids(const int *order, const int *flag, const long long *pos, long long n, int *comm_of)
{
    long long r = blockIdx.x * (long long)blockDim.x + threadIdx.x;
    if (r >= n) return;
    if (flag[r]) comm_of[order[r]] = (int)pos[r];
}

// every non-opener joins its lowest-ranked opener neighbour
__global__ void __launch_bounds__(256) k_join_openers(const long long *rowptr, const int *col, const int *col_rank,
                                                      const int *order, const int *state, long long n, int *comm_of)
{
    for_rows(n, [&](long long x) { return rowptr[x + 1] - rowptr[x]; }, [&](long long x, int sub, int width) {
        const bool joins = x >= 0 && state[x] == 2;
        unsigned best = 0x7fffffff;
        if (joins) {
            const long long r1 = rowptr[x + 1];
            for (long long e = rowptr[x] + sub; e < r1; e += width) {
                const unsigned r = (unsigned)col_rank[e];
                if (r < best && state[col[e]] == 1) best = r;
            }
        }
        WAVE_SYNC();
        best = 0x7fffffffu - best;
        best = 0x7fffffffu - (width == 16 ? row_max_u32(best) : wave_max_u32(best));
        if (joins && sub == width - 1) comm_of[x] = comm_of[order[best]];
    });
}

// one membership per node plus one free slot; in-count within its community
__global__ void __launch_bounds__(256) k_init_slots(const long long *rowptr, const int *col, const int *deg,
                                                    const int *comm_of, long long n, NodeHdr *nh, Slot *slot,
                                                    CommRec *cr)
{
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        nh[n].off = 2 * n;
        nh[n].cnt = 0;
        nh[n].deg = 0;
    }
    for_rows(n, [&](long long x) { return rowptr[x + 1] - rowptr[x]; }, [&](long long x, int sub, int width) {
        int c = 0, in = 0;
        if (x >= 0) {
            c = comm_of[x];
            const long long r1 = rowptr[x + 1];
            for (long long e = rowptr[x] + sub; e < r1; e += width) in += comm_of[col[e]] == c;
        }
        WAVE_SYNC();
        in = width == 16 ? (int)row_sum_u32((unsigned)in) : (int)wave_sum_u32((unsigned)in);
        if (x >= 0 && sub == width - 1) {
            NodeHdr hd;
            hd.off = 2 * x;
            hd.cnt = 1;
            hd.deg = deg[x];
            nh[x] = hd;
            Slot s0 = {c, in}, s1 = {-1, 0};
            slot[2 * x] = s0;
            slot[2 * x + 1] = s1;
            atomicAdd(&cr[c].s, 1);
        }
    });
}

// warm start: checks of a given cover: offsets non-decreasing within [0, total] (bit 0), ids in
// [0, K) (bit 1; K < 0: any id >= 0), no id twice per node (bit 2); chk[1] = largest id.  A
// thread per node, a wave for those with more than CHECK_OWN ids, one atomic per block at the
// end (a wave per node, and one atomic each: 206 us for 1M nodes, now 23).
#define CHECK_OWN 16
__global__ void __launch_bounds__(256) k_cover_check(const long long *off, const int *ids, long long n,
                                                     long long total, int K, int *chk)
{
    __shared__ int s_err[256 / WAVE], s_mx[256 / WAVE];
    const int lane = threadIdx.x & (WAVE - 1);
    int err = 0, mx = -1;
    // one id against the range and those before it in the list
    auto check = [&](long long a0, long long a) {
        const int c = ids[a];
        if (c < 0 || (K >= 0 && c >= K)) err |= 2;
        if (c > mx) mx = c;
        for (long long b = a0; b < a; b++) err |= ids[b] == c ? 4 : 0;
    };
    for (long long x0 = blockIdx.x * (long long)blockDim.x + (threadIdx.x - lane); x0 < n;
         x0 += (long long)gridDim.x * blockDim.x) {
        const long long x = x0 + lane;
        const long long a0 = x < n ? off[x] : 0, a1 = x < n ? off[x + 1] : 0;
        const bool bad = a0 < 0 || a1 < a0 || a1 > total;
        if (bad) err |= 1;
        const bool own = !bad && a1 - a0 <= CHECK_OWN;
        for (long long a = a0; own && a < a1; a++) check(a0, a);
        for (unsigned long long rest = __ballot(!bad && !own); rest; rest &= rest - 1) {
            const int src = __ffsll((long long)rest) - 1;
            const long long w0 = __shfl(a0, src, WAVE), w1 = __shfl(a1, src, WAVE);
            for (long long a = w0 + lane; a < w1; a += WAVE) check(w0, a);
            WAVE_SYNC();
        }
    }
    for (int o = 32; o >= 1; o >>= 1) err |= __shfl_xor(err, o, WAVE);
    mx = (int)wave_max_u32((unsigned)(mx + 1)) - 1;
    if (lane == 0) {
        s_err[threadIdx.x / WAVE] = err;
        s_mx[threadIdx.x / WAVE] = mx;
    }
    __syncthreads();
    if (threadIdx.x != 0) return;
    for (int w = 1; w < 256 / WAVE; w++) {
        err |= s_err[w];
        mx = s_mx[w] > mx ? s_mx[w] : mx;
    }
    if (err) atomicOr(&chk[0], err);
    if (mx >= 0) atomicMax(&chk[1], mx);
}

// warm start: node x's memberships in the given order plus one free slot (slot offset
// off[x] + x); in-count of each = neighbours whose cover lists the community; sizes.
// A row of lanes per node (a wave for the longest; 0.61 -> 0.46 ms for 700,000 nodes); a pass over
// the neighbours' lists counts up to COVER_CHUNK of x's communities at once (a node's ids are distinct, so each neighbour adds at most one to
// each count), so a node with few memberships gathers its neighbourhood once.
#define COVER_CHUNK 8
__global__ void __launch_bounds__(256) k_cover_slots(const long long *rowptr, const int *col, const int *deg,
                                                     const long long *off, const int *ids, long long n, NodeHdr *nh,
                                                     Slot *slot, CommRec *cr)
{
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        nh[n].off = off[n] + n;
        nh[n].cnt = 0;
        nh[n].deg = 0;
    }
    for_rows(n, [&](long long x) { return rowptr[x + 1] - rowptr[x]; }, [&](long long x, int sub, int width) {
        const long long a0 = x >= 0 ? off[x] : 0;
        const int cnt = x >= 0 ? (int)(off[x + 1] - a0) : 0;
        const long long base = a0 + x;
        const long long e0 = x >= 0 ? rowptr[x] : 0, e1 = x >= 0 ? rowptr[x + 1] : 0;
        for (int a = 0; __ballot(a < cnt); a += COVER_CHUNK) {
            const int m = cnt - a < COVER_CHUNK ? cnt - a : COVER_CHUNK;   // (below 1: none left)
            int c[COVER_CHUNK], in[COVER_CHUNK];
#pragma unroll
            for (int k = 0; k < COVER_CHUNK; k++) {
                c[k] = k < m ? ids[a0 + a + k] : -1;   // ids are >= 0: -1 matches nothing
                in[k] = 0;
            }
            for (long long e = m > 0 ? e0 + sub : e1; e < e1; e += width) {
                const int z = col[e];
                const long long b1 = off[z + 1];
                for (long long b = off[z]; b < b1; b++) {
                    const int d = ids[b];
#pragma unroll
                    for (int k = 0; k < COVER_CHUNK; k++) in[k] += d == c[k];
                }
            }
            WAVE_SYNC();
#pragma unroll
            for (int k = 0; k < COVER_CHUNK; k++) {
                if (!__ballot(k < m)) break;
                const int t = width == 16 ? (int)row_sum_u32((unsigned)in[k]) : (int)wave_sum_u32((unsigned)in[k]);
                if (k < m && sub == width - 1) {
                    Slot sl = {c[k], t};
                    slot[base + a + k] = sl;
                    atomicAdd(&cr[c[k]].s, 1);
                }
            }
            WAVE_SYNC();
        }
        if (x >= 0 && sub == width - 1) {
            NodeHdr hd;
            hd.off = base;
            hd.cnt = cnt;
            hd.deg = deg[x];
            nh[x] = hd;
            Slot free_slot = {-1, 0};
            slot[base + cnt] = free_slot;
        }
    });
}

// ------------------------------------------------------------------------------------
// member lists (rebuilt at initialisation and at every iteration end)
// ------------------------------------------------------------------------------------
// capacity: current members plus room for joiners (sum of member degrees, at most n)
__global__ void k_member_extra(const NodeHdr *nh, const Slot *slot, long long n, long long *capx)
{
    long long x = blockIdx.x * (long long)blockDim.x + threadIdx.x;
    if (x >= n) return;
    NodeHdr hd = nh[x];
    for (int t = 0; t < hd.cnt; t++) atomicAdd((unsigned long long *)&capx[slot[hd.off + t].comm], (unsigned long long)hd.deg);
}

__global__ void k_member_cap(long long *capx, const CommRec *cr, int K, long long n)
{
    long long c = blockIdx.x * (long long)blockDim.x + threadIdx.x;
    if (c >= K) return;
    long long ex = capx[c];
    if (ex > n) ex = n;
    capx[c] = cr[c].s + ex;
}

__global__ void k_member_fill(const NodeHdr *nh, const Slot *slot, long long n, int K, const long long *cm_off,
                              int *cm_len, int *cm_node, long long cap)
{
    long long x = blockIdx.x * (long long)blockDim.x + threadIdx.x;
    if (x >= n || cm_off[K] > cap) return;          // over capacity: the host grows it and refills
    NodeHdr hd = nh[x];
    for (int t = 0; t < hd.cnt; t++) {
        int c = slot[hd.off + t].comm;
        int p = atomicAdd(&cm_len[c], 1);
        cm_node[cm_off[c] + p] = (int)x;
    }
}

// ------------------------------------------------------------------------------------
// exact re-sum of every community
// ------------------------------------------------------------------------------------
// Most communities have some ten members, so a row of 16 lanes sums one; those of more than
// ROW_MEMBERS, or with joiners that did not fit their list, are left to the whole wave.  With a
// wave for each, most lanes idle and three 192-bit reductions through LDS: 0.72 -> 0.09 ms
// for the clusters of 1M nodes, 2.29 -> 0.37 ms for those of 4M.
#define ROW_MEMBERS 64
__global__ void __launch_bounds__(256) k_refresh_list(Ctx cx, int count)
{
    const int lane = threadIdx.x & (WAVE - 1), sub = lane & 15;
    const long long nw = (long long)gridDim.x * (blockDim.x / WAVE);
    int bad = 0;
    for (long long i0 = (blockIdx.x * (long long)blockDim.x + threadIdx.x) / WAVE * 4; i0 < count; i0 += 4 * nw) {
        const bool in = i0 + lane / 16 < count;
        const int C = in ? (int)i0 + lane / 16 : (int)i0;
        const int s = cx.cr[C].s;
        const long long base = cx.cm_off[C], cap = cx.cm_off[C + 1] - base;
        const int fill = cx.cm_len[C], ovf = cx.ovf_flag[C];
        const long long len = fill < cap ? fill : cap;
        const bool row = in && len <= ROW_MEMBERS && !ovf;
        u128 a0 = 0, ap = 0, am = 0;
        long long sumi = 0;
        for (long long j = sub; row && j < len; j += 16)
            member_terms(cx, cx.cm_node[base + j], C, s, a0, ap, am, sumi, bad);
        WAVE_SYNC();
        const X192 S0 = row_sum_u128(a0), Sp = row_sum_u128(ap), Sm = row_sum_u128(am);
        const long long ins = (long long)row_sum_u32((unsigned)sumi & 0xffffffu) +
                              ((long long)row_sum_u32((unsigned)(sumi >> 24)) << 24);
        if (row && sub == 15) store_comm(cx, C, s, S0, Sp, Sm, ins, bad);
        WAVE_SYNC();
        unsigned long long rest = __ballot(in && !row && sub == 0);
        while (rest) {
            const int src = __ffsll((long long)rest) - 1;
            rest &= rest - 1;
            const int Cw = __shfl(C, src, WAVE), sw = __shfl(s, src, WAVE);
            const long long bw = __shfl(base, src, WAVE), lw = __shfl(len, src, WAVE);
            X192 b0 = x192_zero(), bp = x192_zero(), bm = x192_zero();
            long long sumw = 0;
            for (long long j = lane; j < lw; j += WAVE)
                member_terms(cx, cx.cm_node[bw + j], Cw, sw, b0, bp, bm, sumw, bad);
            if (cx.ovf_flag[Cw]) {
                const int no = cx.ctr->ovf_cnt;
                for (int e = lane; e < no; e += WAVE)
                    if (cx.ovf_comm[e] == Cw) member_terms(cx, cx.ovf_node[e], Cw, sw, b0, bp, bm, sumw, bad);
            }
            WAVE_SYNC();
            b0 = wave_sum_x192(b0);
            bp = wave_sum_x192(bp);
            bm = wave_sum_x192(bm);
            sumw = wave_sum_i64(sumw);
            if (lane == 0) store_comm(cx, Cw, sw, b0, bp, bm, sumw, bad);
            WAVE_SYNC();
        }
    }
    if (bad) atomicOr(&cx.ctr->error, LF_DEVERR_INEXACT);
}

// ------------------------------------------------------------------------------------
// A6: iteration end
// ------------------------------------------------------------------------------------
// Per iteration some ten launches, each a single pass: the removal of communities with fewer
// than two members and the score's partial sums; the memberships that stay, counted per tile of
// nodes, then copied to the other slot buffer and into the nodes' lines at once; the member
// lists' capacities, summed per tile and placed; the lists filled; the report.  Shared counters
// are folded per block: one atomic per wave on a single address would serialise a launch
// (about 15 ns each).
// Latency bounds the small graphs (each launch of a 2,000-node graph takes 2 to 12 us), so the
// count of launches matters there: an iteration's start and end take some 20 launches
// instead of 63 (300-node job, 17 iterations: 10.2 -> 8.1 ms a run; 120 served jobs 555 -> 420
// ms).  Gathers and atomics bound the large ones: 4M nodes, 7.3M memberships: 1.1 ms an end, of
// which 0.41 the copy with its capacity atomics and 0.31 the list fill.
#define END_TILE 256            // nodes per block: one per thread, so that small graphs spread too
#define CAP_TILE 1024           // communities per block of the list capacities
#define END_PARTS 1024          // most blocks of the pass over the communities

// sum of v over the block's 256 threads before this one, and of all
__device__ __forceinline__ int block_excl_int(int v, int *s_w, int *total)
{
    int wsum;
    const int incl = wave_incl_scan(v, &wsum);
    const int lane = threadIdx.x & (WAVE - 1), wv = threadIdx.x / WAVE;
    __syncthreads();                        // an earlier round's totals are read
    if (lane == 0) s_w[wv] = wsum;
    __syncthreads();
    int off = 0, tot = 0;
    for (int w = 0; w < 256 / WAVE; w++) {
        if (w < wv) off += s_w[w];
        tot += s_w[w];
    }
    *total = tot;
    return off + incl - v;
}

// communities with fewer than `least` members (two; 0 where a batch member leaves within an
// iteration: none) are removed: mark them (tflag = 2), zero their statistics; the live ones
// are counted and their scores summed exactly per block; every community's member list is
// emptied
__global__ void __launch_bounds__(256) k_end_mark(Ctx cx, int least, long long *capx, X256 *part)
{
    __shared__ X256 s_x[256 / WAVE];
    __shared__ int s_live[256 / WAVE];
    X256 acc = x256_zero();
    int live = 0, bad = 0;
    for (long long c = blockIdx.x * (long long)blockDim.x + threadIdx.x; c < cx.K;
         c += (long long)gridDim.x * blockDim.x) {
        CommRec *r = &cx.cr[c];
        const int s = r->s;
        if (s < least) {
            if (s == 1) cx.tflag[c] = 2;
            r->s = 0;
            r->m = 0;
            r->W = 0.0;
            for (int k = 0; k < 5; k++) { r->Sp[k] = 0; r->Sm[k] = 0; }
        } else {
            live += s >= 2;
            x256_add(acc, x256_from_double(r->W, bad));
        }
        cx.cm_len[c] = 0;
        cx.ovf_flag[c] = 0;
        capx[c] = 0;
    }
    if (bad) atomicOr(&cx.ctr->error, LF_DEVERR_INEXACT);
    acc = wave_sum_x256(acc);
    live = wave_sum_int(live);
    const int lane = threadIdx.x & (WAVE - 1), wv = threadIdx.x / WAVE;
    if (lane == 0) {
        s_x[wv] = acc;
        s_live[wv] = live;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < 256 / WAVE; w++) {
            x256_add(acc, s_x[w]);
            live += s_live[w];
        }
        part[blockIdx.x] = acc;
        if (live) atomicAdd(&cx.ctr->live, live);
    }
}

// a membership that stays: not left in this iteration, its community not removed
__device__ __forceinline__ bool stays(const Ctx &cx, int c) { return c >= 0 && cx.tflag[c] != 2; }

__device__ __forceinline__ int count_staying(const Ctx &cx, const NodeLine &l)
{
    int w = 0;
    if (l.off < 0) {
#pragma unroll
        for (int t = 0; t < LINE_SLOTS; t++)
            if (t < l.cnt && stays(cx, l.s[t].comm)) w++;
    } else {
        for (int t0 = 0; t0 < l.cnt; t0 += 4) {        // four slots and their flags per round trip
            int c[4];
#pragma unroll
            for (int q = 0; q < 4; q++) c[q] = t0 + q < l.cnt ? cx.slot[l.off + t0 + q].comm : -1;
#pragma unroll
            for (int q = 0; q < 4; q++) w += stays(cx, c[q]);
        }
    }
    return w;
}

// slots of the next layout per tile of END_TILE nodes: staying memberships + one free slot each
__global__ void __launch_bounds__(256) k_end_count(Ctx cx, long long *tsum)
{
    __shared__ int s_w[256 / WAVE];
    const long long x = (long long)blockIdx.x * END_TILE + threadIdx.x;
    const int v = x < cx.n ? count_staying(cx, cx.ln[x]) + 1 : 0;
    int tot;
    (void)block_excl_int(v, s_w, &tot);
    if (threadIdx.x == 0) tsum[blockIdx.x] = tot;
}

// the staying memberships at their new place (dst), the nodes' headers and lines, and every
// community's room for joiners (sum of member degrees)
__global__ void __launch_bounds__(256) k_end_copy(Ctx cx, const long long *toff, Slot *dst, long long *capx,
                                                  unsigned char *mc8)
{
    __shared__ int s_w[256 / WAVE];
    const long long base = toff[blockIdx.x];
    const long long x = (long long)blockIdx.x * END_TILE + threadIdx.x;
    NodeLine l;
    l.cnt = 0;
    l.off = -1;
    if (x < cx.n) l = cx.ln[x];
    const int w = count_staying(cx, l);
    int tot;
    const long long o = base + block_excl_int(x < cx.n ? w + 1 : 0, s_w, &tot);
    if (x == cx.n) cx.nh[x].off = o;
    if (x >= cx.n) return;
    NodeLine ln;
    ln.cnt = w;
    ln.deg = l.deg;
    ln.off = w + 1 <= LINE_SLOTS ? -1 : o;
#pragma unroll
    for (int t = 0; t < LINE_SLOTS; t++) ln.s[t] = Slot{-1, 0};
    int k = 0;
    for (int t0 = 0; t0 < l.cnt; t0 += LINE_SLOTS) {     // LINE_SLOTS slots and flags per round trip
        Slot sl[LINE_SLOTS];
        bool st[LINE_SLOTS];
#pragma unroll
        for (int q = 0; q < LINE_SLOTS; q++)
            sl[q] = l.off < 0 ? l.s[q] : t0 + q < l.cnt ? cx.slot[l.off + t0 + q] : Slot{-1, 0};
#pragma unroll
        for (int q = 0; q < LINE_SLOTS; q++) st[q] = t0 + q < l.cnt && stays(cx, sl[q].comm);
#pragma unroll
        for (int q = 0; q < LINE_SLOTS; q++)
            if (st[q]) {
                dst[o + k] = sl[q];
                atomicAdd((unsigned long long *)&capx[sl[q].comm], (unsigned long long)l.deg);
#pragma unroll
                for (int u = 0; u < LINE_SLOTS; u++)     // (register indices known at compile time)
                    if (u == k && ln.off < 0) ln.s[u] = sl[q];
                k++;
            }
    }
    dst[o + w] = Slot{-1, 0};
    NodeHdr hd;
    hd.off = o;
    hd.cnt = w;
    hd.deg = l.deg;
    cx.nh[x] = hd;
    cx.ln[x] = ln;
    mc8[x] = w < 255 ? (unsigned char)w : 255;
}

// member-list capacity of a community: its members plus room for joiners
__device__ __forceinline__ long long list_cap(const Ctx &cx, const long long *capx, long long c)
{
    const long long ex = capx[c];
    return cx.cr[c].s + (ex < cx.n ? ex : cx.n);
}

__global__ void __launch_bounds__(256) k_cap_sum(Ctx cx, const long long *capx, long long *tsum)
{
    __shared__ long long s_w[256 / WAVE];
    long long v = 0;
#pragma unroll
    for (int i = 0; i < CAP_TILE / 256; i++) {
        const long long c = (long long)blockIdx.x * CAP_TILE + i * 256 + threadIdx.x;
        if (c < cx.K) v += list_cap(cx, capx, c);
    }
    v = wave_sum_i64(v);
    if ((threadIdx.x & (WAVE - 1)) == 0) s_w[threadIdx.x / WAVE] = v;
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < 256 / WAVE; w++) v += s_w[w];
        tsum[blockIdx.x] = v;
    }
}

// list offsets (K + 1); the removed marks are cleared on the way
__global__ void __launch_bounds__(256) k_cap_place(Ctx cx, const long long *capx, const long long *toff,
                                                   long long *cm_off)
{
    __shared__ long long s_w[256 / WAVE];
    const int lane = threadIdx.x & (WAVE - 1), wv = threadIdx.x / WAVE;
    long long run = toff[blockIdx.x];
    for (int i = 0; i < CAP_TILE / 256; i++) {
        const long long c = (long long)blockIdx.x * CAP_TILE + i * 256 + threadIdx.x;
        const long long v = c < cx.K ? list_cap(cx, capx, c) : 0;
        long long incl = v;
        for (int o = 1; o < WAVE; o <<= 1) {
            const long long t = __shfl_up(incl, o, WAVE);
            if (lane >= o) incl += t;
        }
        __syncthreads();
        if (lane == WAVE - 1) s_w[wv] = incl;
        __syncthreads();
        long long off = run, tot = 0;
        for (int w = 0; w < 256 / WAVE; w++) {
            if (w < wv) off += s_w[w];
            tot += s_w[w];
        }
        run += tot;
        if (c <= cx.K) cm_off[c] = off + incl - v;
        if (c < cx.K) cx.tflag[c] = 0;
    }
}

// exact partition score: per-block X256 partials (the fold is k_score_fold's or the report's)
__global__ void __launch_bounds__(256) k_score_partials(const CommRec *cr, int K, X256 *part, int *err)
{
    __shared__ X256 s_w[256 / WAVE];
    X256 acc = x256_zero();
    int bad = 0;
    for (long long c = blockIdx.x * (long long)blockDim.x + threadIdx.x; c < K; c += (long long)gridDim.x * blockDim.x) {
        X256 v = x256_from_double(cr[c].W, bad);
        x256_add(acc, v);
    }
    acc = wave_sum_x256(acc);
    int lane = threadIdx.x & (WAVE - 1), wv = threadIdx.x / WAVE;
    if (lane == 0) s_w[wv] = acc;
    if (bad) atomicOr(err, LF_DEVERR_INEXACT);
    __syncthreads();
    if (threadIdx.x == 0) {
        X256 s = s_w[0];
        for (int k = 1; k < 256 / WAVE; k++) x256_add(s, s_w[k]);
        part[blockIdx.x] = s;
    }
}

// everything an iteration end reports to the host, written to its pinned record
#define REP_SLOTS 0
#define REP_MEMBERS 1
#define REP_SCORE 2
#define REP_JOINS 3
#define REP_LEAVES 4
#define REP_LIVE 5
#define REP_ERROR 6
__global__ void __launch_bounds__(WAVE) k_end_report(const DevCounters *c, const long long *slots,
                                                     const long long *members, const X256 *part, int np,
                                                     long long *rep)
{
    X256 acc = x256_zero();
    for (int k = threadIdx.x; k < np; k += WAVE) x256_add(acc, part[k]);
    acc = wave_sum_x256(acc);
    if (threadIdx.x != 0) return;
    rep[REP_SLOTS] = *slots;
    rep[REP_MEMBERS] = *members;
    rep[REP_SCORE] = __double_as_longlong(x256_round(acc));
    rep[REP_JOINS] = (long long)c->joins;
    rep[REP_LEAVES] = (long long)c->leaves;
    rep[REP_LIVE] = c->live;
    rep[REP_ERROR] = c->error;
}

__global__ void k_score_fold(const X256 *part, int np, double *out)
{
    X256 acc = x256_zero();
    for (int k = threadIdx.x; k < np; k += WAVE) x256_add(acc, part[k]);
    acc = wave_sum_x256(acc);
    if (threadIdx.x == 0) out[0] = x256_round(acc);
}

// ------------------------------------------------------------------------------------
// host side
// ------------------------------------------------------------------------------------
Ctx lf_ctx(lf_handle *h)
{
    Ctx c;
    memset(&c, 0, sizeof c);   // padding too: the bytes of a Ctx key captured graphs
    c.n = h->n;
    c.K = h->K;
    c.rowptr = h->rowptr;
    c.col = h->col;
    c.deg = h->deg;
    c.order = h->order;
    c.nh = h->nh;
    c.slot = h->slot[h->cur];
    c.ln = h->lines;
    c.cr = h->cr;
    c.cm_off = h->cm_off;
    c.cm_len = h->cm_len;
    c.cm_node = h->cm_node;
    c.tflag = h->tflag;
    c.ovf_node = h->ovf_node;
    c.ovf_comm = h->ovf_comm;
    c.ovf_flag = h->ovf_flag;
    c.dec = h->dec;
    c.ctr = h->ctr;
    for (int k = 0; k < LF_PATH_COUNT; k++) {
        c.plist[k] = h->plist[k];
        c.prec[k] = h->prec[k];
    }
    c.rank = h->rank;
    c.col_rank = h->col_rank;
    c.tpos = h->tpos;
    c.tchunk = h->tchunk;
    c.tbuck = h->tbuck;
    c.tcur = h->tcur;
    c.tvis = h->tvis;
    c.trow = h->trow;
    c.tres = h->tres;
    c.lhdr = h->lhdr;
    c.lpair = h->lpair;
    c.ldeg = h->ldeg;
    c.unit = h->unit;
    c.part_rec = h->part_rec;
    c.part_done = h->part_done;
    c.psum = h->psum;
    c.part_cap = (int)h->part_cap;
    c.stats = (h->profiling >> LF_PROF_COUNTERS_BIT) & 1;
    return c;
}

void lf_free_partition(lf_handle *h)
{
    void **ptrs[] = {(void **)&h->nh, (void **)&h->slot[0], (void **)&h->slot[1], (void **)&h->lines, (void **)&h->cr,
                     (void **)&h->cm_off, (void **)&h->cm_len, (void **)&h->cm_node, (void **)&h->tflag,
                     (void **)&h->ovf_node,
                     (void **)&h->ovf_comm, (void **)&h->ovf_flag, (void **)&h->ctr,
                     (void **)&h->part_done, (void **)&h->vbound,
                     (void **)&h->cls, (void **)&h->clscnt, (void **)&h->clsbase, (void **)&h->plist_all,
                     (void **)&h->prec_all, (void **)&h->mc8, (void **)&h->pre};
    for (void **p : ptrs) {
        lf_dev_free(h, *p);
        *p = nullptr;
    }
    h->K = 0;
    h->slot_capb[0] = h->slot_capb[1] = 0;
    h->cm_cap = 0;
    lf_free_iteration_buffers(h);
    h->graph_version++;
}

static int alloc_member_lists(lf_handle *h)
{
    if (h->cm_node) return LF_OK;
    const long long want = 2 * h->n + 1024;
    return lf_dev_regrow(h, (void **)&h->cm_node, &h->cm_cap, want, sizeof(int));
}

// member lists with capacity for joiners; requires sizes and slots to be current.  Queued
// on the stream without waiting: if the lists outgrow cm_node nothing is written, and the
// total (cm_off[K]) tells the host to grow it and call this again.
static int rebuild_member_lists_async(lf_handle *h)
{
    TmpScope tmp_scope(h);
    hipStream_t st = h->stream;
    const int BS = 256;
    long long n = h->n;
    int K = h->K;
    long long *capx = nullptr;
    LF_TRY(lf_tmp_alloc(h, (void **)&capx, sizeof(long long) * (K + 1)));
    LF_TRY(lf_zero(h, capx, sizeof(long long) * (K + 1)));
    Ctx cx = lf_ctx(h);
    if (n > 0) hipLaunchKernelGGL(k_member_extra, dim3(grid_for(n, BS)), dim3(BS), 0, st, h->nh, cx.slot, n, capx);
    if (K > 0) hipLaunchKernelGGL(k_member_cap, dim3(grid_for(K, BS)), dim3(BS), 0, st, capx, h->cr, K, n);
    LF_TRY(lf_exclusive_scan_i64(h, capx, h->cm_off, K + 1));
    LF_TRY(alloc_member_lists(h));
    LF_TRY(lf_zero(h, h->cm_len, sizeof(int) * (K > 0 ? K : 1)));
    if (n > 0)
        hipLaunchKernelGGL(k_member_fill, dim3(grid_for(n, BS)), dim3(BS), 0, st, h->nh, cx.slot, n, K, h->cm_off,
                           h->cm_len, h->cm_node, h->cm_cap);
    LF_HIP(h, hipGetLastError());
    return LF_OK;
}

// grow cm_node to hold `total` member entries and fill the lists again (waits)
static int grow_member_lists(lf_handle *h, long long total)
{
    if (!h->phase_graphs) LF_HIP(h, hipStreamSynchronize(h->stream));   // a batch member keeps the old list
    // grown two-fold (four-fold for a batch member, whose captured iteration starts and
    // ends a moved buffer invalidates), so a growing cover reallocates only a few times
    // (the batch's spare room within 8 MB)
    long long want = 2 * total + 1024;
    if (h->phase_graphs) want += 2 * total < (2 << 20) ? 2 * total : (2 << 20);
    LF_TRY(lf_dev_regrow(h, (void **)&h->cm_node, &h->cm_cap, want, sizeof(int)));
    return rebuild_member_lists_async(h);
}

int lf_rebuild_member_lists(lf_handle *h)
{
    h->lists_ready = false;
    LF_TRY(rebuild_member_lists_async(h));
    long long total = 0;
    LF_HIP(h, hipMemcpyAsync(&total, h->cm_off + h->K, sizeof(long long), hipMemcpyDeviceToHost, h->stream));
    LF_HIP(h, hipStreamSynchronize(h->stream));
    if (total > h->cm_cap) LF_TRY(grow_member_lists(h, total));
    LF_HIP(h, hipStreamSynchronize(h->stream));
    h->lists_ready = true;
    return LF_OK;
}

// exact partition score into the device double *dw (queued, no wait)
static int partition_score_async(lf_handle *h, double *dw)
{
    TmpScope tmp_scope(h);
    hipStream_t st = h->stream;
    int K = h->K;
    int nb = (int)((K + 255) / 256);
    if (nb > 1024) nb = 1024;
    if (nb < 1) nb = 1;
    X256 *part = nullptr;
    LF_TRY(lf_tmp_alloc(h, (void **)&part, sizeof(X256) * nb));
    hipLaunchKernelGGL(k_score_partials, dim3(nb), dim3(256), 0, st, h->cr, K, part, &h->ctr->error);
    hipLaunchKernelGGL(k_score_fold, dim3(1), dim3(WAVE), 0, st, part, nb, dw);
    LF_HIP(h, hipGetLastError());
    return LF_OK;
}

static int partition_score(lf_handle *h, double *out)
{
    TmpScope tmp_scope(h);
    double *dw = nullptr;
    LF_TRY(lf_tmp_alloc(h, (void **)&dw, sizeof(double)));
    LF_TRY(partition_score_async(h, dw));
    LF_HIP(h, hipMemcpyAsync(out, dw, sizeof(double), hipMemcpyDeviceToHost, h->stream));
    LF_HIP(h, hipStreamSynchronize(h->stream));
    LF_HIP(h, hipGetLastError());
    return LF_OK;
}

int lf_check_dev_error(lf_handle *h)
{
    int e = 0;
    LF_HIP(h, hipMemcpyAsync(&e, &h->ctr->error, sizeof(int), hipMemcpyDeviceToHost, h->stream));
    LF_HIP(h, hipStreamSynchronize(h->stream));
    return lf_dev_error_status(h, e);
}

int lf_dev_error_status(lf_handle *h, int e)
{
    if (e & LF_DEVERR_INEXACT) return lf_set_error(h, LF_EOVERFLOW, "a score term left the exact accumulator's range");
    if (e & LF_DEVERR_SLOTS) return lf_set_error(h, LF_EINTERNAL, "membership slot capacity exceeded");
    if (e & LF_DEVERR_INCOUNT) return lf_set_error(h, LF_EINTERNAL, "in-count bookkeeping inconsistent");
    if (e & LF_DEVERR_ODD) return lf_set_error(h, LF_EINTERNAL, "odd internal degree sum");
    if (e & LF_DEVERR_CAP) return lf_set_error(h, LF_EINTERNAL, "a per-queue work buffer was too small");
    return LF_OK;
}

static int alloc_partition_state(lf_handle *h, long long K, long long slots);
static int finish_partition(lf_handle *h);

int lf_initial_clustering(lf_handle *h)
{
    TmpScope tmp_scope(h);
    hipStream_t st = h->stream;
    const int BS = 256;
    long long n = h->n;
    lf_free_partition(h);
    LF_TRY(lf_dev_alloc(h, (void **)&h->ctr, sizeof(DevCounters)));
    LF_HIP(h, hipMemsetAsync(h->ctr, 0, sizeof(DevCounters), st));
    LF_TRY(lf_prof_begin(h, LF_K_INITCLUST));
    int *state = nullptr, *cursor = nullptr, *comm_of = nullptr, *flag = nullptr, *und = nullptr;
    long long *pos = nullptr;
    size_t nn = (size_t)(n > 0 ? n : 1);
    LF_TRY(lf_tmp_alloc(h, (void **)&state, sizeof(int) * nn));
    LF_TRY(lf_tmp_alloc(h, (void **)&cursor, sizeof(int) * nn));
    LF_TRY(lf_tmp_alloc(h, (void **)&comm_of, sizeof(int) * nn));
    LF_TRY(lf_tmp_alloc(h, (void **)&flag, sizeof(int) * nn));
    LF_TRY(lf_tmp_alloc(h, (void **)&pos, sizeof(long long) * (nn + 1)));
    const int RB = 8;   // rounds between host checks
    LF_TRY(lf_tmp_alloc(h, (void **)&und, sizeof(int) * RB));
    LF_HIP(h, hipMemsetAsync(state, 0, sizeof(int) * nn, st));
    LF_HIP(h, hipMemsetAsync(cursor, 0, sizeof(int) * nn, st));
    int rounds = 0;
    unsigned gr = grid_for(n, BS);
    if (gr > 8192) gr = 8192;
    while (n > 0) {
        LF_HIP(h, hipMemsetAsync(und, 0, sizeof(int) * RB, st));
        for (int r = 0; r < RB; r++)
            hipLaunchKernelGGL(k_lfmis_round, dim3(gr), dim3(BS), 0, st, h->rowptr, h->col, h->col_rank, h->rank, n,
                               state, cursor, und + r);
        rounds += RB;
        int hu[RB];
        LF_HIP(h, hipMemcpyAsync(hu, und, sizeof(int) * RB, hipMemcpyDeviceToHost, st));
        LF_HIP(h, hipStreamSynchronize(st));
        if (hu[RB - 1] == 0) break;
        if (rounds > 64 * (n + 8)) return lf_set_error(h, LF_EINTERNAL, "initial clustering did not converge");
    }
    if (n > 0) {
        hipLaunchKernelGGL(k_opener_flags, dim3(grid_for(n, BS)), dim3(BS), 0, st, h->order, state, n, flag);
    }
    LF_TRY(lf_exclusive_scan_i32_to_i64(h, flag, pos, n));
    long long lastp = 0;
    int lastf = 0;
    if (n > 0) {
        hipLaunchKernelGGL(k_opener_ids, dim3(grid_for(n, BS)), dim3(BS), 0, st, h->order, flag, pos, n, comm_of);
        hipLaunchKernelGGL(k_join_openers, dim3(grid_for(n * 16, BS)), dim3(BS), 0, st, h->rowptr, h->col, h->col_rank,
                           h->order, state, n, comm_of);
        LF_HIP(h, hipMemcpyAsync(&lastp, pos + n - 1, sizeof(long long), hipMemcpyDeviceToHost, st));
        LF_HIP(h, hipMemcpyAsync(&lastf, flag + n - 1, sizeof(int), hipMemcpyDeviceToHost, st));
    }
    LF_HIP(h, hipStreamSynchronize(st));
    LF_HIP(h, hipGetLastError());
    long long K = lastp + lastf;
    if (K >= (1ll << 31) - 1) return lf_set_error(h, LF_EOVERFLOW, "too many communities");
    LF_TRY(alloc_partition_state(h, K, 2 * n));
    if (n >= 0)
        hipLaunchKernelGGL(k_init_slots, dim3(grid_for(n > 0 ? n * 16 : 1, BS)), dim3(BS), 0, st, h->rowptr, h->col,
                           h->deg, comm_of, n, h->nh, h->slot[0], h->cr);
    LF_TRY(finish_partition(h));
    LF_TRY(lf_prof_end(h, LF_K_INITCLUST, rounds + 8));
    LF_TRY(lf_prof_flush(h));
    LF_TRY(lf_check_dev_error(h));
    return LF_OK;
}

// Partition arrays for K community ids and slot storage for `slots` memberships (at least
// one); community records zeroed, no member lists yet.
static int alloc_partition_state(lf_handle *h, long long K, long long slots)
{
    hipStream_t st = h->stream;
    long long n = h->n;
    size_t nn = (size_t)(n > 0 ? n : 1);
    h->K = (int)K;
    size_t KK = (size_t)(K > 0 ? K : 1);
    LF_TRY(lf_dev_alloc(h, (void **)&h->nh, sizeof(NodeHdr) * (nn + 1)));
    h->slot_capb[0] = h->slot_capb[1] = slots > 0 ? slots : 1;
    h->slot_used = slots;
    LF_TRY(lf_dev_alloc(h, (void **)&h->slot[0], sizeof(Slot) * h->slot_capb[0]));
    LF_TRY(lf_dev_alloc(h, (void **)&h->slot[1], sizeof(Slot) * h->slot_capb[1]));
    h->cur = 0;
    LF_TRY(lf_dev_alloc(h, (void **)&h->cr, sizeof(CommRec) * KK));
    LF_TRY(lf_dev_alloc(h, (void **)&h->cm_off, sizeof(long long) * (KK + 1)));
    LF_TRY(lf_dev_alloc(h, (void **)&h->cm_len, sizeof(int) * KK));
    LF_TRY(lf_dev_alloc(h, (void **)&h->tflag, sizeof(int) * KK));
    LF_TRY(lf_dev_alloc(h, (void **)&h->ovf_flag, sizeof(int) * KK));
    LF_TRY(lf_dev_alloc(h, (void **)&h->part_done, sizeof(int) * KK));
    LF_TRY(lf_dev_alloc(h, (void **)&h->vbound, sizeof(long long) * (nn + 1)));
    LF_TRY(lf_dev_alloc(h, (void **)&h->cls, sizeof(int) * nn));
    const size_t ct = LF_PATH_COUNT * (nn / 1024 + 2) + 1;   // counts per path and tile of the path lists
    LF_TRY(lf_dev_alloc(h, (void **)&h->clscnt, sizeof(int) * ct));
    LF_TRY(lf_dev_alloc(h, (void **)&h->clsbase, sizeof(long long) * ct));
    LF_TRY(lf_dev_alloc(h, (void **)&h->plist_all, sizeof(int) * nn));
    LF_TRY(lf_dev_alloc(h, (void **)&h->prec_all, sizeof(NodeRec) * nn));
    for (int k = 0; k < LF_PATH_COUNT; k++) {
        h->prec[k] = h->prec_all;
        h->plist[k] = h->plist_all;
    }
    LF_TRY(lf_dev_alloc(h, (void **)&h->mc8, nn));
    LF_TRY(lf_dev_alloc(h, (void **)&h->pre, sizeof(int) * nn));
    LF_TRY(lf_dev_alloc(h, (void **)&h->ovf_node, sizeof(int) * nn));
    LF_TRY(lf_dev_alloc(h, (void **)&h->ovf_comm, sizeof(int) * nn));
    LF_HIP(h, hipMemsetAsync(h->cr, 0, sizeof(CommRec) * KK, st));
    LF_HIP(h, hipMemsetAsync(h->tflag, 0, sizeof(int) * KK, st));
    LF_HIP(h, hipMemsetAsync(h->ovf_flag, 0, sizeof(int) * KK, st));
    return LF_OK;
}

// With slots, headers and community sizes written: member lists, every community's
// statistics (internal edges, exact sums, score) and the partition score.
static int finish_partition(lf_handle *h)
{
    hipStream_t st = h->stream;
    const int BS = 256;
    const long long K = h->K;
    LF_TRY(lf_rebuild_member_lists(h));
    Ctx cx = lf_ctx(h);
    int rb = (int)((K + 15) / 16);           // a row of lanes per community
    if (rb > 4096) rb = 4096;
    if (rb < 1) rb = 1;
    hipLaunchKernelGGL(k_refresh_list, dim3(rb), dim3(256), 0, st, cx, (int)K);
    LF_HIP(h, hipGetLastError());
    LF_TRY(partition_score(h, &h->Wt));
    return LF_OK;
}

// Warm start from an existing cover (Initial Clustering, last paragraph: an existing
// division can replace the greedy one).  off[n + 1] / ids[total] on the device, each
// node's communities in any order.  Node statistics must exist.
// Checks of a cover on the device (offsets, ids in [0, n_comms) or >= 0 if n_comms < 0, no
// id twice per node); *maxid = the largest id (-1 if none).
int lf_check_cover(lf_handle *h, const long long *off, const int *ids, long long total, int n_comms, int *maxid)
{
    TmpScope tmp_scope(h);
    hipStream_t st = h->stream;
    const int BS = 256;
    const long long n = h->n;
    long long ends[2] = {0, 0};
    LF_HIP(h, hipMemcpyAsync(&ends[0], off, sizeof(long long), hipMemcpyDeviceToHost, st));
    LF_HIP(h, hipMemcpyAsync(&ends[1], off + n, sizeof(long long), hipMemcpyDeviceToHost, st));
    LF_HIP(h, hipStreamSynchronize(st));
    if (ends[0] != 0 || ends[1] != total)
        return lf_set_error(h, LF_EINVAL, "cover offsets must start at 0 and end at total (%lld)", total);
    int *chk = nullptr;                      // [0] error bits, [1] largest id
    LF_TRY(lf_tmp_alloc(h, (void **)&chk, 2 * sizeof(int)));
    const int init[2] = {0, -1};
    LF_HIP(h, hipMemcpyAsync(chk, init, sizeof init, hipMemcpyHostToDevice, st));
    unsigned gc = grid_for(n, BS);
    if (gc > 1024) gc = 1024;
    if (n > 0) hipLaunchKernelGGL(k_cover_check, dim3(gc), dim3(BS), 0, st, off, ids, n, total, n_comms, chk);
    int hc[2];
    LF_HIP(h, hipMemcpyAsync(hc, chk, sizeof hc, hipMemcpyDeviceToHost, st));
    LF_HIP(h, hipStreamSynchronize(st));
    LF_HIP(h, hipGetLastError());
    if (hc[0] & 1) return lf_set_error(h, LF_EINVAL, "cover offsets decrease or leave [0, total]");
    if (hc[0] & 2) return lf_set_error(h, LF_EINVAL, "a community id is negative or not below n_comms");
    if (hc[0] & 4) return lf_set_error(h, LF_EINVAL, "a node lists a community twice");
    *maxid = hc[1];
    return LF_OK;
}

int lf_partition_from_cover(lf_handle *h, const long long *off, const int *ids, long long total, int n_comms)
{
    TmpScope tmp_scope(h);
    hipStream_t st = h->stream;
    const int BS = 256;
    const long long n = h->n;
    int maxid = -1;
    LF_TRY(lf_check_cover(h, off, ids, total, n_comms, &maxid));
    const long long K = n_comms >= 0 ? n_comms : (long long)maxid + 1;
    if (K >= (1ll << 31) - 1) return lf_set_error(h, LF_EOVERFLOW, "too many communities");
    h->state = 1;                            // the previous partition is gone from here on
    lf_free_partition(h);
    LF_TRY(lf_dev_alloc(h, (void **)&h->ctr, sizeof(DevCounters)));
    LF_HIP(h, hipMemsetAsync(h->ctr, 0, sizeof(DevCounters), st));
    LF_TRY(lf_prof_begin(h, LF_K_INITCLUST));
    LF_TRY(alloc_partition_state(h, K, total + n));
    hipLaunchKernelGGL(k_cover_slots, dim3(grid_for(n > 0 ? n * 16 : 1, BS)), dim3(BS), 0, st, h->rowptr, h->col,
                       h->deg, off, ids, n, h->nh, h->slot[0], h->cr);
    LF_TRY(finish_partition(h));
    LF_TRY(lf_prof_end(h, LF_K_INITCLUST, 8));
    LF_TRY(lf_prof_flush(h));
    LF_TRY(lf_check_dev_error(h));
    h->state = 2;
    return LF_OK;
}

// Iteration end, first half (queued): communities with fewer than `least` members removed,
// slots compacted, member lists rebuilt, score reduced, and one report copied to pinned host
// memory.
int lf_iteration_end_enqueue(lf_handle *h, int least)
{
    TmpScope tmp_scope(h);
    hipStream_t st = h->stream;
    const int BS = 256;
    long long n = h->n;
    int K = h->K;
    const Ctx cx = lf_ctx(h);
    const long long nt = n / END_TILE + 1, kt = K / CAP_TILE + 1;       // tiles (position n and id K included)
    int np = (int)grid_for(K, BS);
    if (np > END_PARTS) np = END_PARTS;
    if (np < 1) np = 1;
    long long *capx = nullptr, *nsum = nullptr, *noff = nullptr, *ksum = nullptr, *koff = nullptr;
    X256 *part = nullptr;
    LF_TRY(lf_tmp_alloc(h, (void **)&capx, sizeof(long long) * (K + 1)));
    LF_TRY(lf_tmp_alloc(h, (void **)&nsum, sizeof(long long) * nt));
    LF_TRY(lf_tmp_alloc(h, (void **)&noff, sizeof(long long) * nt));
    LF_TRY(lf_tmp_alloc(h, (void **)&ksum, sizeof(long long) * kt));
    LF_TRY(lf_tmp_alloc(h, (void **)&koff, sizeof(long long) * kt));
    LF_TRY(lf_tmp_alloc(h, (void **)&part, sizeof(X256) * np));
    hipLaunchKernelGGL(k_end_mark, dim3(np), dim3(BS), 0, st, cx, least, capx, part);
    hipLaunchKernelGGL(k_end_count, dim3((unsigned)nt), dim3(BS), 0, st, cx, nsum);
    LF_TRY(lf_exclusive_scan_i64(h, nsum, noff, nt));
    // the new layout holds at most the current one's entries plus one per node (a node's
    // count grows only into its free slot), so the copy needs no wait for its size
    int other = 1 - h->cur;
    const long long bound = h->slot_used + n + 1;
    if (bound > h->slot_capb[other]) {
        const long long want = (h->phase_graphs ? 3 * bound : bound + bound / 2) + 1024;
        LF_TRY(lf_dev_regrow(h, (void **)&h->slot[other], &h->slot_capb[other], want, sizeof(Slot)));
    }
    hipLaunchKernelGGL(k_end_copy, dim3((unsigned)nt), dim3(BS), 0, st, cx, (const long long *)noff, h->slot[other],
                       capx, h->mc8);
    h->cur = other;
    hipLaunchKernelGGL(k_cap_sum, dim3((unsigned)kt), dim3(BS), 0, st, cx, (const long long *)capx, ksum);
    LF_TRY(lf_exclusive_scan_i64(h, ksum, koff, kt));
    hipLaunchKernelGGL(k_cap_place, dim3((unsigned)kt), dim3(BS), 0, st, cx, (const long long *)capx,
                       (const long long *)koff, h->cm_off);
    LF_TRY(alloc_member_lists(h));
    hipLaunchKernelGGL(k_member_fill, dim3(grid_for(n, BS)), dim3(BS), 0, st, h->nh, h->slot[other], n, K, h->cm_off,
                       h->cm_len, h->cm_node, h->cm_cap);
    // the host's one wait of the iteration end: every value it needs in one pinned record
    hipLaunchKernelGGL(k_end_report, dim3(1), dim3(WAVE), 0, st, (const DevCounters *)h->ctr,
                       (const long long *)&h->nh[n].off, (const long long *)h->cm_off + K, (const X256 *)part, np,
                       h->hrep);
    LF_HIP(h, hipGetLastError());
    return LF_OK;
}

// second half: read the report (the caller has waited for it), grow the member lists if
// they did not fit
int lf_iteration_end_complete(lf_handle *h, long long *joins, long long *leaves, long long *live)
{
    hipStream_t st = h->stream;
    const long long *r = h->hrep;
    h->slot_used = r[REP_SLOTS];
    double wt;
    memcpy(&wt, &r[REP_SCORE], sizeof wt);
    h->Wt = wt;
    unsigned long long jl[2] = {(unsigned long long)r[REP_JOINS], (unsigned long long)r[REP_LEAVES]};
    int lv[2] = {(int)r[REP_LIVE], 0};
    h->last_dev_error = (int)r[REP_ERROR];
    *joins = (long long)jl[0];
    *leaves = (long long)jl[1];
    *live = lv[0];
    if (r[REP_MEMBERS] > h->cm_cap) {        // rare: member lists outgrew their buffer
        h->lists_ready = false;              // (if this fails, the next run's first start fills them)
        LF_TRY(grow_member_lists(h, r[REP_MEMBERS]));
        if (!h->phase_graphs) LF_HIP(h, hipStreamSynchronize(st));
        h->lists_ready = true;
    }
    return LF_OK;
}

// memberships (community ids ascending per node) and in-counts, gathered on the device
__global__ void k_member_counts(const NodeHdr *nh, long long n, long long *cnt)
{
    long long x = blockIdx.x * (long long)blockDim.x + threadIdx.x;
    if (x < n) cnt[x] = nh[x].cnt;
    if (x == n) cnt[n] = 0;
}

__global__ void k_member_out(const NodeHdr *nh, const Slot *slot, long long n, const long long *off,
                             int *ids, int *in)
{
    long long x = blockIdx.x * (long long)blockDim.x + threadIdx.x;
    if (x >= n) return;
    NodeHdr hx = nh[x];
    long long o = off[x];
    // insertion sort of a handful of entries, directly in the output range
    for (int t = 0; t < hx.cnt; t++) {
        Slot v = slot[hx.off + t];
        int b = t;
        while (b > 0 && ids[o + b - 1] > v.comm) {
            ids[o + b] = ids[o + b - 1];
            in[o + b] = in[o + b - 1];
            b--;
        }
        ids[o + b] = v.comm;
        in[o + b] = v.in;
    }
}

int lf_fetch_memberships(lf_handle *h, long long *offsets, int *comm_ids, long long capacity,
                         long long *total, int *in_counts)
{
    TmpScope tmp_scope(h);
    hipStream_t st = h->stream;
    const int BS = 256;
    long long n = h->n;
    long long *cnt = nullptr, *doff = nullptr;
    LF_TRY(lf_tmp_alloc(h, (void **)&cnt, sizeof(long long) * (n + 1)));
    LF_TRY(lf_tmp_alloc(h, (void **)&doff, sizeof(long long) * (n + 1)));
    hipLaunchKernelGGL(k_member_counts, dim3(grid_for(n + 1, BS)), dim3(BS), 0, st, h->nh, n, cnt);
    LF_TRY(lf_exclusive_scan_i64(h, cnt, doff, n + 1));
    long long tot = 0;
    LF_HIP(h, hipMemcpyAsync(&tot, doff + n, sizeof(long long), hipMemcpyDeviceToHost, st));
    LF_HIP(h, hipStreamSynchronize(st));
    *total = tot;
    int rc = LF_OK;
    if (offsets && (comm_ids || in_counts)) {
        if (capacity < tot) {
            rc = lf_set_error(h, LF_ERANGE, "capacity %lld < %lld memberships", capacity, tot);
        } else {
            int *dids = nullptr, *din = nullptr;
            LF_TRY(lf_tmp_alloc(h, (void **)&dids, sizeof(int) * (tot > 0 ? tot : 1)));
            LF_TRY(lf_tmp_alloc(h, (void **)&din, sizeof(int) * (tot > 0 ? tot : 1)));
            if (n > 0)
                hipLaunchKernelGGL(k_member_out, dim3(grid_for(n, BS)), dim3(BS), 0, st, h->nh, h->slot[h->cur], n,
                                   doff, dids, din);
            LF_HIP(h, hipMemcpyAsync(offsets, doff, sizeof(long long) * (n + 1), hipMemcpyDeviceToHost, st));
            if (comm_ids && tot > 0)
                LF_HIP(h, hipMemcpyAsync(comm_ids, dids, sizeof(int) * tot, hipMemcpyDeviceToHost, st));
            if (in_counts && tot > 0)
                LF_HIP(h, hipMemcpyAsync(in_counts, din, sizeof(int) * tot, hipMemcpyDeviceToHost, st));
            LF_HIP(h, hipStreamSynchronize(st));
            LF_HIP(h, hipGetLastError());
        }
    }
    return rc;
}
