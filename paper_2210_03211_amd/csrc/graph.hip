// graph.hip -- preprocessing and node statistics on the GPU.
//
//   lf_build_graph   multi-edge removal, self-loop removal, dense labels, symmetric CSR with
//                    sorted rows (Methods, "Preprocessing")
//   lf_node_stats    triangles k_i, local clustering coefficient, global cc (mean of local
//                    CCs) and the node order: CC descending, degree descending, id
//                    ascending (Methods, "Node Order"; WCC-hat subsection for cc)
//
// Triangles: every edge is oriented from the endpoint that is smaller in (degree, id)
// order to the larger one, so each triangle {a < b < c} is found exactly once, at a with
// the oriented edges a->b, a->c and b->c.  For a node u, a wave (or a workgroup for long
// out-lists) stages N+(u) and a bit filter of its members in LDS; groups of 16 lanes walk the
// lists N+(v), v in N+(u), four entries a lane, and what the filter lets pass is queued and
// searched for in the staged N+(u) a full wave at a time.  A hit credits u, v and w; the
// credits of v and w (both in N+(u)) are accumulated in LDS counters and flushed to HBM once
// per (u, position).
#include "method.h"

static int bits_for(long long n)
{
    int b = 1;
    while ((1ll << b) < n) b++;
    return b;
}

// ------------------------------------------------------------------------------------
// A0: graph build
// ------------------------------------------------------------------------------------
__global__ void k_collect_ids(const long long *src, const long long *dst, long long np,
                              unsigned long long *ids, int *err)
{
    long long e = blockIdx.x * (long long)blockDim.x + threadIdx.x;
    if (e >= np) return;
    long long a = src[e], b = dst[e];
    if (a < 0 || b < 0) { atomicOr(err, 1); a = b = 0; }
    bool loop = (a == b);
    ids[2 * e] = loop ? ~0ull : (unsigned long long)a;
    ids[2 * e + 1] = loop ? ~0ull : (unsigned long long)b;
}

__global__ void k_unique_flags_u64(const unsigned long long *k, long long n, unsigned long long sentinel,
                                   int *flag)
{
    long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x;
    if (i >= n) return;
    unsigned long long v = k[i];
    flag[i] = (v != sentinel) && (i == 0 || k[i - 1] != v);
}

// the flagged keys, compacted (twice, if copy is given)
__global__ void k_compact_u64(const unsigned long long *k, const int *flag, const long long *pos,
                              long long n, unsigned long long *out, unsigned long long *copy)
{
    long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x;
    if (i >= n) return;
    if (flag[i]) {
        out[pos[i]] = k[i];
        if (copy) copy[pos[i]] = k[i];
    }
}

// Positions in the sorted ids by their leading ID_BITS bits above the smallest one, so that
// finding an id takes a table entry and the search of what shares it (two or three reads where
// ids are spread evenly) instead of log2(n) dependent reads: relabelling 8.7M pairs over 1M
// ids 1.01 -> 0.37 ms.  Below ID_TABLE_MIN ids the search is short and the table a launch more.
#define ID_BITS 17
#define ID_TABLE_MIN 65536

__device__ __forceinline__ int id_shift(unsigned long long range)
{
    const int bits = range ? 64 - __clzll((long long)range) : 0;
    return bits > ID_BITS ? bits - ID_BITS : 0;
}

// tab[t] = ids below ids[0] + (t << shift), t = 0 .. 2^ID_BITS
__global__ void k_id_table(const unsigned long long *ids, long long n, int *tab)
{
    const long long t = blockIdx.x * (long long)blockDim.x + threadIdx.x;
    if (t > 1 << ID_BITS) return;
    const unsigned long long range = ids[n - 1] - ids[0];
    const int sh = id_shift(range);
    long long lo = 0, hi = n;
    while (lo < hi) {                        // (ids[mid] - ids[0]) >> sh does not overflow
        const long long mid = (lo + hi) >> 1;
        if ((long long)((ids[mid] - ids[0]) >> sh) < t) lo = mid + 1;
        else hi = mid;
    }
    tab[t] = (int)lo;
}

__device__ __forceinline__ long long find_id(const unsigned long long *ids, long long n, const int *tab, int sh,
                                             unsigned long long v)
{
    long long lo = 0, hi = n - 1;
    if (tab) {
        const unsigned long long t = v < ids[0] ? ~0ull : (v - ids[0]) >> sh;
        if (t >= 1 << ID_BITS) return -1;
        lo = tab[t];
        hi = (long long)tab[t + 1] - 1;
    }
    while (lo <= hi) {
        const long long mid = lo + ((hi - lo) >> 1);
        const unsigned long long x = ids[mid];
        if (x == v) return mid;
        if (x < v) lo = mid + 1; else hi = mid - 1;
    }
    return -1;
}

// canonical (min, max) keys; self-loops -> sentinel; ids checked or remapped
__global__ void k_canon_keys(const long long *src, const long long *dst, long long np, long long n,
                             const unsigned long long *uniq_ids, const int *tab, int B,
                             unsigned long long *keys, int *err)
{
    long long e = blockIdx.x * (long long)blockDim.x + threadIdx.x;
    if (e >= np) return;
    long long a = src[e], b = dst[e];
    unsigned long long sentinel = (B >= 32) ? ~0ull : ((1ull << (2 * B)) - 1);
    if (a == b) { keys[e] = sentinel; return; }
    if (uniq_ids) {
        const int sh = tab ? id_shift(uniq_ids[n - 1] - uniq_ids[0]) : 0;
        a = find_id(uniq_ids, n, tab, sh, (unsigned long long)a);
        b = find_id(uniq_ids, n, tab, sh, (unsigned long long)b);
    }
    if (a < 0 || b < 0 || a >= n || b >= n) { atomicOr(err, 1); keys[e] = sentinel; return; }
    if (a > b) { long long t = a; a = b; b = t; }
    keys[e] = ((unsigned long long)a << B) | (unsigned long long)b;
}

// The CSR from the simple edges (a < b) in two orders: fwd by (a, b) and rev, a stable sort of
// it by b.  Row x is the a's of rev's run of b = x (all below x, ascending) followed by the
// b's of fwd's run of a = x (all above, ascending), so no sort of both directions is
// needed: half the bits of half the keys, and degrees follow from the runs without atomics.
// Measured, 4M nodes and 35M edges, 10 ms of it the upload: 19.1 -> 13.3 ms; 1M nodes and 39M
// edges already on the device: 9.5 -> 3.5 ms.

// first entry of each node's run in both orders (n + 1 entries each)
__global__ void k_runs(const unsigned long long *fwd, const unsigned long long *rev, long long ne, int B, long long n,
                       long long *f0, long long *r0)
{
    const long long x = blockIdx.x * (long long)blockDim.x + threadIdx.x;
    if (x > n) return;
    const unsigned long long mask = (1ull << B) - 1;
    long long lo = 0, hi = ne, lo2 = 0, hi2 = ne;
    while (lo < hi || lo2 < hi2) {           // both searches side by side
        const long long m = (lo + hi) >> 1, m2 = (lo2 + hi2) >> 1;
        const bool up = lo < hi && (long long)(fwd[m] >> B) < x;
        const bool up2 = lo2 < hi2 && (long long)(rev[m2] & mask) < x;
        if (lo < hi) {
            if (up) lo = m + 1; else hi = m;
        }
        if (lo2 < hi2) {
            if (up2) lo2 = m2 + 1; else hi2 = m2;
        }
    }
    f0[x] = lo;
    r0[x] = lo2;
}

// maximum over the block of non-negative values, added to *out once per block
__device__ __forceinline__ void block_max(int v, int *out)
{
    __shared__ unsigned s_m[256 / WAVE];
    const unsigned m = wave_max_u32((unsigned)v);
    if ((threadIdx.x & (WAVE - 1)) == 0) s_m[threadIdx.x / WAVE] = m;
    __syncthreads();
    if (threadIdx.x == 0) {
        unsigned t = s_m[0];
        for (int w = 1; w < 256 / WAVE; w++) t = s_m[w] > t ? s_m[w] : t;
        if (t) atomicMax(out, (int)t);
    }
}

__global__ void __launch_bounds__(256) k_rows(const long long *f0, const long long *r0, long long n, int *deg,
                                              long long *rowptr, int *maxdeg)
{
    int mx = 0;
    for (long long x = blockIdx.x * (long long)blockDim.x + threadIdx.x; x <= n;
         x += (long long)gridDim.x * blockDim.x) {
        rowptr[x] = f0[x] + r0[x];
        if (x == n) break;
        const int d = (int)(f0[x + 1] - f0[x] + r0[x + 1] - r0[x]);
        deg[x] = d;
        mx = d > mx ? d : mx;
    }
    __syncthreads();
    block_max(mx, maxdeg);
}

__global__ void k_cols(const unsigned long long *fwd, const unsigned long long *rev, long long ne, int B,
                       const long long *f0, const long long *r0, int *col)
{
    const long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x;
    if (i >= ne) return;
    const unsigned long long mask = (1ull << B) - 1;
    const unsigned long long kf = fwd[i], kr = rev[i];
    col[i + r0[(long long)(kf >> B) + 1]] = (int)(kf & mask);
    col[i + f0[(long long)(kr & mask)]] = (int)(kr >> B);
}

// widened copy and maximum (one atomic per block: every thread's on one address took 0.7 ms
// for 4M values)
__global__ void __launch_bounds__(256) k_deg_to_i64(const int *deg, long long n, long long *out, int *maxdeg)
{
    int mx = 0;
    for (long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x; i < n;
         i += (long long)gridDim.x * blockDim.x) {
        const int d = deg[i];
        out[i] = d;
        mx = d > mx ? d : mx;
    }
    __syncthreads();
    block_max(mx, maxdeg);
}

__global__ void k_set_last(long long *rowptr, long long n, long long val) { rowptr[n] = val; }

__global__ void k_iota_ids(long long *ids, long long n, const unsigned long long *uniq)
{
    long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x;
    if (i >= n) return;
    ids[i] = uniq ? (long long)uniq[i] : i;
}

static inline unsigned grid_for(long long n, int block) { return (unsigned)((n + block - 1) / block); }

// a grid that strides: at most 2048 blocks
static inline unsigned stride_grid(long long n, int block)
{
    const long long g = (n + block - 1) / block;
    return (unsigned)(g < 1 ? 1 : g > 2048 ? 2048 : g);
}

int lf_build_graph(lf_handle *h, long long n, long long np, const long long *src,
                   const long long *dst, unsigned flags)
{
    TmpScope tmp_scope(h);
    hipStream_t st = h->stream;
    const int BS = 256;
    long long *dsrc = nullptr, *ddst = nullptr;
    if (flags & LF_DEVICE_PTR) {
        dsrc = (long long *)src;
        ddst = (long long *)dst;
    } else if (np > 0) {
        LF_TRY(lf_tmp_alloc(h, (void **)&dsrc, sizeof(long long) * np));
        LF_TRY(lf_tmp_alloc(h, (void **)&ddst, sizeof(long long) * np));
        LF_HIP(h, hipMemcpyAsync(dsrc, src, sizeof(long long) * np, hipMemcpyHostToDevice, st));
        LF_HIP(h, hipMemcpyAsync(ddst, dst, sizeof(long long) * np, hipMemcpyHostToDevice, st));
    }
    int *derr = nullptr;
    LF_TRY(lf_tmp_alloc(h, (void **)&derr, sizeof(int) * 4));
    LF_HIP(h, hipMemsetAsync(derr, 0, sizeof(int) * 4, st));

    // scratch sized for the largest use: 2 * np 64-bit keys (ids) and 2 * ne directed keys
    long long kcap = 2 * (np > 0 ? np : 1);
    unsigned long long *ka = nullptr, *kb = nullptr;
    int *flag = nullptr;
    long long *pos = nullptr;
    LF_TRY(lf_tmp_alloc(h, (void **)&ka, sizeof(unsigned long long) * kcap));
    LF_TRY(lf_tmp_alloc(h, (void **)&kb, sizeof(unsigned long long) * kcap));
    LF_TRY(lf_tmp_alloc(h, (void **)&flag, sizeof(int) * kcap));
    LF_TRY(lf_tmp_alloc(h, (void **)&pos, sizeof(long long) * (kcap + 1)));

    unsigned long long *uniq_ids = nullptr;
    if (flags & LF_RELABEL) {
        long long m = 2 * np;
        if (np > 0) hipLaunchKernelGGL(k_collect_ids, dim3(grid_for(np, BS)), dim3(BS), 0, st, dsrc, ddst, np, ka, derr);
        unsigned long long *sorted;
        LF_TRY(lf_sort_u64(h, ka, kb, m, 64, &sorted));
        if (m > 0) hipLaunchKernelGGL(k_unique_flags_u64, dim3(grid_for(m, BS)), dim3(BS), 0, st, sorted, m, ~0ull, flag);
        LF_TRY(lf_exclusive_scan_i32_to_i64(h, flag, pos, m + 0));
        long long last_pos = 0;
        int last_flag = 0;
        if (m > 0) {
            LF_HIP(h, hipMemcpyAsync(&last_pos, pos + m - 1, sizeof(long long), hipMemcpyDeviceToHost, st));
            LF_HIP(h, hipMemcpyAsync(&last_flag, flag + m - 1, sizeof(int), hipMemcpyDeviceToHost, st));
        }
        LF_HIP(h, hipStreamSynchronize(st));
        n = (m > 0) ? last_pos + last_flag : 0;
        LF_TRY(lf_tmp_alloc(h, (void **)&uniq_ids, sizeof(unsigned long long) * (n > 0 ? n : 1)));
        if (m > 0) hipLaunchKernelGGL(k_compact_u64, dim3(grid_for(m, BS)), dim3(BS), 0, st, sorted, flag, pos, m, uniq_ids,
                                       (unsigned long long *)nullptr);
    }
    if (n >= (1ll << 31) - 1) {
        return lf_set_error(h, LF_EOVERFLOW, "n = %lld nodes exceeds the supported 2^31 - 2", n);
    }
    int B = bits_for(n > 1 ? n : 2);
    unsigned long long sentinel = (B >= 32) ? ~0ull : ((1ull << (2 * B)) - 1);
    int *tab = nullptr;
    if (uniq_ids && n >= ID_TABLE_MIN) {
        LF_TRY(lf_tmp_alloc(h, (void **)&tab, sizeof(int) * ((1 << ID_BITS) + 1)));
        hipLaunchKernelGGL(k_id_table, dim3(grid_for((1 << ID_BITS) + 1, BS)), dim3(BS), 0, st, uniq_ids, n, tab);
    }
    if (np > 0)
        hipLaunchKernelGGL(k_canon_keys, dim3(grid_for(np, BS)), dim3(BS), 0, st, dsrc, ddst, np, n,
                           uniq_ids, (const int *)tab, B, ka, derr);
    unsigned long long *sorted;
    LF_TRY(lf_sort_u64(h, ka, kb, np, 2 * B, &sorted));
    if (np > 0) hipLaunchKernelGGL(k_unique_flags_u64, dim3(grid_for(np, BS)), dim3(BS), 0, st, sorted, np, sentinel, flag);
    LF_TRY(lf_exclusive_scan_i32_to_i64(h, flag, pos, np));
    long long last_pos = 0;
    int last_flag = 0, herr[4] = {0, 0, 0, 0};
    if (np > 0) {
        LF_HIP(h, hipMemcpyAsync(&last_pos, pos + np - 1, sizeof(long long), hipMemcpyDeviceToHost, st));
        LF_HIP(h, hipMemcpyAsync(&last_flag, flag + np - 1, sizeof(int), hipMemcpyDeviceToHost, st));
    }
    LF_HIP(h, hipMemcpyAsync(herr, derr, sizeof(int) * 4, hipMemcpyDeviceToHost, st));
    LF_HIP(h, hipStreamSynchronize(st));
    if (herr[0]) return lf_set_error(h, LF_EINVAL, "edge list has an id outside [0, n) (n = %lld)", n);
    long long ne = (np > 0) ? last_pos + last_flag : 0;
    if (2 * ne >= (1ll << 31)) return lf_set_error(h, LF_EOVERFLOW, "2|E| = %lld exceeds 2^31 - 1", 2 * ne);
    // unique canonical keys -> kb (or ka) compacted, and a copy to be sorted by the second
    // id in the other buffer (of 2 np entries)
    unsigned long long *uk = (sorted == ka) ? kb : ka;
    unsigned long long *rev = uk + (np > 0 ? np : 1), *rev_alt = sorted;
    if (np > 0)
        hipLaunchKernelGGL(k_compact_u64, dim3(grid_for(np, BS)), dim3(BS), 0, st, sorted, flag, pos, np, uk, rev);

    LF_TRY(lf_dev_alloc(h, (void **)&h->deg, sizeof(int) * (n > 0 ? n : 1)));
    LF_TRY(lf_dev_alloc(h, (void **)&h->rowptr, sizeof(long long) * (n + 1)));
    LF_TRY(lf_dev_alloc(h, (void **)&h->col, sizeof(int) * (2 * ne + READ_PAD)));
    LF_TRY(lf_dev_alloc(h, (void **)&h->orig_id, sizeof(long long) * (n > 0 ? n : 1)));
    // the sort's alternate buffer is the one compacted from: stream order makes that safe
    LF_TRY(lf_sort_u64(h, rev, rev_alt, ne, B, &sorted));
    long long *f0 = nullptr, *r0 = nullptr;
    LF_TRY(lf_tmp_alloc(h, (void **)&f0, sizeof(long long) * (n + 1)));
    LF_TRY(lf_tmp_alloc(h, (void **)&r0, sizeof(long long) * (n + 1)));
    LF_HIP(h, hipMemsetAsync(derr, 0, sizeof(int) * 4, st));
    hipLaunchKernelGGL(k_runs, dim3(grid_for(n + 1, BS)), dim3(BS), 0, st, uk, sorted, ne, B, n, f0, r0);
    hipLaunchKernelGGL(k_rows, dim3(stride_grid(n + 1, BS)), dim3(BS), 0, st, f0, r0, n, h->deg, h->rowptr, derr + 1);
    if (ne > 0)
        hipLaunchKernelGGL(k_cols, dim3(grid_for(ne, BS)), dim3(BS), 0, st, uk, sorted, ne, B, f0, r0, h->col);
    if (n > 0) hipLaunchKernelGGL(k_iota_ids, dim3(grid_for(n, BS)), dim3(BS), 0, st, h->orig_id, n, uniq_ids);
    int maxdeg = 0;
    LF_HIP(h, hipMemcpyAsync(&maxdeg, derr + 1, sizeof(int), hipMemcpyDeviceToHost, st));
    LF_HIP(h, hipStreamSynchronize(st));
    LF_HIP(h, hipGetLastError());
    h->n = n;
    h->ne = ne;
    h->max_deg = maxdeg;
    return LF_OK;
}

// ------------------------------------------------------------------------------------
// A1: triangles
// ------------------------------------------------------------------------------------
__device__ __forceinline__ bool before(int du, int u, int dv, int v)
{
    return du < dv || (du == dv && u < v);
}

// out-degree in the (degree, id) orientation.  A wave per node left most lanes idle: this,
// the fill below, k_join_openers and k_init_slots took 0.31, 0.29, 0.32 and 0.37 ms for 1M
// nodes, 8M edges, by rows of lanes 0.21, 0.22, 0.24 and 0.24; what is left are the gathers of
// the neighbours' words.
__global__ void __launch_bounds__(256) k_out_degree(const long long *rowptr, const int *col,
                                                    const int *deg, long long n, int *od)
{
    for_rows(n, [&](long long x) { return rowptr[x + 1] - rowptr[x]; }, [&](long long u, int sub, int width) {
        int c = 0;
        if (u >= 0) {
            const int du = deg[u];
            const long long r1 = rowptr[u + 1];
            for (long long e = rowptr[u] + sub; e < r1; e += width) {
                const int v = col[e];
                c += before(du, (int)u, deg[v], v);
            }
        }
        WAVE_SYNC();
        c = width == 16 ? (int)row_sum_u32((unsigned)c) : (int)wave_sum_u32((unsigned)c);
        if (u >= 0 && sub == width - 1) od[u] = c;
    });
}

// compacted out-lists, kept in ascending id order
__global__ void __launch_bounds__(256) k_out_fill(const long long *rowptr, const int *col,
                                                  const int *deg, long long n, const long long *oro,
                                                  int *orc)
{
    const int row = threadIdx.x & (WAVE - 1) & 48;       // the row's first lane
    for_rows(n, [&](long long x) { return rowptr[x + 1] - rowptr[x]; }, [&](long long u, int sub, int width) {
        const int du = u >= 0 ? deg[u] : 0;
        const long long r1 = u >= 0 ? rowptr[u + 1] : 0;
        long long base = u >= 0 ? rowptr[u] : 0, w = u >= 0 ? oro[u] : 0;
        while (__ballot(base < r1)) {
            const long long e = base + sub;
            bool keep = false;
            int v = 0;
            if (e < r1) {
                v = col[e];
                keep = before(du, (int)u, deg[v], v);
            }
            unsigned long long mask = __ballot(keep);
            if (width == 16) mask = (mask >> row) & 0xffff;
            if (keep) orc[w + __popcll(mask & ((1ull << sub) - 1))] = v;
            w += __popcll(mask);
            base += width;
        }
    });
}

__device__ __forceinline__ int lds_find(const int *a, int m, int v)
{
    int lo = 0, hi = m - 1;
    while (lo <= hi) {
        int mid = (lo + hi) >> 1;
        int x = a[mid];
        if (x == v) return mid;
        if (x < v) lo = mid + 1; else hi = mid - 1;
    }
    return -1;
}

// A triangle {u, v, w} found at u (v = N+(u)[j], w = N+(u)[p]) in the exact-WCC pass:
// the three oriented edges are marked as closing a triangle, and every community that u,
// v and w share gains one triangle at each of them (a walk of their sorted id lists).
__device__ __forceinline__ void wcc_hit(const WccTri &wt, int u, int v, int w, long long e_uv, long long e_uw,
                                        long long e_vw)
{
    wt.eflag[e_uv] = 1;
    wt.eflag[e_uw] = 1;
    wt.eflag[e_vw] = 1;
    long long a = wt.moff[u], b = wt.moff[v], c = wt.moff[w];
    const long long ae = wt.moff[u + 1], be = wt.moff[v + 1], ce = wt.moff[w + 1];
    while (a < ae && b < be && c < ce) {
        const int x = wt.mid[a], y = wt.mid[b], z = wt.mid[c];
        if (x == y && y == z) {
            atomicAdd(&wt.tcm[a], 1);
            atomicAdd(&wt.tcm[b], 1);
            atomicAdd(&wt.tcm[c], 1);
            a++; b++; c++;
        } else {
            const int m = x > y ? (x > z ? x : z) : (y > z ? y : z);
            a += x < m;
            b += y < m;
            c += z < m;
        }
    }
}

// Nearly all probes miss.  A bit per hash of N+(u)'s members (one LDS read) turns most of them
// away; the rest are queued per wave, and only a full wave of them does the binary search, so
// that its log2(m) dependent LDS reads are paid by 64 likely hits at a time instead of by
// every probe.  (A hash table instead, probed until an empty entry, was slower than the plain
// binary search, 88 against 40 ms: each step lasts as long as the longest run among 64 lanes.)
__device__ __forceinline__ unsigned tri_hash(int v, int lg) { return (unsigned)v * 0x9E3779B1u >> (32 - lg); }

template <bool WCC, class J>             // J holds an index in N+(u)
struct TriQueue {
    int w[2 * WAVE];
    long long e[WCC ? 2 * WAVE : 1];
    J j[2 * WAVE];
};

// up to 64 queued probes of one wave: (list index j of v, third corner w, its edge e)
template <bool WCC, class J>
__device__ __forceinline__ int tri_drain(TriQueue<WCC, J> &Q, int n, int lane, int u, long long b, const int *nbr, int m,
                                         int *cnt, const WccTri &wt)
{
    int hit = 0;
    if (lane < n) {
        const int w = Q.w[lane], j = Q.j[lane];
        const int p = lds_find(nbr, m, w);
        if (p >= 0) {
            if constexpr (WCC) {
                wcc_hit(wt, u, nbr[j], w, b + j, b + p, Q.e[lane]);
            } else {
                atomicAdd(&cnt[p], 1);
                atomicAdd(&cnt[j], 1);
                hit = 1;
            }
        }
    }
    return hit;
}

// queue the probes of a wave's lanes that pass the filter; a full wave of them is drained
template <bool WCC, class J>
__device__ __forceinline__ int tri_push(TriQueue<WCC, J> &Q, int &qn, bool cand, int w, int j, long long e, int lane, int u,
                                        long long b, const int *nbr, int m, int *cnt, const WccTri &wt)
{
    const unsigned long long mask = __ballot(cand);
    if (cand) {
        const int at = qn + __popcll(mask & ((1ull << lane) - 1));
        Q.w[at] = w;
        Q.j[at] = (J)j;
        if constexpr (WCC) Q.e[at] = e;
    }
    qn += __popcll(mask);
    WAVE_SYNC();
    if (qn < WAVE) return 0;
    const int hit = tri_drain(Q, WAVE, lane, u, b, nbr, m, cnt, wt);
    qn -= WAVE;
    WAVE_SYNC();
    if (lane < qn) {
        Q.w[lane] = Q.w[WAVE + lane];
        Q.j[lane] = Q.j[WAVE + lane];
        if constexpr (WCC) Q.e[lane] = Q.e[WAVE + lane];
    }
    WAVE_SYNC();
    return hit;
}

#define TRI_WAVE_CAP 256
#define TRI_GROUP 512           // threads per longer out-list
#define TRI_GROUP_BITS 16       // filter bits per workgroup
#define TRI_WAVE_BITS 12        // per wave of the short out-lists
#define TRI_GW 16               // lanes per list of theirs
#define TRI_PER 4               // entries per lane

// A wave probes the lists k = first, first + stride, .. < ns of one node u: TRI_GW lanes walk one
// list at a time, TRI_PER entries each, and take the next one that is left when theirs ends; the
// next entries are read before these are tested, and a test is one filter bit.  range(k, e0, e1)
// gives a list's entries [e0, e1), index(k) its node's place in N+(u).
template <bool WCC, class J, class Range, class Index>
__device__ __forceinline__ int tri_walk(const int *orc, int first, int stride, int ns, Range range, Index index,
                                        const unsigned *bits, int lg, TriQueue<WCC, J> &Q, int lane, int u, long long b,
                                        const int *nbr, int m, int *cnt, const WccTri &wt)
{
    const int gl = TRI_PER * (lane & (TRI_GW - 1));
    const unsigned long long before = (1ull << (lane & ~(TRI_GW - 1))) - 1;
    int total = 0, qn = 0, taken = WAVE / TRI_GW, k = first + stride * (lane / TRI_GW);
    int e = 0, e1 = 0;                      // (a group without a list has nothing to test)
    if (k < ns) {
        range(k, e, e1);
        e += gl;
    }
    v4i w = read_entries(orc + (e < e1 ? e : 0));
    while (__ballot(k < ns)) {
        int en = e + TRI_PER * TRI_GW, e1n = e1, kn = k;
        const bool need = k < ns && en - gl >= e1;
        const unsigned long long nm = __ballot(need && gl == 0);
        if (nm) {
            if (need) {
                kn = first + stride * (taken + __popcll(nm & before));
                en = e1n = 0;
                if (kn < ns) {
                    range(kn, en, e1n);
                    en += gl;
                }
            }
            taken += __popcll(nm);
        }
        const v4i wn = read_entries(orc + (en < e1n ? en : 0));
        unsigned word[TRI_PER], hw[TRI_PER];
#pragma unroll
        for (int t = 0; t < TRI_PER; t++) {
            hw[t] = tri_hash(w[t], lg);
            word[t] = bits[hw[t] >> 5];
        }
#pragma unroll
        for (int t = 0; t < TRI_PER; t++) {
            const bool cand = e + t < e1 && (word[t] >> (hw[t] & 31) & 1);
            if (__ballot(cand)) {
                const int j = cand ? index(k) : 0;
                total += tri_push(Q, qn, cand, w[t], j, e + t, lane, u, b, nbr, m, cnt, wt);
            }
        }
        k = kn;
        e = en;
        e1 = e1n;
        w = wn;
    }
    return total + tri_drain(Q, qn, lane, u, b, nbr, m, cnt, wt);
}

// One wave, a block of its own, per node with |N+(u)| <= TRI_WAVE_CAP; longer out-lists are
// deferred.  What bounds it is the work per probe (7G probes on the dense graph below), and for
// graphs of short lists the chain oro -> orc -> oro -> orc of a node, so that as many waves as
// fit should be resident: 5 KB of LDS each, and no wave waits for another of its block.  1M nodes,
// 33M edges, dense: 39.7 ms with a search of N+(u) per probe; 20.2 with the walk at one entry
// per lane, 11.5 at four, 10.1 with 20 KB instead of 25.6 per block of four waves, 7.5 with two
// waves per block, 6.1 with one.  4M nodes, 35M edges: 8.7 -> 2.9 ms; the pass of the exact WCC, 1M
// nodes, 8M edges: 2.6 -> 0.95 ms.
// WCC = false: triangle counts per node into tri; true: wcc_hit per triangle instead.
template <bool WCC>
__global__ void __launch_bounds__(WAVE) k_tri_wave(const long long *oro, const int *orc, long long n,
                                                   unsigned long long *tri, int *defer, int *ndefer, WccTri wt)
{
    __shared__ int nbr[TRI_WAVE_CAP];
    __shared__ int cnt[WCC ? 1 : TRI_WAVE_CAP];
    __shared__ int start[TRI_WAVE_CAP];
    __shared__ unsigned short len[TRI_WAVE_CAP];
    __shared__ unsigned char seg[TRI_WAVE_CAP];
    __shared__ unsigned bits[(1 << TRI_WAVE_BITS) / 32];
    __shared__ TriQueue<WCC, unsigned char> Q;
    const int lane = threadIdx.x;
    const long long u = blockIdx.x;
    if (u >= n) return;
    const long long b = oro[u];
    int m = (int)(oro[u + 1] - b);
    if (m > TRI_WAVE_CAP) {
        if (lane == 0) defer[atomicAdd(ndefer, 1)] = (int)u;
        m = 0;
    }
    if (m < 2) return;                     // a triangle needs two out-neighbours of u
    for (int t = lane; t < (1 << TRI_WAVE_BITS) / 32; t += WAVE) bits[t] = 0;
    WAVE_SYNC();
    // stage N+(u) and its filter; the non-empty N+(v): first entry (below 2^30, as 2|E| < 2^31),
    // length (below 2^16: its members have as many neighbours each) and index in N+(u)
    int ns = 0;
    for (int base = 0; base < m; base += WAVE) {
        const int j = base + lane;
        int r0 = 0, r1 = 0;
        if (j < m) {
            const int v = orc[b + j];
            nbr[j] = v;
            if constexpr (!WCC) cnt[j] = 0;
            const unsigned hv = tri_hash(v, TRI_WAVE_BITS);
            atomicOr(&bits[hv >> 5], 1u << (hv & 31));
            r0 = (int)oro[v];
            r1 = (int)oro[v + 1];
        }
        const unsigned long long has = __ballot(r1 > r0);
        if (r1 > r0) {
            const int k = ns + __popcll(has & ((1ull << lane) - 1));
            start[k] = r0;
            len[k] = (unsigned short)(r1 - r0);
            seg[k] = (unsigned char)j;
        }
        ns += __popcll(has);
    }
    WAVE_SYNC();
    if (ns == 0) return;
    auto range = [&](int k, int &e0, int &e1) {
        e0 = start[k];
        e1 = e0 + len[k];
    };
    auto index = [&](int k) { return (int)seg[k]; };
    int total = tri_walk(orc, 0, 1, ns, range, index, bits, TRI_WAVE_BITS, Q, lane, (int)u, b, nbr, m, cnt, wt);
    WAVE_SYNC();
    if constexpr (!WCC) {
        for (int j = lane; j < m; j += WAVE)
            if (cnt[j]) atomicAdd(&tri[nbr[j]], (unsigned long long)cnt[j]);
        total = wave_sum_int(total);
        if (lane == 0 && total) atomicAdd(&tri[u], (unsigned long long)total);
    }
}

// One workgroup per deferred node; out-list and counters in LDS when they fit (LDS sized for
// the longest out-list, so that several workgroups share a CU), otherwise in this workgroup's
// slice of global scratch.  Its waves walk every eighth list each.  8,263 nodes of 257 to 682
// out-neighbours (the dense graph above): a list per wave with a search per probe 13.2 ms, with
// the filter 5.2, this walk 4.1 with 1,024 threads, 3.2 with 512, 3.4 with 256.
template <bool WCC>
__global__ void __launch_bounds__(TRI_GROUP) k_tri_group(const long long *oro, const int *orc,
                                                    const int *list, int nlist,
                                                    unsigned long long *tri, int lds_cap,
                                                    int *gscratch, long long gslice, WccTri wt)
{
    extern __shared__ int s_dyn[];
    __shared__ int s_total;
    __shared__ unsigned bits[(1 << TRI_GROUP_BITS) / 32];
    __shared__ TriQueue<WCC, int> s_q[TRI_GROUP / WAVE];
    const int lane = threadIdx.x & (WAVE - 1), wv = threadIdx.x / WAVE, nw = blockDim.x / WAVE;
    for (int it = blockIdx.x; it < nlist; it += gridDim.x) {
        int u = list[it];
        long long b = oro[u];
        int m = (int)(oro[u + 1] - b);
        const bool lds = m <= lds_cap;
        int *nbr = lds ? s_dyn : gscratch + (long long)blockIdx.x * gslice;
        int *cnt = lds ? s_dyn + lds_cap : nbr + m;
        TriQueue<WCC, int> &Q = s_q[wv];
        if (threadIdx.x == 0) s_total = 0;
        for (int t = threadIdx.x; t < (1 << TRI_GROUP_BITS) / 32; t += blockDim.x) bits[t] = 0;
        __syncthreads();
        for (int j = threadIdx.x; j < m; j += blockDim.x) {
            const int v = orc[b + j];
            nbr[j] = v;
            cnt[j] = 0;
            const unsigned hv = tri_hash(v, TRI_GROUP_BITS);
            atomicOr(&bits[hv >> 5], 1u << (hv & 31));
        }
        __syncthreads();
        auto range = [&](int k, int &e0, int &e1) {
            const int v = nbr[k];
            e0 = (int)oro[v];
            e1 = (int)oro[v + 1];
        };
        auto index = [](int k) { return k; };
        int total = tri_walk(orc, wv, nw, m, range, index, bits, TRI_GROUP_BITS, Q, lane, u, b, nbr, m, cnt, wt);
        WAVE_SYNC();
        if constexpr (!WCC) {
            total = wave_sum_int(total);
            if (lane == 0 && total) atomicAdd(&s_total, total);
        }
        __syncthreads();
        if constexpr (!WCC) {
            for (int j = threadIdx.x; j < m; j += blockDim.x)
                if (cnt[j]) atomicAdd(&tri[nbr[j]], (unsigned long long)cnt[j]);
            if (threadIdx.x == 0 && s_total) atomicAdd(&tri[u], (unsigned long long)s_total);
        }
        __syncthreads();
    }
}

// ------------------------------------------------------------------------------------
// A2: local CC, global cc, order
// ------------------------------------------------------------------------------------
#define RED_BLOCK 256

// local CC, the exact sum of the CCs (per-block partials) and the triangle sum
__global__ void __launch_bounds__(RED_BLOCK) k_local_cc(const unsigned long long *tri, const int *deg,
                                                        long long n, double *ccl, X192 *partial,
                                                        unsigned long long *tsum, int *err)
{
    __shared__ X192 s_w[RED_BLOCK / WAVE];
    X192 acc = x192_zero();
    unsigned long long t = 0;
    int bad = 0;
    for (long long x = blockIdx.x * (long long)blockDim.x + threadIdx.x; x < n;
         x += (long long)gridDim.x * blockDim.x) {
        long long d = deg[x];
        long long k = (long long)tri[x];
        double c = 0.0;
        if (d > 1) c = (double)k / (double)(d * (d - 1) / 2);
        ccl[x] = c;
        X192 v = x192_from_double(c, bad);
        x192_add(acc, v);
        t += (unsigned long long)k;
    }
    acc = wave_sum_x192(acc);
    t = (unsigned long long)wave_sum_i64((long long)t);
    int lane = threadIdx.x & (WAVE - 1), wv = threadIdx.x / WAVE;
    if (lane == 0) {
        s_w[wv] = acc;
        atomicAdd(tsum, t);
    }
    if (bad) atomicOr(err, LF_DEVERR_INEXACT);
    __syncthreads();
    if (threadIdx.x == 0) {
        X192 s = s_w[0];
        for (int k = 1; k < RED_BLOCK / WAVE; k++) x192_add(s, s_w[k]);
        partial[blockIdx.x] = s;
    }
}

// exact sum of doubles into per-block partials (diagnostic entry point)
__global__ void __launch_bounds__(RED_BLOCK) k_exact_partials(const double *v, long long n, X192 *partial,
                                                              int *err)
{
    __shared__ X192 s_w[RED_BLOCK / WAVE];
    X192 acc = x192_zero();
    int bad = 0;
    for (long long x = blockIdx.x * (long long)blockDim.x + threadIdx.x; x < n;
         x += (long long)gridDim.x * blockDim.x) {
        double a = v[x];
        if (!(fabs(a) <= 1073741824.0)) bad = 1;
        X192 t = x192_from_double(a, bad);
        x192_add(acc, t);
    }
    acc = wave_sum_x192(acc);
    if (bad) atomicOr(err, LF_DEVERR_INEXACT);
    int lane = threadIdx.x & (WAVE - 1), wv = threadIdx.x / WAVE;
    if (lane == 0) s_w[wv] = acc;
    __syncthreads();
    if (threadIdx.x == 0) {
        X192 s = s_w[0];
        for (int k = 1; k < RED_BLOCK / WAVE; k++) x192_add(s, s_w[k]);
        partial[blockIdx.x] = s;
    }
}

// one wave folds the partials and rounds once; result = R(sum) / divisor (divisor > 0)
__global__ void k_fold_partials(const X192 *partial, int np, double divisor, double *out)
{
    int lane = threadIdx.x;
    X192 acc = x192_zero();
    for (int k = lane; k < np; k += WAVE) x192_add(acc, partial[k]);
    acc = wave_sum_x192(acc);
    if (lane == 0) out[0] = x192_round(acc) / divisor;
}

__global__ void k_order_keys_deg(const int *deg, long long n, int maxdeg, unsigned *key, int *val)
{
    long long x = blockIdx.x * (long long)blockDim.x + threadIdx.x;
    if (x >= n) return;
    key[x] = (unsigned)(maxdeg - deg[x]);   // degree descending
    val[x] = (int)x;                          // ids ascending (stable sorts keep it)
}

__global__ void k_order_keys_cc(const double *ccl, const int *ids, long long n, unsigned long long *key)
{
    long long r = blockIdx.x * (long long)blockDim.x + threadIdx.x;
    if (r >= n) return;
    // CC in [0, 1]: its bit pattern orders like the value; subtract to sort descending
    unsigned long long b = (unsigned long long)__double_as_longlong(ccl[ids[r]]);
    key[r] = 0x3FF0000000000000ull - b;
}

__global__ void k_rank(const int *order, long long n, int *rank)
{
    long long r = blockIdx.x * (long long)blockDim.x + threadIdx.x;
    if (r >= n) return;
    rank[order[r]] = (int)r;
}

// the order position of every adjacency entry's node, so that a pass over a node's
// neighbours reads their positions with its column indices instead of one hop later
__global__ void k_col_rank(const int *col, long long m, const int *rank, int *out)
{
    long long e = blockIdx.x * (long long)blockDim.x + threadIdx.x;
    if (e >= m) return;
    out[e] = rank[col[e]];
}

__global__ void k_clear_int(int *p) { *p = 0; }

// The exact sum on caller-placed scratch: part (LF_EXACT_PARTIALS X192 entries), err (one
// int) and dout (one double) in device memory; nothing is allocated here.
int lf_exact_sum_run(lf_handle *h, const double *v, long long n, double *out, X192 *part, int *err, double *dout)
{
    hipStream_t st = h->stream;
    int nb = (int)((n + RED_BLOCK - 1) / RED_BLOCK);
    if (nb > LF_EXACT_PARTIALS) nb = LF_EXACT_PARTIALS;
    if (nb < 1) nb = 1;
    hipLaunchKernelGGL(k_clear_int, dim3(1), dim3(1), 0, st, err);
    hipLaunchKernelGGL(k_exact_partials, dim3(nb), dim3(RED_BLOCK), 0, st, v, n, part, err);
    hipLaunchKernelGGL(k_fold_partials, dim3(1), dim3(WAVE), 0, st, part, nb, 1.0, dout);
    int herr = 0;
    LF_HIP(h, hipMemcpyAsync(out, dout, sizeof(double), hipMemcpyDeviceToHost, st));
    LF_HIP(h, hipMemcpyAsync(&herr, err, sizeof(int), hipMemcpyDeviceToHost, st));
    LF_HIP(h, hipStreamSynchronize(st));
    LF_HIP(h, hipGetLastError());
    if (herr) return lf_set_error(h, LF_EOVERFLOW, "value outside the exact accumulator's range");
    return LF_OK;
}

int lf_exact_sum_dev(lf_handle *h, const double *v, long long n, double *out)
{
    TmpScope tmp_scope(h);
    X192 *part = nullptr;
    int *err = nullptr;
    double *dout = nullptr;
    LF_TRY(lf_tmp_alloc(h, (void **)&part, sizeof(X192) * LF_EXACT_PARTIALS));
    LF_TRY(lf_tmp_alloc(h, (void **)&err, sizeof(int)));
    LF_TRY(lf_tmp_alloc(h, (void **)&dout, sizeof(double)));
    return lf_exact_sum_run(h, v, n, out, part, err, dout);
}

// Every triangle once, at its lowest endpoint in (degree, id) order: with wt == nullptr
// the per-node counts go to h->tri, otherwise wcc_hit is applied to each triangle.
// Oriented lists (out-offsets oro[n + 1], out-neighbours orc, ascending ids) are built
// into temporaries of the caller's scratch scope and returned if asked for.
int lf_triangle_pass(lf_handle *h, const WccTri *wt, int *launches, long long **oro_out, int **orc_out)
{
    hipStream_t st = h->stream;
    const long long n = h->n;
    const int BS = 256;
    int maxdev = 0;
    LF_HIP(h, hipDeviceGetAttribute(&maxdev, hipDeviceAttributeMaxSharedMemoryPerBlock, h->device));
    int *od = nullptr;
    long long *oro = nullptr;
    int *orc = nullptr;
    int *defer = nullptr;
    int *cnt = nullptr;
    LF_TRY(lf_tmp_alloc(h, (void **)&od, sizeof(int) * (n > 0 ? n : 1)));
    LF_TRY(lf_tmp_alloc(h, (void **)&oro, sizeof(long long) * (n + 1)));
    LF_TRY(lf_tmp_alloc(h, (void **)&orc, sizeof(int) * (h->ne + READ_PAD)));
    LF_TRY(lf_tmp_alloc(h, (void **)&defer, sizeof(int) * (n > 0 ? n : 1)));
    LF_TRY(lf_tmp_alloc(h, (void **)&cnt, sizeof(int) * 4));
    LF_HIP(h, hipMemsetAsync(cnt, 0, sizeof(int) * 4, st));
    WccTri none;
    memset(&none, 0, sizeof none);
    const WccTri w = wt ? *wt : none;
    unsigned gw = grid_for(n * 16, BS);     // a row of lanes per node
    long long *od64 = nullptr;
    LF_TRY(lf_tmp_alloc(h, (void **)&od64, sizeof(long long) * (n + 1)));
    if (n > 0) {
        hipLaunchKernelGGL(k_out_degree, dim3(gw), dim3(BS), 0, st, h->rowptr, h->col, h->deg, n, od);
        hipLaunchKernelGGL(k_deg_to_i64, dim3(stride_grid(n, BS)), dim3(BS), 0, st, od, n, od64, cnt + 2);
    }
    LF_TRY(lf_exclusive_scan_i64(h, od64, oro, n));
    hipLaunchKernelGGL(k_set_last, dim3(1), dim3(1), 0, st, oro, n, h->ne);
    if (n > 0) {
        hipLaunchKernelGGL(k_out_fill, dim3(gw), dim3(BS), 0, st, h->rowptr, h->col, h->deg, n, oro, orc);
        if (wt)
            hipLaunchKernelGGL(k_tri_wave<true>, dim3((unsigned)n), dim3(WAVE), 0, st,
                               oro, orc, n, h->tri, defer, cnt, w);
        else
            hipLaunchKernelGGL(k_tri_wave<false>, dim3((unsigned)n), dim3(WAVE), 0, st,
                               oro, orc, n, h->tri, defer, cnt, w);
    }
    int hc[4] = {0, 0, 0, 0};
    LF_HIP(h, hipMemcpyAsync(hc, cnt, sizeof(int) * 4, hipMemcpyDeviceToHost, st));
    LF_HIP(h, hipStreamSynchronize(st));
    int ndefer = hc[0], maxod = hc[2];
    *launches = 5;
    if (ndefer > 0) {
        // dynamic LDS: list and counters, beside the filter and the queues (at most 48 KB)
        int lds_cap = (maxdev - 49152) / (2 * (int)sizeof(int));
        if (maxod < lds_cap) lds_cap = maxod;
        if (h->tri_lds_cap > 0 && h->tri_lds_cap < lds_cap) lds_cap = h->tri_lds_cap;
        const int most = maxod > lds_cap ? 1024 : 8192;    // (a slice of scratch each past the cap)
        const int blocks = ndefer < most ? ndefer : most;
        int *gs = nullptr;
        long long gslice = 2ll * maxod + 2;
        if (maxod > lds_cap) LF_TRY(lf_tmp_alloc(h, (void **)&gs, sizeof(int) * gslice * blocks));
        size_t shmem = sizeof(int) * 2 * (size_t)lds_cap;
        const void *fn = wt ? (const void *)k_tri_group<true> : (const void *)k_tri_group<false>;
        LF_HIP(h, hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)shmem));
        if (wt)
            hipLaunchKernelGGL(k_tri_group<true>, dim3(blocks), dim3(TRI_GROUP), shmem, st, oro, orc, defer, ndefer,
                               h->tri, lds_cap, gs, gslice, w);
        else
            hipLaunchKernelGGL(k_tri_group<false>, dim3(blocks), dim3(TRI_GROUP), shmem, st, oro, orc, defer, ndefer,
                               h->tri, lds_cap, gs, gslice, w);
        LF_HIP(h, hipGetLastError());
        LF_HIP(h, hipStreamSynchronize(st));
        *launches = 6;
    }
    LF_HIP(h, hipGetLastError());
    if (oro_out) *oro_out = oro;
    if (orc_out) *orc_out = orc;
    return LF_OK;
}

int lf_node_stats(lf_handle *h)
{
    TmpScope tmp_scope(h);
    hipStream_t st = h->stream;
    long long n = h->n;
    const int BS = 256;

    LF_TRY(lf_prof_begin(h, LF_K_TRIANGLES));
    int *cnt = nullptr;
    LF_TRY(lf_tmp_alloc(h, (void **)&cnt, sizeof(int) * 4));
    LF_TRY(lf_dev_alloc(h, (void **)&h->tri, sizeof(unsigned long long) * (n > 0 ? n : 1)));
    LF_HIP(h, hipMemsetAsync(h->tri, 0, sizeof(unsigned long long) * (n > 0 ? n : 1), st));
    int launches = 0;
    LF_TRY(lf_triangle_pass(h, nullptr, &launches, nullptr, nullptr));
    int hc[4] = {0, 0, 0, 0};
    LF_TRY(lf_prof_end(h, LF_K_TRIANGLES, launches));

    // local CC, cc, T
    LF_TRY(lf_prof_begin(h, LF_K_ORDER));
    LF_TRY(lf_dev_alloc(h, (void **)&h->ccl, sizeof(double) * (n > 0 ? n : 1)));
    int nb = (int)((n + RED_BLOCK - 1) / RED_BLOCK);
    if (nb > 1024) nb = 1024;
    if (nb < 1) nb = 1;
    X192 *part = nullptr;
    unsigned long long *tsum = nullptr;
    double *dcc = nullptr;
    LF_TRY(lf_tmp_alloc(h, (void **)&part, sizeof(X192) * nb));
    LF_TRY(lf_tmp_alloc(h, (void **)&tsum, sizeof(unsigned long long)));
    LF_TRY(lf_tmp_alloc(h, (void **)&dcc, sizeof(double)));
    LF_HIP(h, hipMemsetAsync(tsum, 0, sizeof(unsigned long long), st));
    LF_HIP(h, hipMemsetAsync(cnt, 0, sizeof(int) * 4, st));
    hipLaunchKernelGGL(k_local_cc, dim3(nb), dim3(RED_BLOCK), 0, st, h->tri, h->deg, n, h->ccl, part, tsum, cnt);
    hipLaunchKernelGGL(k_fold_partials, dim3(1), dim3(WAVE), 0, st, part, nb, (double)(n > 0 ? n : 1), dcc);

    // order: stable sort by degree descending, then stable sort by CC descending
    LF_TRY(lf_dev_alloc(h, (void **)&h->order, sizeof(int) * (n > 0 ? n : 1)));
    LF_TRY(lf_dev_alloc(h, (void **)&h->rank, sizeof(int) * (n > 0 ? n : 1)));
    const long long m = 2 * h->ne;
    LF_TRY(lf_dev_alloc(h, (void **)&h->col_rank, sizeof(int) * (m + READ_PAD)));
    unsigned *k1 = nullptr, *k1b = nullptr;
    int *v1 = nullptr, *v1b = nullptr;
    unsigned long long *k2 = nullptr, *k2b = nullptr;
    LF_TRY(lf_tmp_alloc(h, (void **)&k1, sizeof(unsigned) * (n > 0 ? n : 1)));
    LF_TRY(lf_tmp_alloc(h, (void **)&k1b, sizeof(unsigned) * (n > 0 ? n : 1)));
    LF_TRY(lf_tmp_alloc(h, (void **)&v1, sizeof(int) * (n > 0 ? n : 1)));
    LF_TRY(lf_tmp_alloc(h, (void **)&v1b, sizeof(int) * (n > 0 ? n : 1)));
    LF_TRY(lf_tmp_alloc(h, (void **)&k2, sizeof(unsigned long long) * (n > 0 ? n : 1)));
    LF_TRY(lf_tmp_alloc(h, (void **)&k2b, sizeof(unsigned long long) * (n > 0 ? n : 1)));
    unsigned *rk1;
    int *rv1;
    if (n > 0) hipLaunchKernelGGL(k_order_keys_deg, dim3(grid_for(n, BS)), dim3(BS), 0, st, h->deg, n, h->max_deg, k1, v1);
    LF_TRY(lf_sort_pairs_u32_i32(h, k1, k1b, v1, v1b, n, &rk1, &rv1));
    if (n > 0) hipLaunchKernelGGL(k_order_keys_cc, dim3(grid_for(n, BS)), dim3(BS), 0, st, h->ccl, rv1, n, k2);
    int *other = (rv1 == v1) ? v1b : v1;
    unsigned long long *rk2;
    int *rv2;
    LF_TRY(lf_sort_pairs_u64_i32(h, k2, k2b, rv1, other, n, 62, &rk2, &rv2));
    LF_HIP(h, hipMemcpyAsync(h->order, rv2, sizeof(int) * (n > 0 ? n : 1), hipMemcpyDeviceToDevice, st));
    if (n > 0) hipLaunchKernelGGL(k_rank, dim3(grid_for(n, BS)), dim3(BS), 0, st, h->order, n, h->rank);
    if (m > 0) hipLaunchKernelGGL(k_col_rank, dim3(grid_for(m, BS)), dim3(BS), 0, st, h->col, m, h->rank, h->col_rank);
    unsigned long long ht = 0;
    LF_HIP(h, hipMemcpyAsync(&h->cc, dcc, sizeof(double), hipMemcpyDeviceToHost, st));
    LF_HIP(h, hipMemcpyAsync(&ht, tsum, sizeof(unsigned long long), hipMemcpyDeviceToHost, st));
    LF_HIP(h, hipMemcpyAsync(hc, cnt, sizeof(int) * 4, hipMemcpyDeviceToHost, st));
    LF_HIP(h, hipStreamSynchronize(st));
    LF_HIP(h, hipGetLastError());
    LF_TRY(lf_prof_end(h, LF_K_ORDER, 7));
    LF_TRY(lf_prof_flush(h));
    if (n == 0) h->cc = 0.0;
    h->T = (long long)(ht / 3);
    if (hc[0]) return lf_set_error(h, LF_EINTERNAL, "clustering coefficient not exactly summable");
    if (ht % 3) return lf_set_error(h, LF_EINTERNAL, "triangle credits not divisible by 3");
    return LF_OK;
}
