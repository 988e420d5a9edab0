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
// out-lists) stages N+(u) in LDS, walks the concatenation of N+(v) over v in N+(u) with
// all its lanes, and binary-searches each w in the staged N+(u).  A hit credits u, v and
// w; the credits of v and w (both in N+(u)) are accumulated in LDS counters and flushed
// to HBM once per (u, position).
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

__device__ __forceinline__ long long find_sorted_u64(const unsigned long long *a, long long n,
                                                     unsigned long long v)
{
    long long lo = 0, hi = n - 1;
    while (lo <= hi) {
        long long mid = lo + ((hi - lo) >> 1);
        unsigned long long x = a[mid];
        if (x == v) return mid;
        if (x < v) lo = mid + 1; else hi = mid - 1;
    }
    return -1;
}

// canonical (min, max) keys; self-loops -> sentinel; ids checked or remapped
__global__ void k_canon_keys(const long long *src, const long long *dst, long long np, long long n,
                             const unsigned long long *uniq_ids, int B, unsigned long long *keys,
                             int *err)
{
    long long e = blockIdx.x * (long long)blockDim.x + threadIdx.x;
    if (e >= np) return;
    long long a = src[e], b = dst[e];
    unsigned long long sentinel = (B >= 32) ? ~0ull : ((1ull << (2 * B)) - 1);
    if (a == b) { keys[e] = sentinel; return; }
    if (uniq_ids) {
        a = find_sorted_u64(uniq_ids, n, (unsigned long long)a);
        b = find_sorted_u64(uniq_ids, n, (unsigned long long)b);
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
    if (np > 0)
        hipLaunchKernelGGL(k_canon_keys, dim3(grid_for(np, BS)), dim3(BS), 0, st, dsrc, ddst, np, n,
                           uniq_ids, B, ka, derr);
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
    LF_TRY(lf_dev_alloc(h, (void **)&h->col, sizeof(int) * (2 * ne > 0 ? 2 * ne : 1)));
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

// out-degree in the (degree, id) orientation; one wave per node
__global__ void __launch_bounds__(256) k_out_degree(const long long *rowptr, const int *col,
                                                    const int *deg, long long n, int *od)
{
    long long u = (blockIdx.x * (long long)blockDim.x + threadIdx.x) / WAVE;
    int lane = threadIdx.x & (WAVE - 1);
    if (u >= n) return;
    int du = deg[u];
    int c = 0;
    for (long long e = rowptr[u] + lane; e < rowptr[u + 1]; e += WAVE) {
        int v = col[e];
        c += before(du, (int)u, deg[v], v);
    }
    c = wave_sum_int(c);
    if (lane == 0) od[u] = c;
}

// compacted out-lists, kept in ascending id order
__global__ void __launch_bounds__(256) k_out_fill(const long long *rowptr, const int *col,
                                                  const int *deg, long long n, const long long *oro,
                                                  int *orc)
{
    long long u = (blockIdx.x * (long long)blockDim.x + threadIdx.x) / WAVE;
    int lane = threadIdx.x & (WAVE - 1);
    if (u >= n) return;
    int du = deg[u];
    long long w = oro[u];
    for (long long base = rowptr[u]; base < rowptr[u + 1]; base += WAVE) {
        long long e = base + lane;
        bool keep = false;
        int v = 0;
        if (e < rowptr[u + 1]) {
            v = col[e];
            keep = before(du, (int)u, deg[v], v);
        }
        unsigned long long mask = __ballot(keep);
        int rank = __popcll(mask & ((1ull << lane) - 1));
        if (keep) orc[w + rank] = v;
        w += __popcll(mask);
    }
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
// every probe.  k_tri_group on 1M nodes, 39M edges: 13.2 -> 5.2 ms.  (A hash table instead,
// probed until an empty entry, was slower than the plain binary search, 88 against 40 ms in
// k_tri_wave: each step lasts as long as the longest run among 64 lanes.)
__device__ __forceinline__ unsigned tri_hash(int v, int lg) { return (unsigned)v * 0x9E3779B1u >> (32 - lg); }

template <bool WCC>
struct TriQueue {
    int w[2 * WAVE], j[2 * WAVE];
    long long e[WCC ? 2 * WAVE : 1];
};

// up to 64 queued probes of one wave: (list index j of v, third corner w, its edge e)
template <bool WCC>
__device__ __forceinline__ int tri_drain(TriQueue<WCC> &Q, int n, int lane, int u, long long b, const int *nbr, int m,
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
template <bool WCC>
__device__ __forceinline__ int tri_push(TriQueue<WCC> &Q, int &qn, bool cand, int w, int j, long long e, int lane, int u,
                                        long long b, const int *nbr, int m, int *cnt, const WccTri &wt)
{
    const unsigned long long mask = __ballot(cand);
    if (cand) {
        const int at = qn + __popcll(mask & ((1ull << lane) - 1));
        Q.w[at] = w;
        Q.j[at] = j;
        if constexpr (WCC) Q.e[at] = e;
    }
    qn += __popcll(mask);
    WAVE_SYNC();
    if (qn < WAVE) return 0;
    const int hit = tri_drain<WCC>(Q, WAVE, lane, u, b, nbr, m, cnt, wt);
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
#define TRI_GROUP_BITS 16       // filter bits per workgroup
#define TRI_WAVES 4

// the wave's bitwise or of x (every lane active)
__device__ __forceinline__ unsigned op_or(unsigned a, unsigned b) { return a | b; }
__device__ __forceinline__ unsigned wave_or_u32(unsigned x)
{
    DPP_INCLUSIVE(x, op_or);
    return (unsigned)__builtin_amdgcn_readlane((int)x, WAVE - 1);
}

// one wave per node with |N+(u)| <= TRI_WAVE_CAP; longer out-lists are deferred.  The waves
// of a block share nothing and never meet: with block barriers around the probe loop a
// block lasted as long as the heaviest of its four nodes.  Probes are taken 64 at a time;
// which out-neighbour's list a lane is in follows from one mask of the list starts within
// the 64 (empty lists are left out) instead of a binary search per probe.  What bounds it is
// the search of w in N+(u), log2(m) dependent LDS reads.  Measured: 4M nodes, 35M edges
// 11.1 -> 8.7 ms; 1M nodes, 39M edges, dense 54.4 -> 39.7 ms.  With k_tri_group's filter and
// queue here too: 9.4 and 37.1 ms, their LDS leaving fewer waves on a CU.
// WCC = false: triangle counts per node into tri; true: wcc_hit per triangle instead.
template <bool WCC>
__global__ void __launch_bounds__(256) k_tri_wave(const long long *oro, const int *orc, long long n,
                                                  unsigned long long *tri, int *defer, int *ndefer, WccTri wt)
{
    __shared__ int s_nbr[TRI_WAVES][TRI_WAVE_CAP];
    __shared__ int s_pre[TRI_WAVES][TRI_WAVE_CAP];
    __shared__ int s_cnt[TRI_WAVES][TRI_WAVE_CAP];
    __shared__ short s_seg[TRI_WAVES][TRI_WAVE_CAP];
    int wv = threadIdx.x / WAVE, lane = threadIdx.x & (WAVE - 1);
    long long u = blockIdx.x * (long long)TRI_WAVES + wv;
    long long b = 0;
    int m = 0;
    if (u < n) {
        b = oro[u];
        m = (int)(oro[u + 1] - b);
    }
    if (m > TRI_WAVE_CAP) {
        if (lane == 0) defer[atomicAdd(ndefer, 1)] = (int)u;
        m = 0;
    }
    if (m < 2) m = 0;                      // a triangle needs two out-neighbours of u
    int *nbr = s_nbr[wv], *pre = s_pre[wv], *cnt = s_cnt[wv];
    short *seg = s_seg[wv];
    // stage N+(u); the non-empty N+(v): their index in N+(u) and first probe
    int W = 0, ns = 0;                      // probes, non-empty lists
    for (int base = 0; base < m; base += WAVE) {
        const int j = base + lane;
        int len = 0;
        if (j < m) {
            const int v = orc[b + j];
            nbr[j] = v;
            cnt[j] = 0;
            len = (int)(oro[v + 1] - oro[v]);
        }
        int tot;
        const int incl = wave_incl_scan(len, &tot);
        const unsigned long long has = __ballot(len > 0);
        if (len > 0) {
            const int k = ns + __popcll(has & ((1ull << lane) - 1));
            pre[k] = W + incl - len;
            seg[k] = (short)j;
        }
        W += tot;
        ns += __popcll(has);
    }
    WAVE_SYNC();
    int total = 0;
    int s0 = 0;                             // list of the chunk's first probe
    for (int f0 = 0; f0 < W; f0 += WAVE) {  // same trip count on every lane
        // list starts after f0 within the chunk: at most 63 of them, in lists s0 + 1 ..
        const int q = s0 + 1 + lane;
        const int at = q < ns ? pre[q] - f0 : WAVE;
        const unsigned lo = wave_or_u32(at < 32 ? 1u << at : 0u);
        const unsigned hi = wave_or_u32(at >= 32 && at < WAVE ? 1u << (at - 32) : 0u);
        const unsigned long long starts = ((unsigned long long)hi << 32) | lo;
        const int f = f0 + lane;
        if (f < W) {
            const int s = s0 + __popcll(starts & ((2ull << lane) - 1));
            const int j = seg[s], v = nbr[j];
            const long long evw = oro[v] + (f - pre[s]);
            const int w = orc[evw];
            const int p = lds_find(nbr, m, w);
            if (p >= 0) {
                if constexpr (WCC) {
                    wcc_hit(wt, (int)u, v, w, b + j, b + p, evw);
                } else {
                    atomicAdd(&cnt[p], 1);
                    atomicAdd(&cnt[j], 1);
                    total++;
                }
            }
        }
        s0 += __popcll(starts);
        // the next chunk may open exactly at a list's start
        if (s0 + 1 < ns && pre[s0 + 1] == f0 + WAVE) s0++;
    }
    WAVE_SYNC();
    if constexpr (!WCC) {
        for (int j = lane; j < m; j += WAVE)
            if (cnt[j]) atomicAdd(&tri[nbr[j]], (unsigned long long)cnt[j]);
        total = wave_sum_int(total);
        if (lane == 0 && total) atomicAdd(&tri[u], (unsigned long long)total);
    }
}

// one workgroup per deferred node; out-list and counters in LDS when they fit (LDS sized for
// the longest out-list, so that two workgroups share a CU), otherwise in this workgroup's slice
// of global scratch.  A wave takes one N+(v) at a time (those of a hub's out-neighbours are
// long).
template <bool WCC>
__global__ void __launch_bounds__(1024) k_tri_group(const long long *oro, const int *orc,
                                                    const int *list, int nlist,
                                                    unsigned long long *tri, int lds_cap,
                                                    int *gscratch, long long gslice, WccTri wt)
{
    extern __shared__ int s_dyn[];
    __shared__ int s_total;
    __shared__ unsigned bits[(1 << TRI_GROUP_BITS) / 32];
    __shared__ TriQueue<WCC> s_q[1024 / WAVE];
    const int lane = threadIdx.x & (WAVE - 1), wv = threadIdx.x / WAVE, nw = blockDim.x / WAVE;
    for (int it = blockIdx.x; it < nlist; it += gridDim.x) {
        int u = list[it];
        long long b = oro[u];
        int m = (int)(oro[u + 1] - b);
        const bool lds = m <= lds_cap;
        int *nbr = lds ? s_dyn : gscratch + (long long)blockIdx.x * gslice;
        int *cnt = lds ? s_dyn + lds_cap : nbr + m;
        TriQueue<WCC> &Q = s_q[wv];
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
        int total = 0, qn = 0;
        for (int j = wv; j < m; j += nw) {
            const int v = nbr[j];
            const long long e1 = oro[v + 1];
            for (long long e0 = oro[v]; e0 < e1; e0 += WAVE) {
                const long long evw = e0 + lane;
                bool cand = false;
                int w = 0;
                if (evw < e1) {
                    w = orc[evw];
                    const unsigned hw = tri_hash(w, TRI_GROUP_BITS);
                    cand = (bits[hw >> 5] >> (hw & 31)) & 1;
                }
                WAVE_SYNC();
                total += tri_push<WCC>(Q, qn, cand, w, j, evw, lane, u, b, nbr, m, cnt, wt);
            }
        }
        total += tri_drain<WCC>(Q, qn, lane, u, b, nbr, m, cnt, wt);
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
    LF_TRY(lf_tmp_alloc(h, (void **)&orc, sizeof(int) * (h->ne > 0 ? h->ne : 1)));
    LF_TRY(lf_tmp_alloc(h, (void **)&defer, sizeof(int) * (n > 0 ? n : 1)));
    LF_TRY(lf_tmp_alloc(h, (void **)&cnt, sizeof(int) * 4));
    LF_HIP(h, hipMemsetAsync(cnt, 0, sizeof(int) * 4, st));
    WccTri none;
    memset(&none, 0, sizeof none);
    const WccTri w = wt ? *wt : none;
    unsigned gw = grid_for(n * WAVE, BS);
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
            hipLaunchKernelGGL(k_tri_wave<true>, dim3(grid_for(n, TRI_WAVES)), dim3(TRI_WAVES * WAVE), 0, st,
                               oro, orc, n, h->tri, defer, cnt, w);
        else
            hipLaunchKernelGGL(k_tri_wave<false>, dim3(grid_for(n, TRI_WAVES)), dim3(TRI_WAVES * WAVE), 0, st,
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
        int blocks = ndefer < 1024 ? ndefer : 1024;
        int *gs = nullptr;
        long long gslice = 2ll * maxod + 2;
        if (maxod > lds_cap) LF_TRY(lf_tmp_alloc(h, (void **)&gs, sizeof(int) * gslice * blocks));
        size_t shmem = sizeof(int) * 2 * (size_t)lds_cap;
        const void *fn = wt ? (const void *)k_tri_group<true> : (const void *)k_tri_group<false>;
        LF_HIP(h, hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)shmem));
        if (wt)
            hipLaunchKernelGGL(k_tri_group<true>, dim3(blocks), dim3(1024), shmem, st, oro, orc, defer, ndefer,
                               h->tri, lds_cap, gs, gslice, w);
        else
            hipLaunchKernelGGL(k_tri_group<false>, dim3(blocks), dim3(1024), shmem, st, oro, orc, defer, ndefer,
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
    LF_TRY(lf_dev_alloc(h, (void **)&h->col_rank, sizeof(int) * (m > 0 ? m : 1)));
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
