// method.h -- device arithmetic of the LazyFox method (WCC-hat node terms, community
// density, candidate changes), shared by the initialisation and the iteration kernels.
//
// WCC-hat (Methods, WCC-hat subsection): for a member x of community C with
// d = deg(x,V), i = deg(x,C), s = |C| and density p,
//     WCC-hat(x,C) = E[t(x,C)] / E[t(x,V)] * deg(x,V) / (|C\{x}| + deg(x,V\C))
// with E[t(x,C)] = C(i,2) p and E[t(x,V)] = C(d,2) cc, i.e. p * g(i,d,s) / cc with
//     g(i,d,s) = i(i-1) / ((d-1)(s-1+d-i)),   0 if i < 2 or d < 2 (E[t] = 0).
// cc is a positive constant, so the method's comparisons use the cc-free score
// W(C) = fl(p * R(sum_{y in C} g)), R = exact sum rounded once to nearest-even.
#pragma once
#include "lf_internal.h"

#define WAVE 64

#define WAVE_SYNC()                                                                        \
    do {                                                                                   \
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");                             \
        __builtin_amdgcn_wave_barrier();                                                   \
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");                             \
    } while (0)

// Numerator and denominator are products of two integers below 2^33, each exact in FP64, so
// one FP64 multiplication rounds the product exactly as a conversion of the 64-bit integer
// product would (half the instructions of the integer product and its conversion).
__device__ __forceinline__ double g_term(int i, int d, int s)
{
    if (d < 2 || i < 2) return 0.0;
    const double num = (double)i * (double)(i - 1);
    const double den = (double)(d - 1) * ((double)(s - 1) + (double)(d - i));
    return num / den;
}

// density of a community with s members and m internal edges
__device__ __forceinline__ double density(int s, long long m)
{
    if (s < 2) return 0.0;
    return (double)(2 * m) / ((double)s * (double)(s - 1));
}

__device__ __forceinline__ X192 rec_load(const unsigned *p)
{
    X192 r;
    r.w0 = (u64)p[0] | ((u64)p[1] << 32);
    r.w1 = (u64)p[2] | ((u64)p[3] << 32);
    r.w2 = (u64)p[4];
    return r;
}

__device__ __forceinline__ void rec_store(unsigned *p, const X192 &v, int &bad)
{
    p[0] = (unsigned)v.w0;
    p[1] = (unsigned)(v.w0 >> 32);
    p[2] = (unsigned)v.w1;
    p[3] = (unsigned)(v.w1 >> 32);
    p[4] = (unsigned)v.w2;
    if (v.w2 >> 32) bad = 1;           // a stored sum is never negative nor >= 2^40
}

// write a re-summed community (members' exact sums at sizes s, s+1, s-1 and in-count sum)
__device__ __forceinline__ void store_comm(const Ctx &cx, int C, int s, X192 a0, X192 ap, X192 am,
                                           long long sumi, int &bad)
{
    if (sumi & 1) atomicOr(&cx.ctr->error, LF_DEVERR_ODD);
    long long m = sumi / 2;
    CommRec *r = &cx.cr[C];
    r->m = m;
    r->W = density(s, m) * x192_round(a0);
    rec_store(r->Sp, ap, bad);
    rec_store(r->Sm, am, bad);
    cx.tflag[C] = 0;
}

// Values read together: without this the compiler moves a read behind the branches that do not
// need it, where it is a round trip of its own.  All the operands have arrived behind it.
template <class A>
__device__ __forceinline__ void arrived(A &a) { asm volatile("" : "+v"(a)); }
template <class A, class B>
__device__ __forceinline__ void arrived(A &a, B &b) { asm volatile("" : "+v"(a), "+v"(b)); }
template <class A, class B, class C>
__device__ __forceinline__ void arrived(A &a, B &b, C &c) { asm volatile("" : "+v"(a), "+v"(b), "+v"(c)); }
template <class A, class B, class C, class D>
__device__ __forceinline__ void arrived(A &a, B &b, C &c, D &d)
{
    asm volatile("" : "+v"(a), "+v"(b), "+v"(c), "+v"(d));
}
template <class A, class B, class C, class D, class E>
__device__ __forceinline__ void arrived(A &a, B &b, C &c, D &d, E &e)
{
    asm volatile("" : "+v"(a), "+v"(b), "+v"(c), "+v"(d), "+v"(e));
}

typedef int v4i __attribute__((ext_vector_type(4)));

// a node's line in four 16-byte reads; valid once all four have arrived
struct RawLine {
    v4i q[4];
};

__device__ __forceinline__ RawLine read_line(const NodeLine *p)
{
    const v4i *v = (const v4i *)p;
    return RawLine{{v[0], v[1], v[2], v[3]}};
}

__device__ __forceinline__ NodeLine as_line(const RawLine &r) { return __builtin_bit_cast(NodeLine, r); }

// position of community c among a node's cnt slots (-1 if absent); *in gets its in-count
__device__ __forceinline__ int find_slot_in(const Slot *slot, long long off, int cnt, int c, int *in)
{
    for (int t = 0; t < cnt; t += 4) {         // four independent loads per round trip
        long long w[4];
#pragma unroll
        for (int k = 0; k < 4; k++) w[k] = *(const long long *)&slot[off + (t + k < cnt ? t + k : t)];
        arrived(w[0], w[1], w[2], w[3]);
#pragma unroll
        for (int k = 0; k < 4; k++)
            if ((int)w[k] == c) {
                *in = (int)(w[k] >> 32);
                return t + k;
            }
    }
    return -1;
}

// correction of one neighbour y (in C with in-count i, degree dy) when x joins C (its
// in-count rises by one, the size to s+1) or leaves C (falls by one, size s-1)
__device__ __forceinline__ u128 visit_term(bool leave, int i, int dy, int s, int &bad)
{
    const int sn = leave ? s - 1 : s + 1;
    const double gn = g_term(leave ? i - 1 : i + 1, dy, sn);
    const double go = g_term(i, dy, sn);
    return fx128(gn, bad) - fx128(go, bad);
}

// the fields of C's record a candidate evaluation needs (S = S- for a leave, S+ for a join)
struct CandRec {
    double W;
    unsigned S[5];
    int m;                                   // below 2^30 (2|E| < 2^31)
    int s;
};

__device__ __forceinline__ void load_cand(const Ctx &cx, int C, bool leave, CandRec &r)
{
    const CommRec *p = &cx.cr[C];
    r.s = p->s;
    r.m = (int)p->m;
    r.W = p->W;
    const unsigned *S = leave ? p->Sm : p->Sp;
#pragma unroll
    for (int k = 0; k < 5; k++) r.S[k] = S[k];
}

// change of C's cc-free score when x (degree dx, k neighbours in C) joins / leaves C;
// corr = exact sum of the neighbours' corrections
__device__ __forceinline__ double cand_delta(const CandRec &r, bool leave, int k, int dx, u128 corr, int &bad)
{
    const int sn = leave ? r.s - 1 : r.s + 1;
    const u128 own = fx128(g_term(k, dx, sn), bad);
    X192 S = rec_load(r.S);
    x192_add(S, x192_sext128(leave ? corr - own : corr + own));
    return density(sn, leave ? r.m - k : r.m + k) * x192_round(S) - r.W;
}

// strictly positive changes only; larger wins; equal -> lower community id
__device__ __forceinline__ void better(double d, int c, double &bd, int &bc)
{
    if (!(d > 0.0)) return;
    if (bc < 0 || d > bd || (d == bd && c < bc)) { bd = d; bc = c; }
}

// Cross-lane reductions over a whole wave with DPP moves (every lane active): within rows of
// 16 lanes by shifts, then across the rows by broadcasts of each row's last lane.  A step
// is one VALU instruction; a shuffle through LDS costs some 60 cycles of latency each.
#define DPP_STEP(x, op, ctrl, rows) x = op(x, (unsigned)__builtin_amdgcn_update_dpp(0, (int)(x), ctrl, rows, 0xf, false))
#define DPP_INCLUSIVE(x, op)                                                               \
    do {                                                                                   \
        DPP_STEP(x, op, 0x111, 0xf);                                                       \
        DPP_STEP(x, op, 0x112, 0xf);                                                       \
        DPP_STEP(x, op, 0x114, 0xf);                                                       \
        DPP_STEP(x, op, 0x118, 0xf);                                                       \
        DPP_STEP(x, op, 0x142, 0xa);                                                       \
        DPP_STEP(x, op, 0x143, 0xc);                                                       \
    } while (0)

__device__ __forceinline__ unsigned op_add(unsigned a, unsigned b) { return a + b; }
__device__ __forceinline__ unsigned op_max(unsigned a, unsigned b) { return a > b ? a : b; }

// inclusive prefix sum over the wave's lanes; *total = the sum of all 64
__device__ __forceinline__ int wave_incl_scan(int v, int *total)
{
    unsigned x = (unsigned)v;
    DPP_INCLUSIVE(x, op_add);
    *total = __builtin_amdgcn_readlane((int)x, WAVE - 1);
    return (int)x;
}

// the sum of the lanes' values, the same on every lane
__device__ __forceinline__ unsigned wave_sum_u32(unsigned x)
{
    DPP_INCLUSIVE(x, op_add);
    return (unsigned)__builtin_amdgcn_readlane((int)x, WAVE - 1);
}

// the sum over the lane's row of 16 lanes, valid on the row's last lane
__device__ __forceinline__ unsigned row_sum_u32(unsigned x)
{
    DPP_STEP(x, op_add, 0x111, 0xf);
    DPP_STEP(x, op_add, 0x112, 0xf);
    DPP_STEP(x, op_add, 0x114, 0xf);
    DPP_STEP(x, op_add, 0x118, 0xf);
    return x;
}

// the largest of the row's values (unsigned), valid on its last lane
__device__ __forceinline__ unsigned row_max_u32(unsigned x)
{
    DPP_STEP(x, op_max, 0x111, 0xf);
    DPP_STEP(x, op_max, 0x112, 0xf);
    DPP_STEP(x, op_max, 0x114, 0xf);
    DPP_STEP(x, op_max, 0x118, 0xf);
    return x;
}

// four entries of an adjacency or out-list from p on, in one read (the arrays are padded by
// READ_PAD entries)
#define READ_PAD 4
__device__ __forceinline__ v4i read_entries(const int *p)
{
    v4i r;
    __builtin_memcpy(&r, p, sizeof r);
    return r;
}

// the sum over the lane's 8 lanes of a row, valid on the last of them
__device__ __forceinline__ unsigned oct_sum_u32(unsigned x)
{
    DPP_STEP(x, op_add, 0x111, 0xf);
    DPP_STEP(x, op_add, 0x112, 0xf);
    DPP_STEP(x, op_add, 0x114, 0xf);
    return x;
}

// Passes over all nodes' neighbours: most nodes have far fewer than 64, so a row of 16 lanes
// takes a node (four per wave) and only those of more than ROW_DEG neighbours get the whole
// wave, one after the other.  body(x, sub, width) runs with the node's 16 or 64 lanes (the other
// rows' nodes beside it); all lanes of the wave call it, x < 0 where there is no node.
#define ROW_DEG 256
template <class Degree, class Body>
__device__ __forceinline__ void for_rows(long long n, Degree degree, Body body)
{
    const int lane = threadIdx.x & (WAVE - 1), sub = lane & 15;
    const long long x = (blockIdx.x * (long long)blockDim.x + threadIdx.x) / 16;
    if (x - lane / 16 >= n) return;          // uniform over the wave
    const bool in = x < n, longer = in && degree(x) > ROW_DEG;
    body(in && !longer ? x : -1, sub, 16);
    for (unsigned long long rest = __ballot(longer && sub == 0); rest; rest &= rest - 1) {
        WAVE_SYNC();
        body(x - lane / 16 + (__ffsll((long long)rest) - 1) / 16, lane, WAVE);
    }
}

// the largest of the lanes' values (unsigned), the same on every lane
__device__ __forceinline__ unsigned wave_max_u32(unsigned x)
{
    DPP_INCLUSIVE(x, op_max);
    return (unsigned)__builtin_amdgcn_readlane((int)x, WAVE - 1);
}

// Exact sum of lanes' 128-bit values: each is cut into six 24-bit limbs, whose sums over 64
// lanes fit 32-bit words, so a limb is one DPP reduction (no carries, no LDS).
template <class Sum>
__device__ __forceinline__ X192 sum_limbs(u128 v, Sum sum)
{
    const unsigned w0 = (unsigned)v, w1 = (unsigned)(v >> 32), w2 = (unsigned)(v >> 64), w3 = (unsigned)(v >> 96);
    const u64 t0 = sum(w0 & 0xffffffu);
    const u64 t1 = sum((w0 >> 24) | ((w1 & 0xffffu) << 8));
    const u64 t2 = sum((w1 >> 16) | ((w2 & 0xffu) << 16));
    const u64 t3 = sum(w2 >> 8);
    const u64 t4 = sum(w3 & 0xffffffu);
    const u64 t5 = sum(w3 >> 24);
    const u64 lo = t0 + (t1 << 24), mid = t2 + (t3 << 24), hi = t4 + (t5 << 24);   // at 2^0, 2^48, 2^96
    X192 r = {lo, 0, 0};
    x192_add(r, X192{mid << 48, mid >> 16, 0});
    x192_add(r, X192{0, hi << 32, hi >> 32});
    return r;
}
__device__ __forceinline__ X192 wave_sum_u128(u128 v)     // the wave's, on every lane
{
    return sum_limbs(v, [](unsigned x) { return wave_sum_u32(x); });
}
__device__ __forceinline__ X192 row_sum_u128(u128 v)      // the row's, on its last lane
{
    return sum_limbs(v, [](unsigned x) { return row_sum_u32(x); });
}

// best (change, community) of the wave's lanes, on every lane: the largest positive change
// (positive doubles order like their bits), the lowest id among equals.  Most nodes have no
// improving move, so the common case is one ballot.
__device__ __forceinline__ void wave_best(double &bd, int &bc)
{
    if (!__ballot(bc >= 0)) return;
    const unsigned long long bits = bc >= 0 ? (unsigned long long)__double_as_longlong(bd) : 0ull;
    const unsigned hi = wave_max_u32((unsigned)(bits >> 32));
    const unsigned lo = wave_max_u32((unsigned)(bits >> 32) == hi ? (unsigned)bits : 0u);
    const unsigned long long top = ((unsigned long long)hi << 32) | lo;
    // ids are >= 0: the lowest id is the largest complement
    bc = (int)(0x7fffffffu - wave_max_u32(bits == top ? 0x7fffffffu - (unsigned)bc : 0u));
    bd = __longlong_as_double((long long)top);
}

// the g-terms of one member of C with in-count i and degree d at sizes s, s+1, s-1.  A term is
// at most 2: i <= s - 1 and i <= d, so at size s - 1 at most i / (i - 1), which is 2 where i = d = 2 and
// s = 3.  An unsigned 128-bit accumulator (below 2^8) holds fewer than TERMS_U128 of them.
#define TERMS_U128 128
__device__ __forceinline__ void acc_add(X192 &a, u128 t) { x192_add(a, x192_sext128(t)); }
__device__ __forceinline__ void acc_add(u128 &a, u128 t) { a += t; }

template <class Acc>
__device__ __forceinline__ void member_add(int i, int d, int s, Acc &a0, Acc &ap, Acc &am, long long &sumi, int &bad)
{
    sumi += i;
    acc_add(a0, fx128(g_term(i, d, s), bad));
    __builtin_amdgcn_sched_barrier(0);       // one division at a time: fewer registers, more waves
    acc_add(ap, fx128(g_term(i, d, s + 1), bad));
    __builtin_amdgcn_sched_barrier(0);
    acc_add(am, fx128(g_term(i, d, s - 1), bad));
}

// exact g-sums of one member y of C (at sizes s, s+1, s-1) if y is still in C
template <class Acc>
__device__ __forceinline__ void member_terms(const Ctx &cx, int y, int C, int s, Acc &a0, Acc &ap,
                                             Acc &am, long long &sumi, int &bad)
{
    NodeHdr hy = cx.nh[y];
    int in = 0;
    int t = find_slot_in(cx.slot, hy.off, hy.cnt, C, &in);
    if (t < 0) return;                       // left C earlier in this iteration
    member_add(in, hy.deg, s, a0, ap, am, sumi, bad);
}

// ---- membership lines (the queue kernels' view of the memberships) --------------------
// position of community c among the memberships of the node with line l (-1 if absent)
// and its in-count: inline memberships come from the line itself
__device__ __forceinline__ int line_find(const Ctx &cx, const NodeLine &l, int c, int *in)
{
    if (l.off < 0) {
        int a = -1, iv = 0;
#pragma unroll
        for (int t = 0; t < LINE_SLOTS; t++)
            if (t < l.cnt && l.s[t].comm == c) {
                a = t;
                iv = l.s[t].in;
            }
        *in = iv;
        return a;
    }
    return find_slot_in(cx.slot, l.off, l.cnt, c, in);
}

// member_terms on the membership lines
__device__ __forceinline__ void member_terms_of(const Ctx &cx, const NodeLine &ly, int C, int s, u128 &a0, u128 &ap,
                                                u128 &am, long long &sumi, int &bad)
{
    int in = 0;
    if (line_find(cx, ly, C, &in) < 0) return;   // left C earlier in this iteration
    member_add(in, ly.deg, s, a0, ap, am, sumi, bad);
}

__device__ __forceinline__ void member_terms_line(const Ctx &cx, int y, int C, int s, u128 &a0, u128 &ap,
                                                  u128 &am, long long &sumi, int &bad)
{
    RawLine r = read_line(cx.ln + y);
    arrived(r.q[0], r.q[1], r.q[2], r.q[3]);
    member_terms_of(cx, as_line(r), C, s, a0, ap, am, sumi, bad);
}

__device__ __forceinline__ unsigned hash_tab(int c) { return (unsigned)c * 0x9E3779B1u; }

