// Steps a2 + a3: triangulation of the separated cycles, edge<->triangle incidence, and the
// message-passing iterations (paper Sec. 3.2.1, eq. 5 and 6; Sec. 3.2.3, algorithm
// "Parallel-Message-Passing").
//
// Triangulation (the paper only says that longer cycles are triangulated): fan from v0 --
// triangles {v0,v_m,v_{m+1}}, chords (v0,v_m); unseen chords join the edge list with cost 0 and
// the list stays canonical.  Triangles are the sorted set of distinct node triples u<v<w, keyed
// as (edge id of (u,v), in-row distance to edge (u,w)); slots of a triangle are its edges
// (u,v),(u,w),(v,w).
//
// Message passing keeps c_e (reduced edge costs, eq. 6a) and c_t (triangle costs, eq. 6b).
// One iteration = edges->triangles (every edge in N_e triangles hands each of them c_e/N_e and
// drops to 0) + triangles->edges (six min-marginal updates with weights 1/3,1/2,1,1/2,1,1).
// It runs as two kernels without atomics:
//   triangle kernel: gathers the three shares, does the six updates in registers, writes c_t and
//                    the three outgoing messages;
//   edge kernel:     one thread per edge that lies in a triangle; adds its messages in ascending
//                    triangle order (slot list built once per round by a stable sort) and stores
//                    the next share c_e/N_e.  Work is proportional to the triangles, not the edges.
// Inside the iterations an edge is known by its number among the edges that lie in a triangle (the
// "active" edges): the shares form a dense array, and the edge id is looked at when the first shares
// come in and when the final costs go out.
#include <hip/hip_ext.h>

#include "prim.h"
#include "steps.h"

namespace rama {

namespace {

// ---------------------------------------------------------------------------------------------
// cycle access: one flat index space over the fan pieces of all cycles
// ---------------------------------------------------------------------------------------------
// list k < kCycleLists: the (k+3)-cycles; list kCycleLists: triangles kept from earlier dual rounds
// on this graph (sorted node triples), which re-enter as 3-cycles
constexpr int kCycleSets = kCycleLists + 1;
__host__ __device__ constexpr int set_len(int k) { return k < kCycleLists ? k + 3 : 3; }
struct CycleSet {
    const int32_t *c[kCycleSets];
    uint32_t cyc_end[kCycleSets];    // running totals over the lists (all below 2^31): cycles,
    uint32_t fan_end[kCycleSets];    // fan triangles (L-2 per cycle)
    uint32_t chord_end[kCycleSets];  // and chords (L-3 per cycle)
};

// The list an index falls into is found by a chain of compile-time cases: every access to the
// set's arrays then has a constant index and the set stays in scalar registers (a loop with an early
// exit made the compiler copy it to private memory, 128 bytes written per thread).
template <int K>
__device__ __forceinline__ void chord_pick(const CycleSet &s, uint32_t q, int32_t &a, int32_t &b)
{
    // q-th chord: an L-cycle gives the L-3 chords (v0,v_m), m = 2..L-2; list K has K chords per cycle
    if constexpr (K >= kCycleLists) {
        a = b = 0;
    } else {
        if (q < s.chord_end[K]) {
            const uint32_t r = q - s.chord_end[K - 1], cyc = r / (uint32_t)K;
            const int32_t *v = s.c[K] + (uint32_t)(K + 3) * cyc;
            a = v[0]; b = v[2 + (r - cyc * (uint32_t)K)];
        } else {
            chord_pick<K + 1>(s, q, a, b);
        }
    }
}
__device__ __forceinline__ void chord_of(const CycleSet &s, uint32_t q, int32_t &a, int32_t &b)
{
    chord_pick<1>(s, q, a, b);   // 3-cycles and kept triangles have no chords
}

template <int K>
__device__ __forceinline__ void fan_pick(const CycleSet &s, uint32_t q, int32_t &a, int32_t &b, int32_t &c)
{
    // q-th fan triangle (unsorted nodes): an L-cycle gives {v0,v_m,v_{m+1}}, m = 1..L-2
    if constexpr (K >= kCycleSets) {
        a = b = c = 0;
    } else {
        if (q < s.fan_end[K]) {
            constexpr uint32_t per = (uint32_t)(set_len(K) - 2);
            uint32_t r = q;
            if constexpr (K > 0) r -= s.fan_end[K - 1];
            const uint32_t cyc = r / per;
            const int32_t *v = s.c[K] + (uint32_t)set_len(K) * cyc;   // list sizes stay below 2^31 entries
            const uint32_t mm = 1u + (r - cyc * per);
            a = v[0]; b = v[mm]; c = v[mm + 1];
        } else {
            fan_pick<K + 1>(s, q, a, b, c);
        }
    }
}
__device__ __forceinline__ void fan_triangle(const CycleSet &s, uint32_t q, int32_t &a, int32_t &b, int32_t &c)
{
    fan_pick<0>(s, q, a, b, c);
}

template <int K>
__device__ __forceinline__ void cycle_pick(const CycleSet &s, uint32_t q, const int32_t *&v, int &L)
{
    if constexpr (K >= kCycleSets) {
        v = nullptr; L = 0;
    } else {
        if (q < s.cyc_end[K]) {
            uint32_t r = q;
            if constexpr (K > 0) r -= s.cyc_end[K - 1];
            v = s.c[K] + (size_t)set_len(K) * r;
            L = set_len(K);
        } else {
            cycle_pick<K + 1>(s, q, v, L);
        }
    }
}

__device__ __forceinline__ void sort3(int32_t &a, int32_t &b, int32_t &c)
{
    int32_t t;
    if (a > b) { t = a; a = b; b = t; }
    if (b > c) { t = b; b = c; c = t; }
    if (a > b) { t = a; a = b; b = t; }
}

// every cycle: nodes in range and distinct, every cycle edge present in the graph
__global__ __launch_bounds__(kBlock) void k_validate_cycles(CycleSet s, int32_t n, const int32_t *rowptr,
                                                            const int32_t *j, int32_t *flag)
{
    size_t q = (size_t)blockIdx.x * kBlock + threadIdx.x;
    if (q >= s.cyc_end[kCycleSets - 1]) return;
    const int32_t *v;
    int L;
    cycle_pick<0>(s, (uint32_t)q, v, L);
    int32_t x[kMaxCycleLen];
    bool bad = false;
    for (int a = 0; a < L; ++a) {
        x[a] = v[a];
        if (x[a] < 0 || x[a] >= n) bad = true;
        for (int b = 0; b < a; ++b) if (x[b] == x[a]) bad = true;
    }
    if (!bad)
        for (int a = 0; a < L; ++a) {
            int32_t p = x[a], r = x[(a + 1) % L];
            if (find_edge_in_row(rowptr, j, min(p, r), max(p, r)) < 0) bad = true;
        }
    if (bad) *flag = 1;
}

__global__ __launch_bounds__(kBlock) void k_chord_keys(CycleSet s, size_t nch, int nbits, uint64_t *key)
{
    size_t q = (size_t)blockIdx.x * kBlock + threadIdx.x;
    if (q >= nch) return;
    int32_t a, b;
    chord_of(s, (uint32_t)q, a, b);
    key[q] = ((uint64_t)(uint32_t)min(a, b) << nbits) | (uint32_t)max(a, b);
}

// Cycles of five and more nodes are listed walk by walk, and walks from one repulsive edge share most of their nodes: on a
// neighbour graph a chord comes up twelve times on average and a fan triangle six times.  A workgroup enters the 2048
// candidates of its tile -- the walks of a few dozen repulsive edges -- into a hash set in LDS and hands on what
// it sees for the first time, in any order (the sort behind puts it in order and drops what tiles have in common).
// The set holds the candidates' numbers within the tile; equality is decided on the nodes themselves.
// Bounded by LDS latency.  6-NN graph of 10^6 points (2.4e7 chord and 3.7e7 triangle candidates): solve 13.76 -> 12.53 ms
// against dropping only repeats of the cycle before (chords) and none (triangles); the chords' sort gets 4 instead of 17
// million keys.
constexpr int kSetItems = 8;
constexpr int kSetTile = kBlock * kSetItems, kSetSlots = 2 * kSetTile;
template <int NODES>
struct TileSet {
    int32_t node[NODES][kSetTile];
    uint32_t slot[kSetSlots];       // candidate, or kSetTile: empty; later the list of the new ones
    uint32_t base;
    __device__ __forceinline__ void clear()
    {
        for (int k = threadIdx.x; k < kSetSlots; k += kBlock) slot[k] = (uint32_t)kSetTile;
    }
    // true iff candidate `me` (whose nodes are in place, as are all others') is the one that stands for its equals
    __device__ __forceinline__ bool enter(uint32_t me)
    {
        constexpr uint32_t mix[3] = {0x9E3779B1u, 0x85EBCA6Bu, 0xC2B2AE35u};
        uint32_t h = 0;
#pragma unroll
        for (int k = 0; k < NODES; ++k) h = (h ^ (uint32_t)node[k][me]) * mix[k];
        h >>= 32 - __builtin_ctz(kSetSlots);
        for (;;) {      // half of the slots stay empty: the walk ends
            const uint32_t old = atomicCAS(&slot[h], (uint32_t)kSetTile, me);
            if (old == (uint32_t)kSetTile) return true;
            bool same = true;
#pragma unroll
            for (int k = 0; k < NODES; ++k) same = same && node[k][old] == node[k][me];
            if (same) return false;
            h = (h + 1) & (kSetSlots - 1);
        }
    }
    // packs the candidates marked in `fresh` (bit q: candidate q * kBlock + tid) into the front of slot[]; returns their
    // number, and in base the place `counter` gives them
    __device__ __forceinline__ uint32_t pack(uint32_t fresh, uint32_t *counter)
    {
        uint32_t total;
        uint32_t at = block_inclusive_scan((uint32_t)__popc(fresh), &total) - (uint32_t)__popc(fresh);      // all have entered
        for (; fresh; fresh &= fresh - 1) slot[at++] = (uint32_t)((__ffs((int)fresh) - 1) * kBlock) + threadIdx.x;
        if (threadIdx.x == 0) base = total ? atomicAdd(counter, total) : 0u;
        __syncthreads();
        return total;
    }
};

__global__ __launch_bounds__(kBlock) void k_new_chords(CycleSet s, size_t nch, int nbits, uint64_t *key, uint32_t *counter)
{
    __shared__ TileSet<2> set;
    const size_t tile = (size_t)blockIdx.x * kSetTile;
    set.clear();
#pragma unroll
    for (int q = 0; q < kSetItems; ++q) {
        const uint32_t x = (uint32_t)q * kBlock + threadIdx.x;
        if (tile + x < nch) {
            int32_t a, b;
            chord_of(s, (uint32_t)(tile + x), a, b);
            set.node[0][x] = min(a, b); set.node[1][x] = max(a, b);
        }
    }
    __syncthreads();
    uint32_t fresh = 0;
#pragma unroll
    for (int q = 0; q < kSetItems; ++q) {
        const uint32_t x = (uint32_t)q * kBlock + threadIdx.x;
        if (tile + x < nch && set.enter(x)) fresh |= 1u << q;
    }
    const uint32_t total = set.pack(fresh, counter);
    for (uint32_t k = threadIdx.x; k < total; k += kBlock) {
        const uint32_t x = set.slot[k];
        key[set.base + k] = ((uint64_t)(uint32_t)set.node[0][x] << nbits) | (uint32_t)set.node[1][x];
    }
}

// For every sorted chord key: where it would be inserted in the canonical edge list, or -1 if
// it repeats the previous key or is an edge already.  One binary search per chord, done once.
__global__ __launch_bounds__(kBlock) void k_chord_lookup(size_t nch, const uint64_t *key, const int32_t *rowptr,
                                                         const int32_t *j, int nbits, int32_t *where)
{
    size_t q = (size_t)blockIdx.x * kBlock + threadIdx.x;
    if (q >= nch) return;
    uint64_t k = key[q];
    if (q > 0 && key[q - 1] == k) { where[q] = -1; return; }
    int32_t u = (int32_t)(k >> nbits), v = (int32_t)(k & ((1ull << nbits) - 1ull));
    int32_t lo = rowptr[u], hi = rowptr[u + 1];
    const int32_t end = hi;
    while (lo < hi) {
        int32_t mid = lo + ((hi - lo) >> 1);
        if (j[mid] < v) lo = mid + 1; else hi = mid;
    }
    where[q] = (lo < end && j[lo] == v) ? -1 : lo;
}
struct NewChordFlag {
    static constexpr int bytes = 4;   // bytes read per item
    static constexpr const char *tag = "NewChordFlag";
    const int32_t *where;
    __device__ __forceinline__ uint32_t operator()(size_t q) const { return where[q] >= 0 ? 1u : 0u; }
};

// compacts the new chords together with the number of graph edges that precede each
__global__ __launch_bounds__(kBlock) void k_emit_chords(size_t nch, const uint64_t *key, const int32_t *where,
                                                        const uint32_t *pos, int nbits, int32_t *ci, int32_t *cj,
                                                        int32_t *before)
{
    size_t q = (size_t)blockIdx.x * kBlock + threadIdx.x;
    if (q >= nch) return;
    int32_t w = where[q];
    if (w < 0) return;
    uint64_t k = key[q];
    uint32_t p = pos[q];
    ci[p] = (int32_t)(k >> nbits);
    cj[p] = (int32_t)(k & ((1ull << nbits) - 1ull));
    before[p] = w;
}

// merge of the canonical edge list with the (sorted, disjoint) new chords.
// ins[v] = number of chords with before < v, so ins[e + 1] chords come before graph edge e (row bounds of
// `before`).  A workgroup writes its 256 edges and the chords that sit between them (and in front of its first
// edge; the last workgroup also those behind the last edge): one contiguous stretch of the output, written
// at one time.  With chord k handled by thread k instead, every output cache line was written twice, at two
// far-apart moments (3.0 GB written for a 1.56 GB list at the 320^3 grid).
__global__ __launch_bounds__(kBlock) void k_merge_edges(size_t m, const int32_t *i, const int32_t *j, const float *c,
                                                        const int32_t *ins, const int32_t *ci, const int32_t *cj,
                                                        const int32_t *before, int32_t *io, int32_t *jo, float *co)
{
    const size_t e0 = (size_t)blockIdx.x * kBlock, e = e0 + threadIdx.x;
    const size_t e1 = e0 + kBlock < m ? e0 + kBlock : m;
    if (e < m) {
        size_t d = e + (size_t)ins[e + 1];
        io[d] = i[e]; jo[d] = j[e]; co[d] = c[e];
    }
    const size_t k0 = (size_t)ins[e0], k1 = (size_t)ins[e1 == m ? m + 1 : e1];
    for (size_t k = k0 + threadIdx.x; k < k1; k += kBlock) {
        size_t d = (size_t)before[k] + k;
        io[d] = ci[k]; jo[d] = cj[k]; co[d] = 0.0f;
    }
}

// longest row of the upper CSR (bounds the in-row distance between two edges of one row)
// (a workgroup takes 4096 rows: one atomic per 4096 rows on the result word)
constexpr int kMaxRowItems = 16;
__global__ __launch_bounds__(kBlock) void k_max_row(int32_t n, const int32_t *rowptr, uint32_t *out)
{
    const size_t base = (size_t)blockIdx.x * (kBlock * kMaxRowItems) + threadIdx.x;
    uint32_t longest = 0;
#pragma unroll
    for (int q = 0; q < kMaxRowItems; ++q) {
        const size_t v = base + (size_t)q * kBlock;
        if (v < (size_t)n) {
            const uint32_t len = (uint32_t)(rowptr[v + 1] - rowptr[v]);
            longest = len > longest ? len : longest;
        }
    }
    block_max_into(longest, out);
}

// A triangle u<v<w is keyed by (position e0 of edge (u,v), distance e1-e0 to edge (u,w) in the
// same row): ascending keys = ascending (u,v,w), and the key needs only
// bits(|E'|) + bits(longest row) bits -- four 8-bit passes of 32-bit keys on grid-like graphs.
template <typename KT>
__global__ __launch_bounds__(kBlock) void k_triangle_keys(CycleSet s, size_t nt, const int32_t *rowptr,
                                                          const int32_t *j, int dbits, KT *key, int32_t *flag)
{
    size_t q = (size_t)blockIdx.x * kBlock + threadIdx.x;
    if (q >= nt) return;
    int32_t a, b, c;
    fan_triangle(s, (uint32_t)q, a, b, c);
    sort3(a, b, c);
    int32_t e0, e1;
    find_two_in_row(rowptr, j, a, b, c, e0, e1);
    if (e0 < 0 || e1 < 0) { *flag = 1; e0 = 0; e1 = 0; }
    key[q] = ((KT)(uint32_t)e0 << dbits) | (KT)(uint32_t)(e1 - e0);
}

// the same keys, without the triangles that repeat one of their tile (see TileSet); *counter: their number
template <typename KT>
__global__ __launch_bounds__(kBlock) void k_new_triangle_keys(CycleSet s, size_t nt, const int32_t *rowptr, const int32_t *j, int dbits,
                                                              KT *key, int32_t *flag, uint32_t *counter)
{
    __shared__ TileSet<3> set;
    const size_t tile = (size_t)blockIdx.x * kSetTile;
    set.clear();
#pragma unroll
    for (int q = 0; q < kSetItems; ++q) {
        const uint32_t x = (uint32_t)q * kBlock + threadIdx.x;
        if (tile + x < nt) {
            int32_t a, b, c;
            fan_triangle(s, (uint32_t)(tile + x), a, b, c);
            sort3(a, b, c);
            set.node[0][x] = a; set.node[1][x] = b; set.node[2][x] = c;
        }
    }
    __syncthreads();
    uint32_t fresh = 0;
#pragma unroll
    for (int q = 0; q < kSetItems; ++q) {
        const uint32_t x = (uint32_t)q * kBlock + threadIdx.x;
        if (tile + x < nt && set.enter(x)) fresh |= 1u << q;
    }
    const uint32_t total = set.pack(fresh, counter);
    for (uint32_t k = threadIdx.x; k < total; k += kBlock) {
        const uint32_t x = set.slot[k];
        int32_t e0, e1;
        find_two_in_row(rowptr, j, set.node[0][x], set.node[1][x], set.node[2][x], e0, e1);
        if (e0 < 0 || e1 < 0) { *flag = 1; e0 = 0; e1 = 0; }
        key[set.base + k] = ((KT)(uint32_t)e0 << dbits) | (KT)(uint32_t)(e1 - e0);
    }
}

template <typename KT>
struct HeadFlagT {
    static constexpr int bytes = (int)sizeof(KT);   // bytes read per item
    static constexpr const char *tag = sizeof(KT) == 8 ? "HeadFlag64" : "HeadFlag32";
    const KT *key;
    __device__ __forceinline__ uint32_t operator()(size_t e) const { return ((e == 0) | (key[e] != key[e ? e - 1 : 0])) ? 1u : 0u; }
};

// Consumer of the scan over the heads of the sorted triangle keys.  The head of run t is triangle t:
// it writes its three edge ids and the (edge, slot) pairs for the incidence sort.  Triangles kept from
// an earlier dual round take their costs along: `origin` (optional) is the fan index each sorted key
// came from, the kept triangles occupy the fan indices [kept_begin, kept_end) in their old order, and
// the run a key lies in is the triangle's new index.
template <typename KT>
struct TrianglesEmit {
    static constexpr const char *tag = sizeof(KT) == 8 ? "Triangles64" : "Triangles";
    static constexpr bool long_chain = true;   // key -> nodes -> row -> entry: four loads that wait for each other
    const KT *key;
    const int32_t *rowptr, *j;
    int dbits;
    uint32_t *skey;           // per slot 3t+k the edge id: the keys of the incidence sort, whose values are the slots themselves
    const int32_t *flag_in;   // raised by the kernel that built the keys
    int32_t *flag;            // where the host will look: flag_in is carried over
    const uint32_t *origin;
    uint32_t kept_begin, kept_end;
    const float *ct_old;
    float *ct;
    bool zero_new;            // new triangles get their zero costs stored (not needed when the first iteration knows)
    struct Item { int32_t e0, e1, begin, end, node; uint32_t from; };     // edges (u,v), (u,w); row of v; w; where the key came from
    __device__ __forceinline__ Item load(size_t q) const
    {
        const KT k = key[q];
        const int32_t e0 = (int32_t)(k >> dbits), e1 = e0 + (int32_t)(k & (((KT)1 << dbits) - 1)), v = j[e0];
        return {e0, e1, rowptr[v], rowptr[v + 1], j[e1], origin ? origin[q] : 0u};
    }
    __device__ __forceinline__ void operator()(size_t q, uint32_t head, uint32_t runs_before, const Item &x) const
    {
        const size_t t = (size_t)runs_before + head - 1;   // the run q lies in (the first key is a head)
        if (q == 0 && *flag_in) *flag = 1;
        if (origin) {
            const uint32_t o = x.from;
            if (o >= kept_begin && o < kept_end) {
                const size_t old = o - kept_begin;
                ct[3 * t] = ct_old[3 * old]; ct[3 * t + 1] = ct_old[3 * old + 1]; ct[3 * t + 2] = ct_old[3 * old + 2];
            }
        }
        if (!head) return;
        if (!origin && zero_new) { ct[3 * t] = 0.0f; ct[3 * t + 1] = 0.0f; ct[3 * t + 2] = 0.0f; }   // a new triangle starts at zero
        int32_t e2 = find_edge_between(j, x.begin, x.end, x.node);
        if (e2 < 0) { *flag = 1; e2 = 0; }
        skey[3 * t + 0] = (uint32_t)x.e0; skey[3 * t + 1] = (uint32_t)x.e1; skey[3 * t + 2] = (uint32_t)e2;
    }
};

// node triple (u,v,w) of every triangle from its edges (u,v) and (u,w); tri_act holds their numbers among the active edges
__global__ __launch_bounds__(kBlock) void k_triangle_nodes(size_t T, const uint32_t *tri_act, const uint32_t *act_edge,
                                                           const int32_t *i, const int32_t *j, int32_t *nodes)
{
    size_t t = (size_t)blockIdx.x * kBlock + threadIdx.x;
    if (t >= T) return;
    const uint32_t e0 = act_edge[tri_act[3 * t]], e1 = act_edge[tri_act[3 * t + 1]];
    nodes[3 * t] = i[e0]; nodes[3 * t + 1] = j[e0]; nodes[3 * t + 2] = j[e1];
}

// ---------------------------------------------------------------------------------------------
// message passing
// ---------------------------------------------------------------------------------------------
// edges that lie in at least one triangle ("active"): runs of equal edge id in the sorted slot list
struct HeadFlag32 {
    static constexpr int bytes = 4;   // bytes read per item
    static constexpr const char *tag = "HeadFlag32";
    const uint32_t *key;
    __device__ __forceinline__ uint32_t operator()(size_t p) const { return ((p == 0) | (key[p] != key[p ? p - 1 : 0])) ? 1u : 0u; }
};

// consumer of the scan over HeadFlag32: run number a of the sorted slot list starts at p and belongs
// to edge skey[p]; the entry behind the last run closes it.  Every slot learns the number of its run:
// the message passing addresses edges by their number among the active edges, so that the shares it
// gathers lie densely (on the 320^3 grid one edge in five is active; indexed by edge id the share
// array cost the triangle update 25 bytes of fetches per triangle beyond the 12 it uses).
struct ActiveEdgesEmit {
    static constexpr const char *tag = "ActiveEdges";
    const uint32_t *skey, *sval;
    uint32_t ns, na;
    uint32_t *act_edge, *act_start, *tri_act;
    struct Item { uint32_t edge, slot; };
    __device__ __forceinline__ Item load(size_t p) const { return {skey[p], sval[p]}; }
    __device__ __forceinline__ void operator()(size_t p, uint32_t head, uint32_t before, const Item &x) const
    {
        if (p == 0) act_start[na] = ns;
        const uint32_t a = before + head - 1u;   // the first slot is a head
        tri_act[x.slot] = a;
        if (!head) return;
        act_edge[a] = x.edge;
        act_start[a] = (uint32_t)p;
    }
};

__global__ __launch_bounds__(kBlock) void k_edge_init(size_t na, const uint32_t *act_edge, const uint32_t *act_start,
                                                      const float *ce, float *share)
{
    size_t a = (size_t)blockIdx.x * kBlock + threadIdx.x;
    if (a >= na) return;
    share[a] = ce[act_edge[a]] / (float)(act_start[a + 1] - act_start[a]);
}

// FIRST: the triangles are new and this is their first iteration: their costs are zero and have not been stored
// (the sum with zero stays, so that the result is the same bit for bit, signs of zeros included).
template <bool FIRST>
__global__ __launch_bounds__(kBlock) void k_triangle_update(size_t T, const uint32_t *tri_act, const float *share,
                                                            float *ct, float *msg)
{
    size_t t = (size_t)xcd_block() * kBlock + threadIdx.x;
    if (t >= T) return;
    const uint32_t e0 = tri_act[3 * t], e1 = tri_act[3 * t + 1], e2 = tri_act[3 * t + 2];
    // edges -> triangles
    float a = (FIRST ? 0.0f : ct[3 * t]) + share[e0];
    float b = (FIRST ? 0.0f : ct[3 * t + 1]) + share[e1];
    float c = (FIRST ? 0.0f : ct[3 * t + 2]) + share[e2];
    // triangles -> edges
    float oa, ob, oc;
    triangle_to_edges(a, b, c, oa, ob, oc);
    ct[3 * t] = a; ct[3 * t + 1] = b; ct[3 * t + 2] = c;
    msg[3 * t] = oa; msg[3 * t + 1] = ob; msg[3 * t + 2] = oc;
}

// Triangles -> edges.  An edge in no triangle is never touched and keeps its cost.  Between iterations
// only the share travels on (the next triangle update reads nothing else), so c_e itself is stored
// only when somebody reads it: after the last iteration, or for the bound.
// A workgroup's 1024 consecutive active edges own one contiguous piece of the slot list.  Its threads
// fetch the slots and messages of that piece side by side into LDS -- coalesced slot reads, and
// neighbouring lanes gather the messages of neighbouring slots, which fall into far fewer cache lines
// per load instruction than one-thread-per-edge loops do -- and then every thread adds up its own
// runs from LDS, in slot order (ordered sum: bit-reproducible).  Against the per-edge loop this took
// the kernel from 14.7 to 11.5 ms per solve at the 320^3 grid.
// Few active edges do not fill the chip with 1024 per workgroup, so up to 2^21 of them come 256 to a workgroup: 8.2 -> 3.7 us
// a launch in the solve of a 128^2 long-range grid, two dual rounds on a 180x181 one 2.99 -> 2.87 ms.  The line at 2^18, 2^20
// or 2^22 measures the same there and on the larger graphs; 256 for every length costs the 320^3 grid 94.4 -> 96.2 ms.
constexpr int kEdgesPerThread = 4;
constexpr size_t kFewEdges = size_t(1) << 21;
constexpr int kSlotsPerThread = 8;
constexpr int kEdgeChunk = kSlotsPerThread * kBlock;
template <bool STORE_CE, int PER>
__global__ __launch_bounds__(kBlock) void k_edge_update(size_t na, const uint32_t *act_edge, const uint32_t *act_start,
                                                               const uint32_t *slot, const float *msg, float *ce, float *share)
{
    __shared__ float sm[kEdgeChunk];
    const size_t a0 = (size_t)xcd_block() * (kBlock * PER);
    if (a0 >= na) return;      // the whole workgroup
    const size_t alast = a0 + kBlock * PER < na ? a0 + kBlock * PER : na;
    const uint32_t P0 = act_start[a0], P1 = act_start[alast];
    uint32_t p0[PER], p1[PER];
    float acc[PER];
#pragma unroll
    for (int j = 0; j < PER; ++j) {
        const size_t a = a0 + (size_t)j * kBlock + threadIdx.x;
        p0[j] = 0; p1[j] = 0; acc[j] = 0.0f;
        if (a < na) { p0[j] = act_start[a]; p1[j] = act_start[a + 1]; }
    }
    for (uint32_t cb = P0; cb < P1; cb += kEdgeChunk) {
        const uint32_t cend = cb + kEdgeChunk < P1 ? cb + kEdgeChunk : P1;
        uint32_t q[kSlotsPerThread];
#pragma unroll
        for (int k = 0; k < kSlotsPerThread; ++k) {
            const uint32_t p = cb + (uint32_t)k * kBlock + threadIdx.x;
            q[k] = p < cend ? slot[p] : 0xffffffffu;
        }
#pragma unroll
        for (int k = 0; k < kSlotsPerThread; ++k)
            if (q[k] != 0xffffffffu) sm[k * kBlock + threadIdx.x] = msg[q[k]];
        __syncthreads();
#pragma unroll
        for (int j = 0; j < PER; ++j) {
            const uint32_t lo = p0[j] > cb ? p0[j] : cb, hi = p1[j] < cend ? p1[j] : cend;
            for (uint32_t p = lo; p < hi; ++p) acc[j] = acc[j] + sm[p - cb];
        }
        __syncthreads();
    }
#pragma unroll
    for (int j = 0; j < PER; ++j) {
        const size_t a = a0 + (size_t)j * kBlock + threadIdx.x;
        if (a < na) {
            if (STORE_CE) ce[act_edge[a]] = acc[j];
            share[a] = acc[j] / (float)(p1[j] - p0[j]);
        }
    }
}

struct EdgeLB {
    static constexpr int bytes = 4;   // bytes read per item
    static constexpr const char *tag = "EdgeLB";
    const float *ce;
    __device__ __forceinline__ double operator()(size_t e) const { float w = ce[e]; return w < 0.0f ? (double)w : 0.0; }
};
struct TriLB {
    static constexpr int bytes = 12;   // bytes read per item
    static constexpr const char *tag = "TriLB";
    const float *ct;
    __device__ __forceinline__ double operator()(size_t t) const
    {
        TriCosts l = labeling_costs(ct[3 * t], ct[3 * t + 1], ct[3 * t + 2]);
        return (double)fminf(fminf(fminf(0.0f, l.l110), fminf(l.l101, l.l011)), l.l111);
    }
};

// LB(lambda), eq. 5.  After a full iteration c_e and c_t are the stored state.
rama_status lower_bound_now(Ctx &ctx, const float *ce, size_t m, const float *ct, size_t T, double *dev_out)
{
    RAMA_TRY(device_sum(ctx, EdgeLB{ce}, m, dev_out, false));
    if (T > 0) RAMA_TRY(device_sum(ctx, TriLB{ct}, T, dev_out, true));
    return RAMA_OK;
}

rama_status copy_graph(Ctx &ctx, const Graph &g, Graph &out)
{
    out.n = g.n; out.m = g.m;
    out.sign_sums.reset();
    size_t m = (size_t)(g.m > 0 ? g.m : 1);
    RAMA_TRY(out.i.alloc(ctx, m));
    RAMA_TRY(out.j.alloc(ctx, m));
    RAMA_TRY(out.c.alloc(ctx, m));
    if (g.m > 0) {
        HIP_TRY(ctx, hipMemcpyAsync(out.i.get(), g.i.get(), (size_t)g.m * 4, hipMemcpyDeviceToDevice, ctx.stream));
        HIP_TRY(ctx, hipMemcpyAsync(out.j.get(), g.j.get(), (size_t)g.m * 4, hipMemcpyDeviceToDevice, ctx.stream));
        HIP_TRY(ctx, hipMemcpyAsync(out.c.get(), g.c.get(), (size_t)g.m * 4, hipMemcpyDeviceToDevice, ctx.stream));
    }
    return RAMA_OK;
}

// From the triangles' edges (skey: three per triangle, in ascending order of the triangles) to the reduced costs in aug.c.
// inc_heads: a plan over the 3T slots with two spare words, the first of which is raised when a cycle uses an edge that is
// not in the graph.  ct: the triangles' costs; with ct_lazy they are zero and have no memory yet.
rama_status pass_messages(Ctx &ctx, Graph &aug, size_t T, Buf<uint32_t> &skey, ScanPlan<uint32_t> &inc_heads, Buf<float> &ct, bool ct_lazy,
                          int k_iters, double *lower_bound, double *lb_trace, double *lb_dev, DualState *next)
{
    const size_t ma = (size_t)aug.m;
    if (messages_fit(T) && ct_lazy && !next) {      // with ct_lazy there are iterations and no trace
        bool raised = false;
        RAMA_TRY(ct.alloc(ctx, 3 * T));
        RAMA_TRY(messages_few(ctx, skey.get(), T, k_iters, aug.c.get(), ct.get(), inc_heads.extra_ptr(), &raised));
        if (raised) return fail(ctx, RAMA_ERR_BAD_GRAPH, "a cycle uses an edge that is not in the graph");
        if (!lower_bound) return RAMA_OK;
        RAMA_TRY(lower_bound_now(ctx, aug.c.get(), ma, ct.get(), T, lb_dev));
        return read_back(ctx, lower_bound, lb_dev, 8);
    }
    Buf<uint32_t> slot, tri_act;   // tri_act: per triangle slot its edge's number among the active edges
    RAMA_TRY(slot.alloc(ctx, 3 * T));
    // ---- incidence: slots of every edge in ascending triangle order ----------------------------
    // (if the flag is up, the edge ids below are placeholders -- all valid indices -- and the result is discarded)
    Buf<uint32_t> inc_head_sums;   // heads per scan tile, if the sort's last kernel could count them
    SortAgain<uint32_t, uint32_t> again;
    again.flag = inc_heads.extra_ptr() + 1;
    RAMA_TRY((radix_sort_pairs<uint32_t, uint32_t>(ctx, skey, slot, 3 * T, bits_for((uint64_t)ma), true, &inc_head_sums, (uint64_t)ma, &again)));   // values: the slots 0..3T-1
    Buf<uint32_t> act_edge, act_start;
    size_t na = 0;
    {
        ScanPlan<uint32_t> &heads = inc_heads;
        RAMA_TRY((count_heads<uint32_t, uint32_t>(ctx, skey, &slot, 3 * T, bits_for((uint64_t)ma), [](const uint32_t *k) { return HeadFlag32{k}; }, heads, 1,
                                                  inc_head_sums, again)));
        if (heads.extra_value[0]) return fail(ctx, RAMA_ERR_BAD_GRAPH, "a cycle uses an edge that is not in the graph");
        na = heads.total;
        RAMA_TRY(act_edge.alloc(ctx, na));
        RAMA_TRY(act_start.alloc(ctx, na + 1));
        RAMA_TRY(tri_act.alloc(ctx, 3 * T));
        RAMA_TRY((scan_emit<uint32_t>(ctx, HeadFlag32{skey.get()},
                                      ActiveEdgesEmit{skey.get(), slot.get(), (uint32_t)(3 * T), (uint32_t)na, act_edge.get(),
                                                      act_start.get(), tri_act.get()},
                                      heads, (double)(na * 8 + 3 * T * 8))));
    }
    skey.reset();
    // ---- iterations ----------------------------------------------------------------------------
    Buf<float> share, msg;
    if (ct_lazy) RAMA_TRY(ct.alloc(ctx, 3 * T));
    RAMA_TRY(share.alloc(ctx, na));
    RAMA_TRY(msg.alloc(ctx, 3 * T));
    float *ce = aug.c.get();
    {
        ProfScope ps_(ctx, "k_edge_init", (double)(na * 16));
        k_edge_init<<<grid_for(na), kBlock, 0, ctx.stream>>>(na, act_edge.get(), act_start.get(), ce, share.get());
    }
    LAUNCH_TRY(ctx, "edge_init");
    if (lb_trace) {
        RAMA_TRY(lower_bound_now(ctx, ce, ma, ct.get(), T, lb_dev));
        RAMA_TRY(read_back(ctx, &lb_trace[0], lb_dev, 8));
    }
    for (int it = 1; it <= k_iters; ++it) {
        const bool first = it == 1 && ct_lazy;
        if (ctx.prof.wants("k_triangle_update")) {   // timed by the dispatch's own start and stop stamps
            hipEvent_t ea, eb;
            ctx.prof.begin_stamped("k_triangle_update", (double)(T * (first ? 48 : 60)), &ea, &eb);
            if (first)
                hipExtLaunchKernelGGL(k_triangle_update<true>, dim3(xcd_grid(grid_for(T))), dim3(kBlock), 0, ctx.stream, ea, eb, 0, (size_t)T,
                                      (const uint32_t *)tri_act.get(), (const float *)share.get(), (float *)ct.get(), (float *)msg.get());
            else
                hipExtLaunchKernelGGL(k_triangle_update<false>, dim3(xcd_grid(grid_for(T))), dim3(kBlock), 0, ctx.stream, ea, eb, 0, (size_t)T,
                                      (const uint32_t *)tri_act.get(), (const float *)share.get(), (float *)ct.get(), (float *)msg.get());
        } else if (first) {
            k_triangle_update<true><<<xcd_grid(grid_for(T)), kBlock, 0, ctx.stream>>>(T, tri_act.get(), share.get(), ct.get(), msg.get());
        } else {
            k_triangle_update<false><<<xcd_grid(grid_for(T)), kBlock, 0, ctx.stream>>>(T, tri_act.get(), share.get(), ct.get(), msg.get());
        }
        LAUNCH_TRY(ctx, "triangle_update");
        {
            const bool store_ce = it == k_iters || lb_trace != nullptr;
            ProfScope ps_(ctx, store_ce ? "k_edge_update<true>" : "k_edge_update<false>", (double)(na * (store_ce ? 16 : 8) + 3 * T * 8));
            auto update = [&](auto store, auto per) {
                constexpr int kPer = decltype(per)::value;
                k_edge_update<decltype(store)::value, kPer><<<xcd_grid(grid_for(na, kBlock * kPer)), kBlock, 0, ctx.stream>>>(
                    na, act_edge.get(), act_start.get(), slot.get(), msg.get(), ce, share.get());
            };
            using std::integral_constant;
            if (na <= kFewEdges) {
                if (store_ce) update(std::true_type{}, integral_constant<int, 1>{});
                else update(std::false_type{}, integral_constant<int, 1>{});
            } else {
                if (store_ce) update(std::true_type{}, integral_constant<int, kEdgesPerThread>{});
                else update(std::false_type{}, integral_constant<int, kEdgesPerThread>{});
            }
        }
        LAUNCH_TRY(ctx, "edge_update");
        if (lb_trace) {
            RAMA_TRY(lower_bound_now(ctx, ce, ma, ct.get(), T, lb_dev));
            RAMA_TRY(read_back(ctx, &lb_trace[it], lb_dev, 8));
        }
    }
    if (lower_bound) {
        if (lb_trace) *lower_bound = lb_trace[k_iters];
        else {
            RAMA_TRY(lower_bound_now(ctx, ce, ma, ct.get(), T, lb_dev));
            RAMA_TRY(read_back(ctx, lower_bound, lb_dev, 8));
        }
    }
    if (next) {
        next->T = T;
        RAMA_TRY(next->tri_nodes.alloc(ctx, 3 * T));
        {
            ProfScope ps_(ctx, "k_triangle_nodes", (double)(T * 36));
            k_triangle_nodes<<<grid_for(T), kBlock, 0, ctx.stream>>>(T, tri_act.get(), act_edge.get(), aug.i.get(), aug.j.get(),
                                                                  next->tri_nodes.get());
        }
        LAUNCH_TRY(ctx, "triangle_nodes");
        next->ct = std::move(ct);
    }
    return RAMA_OK;
}

}  // namespace

rama_status dual_update(Ctx &ctx, const Graph &g, int lists, const int32_t *const *cycles, const int64_t *n_cycles,
                        bool validate_cycles, int k_iters, Graph &out, double *lower_bound, double *lb_trace,
                        DualInfo *info, DualState *prev, DualState *next, Graph *donor)
{
    if (lists < 0 || lists > kCycleLists || k_iters < 0 || (lists > 0 && (!cycles || !n_cycles)))
        return fail(ctx, RAMA_ERR_INVALID_ARG, "message passing: bad cycle lists or iteration count");
    RAMA_TRY(zero_page_recycle(ctx));
    CycleSet cs;
    size_t ncyc = 0, nfan = 0, nch = 0;
    double cycle_bytes = 0.0;
    const size_t T_kept = prev ? prev->T : 0;
    for (int k = 0; k < kCycleSets; ++k) {
        cs.c[k] = nullptr;
        if (k == kCycleLists) {
            cs.c[k] = prev ? prev->tri_nodes.get() : nullptr;
            ncyc += T_kept;
            nfan += T_kept;
        } else if (k < lists) {
            if (n_cycles[k] < 0) return fail(ctx, RAMA_ERR_INVALID_ARG, "message passing: negative count");
            if (n_cycles[k] > 0 && !cycles[k]) return fail(ctx, RAMA_ERR_INVALID_ARG, "message passing: null cycle list");
            cs.c[k] = cycles[k];
            ncyc += (size_t)n_cycles[k];
            nfan += (size_t)(k + 1) * (size_t)n_cycles[k];
            nch += (size_t)k * (size_t)n_cycles[k];
            cycle_bytes += 4.0 * (k + 3) * (double)n_cycles[k];
        }
        if (3 * nfan >= (size_t(1) << 31)) return fail(ctx, RAMA_ERR_CAPACITY, "triangle slots reach 2^31");
        cs.cyc_end[k] = (uint32_t)ncyc; cs.fan_end[k] = (uint32_t)nfan; cs.chord_end[k] = (uint32_t)nch;
    }
    const size_t m = (size_t)g.m;
    if (3 * nfan >= (size_t(1) << 31) || m + nch >= (size_t(1) << 31))
        return fail(ctx, RAMA_ERR_CAPACITY, "triangle slots or augmented edges reach 2^31");
    if (info) info->n_triangles = 0;
    Buf<double> lb_dev;
    RAMA_TRY(lb_dev.alloc(ctx, 1));
    if (nfan == 0 || m == 0) {
        if (nfan > 0) return fail(ctx, RAMA_ERR_BAD_GRAPH, "cycles given for a graph without edges");
        RAMA_TRY(copy_graph(ctx, g, out));
        double lb = 0.0;
        if (lower_bound || lb_trace) RAMA_TRY(negative_cost_sum(ctx, g.c.get(), g.m, &lb));
        if (lower_bound) *lower_bound = lb;
        if (lb_trace) for (int k = 0; k <= k_iters; ++k) lb_trace[k] = lb;
        return RAMA_OK;
    }
    const int32_t n = g.n;
    const int nbits = bits_for((uint64_t)n);
    // "a cycle uses an edge that is not in the graph": raised by the kernels that look edges up, read by the
    // host together with the next count it waits for anyway
    Buf<int32_t> flag;   // [0]: the flag, [1]: the longest row of the upper adjacency (filled in further down)
    RAMA_TRY(zeroed<int32_t>(ctx, 2, flag));
    // rows of the canonical edge list (upper CSR)
    Buf<int32_t> rowptr;
    RAMA_TRY(rowptr.alloc(ctx, (size_t)n + 1));
    RAMA_TRY((row_bounds<int32_t, int32_t>(ctx, g.i.get(), m, n, rowptr.get())));
    if (validate_cycles) {
        {
            ProfScope ps_(ctx, "k_validate_cycles", cycle_bytes);
            k_validate_cycles<<<grid_for(ncyc), kBlock, 0, ctx.stream>>>(cs, n, rowptr.get(), g.j.get(), flag.get());
        }
        LAUNCH_TRY(ctx, "validate_cycles");
        int32_t hf = 0;
        RAMA_TRY(read_back(ctx, &hf, flag.get(), 4));
        if (hf) return fail(ctx, RAMA_ERR_BAD_GRAPH, "a cycle has repeated / out-of-range nodes or uses an edge that is not in the graph");
    }
    // ---- chords -> augmented edge list -------------------------------------------------------
    Graph aug;
    aug.n = n;
    uint32_t nnew = 0;
    const bool many_repeats = cs.chord_end[kCycleLists - 1] > cs.chord_end[1];      // cycles of five and more nodes
    if (nch > 0) {
        Buf<uint64_t> ckey;
        RAMA_TRY(ckey.alloc(ctx, nch));
        if (many_repeats) {
            Buf<uint32_t> fresh;
            RAMA_TRY(zeroed<uint32_t>(ctx, 1, fresh));
            {
                ProfScope ps_(ctx, "k_new_chords", (double)(nch * 8));
                k_new_chords<<<grid_for(nch, kSetTile), kBlock, 0, ctx.stream>>>(cs, nch, nbits, ckey.get(), fresh.get());
            }
            LAUNCH_TRY(ctx, "new_chords");
            uint32_t left = 0;
            RAMA_TRY(read_back(ctx, &left, fresh.get(), 4));
            nch = left;        // at least one
        } else {
            ProfScope ps_(ctx, "k_chord_keys", (double)(nch * 24));
            k_chord_keys<<<grid_for(nch), kBlock, 0, ctx.stream>>>(cs, nch, nbits, ckey.get());
        }
        LAUNCH_TRY(ctx, "chord_keys");
        RAMA_TRY((radix_sort_keys<uint64_t>(ctx, ckey, nch, 2 * nbits, nullptr, (uint64_t)n << nbits)));
        Buf<uint32_t> cpos;
        Buf<int32_t> where;
        RAMA_TRY(cpos.alloc(ctx, nch + 1));
        RAMA_TRY(where.alloc(ctx, nch));
        {
            ProfScope ps_(ctx, "k_chord_lookup", (double)(nch * 20));
            k_chord_lookup<<<grid_for(nch), kBlock, 0, ctx.stream>>>(nch, ckey.get(), rowptr.get(), g.j.get(), nbits,
                                                                    where.get());
        }
        LAUNCH_TRY(ctx, "chord_lookup");
        RAMA_TRY((exclusive_scan<uint32_t>(ctx, NewChordFlag{where.get()}, cpos.get(), nch)));
        RAMA_TRY(read_back(ctx, &nnew, cpos.get() + nch, 4));
        if (nnew > 0) {
            Buf<int32_t> ci, cj, before, ins;
            RAMA_TRY(ci.alloc(ctx, nnew));
            RAMA_TRY(cj.alloc(ctx, nnew));
            RAMA_TRY(before.alloc(ctx, nnew));
            RAMA_TRY(ins.alloc(ctx, m + 2));
            {
                ProfScope ps_(ctx, "k_emit_chords", (double)(nch * 16 + (size_t)nnew * 12));
                k_emit_chords<<<grid_for(nch), kBlock, 0, ctx.stream>>>(nch, ckey.get(), where.get(), cpos.get(), nbits,
                                                                       ci.get(), cj.get(), before.get());
            }
            LAUNCH_TRY(ctx, "emit_chords");
            // ins[v] = number of chords with before < v ; chords placed before edge e: before <= e -> ins[e+1]
            RAMA_TRY((row_bounds<int32_t, int32_t>(ctx, before.get(), nnew, (int64_t)m + 1, ins.get())));
            aug.m = (int64_t)(m + nnew);
            RAMA_TRY(aug.i.alloc(ctx, (size_t)aug.m));
            RAMA_TRY(aug.j.alloc(ctx, (size_t)aug.m));
            RAMA_TRY(aug.c.alloc(ctx, (size_t)aug.m));
            {
                ProfScope ps_(ctx, "k_merge_edges", (double)(m * 16 + (size_t)nnew * 12 + (m + nnew) * 12));
                k_merge_edges<<<grid_for(m), kBlock, 0, ctx.stream>>>(m, g.i.get(), g.j.get(), g.c.get(), ins.get(), ci.get(),
                                                                 cj.get(), before.get(), aug.i.get(), aug.j.get(),
                                                                 aug.c.get());
            }
            LAUNCH_TRY(ctx, "merge_edges");
            RAMA_TRY((row_bounds<int32_t, int32_t>(ctx, aug.i.get(), (size_t)aug.m, n, rowptr.get())));
        }
    }
    if (nnew == 0) {
        // no chord to add: the augmented graph is the input graph.  `donor` (the same graph, owned by a
        // caller that replaces it by the result anyway) hands its arrays over instead of being copied;
        // nothing below reads g.
        if (donor) {
            aug.n = g.n; aug.m = g.m;
            aug.i = std::move(donor->i); aug.j = std::move(donor->j); aug.c = std::move(donor->c);
        } else {
            RAMA_TRY(copy_graph(ctx, g, aug));
        }
    }
    const size_t ma = (size_t)aug.m;
    // ---- triangles -----------------------------------------------------------------------------
    // Where one workgroup sorts the keys by itself nobody waits to hear of the longest row.  (A sort of more keys has longer
    // buckets of equal leading bits with a wider second field: 3.4e5 keys 45 us slower, the wait takes 20.)
    int dbits = bits_for((uint64_t)n);
    if (bits_for((uint64_t)ma) + dbits > 31 || nfan > (size_t)LocalSort<uint32_t>::cap) {
        uint32_t *maxrow = (uint32_t *)(flag.get() + 1);
        {
            ProfScope ps_(ctx, "k_max_row", (double)(((size_t)n + 1) * 4));
            k_max_row<<<grid_for((size_t)n, kBlock * kMaxRowItems), kBlock, 0, ctx.stream>>>(n, rowptr.get(), maxrow);
        }
        LAUNCH_TRY(ctx, "max_row");
        uint32_t hmax = 0;
        RAMA_TRY(read_back(ctx, &hmax, maxrow, 4));
        dbits = bits_for((uint64_t)hmax + 1);
    }
    const int kbits = bits_for((uint64_t)ma) + dbits;
    Buf<uint32_t> skey;
    size_t T = 0;
    Buf<float> ct;
    ScanPlan<uint32_t> inc_heads;   // scan over the sorted slot list (incidence); its spare word carries the flag to the host
    // new triangles start at zero costs; when iterations follow at once, nobody stores or fetches those zeros
    // (the first triangle update knows).  Someone who looks at c_t before the first iteration needs them: the
    // bound trace, a call without iterations, a caller who keeps the triangles.  Their memory is asked for behind the
    // incidence sort then, whose two pairs of slot arrays are what a round needs most memory for.
    const bool ct_lazy = T_kept == 0 && k_iters > 0 && lb_trace == nullptr;
    auto triangles = [&](auto key_tag) -> rama_status {
        using KT = decltype(key_tag);
        Buf<KT> tkey;
        Buf<uint32_t> origin;
        RAMA_TRY(tkey.alloc(ctx, nfan));
        size_t nkeys = nfan;
        if (many_repeats && T_kept == 0) {
            Buf<uint32_t> fresh;
            RAMA_TRY(zeroed<uint32_t>(ctx, 1, fresh));
            {
                ProfScope ps_(ctx, "k_new_triangle_keys", (double)(nfan * 12));
                k_new_triangle_keys<KT><<<grid_for(nfan, kSetTile), kBlock, 0, ctx.stream>>>(cs, nfan, rowptr.get(), aug.j.get(), dbits,
                                                                                            tkey.get(), flag.get(), fresh.get());
            }
            LAUNCH_TRY(ctx, "new_triangle_keys");
            uint32_t left = 0;
            RAMA_TRY(read_back(ctx, &left, fresh.get(), 4));
            nkeys = left;      // at least one
        } else {
            ProfScope ps_(ctx, "k_triangle_keys", (double)(nfan * (12 + sizeof(KT))));
            k_triangle_keys<KT><<<grid_for(nfan), kBlock, 0, ctx.stream>>>(cs, nfan, rowptr.get(), aug.j.get(), dbits,
                                                                          tkey.get(), flag.get());
        }
        LAUNCH_TRY(ctx, "triangle_keys");
        Buf<uint32_t> head_sums;   // heads per scan tile, if the sort's last kernel could count them
        ScanPlan<uint32_t> heads;
        RAMA_TRY((scan_plan_alloc<uint32_t>(ctx, nkeys, 1, heads)));
        SortAgain<KT, uint32_t> again;
        again.flag = heads.extra_ptr();
        if (T_kept > 0) {   // the sort also has to tell where the kept triangles end up
            RAMA_TRY(origin.alloc(ctx, nfan));
            RAMA_TRY((radix_sort_pairs<KT, uint32_t>(ctx, tkey, origin, nfan, kbits, true, &head_sums, kbits < 64 ? (uint64_t)ma << dbits : 0, &again)));   // values: the fan indices 0..nfan-1
        } else {
            RAMA_TRY((radix_sort_keys<KT>(ctx, tkey, nkeys, kbits, &head_sums, kbits < 64 ? (uint64_t)ma << dbits : 0, &again)));
        }
        RAMA_TRY((count_heads<KT, uint32_t>(ctx, tkey, T_kept > 0 ? &origin : nullptr, nkeys, kbits, [](const KT *k) { return HeadFlagT<KT>{k}; }, heads, 0,
                                            head_sums, again)));
        T = heads.total;
        if (!ct_lazy) RAMA_TRY(ct.alloc(ctx, 3 * T));
        if (T_kept > 0) RAMA_TRY(fill<float>(ctx, ct.get(), 0.0f, 3 * T));   // otherwise the consumer below zeroes what it creates
        RAMA_TRY(skey.alloc(ctx, 3 * T));
        RAMA_TRY((scan_plan_alloc<uint32_t>(ctx, 3 * T, 2, inc_heads)));
        TrianglesEmit<KT> te{tkey.get(), rowptr.get(), aug.j.get(), dbits, skey.get(), flag.get(),
                             (int32_t *)inc_heads.extra_ptr(), T_kept > 0 ? origin.get() : nullptr, cs.fan_end[kCycleLists - 1], cs.fan_end[kCycleLists],
                             T_kept > 0 ? prev->ct.get() : nullptr, ct.get(), !ct_lazy};
        RAMA_TRY((scan_emit<uint32_t>(ctx, HeadFlagT<KT>{tkey.get()}, te, heads, (double)(T * 20 + T_kept * 24))));
        return RAMA_OK;
    };
    if (kbits <= 32) RAMA_TRY(triangles(uint32_t{}));
    else RAMA_TRY(triangles(uint64_t{}));
    if (info) info->n_triangles = (int64_t)T;
    // the kept triangles are taken over, and the keys are gone: the incidence sort needs the memory
    if (prev) { prev->tri_nodes.reset(); prev->ct.reset(); }
    rowptr.reset();
    RAMA_TRY(pass_messages(ctx, aug, T, skey, inc_heads, ct, ct_lazy, k_iters, lower_bound, lb_trace, lb_dev.get(), next));
    out.n = aug.n; out.m = aug.m;
    out.i = std::move(aug.i); out.j = std::move(aug.j); out.c = std::move(aug.c);
    out.sign_sums.reset();   // the costs are new
    return RAMA_OK;
}

// A round whose predecessor had this many triangles at most is tried by one workgroup first: their number shrinks from round
// to round, mostly to a third or a fifth.  A try that succeeds takes 33 to 75 us for separation and messages where the list
// takes 115 to 160, a try that fails costs 20 to 30 at 10^5 edges, and up to the time of the counting pass at 10^7.
constexpr int64_t kTryFewFrom = 8192;

rama_status triangle_round(Ctx &ctx, Graph &g, int k_iters, int64_t last, bool any, double *lower_bound, TriangleCounts &out,
                           const std::function<void()> &separated)
{
    RAMA_TRY(zero_page_recycle(ctx));
    out = TriangleCounts{};
    if (g.m == 0) return RAMA_OK;
    Buf<int32_t> rowptr;
    RAMA_TRY(rowptr.alloc(ctx, (size_t)g.n + 1));
    RAMA_TRY((row_bounds<int32_t, int32_t>(ctx, g.i.get(), (size_t)g.m, g.n, rowptr.get())));
    TriangleSurvey survey;
    RAMA_TRY(triangle_survey(ctx, g, rowptr.get(), any, survey));
    if (last >= 0 && last <= kTryFewFrom && !lower_bound) {
        bool done = false;
        RAMA_TRY(triangles_few(ctx, g, rowptr.get(), survey, k_iters, out, &done, separated));
        if (done || out.dense) return RAMA_OK;
    }
    Buf<uint32_t> skey;
    RAMA_TRY(triangles_list(ctx, g, rowptr.get(), survey, skey, out));
    if (out.dense) return RAMA_OK;
    separated();
    rowptr.reset();
    const size_t T = (size_t)out.triangles;
    if (T == 0) return RAMA_OK;
    ScanPlan<uint32_t> inc_heads;
    RAMA_TRY((scan_plan_alloc<uint32_t>(ctx, 3 * T, 2, inc_heads)));
    Buf<float> ct;
    Buf<double> lb_dev;
    RAMA_TRY(lb_dev.alloc(ctx, 1));
    RAMA_TRY(pass_messages(ctx, g, T, skey, inc_heads, ct, true, k_iters, lower_bound, nullptr, lb_dev.get(), nullptr));
    g.sign_sums.reset();      // the costs are new
    return RAMA_OK;
}

}  // namespace rama
