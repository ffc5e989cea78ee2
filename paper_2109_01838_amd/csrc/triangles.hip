// Separation and message passing of a round that separates triangles only (every round behind the first, by default).
//
// A conflicted triangle u < v < w has exactly one repulsive edge and two attractive ones (paper Sec. 3.2.2).  On the
// canonical list its edges (u,v), (u,w), (v,w) stand in this order, and ascending pairs of places (of (u,v), of (u,w)) are
// ascending triples (u,v,w).  So the triangles come out of the list itself: for every edge (u,v), the common entries of
// the rest of row u and of row v, with the signs looked at on the way -- no attractive adjacency (which takes a sort of
// the lower neighbours), no list of cycles, no keys and no sort to put the triangles in order.  The work is the sum over
// the edges of the shorter of the two stretches, whatever the degrees.
//
// Two ways from there:
//   few     at most kFewTriangles: listed in any order by one launch, and one workgroup does the incidence and all
//           iterations (k_messages_few); the host hears of it when it is over;
//   many    counted tile by tile, scanned, listed in order; the incidence sort and the iterations of dual.hip follow.
//
// Measured against the lists of cycles (cycles.hip, then chords, keys and their sort in dual.hip), us for the separation and
// the message passing of a round: 9.4e7 edges with 1.5e7 triangles 4800 instead of 6900, 1.6e6 with 3.1e5 300 instead of 433,
// 3.2e5 with 2.5e4 of a volume's late round 124 instead of 273, 8.1e4 with 246 triangles 40 instead of 185.  Solves:
// 128^2 long-range grid 2.79 -> 2.28 ms, 512^2 7.0 -> 5.9, 6-NN graph of 10^6 points 11.5 -> 9.95, 61x97x131 volume 7.2 -> 5.8,
// 320^3 volume 84.4 -> 78.1.
#include "prim.h"
#include "steps.h"

namespace rama {

namespace {

// ---------------------------------------------------------------------------------------------
// triangles of a tile of consecutive edges
// ---------------------------------------------------------------------------------------------
// A workgroup takes EDGES consecutive edges (u,v).  Each is tried with every entry of the shorter of two stretches -- the
// rest of row u behind the edge, and row v -- and the entry is searched in the longer one.  The tries are dealt out evenly
// over the threads (their numbers, summed up, are in LDS), so neither a long row nor an edge without tries leaves a lane
// waiting.  In order of their numbers the tries meet the triangles in ascending order.
enum TriangleMode { kTriList, kTriCount, kTriFill };

struct TriangleGraph {
    const int32_t *rowptr, *i, *j;
    const float *c;
    size_t m;
    const uint64_t *signs;      // attractive edges | repulsive edges << 32
};
__device__ __forceinline__ bool both_signs(uint64_t signs) { return (uint32_t)signs != 0u && (signs >> 32) != 0u; }

constexpr int kTriBatch = 2;                   // tries a thread has under way at a time
// triangles of a tile that the counting pass keeps: contracted grids and neighbour graphs have about one to five edges
constexpr int tri_room(int edges) { return edges * 7 / 16 + 8; }
template <int EDGES>
struct TriangleTile {
    uint32_t before[EDGES];                    // tries of the tile's edges in front
    int32_t scan[EDGES], lo[EDGES], hi[EDGES]; // start of the stretch that is walked; the stretch that is searched
    uint8_t kind[EDGES];                       // bit 0: the edge is repulsive, bit 1: row v is walked
    uint32_t wave[2][kTriBatch * (kBlock / 64)];
    uint32_t over;
};

// The counter of a list that takes no more than `cap`, and a word that says it is full, once per XCD, each in a cache line of
// its own: 6.2e4 waves that look at the counter itself, one after the other in one line, took 65 us.
constexpr int kListLine = 32, kListWords = kListLine * 9;
__device__ __forceinline__ uint32_t *list_over(uint32_t *counter, uint32_t xcd) { return counter + kListLine * (1u + xcd); }

// Bounded by the latency of a try's chain (its edge by bisection in LDS, the entry, three to five probes, the sign), so
// what counts is the number of tries under way: two to a thread, every step made for both before the next; 64 edges to a
// workgroup on short lists and on dense rows, 256 beyond (see wide_tiles).
// The listing pass is over as soon as there are more than cap triangles: the wave that brings the counter beyond cap tells it.
// (Run to its end, with an atomic for every wave that finds any, it took 2 ms for the 2.1e6 triangles of 9.6e6 edges, 11 for
// 8.8e6 of 3.9e7.)
// The counting pass keeps what it finds, tile by tile in `list`, as long as the tile's room lasts, and the fill pass copies
// it to its place; tiles with more triangles are searched again.  (One list for all tiles, its next free place behind an
// atomic counter, took 12 ns per tile: 7.9 instead of 2.5 ms for 650000 of them.)
template <int MODE, int EDGES>
__global__ __launch_bounds__(kBlock) void k_triangles(TriangleGraph g, uint32_t nb, uint32_t *list, uint32_t cap, uint32_t *counter,
                                                      uint64_t *sums, const uint64_t *offs, uint32_t *slots)
{
    constexpr int kWaves = kBlock / 64;
    __shared__ TriangleTile<EDGES> S;
    constexpr uint32_t kRoom = (uint32_t)tri_room(EDGES);
    const uint32_t tile = xcd_block();
    if (tile >= nb) return;      // the whole workgroup (padding of the grid)
    const int tid = (int)threadIdx.x, lane = lane_id(), w = tid >> 6;
    uint64_t at = 0;
    if constexpr (MODE != kTriFill) {
        if (!both_signs(*g.signs)) {      // no triangle in the whole graph
            if (MODE == kTriCount && tid == 0) sums[tile] = 0;
            return;
        }
    }
    if constexpr (MODE == kTriFill) {
        at = offs[tile];
        const uint32_t n = (uint32_t)(offs[tile + 1] - at);
        if (n <= kRoom) {      // the whole workgroup
            const uint32_t *from = list + 3 * (size_t)kRoom * tile;
            for (uint32_t k = (uint32_t)tid; k < 3 * n; k += kBlock) slots[3 * (size_t)at + k] = from[k];
            return;
        }
    }
    const size_t e_first = (size_t)tile * EDGES;
    uint32_t tries = 0;
    if constexpr (MODE == kTriList) {
        if (tid == 0) S.over = __hip_atomic_load(list_over(counter, blockIdx.x & 7u), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    if (tid < EDGES) {
        const size_t e = e_first + (size_t)tid;
        if (e < g.m) {
            const int32_t v = g.j[e];
            const float c = g.c[e];
            const int32_t a0 = (int32_t)e + 1, a1 = g.rowptr[g.i[e] + 1], b0 = g.rowptr[v], b1 = g.rowptr[v + 1];
            const bool walk_v = b1 - b0 < a1 - a0;
            tries = c > 0.0f || c < 0.0f ? (uint32_t)(walk_v ? b1 - b0 : a1 - a0) : 0u;
            S.scan[tid] = walk_v ? b0 : a0;
            S.lo[tid] = walk_v ? a0 : b0;
            S.hi[tid] = walk_v ? a1 : b1;
            S.kind[tid] = (uint8_t)((c < 0.0f ? 1 : 0) | (walk_v ? 2 : 0));
        }
    }
    const uint32_t inc = wave_inclusive_scan(tries);
    if (lane == 63) S.wave[0][w] = inc;
    __syncthreads();
    uint32_t total = 0, pre = 0;
#pragma unroll
    for (int k = 0; k < kWaves; ++k) {
        const uint32_t x = S.wave[0][k];
        pre += k < w ? x : 0u;
        total += x;
    }
    if (tid < EDGES) S.before[tid] = pre + inc - tries;
    __syncthreads();
    if constexpr (MODE == kTriList) {
        if (S.over) return;      // the whole workgroup; behind this point there is no barrier, and a wave may leave by itself
    }
    uint32_t found = 0;
    for (uint32_t p0 = 0, turn = 1; p0 < total; p0 += kTriBatch * kBlock, ++turn) {      // the same number of turns for all threads
        int t[kTriBatch];
        int32_t y[kTriBatch], lo[kTriBatch], hi[kTriBatch], node[kTriBatch], e1[kTriBatch], e2[kTriBatch];
        float cy[kTriBatch], cz[kTriBatch];
        uint32_t kind[kTriBatch];
#pragma unroll
        for (int q = 0; q < kTriBatch; ++q) {
            const uint32_t p = p0 + (uint32_t)(q * kBlock + tid);
            t[q] = 0;      // the last edge with at most p tries before its own
#pragma unroll
            for (int step = EDGES / 2; step > 0; step >>= 1)
                if (S.before[t[q] + step] <= p) t[q] += step;
            const bool any = p < total;
            y[q] = any ? S.scan[t[q]] + (int32_t)(p - S.before[t[q]]) : (int32_t)e_first;
            lo[q] = any ? S.lo[t[q]] : 0;
            hi[q] = any ? S.hi[t[q]] : 0;
            kind[q] = S.kind[t[q]];
        }
#pragma unroll
        for (int q = 0; q < kTriBatch; ++q) { cy[q] = g.c[y[q]]; node[q] = g.j[y[q]]; }
#pragma unroll
        for (int q = 0; q < kTriBatch; ++q) {      // exactly one of the three edges is repulsive, none is zero
            if (!(cy[q] > 0.0f || (cy[q] < 0.0f && !(kind[q] & 1u)))) { lo[q] = 0; hi[q] = 0; }
        }
        int32_t row[kTriBatch][8], z[kTriBatch];
#pragma unroll
        for (int q = 0; q < kTriBatch; ++q) __builtin_memcpy(row[q], g.j + lo[q], sizeof(row[q]));      // device arrays end with slack
#pragma unroll
        for (int q = 0; q < kTriBatch; ++q) {
            z[q] = -1;
#pragma unroll
            for (int k = 0; k < 8; ++k)
                if (lo[q] + k < hi[q] && row[q][k] == node[q]) z[q] = lo[q] + k;
            if (z[q] < 0 && hi[q] - lo[q] > 8 && row[q][7] < node[q]) z[q] = find_edge_between(g.j, lo[q] + 8, hi[q], node[q]);
        }
#pragma unroll
        for (int q = 0; q < kTriBatch; ++q) cz[q] = g.c[z[q] < 0 ? (int32_t)e_first : z[q]];
        uint64_t hits[kTriBatch];
#pragma unroll
        for (int q = 0; q < kTriBatch; ++q) {
            const bool hit = z[q] >= 0 && ((kind[q] & 1u) || cy[q] < 0.0f ? cz[q] > 0.0f : cz[q] < 0.0f);
            e1[q] = !hit ? -1 : kind[q] & 2u ? z[q] : y[q];
            e2[q] = kind[q] & 2u ? y[q] : z[q];
            hits[q] = __ballot(hit);
        }
        auto put = [&](uint32_t *to, size_t k, int q) {
            to[3 * k] = (uint32_t)(e_first + (size_t)t[q]); to[3 * k + 1] = (uint32_t)e1[q]; to[3 * k + 2] = (uint32_t)e2[q];
        };
        if constexpr (MODE == kTriList) {
            bool full = false;
#pragma unroll
            for (int q = 0; q < kTriBatch; ++q)
                if (hits[q]) {      // uniform in the wave
                    const uint32_t n = (uint32_t)__popcll(hits[q]);
                    uint32_t base = 0;
                    if (lane == 0) base = atomicAdd(counter, n);
                    base = (uint32_t)__builtin_amdgcn_readfirstlane((int)base);
                    if (base <= cap && base + n > cap && lane < 8)      // one wave
                        __hip_atomic_store(list_over(counter, (uint32_t)lane), 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    full |= base > cap;
                    base += (uint32_t)__popcll(hits[q] & ((1ull << lane) - 1ull));
                    if (e1[q] >= 0 && base < cap) put(list, base, q);
                }
            if (full) return;
        } else {
            if (lane == 0) {
#pragma unroll
                for (int q = 0; q < kTriBatch; ++q) S.wave[turn & 1u][q * kWaves + w] = (uint32_t)__popcll(hits[q]);
            }
            __syncthreads();
            uint32_t mine[kTriBatch] = {}, all = 0;
#pragma unroll
            for (int k = 0; k < kTriBatch * kWaves; ++k) {
                const uint32_t x = S.wave[turn & 1u][k];
#pragma unroll
                for (int q = 0; q < kTriBatch; ++q) mine[q] += k < q * kWaves + w ? x : 0u;
                all += x;
            }
#pragma unroll
            for (int q = 0; q < kTriBatch; ++q)
                if (e1[q] >= 0) {
                    const uint32_t k = found + mine[q] + (uint32_t)__popcll(hits[q] & ((1ull << lane) - 1ull));
                    if constexpr (MODE == kTriFill) put(slots, (size_t)at + k, q);
                    else if (k < kRoom) put(list, (size_t)kRoom * tile + k, q);
                }
            found += all;
        }
    }
    if constexpr (MODE == kTriCount) {
        if (tid == 0) sums[tile] = found;      // the same in all threads
    }
}

// sum of nb packed sign counts, by one workgroup
__global__ __launch_bounds__(kBlock) void k_total_signs(const uint64_t *sums, size_t nb, uint64_t *out)
{
    uint64_t s = 0;
    for (size_t k = threadIdx.x; k < nb; k += kBlock) s += sums[k];
    uint64_t all;
    (void)block_inclusive_scan(s, &all);
    if (threadIdx.x == 0) *out = all;
}

// ---------------------------------------------------------------------------------------------
// message passing over few triangles: everything by one workgroup
// ---------------------------------------------------------------------------------------------
// The edges that lie in a triangle get dense numbers from a hash table in LDS (any order will do: the number is only a
// place for the share), every edge's slots are put in ascending order of their triangles by comparing, and the
// iterations run between barriers with the triangles' costs in registers.  The arithmetic and the order of every sum are
// those of k_triangle_update and k_edge_update.
// One workgroup bound by LDS latency and barriers: 3 launches and one wait for a whole round's separation and message
// passing instead of some fifty launches and five waits, which is what such a round was (150 to 220 us with a handful
// of triangles).
constexpr int kFewThreads = 1024;
constexpr int kFewTriangles = 2048;
constexpr int kFewPer = kFewTriangles / kFewThreads;           // triangles per thread
constexpr int kFewSlots = 3 * kFewTriangles;
constexpr int kFewRuns = kFewSlots / kFewThreads;              // runs of slots per thread, at most
constexpr int kFewTable = 8192, kFewEntries = kFewTable / kFewThreads;
constexpr uint32_t kNoEdge = 0xffffffffu;
static_assert(kFewSlots < kFewTable && kFewSlots < (1 << 16) && 4 * kFewTriangles <= (1 << 16), "the table keeps room; 16-bit places and slots");
struct FewShared {
    union {
        struct { uint32_t edge[kFewTable], count[kFewTable]; } table;                   // then: number of the edge, start of its slots
        struct { float share[kFewSlots], msg[4 * kFewTriangles]; } pass;
    };
    uint64_t key[kFewTriangles];       // (u,v) << 32 | (u,w), as places in the edge list
    uint32_t act_edge[kFewSlots];
    uint16_t start[kFewSlots + 1];
    uint16_t arrived[kFewSlots], slot[kFewSlots];       // 4 * triangle + which: as they came, in order
    uint32_t wave[kFewThreads / 64];
};

// counter (optional): the number of triangles, which n_triangles is otherwise.  ct (optional) gets their costs in the end.
// mail[1]: number of triangles, mail[2]: *signs (optional), mail[3]: *flag (optional).
// Nothing is done for more than kFewTriangles.
__global__ __launch_bounds__(kFewThreads) void k_messages_few(const uint32_t *list, const uint32_t *counter, uint32_t n_triangles, const uint64_t *signs,
                                                              int iters, float *ce, float *ct, const uint32_t *flag, uint64_t *mail, uint64_t seq)
{
    __shared__ FewShared S;
    const int tid = (int)threadIdx.x, lane = lane_id(), w = tid >> 6;
    const uint32_t T = counter ? *counter : n_triangles;
    if (T > 0 && T <= (uint32_t)kFewTriangles) {      // uniform
        uint32_t e[kFewPer][3];
        uint32_t h[kFewPer][3];      // place in the table | arrival << 16
        for (int k = tid; k < kFewTable; k += kFewThreads) { S.table.edge[k] = kNoEdge; S.table.count[k] = 0; }
#pragma unroll
        for (int q = 0; q < kFewPer; ++q) {
            const uint32_t t = (uint32_t)(tid + q * kFewThreads);
#pragma unroll
            for (int k = 0; k < 3; ++k) { e[q][k] = t < T ? list[3 * t + k] : kNoEdge; h[q][k] = 0; }
            if (t < T) S.key[t] = (uint64_t)e[q][0] << 32 | e[q][1];
        }
        __syncthreads();
#pragma unroll
        for (int q = 0; q < kFewPer; ++q)
            if ((uint32_t)(tid + q * kFewThreads) < T) {
#pragma unroll
                for (int k = 0; k < 3; ++k) {
                    uint32_t x = (e[q][k] * 0x9E3779B1u) >> (32 - __builtin_ctz(kFewTable));
                    for (;;) {      // a quarter of the table stays empty: the walk ends
                        const uint32_t old = atomicCAS(&S.table.edge[x], kNoEdge, e[q][k]);
                        if (old == kNoEdge || old == e[q][k]) break;
                        x = (x + 1) & (kFewTable - 1);
                    }
                    h[q][k] = x | atomicAdd(&S.table.count[x], 1u) << 16;
                }
            }
        __syncthreads();
        // numbers for the edges, places for their slots: one scan over the table with both in a word
        uint32_t key[kFewEntries], cnt[kFewEntries], mine = 0;
#pragma unroll
        for (int k = 0; k < kFewEntries; ++k) {
            key[k] = S.table.edge[tid * kFewEntries + k];
            cnt[k] = S.table.count[tid * kFewEntries + k];
            mine += cnt[k] ? cnt[k] | 1u << 16 : 0u;
        }
        const uint32_t inc = wave_inclusive_scan(mine);
        if (lane == 63) S.wave[w] = inc;
        __syncthreads();
        uint32_t run = inc - mine, na = 0;
#pragma unroll
        for (int k = 0; k < kFewThreads / 64; ++k) {
            const uint32_t x = S.wave[k];
            run += k < w ? x : 0u;
            na += x >> 16;
        }
#pragma unroll
        for (int k = 0; k < kFewEntries; ++k)
            if (cnt[k]) {
                const uint32_t a = run >> 16;
                S.table.edge[tid * kFewEntries + k] = a;
                S.table.count[tid * kFewEntries + k] = run & 0xffffu;
                S.act_edge[a] = key[k];
                S.start[a] = (uint16_t)run;
                run += cnt[k] | 1u << 16;
            }
        if (tid == 0) S.start[na] = (uint16_t)(3u * T);
        __syncthreads();
#pragma unroll
        for (int q = 0; q < kFewPer; ++q) {
            const uint32_t t = (uint32_t)(tid + q * kFewThreads);
            if (t < T) {
#pragma unroll
                for (int k = 0; k < 3; ++k) {
                    const uint32_t x = h[q][k] & 0xffffu, at = S.table.count[x] + (h[q][k] >> 16);
                    e[q][k] = S.table.edge[x];      // from here on: the edge's number
                    S.arrived[at] = (uint16_t)(4u * t + (uint32_t)k);
                }
            }
        }
        __syncthreads();
#pragma unroll
        for (int q = 0; q < kFewPer; ++q) {
            const uint32_t t = (uint32_t)(tid + q * kFewThreads);
            if (t < T) {
                const uint64_t self = S.key[t];
#pragma unroll
                for (int k = 0; k < 3; ++k) {
                    const uint32_t s0 = S.start[e[q][k]], s1 = S.start[e[q][k] + 1];
                    uint32_t at = s0;
                    for (uint32_t p = s0; p < s1; ++p) at += S.key[S.arrived[p] >> 2] < self ? 1u : 0u;
                    S.slot[at] = (uint16_t)(4u * t + (uint32_t)k);
                }
            }
        }
        uint32_t edge[kFewRuns], first[kFewRuns], len[kFewRuns];
#pragma unroll
        for (int r = 0; r < kFewRuns; ++r) {
            const uint32_t a = (uint32_t)(tid + r * kFewThreads);
            edge[r] = 0; first[r] = 0; len[r] = 0;
            if (a < na) {
                edge[r] = S.act_edge[a];
                first[r] = S.start[a];
                len[r] = S.start[a + 1] - first[r];
                S.pass.share[a] = ce[edge[r]] / (float)len[r];      // the table is no longer looked at
            }
        }
        __syncthreads();
        float a[kFewPer] = {}, b[kFewPer] = {}, c[kFewPer] = {};
        for (int it = 1; it <= iters; ++it) {
#pragma unroll
            for (int q = 0; q < kFewPer; ++q) {
                const uint32_t t = (uint32_t)(tid + q * kFewThreads);
                if (t < T) {
                    a[q] = a[q] + S.pass.share[e[q][0]]; b[q] = b[q] + S.pass.share[e[q][1]]; c[q] = c[q] + S.pass.share[e[q][2]];
                    float oa, ob, oc;
                    triangle_to_edges(a[q], b[q], c[q], oa, ob, oc);
                    S.pass.msg[4 * t] = oa; S.pass.msg[4 * t + 1] = ob; S.pass.msg[4 * t + 2] = oc;
                }
            }
            __syncthreads();
#pragma unroll
            for (int r = 0; r < kFewRuns; ++r)
                if (len[r]) {
                    float acc = 0.0f;
                    for (uint32_t p = 0; p < len[r]; ++p) acc = acc + S.pass.msg[S.slot[first[r] + p]];
                    if (it == iters) ce[edge[r]] = acc;
                    else S.pass.share[tid + r * kFewThreads] = acc / (float)len[r];
                }
            __syncthreads();
        }
        if (ct) {      // uniform
#pragma unroll
            for (int q = 0; q < kFewPer; ++q) {
                const uint32_t t = (uint32_t)(tid + q * kFewThreads);
                if (t < T) { ct[3 * t] = a[q]; ct[3 * t + 1] = b[q]; ct[3 * t + 2] = c[q]; }
            }
        }
    }
    __syncthreads();
    if (tid == 0) { mail[1] = (uint64_t)T; mail[2] = signs ? *signs : 0ull; mail[3] = flag ? (uint64_t)*flag : 0ull; }
    mail_send(mail, seq);
}

// Tiles of 256 edges: long lists.  With long rows (seven edges to a node and more) 64 fill the chip sooner and keep a
// workgroup's tries few: 4.2e7 edges 1090 us with 256 and 1970 with 64, 2.2e6 edges with sixteen to a node 227 and 194,
// 9.6e5 with six to a node 71 and 74.
inline bool wide_tiles(size_t m, size_t n) { return m >= (size_t(1) << 22) || (m >= (size_t(1) << 18) && m <= 6 * n); }
inline unsigned triangle_tiles(size_t m, size_t n) { return grid_for(m, wide_tiles(m, n) ? kBlock : 64); }

template <int MODE>
rama_status run_triangles(Ctx &ctx, const char *name, const TriangleGraph &tg, size_t n, uint32_t *list, uint32_t cap, uint32_t *counter,
                          uint64_t *sums, const uint64_t *offs, uint32_t *slots, double bytes)
{
    const uint32_t nb = triangle_tiles(tg.m, n);
    ProfScope ps_(ctx, name, bytes);
    if (wide_tiles(tg.m, n)) k_triangles<MODE, kBlock><<<xcd_grid(nb), kBlock, 0, ctx.stream>>>(tg, nb, list, cap, counter, sums, offs, slots);
    else k_triangles<MODE, 64><<<xcd_grid(nb), kBlock, 0, ctx.stream>>>(tg, nb, list, cap, counter, sums, offs, slots);
    LAUNCH_TRY(ctx, "triangles");
    return RAMA_OK;
}

// sums: sign counts per tile of kScanTile edges
rama_status total_signs(Ctx &ctx, const uint64_t *sums, size_t m, uint64_t *out)
{
    const size_t nb = grid_for(m, kScanTile);
    {
        ProfScope ps_(ctx, "k_total_signs", (double)(nb * 8));
        k_total_signs<<<1, kBlock, 0, ctx.stream>>>(sums, nb, out);
    }
    LAUNCH_TRY(ctx, "total_signs");
    return RAMA_OK;
}

}  // namespace

rama_status triangles_few(Ctx &ctx, Graph &g, const int32_t *rowptr, int k_iters, TriangleCounts &out, bool *done, const std::function<void()> &separated)
{
    *done = false;
    if (!g.sign_sums.get()) return RAMA_OK;
    Buf<uint32_t> list, counter;
    Buf<uint64_t> signs;
    RAMA_TRY(list.alloc(ctx, (size_t)kFewSlots));
    RAMA_TRY(zeroed<uint32_t>(ctx, (size_t)kListWords, counter));
    RAMA_TRY(signs.alloc(ctx, 1));
    RAMA_TRY(total_signs(ctx, g.sign_sums.get(), (size_t)g.m, signs.get()));
    RAMA_TRY(run_triangles<kTriList>(ctx, "k_triangles", TriangleGraph{rowptr, g.i.get(), g.j.get(), g.c.get(), (size_t)g.m, signs.get()}, (size_t)g.n,
                                     list.get(), (uint32_t)kFewTriangles, counter.get(), nullptr, nullptr, nullptr, (double)g.m * 12 + (double)g.n * 4));
    separated();
    const uint64_t seq = ++ctx.mail_seq;
    {
        ProfScope ps_(ctx, "k_messages_few", (double)(kFewSlots * 4));
        k_messages_few<<<1, kFewThreads, 0, ctx.stream>>>(list.get(), counter.get(), 0, signs.get(), k_iters, g.c.get(), nullptr, nullptr, mailbox(ctx), seq);
    }
    LAUNCH_TRY(ctx, "messages_few");
    RAMA_TRY(wait_mail(ctx, seq));
    const volatile uint64_t *mail = mailbox(ctx);
    const uint64_t found = mail[1], by_sign = mail[2];
    if (found > (uint64_t)kFewTriangles) return RAMA_OK;
    out.triangles = (int64_t)found;
    out.attractive = (int64_t)(uint32_t)by_sign; out.repulsive = (int64_t)(by_sign >> 32);
    if (found) g.sign_sums.reset();      // the costs are new
    *done = true;
    return RAMA_OK;
}

bool messages_fit(size_t T) { return T > 0 && T <= (size_t)kFewTriangles; }
rama_status messages_few(Ctx &ctx, const uint32_t *edges, size_t T, int k_iters, float *ce, float *ct, const uint32_t *flag, bool *raised)
{
    const uint64_t seq = ++ctx.mail_seq;
    {
        ProfScope ps_(ctx, "k_messages_few", (double)(T * 24));
        k_messages_few<<<1, kFewThreads, 0, ctx.stream>>>(edges, nullptr, (uint32_t)T, nullptr, k_iters, ce, ct, flag, mailbox(ctx), seq);
    }
    LAUNCH_TRY(ctx, "messages_few");
    RAMA_TRY(wait_mail(ctx, seq));
    *raised = ((const volatile uint64_t *)mailbox(ctx))[3] != 0;
    return RAMA_OK;
}

rama_status triangles_list(Ctx &ctx, const Graph &g, const int32_t *rowptr, Buf<uint32_t> &slots, TriangleCounts &out)
{
    const size_t m = (size_t)g.m, n = (size_t)g.n;
    const unsigned nb = triangle_tiles(m, n), nb_signs = grid_for(m, kScanTile);
    Buf<uint64_t> sums, offs, signs;      // offs: nb places, the number of triangles, the sign counts
    RAMA_TRY(sums.alloc(ctx, nb));
    RAMA_TRY(offs.alloc(ctx, (size_t)nb + 2));
    const TriangleGraph tg{rowptr, g.i.get(), g.j.get(), g.c.get(), m, offs.get() + nb + 1};
    Buf<uint32_t> kept;
    RAMA_TRY(kept.alloc(ctx, 3 * (size_t)nb * (size_t)tri_room(wide_tiles(m, n) ? kBlock : 64)));
    if (!g.sign_sums.get()) {
        RAMA_TRY(signs.alloc(ctx, nb_signs));
        ProfScope ps_(ctx, kernel_name<SignFlags>("k_scan_reduce"), (double)(m * 4));
        k_scan_reduce<uint64_t, SignFlags><<<nb_signs, kBlock, 0, ctx.stream>>>(SignFlags{g.c.get()}, signs.get(), m, (uint64_t *)nullptr, (uint32_t *)nullptr,
                                                                               (uint64_t *)nullptr, 0, (const uint64_t *)nullptr, 0);
    }
    LAUNCH_TRY(ctx, "scan_reduce");
    RAMA_TRY(total_signs(ctx, g.sign_sums.get() ? g.sign_sums.get() : signs.get(), m, offs.get() + nb + 1));
    RAMA_TRY(run_triangles<kTriCount>(ctx, "k_count_cycles<3>", tg, n, kept.get(), 0, nullptr, sums.get(), nullptr, nullptr,
                                      (double)m * 12 + (double)n * 4 + (double)nb * 12));
    uint64_t back[2];
    if (nb <= kScanMidMax) {
        const uint64_t seq = ++ctx.mail_seq;
        {
            ProfScope ps_(ctx, "k_scan_mid", (double)((size_t)nb * 16));
            k_scan_mid<uint64_t><<<1, kBlock, 0, ctx.stream>>>(sums.get(), offs.get(), nb, mailbox(ctx), seq, offs.get() + nb + 1, 1);
        }
        LAUNCH_TRY(ctx, "scan_mid");
        RAMA_TRY(wait_mail(ctx, seq));
        const volatile uint64_t *mail = mailbox(ctx);
        back[0] = mail[1]; back[1] = mail[2];
    } else {
        RAMA_TRY((exclusive_scan<uint64_t, PtrInput<uint64_t>>(ctx, PtrInput<uint64_t>{sums.get()}, offs.get(), nb)));
        RAMA_TRY(read_back(ctx, back, offs.get() + nb, sizeof back));
    }
    out.attractive = (int64_t)(uint32_t)back[1]; out.repulsive = (int64_t)(back[1] >> 32);
    out.triangles = 0;
    RAMA_TRY(adjacency_fits(ctx, (uint64_t)out.attractive));
    RAMA_TRY(list_fits(ctx, 0, (int64_t)(back[0] < (uint64_t(1) << 31) ? back[0] : (uint64_t(1) << 31))));
    out.triangles = (int64_t)back[0];
    if (out.triangles == 0) return RAMA_OK;
    RAMA_TRY(slots.alloc(ctx, 3 * (size_t)back[0]));
    return run_triangles<kTriFill>(ctx, "k_fill_cycles<3>", tg, n, kept.get(), 0, nullptr, nullptr, offs.get(), slots.get(),
                                   (double)nb * 20 + (double)back[0] * 24);
}

}  // namespace rama
