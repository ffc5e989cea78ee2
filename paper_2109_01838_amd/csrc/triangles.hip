// Separation and message passing of a round that separates triangles only (every round behind the first, by default).
//
// A conflicted triangle u < v < w has exactly one repulsive edge and two attractive ones (paper Sec. 3.2.2).  On the
// canonical list its edges (u,v), (u,w), (v,w) stand in this order, and ascending pairs of places (of (u,v), of (u,w)) are
// ascending triples (u,v,w).  So the triangles come out of the list itself: for every edge (u,v), the common entries of
// the rest of row u and of row v, with the signs looked at on the way -- no attractive adjacency (which takes a sort of
// the lower neighbours), no list of cycles, no keys and no sort to put the triangles in order.  The work is the sum over
// all edges of the shorter of the two stretches, of which a dense graph has many that can be no triangle's: a survey tells,
// and such a round goes through the lists of cycles (see kDenseTries).
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
    const uint64_t *survey;     // see k_survey
    uint64_t most_tries;        // of its sample
};

// What is tried for edge e: the entries of the shorter of two stretches, [a0,a1) the rest of its row and [b0,b1) the row of
// its second node.
struct EdgeTries {
    int32_t a0, a1, b0, b1;
    float c;
    bool walk_v;
    uint32_t n;
};
__device__ __forceinline__ EdgeTries edge_tries(const TriangleGraph &g, size_t e)
{
    EdgeTries t;
    const int32_t v = g.j[e];
    t.c = g.c[e];
    t.a0 = (int32_t)e + 1; t.a1 = g.rowptr[g.i[e] + 1]; t.b0 = g.rowptr[v]; t.b1 = g.rowptr[v + 1];
    t.walk_v = t.b1 - t.b0 < t.a1 - t.a0;
    t.n = t.c > 0.0f || t.c < 0.0f ? (uint32_t)(t.walk_v ? t.b1 - t.b0 : t.a1 - t.a0) : 0u;
    return t;
}

// In front of the search, survey[0]: attractive edges | repulsive edges << 32, survey[1]: tries of a sample of the edges, 64 in
// a row at up to kSurveySpots places spread evenly.  The search leaves at once when there is no edge of one sign, and when
// its tries are many (see kDenseTries).  3.8 us in front of a round: one chain edge -> row bounds -> sum.
constexpr int kSurveyThreads = 1024, kSurveyGroups = 64, kSurveySpots = kSurveyGroups * (kSurveyThreads / 64);
constexpr size_t survey_sample(size_t m) { return m < (size_t)kSurveySpots * 64 ? m : (size_t)kSurveySpots * 64; }
// sums: n_sums packed sign counts; survey[1] is zero on entry
__global__ __launch_bounds__(kSurveyThreads) void k_survey(TriangleGraph g, const uint64_t *sums, unsigned n_sums, uint64_t *survey)
{
    __shared__ unsigned long long s_all;
    const int tid = (int)threadIdx.x;
    if (tid == 0) s_all = 0;
    __syncthreads();
    uint64_t x = 0;
    if (blockIdx.x == kSurveyGroups) {
        for (unsigned k = (unsigned)tid; k < n_sums; k += kSurveyThreads) x += sums[k];
    } else {
        const size_t spot = (size_t)blockIdx.x * (kSurveyThreads / 64) + (size_t)(tid >> 6);
        const size_t first = g.m <= (size_t)kSurveySpots * 64 ? spot * 64 : spot * g.m / kSurveySpots;
        const size_t e = first + (size_t)lane_id();
        if (e < g.m) x = edge_tries(g, e).n;
    }
    x = wave_sum(x);
    if (lane_id() == 0 && x) atomicAdd(&s_all, (unsigned long long)x);
    __syncthreads();
    if (tid == 0) {
        if (blockIdx.x == kSurveyGroups) survey[0] = s_all;
        else if (s_all) atomicAdd((unsigned long long *)&survey[1], s_all);
    }
}
__host__ __device__ inline bool both_signs(uint64_t signs) { return (uint32_t)signs != 0u && (signs >> 32) != 0u; }
__device__ __forceinline__ bool not_searched(const TriangleGraph &g) { return !both_signs(g.survey[0]) || g.survey[1] > g.most_tries; }

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
        if (not_searched(g)) {
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
            const EdgeTries t = edge_tries(g, e);
            tries = t.n;
            S.scan[tid] = t.walk_v ? t.b0 : t.a0;
            S.lo[tid] = t.walk_v ? t.a0 : t.b0;
            S.hi[tid] = t.walk_v ? t.a1 : t.b1;
            S.kind[tid] = (uint8_t)((t.c < 0.0f ? 1 : 0) | (t.walk_v ? 2 : 0));
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
// Slots of an edge in more triangles than this are not compared with each other but put in order by a bit per triangle and the
// counts of the bits in front, which takes triangles that come in ascending order.  Message passing with one iteration, us,
// all compared | as it is: one edge in 2048 triangles 505 | 194 (by the kernels for any number 260), in 512 194 | 154, in 256
// 150 either way.
constexpr uint32_t kLongRun = 256;
constexpr int kLongRuns = kFewSlots / ((int)kLongRun + 1), kLongWords = kFewTriangles / 32;
static_assert(kLongWords == 64, "a wave adds up the words of a run");
static_assert(kFewSlots < kFewTable && kFewSlots < (1 << 16) && 4 * kFewTriangles <= (1 << 16), "the table keeps room; 16-bit places and slots");
struct FewShared {
    union {
        struct { uint32_t edge[kFewTable], count[kFewTable]; } table;                   // then: number of the edge, start of its slots
        struct { float share[kFewSlots], msg[4 * kFewTriangles]; } pass;
        struct { float share[kFewSlots]; uint32_t bits[kLongRuns][kLongWords], before[kLongRuns][kLongWords]; } runs;      // before the first messages
    };
    uint64_t key[kFewTriangles];       // (u,v) << 32 | (u,w), as places in the edge list
    uint32_t act_edge[kFewSlots];
    uint16_t start[kFewSlots + 1];
    uint16_t arrived[kFewSlots], slot[kFewSlots];       // 4 * triangle + which: as they came, in order
    uint32_t wave[kFewThreads / 64], n_long;
};

// counter (optional): the number of triangles, which come in any order; otherwise there are n_triangles, ascending.  ct (optional)
// gets their costs in the end.
// mail[1]: number of triangles, mail[2], mail[4]: the survey (optional), mail[3]: *flag (optional).
// Nothing is done for more than kFewTriangles, nor for triangles in any order with a run longer than kLongRun (mail[1] is then
// kFewTriangles + 1).
__global__ __launch_bounds__(kFewThreads) void k_messages_few(const uint32_t *list, const uint32_t *counter, uint32_t n_triangles, const uint64_t *survey,
                                                              int iters, float *ce, float *ct, const uint32_t *flag, MailWord *mail, uint64_t seq)
{
    __shared__ FewShared S;
    const int tid = (int)threadIdx.x, lane = lane_id(), w = tid >> 6;
    const uint32_t T = counter ? *counter : n_triangles;
    bool left = false;      // uniform
    if (tid == 0) S.n_long = 0;
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
        uint32_t edge[kFewRuns], first[kFewRuns], len[kFewRuns], longest = 0;
#pragma unroll
        for (int r = 0; r < kFewRuns; ++r) {
            const uint32_t a = (uint32_t)(tid + r * kFewThreads);
            edge[r] = 0; first[r] = 0; len[r] = 0;
            if (a < na) {
                edge[r] = S.act_edge[a];
                first[r] = S.start[a];
                len[r] = S.start[a + 1] - first[r];
                longest = max(longest, len[r]);
            }
        }
        const bool any_long = __syncthreads_or(longest > kLongRun) != 0;      // behind it the table is no longer looked at
        left = any_long && counter;
        if (any_long && !left) {
#pragma unroll
            for (int r = 0; r < kFewRuns; ++r)
                if (len[r] > kLongRun) S.arrived[first[r]] = (uint16_t)atomicAdd(&S.n_long, 1u);      // the run's number
            for (int k = tid; k < kLongRuns * kLongWords; k += kFewThreads) (&S.runs.bits[0][0])[k] = 0;
            __syncthreads();
#pragma unroll
            for (int q = 0; q < kFewPer; ++q) {
                const uint32_t t = (uint32_t)(tid + q * kFewThreads);
                if (t < T) {
#pragma unroll
                    for (int k = 0; k < 3; ++k) {
                        const uint32_t s0 = S.start[e[q][k]];
                        if (S.start[e[q][k] + 1] - s0 > kLongRun) atomicOr(&S.runs.bits[S.arrived[s0]][t >> 5], 1u << (t & 31u));
                    }
                }
            }
            __syncthreads();
            for (uint32_t r = (uint32_t)w; r < S.n_long; r += kFewThreads / 64) {
                const uint32_t n = (uint32_t)__popc(S.runs.bits[r][lane]);
                S.runs.before[r][lane] = wave_inclusive_scan(n) - n;
            }
            __syncthreads();
        }
#pragma unroll
        for (int q = 0; q < kFewPer; ++q) {
            const uint32_t t = (uint32_t)(tid + q * kFewThreads);
            if (t < T && !left) {
                const uint64_t self = S.key[t];
#pragma unroll
                for (int k = 0; k < 3; ++k) {
                    const uint32_t s0 = S.start[e[q][k]], s1 = S.start[e[q][k] + 1];
                    uint32_t at = s0;
                    if (s1 - s0 > kLongRun) {
                        const uint32_t r = S.arrived[s0];
                        at += S.runs.before[r][t >> 5] + (uint32_t)__popc(S.runs.bits[r][t >> 5] & ((1u << (t & 31u)) - 1u));
                    } else {
                        for (uint32_t p = s0; p < s1; ++p) at += S.key[S.arrived[p] >> 2] < self ? 1u : 0u;
                    }
                    S.slot[at] = (uint16_t)(4u * t + (uint32_t)k);
                }
            }
        }
#pragma unroll
        for (int r = 0; r < kFewRuns; ++r)
            if (len[r]) S.pass.share[tid + r * kFewThreads] = ce[edge[r]] / (float)len[r];
        __syncthreads();
        float a[kFewPer] = {}, b[kFewPer] = {}, c[kFewPer] = {};
        for (int it = 1; it <= iters && !left; ++it) {
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
    if (tid == 0) {
        mail_put(mail + 1, left ? (uint64_t)kFewTriangles + 1 : (uint64_t)T);
        mail_put(mail + 2, survey ? survey[0] : (uint64_t)0);
        mail_put(mail + 3, flag ? (uint64_t)*flag : (uint64_t)0);
        mail_put(mail + 4, survey ? survey[1] : (uint64_t)0);
    }
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

// With more tries per edge than kDenseTries, and kManyTries in all, the lists of cycles are the better way: their search starts
// from the repulsive edges and intersects attractive neighbours only, which on dense graphs is a small part of the tries.
// Separation and messages of a round in us, edge list | cycle lists (survey and this search's empty launch included), by
// tries per edge.  Random graphs: 5.4 (10^6 edges) 165 | 338, 7.5 (7.6e5) 121 | 334, 10.5 (9.5e5) 299 | 324, 13.1 (9.0e5)
// 304 | 340, 16.0 (8.4e5) 342 | 379, 16.1 (8.4e6) 1913 | 1311, 20 (9.3e5) 395 | 393, 30 (8.3e6) 2970 | 1862, 45 (9.6e5) 698 |
// 536, 133 (10^6) 3553 | 1644.  Where rows lie close together the line could stand higher: long-range grid 13.4 (10^6) 222 |
// 350, windows 11.4 (2.1e6) 1703 | 1858, 19 (3.6e6) 4500 | 5001, 48 (1.9e6) 596 | 559.  Few tries in all: 13 (6.8e4 edges) 44 |
// 136, 23 (2.3e5) 64 | 112, 59 (1.7e4) 107 | 138.
constexpr uint64_t kDenseTries = 16, kManyTries = uint64_t(1) << 21;
// the same for the sample of m edges
constexpr uint64_t most_tries(size_t m)
{
    const uint64_t dense = kDenseTries * (uint64_t)survey_sample(m), many = m ? kManyTries * (uint64_t)survey_sample(m) / m : 0;
    return dense > many ? dense : many;
}
static_assert(most_tries(0) == 0 && most_tries(1) == kManyTries && most_tries(survey_sample(~size_t(0))) == kManyTries, "short lists");
static_assert(most_tries(size_t(1) << 18) == kDenseTries << 16 && most_tries((size_t(1) << 31) - 1) == kDenseTries << 16, "long lists");

rama_status take_survey(Ctx &ctx, TriangleCounts &out, uint64_t signs, uint64_t tries, const TriangleSurvey &survey)
{
    out.attractive = (int64_t)(uint32_t)signs; out.repulsive = (int64_t)(signs >> 32);
    out.dense = both_signs(signs) && tries > survey.most_tries;
    return adjacency_fits(ctx, (uint64_t)out.attractive, (uint64_t)out.repulsive);
}
TriangleGraph triangle_graph(const Graph &g, const int32_t *rowptr, const TriangleSurvey &survey)
{
    return {rowptr, g.i.get(), g.j.get(), g.c.get(), (size_t)g.m, survey.words.get(), survey.most_tries};
}

}  // namespace

rama_status triangle_survey(Ctx &ctx, const Graph &g, const int32_t *rowptr, bool any, TriangleSurvey &survey)
{
    const size_t m = (size_t)g.m;
    const unsigned n_sums = grid_for(m, kScanTile);
    survey.most_tries = any ? ~uint64_t(0) : most_tries(m);
    RAMA_TRY(zeroed<uint64_t>(ctx, 2, survey.words));
    Buf<uint64_t> signs;
    if (!g.sign_sums.get()) {
        RAMA_TRY(signs.alloc(ctx, n_sums));
        ProfScope ps_(ctx, kernel_name<SignFlags>("k_scan_reduce"), (double)(m * 4));
        k_scan_reduce<uint64_t, SignFlags><<<n_sums, kBlock, 0, ctx.stream>>>(SignFlags{g.c.get()}, signs.get(), m, (uint64_t *)nullptr, (uint32_t *)nullptr,
                                                                             (MailWord *)nullptr, 0, (const uint64_t *)nullptr, 0);
    }
    LAUNCH_TRY(ctx, "scan_reduce");
    {
        ProfScope ps_(ctx, "k_survey", (double)((size_t)n_sums * 8 + survey_sample(m) * 12));
        k_survey<<<kSurveyGroups + 1, kSurveyThreads, 0, ctx.stream>>>(triangle_graph(g, rowptr, survey), g.sign_sums.get() ? g.sign_sums.get() : signs.get(),
                                                                    n_sums, survey.words.get());
    }
    LAUNCH_TRY(ctx, "survey");
    return RAMA_OK;
}

rama_status triangles_few(Ctx &ctx, Graph &g, const int32_t *rowptr, const TriangleSurvey &survey, int k_iters, TriangleCounts &out, bool *done,
                          const std::function<void()> &separated)
{
    *done = false;
    Buf<uint32_t> list, counter;
    RAMA_TRY(list.alloc(ctx, (size_t)kFewSlots));
    RAMA_TRY(zeroed<uint32_t>(ctx, (size_t)kListWords, counter));
    RAMA_TRY(run_triangles<kTriList>(ctx, "k_triangles<list>", triangle_graph(g, rowptr, survey), (size_t)g.n, list.get(), (uint32_t)kFewTriangles, counter.get(),
                                     nullptr, nullptr, nullptr, (double)g.m * 12 + (double)g.n * 4));
    separated();
    const uint64_t seq = ++ctx.mail_seq;
    {
        ProfScope ps_(ctx, "k_messages_few", (double)(kFewSlots * 4));
        k_messages_few<<<1, kFewThreads, 0, ctx.stream>>>(list.get(), counter.get(), 0, survey.words.get(), k_iters, g.c.get(), nullptr, nullptr, mailbox(ctx), seq);
    }
    LAUNCH_TRY(ctx, "messages_few");
    RAMA_TRY(wait_mail(ctx, seq));
    const volatile uint64_t *mail = mail_words(ctx);
    const uint64_t found = mail[1];
    RAMA_TRY(take_survey(ctx, out, mail[2], mail[4], survey));
    if (out.dense || found > (uint64_t)kFewTriangles) return RAMA_OK;
    out.triangles = (int64_t)found;
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
    *raised = mail_words(ctx)[3] != 0;
    return RAMA_OK;
}

rama_status triangles_list(Ctx &ctx, const Graph &g, const int32_t *rowptr, const TriangleSurvey &survey, Buf<uint32_t> &slots, TriangleCounts &out)
{
    const size_t m = (size_t)g.m, n = (size_t)g.n;
    const unsigned nb = triangle_tiles(m, n);
    const TriangleGraph tg = triangle_graph(g, rowptr, survey);
    Buf<uint64_t> sums, offs;      // offs: nb places, the number of triangles
    RAMA_TRY(sums.alloc(ctx, nb));
    RAMA_TRY(offs.alloc(ctx, (size_t)nb + 1));
    Buf<uint32_t> kept;
    RAMA_TRY(kept.alloc(ctx, 3 * (size_t)nb * (size_t)tri_room(wide_tiles(m, n) ? kBlock : 64)));
    RAMA_TRY(run_triangles<kTriCount>(ctx, "k_triangles<count>", tg, n, kept.get(), 0, nullptr, sums.get(), nullptr, nullptr,
                                      (double)m * 12 + (double)n * 4 + (double)nb * 12));
    uint64_t back[3];
    if (nb <= kScanMidMax) {
        const uint64_t seq = ++ctx.mail_seq;
        {
            ProfScope ps_(ctx, "k_scan_mid", (double)((size_t)nb * 16));
            k_scan_mid<uint64_t><<<1, kBlock, 0, ctx.stream>>>(sums.get(), offs.get(), nb, mailbox(ctx), seq, survey.words.get(), 2);
        }
        LAUNCH_TRY(ctx, "scan_mid");
        RAMA_TRY(wait_mail(ctx, seq));
        const volatile uint64_t *mail = mail_words(ctx);
        for (int k = 0; k < 3; ++k) back[k] = mail[1 + k];
    } else {
        RAMA_TRY((exclusive_scan<uint64_t, PtrInput<uint64_t>>(ctx, PtrInput<uint64_t>{sums.get()}, offs.get(), nb)));
        RAMA_TRY(read_back(ctx, back, offs.get() + nb, 8, survey.words.get(), 16));
    }
    out.triangles = 0;
    RAMA_TRY(take_survey(ctx, out, back[1], back[2], survey));
    if (out.dense) return RAMA_OK;
    RAMA_TRY(list_fits(ctx, 0, (int64_t)(back[0] < (uint64_t(1) << 31) ? back[0] : (uint64_t(1) << 31))));
    out.triangles = (int64_t)back[0];
    if (out.triangles == 0) return RAMA_OK;
    RAMA_TRY(slots.alloc(ctx, 3 * (size_t)back[0]));
    return run_triangles<kTriFill>(ctx, "k_triangles<fill>", tg, n, kept.get(), 0, nullptr, nullptr, offs.get(), slots.get(),
                                   (double)nb * 20 + (double)back[0] * 24);
}

}  // namespace rama
