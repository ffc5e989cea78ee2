// Step a0: problem statement -> canonical device graph (paper Sec. 3: graph and cost vector;
// Lemma 1(b): parallel edges carry the sum of their costs).
#include "prim.h"
#include <algorithm>
#include <vector>

namespace rama {

namespace {

// flags[0]: endpoint out of range or non-finite cost; flags[1]: list is not canonical;
// flags[2]: largest |i-j| of a valid edge; flags[3]: number of places where the oriented pair (min, max) is smaller
// than the one before it (few of them: the list is a handful of sorted runs, e.g. one per grid direction); flags[4]: there is
// a self-loop or a pair equal to the one before it; flags[5]: there is a positive cost; flags[6..]: the first kMaxRuns - 1 of the
// places counted in flags[3], in any order.  A workgroup takes one tile of the scan over NotLoop (kScanTile edges) and leaves the number of edges
// that are no self-loops in tile_sums, so that scan needs no counting pass.
constexpr int kMaxRuns = 16;
constexpr int kFirstRun = 6, kFlagWords = kFirstRun + kMaxRuns - 1;
__global__ __launch_bounds__(kBlock) void k_validate(int32_t n, size_t m, const int32_t *i, const int32_t *j,
                                                     const float *c, int32_t *flags, uint32_t *tile_sums)
{
    const size_t base = (size_t)blockIdx.x * kScanTile + threadIdx.x;
    uint32_t diff = 0, kept = 0, down = 0;      // down: a bit per place of this thread
    bool plain = true;
    bool ordered = true, valid = true;
    // all edges are read at once, and those in front of a wave's stretches; the others' neighbours come from the lane in front
    int32_t ea[kScanItems], eb[kScanItems], ep[kScanItems], eq[kScanItems];
    float ew[kScanItems];
#pragma unroll
    for (int q = 0; q < kScanItems; ++q) {
        const size_t e = base + (size_t)q * kBlock, at = e < m ? e : m - 1;
        const size_t first = e - (size_t)lane_id(), before = first == 0 ? 0 : (first < m ? first : m) - 1;      // uniform in the wave
        ea[q] = i[at]; eb[q] = j[at]; ew[q] = c[at]; ep[q] = i[before]; eq[q] = j[before];
    }
#pragma unroll
    for (int q = 0; q < kScanItems; ++q) {
        const int32_t a = __shfl_up(ea[q], 1, 64), b = __shfl_up(eb[q], 1, 64);
        if (lane_id() != 0) { ep[q] = a; eq[q] = b; }
    }
#pragma unroll
    for (int q = 0; q < kScanItems; ++q) {
        const size_t e = base + (size_t)q * kBlock;
        if (e >= m) continue;
        const int32_t a = ea[q], b = eb[q];
        const float w = ew[q];
        kept += (a != b ? 1u : 0u) + (w > 0.0f ? 1u << 16 : 0u);      // the positive ones in the upper half
        bool bad = a < 0 || a >= n || b < 0 || b >= n || !(fabsf(w) <= 3.402823466e+38f);
        if (bad) {
            valid = false;
        } else {
            const uint32_t d = (uint32_t)abs(a - b);
            diff = d > diff ? d : diff;
            bool canon = a < b;
            if (e > 0) {
                const int32_t pa = ep[q], pb = eq[q];
                canon = canon && (pa < a || (pa == a && pb < b));
                const int32_t lo = min(a, b), hi = max(a, b), plo = min(pa, pb), phi = max(pa, pb);
                down |= (lo < plo || (lo == plo && hi < phi)) ? 1u << q : 0u;
                plain = plain && !(lo == plo && hi == phi);
            }
            plain = plain && a != b;
            ordered = ordered && canon;
        }
    }
    // a flag is stored once a wave and not where it is seen to be set: stores to one word are carried out one after the other
    // (2.3e6 edges in arbitrary order 91 -> 18 us)
    auto raise = [&](bool any, int32_t *flag) {
        if (__ballot(any) && lane_id() == 0 && !*(volatile int32_t *)flag) *flag = 1;
    };
    raise(!valid, &flags[0]); raise(!ordered, &flags[1]); raise(!plain, &flags[4]);
    static_assert(kScanTile < (1 << 16), "two counts in a word");
    kept = block_sum(kept);
    const uint32_t downs = block_sum((uint32_t)__popc(down));
    if (threadIdx.x == 0) {
        tile_sums[blockIdx.x] = kept & 0xffffu;
        if (kept >> 16 && !*(volatile int32_t *)&flags[5]) flags[5] = 1;
    }
    if (downs > 0 && downs < (uint32_t)kMaxRuns) {      // uniform
        for (; down; down &= down - 1) {
            const uint32_t at = atomicAdd((uint32_t *)&flags[3], 1u);
            if (at < (uint32_t)(kMaxRuns - 1)) flags[kFirstRun + at] = (int32_t)(base + (size_t)(__ffs((int)down) - 1) * kBlock);
        }
    } else if (downs && threadIdx.x == 0 && *(volatile uint32_t *)&flags[3] < (uint32_t)kMaxRuns) {
        atomicAdd((uint32_t *)&flags[3], downs);        // too many for a list of runs
    }
    block_max_into(diff, (uint32_t *)&flags[2]);
}

struct NotLoop {
    static constexpr int bytes = 8;   // bytes read per item
    static constexpr const char *tag = "NotLoop";
    const int32_t *i, *j;
    __device__ __forceinline__ uint32_t operator()(size_t e) const { return i[e] != j[e] ? 1u : 0u; }
};

// consumer of the scan over NotLoop: edge e that is no self-loop goes to place p
struct PackEdgesEmit {
    static constexpr const char *tag = "PackEdges";
    const int32_t *i, *j;
    const float *c;
    int dbits;
    uint64_t *key;
    uint32_t *val;
    struct Item { int32_t a, b; float c; };
    __device__ __forceinline__ Item load(size_t e) const { return {i[e], j[e], c[e]}; }
    __device__ __forceinline__ void operator()(size_t, uint32_t keep, uint32_t p, const Item &x) const
    {
        if (!keep) return;
        key[p] = edge_key((uint32_t)min(x.a, x.b), (uint32_t)max(x.a, x.b), dbits);
        val[p] = __float_as_uint(x.c);
    }
};

// the same as a source of the sort
struct InputEdges {
    const int32_t *i, *j;
    const float *c;
    int dbits;
    __device__ __forceinline__ uint64_t key(size_t e) const
    {
        const int32_t a = i[e], b = j[e];
        return edge_key((uint32_t)min(a, b), (uint32_t)max(a, b), dbits);
    }
    __device__ __forceinline__ bool takes_part(uint64_t k) const { return (k & ((uint64_t(1) << dbits) - 1u)) != 0u; }   // hi > lo
    __device__ __forceinline__ uint32_t value(size_t e) const { return __float_as_uint(c[e]); }
};

struct HeadFlag {
    static constexpr int bytes = 8;   // bytes read per item
    static constexpr const char *tag = "HeadFlag";
    const uint64_t *key;
    __device__ __forceinline__ uint32_t operator()(size_t e) const { return ((e == 0) | (key[e] != key[e ? e - 1 : 0])) ? 1u : 0u; }
};

// ---- a list that consists of a few sorted runs, none of which repeats a pair: one pass ---------------------------
// Grids written direction by direction.  A workgroup takes the edges of a range of nodes (as first endpoint): one stretch
// of every run.  It counts the edges per node in LDS, places them node by node, orders the few of a node by their second
// endpoint by comparing them with each other, and writes a stretch of the canonical list: every edge is read once and
// written once, where packing, merging run by run and summing equal pairs moves it five times.  A pair that occurs
// in two runs, a range with more edges than fit and a node with more than kRowMax of them raise *flag: the list is then
// canonicalised the general way.
// Bounded by LDS latency and the barriers between the steps: 0.79 ms for 9.8e7 edges of the 320^3 grid, where a copy of the
// 24 bytes per edge takes 0.45 and packing, merging and summing took 2.7; 84 us for the 1.2e7 of a 160^3 one.
constexpr int kRangeEdges = 3072, kRangeNodes = 1024, kRowMax = 64;
constexpr int kRangeItems = kRangeEdges / kBlock;
struct Runs {
    uint32_t start[kMaxRuns + 1];
    int n;
};

// bounds[t * runs + r] = first place of run r whose smaller endpoint is at least t * width
__global__ __launch_bounds__(kBlock) void k_range_bounds(Runs runs, const int32_t *i, const int32_t *j, uint32_t ranges, uint32_t width,
                                                         uint32_t *bounds)
{
    const uint32_t q = blockIdx.x * kBlock + threadIdx.x;
    if (q >= (ranges + 1) * (uint32_t)runs.n) return;
    const uint32_t t = q / (uint32_t)runs.n, r = q - t * (uint32_t)runs.n;
    uint32_t lo = 0, hi = 0;
#pragma unroll
    for (int k = 0; k < kMaxRuns; ++k)
        if (k == (int)r) { lo = runs.start[k]; hi = runs.start[k + 1]; }
    const uint64_t from = (uint64_t)t * width;      // beyond the last node for the last bound
    while (lo < hi) {
        const uint32_t mid = lo + (hi - lo) / 2;
        if ((uint64_t)(uint32_t)min(i[mid], j[mid]) < from) lo = mid + 1; else hi = mid;
    }
    bounds[q] = lo;
}

__global__ __launch_bounds__(kBlock) void k_interleave_runs(Runs runs, const int32_t *i, const int32_t *j, const float *c, uint32_t width,
                                                            const uint32_t *bounds, int32_t *io, int32_t *jo, float *co,
                                                            unsigned long long *sign_sums, int32_t *flag)
{
    __shared__ uint32_t s_row[kRangeNodes + 1];
    __shared__ uint32_t s_diff[kRangeEdges];
    __shared__ float s_cost[kRangeEdges];
    __shared__ uint16_t s_node[kRangeEdges];
    __shared__ uint32_t s_from[kMaxRuns], s_before[kMaxRuns + 1], s_out;
    const uint32_t tid = threadIdx.x, R = (uint32_t)runs.n;
    const uint32_t v0 = blockIdx.x * width;
    if (tid == 0) {
        uint32_t total = 0, out = 0;
        for (uint32_t r = 0; r < R; ++r) {
            const uint32_t a = bounds[(size_t)blockIdx.x * R + r], b = bounds[(size_t)(blockIdx.x + 1) * R + r];
            s_from[r] = a; s_before[r] = total;
            total += b - a;
            out += a - runs.start[r];
        }
        s_before[R] = total;
        s_out = out;
    }
    for (uint32_t v = tid; v <= (uint32_t)kRangeNodes; v += kBlock) s_row[v] = 0;
    __syncthreads();
    const uint32_t total = s_before[R], out0 = s_out;
    if (total > (uint32_t)kRangeEdges) {      // uniform
        if (tid == 0) *flag = 1;
        return;
    }
    uint32_t node[kRangeItems], slot[kRangeItems], diff[kRangeItems];
    float cost[kRangeItems];
#pragma unroll
    for (int q = 0; q < kRangeItems; ++q) {
        const uint32_t x = (uint32_t)q * kBlock + tid;
        node[q] = 0; slot[q] = 0; diff[q] = 0; cost[q] = 0.0f;
        if (x < total) {
            uint32_t r = 0;
            while (r + 1 < R && s_before[r + 1] <= x) ++r;
            const size_t e = (size_t)s_from[r] + (x - s_before[r]);
            const int32_t a = i[e], b = j[e];
            node[q] = (uint32_t)min(a, b) - v0;
            diff[q] = (uint32_t)abs(a - b);
            cost[q] = c[e];
            slot[q] = atomicAdd(&s_row[node[q]], 1u);      // any order: the node's edges are put into order below
        }
    }
    __syncthreads();
    constexpr int kPer = kRangeNodes / kBlock;
    uint32_t n_row[kPer], mine = 0, all;
#pragma unroll
    for (int q = 0; q < kPer; ++q) { n_row[q] = s_row[tid * kPer + q]; mine += n_row[q]; }
    uint32_t run = block_inclusive_scan(mine, &all) - mine;
#pragma unroll
    for (int q = 0; q < kPer; ++q) { s_row[tid * kPer + q] = run; run += n_row[q]; }
    if (tid == kBlock - 1) s_row[kRangeNodes] = run;
    __syncthreads();
#pragma unroll
    for (int q = 0; q < kRangeItems; ++q) {
        const uint32_t x = (uint32_t)q * kBlock + tid;
        if (x < total) {
            const uint32_t p = s_row[node[q]] + slot[q];
            s_diff[p] = diff[q]; s_cost[p] = cost[q]; s_node[p] = (uint16_t)node[q];
        }
    }
    __syncthreads();
    // signs of the costs per tile of outputs (see reduce_runs): positive in the low half of a word, negative in the high half
    const uint32_t tile0 = out0 / (uint32_t)kScanTile;
    uint32_t sign[3] = {0u, 0u, 0u};      // the outputs lie in up to three tiles
    bool bad = false;
#pragma unroll
    for (int q = 0; q < kRangeItems; ++q) {
        const uint32_t x = (uint32_t)q * kBlock + tid;
        if (x < total) {
            const uint32_t v = s_node[x], d = s_diff[x], r0 = s_row[v], r1 = s_row[v + 1];
            uint32_t rank = 0, equal = 0;
            if (r1 - r0 <= (uint32_t)kRowMax)
                for (uint32_t p = r0; p < r1; ++p) { rank += s_diff[p] < d ? 1u : 0u; equal += s_diff[p] == d ? 1u : 0u; }
            bad |= equal != 1u;
            const uint32_t o = out0 + r0 + rank;
            const float w = s_cost[x];
            io[o] = (int32_t)(v0 + v);
            jo[o] = (int32_t)(v0 + v + d);
            co[o] = w;
            const uint32_t t = o / (uint32_t)kScanTile - tile0, one = w > 0.0f ? 1u : w < 0.0f ? 1u << 16 : 0u;
#pragma unroll
            for (int k = 0; k < 3; ++k) sign[k] += t == (uint32_t)k ? one : 0u;
        }
    }
    if (bad) *flag = 1;
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        const uint32_t sum = block_sum(sign[k]);
        if (tid == 0 && sum) atomicAdd(&sign_sums[tile0 + k], (unsigned long long)(sum & 0xffffu) | (unsigned long long)(sum >> 16) << 32);
    }
}

// start: the runs' first places, ascending, and m behind them; *done stays false when the list needs the general way
rama_status interleave_runs(Ctx &ctx, int32_t n, size_t m, const int32_t *i, const int32_t *j, const float *c,
                            const std::vector<uint32_t> &start, Graph &out, bool *done)
{
    *done = false;
    Runs runs;
    runs.n = (int)start.size() - 1;
    for (int r = 0; r <= kMaxRuns; ++r) runs.start[r] = r <= runs.n ? start[(size_t)r] : (uint32_t)m;
    // nodes per workgroup: nine tenths of what it holds on average
    const uint64_t fit = (uint64_t)kRangeEdges * 9 / 10 * (uint64_t)n / m;
    const uint32_t width = (uint32_t)(fit < 1 ? 1 : fit > (uint64_t)kRangeNodes ? (uint64_t)kRangeNodes : fit);
    const uint32_t ranges = (uint32_t)(((uint64_t)n + width - 1) / width);
    if ((uint64_t)ranges > (uint64_t)m / 64 + 64) return RAMA_OK;      // next to no edges per workgroup
    Buf<uint32_t> bounds;
    Buf<int32_t> flag;
    RAMA_TRY(bounds.alloc(ctx, ((size_t)ranges + 1) * (size_t)runs.n));
    RAMA_TRY(zeroed<int32_t>(ctx, 1, flag));
    RAMA_TRY(out.i.alloc(ctx, m));
    RAMA_TRY(out.j.alloc(ctx, m));
    RAMA_TRY(out.c.alloc(ctx, m));
    const size_t tiles = (m + kScanTile - 1) / kScanTile;
    RAMA_TRY(out.sign_sums.alloc(ctx, tiles + 2));
    RAMA_TRY(fill<uint64_t>(ctx, out.sign_sums.get(), 0ull, tiles + 2));
    {
        ProfScope ps_(ctx, "k_range_bounds", (double)((size_t)ranges * runs.n * 4));
        k_range_bounds<<<grid_for(((size_t)ranges + 1) * (size_t)runs.n), kBlock, 0, ctx.stream>>>(runs, i, j, ranges, width, bounds.get());
    }
    LAUNCH_TRY(ctx, "range_bounds");
    {
        ProfScope ps_(ctx, "k_interleave_runs", (double)(m * 24));
        k_interleave_runs<<<ranges, kBlock, 0, ctx.stream>>>(runs, i, j, c, width, bounds.get(), out.i.get(), out.j.get(), out.c.get(),
                                                             (unsigned long long *)out.sign_sums.get(), flag.get());
    }
    LAUNCH_TRY(ctx, "interleave_runs");
    int32_t bad = 0;
    RAMA_TRY(read_back(ctx, &bad, flag.get(), 4));
    if (bad) {      // the general way needs the memory
        out.sign_sums.reset();
        out.i.reset(); out.j.reset(); out.c.reset();
        return RAMA_OK;
    }
    out.m = (int64_t)m;
    *done = true;
    return RAMA_OK;
}

// ---- a list that consists of a few sorted runs is merged instead of sorted --------------------------------------
constexpr int kMergeRuns = 8;
constexpr int kMergeTile = 2048;

// places p >= 1 with key[p] < key[p-1]: out[0] counts them, out[1..] takes the first kMergeRuns - 1 (in any order)
__global__ __launch_bounds__(kBlock) void k_find_descents(const uint64_t *key, size_t n, uint32_t *out)
{
    const size_t p = (size_t)blockIdx.x * kBlock + threadIdx.x;
    if (p == 0 || p >= n) return;
    if (key[p] < key[p - 1]) {
        const uint32_t k = atomicAdd(out, 1u);
        if (k < (uint32_t)(kMergeRuns - 1)) out[1 + k] = (uint32_t)p;
    }
}

// Merge path: split[t] = how many of the first t * kMergeTile merged elements come from a (a's elements go first among
// equal keys, which keeps the merge stable).
__global__ __launch_bounds__(kBlock) void k_merge_partition(const uint64_t *a, uint32_t na, const uint64_t *b, uint32_t nb,
                                                            uint32_t ntiles, uint32_t *split)
{
    const uint32_t t = blockIdx.x * kBlock + threadIdx.x;
    if (t > ntiles) return;
    const uint64_t d64 = (uint64_t)t * kMergeTile;
    const uint32_t diag = d64 < (uint64_t)na + nb ? (uint32_t)d64 : na + nb;
    uint32_t lo = diag > nb ? diag - nb : 0u, hi = diag < na ? diag : na;
    while (lo < hi) {
        const uint32_t mid = lo + (hi - lo) / 2;
        if (a[mid] <= b[diag - 1 - mid]) lo = mid + 1;
        else hi = mid;
    }
    split[t] = lo;
}

// One tile of the merged list: its pieces of a and b go to LDS side by side, every element finds its place by a
// bisection of the other piece, and the tile is written out in order.
__global__ __launch_bounds__(kBlock) void k_merge_pairs(const uint64_t *ak, const uint32_t *av, uint32_t na, const uint64_t *bk,
                                                        const uint32_t *bv, uint32_t nb, const uint32_t *split, uint64_t *ok,
                                                        uint32_t *ov)
{
    __shared__ uint64_t sk[kMergeTile];
    __shared__ uint32_t sv[kMergeTile];
    constexpr int kPer = kMergeTile / kBlock;
    const uint32_t t = blockIdx.x;
    const uint32_t diag0 = t * (uint32_t)kMergeTile;
    const uint32_t diag1 = (uint64_t)diag0 + kMergeTile < (uint64_t)na + nb ? diag0 + kMergeTile : na + nb;
    const uint32_t a0 = split[t], a1 = split[t + 1], b0 = diag0 - a0;
    const uint32_t cnt_a = a1 - a0, total = diag1 - diag0, cnt_b = total - cnt_a;
    for (uint32_t x = threadIdx.x; x < total; x += kBlock) {
        if (x < cnt_a) { sk[x] = ak[a0 + x]; sv[x] = av[a0 + x]; }
        else { sk[x] = bk[b0 + (x - cnt_a)]; sv[x] = bv[b0 + (x - cnt_a)]; }
    }
    __syncthreads();
    uint64_t k[kPer];
    uint32_t v[kPer], r[kPer];
#pragma unroll
    for (int q = 0; q < kPer; ++q) {
        const uint32_t x = threadIdx.x + (uint32_t)q * kBlock;
        r[q] = 0xffffffffu;
        if (x >= total) continue;
        k[q] = sk[x]; v[q] = sv[x];
        uint32_t lo, hi;
        if (x < cnt_a) {           // elements of b that are smaller
            lo = 0; hi = cnt_b;
            while (lo < hi) { const uint32_t mid = (lo + hi) / 2; if (sk[cnt_a + mid] < k[q]) lo = mid + 1; else hi = mid; }
            r[q] = x + lo;
        } else {                   // elements of a that are smaller or equal
            lo = 0; hi = cnt_a;
            while (lo < hi) { const uint32_t mid = (lo + hi) / 2; if (sk[mid] <= k[q]) lo = mid + 1; else hi = mid; }
            r[q] = (x - cnt_a) + lo;
        }
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < kPer; ++q)
        if (r[q] != 0xffffffffu) { sk[r[q]] = k[q]; sv[r[q]] = v[q]; }
    __syncthreads();
    for (uint32_t x = threadIdx.x; x < total; x += kBlock) { ok[diag0 + x] = sk[x]; ov[diag0 + x] = sv[x]; }
}

// key/val consist of the sorted runs [start[r], start[r+1]), r < runs: rounds of pairwise stable merges
rama_status merge_runs(Ctx &ctx, Buf<uint64_t> &key, Buf<uint32_t> &val, size_t n, std::vector<uint32_t> start)
{
    Buf<uint64_t> key2;
    Buf<uint32_t> val2, split;
    RAMA_TRY(key2.alloc(ctx, n));
    RAMA_TRY(val2.alloc(ctx, n));
    RAMA_TRY(split.alloc(ctx, n / kMergeTile + 2));
    while (start.size() > 2) {
        std::vector<uint32_t> next;
        for (size_t r = 0; r + 1 < start.size(); r += 2) {
            const uint32_t s0 = start[r], s1 = start[r + 1];
            next.push_back(s0);
            if (r + 2 >= start.size()) {   // a run without a partner moves over as it is
                HIP_TRY(ctx, hipMemcpyAsync(key2.get() + s0, key.get() + s0, (size_t)(s1 - s0) * 8, hipMemcpyDeviceToDevice, ctx.stream));
                HIP_TRY(ctx, hipMemcpyAsync(val2.get() + s0, val.get() + s0, (size_t)(s1 - s0) * 4, hipMemcpyDeviceToDevice, ctx.stream));
                continue;
            }
            const uint32_t s2 = start[r + 2], na = s1 - s0, nb = s2 - s1;
            const uint32_t ntiles = (na + nb + kMergeTile - 1) / kMergeTile;
            {
                ProfScope ps_(ctx, "k_merge_partition", (double)ntiles * 4);
                k_merge_partition<<<grid_for((size_t)ntiles + 1), kBlock, 0, ctx.stream>>>(key.get() + s0, na, key.get() + s1, nb, ntiles,
                                                                                      split.get());
            }
            LAUNCH_TRY(ctx, "merge_partition");
            {
                ProfScope ps_(ctx, "k_merge_pairs", (double)(na + nb) * 24);
                k_merge_pairs<<<ntiles, kBlock, 0, ctx.stream>>>(key.get() + s0, val.get() + s0, na, key.get() + s1, val.get() + s1, nb,
                                                               split.get(), key2.get() + s0, val2.get() + s0);
            }
            LAUNCH_TRY(ctx, "merge_pairs");
        }
        next.push_back(start.back());
        start.swap(next);
        key.swap(key2);
        val.swap(val2);
    }
    return RAMA_OK;
}

}  // namespace

rama_status canonicalise(Ctx &ctx, int32_t n, int64_t m, const int32_t *i, const int32_t *j, const float *c, Graph &out)
{
    ctx.sorts_unseen = true;      // every call begins here
    if (n < 0 || m < 0 || (m > 0 && (!i || !j || !c))) return fail(ctx, RAMA_ERR_INVALID_ARG, "canonicalise: bad arguments");
    if (m >= (int64_t(1) << 31) - 1) return fail(ctx, RAMA_ERR_CAPACITY, "edge count reaches 2^31");
    out.n = n;
    out.m = 0;
    RAMA_TRY(zero_page_recycle(ctx));
    if (m == 0) {
        RAMA_TRY(out.i.alloc(ctx, 1));
        RAMA_TRY(out.j.alloc(ctx, 1));
        RAMA_TRY(out.c.alloc(ctx, 1));
        return RAMA_OK;
    }
    Buf<int32_t> flags;
    RAMA_TRY(zeroed<int32_t>(ctx, kFlagWords, flags));
    ScanPlan<uint32_t> keep;
    RAMA_TRY((scan_plan_alloc<uint32_t>(ctx, (size_t)m, 0, keep)));
    {
        ProfScope ps_(ctx, "k_validate", (double)((size_t)m * 12));
        k_validate<<<keep.nb, kBlock, 0, ctx.stream>>>(n, (size_t)m, i, j, c, flags.get(), keep.sums.get());
    }
    LAUNCH_TRY(ctx, "validate");
    int32_t hf[kFlagWords];
    RAMA_TRY(read_back(ctx, hf, flags.get(), sizeof hf));
    if (hf[0]) return fail(ctx, RAMA_ERR_BAD_GRAPH, "edge endpoint outside [0,n_nodes) or non-finite cost");
    out.none_attractive = hf[5] == 0;      // sums of parallel edges are none either
    if (!hf[1]) {  // already canonical: plain copy
        RAMA_TRY(out.i.alloc(ctx, m));
        RAMA_TRY(out.j.alloc(ctx, m));
        RAMA_TRY(out.c.alloc(ctx, m));
        HIP_TRY(ctx, hipMemcpyAsync(out.i.get(), i, (size_t)m * 4, hipMemcpyDeviceToDevice, ctx.stream));
        HIP_TRY(ctx, hipMemcpyAsync(out.j.get(), j, (size_t)m * 4, hipMemcpyDeviceToDevice, ctx.stream));
        HIP_TRY(ctx, hipMemcpyAsync(out.c.get(), c, (size_t)m * 4, hipMemcpyDeviceToDevice, ctx.stream));
        out.m = m;
        return RAMA_OK;
    }
    if (hf[3] < kMaxRuns && !hf[4] && m > (int64_t)LocalSort<uint64_t>::cap) {
        std::vector<uint32_t> start(hf + kFirstRun, hf + kFirstRun + hf[3]);
        start.push_back(0u);
        start.push_back((uint32_t)m);
        std::sort(start.begin(), start.end());
        bool done = false;
        RAMA_TRY(interleave_runs(ctx, n, (size_t)m, i, j, c, start, out, &done));
        if (done) return RAMA_OK;
    }
    const int nbits = bits_for((uint64_t)n), dbits = bits_for((uint64_t)hf[2] + 1);
    RAMA_TRY((scan_totals<uint32_t>(ctx, NotLoop{i, j}, keep, keep.sums.get())));   // tile sums: left by k_validate
    const uint32_t kept = keep.total;
    if (kept == 0) {
        RAMA_TRY(out.i.alloc(ctx, 1));
        RAMA_TRY(out.j.alloc(ctx, 1));
        RAMA_TRY(out.c.alloc(ctx, 1));
        return RAMA_OK;
    }
    Buf<uint64_t> key;
    Buf<uint32_t> val;
    RAMA_TRY(key.alloc(ctx, kept));
    RAMA_TRY(val.alloc(ctx, kept));
    Buf<uint32_t> head_sums;   // heads per scan tile, if the sort's last kernel could count them
    ScanPlan<uint32_t> runs;
    RAMA_TRY((scan_plan_alloc<uint32_t>(ctx, kept, 1, runs)));
    SortAgain<uint64_t, uint32_t> again;
    again.flag = runs.extra_ptr();
    const bool few_runs = hf[3] < kMergeRuns;
    if (!few_runs && sort_takes_source(kept, (size_t)m)) {      // the sort's first pass reads the edges itself
        Buf<uint64_t> key2;
        Buf<uint32_t> val2;
        RAMA_TRY(key2.alloc(ctx, kept));
        RAMA_TRY(val2.alloc(ctx, kept));
        keep.offs.reset();
        RAMA_TRY((radix_sort_source<uint64_t, uint32_t>(ctx, InputEdges{i, j, c, dbits}, (size_t)m, key, val, key2, val2, kept, nbits + dbits,
                                                        &head_sums, (uint64_t)n << dbits, &again)));
    } else {
        RAMA_TRY((scan_emit<uint32_t>(ctx, NotLoop{i, j}, PackEdgesEmit{i, j, c, dbits, key.get(), val.get()}, keep,
                                      (double)((size_t)m * 4 + (size_t)kept * 12))));
        keep.offs.reset();
        bool merged = false;
        if (few_runs && kept > (uint32_t)LocalSort<uint64_t>::cap) {
            // few places where the order breaks: the packed list is a handful of sorted runs (dropping self-loops cannot
            // add any): find their starts and merge them, one pass per doubling, instead of sorting by all key bits
            Buf<uint32_t> desc;
            RAMA_TRY(zeroed<uint32_t>(ctx, kMergeRuns, desc));
            {
                ProfScope ps_(ctx, "k_find_descents", (double)kept * 8);
                k_find_descents<<<grid_for(kept), kBlock, 0, ctx.stream>>>(key.get(), kept, desc.get());
            }
            LAUNCH_TRY(ctx, "find_descents");
            uint32_t hd[kMergeRuns];
            RAMA_TRY(read_back(ctx, hd, desc.get(), sizeof hd));
            if (hd[0] < (uint32_t)kMergeRuns) {
                std::vector<uint32_t> start(hd + 1, hd + 1 + hd[0]);
                start.push_back(0u);
                start.push_back(kept);
                std::sort(start.begin(), start.end());
                RAMA_TRY(merge_runs(ctx, key, val, kept, start));
                merged = true;
            }
        }
        if (!merged)
            RAMA_TRY((radix_sort_pairs<uint64_t, uint32_t>(ctx, key, val, kept, nbits + dbits, false, &head_sums, (uint64_t)n << dbits, &again)));
    }
    RAMA_TRY((count_heads<uint64_t, uint32_t>(ctx, key, &val, kept, nbits + dbits, [](const uint64_t *k) { return HeadFlag{k}; }, runs, 0, head_sums, again)));
    const uint32_t uniq = runs.total;
    RAMA_TRY(out.i.alloc(ctx, uniq));
    RAMA_TRY(out.j.alloc(ctx, uniq));
    RAMA_TRY(out.c.alloc(ctx, uniq));
    RAMA_TRY(reduce_runs(ctx, runs, key.get(), val.get(), dbits, out.i.get(), out.j.get(), out.c.get(), &out.sign_sums));
    out.m = uniq;
    return RAMA_OK;
}

namespace {
struct NegPart {
    static constexpr int bytes = 4;   // bytes read per item
    static constexpr const char *tag = "NegPart";
    const float *c;
    __device__ __forceinline__ double operator()(size_t e) const { float w = c[e]; return w < 0.0f ? (double)w : 0.0; }
};
}  // namespace

rama_status negative_cost_sum(Ctx &ctx, const float *c, int64_t m, double *out)
{
    Buf<double> d;
    RAMA_TRY(d.alloc(ctx, 1));
    RAMA_TRY(device_sum(ctx, NegPart{c}, (size_t)m, d.get(), false));
    return read_back(ctx, out, d.get(), 8);
}

}  // namespace rama
