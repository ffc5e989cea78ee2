// Whole rounds of the solver on graphs that one workgroup can hold (up to 8192 edges and 6144 nodes).
//
// A round of a small graph through the stage kernels is some sixty launches and ten host waits, 250 to 1100 us whatever
// the size: nothing but latency (2.3 us per dependent launch, 9 us per count the host waits for).  Here one workgroup of
// 1024 threads keeps the edge list in LDS and runs round after round -- triangles, message passing, matching or
// spanning forest, contraction -- between barriers, and the host hears of it when it is over.  The arithmetic, its order
// and every tie are those of the stage kernels, so the results are the same bit for bit.
//
// Bounded by barriers, LDS latency and the instructions that sixteen waves on one CU issue, so what counts is that a step
// of a short list takes few of them: loops over a thread's items end where the list does, triangles' slots and contracted
// edges find their places by counting and comparing instead of by passes, and barriers wait for LDS only.  Measured per round,
// with passes and loops of full length | as it is: 36 edges 17 | 10 us, 438 edges with a triangle 31 | 20, 2678 edges 43 | 33,
// 6210 edges 120 | 93 (through the stage kernels 250 to 1100 whatever the size); all rounds of a 32^2 grid 220 | 130, of a 128^2
// long-range grid 285 | 202, of the contraction of a 300x301 one 323 | 258.
#include "prim.h"
#include "steps.h"

namespace rama {

namespace {

constexpr int kTailThreads = 1024;
constexpr int kTailWaves = kTailThreads / 64;
constexpr int kTailItems = kTailEdges / kTailThreads;          // edges per thread
constexpr int kTailNodeItems = kTailNodes / kTailThreads;      // nodes per thread
constexpr int kTriItems = kTailTriangles / kTailThreads;
constexpr int kSlotItems = 3 * kTailTriangles / kTailThreads;
constexpr int kNodeBits = 13;
constexpr uint32_t kNodeMask = (1u << kNodeBits) - 1u;
static_assert(kTailNodes <= (1 << kNodeBits) - 1 && kTailEdges <= (1 << 13) && 3 * kTailTriangles <= kTailEdges, "field widths");
static_assert(kTailEdges % kTailThreads == 0 && kTailNodes % (2 * kTailThreads) == 0, "whole items per thread");

// the work area (in 4-byte words), used by one step after another:
//   sort        keys [0, 8192), values [8192, 16384), digit counts of the 16 waves [16384, 20480)
//   separation  row ends [0, 3136) (16 bits each), cursors, then first edges of the rows [3136, 6272), adjacency [6272, 14464) (16-bit edge numbers),
//               triangles found: keys [14464, 16512), third edges [16512, 17536) (16 bits each), entries each
//               repulsive edge is tried with [17536, 21632) (16 bits each), their sums per thread [21632, 22656)
//   messages    slots of every edge [0, 8192), as they came [8192, 11264) and in order [11264, 14336) (16 bits each), or sorted
//               slots as the sort left them; messages [14336, 20480)
//   matching    rank words [0, 12288), mates [12288, 15360) (16 bits each)
//   forest      rank words [0, 12288), later depth, parent, edge to it (16 bits each) [0, 9216); components
//               [12288, 15360), hooks [15360, 18432), forest bits [18432, 18688), removed bits [18688, 18944)
//   mapping     representatives [0, 6144), new numbers [6144, 9216) (16 bits each)
constexpr int kWorkWords = 22656;
constexpr int kSortVal = kTailEdges, kSortHist = 2 * kTailEdges;
constexpr int kSepCur = 3136, kSepAdj = 6272, kSepKey = 14464, kSepThird = 16512, kSepTries = 17536, kSepBefore = 21632;
constexpr int kMsg = 14336, kArrived = 8192, kSlot = 11264;
constexpr int kMate = 12288, kComp = 12288, kHook = 15360, kInForest = 18432, kRemoved = 18688;
constexpr int kDepth = 0, kUp = 3072, kUpEdge = 6144;
constexpr int kRep = 0, kNew = 6144;
static_assert(kSepCur * 2 >= kTailNodes + 1 && kSepAdj + kTailEdges <= kSepKey && kSepThird + kTailTriangles / 2 <= kSepTries &&
              kSepTries + kTailEdges / 2 <= kSepBefore && kSepBefore + kTailThreads <= kWorkWords, "separation");
static_assert(kArrived >= kTailEdges && kArrived + 3 * kTailTriangles / 2 <= kSlot && kSlot + 3 * kTailTriangles / 2 <= kMsg && kMsg <= kSepKey, "slots");
static_assert(kSortVal + 3 * kTailTriangles <= kMsg && kMsg + 3 * kTailTriangles <= kWorkWords, "messages");
static_assert(2 * kTailNodes <= kMate && kMate + kTailNodes / 2 <= kHook && kHook + kTailNodes / 2 <= kInForest, "matching, forest");
static_assert(kInForest + kTailEdges / 32 <= kRemoved && kRemoved + kTailEdges / 32 <= kWorkWords, "forest bits");
static_assert(kSortHist + kTailWaves * kRadix <= kWorkWords, "sort");

struct alignas(8) TailShared {
    uint32_t key[kTailEdges];      // lo << 13 | hi, ascending
    float cost[kTailEdges];
    uint32_t work[kWorkWords];
    uint32_t wave[kTailWaves];
    uint32_t digit[4];
    uint32_t count[6];
};
static_assert(alignof(TailShared) % 8 == 0 && offsetof(TailShared, work) % 8 == 0, "the work area holds 64-bit rank words, whose LDS atomics fault elsewhere");

struct TailArgs {
    int32_t n, m;
    const int32_t *i, *j;          // graph in, graph out (the arrays may be the same)
    const float *c;
    int32_t *io, *jo;
    float *co;
    int32_t *fmap;                 // [n]: node of the first graph -> node of the last
    int separate, iters, cap, max_rounds;
    float tau, forest_ratio;
    MailWord *mail;
    uint64_t seq;
};

__device__ __forceinline__ int tail_lane() { return (int)(threadIdx.x & 63u); }
__device__ __forceinline__ int tail_wave() { return __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)); }

// exclusive scan over the 1024 threads
__device__ __forceinline__ uint32_t tail_scan(uint32_t v, uint32_t *total, uint32_t *s_wave)
{
    const uint32_t inc = wave_inclusive_scan(v);
    const int w = tail_wave();
    if (tail_lane() == 63) s_wave[w] = inc;
    __syncthreads();
    uint32_t x = s_wave[tail_lane() & (kTailWaves - 1)];
    x = wave_inclusive_scan(tail_lane() < kTailWaves ? x : 0u);
    const uint32_t before = w ? (uint32_t)__builtin_amdgcn_readlane((int)x, w - 1) : 0u;
    *total = (uint32_t)__builtin_amdgcn_readlane((int)x, kTailWaves - 1);
    __syncthreads();
    return before + inc - v;
}

// Stable sort of cnt (key, value) pairs by the key's low `bits` bits.  Item r of lane l in wave w is number
// (w*rows + r)*64 + l, rows = ceil(cnt / 1024); the result is in work[0..) and work[kSortVal..).  The passes are those
// of k_rs_local.
__device__ __forceinline__ void tail_sort(TailShared &S, uint32_t (&key)[kTailItems], uint32_t (&val)[kTailItems], uint32_t cnt, int bits)
{
    uint32_t *skey = S.work, *sval = S.work + kSortVal;
    uint32_t *whist = S.work + kSortHist;
    const int tid = (int)threadIdx.x, lane = tail_lane(), w = tail_wave();
    const int rows = (int)((cnt + kTailThreads - 1) / kTailThreads);
    const uint32_t base = (uint32_t)(w * rows * 64 + lane);
    const uint64_t lt = (1ull << lane) - 1ull;
    uint32_t rank[kTailItems];
    const int passes = (bits + kRadixBits - 1) / kRadixBits;
    int shift = 0, remaining = bits;
    for (int p = 0; p < passes; ++p) {
        const int b = (remaining + (passes - p) - 1) / (passes - p);
        const uint32_t mask = (1u << b) - 1u;
        for (int k = tid; k < kTailWaves * kRadix; k += kTailThreads) whist[k] = 0;
        __syncthreads();
#pragma unroll
        for (int r = 0; r < kTailItems; ++r)
            if (r < rows) {
                const bool valid = base + (uint32_t)r * 64u < cnt;
                const uint32_t d = (key[r] >> shift) & mask;
                const uint64_t same = match_digit(d, b, __ballot(valid));
                uint32_t *h = whist + w * kRadix + d;
                const uint32_t before = *h;
                rank[r] = before + (uint32_t)__popcll(same & lt);
                __builtin_amdgcn_wave_barrier();
                if (valid && lane == __ffsll((long long)same) - 1) *h = before + (uint32_t)__popcll(same);
                __builtin_amdgcn_wave_barrier();
            }
        __syncthreads();
        uint32_t c[kTailWaves], tot = 0;
        if (tid < kRadix) {
#pragma unroll
            for (int k = 0; k < kTailWaves; ++k) { c[k] = whist[k * kRadix + tid]; tot += c[k]; }
        }
        const uint32_t inc = wave_inclusive_scan(tot);
        if (tid < kRadix && lane == 63) S.digit[w] = inc;
        __syncthreads();
        if (tid < kRadix) {
            uint32_t run = inc - tot;
#pragma unroll
            for (int k = 0; k < 3; ++k)
                if (k < w) run += S.digit[k];
#pragma unroll
            for (int k = 0; k < kTailWaves; ++k) { whist[k * kRadix + tid] = run; run += c[k]; }
        }
        __syncthreads();
#pragma unroll
        for (int r = 0; r < kTailItems; ++r)
            if (r < rows && base + (uint32_t)r * 64u < cnt) {
                const uint32_t at = whist[w * kRadix + ((key[r] >> shift) & mask)] + rank[r];
                skey[at] = key[r];
                sval[at] = val[r];
            }
        __syncthreads();
        if (p + 1 < passes) {
#pragma unroll
            for (int r = 0; r < kTailItems; ++r)
                if (r < rows && base + (uint32_t)r * 64u < cnt) {
                    key[r] = skey[base + (uint32_t)r * 64u];
                    val[r] = sval[base + (uint32_t)r * 64u];
                }
        }
        shift += b;
        remaining -= b;
    }
}

__device__ __forceinline__ int tail_bits(uint32_t n)      // bits for values in [0, n)
{
    return n <= 2u ? 1 : 32 - __clz((int)(n - 1u));
}

// items of a list of `count` that a thread takes: loops over a thread's items end there (uniform), so that a short list does
// not pay for the longest one
__device__ __forceinline__ int tail_per_thread(int count) { return (count + kTailThreads - 1) / kTailThreads; }

// Triangles with one repulsive edge (a round that separates up to length 3).  Returns their number if it is at most
// kTailTriangles; they are in work[kSepKey..) -- (first edge, second edge) -- and work[kSepThird..), in any order.
// With more of them a thread stops at the first one it has no place for, and the return is some larger number.
__device__ __forceinline__ uint32_t tail_triangles(TailShared &S, int n, int m, uint32_t &n_attractive, uint32_t &n_repulsive)
{
    const int tid = (int)threadIdx.x, per = tail_per_thread(m), per_node = tail_per_thread(n);
    uint16_t *row_end = (uint16_t *)S.work, *adj = (uint16_t *)(S.work + kSepAdj);
    for (int k = tid; 2 * k < n; k += kTailThreads) S.work[k] = 0;      // degrees
    if (tid < 3) S.count[tid] = 0;
    lds_barrier();
    uint32_t pos = 0, neg = 0;
#pragma unroll
    for (int q = 0; q < kTailItems; ++q) {
        if (q >= per) break;
        const int e = tid + q * kTailThreads;
        const float c = e < m ? S.cost[e] : 0.0f;
        neg += c < 0.0f ? 1u : 0u;
        if (c > 0.0f) {
            ++pos;
            const uint32_t u = S.key[e] >> kNodeBits, v = S.key[e] & kNodeMask;
            atomicAdd(&S.work[u >> 1], 1u << (16 * (u & 1)));      // at most 8191 per node: no carry between the halves
            atomicAdd(&S.work[v >> 1], 1u << (16 * (v & 1)));
        }
    }
    pos = wave_sum(pos); neg = wave_sum(neg);
    if (tail_lane() == 0 && (pos | neg)) { atomicAdd(&S.count[0], pos); atomicAdd(&S.count[1], neg); }
    lds_barrier();
    n_attractive = S.count[0]; n_repulsive = S.count[1];
    if (n_attractive == 0 || n_repulsive == 0) return 0;
    uint32_t deg[kTailNodeItems], mine = 0, all;
#pragma unroll
    for (int q = 0; q < kTailNodeItems; ++q) {
        const int v = tid * per_node + q;
        deg[q] = q < per_node && v < n ? row_end[v] : 0u;
        mine += deg[q];
    }
    uint32_t run = tail_scan(mine, &all, S.wave);
    uint16_t *cursor = (uint16_t *)(S.work + kSepCur);
#pragma unroll
    for (int q = 0; q < kTailNodeItems; ++q) {
        const int v = tid * per_node + q;
        if (q < per_node && v < n) {
            cursor[v] = (uint16_t)run;
            run += deg[q];
            row_end[v] = (uint16_t)run;
        }
    }
    lds_barrier();
#pragma unroll
    for (int q = 0; q < kTailItems; ++q) {
        if (q >= per) break;
        const int e = tid + q * kTailThreads;
        if (e < m && S.cost[e] > 0.0f) {
            const uint32_t u = S.key[e] >> kNodeBits, v = S.key[e] & kNodeMask;
            const uint32_t au = atomicAdd(&S.work[kSepCur + (u >> 1)], 1u << (16 * (u & 1)));
            const uint32_t av = atomicAdd(&S.work[kSepCur + (v >> 1)], 1u << (16 * (v & 1)));
            adj[(au >> (16 * (u & 1))) & 0xffffu] = (uint16_t)e;
            adj[(av >> (16 * (v & 1))) & 0xffffu] = (uint16_t)e;
        }
    }
    lds_barrier();
    // Every repulsive edge is tried with each entry of the shorter of its rows; the tries are dealt out evenly over the
    // threads (an edge per thread and turn left most of a wave waiting for its longest row), a stretch of them to each, which
    // finds its first edge once.  The third edge is looked for in its row of the list; the rows begin at row_first, which
    // takes the cursors' place.
    uint16_t *row_first = cursor, *tries = (uint16_t *)(S.work + kSepTries), *third = (uint16_t *)(S.work + kSepThird);
    uint32_t *before = S.work + kSepBefore;      // tries of the edges of the threads in front; thread t: edges t * per ..
    for (int v = tid; v <= n; v += kTailThreads) {
        const uint32_t key = (uint32_t)v << kNodeBits;
        int lo = 0, hi = m;
        while (lo < hi) {
            const int mid = (lo + hi) >> 1;
            if (S.key[mid] < key) lo = mid + 1; else hi = mid;
        }
        row_first[v] = (uint16_t)lo;
    }
    auto rows_of = [&](int e, uint32_t &s, uint32_t &o, int &s0) {      // s: the end with the shorter row, which starts at s0
        s = S.key[e] >> kNodeBits; o = S.key[e] & kNodeMask;
        s0 = s ? row_end[s - 1] : 0;
        int len = row_end[s] - s0;
        const int o0 = o ? row_end[o - 1] : 0, len_o = row_end[o] - o0;
        if (len > len_o) { const uint32_t t = s; s = o; o = t; s0 = o0; len = len_o; }
        return len;
    };
    uint32_t sum = 0, all_tries;
    uint32_t s, o;
    int s0;
#pragma unroll
    for (int q = 0; q < kTailItems; ++q) {
        if (q >= per) break;
        const int e = tid * per + q;
        if (e < m) {
            const uint32_t len = S.cost[e] < 0.0f ? (uint32_t)rows_of(e, s, o, s0) : 0u;
            tries[e] = (uint16_t)len;
            sum += len;
        }
    }
    before[tid] = tail_scan(sum, &all_tries, S.wave);
    lds_barrier();
    const uint32_t stretch = (all_tries + kTailThreads - 1) / kTailThreads, first = (uint32_t)tid * stretch;
    const uint32_t last = first + stretch < all_tries ? first + stretch : all_tries;
    if (first < last) {
        int t = 0;      // the last thread with at most `first` tries before its own
#pragma unroll
        for (int step = kTailThreads / 2; step > 0; step >>= 1)
            if (before[t + step] <= first) t += step;
        int e = t * per;
        uint32_t k = first - before[t], len = tries[e];
        while (k >= len) { k -= len; len = tries[++e]; }
        (void)rows_of(e, s, o, s0);
        for (uint32_t p = first;;) {
            const int a = adj[s0 + (int)k];
            const uint32_t u = S.key[a] >> kNodeBits, v = S.key[a] & kNodeMask, x = u == s ? v : u, x0 = min(x, o);
            const uint32_t wanted = x0 << kNodeBits | max(x, o);
            int lo = row_first[x0], hi = row_first[x0 + 1];
            const int end = hi;
            while (lo < hi) {
                const int mid = (lo + hi) >> 1;
                if (S.key[mid] < wanted) lo = mid + 1; else hi = mid;
            }
            if (lo < end && S.key[lo] == wanted && S.cost[lo] > 0.0f) {
                // the edges (u,v), (u,w), (v,w) of a triangle u < v < w stand in this order in the list
                const int b = lo, e0 = min(e, min(a, b)), e2 = max(e, max(a, b)), e1 = e + a + b - e0 - e2;
                const uint32_t at = atomicAdd(&S.count[2], 1u);
                if (at >= (uint32_t)kTailTriangles) break;
                S.work[kSepKey + at] = (uint32_t)e0 << 13 | (uint32_t)e1;
                third[at] = (uint16_t)e2;
            }
            if (++p >= last) break;
            if (++k >= len) {      // there are tries left, so an edge behind this one has some
                k = 0;
                do len = tries[++e]; while (len == 0);
                (void)rows_of(e, s, o, s0);
            }
        }
    }
    lds_barrier();
    return S.count[2];
}

// Places of a stable sort of the keys of the items in `in` (bit r: item r) by their `bits` bits, as local_sort does it: the top
// bits make buckets, and a key finds its place among its bucket's by comparing a word that ends with the place it came from,
// which is base + 64 r.  Keys and values are then in work[0..) and work[kSortVal..); false, and nothing done, if a bucket
// is too long.
constexpr int kTailBucketBits = 12, kTailBucketMax = 160;
__device__ __forceinline__ bool tail_bucket_sort(TailShared &S, const uint32_t (&key)[kTailItems], const uint32_t (&val)[kTailItems], uint32_t in,
                                                 int rows, uint32_t base, int bits)
{
    static_assert((1 << kTailBucketBits) == 4 * kTailThreads && kSortHist + 2 * kTailThreads <= kWorkWords, "two words of two counters to a thread");
    const int tid = (int)threadIdx.x, shift = bits > kTailBucketBits ? bits - kTailBucketBits : 0;
    uint32_t *count = S.work + kSortHist;
    const uint16_t *end = reinterpret_cast<const uint16_t *>(count);
    count[2 * tid] = 0; count[2 * tid + 1] = 0;
    if (tid == 0) S.count[3] = 0;
    lds_barrier();
    uint32_t at[kTailItems];
#pragma unroll
    for (int r = 0; r < kTailItems; ++r) {
        if (r >= rows) break;
        if (in & (1u << r)) {
            const uint32_t b = key[r] >> shift;
            at[r] = (atomicAdd(&count[b >> 1], 1u << (16 * (b & 1))) >> (16 * (b & 1))) & 0xffffu;      // at most 8192 in all: no carry
        }
    }
    lds_barrier();
    const uint32_t x = count[2 * tid], y = count[2 * tid + 1];
    const uint32_t c0 = x & 0xffffu, c1 = x >> 16, c2 = y & 0xffffu, c3 = y >> 16;
    if (max(max(c0, c1), max(c2, c3)) > (uint32_t)kTailBucketMax) S.count[3] = 1;
    uint32_t all;
    const uint32_t run = tail_scan(c0 + c1 + c2 + c3, &all, S.wave);
    if (S.count[3]) {      // uniform; nobody changes it before the next barrier
        lds_barrier();
        return false;
    }
    count[2 * tid] = (run + c0) | (run + c0 + c1) << 16;
    count[2 * tid + 1] = (run + c0 + c1 + c2) | (run + c0 + c1 + c2 + c3) << 16;
    lds_barrier();
    const uint32_t low = (1u << shift) - 1u;
#pragma unroll
    for (int r = 0; r < kTailItems; ++r) {
        if (r >= rows) break;
        if (in & (1u << r)) {
            const uint32_t b = key[r] >> shift;
            S.work[(b ? end[b - 1] : 0u) + at[r]] = (key[r] & low) << 13 | (base + (uint32_t)r * 64u);
        }
    }
    lds_barrier();
#pragma unroll
    for (int r = 0; r < kTailItems; ++r) {
        if (r >= rows) break;
        if (in & (1u << r)) {
            const uint32_t b = key[r] >> shift, b0 = b ? end[b - 1] : 0u, b1 = end[b];
            const uint32_t self = (key[r] & low) << 13 | (base + (uint32_t)r * 64u);
            at[r] = b0;
            for (uint32_t p = b0; p < b1; p += 4) {      // four words under way at a time
                uint32_t x[4];
#pragma unroll
                for (int k = 0; k < 4; ++k) x[k] = S.work[p + k];
#pragma unroll
                for (int k = 0; k < 4; ++k) at[r] += p + k < b1 && x[k] < self ? 1u : 0u;
            }
        }
    }
    lds_barrier();
#pragma unroll
    for (int r = 0; r < kTailItems; ++r) {
        if (r >= rows) break;
        if (in & (1u << r)) { S.work[at[r]] = key[r]; S.work[kSortVal + at[r]] = val[r]; }
    }
    lds_barrier();
    return true;
}

// message passing where an edge has many slots: triangles, then slots, put into order by sorts
__device__ __forceinline__ void tail_messages_sorted(TailShared &S, int m, uint32_t T, int iters)
{
    const int tid = (int)threadIdx.x, lane = tail_lane(), w = tail_wave();
    const int ebits = tail_bits((uint32_t)m);
    uint32_t *skey = S.work, *sval = S.work + kSortVal;
    uint32_t key[kTailItems] = {}, val[kTailItems] = {};
    {
        const uint32_t rows = (T + kTailThreads - 1) / kTailThreads, base = (uint32_t)w * rows * 64u + (uint32_t)lane;
#pragma unroll
        for (int r = 0; r < kTriItems; ++r)
            if ((uint32_t)r < rows && base + (uint32_t)r * 64u < T) {
                key[r] = S.work[kSepKey + base + (uint32_t)r * 64u];
                val[r] = reinterpret_cast<const uint16_t *>(S.work + kSepThird)[base + (uint32_t)r * 64u];
            }
    }
    __syncthreads();
    tail_sort(S, key, val, T, 13 + ebits);
    uint32_t e0[kTriItems] = {}, e1[kTriItems] = {}, e2[kTriItems] = {};
#pragma unroll
    for (int q = 0; q < kTriItems; ++q) {
        const uint32_t t = (uint32_t)(tid + q * kTailThreads);
        if (t < T) { e0[q] = skey[t] >> 13; e1[q] = skey[t] & 8191u; e2[q] = sval[t]; }
    }
    // slots 3t, 3t+1, 3t+2 of triangle t, sorted by edge (stable: an edge's slots ascend)
    const uint32_t ns = 3 * T;
    {
        const uint32_t rows = (ns + kTailThreads - 1) / kTailThreads, base = (uint32_t)w * rows * 64u + (uint32_t)lane;
#pragma unroll
        for (int r = 0; r < kSlotItems; ++r) {
            const uint32_t s = base + (uint32_t)r * 64u;
            if ((uint32_t)r < rows && s < ns) {
                const uint32_t t = s / 3u, k = s - 3u * t;
                key[r] = k == 0 ? skey[t] >> 13 : k == 1 ? skey[t] & 8191u : sval[t];
                val[r] = s;
            }
        }
    }
    __syncthreads();
    tail_sort(S, key, val, ns, ebits);
    uint32_t len[kSlotItems], edge[kSlotItems];
#pragma unroll
    for (int q = 0; q < kSlotItems; ++q) {      // the run of slots that starts at place p
        const uint32_t p = (uint32_t)(tid + q * kTailThreads);
        len[q] = 0; edge[q] = 0;
        if (p < ns && (p == 0 || skey[p] != skey[p - 1])) {
            edge[q] = skey[p];
            uint32_t end = p + 1;
            while (end < ns && skey[end] == edge[q]) ++end;
            len[q] = end - p;
            S.cost[edge[q]] = S.cost[edge[q]] / (float)len[q];      // from here to the last iteration: the share
        }
    }
    __syncthreads();
    float *msg = reinterpret_cast<float *>(S.work + kMsg);
    float a[kTriItems] = {}, b[kTriItems] = {}, c[kTriItems] = {};
    for (int it = 1; it <= iters; ++it) {
#pragma unroll
        for (int q = 0; q < kTriItems; ++q) {
            const uint32_t t = (uint32_t)(tid + q * kTailThreads);
            if (t < T) {
                a[q] = a[q] + S.cost[e0[q]]; b[q] = b[q] + S.cost[e1[q]]; c[q] = c[q] + S.cost[e2[q]];
                float oa, ob, oc;
                triangle_to_edges(a[q], b[q], c[q], oa, ob, oc);
                msg[3 * t] = oa; msg[3 * t + 1] = ob; msg[3 * t + 2] = oc;
            }
        }
        __syncthreads();
#pragma unroll
        for (int q = 0; q < kSlotItems; ++q)
            if (len[q]) {
                const uint32_t p = (uint32_t)(tid + q * kTailThreads);
                float acc = 0.0f;
                for (uint32_t s = 0; s < len[q]; ++s) acc = acc + msg[sval[p + s]];
                S.cost[edge[q]] = it == iters ? acc : acc / (float)len[q];
            }
        __syncthreads();
    }
}

// The slots of an edge -- its places in triangles -- in the order of the triangles, by counting and comparing (see k_messages_few):
// work[e]: the first of edge e's slots | their number << 16, slot[]: 3 * triangle + which.  The triangles stay where they
// are.  false, and nothing else done, if an edge has more than kTailRun slots.
constexpr uint32_t kTailRun = 48;
__device__ __forceinline__ bool tail_slots(TailShared &S, int m, uint32_t T, uint32_t (&e)[kTriItems][3])
{
    const int tid = (int)threadIdx.x, per = tail_per_thread(m);
    uint16_t *arrived = (uint16_t *)(S.work + kArrived), *slot = (uint16_t *)(S.work + kSlot);
    for (int k = tid; k < m; k += kTailThreads) S.work[k] = 0;
    if (tid == 0) S.count[3] = 0;
    uint32_t key[kTriItems], at[kTriItems][3];
#pragma unroll
    for (int q = 0; q < kTriItems; ++q) {
        const uint32_t t = (uint32_t)(tid + q * kTailThreads);
        key[q] = t < T ? S.work[kSepKey + t] : 0u;
        e[q][0] = key[q] >> 13; e[q][1] = key[q] & 8191u;
        e[q][2] = t < T ? reinterpret_cast<const uint16_t *>(S.work + kSepThird)[t] : 0u;
    }
    lds_barrier();
#pragma unroll
    for (int q = 0; q < kTriItems; ++q)
        if ((uint32_t)(tid + q * kTailThreads) < T)
#pragma unroll
            for (int k = 0; k < 3; ++k) at[q][k] = atomicAdd(&S.work[e[q][k]], 1u);
    lds_barrier();
    uint32_t c[kTailItems], mine = 0, all, longest = 0;
#pragma unroll
    for (int q = 0; q < kTailItems; ++q) {
        const int x = tid * per + q;
        c[q] = q < per && x < m ? S.work[x] : 0u;
        mine += c[q];
        longest = max(longest, c[q]);
    }
    if (longest > kTailRun) S.count[3] = 1;
    uint32_t run = tail_scan(mine, &all, S.wave);
    if (S.count[3]) {      // uniform
        lds_barrier();
        return false;
    }
#pragma unroll
    for (int q = 0; q < kTailItems; ++q) {
        const int x = tid * per + q;
        if (q < per && x < m) S.work[x] = run | c[q] << 16;
        run += c[q];
    }
    lds_barrier();
#pragma unroll
    for (int q = 0; q < kTriItems; ++q) {
        const uint32_t t = (uint32_t)(tid + q * kTailThreads);
        if (t < T)
#pragma unroll
            for (int k = 0; k < 3; ++k) arrived[(S.work[e[q][k]] & 0xffffu) + at[q][k]] = (uint16_t)t;
    }
    lds_barrier();
#pragma unroll
    for (int q = 0; q < kTriItems; ++q) {
        const uint32_t t = (uint32_t)(tid + q * kTailThreads);
        if (t < T)
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                const uint32_t x = S.work[e[q][k]], p0 = x & 0xffffu, p1 = p0 + (x >> 16);
                uint32_t to = p0;
                for (uint32_t p = p0; p < p1; ++p) to += S.work[kSepKey + arrived[p]] < key[q] ? 1u : 0u;
                slot[to] = (uint16_t)(3u * t + (uint32_t)k);
            }
    }
    lds_barrier();
    return true;
}

// `iters` iterations of message passing over the T <= kTailTriangles triangles tail_triangles left behind
__device__ __forceinline__ void tail_messages(TailShared &S, int m, uint32_t T, int iters)
{
    const int tid = (int)threadIdx.x, per = tail_per_thread(m);
    uint32_t e[kTriItems][3];
    if (!tail_slots(S, m, T, e)) return tail_messages_sorted(S, m, T, iters);
    const uint16_t *slot = (const uint16_t *)(S.work + kSlot);
    uint32_t run[kTailItems];      // of the edges tid, tid + kTailThreads ..: first slot | slots << 16
#pragma unroll
    for (int q = 0; q < kTailItems; ++q) {
        const int x = tid + q * kTailThreads;
        run[q] = q < per && x < m ? S.work[x] : 0u;
        if (run[q] >> 16) S.cost[x] = S.cost[x] / (float)(run[q] >> 16);      // from here to the last iteration: the share
    }
    lds_barrier();
    float *msg = reinterpret_cast<float *>(S.work + kMsg);
    float a[kTriItems] = {}, b[kTriItems] = {}, c[kTriItems] = {};
    for (int it = 1; it <= iters; ++it) {
#pragma unroll
        for (int q = 0; q < kTriItems; ++q) {
            const uint32_t t = (uint32_t)(tid + q * kTailThreads);
            if (t < T) {
                a[q] = a[q] + S.cost[e[q][0]]; b[q] = b[q] + S.cost[e[q][1]]; c[q] = c[q] + S.cost[e[q][2]];
                float oa, ob, oc;
                triangle_to_edges(a[q], b[q], c[q], oa, ob, oc);
                msg[3 * t] = oa; msg[3 * t + 1] = ob; msg[3 * t + 2] = oc;
            }
        }
        lds_barrier();
#pragma unroll
        for (int q = 0; q < kTailItems; ++q) {
            if (q >= per) break;
            const uint32_t len = run[q] >> 16, p0 = run[q] & 0xffffu;
            if (len) {
                float acc = 0.0f;
                for (uint32_t p = p0; p < p0 + len; ++p) acc = acc + msg[slot[p]];
                S.cost[tid + q * kTailThreads] = it == iters ? acc : acc / (float)len;
            }
        }
        lds_barrier();
    }
}

// handshake matching (see k_handshake_finish); mates (0xffff: none) in work[kMate..); returns the number of pairs
__device__ __forceinline__ uint32_t tail_matching(TailShared &S, int n, int m, float tau, int cap)
{
    constexpr unsigned long long kMatched = ~0ull;      // in a node's word: no candidate's rank
    const int tid = (int)threadIdx.x, per = tail_per_thread(m);
    unsigned long long *best = reinterpret_cast<unsigned long long *>(S.work);
    uint16_t *mate = (uint16_t *)(S.work + kMate);
    uint32_t *any = S.count + 4;      // [2]: candidates left in this round, in the next one
    for (int k = tid; 2 * k < n; k += kTailThreads) S.work[kMate + k] = 0xffffffffu;
    for (int v = tid; v < n; v += kTailThreads) best[v] = 0ull;
    if (tid < 2) any[tid] = 0u;
    uint32_t alive = 0, made = 0, uv[kTailItems];
    unsigned long long rank[kTailItems];
#pragma unroll
    for (int q = 0; q < kTailItems; ++q) {
        const int e = tid + q * kTailThreads;
        uv[q] = 0; rank[q] = 0;
        if (q < per && e < m && S.cost[e] > tau) {
            alive |= 1u << q;
            uv[q] = S.key[e];
            rank[q] = edge_rank(S.cost[e], (uint32_t)e);
        }
    }
    lds_barrier();
    auto propose = [&] {
#pragma unroll
        for (int q = 0; q < kTailItems; ++q) {
            if (q >= per) break;
            if (alive & (1u << q)) {
                atomicMax(&best[uv[q] >> kNodeBits], rank[q]);
                atomicMax(&best[uv[q] & kNodeMask], rank[q]);
            }
        }
    };
    if (__ballot(alive != 0u) && tail_lane() == 0) any[0] = 1u;
    propose();
    for (int r = 0; r < cap; ++r) {
        lds_barrier();
        if (!any[r & 1]) break;      // uniform
        if (tid == 0) any[(r + 1) & 1] = 0u;
#pragma unroll
        for (int q = 0; q < kTailItems; ++q) {
            if (q >= per) break;
            if (alive & (1u << q)) {
                const uint32_t u = uv[q] >> kNodeBits, v = uv[q] & kNodeMask;
                if (best[u] == rank[q] && best[v] == rank[q]) {
                    mate[u] = (uint16_t)v; mate[v] = (uint16_t)u;
                    best[u] = kMatched; best[v] = kMatched;      // whoever reads it in this step has lost either way
                    ++made;
                }
            }
        }
        lds_barrier();
#pragma unroll
        for (int q = 0; q < kTailItems; ++q) {
            if (q >= per) break;
            if (alive & (1u << q)) {
                const uint32_t u = uv[q] >> kNodeBits, v = uv[q] & kNodeMask;
                if (best[u] == kMatched || best[v] == kMatched) alive &= ~(1u << q);
                else { best[u] = 0ull; best[v] = 0ull; }
            }
        }
        if (__ballot(alive != 0u) && tail_lane() == 0) any[(r + 1) & 1] = 1u;
        lds_barrier();
        propose();
    }
    uint32_t all;
    (void)tail_scan(made, &all, S.wave);
    return all;
}

// S by the spanning forest without conflicts; returns |S|, representatives (smallest node of the component of (V,S)) in
// work[kRep..)
__device__ __forceinline__ uint32_t tail_forest(TailShared &S, int n, int m, float tau)
{
    const int tid = (int)threadIdx.x;
    unsigned long long *best = reinterpret_cast<unsigned long long *>(S.work);
    uint16_t *comp = (uint16_t *)(S.work + kComp), *hook = (uint16_t *)(S.work + kHook);
    for (int v = tid; v < kTailNodes; v += kTailThreads) { comp[v] = (uint16_t)v; hook[v] = (uint16_t)v; best[v] = 0ull; }
    for (int k = tid; k < kTailEdges / 32; k += kTailThreads) { S.work[kInForest + k] = 0u; S.work[kRemoved + k] = 0u; }
    uint32_t alive = 0;
#pragma unroll
    for (int q = 0; q < kTailItems; ++q) {
        const int e = tid + q * kTailThreads;
        if (e < m && S.cost[e] > tau) alive |= 1u << q;
    }
    // Boruvka rounds; every one at least halves the number of components that have a candidate left
    for (int round = 0; round < 64; ++round) {
        if (!__syncthreads_or(alive != 0u)) break;
        for (int q = 0; q < kTailItems; ++q) {
            const int e = tid + q * kTailThreads;
            if (!(alive & (1u << q))) continue;
            const uint32_t cu = comp[S.key[e] >> kNodeBits], cv = comp[S.key[e] & kNodeMask];
            const unsigned long long r = edge_rank(S.cost[e], (uint32_t)e);
            atomicMax(&best[cu], r);
            atomicMax(&best[cv], r);
        }
        __syncthreads();
        for (int q = 0; q < kTailItems; ++q) {
            const int e = tid + q * kTailThreads;
            if (!(alive & (1u << q))) continue;
            const uint32_t cu = comp[S.key[e] >> kNodeBits], cv = comp[S.key[e] & kNodeMask];
            const unsigned long long r = edge_rank(S.cost[e], (uint32_t)e);
            const bool bu = best[cu] == r, bv = best[cv] == r;
            if (!(bu || bv)) continue;
            atomicOr(&S.work[kInForest + (e >> 5)], 1u << (e & 31));
            if (bu && !(bv && cu < cv)) hook[cu] = (uint16_t)cv;
            if (bv && !(bu && cv < cu)) hook[cv] = (uint16_t)cu;
        }
        __syncthreads();
        for (int v = tid; v < n; v += kTailThreads) {
            uint32_t r = comp[v], h = hook[r];
            while (h != r) { r = h; h = hook[r]; }      // the hook graph is a forest: every chain ends in a root
            comp[v] = (uint16_t)r;
        }
        __syncthreads();
        for (int v = tid; v < n; v += kTailThreads) { best[v] = 0ull; hook[v] = (uint16_t)v; }   // comp[] holds roots only
        for (int q = 0; q < kTailItems; ++q) {
            const int e = tid + q * kTailThreads;
            if ((alive & (1u << q)) && comp[S.key[e] >> kNodeBits] == comp[S.key[e] & kNodeMask]) alive &= ~(1u << q);
        }
    }
    // rooting at the component representatives, breadth first
    uint16_t *depth = (uint16_t *)(S.work + kDepth), *up = (uint16_t *)(S.work + kUp), *up_edge = (uint16_t *)(S.work + kUpEdge);
    for (int v = tid; v < n; v += kTailThreads) { depth[v] = comp[v] == v ? 0 : 0xffffu; up[v] = (uint16_t)v; }
    uint32_t tree = 0;      // own forest edges
#pragma unroll
    for (int q = 0; q < kTailItems; ++q) {
        const int e = tid + q * kTailThreads;
        if (e < m && (S.work[kInForest + (e >> 5)] >> (e & 31)) & 1u) tree |= 1u << q;
    }
    __syncthreads();
    for (uint32_t lvl = 0; lvl < (uint32_t)n; ++lvl) {      // the sweep behind the deepest level changes nothing
        bool changed = false;
        for (int q = 0; q < kTailItems; ++q) {
            if (!(tree & (1u << q))) continue;
            const int e = tid + q * kTailThreads;
            const uint32_t a = S.key[e] >> kNodeBits, b = S.key[e] & kNodeMask;
            const uint32_t da = depth[a], db = depth[b];
            // a tree: nobody else reaches the child on this level
            if (da == lvl && db == 0xffffu) { depth[b] = (uint16_t)(lvl + 1); up[b] = (uint16_t)a; up_edge[b] = (uint16_t)e; changed = true; }
            else if (db == lvl && da == 0xffffu) { depth[a] = (uint16_t)(lvl + 1); up[a] = (uint16_t)b; up_edge[a] = (uint16_t)e; changed = true; }
        }
        if (!__syncthreads_or(changed)) break;
    }
    for (int q = 0; q < kTailItems; ++q) {      // the lowest edge on the tree path of every repulsive edge
        const int e = tid + q * kTailThreads;
        if (e >= m || !(S.cost[e] < 0.0f)) continue;
        uint32_t a = S.key[e] >> kNodeBits, b = S.key[e] & kNodeMask;
        if (comp[a] != comp[b]) continue;
        uint32_t da = depth[a], db = depth[b], low_e = 0;
        unsigned long long low = ~0ull;
        while (a != b) {
            uint32_t pe;
            if (da >= db) { pe = up_edge[a]; a = up[a]; --da; } else { pe = up_edge[b]; b = up[b]; --db; }
            const unsigned long long r = edge_rank(S.cost[pe], pe);
            if (r < low) { low = r; low_e = pe; }
        }
        if (low != ~0ull) atomicOr(&S.work[kRemoved + (low_e >> 5)], 1u << (low_e & 31));
    }
    __syncthreads();
    uint32_t kept = 0;
    for (int q = 0; q < kTailItems; ++q) {
        const int e = tid + q * kTailThreads;
        if ((tree & (1u << q)) && (S.work[kRemoved + (e >> 5)] >> (e & 31)) & 1u) tree &= ~(1u << q);
        kept += (tree >> q) & 1u;
    }
    uint32_t all;
    (void)tail_scan(kept, &all, S.wave);
    // components: hooking of the larger root onto the smaller until nothing changes (see k_forest_components)
    uint32_t *rep = S.work + kRep;
    for (int v = tid; v < n; v += kTailThreads) rep[v] = (uint32_t)v;
    __syncthreads();
    for (;;) {
        bool changed = false;
        for (int q = 0; q < kTailItems; ++q) {
            if (!(tree & (1u << q))) continue;
            const uint32_t k = S.key[tid + q * kTailThreads];
            uint32_t a = k >> kNodeBits, b = k & kNodeMask;
            for (uint32_t p = rep[a]; p != a; p = rep[a]) a = p;
            for (uint32_t p = rep[b]; p != b; p = rep[b]) b = p;
            if (a != b) { atomicMin(&rep[max(a, b)], min(a, b)); changed = true; }
        }
        if (!__syncthreads_or(changed)) break;
    }
    for (int v = tid; v < n; v += kTailThreads) {
        uint32_t r = rep[v];
        for (uint32_t p = rep[r]; p != r; p = rep[r]) r = p;
        rep[v] = r;      // a shorter way to the same root: no walk of another thread goes wrong
    }
    __syncthreads();
    return all;
}

__global__ __launch_bounds__(kTailThreads) void k_tail_rounds(TailArgs A)
{
    __shared__ TailShared S;
    const int tid = (int)threadIdx.x, lane = tail_lane(), w = tail_wave();
    int n = A.n, m = A.m;
    for (int e = tid; e < m; e += kTailThreads) {
        S.key[e] = (uint32_t)A.i[e] << kNodeBits | (uint32_t)A.j[e];
        S.cost[e] = A.c[e];
    }
    for (int v = tid; v < A.n; v += kTailThreads) A.fmap[v] = v;
    __syncthreads();
    MailWord *rec = A.mail + 3;
    uint32_t status = kTailMore, rounds = 0;
    while (rounds < (uint32_t)A.max_rounds) {
        const uint64_t t0 = wall_clock64();
        uint32_t T = 0, n_attractive = 0, n_repulsive = 0;
        if (A.separate) T = tail_triangles(S, n, m, n_attractive, n_repulsive);
        if (T > (uint32_t)kTailTriangles) { status = kTailTooMany; break; }
        const uint64_t t1 = wall_clock64();
        if (T) tail_messages(S, m, T, A.iters);
        const uint64_t t2 = wall_clock64();
        uint32_t ns = tail_matching(S, n, m, A.tau, A.cap);
        bool forest = false;
        uint32_t *rep = S.work + kRep;
        uint16_t *fnew = (uint16_t *)(S.work + kNew);
        if (ns && A.forest_ratio > 0.0f && (double)ns < (double)A.forest_ratio * (double)n) {
            forest = true;
            ns = tail_forest(S, n, m, A.tau);
        } else if (ns) {
            const uint16_t *mate = (const uint16_t *)(S.work + kMate);
            for (int v = tid; v < n; v += kTailThreads) rep[v] = mate[v] < v ? mate[v] : (uint32_t)v;
            __syncthreads();
        }
        const int n_old = n, m_old = m;
        if (ns) {
            // new numbers: ranks of the representatives
            uint32_t root = 0, n_new;
            const int per_node = tail_per_thread(n);
#pragma unroll
            for (int q = 0; q < kTailNodeItems; ++q) {
                if (q >= per_node) break;
                const int v = tid * per_node + q;
                root += v < n && rep[v] == (uint32_t)v ? 1u : 0u;
            }
            uint32_t run = tail_scan(root, &n_new, S.wave);
#pragma unroll
            for (int q = 0; q < kTailNodeItems; ++q) {
                if (q >= per_node) break;
                const int v = tid * per_node + q;
                if (v < n && rep[v] == (uint32_t)v) fnew[v] = (uint16_t)run++;
            }
            lds_barrier();
            for (int v = tid; v < n; v += kTailThreads)
                if (rep[v] != (uint32_t)v) fnew[v] = fnew[rep[v]];
            lds_barrier();
            for (int v = tid; v < A.n; v += kTailThreads) A.fmap[v] = fnew[A.fmap[v]];   // always the same thread's entries
            // relabelled edges without the loops, sorted, runs summed in order
            const int nb = tail_bits(n_new);
            const uint32_t fmask = (1u << nb) - 1u, loop_key = 0xffffffffu >> (32 - 2 * nb);
            const uint32_t rows = ((uint32_t)m + kTailThreads - 1) / kTailThreads, base = (uint32_t)w * rows * 64u + (uint32_t)lane;
            uint32_t key[kTailItems] = {}, val[kTailItems] = {}, stays = 0, kept;      // bit r: edge r stays
#pragma unroll
            for (int r = 0; r < kTailItems; ++r) {
                const uint32_t e = base + (uint32_t)r * 64u;
                if ((uint32_t)r < rows && e < (uint32_t)m) {
                    const uint32_t a = fnew[S.key[e] >> kNodeBits], b = fnew[S.key[e] & kNodeMask];
                    key[r] = a == b ? loop_key : min(a, b) << nb | max(a, b);
                    val[r] = __float_as_uint(S.cost[e]);
                    stays |= a != b ? 1u << r : 0u;
                }
            }
            (void)tail_scan((uint32_t)__popc(stays), &kept, S.wave);
            if (!tail_bucket_sort(S, key, val, stays, (int)rows, base, 2 * nb)) tail_sort(S, key, val, (uint32_t)m, 2 * nb);      // loops come last
            const uint32_t *skey = S.work, *sval = S.work + kSortVal;
            uint32_t heads = 0, place[kTailItems], carry = 0;
#pragma unroll
            for (int r = 0; r < kTailItems; ++r) {
                const uint32_t p = base + (uint32_t)r * 64u;
                const bool head = (uint32_t)r < rows && p < kept && (p == 0 || skey[p] != skey[p - 1]);
                const uint64_t vote = __ballot(head);
                place[r] = carry + (uint32_t)__popcll(vote & ((1ull << lane) - 1ull));
                carry += (uint32_t)__popcll(vote);
                heads |= head ? 1u << r : 0u;
            }
            uint32_t m_new;
            const uint32_t first = tail_scan(lane == 0 ? carry : 0u, &m_new, S.wave);
            const uint32_t before = (uint32_t)__builtin_amdgcn_readfirstlane((int)first);      // heads of the waves in front
#pragma unroll
            for (int r = 0; r < kTailItems; ++r)
                if (heads & (1u << r)) {
                    uint32_t p = base + (uint32_t)r * 64u;
                    const uint32_t k = skey[p];
                    float acc = __uint_as_float(sval[p]);
                    for (++p; p < kept && skey[p] == k; ++p) acc = acc + __uint_as_float(sval[p]);
                    S.key[before + place[r]] = (k >> nb) << kNodeBits | (k & fmask);
                    S.cost[before + place[r]] = acc;
                }
            __syncthreads();
            n = (int)n_new; m = (int)m_new;
        }
        if (tid == 0) {
            const uint64_t t3 = wall_clock64();
            mail_put(rec + 0, (uint64_t)(uint32_t)n_old | (uint64_t)(uint32_t)m_old << 32);
            mail_put(rec + 1, (uint64_t)n_attractive | (uint64_t)n_repulsive << 32);
            mail_put(rec + 2, (uint64_t)T | (uint64_t)(forest ? 1u : 0u) << 32);
            mail_put(rec + 3, (uint64_t)ns);
            mail_put(rec + 4, (uint64_t)(uint32_t)(t1 - t0) | (uint64_t)(uint32_t)(t2 - t1) << 32);
            mail_put(rec + 5, (uint64_t)(t3 - t2));
        }
        rec += kTailRecord;
        ++rounds;
        if (ns == 0) { status = kTailDone; break; }
    }
    for (int e = tid; e < m; e += kTailThreads) {
        A.io[e] = (int32_t)(S.key[e] >> kNodeBits);
        A.jo[e] = (int32_t)(S.key[e] & kNodeMask);
        A.co[e] = S.cost[e];
    }
    if (tid == 0) {
        mail_put(A.mail + 1, (uint64_t)status | (uint64_t)rounds << 32);
        mail_put(A.mail + 2, (uint64_t)(uint32_t)n | (uint64_t)(uint32_t)m << 32);
    }
    mail_send(A.mail, A.seq);
}

}  // namespace

rama_status tail_rounds(Ctx &ctx, const Graph &g, Graph &out, bool separate, int k_iters, float tau, int rounds_cap,
                        float forest_ratio, int max_rounds, Buf<int32_t> &fmap, TailResult &res)
{
    if (!tail_fits(g)) return fail(ctx, RAMA_ERR_INVALID_ARG, "tail_rounds: graph too large");
    RAMA_TRY(fmap.alloc(ctx, (size_t)(g.n > 0 ? g.n : 1)));
    static_assert(3 + kTailMaxRounds * kTailRecord <= (int)Ctx::kMailWords, "a record per round in one message");
    if (max_rounds <= 0 || max_rounds > kTailMaxRounds) max_rounds = kTailMaxRounds;
    const uint64_t seq = ++ctx.mail_seq;
    {
        ProfScope ps_(ctx, "k_tail_rounds", (double)((size_t)g.m * 24 + (size_t)g.n * 4));
        k_tail_rounds<<<1, kTailThreads, 0, ctx.stream>>>(TailArgs{g.n, (int32_t)g.m, g.i.get(), g.j.get(), g.c.get(), out.i.get(), out.j.get(),
                                                                  out.c.get(), fmap.get(), separate ? 1 : 0, k_iters, rounds_cap > 0 ? rounds_cap : 0,
                                                                  max_rounds, tau, forest_ratio, mailbox(ctx), seq});
    }
    LAUNCH_TRY(ctx, "tail_rounds");
    RAMA_TRY(wait_mail(ctx, seq));
    const volatile uint64_t *mail = mail_words(ctx);
    auto lo = [](uint64_t x) { return (int64_t)(uint32_t)x; };
    auto hi = [](uint64_t x) { return (int64_t)(x >> 32); };
    res.status = (int)lo(mail[1]);
    res.rounds.clear();
    for (int r = 0; r < (int)hi(mail[1]); ++r) {
        const volatile uint64_t *w = mail + 3 + r * kTailRecord;
        rama_round_stats R;
        memset(&R, 0, sizeof R);
        R.n_nodes = (int32_t)lo(w[0]); R.n_edges = hi(w[0]); R.n_edges_aug = hi(w[0]);
        R.n_attractive = separate ? lo(w[1]) : -1; R.n_repulsive = separate ? hi(w[1]) : -1;
        R.n_cycles[0] = lo(w[2]); R.n_triangles = lo(w[2]); R.used_forest = (int32_t)hi(w[2]);
        R.n_contracted = lo(w[3]);
        R.ms_cycles = (double)lo(w[4]) / ctx.wall_khz; R.ms_dual = (double)hi(w[4]) / ctx.wall_khz;
        R.ms_contract = (double)w[5] / ctx.wall_khz;
        res.rounds.push_back(R);
    }
    out.n = (int32_t)lo(mail[2]);
    out.m = hi(mail[2]);
    out.sign_sums.reset();
    return RAMA_OK;
}

}  // namespace rama
