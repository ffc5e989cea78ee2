// Step a1: conflicted-cycle separation (paper Sec. 3.2.2, definition "Conflicted cycles" and the
// lemma on searching per repulsive edge; appendix algorithm "Parallel Conf. 5-Cycles").
//
// For every repulsive edge (v0,vL), v0<vL, all attractive simple paths of 2, 3 and 4 hops
// between its endpoints are enumerated on the positive neighbourhoods N+ held as a CSR with
// ascending rows:
//   3-cycles: v1 in N+(v0) & N+(vL)
//   4-cycles: v1 in N+(v0), v2 in N+(v1) & N+(vL)
//   5-cycles: v1 in N+(v0), v2 in N+(v1), v3 in N+(v2) & N+(vL); the same set as the appendix
//             algorithm's pairs (v1,v3) in N+(v0) x N+(vL) with common neighbour v2
// A count pass, a scan and a fill pass produce the lists already in their final order
// (v0, vL, then the path v1, v2, v3), because repulsive edges are visited in canonical order
// and every row is ascending.
#include "prim.h"
#include "steps.h"

namespace rama {

namespace {

// consumer of the scan over SignFlags: an attractive edge goes to place low(prefix) of the attractive
// list (the lower half of the adjacency is sorted from its pairs read as (j,i)), a repulsive one
// to place high(prefix) of the repulsive list
struct SplitSignEmit {
    static constexpr const char *tag = "SplitSign";
    const int32_t *i, *j;
    int32_t *pi, *pj;
    int32_t *ri, *rj;
    struct Item { int32_t a, b; };
    __device__ __forceinline__ Item load(size_t e) const { return {i[e], j[e]}; }
    __device__ __forceinline__ void operator()(size_t, uint64_t sign, uint64_t prefix, const Item &x) const
    {
        if (sign == 0) return;
        if (sign == 1ull) {
            const uint32_t p = (uint32_t)prefix;
            pi[p] = x.a; pj[p] = x.b;
        } else {
            const uint32_t p = (uint32_t)(prefix >> 32);
            ri[p] = x.a; rj[p] = x.b;
        }
    }
};

// row pointers of N+ = lower + upper part; *longest (optional) collects the longest row
__global__ __launch_bounds__(kBlock) void k_add_ptr(int32_t n, const int32_t *a, const int32_t *b, int32_t *out,
                                                    uint32_t *longest)
{
    int32_t v = blockIdx.x * kBlock + threadIdx.x;
    if (v <= n) out[v] = a[v] + b[v];
    if (longest) block_max_into(v < n ? (uint32_t)((a[v + 1] - a[v]) + (b[v + 1] - b[v])) : 0u, longest);
}

// row v of N+ = [lower neighbours u<v, ascending][upper neighbours w>v, ascending]
__global__ __launch_bounds__(kBlock) void k_fill_adj(size_t mp, const int32_t *pi, const int32_t *pj,
                                                     const uint32_t *lj, const uint32_t *li, const int32_t *up_ptr,
                                                     const int32_t *low_ptr, const int32_t *rowptr, int32_t *nb)
{
    size_t e = (size_t)blockIdx.x * kBlock + threadIdx.x;
    if (e >= mp) return;
    {   // upper entry of edge e: row pi[e]
        int32_t u = pi[e];
        int32_t lowdeg = low_ptr[u + 1] - low_ptr[u];
        nb[rowptr[u] + lowdeg + ((int32_t)e - up_ptr[u])] = pj[e];
    }
    {   // lower entry at sorted position e: row lj[e]
        int32_t v = (int32_t)lj[e];
        nb[rowptr[v] + ((int32_t)e - low_ptr[v])] = (int32_t)li[e];
    }
}

struct Adj {
    const int32_t *ptr;
    const int32_t *nb;
};

// both rows (at most N entries each) are fetched whole with 16-byte loads -- one wait instead of a
// chain of dependent probes -- and compared in registers; f is called for the common entries in
// ascending order.  The array is padded by kWideRow entries; what lies behind a row's end is masked out.
template <int N, typename F>
__device__ __forceinline__ void intersect_in_registers(const Adj &g, int32_t a0, int32_t a1, int32_t b0, int32_t b1, F &&f)
{
    int32_t ra[N], rb[N];
    __builtin_memcpy(ra, g.nb + a0, sizeof(ra));
    __builtin_memcpy(rb, g.nb + b0, sizeof(rb));
#pragma unroll
    for (int k = 0; k < N; ++k) {
        ra[k] = a0 + k < a1 ? ra[k] : -1;
        rb[k] = b0 + k < b1 ? rb[k] : -2;
    }
#pragma unroll
    for (int k = 0; k < N; ++k) {
        bool hit = false;
#pragma unroll
        for (int q = 0; q < N; ++q) hit |= (ra[k] == rb[q]);
        if (hit) f(ra[k]);
    }
}

// calls f(x) for every x in row a & row b, ascending.  Rows of up to kWideRow entries -- nearly all
// rows of the contracted graphs -- are compared in registers; longer ones: walk the shorter row,
// bisect the longer (a chain of dependent loads: measured, this fallback used to take half of the
// triangle search's time when it started at nine entries).
constexpr int kShortRow = 8;
constexpr int kWideRow = 16;
template <typename F>
__device__ __forceinline__ void intersect_rows(const Adj &g, int32_t a, int32_t b, F &&f)
{
    int32_t a0 = g.ptr[a], a1 = g.ptr[a + 1], b0 = g.ptr[b], b1 = g.ptr[b + 1];
    if (a0 == a1 || b0 == b1) return;
    if (a1 - a0 <= kShortRow && b1 - b0 <= kShortRow) {
        intersect_in_registers<kShortRow>(g, a0, a1, b0, b1, f);
        return;
    }
    if (a1 - a0 <= kWideRow && b1 - b0 <= kWideRow) {
        intersect_in_registers<kWideRow>(g, a0, a1, b0, b1, f);
        return;
    }
    if (a1 - a0 > b1 - b0) { int32_t t = a0; a0 = b0; b0 = t; t = a1; a1 = b1; b1 = t; }
    for (int32_t p = a0; p < a1 && b0 < b1; ++p) {
        int32_t x = g.nb[p];
        int32_t lo = b0, hi = b1;
        while (lo < hi) {
            int32_t mid = lo + ((hi - lo) >> 1);
            if (g.nb[mid] < x) lo = mid + 1; else hi = mid;
        }
        b0 = lo;
        if (lo < b1 && g.nb[lo] == x) { f(x); b0 = lo + 1; }
    }
}

// N+(vL) of the repulsive edge under work: kept in registers when it has at most 8 entries
// (always the case on grid-like inputs), otherwise searched in memory
constexpr int kRowRegs = 8;
struct EndRow {
    int32_t r[kRowRegs];
    int32_t b0, b1;
    const int32_t *nb;
    bool in_regs;
    // The rows of the entries, for closing the last hop from vL's side (the appendix algorithm's meeting
    // in the middle): the walk is at its last inner node `tail`, and instead of fetching N+(tail) and
    // testing its entries against N+(vL), every entry v of N+(vL) tests whether tail is in N+(v).  These
    // rows are the same for the whole search of one repulsive edge, so they are fetched once, where the
    // walk would fetch one row per path that reaches its last level.
    int32_t rows[kRowRegs][kRowRegs];
    bool rows_ok;   // N+(vL) and the rows of all its entries have at most kRowRegs entries and are loaded
    __device__ __forceinline__ void load(const Adj &g, int32_t vl)
    {
        nb = g.nb; b0 = g.ptr[vl]; b1 = g.ptr[vl + 1];
        in_regs = (b1 - b0) <= kRowRegs;
        rows_ok = false;
#pragma unroll
        for (int k = 0; k < kRowRegs; ++k) r[k] = (in_regs && b0 + k < b1) ? nb[b0 + k] : -1;
    }
    __device__ __forceinline__ void load_rows(const Adj &g)
    {
        bool ok = in_regs;
        int32_t p0[kRowRegs], p1[kRowRegs];
#pragma unroll
        for (int k = 0; k < kRowRegs; ++k) {
            p0[k] = 0; p1[k] = 0;
            if (r[k] >= 0) { p0[k] = g.ptr[r[k]]; p1[k] = g.ptr[r[k] + 1]; }
            ok &= (p1[k] - p0[k]) <= kRowRegs;
        }
#pragma unroll
        for (int k = 0; k < kRowRegs; ++k) {
            // two 16-byte loads per row (the array is padded); what lies behind the row's end becomes -1
            int32_t row[kRowRegs];
            __builtin_memcpy(row, nb + p0[k], sizeof(row));
#pragma unroll
            for (int q = 0; q < kRowRegs; ++q) rows[k][q] = (ok && p0[k] + q < p1[k]) ? row[q] : -1;
        }
        rows_ok = ok;
    }
    // entry k of N+(vL) has `x` in its row
    __device__ __forceinline__ bool row_has(int k, int32_t x) const
    {
        bool f = false;
#pragma unroll
        for (int q = 0; q < kRowRegs; ++q) f |= (rows[k][q] == x);
        return f;
    }
    __device__ __forceinline__ bool has(int32_t x) const
    {
        if (in_regs) {
            bool f = false;
#pragma unroll
            for (int k = 0; k < kRowRegs; ++k) f |= (r[k] == x);
            return f;
        }
        int32_t lo = b0, hi = b1;
        while (lo < hi) {
            int32_t mid = lo + ((hi - lo) >> 1);
            if (nb[mid] < x) lo = mid + 1; else hi = mid;
        }
        return lo < b1 && nb[lo] == x;
    }
};

// Depth-first walk v0 -> v1 -> v2 -> ... along N+, closing on N+(vL) at every depth: a node v_K
// reached over K attractive hops that lies in N+(vL) closes the (K+2)-cycle (v0,..,v_K,vL).  For
// length 5 these are the appendix algorithm's pairs (v1,v3) with common neighbour v2, visited
// path-first.  vL and v0 are never in N+(vL) / N+(v0) of a repulsive edge and a row never holds its
// own node, so a closing node only has to differ from the inner path nodes; a node the walk
// continues through must also differ from v0 and vL.  Rows are ascending, so every list comes out
// in path order.  The recursion is over a compile-time depth: it unrolls into nested loops with
// the path in registers.
// [r0, r1) is the row of path[K-1]: the level above fetched the bounds while it was still busy with
// the previous neighbour, so that a level does not start with a load it has to wait for.
template <int K, int MAXL, typename Emit>
__device__ __forceinline__ void extend_path(const Adj &g, const EndRow &end, int32_t vl, int max_len,
                                            int32_t (&path)[MAXL], Emit &emit, int32_t r0, int32_t r1)
{
    if constexpr (K >= 3) {
        if (K + 3 > max_len && end.rows_ok) {
            // Last level, met from vL's side: no row of the tail is fetched at all.  N+(vL) is ascending,
            // so the closing nodes come in the same order as from the tail's row.
            const int32_t tail = path[K - 1];
#pragma unroll
            for (int k = 0; k < kRowRegs; ++k) {
                const int32_t v = end.r[k];
                bool inner = false;
#pragma unroll
                for (int q = 1; q < K - 1; ++q) inner |= (path[q] == v);
                if (v >= 0 && !inner && end.row_has(k, tail)) { path[K] = v; emit.template cycle<K + 2>(path); }
            }
            return;
        }
    }
    if (K + 3 > max_len && r1 - r0 <= kShortRow) {
        // Last level (nothing continues below) and a short row: its entries come in with two 16-byte
        // loads instead of one dependent load per turn of a loop -- the walk spends most of its time
        // waiting for exactly these loads.  (The array is padded; entries behind the row's end are skipped.)
        int32_t row[kShortRow];
        __builtin_memcpy(row, g.nb + r0, sizeof(row));
#pragma unroll
        for (int k = 0; k < kShortRow; ++k) {
            if (r0 + k < r1) {
                const int32_t v = row[k];
                bool inner = false;
#pragma unroll
                for (int q = 1; q < K - 1; ++q) inner |= (path[q] == v);
                if (!inner && end.has(v)) { path[K] = v; emit.template cycle<K + 2>(path); }
            }
        }
        return;
    }
    // the level below needs its row's bounds -- unless it is the last one and closes from vL's side
    const bool deeper = (K + 3 <= MAXL) && (K + 3 <= max_len) && !(K >= 2 && K + 4 > max_len && end.rows_ok);
    int32_t vn = r0 < r1 ? g.nb[r0] : 0, n0 = 0, n1 = 0;      // the neighbour of the coming turn and its row
    if (deeper && r0 < r1) { n0 = g.ptr[vn]; n1 = g.ptr[vn + 1]; }
    for (int32_t p = r0; p < r1; ++p) {
        const int32_t v = vn, c0 = n0, c1 = n1;
        if (p + 1 < r1) {
            vn = g.nb[p + 1];
            if (deeper) { n0 = g.ptr[vn]; n1 = g.ptr[vn + 1]; }
        }
        bool inner = false;
#pragma unroll
        for (int q = 1; q < K - 1; ++q) inner |= (path[q] == v);
        if (inner) continue;
        if (end.has(v)) { path[K] = v; emit.template cycle<K + 2>(path); }
        if constexpr (K + 3 <= MAXL) {
            if (K + 3 > max_len || v == vl || v == path[0]) continue;
            path[K] = v;
            extend_path<K + 1, MAXL>(g, end, vl, max_len, path, emit, c0, c1);
        }
    }
}
template <int K, int MAXL, typename Emit>
__device__ __forceinline__ void extend_path(const Adj &g, const EndRow &end, int32_t vl, int max_len,
                                            int32_t (&path)[MAXL], Emit &emit)
{
    const int32_t tail = path[K - 1];
    extend_path<K, MAXL>(g, end, vl, max_len, path, emit, g.ptr[tail], g.ptr[tail + 1]);
}

template <int MAXL, bool MEET = false, typename Emit>
__device__ __forceinline__ void enumerate_cycles(const Adj &g, int32_t v0, int32_t vl, int max_len, Emit &emit)
{
    int32_t path[MAXL];
    path[0] = v0;
    if (max_len <= 3) {
        intersect_rows(g, v0, vl, [&](int32_t v1) { path[1] = v1; emit.template cycle<3>(path); });
        return;
    }
    EndRow end;
    end.load(g, vl);
    if (end.b0 == end.b1) return;
    if constexpr (MEET)
        if (max_len >= 5) end.load_rows(g);   // the last level (three or more hops from v0) closes from vL's side
    extend_path<1, MAXL>(g, end, vl, max_len, path, emit);
}

// the walk below one given first hop v1 (what the walk from v0 does for each entry of its row)
template <int MAXL, typename Emit>
__device__ __forceinline__ void walk_from_first(const Adj &g, const EndRow &end, int32_t v0, int32_t v1, int32_t vl,
                                                int max_len, Emit &emit)
{
    int32_t path[MAXL];
    path[0] = v0; path[1] = v1;
    if (end.has(v1)) emit.template cycle<3>(path);
    if constexpr (MAXL >= 4)
        if (max_len >= 4) extend_path<2, MAXL>(g, end, vl, max_len, path, emit);
}

// A repulsive edge whose first endpoint has a long attractive row is "heavy": one thread would walk
// the whole row alone while its wave waits.  The per-thread kernels put such edges on a list
// instead, and a second kernel gives each listed edge to a whole wave, one first hop per lane.
// (Walks of length 3 are row intersections and stay with the per-thread kernels.)
constexpr size_t kListHitsFrom = size_t(1) << 17;
constexpr int kHeavyRow = 128;
constexpr unsigned kHeavyGroups = 512;
constexpr unsigned kSpillGroups = 768;     // three workgroups per CU: what their LDS allows
constexpr int kWalkRow = 16;               // see WalkList
constexpr uint32_t kWalkFrom = 4096;
static_assert(kWalkRow <= kHeavyRow, "what is walked by a thread is not heavy");
__device__ __forceinline__ bool heavy_edge(const Adj &g, int32_t v0, int max_len)
{
    return max_len >= 4 && g.ptr[v0 + 1] - g.ptr[v0] > kHeavyRow;
}

template <int MAXL>
struct CountEmit {
    uint32_t n[MAXL - 2];
    __device__ __forceinline__ void clear()
    {
#pragma unroll
        for (int k = 0; k < MAXL - 2; ++k) n[k] = 0;
    }
    template <int L>
    __device__ __forceinline__ void cycle(const int32_t (&)[MAXL])
    {
        n[L - 3] += (n[L - 3] != 0xffffffffu);   // saturates; the host reports it
    }
};

template <int MAXL>
struct FillEmit {
    int32_t vl;
    int32_t *o[MAXL - 2];
    template <int L>
    __device__ __forceinline__ void cycle(const int32_t (&path)[MAXL])
    {
        int32_t *w = o[L - 3];
#pragma unroll
        for (int q = 0; q < L - 1; ++q) w[q] = path[q];
        w[L - 1] = vl;
        o[L - 3] = w + L;
    }
};

// per-list arrays of one repulsive-edge table: list k (the (k+3)-cycles) starts at k*stride
template <typename T, int N>
struct ListPtrs {
    T *p[N];
};

// counts per repulsive edge and length.  shortest_only: deepen the walk one length at a time
// and stop at the first length that closes a cycle (the hop distance in (V,E+) plus one); only
// that length's count is kept.  All lanes of a wave call this together; `valid` says whether the
// lane has an edge r.
template <int MAXL, bool MEET>
__device__ __forceinline__ void count_edge(bool valid, size_t r, const int32_t *ri, const int32_t *rj, const Adj &g,
                                           int max_len, int flags, const ListPtrs<uint32_t, MAXL - 2> &cnt,
                                           uint32_t *heavy, uint32_t *n_heavy, uint32_t *saturated)
{
    const bool shortest_only = flags != 0;
    const bool is_heavy = valid && heavy_edge(g, ri[r], max_len);
    const unsigned long long vote = __ballot(is_heavy);
    if (vote) {   // the wave's heavy edges join the list with one atomic
        const int lane = (int)(threadIdx.x & 63);
        uint32_t base = 0;
        if (lane == __ffsll((long long)vote) - 1) base = atomicAdd(n_heavy, (uint32_t)__popcll(vote));
        base = (uint32_t)__shfl((int)base, __ffsll((long long)vote) - 1, 64);
        if (is_heavy) heavy[base + (uint32_t)__popcll(vote & ((1ull << lane) - 1ull))] = (uint32_t)r;
    }
    if (!valid || is_heavy) return;
    CountEmit<MAXL> em;
    em.clear();
    if (!shortest_only) {
        enumerate_cycles<MAXL, MEET>(g, ri[r], rj[r], max_len, em);
    } else {
        for (int L = 3; L <= max_len; ++L) {
            em.clear();
            enumerate_cycles<MAXL, MEET>(g, ri[r], rj[r], L, em);
            uint32_t any = 0;   // only length L can have closed: shorter ones were tried before
#pragma unroll
            for (int k = 0; k < MAXL - 2; ++k) any |= em.n[k];
            if (any) break;
        }
    }
    bool sat = false;
#pragma unroll
    for (int k = 0; k < MAXL - 2; ++k)
        if (k + 3 <= max_len) { cnt.p[k][r] = em.n[k]; sat |= (em.n[k] == 0xffffffffu); }
    if (sat) *saturated = 1u;   // a count that reached 2^32-1 may have lost cycles: the host turns this into an error
}

template <int MAXL, bool MEET>
__global__ __launch_bounds__(kBlock) void k_count_cycles(size_t nr, const int32_t *ri, const int32_t *rj, Adj g,
                                                         int max_len, int flags,
                                                         ListPtrs<uint32_t, MAXL - 2> cnt, uint32_t *heavy,
                                                         uint32_t *n_heavy, uint32_t *saturated)
{
    const size_t r = (size_t)blockIdx.x * kBlock + threadIdx.x;
    count_edge<MAXL, MEET>(r < nr, r, ri, rj, g, max_len, flags, cnt, heavy, n_heavy, saturated);
}

// ---- counts up to length 5 on graphs all of whose attractive rows have at most R entries -----------
// The walk with its last level closed from vL's side, written out for rows that are known to be short: every row comes
// in whole by 16-byte loads that do not wait for each other (the bounds of all first hops' rows at once, the row of the
// coming v1 while this one is worked on), where the walk above fetches entry after entry, and R fixes how many
// comparisons a pair (v1,v2) costs.  What bounds it: those R*R comparisons for each of up to R*R pairs.  320^3 grid (3.1e7
// repulsive edges): 4.4 ms for the walk, 2.2 here.
template <int R>
__global__ __launch_bounds__(kBlock) void k_count_cycles_short(size_t nr, const int32_t *ri, const int32_t *rj, Adj g, ListPtrs<uint32_t, 3> cnt)
{
    const size_t r = (size_t)blockIdx.x * kBlock + threadIdx.x;
    if (r >= nr) return;
    const int32_t v0 = ri[r], vl = rj[r];
    const int32_t a0 = g.ptr[v0], a1 = g.ptr[v0 + 1], b0 = g.ptr[vl], b1 = g.ptr[vl + 1];
    uint32_t n3 = 0, n4 = 0, n5 = 0;
    if (a0 < a1 && b0 < b1) {
        int32_t ra[R], rb[R], pa0[R], pa1[R], rows[R][R];
        __builtin_memcpy(ra, g.nb + a0, sizeof(ra));      // the array is padded; what lies behind a row's end becomes -1, -2
        __builtin_memcpy(rb, g.nb + b0, sizeof(rb));
#pragma unroll
        for (int k = 0; k < R; ++k) {
            ra[k] = a0 + k < a1 ? ra[k] : -1;
            rb[k] = b0 + k < b1 ? rb[k] : -2;
        }
#pragma unroll
        for (int k = 0; k < R; ++k) {
            int32_t p0 = 0, p1 = 0;
            pa0[k] = 0; pa1[k] = 0;
            if (ra[k] >= 0) { pa0[k] = g.ptr[ra[k]]; pa1[k] = g.ptr[ra[k] + 1]; }
            if (rb[k] >= 0) { p0 = g.ptr[rb[k]]; p1 = g.ptr[rb[k] + 1]; }
            int32_t row[R];
            __builtin_memcpy(row, g.nb + p0, sizeof(row));
#pragma unroll
            for (int q = 0; q < R; ++q) rows[k][q] = p0 + q < p1 ? row[q] : -2;
        }
        int32_t coming[R];
        __builtin_memcpy(coming, g.nb + pa0[0], sizeof(coming));
#pragma unroll
        for (int a = 0; a < R; ++a) {
            int32_t row[R];
#pragma unroll
            for (int q = 0; q < R; ++q) row[q] = pa0[a] + q < pa1[a] ? coming[q] : -1;
            if (a + 1 < R) __builtin_memcpy(coming, g.nb + pa0[a + 1 < R ? a + 1 : a], sizeof(coming));
            const int32_t v1 = ra[a];
            if (v1 < 0) continue;
#pragma unroll
            for (int k = 0; k < R; ++k) n3 += rb[k] == v1 ? 1u : 0u;
#pragma unroll
            for (int q = 0; q < R; ++q) {
                const int32_t v2 = row[q];
                if (v2 < 0 || v2 == v0) continue;
#pragma unroll
                for (int k = 0; k < R; ++k) n4 += rb[k] == v2 ? 1u : 0u;
                if (v2 == vl) continue;
#pragma unroll
                for (int k = 0; k < R; ++k) {
                    bool hit = false;
#pragma unroll
                    for (int x = 0; x < R; ++x) hit |= rows[k][x] == v2;
                    n5 += hit && rb[k] != v1 ? 1u : 0u;
                }
            }
        }
    }
    cnt.p[0][r] = n3; cnt.p[1][r] = n4; cnt.p[2][r] = n5;
}

// Edges the hashed search has no room for.  Those whose v0 has few attractive neighbours (up to kWalkRow) leave most of a
// wave idle: when there are many of them (kWalkFrom) they are walked by a thread each, in front of the heavy ones.
// Separation up to length 5, ms, wave per edge | thread per edge: leaves of a star, 10^5 edges with one neighbour 2718 | 43;
// leaves of eight hubs, four neighbours, 36000 edges 236 | 28; of 32 hubs, sixteen neighbours, 60000 edges 114 | 73, 2000
// edges 44 | 520; skewed degrees (10^4 nodes, few such edges) 12.5 | 46; of 64 hubs, 32 neighbours, 30000 edges 77 | 183.
// They stand at the back of the heavy edges' array: entry q is last[-q].
struct WalkList {
    uint32_t *last = nullptr, *n = nullptr;
    __device__ __forceinline__ uint32_t by_threads() const { return n && *n >= kWalkFrom ? *n : 0u; }
    __device__ __forceinline__ uint32_t by_waves() const { return n && *n < kWalkFrom ? *n : 0u; }
    __device__ __forceinline__ uint32_t operator[](size_t q) const { return *(last - q); }
};
// the counts of the listed edges that are walked by a thread each (fixed grid, every workgroup strides over the list)
template <int MAXL, bool MEET>
__global__ __launch_bounds__(kBlock) void k_count_cycles_listed(WalkList list, const int32_t *ri, const int32_t *rj, Adj g, int max_len,
                                                                int flags, ListPtrs<uint32_t, MAXL - 2> cnt, uint32_t *saturated)
{
    const size_t n = list.by_threads();
    for (size_t base = (size_t)blockIdx.x * kBlock; base < n; base += (size_t)gridDim.x * kBlock) {
        const size_t q = base + threadIdx.x;
        const bool valid = q < n;
        count_edge<MAXL, MEET>(valid, valid ? list[q] : 0, ri, rj, g, max_len, flags, cnt, nullptr, nullptr, saturated);
    }
}

// counts of the listed heavy edges: a wave per edge, lane l takes the first hops l, l+64, ...
template <int MAXL>
__global__ __launch_bounds__(kBlock) void k_count_cycles_heavy(const uint32_t *heavy, const uint32_t *n_heavy, WalkList walk,
                                                               const int32_t *ri, const int32_t *rj, Adj g, int max_len,
                                                               int shortest_only, ListPtrs<uint32_t, MAXL - 2> cnt,
                                                               uint32_t *saturated)
{
    const uint32_t n_own = *n_heavy, nh = n_own + walk.by_waves();
    const int lane = (int)(threadIdx.x & 63);
    for (uint32_t h = blockIdx.x * (kBlock / 64) + (threadIdx.x >> 6); h < nh; h += gridDim.x * (kBlock / 64)) {
        const uint32_t r = h < n_own ? heavy[h] : walk[h - n_own];
        const int32_t v0 = ri[r], vl = rj[r];
        EndRow end;
        end.load(g, vl);
        const int32_t r0 = g.ptr[v0], r1 = g.ptr[v0 + 1];
        unsigned long long tot[MAXL - 2];
        for (int L = shortest_only ? 3 : max_len; L <= max_len; ++L) {
            CountEmit<MAXL> em;
            em.clear();
            if (end.b0 != end.b1)
                for (int32_t p = r0 + lane; p < r1; p += 64) walk_from_first<MAXL>(g, end, v0, g.nb[p], vl, L, em);
            unsigned long long any = 0;
#pragma unroll
            for (int k = 0; k < MAXL - 2; ++k) {
                tot[k] = wave_sum((unsigned long long)em.n[k]);
                any |= tot[k];
            }
            if (any) break;   // plain search: single pass at full depth; shortest only: first length that closes
        }
        if (lane == 0) {
#pragma unroll
            for (int k = 0; k < MAXL - 2; ++k)
                if (k + 3 <= max_len) {
                    cnt.p[k][r] = tot[k] >= 0xffffffffull ? 0xffffffffu : (uint32_t)tot[k];
                    if (tot[k] >= 0xffffffffull) *saturated = 1u;
                }
        }
    }
}

template <int MAXL>
struct HasCycles {
    static constexpr int bytes = 4;   // bytes read per item: at least one count (one per list searched)
    static constexpr const char *tag = MAXL > 5 ? "HasCycles7" : "HasCycles";
    ListPtrs<uint32_t, MAXL - 2> cnt;
    int live;   // bit mask of the lists that hold any cycle
    __device__ __forceinline__ uint32_t operator()(size_t r) const
    {
        uint32_t any = 0;
#pragma unroll
        for (int k = 0; k < MAXL - 2; ++k)
            if (live & (1 << k)) any |= cnt.p[k][r];
        return any ? 1u : 0u;
    }
};

// consumer of the scan over HasCycles: the repulsive edges that close a cycle
struct CollectHitsEmit {
    static constexpr const char *tag = "CollectHits";
    uint32_t *hit;
    __device__ __forceinline__ void operator()(size_t r, uint32_t any, uint32_t p) const
    {
        if (any) hit[p] = (uint32_t)r;
    }
};

// the list totals (last entry of every offset array) and the saturation flag, side by side for one read-back
template <int NL>
__global__ void k_cycle_totals(ListPtrs<uint64_t, NL> off, size_t mr, int lists, const uint32_t *saturated, uint64_t *summary)
{
    const int k = (int)threadIdx.x;
    if (k < lists) summary[k] = off.p[k][mr];
    if (k == NL) summary[NL] = *saturated;
}

// The places of all lists by two launches: tile sums (blockIdx.y: the list), then every workgroup adds up those in front of
// its tile.  Up to kPlaceTiles tiles; against two or three launches a list and one for the totals, cycles up to length 5 of a
// 6-NN graph of 3*10^5 points 0.509 -> 0.480 ms.
constexpr unsigned kPlaceTiles = 1024;
template <int NL>
__global__ __launch_bounds__(kBlock) void k_place_sums(ListPtrs<uint32_t, NL> cnt, size_t mr, uint64_t *sums)
{
    const uint32_t *c = cnt.p[0];
#pragma unroll
    for (int k = 1; k < NL; ++k)
        if ((int)blockIdx.y == k) c = cnt.p[k];
    const size_t base = (size_t)blockIdx.x * kScanTile + threadIdx.x;
    uint32_t x[kScanItems];
    uint64_t s = 0;
#pragma unroll
    for (int q = 0; q < kScanItems; ++q) x[q] = item_or_last<uint32_t>(PtrInput<uint32_t>{c}, base + (size_t)q * kBlock, mr);
#pragma unroll
    for (int q = 0; q < kScanItems; ++q) s += x[q];
    s = block_sum(s);
    if (threadIdx.x == 0) sums[(size_t)blockIdx.y * gridDim.x + blockIdx.x] = s;
}
// sums: null with a single tile
template <int NL>
__global__ __launch_bounds__(kBlock) void k_places(ListPtrs<uint32_t, NL> cnt, ListPtrs<uint64_t, NL> off, size_t mr, const uint64_t *sums, uint64_t *summary)
{
    __shared__ uint64_t wave_tot[kBlock / 64];
    const uint32_t *c = cnt.p[0];
    uint64_t *out = off.p[0];
#pragma unroll
    for (int k = 1; k < NL; ++k)
        if ((int)blockIdx.y == k) { c = cnt.p[k]; out = off.p[k]; }
    const int w = threadIdx.x >> 6;
    const size_t base = (size_t)blockIdx.x * kScanTile + (size_t)w * kScanWaveItems + lane_id();
    uint32_t x[kScanItems];
    uint64_t v[kScanItems], pre = 0, carry = 0;
#pragma unroll
    for (int q = 0; q < kScanItems; ++q) x[q] = item_or_last<uint32_t>(PtrInput<uint32_t>{c}, base + (size_t)q * 64, mr);
    for (unsigned t = threadIdx.x; t < blockIdx.x; t += kBlock) pre += sums[(size_t)blockIdx.y * gridDim.x + t];
#pragma unroll
    for (int q = 0; q < kScanItems; ++q) {
        const uint64_t inc = wave_inclusive_scan((uint64_t)x[q]);
        v[q] = inc - x[q] + carry;
        carry += wave_last(inc);
    }
    if (lane_id() == 0) wave_tot[w] = carry;
    pre = block_sum(pre);      // its barriers are wave_tot's as well
#pragma unroll
    for (int k = 0; k < kBlock / 64 - 1; ++k)
        if (k < w) pre += wave_tot[k];
#pragma unroll
    for (int q = 0; q < kScanItems; ++q) {
        const size_t k = base + (size_t)q * 64;
        if (k < mr) out[k] = v[q] + pre;
    }
    if (blockIdx.x == gridDim.x - 1 && threadIdx.x == kBlock - 1) {
        out[mr] = pre + carry;
        summary[blockIdx.y] = pre + carry;
    }
}

// second walk, only over the repulsive edges that have cycles and only as deep as their
// longest cycle; writes every list at the offsets of the scan
template <int MAXL, bool MEET>
__device__ __forceinline__ void fill_edge(uint32_t r, const int32_t *ri, const int32_t *rj, const Adj &g, int live,
                                          int max_len, const ListPtrs<uint32_t, MAXL - 2> &cnt,
                                          const ListPtrs<uint64_t, MAXL - 2> &off, const ListPtrs<int32_t, MAXL - 2> &out)
{
    if (heavy_edge(g, ri[r], max_len)) return;   // written by k_fill_cycles_heavy
    int depth = 0;
    FillEmit<MAXL> em;
    em.vl = rj[r];
#pragma unroll
    for (int k = 0; k < MAXL - 2; ++k) {
        em.o[k] = nullptr;
        if (live & (1 << k)) {   // `live`: bit k set iff list k holds any cycle at all (the arrays of empty lists are not touched)
            if (cnt.p[k][r]) depth = k + 3;
            em.o[k] = out.p[k] + (size_t)(k + 3) * off.p[k][r];
        }
    }
    if (depth) enumerate_cycles<MAXL, MEET>(g, ri[r], em.vl, depth, em);
}

template <int MAXL, bool MEET>
__global__ __launch_bounds__(kBlock) void k_fill_cycles(size_t nh, const uint32_t *hit, const int32_t *ri,
                                                        const int32_t *rj, Adj g, int live, int max_len,
                                                        ListPtrs<uint32_t, MAXL - 2> cnt,
                                                        ListPtrs<uint64_t, MAXL - 2> off,
                                                        ListPtrs<int32_t, MAXL - 2> out)
{
    size_t h = (size_t)blockIdx.x * kBlock + threadIdx.x;
    if (h >= nh) return;
    fill_edge<MAXL, MEET>(hit ? hit[h] : (uint32_t)h, ri, rj, g, live, max_len, cnt, off, out);
}

// the same for the edges k_count_cycles_listed counted
template <int MAXL, bool MEET>
__global__ __launch_bounds__(kBlock) void k_fill_cycles_listed(WalkList list, const int32_t *ri, const int32_t *rj, Adj g, int live, int max_len,
                                                               ListPtrs<uint32_t, MAXL - 2> cnt, ListPtrs<uint64_t, MAXL - 2> off,
                                                               ListPtrs<int32_t, MAXL - 2> out)
{
    const size_t n = list.by_threads();
    for (size_t q = (size_t)blockIdx.x * kBlock + threadIdx.x; q < n; q += (size_t)gridDim.x * kBlock)
        fill_edge<MAXL, MEET>(list[q], ri, rj, g, live, max_len, cnt, off, out);
}

// ---- hashed search for cycles of length up to 5 --------------------------------------------------
// The same meeting in the middle on rows that are too long for registers.  G lanes share a repulsive edge.  They enter every node of the rows of N+(vL)'s entries v3 into a hash table in LDS, with
// one bit per v3 whose row holds the node (and one more bit for the nodes of N+(vL) itself); a pair (v1, v2),
// v2 in N+(v1), then needs one look into the table: its bits say which v3 close (v0,v1,v2,v3,vL) and whether
// (v0,v1,v2,vL) is a cycle.  That is d^2 entries and d^2 looks per edge, where the walk makes d^3 steps that each
// wait for a row.  What bounds the kernels: LDS latency (a look is a chain of a row search, a probe and the bits) at the
// ten to sixteen waves per CU that the tables leave room for.
// Edges whose rows or entries do not fit the table go to a list that a second launch works off with a table of 4096
// places; what does not fit there either is walked (more than 64 attractive neighbours at v0, more than 63 at vL, or rows
// behind these that hold more entries than the table), by a wave or a thread each (see WalkList).
constexpr uint32_t kNoKey = 0xffffffffu;
constexpr uint32_t kHashPairs = 1u << 24;      // beyond that a 32-bit count could overflow
constexpr int kSpillSlots = 4096;
template <int G, int SLOTS>
struct alignas(16) HashStage {
    static constexpr int W = G > 32 ? 2 : 1;   // words of a bit mask over N+(vL); the last bit is "in N+(vL)"
    uint32_t key[SLOTS];
    uint32_t mask[W][SLOTS];
    // N+(v0); per entry the number of pairs before its row (the largest int behind the last one) and where item 0
    // would sit in the adjacency array if the row's items were numbered from that on
    int32_t rowA[G], offA[G], fromA[G];
    int32_t rowB[G], offB[G], fromB[G];        // the same of N+(vL)
    std::conditional_t<(G > 32), uint64_t, uint32_t> others[G];      // of N+(v0)'s entries: the bits of N+(vL) but the one of the entry itself
};
// LDS that one wave shares: orders what its lanes wrote before against what they read behind
__device__ __forceinline__ void wave_lds_fence()
{
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}
template <int G>
__device__ __forceinline__ uint32_t lanes_exclusive_scan(uint32_t v, uint32_t *total)
{
    uint32_t inc;
    if constexpr (G == 64) {
        inc = wave_inclusive_scan(v);
        *total = wave_last(inc);
    } else {
        const int gl = (int)(threadIdx.x & (G - 1));
        inc = v;
#pragma unroll
        for (int off = 1; off < G; off <<= 1) {
            const uint32_t t = (uint32_t)__shfl_up((int)inc, off, G);
            if (gl >= off) inc += t;
        }
        *total = (uint32_t)__shfl((int)inc, G - 1, G);
    }
    return inc - v;
}
template <int G>
__device__ __forceinline__ uint64_t lanes_ballot(bool p)
{
    const uint64_t b = __ballot(p);
    if constexpr (G == 64) return b;
    else return (b >> (lane_id() & (64 - G))) & ((1ull << G) - 1ull);
}
template <int G>
__device__ __forceinline__ uint32_t lanes_sum(uint32_t v)
{
#pragma unroll
    for (int off = G / 2; off > 0; off >>= 1) v += (uint32_t)__shfl_xor((int)v, off, G);
    return v;
}
template <int SLOTS>
__device__ __forceinline__ uint32_t hash_slot(uint32_t v)
{
    static_assert((SLOTS & (SLOTS - 1)) == 0, "power of two");
    return (v * 0x9E3779B1u) >> (32 - __builtin_ctz(SLOTS));
}
// the table is never full (hash_stage sees to that): both loops end
template <int G, int SLOTS>
__device__ __forceinline__ uint32_t hash_enter(HashStage<G, SLOTS> &S, uint32_t v)
{
    uint32_t h = hash_slot<SLOTS>(v);
    for (;;) {
        const uint32_t old = atomicCAS(&S.key[h], kNoKey, v);
        if (old == kNoKey || old == v) return h;
        h = (h + 1) & (SLOTS - 1);
    }
}
template <int G, int SLOTS>
__device__ __forceinline__ uint64_t hash_look(const HashStage<G, SLOTS> &S, uint32_t v)
{
    uint32_t h = hash_slot<SLOTS>(v);
    for (;;) {
        const uint32_t k = S.key[h];
        if (k == v) break;
        if (k == kNoKey) return 0ull;
        h = (h + 1) & (SLOTS - 1);
    }
    uint64_t m = S.mask[0][h];
    if constexpr (HashStage<G, SLOTS>::W == 2) m |= (uint64_t)S.mask[1][h] << 32;
    return m;
}
// A lane's next kHashBatch items, G apart, take every step together: one after the other, each would wait for its own chain
// (the row by bisection, the entry, the first place of the table).
// Measured with item after item, a search for every item's row and a second look for every pair that closes a 5-cycle | as it is,
// count + fill in us: 6-NN graph of 3*10^5 points 118 + 139 | 90 + 108, of 10^6 402 + 455 | 304 + 353, 512^2 long-range grid 298 + 176
// | 270 + 145, 180x181 one behind a dual round (64 lanes) 226 + 218 | 199 + 183.
constexpr int kHashBatch = 4;
// row[q]: the row of item w[q], one of the items base .. base + G * kHashBatch - 1; off[k] (`mine`: lane k's) items come before row
// k, the largest int behind the last row.  No row is empty: its node's neighbour is in it.
template <int G>
__device__ __forceinline__ void rows_of_items(const int32_t *off, int32_t mine, uint32_t base, const int32_t (&w)[kHashBatch], int (&row)[kHashBatch])
{
    if constexpr (G * kHashBatch == 64) {      // a bit for the first item of every row: rows are counted, not searched
        const uint32_t at = (uint32_t)mine - base;
        uint32_t lo = at < 32u ? 1u << at : 0u, hi = at >= 32u && at < 64u ? 1u << (at - 32u) : 0u;
        lo |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)lo, 0x128, 0xf, 0xf, false);      // row_ror:8 4 2 1: all sixteen lanes' bits
        hi |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)hi, 0x128, 0xf, 0xf, false);
        lo |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)lo, 0x124, 0xf, 0xf, false);
        hi |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)hi, 0x124, 0xf, 0xf, false);
        lo |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)lo, 0x122, 0xf, 0xf, false);
        hi |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)hi, 0x122, 0xf, 0xf, false);
        lo |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)lo, 0x121, 0xf, 0xf, false);
        hi |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)hi, 0x121, 0xf, 0xf, false);
        const int in_front = __popcll(lanes_ballot<G>((uint32_t)mine < base)) - 1;
#pragma unroll
        for (int q = 0; q < kHashBatch; ++q) {
            const uint32_t p = (uint32_t)w[q] - base;      // bits 0 .. p
            row[q] = in_front + __popc(lo & (p >= 31u ? ~0u : (2u << p) - 1u)) + __popc(p >= 32u ? hi & (p >= 63u ? ~0u : (2u << (p - 32u)) - 1u) : 0u);
        }
    } else {
#pragma unroll
        for (int q = 0; q < kHashBatch; ++q) row[q] = 0;
#pragma unroll
        for (int step = G / 2; step > 0; step >>= 1) {
            int32_t x[kHashBatch];
#pragma unroll
            for (int q = 0; q < kHashBatch; ++q) x[q] = off[row[q] + step];
#pragma unroll
            for (int q = 0; q < kHashBatch; ++q) row[q] += x[q] <= w[q] ? step : 0;
        }
    }
}
// v[q] (< 0: none) get their places in the table, and `bit[q]` in the mask there
template <int G, int SLOTS>
__device__ __forceinline__ void hash_enter_items(HashStage<G, SLOTS> &S, const int32_t (&v)[kHashBatch], const int (&bit)[kHashBatch])
{
    constexpr int W = HashStage<G, SLOTS>::W;
    uint32_t h[kHashBatch], old[kHashBatch];
#pragma unroll
    for (int q = 0; q < kHashBatch; ++q) {
        h[q] = hash_slot<SLOTS>((uint32_t)v[q]);
        old[q] = v[q] >= 0 ? atomicCAS(&S.key[h[q]], kNoKey, (uint32_t)v[q]) : kNoKey;
    }
#pragma unroll
    for (int q = 0; q < kHashBatch; ++q)
        if (v[q] >= 0) {
            while (old[q] != kNoKey && old[q] != (uint32_t)v[q]) {
                h[q] = (h[q] + 1) & (SLOTS - 1);
                old[q] = atomicCAS(&S.key[h[q]], kNoKey, (uint32_t)v[q]);
            }
            atomicOr(&S.mask[W == 2 ? bit[q] >> 5 : 0][h[q]], 1u << (bit[q] & 31));
        }
}
// hash_look for v[q]
template <int G, int SLOTS>
__device__ __forceinline__ void hash_look_items(const HashStage<G, SLOTS> &S, const int32_t (&v)[kHashBatch], uint64_t (&m)[kHashBatch])
{
    uint32_t h[kHashBatch], k[kHashBatch];
#pragma unroll
    for (int q = 0; q < kHashBatch; ++q) {
        h[q] = hash_slot<SLOTS>((uint32_t)v[q]);
        k[q] = S.key[h[q]];
        m[q] = S.mask[0][h[q]];
        if constexpr (HashStage<G, SLOTS>::W == 2) m[q] |= (uint64_t)S.mask[1][h[q]] << 32;
    }
#pragma unroll
    for (int q = 0; q < kHashBatch; ++q)
        if (k[q] != (uint32_t)v[q]) {
            m[q] = 0;
            while (k[q] != kNoKey) {
                h[q] = (h[q] + 1) & (SLOTS - 1);
                k[q] = S.key[h[q]];
                if (k[q] != (uint32_t)v[q]) continue;
                m[q] = S.mask[0][h[q]];
                if constexpr (HashStage<G, SLOTS>::W == 2) m[q] |= (uint64_t)S.mask[1][h[q]] << 32;
                break;
            }
        }
}

struct HashEdge {
    int32_t v0, vl;
    int dA, dB;
    uint32_t pairs;     // number of (v1, v2) pairs
    int32_t my_v1;      // lane k < dA: rowA[k]
    int32_t my_off;     // offA[lane]
    bool three;         // my_v1 is in N+(vL)
    bool live;          // the edge is searched here (valid, both rows non-empty, everything fits)
    bool spilled;       // it does not fit
};

template <int G, int SLOTS>
__device__ __forceinline__ HashEdge hash_stage(HashStage<G, SLOTS> &S, bool valid, int32_t v0, int32_t vl, const Adj &g, int max_len)
{
    constexpr int W = HashStage<G, SLOTS>::W;
    constexpr int kFlag = G > 32 ? 31 : G - 1;   // bit of the last mask word: in N+(vL)
    const int gl = (int)(threadIdx.x & (G - 1));
    HashEdge E;
    E.v0 = v0; E.vl = vl; E.my_v1 = -1; E.my_off = 0x7fffffff; E.three = false; E.pairs = 0;
    int32_t pa0 = 0, pa1 = 0, pb0 = 0, pb1 = 0;
    if (valid) { pa0 = g.ptr[v0]; pa1 = g.ptr[v0 + 1]; pb0 = g.ptr[vl]; pb1 = g.ptr[vl + 1]; }
    E.dA = pa1 - pa0; E.dB = pb1 - pb0;
    const bool search = valid && E.dA > 0 && E.dB > 0;
    const bool fits = E.dA <= G && E.dB <= G - 1;
    int32_t startA = 0, startB = 0, v3 = -1;
    uint32_t lenA = 0, lenB = 0;
    if (search && fits) {
        if (gl < E.dA) {
            E.my_v1 = g.nb[pa0 + gl];
            startA = g.ptr[E.my_v1];
            lenA = (uint32_t)(g.ptr[E.my_v1 + 1] - startA);
        }
        if (gl < E.dB) {
            v3 = g.nb[pb0 + gl];
            if (max_len >= 5) {
                startB = g.ptr[v3];
                lenB = (uint32_t)(g.ptr[v3 + 1] - startB);
            }
        }
    }
    // a heavy row among N+(v0)'s entries is no trouble here (its pairs are only looked up), one among N+(vL)'s does not fit
    uint32_t entries;
    const uint32_t beforeA = lanes_exclusive_scan<G>(lenA, &E.pairs), beforeB = lanes_exclusive_scan<G>(lenB, &entries);
    E.spilled = search && (!fits || entries + (uint32_t)E.dB > (uint32_t)(SLOTS / 8 * 7) || E.pairs > kHashPairs);
    E.live = search && !E.spilled;
    if (!E.live) return E;
    wave_lds_fence();      // the stage may still be in use for the edge before this one
    const int32_t my_offB = gl < E.dB ? (int32_t)beforeB : 0x7fffffff;
    E.my_off = gl < E.dA ? (int32_t)beforeA : 0x7fffffff;
    S.rowA[gl] = E.my_v1; S.fromA[gl] = startA - (int32_t)beforeA; S.offA[gl] = E.my_off;
    S.rowB[gl] = v3; S.fromB[gl] = startB - (int32_t)beforeB; S.offB[gl] = my_offB;
    for (int k = gl * 4; k < SLOTS; k += G * 4) {
        *reinterpret_cast<uint4 *>(&S.key[k]) = make_uint4(kNoKey, kNoKey, kNoKey, kNoKey);
#pragma unroll
        for (int q = 0; q < W; ++q) *reinterpret_cast<uint4 *>(&S.mask[q][k]) = make_uint4(0, 0, 0, 0);
    }
    wave_lds_fence();
    if (v3 >= 0) atomicOr(&S.mask[W - 1][hash_enter(S, (uint32_t)v3)], 1u << kFlag);
    for (uint32_t base = 0; base < entries; base += G * kHashBatch) {
        int32_t w[kHashBatch], v2[kHashBatch];
        int row[kHashBatch];
#pragma unroll
        for (int q = 0; q < kHashBatch; ++q) w[q] = (int32_t)min(base + (uint32_t)(q * G + gl), entries - 1);
        rows_of_items<G>(S.offB, my_offB, base, w, row);
#pragma unroll
        for (int q = 0; q < kHashBatch; ++q) v2[q] = g.nb[S.fromB[row[q]] + w[q]];
#pragma unroll
        for (int q = 0; q < kHashBatch; ++q)
            if (base + (uint32_t)(q * G + gl) >= entries || v2[q] == v0 || v2[q] == vl) v2[q] = -1;
        hash_enter_items(S, v2, row);
    }
    wave_lds_fence();
    if (E.my_v1 >= 0) {      // v3 == v1 closes no cycle; it can only come up where v1 is in N+(vL)
        uint64_t others = ~0ull;
        E.three = ((hash_look(S, (uint32_t)E.my_v1) >> (G - 1)) & 1ull) != 0;
        if (E.three) {
            int lo = 0, hi = E.dB;
            while (lo < hi) {
                const int mid = (lo + hi) >> 1;
                if (S.rowB[mid] < E.my_v1) lo = mid + 1; else hi = mid;
            }
            others = ~(1ull << lo);
        }
        S.others[gl] = (std::remove_reference_t<decltype(S.others[0])>)others;
    }
    wave_lds_fence();
    return E;
}

// what the table says about the pairs base + q * G + lane: v1, v2, whether (v0,v1,v2,vl) is a cycle, which v3 close a 5-cycle
// (nothing of the pairs behind the last one)
template <int G, int SLOTS>
__device__ __forceinline__ void hash_pairs(const HashStage<G, SLOTS> &S, const HashEdge &E, const Adj &g, uint32_t base, int32_t (&v1)[kHashBatch],
                                           int32_t (&v2)[kHashBatch], bool (&four)[kHashBatch], uint64_t (&fives)[kHashBatch])
{
    constexpr uint64_t kFlagBit = 1ull << (G - 1);
    const uint32_t first = base + (uint32_t)(threadIdx.x & (G - 1));
    int32_t w[kHashBatch];
    int row[kHashBatch];
    uint64_t m[kHashBatch], others[kHashBatch];
#pragma unroll
    for (int q = 0; q < kHashBatch; ++q) w[q] = (int32_t)min(first + (uint32_t)(q * G), E.pairs - 1);
    rows_of_items<G>(S.offA, E.my_off, base, w, row);
#pragma unroll
    for (int q = 0; q < kHashBatch; ++q) { v1[q] = S.rowA[row[q]]; v2[q] = g.nb[S.fromA[row[q]] + w[q]]; others[q] = S.others[row[q]]; }
    hash_look_items(S, v2, m);                         // v0 and vl are not in the table
#pragma unroll
    for (int q = 0; q < kHashBatch; ++q) {
        if (first + (uint32_t)(q * G) >= E.pairs) m[q] = 0;
        four[q] = (m[q] & kFlagBit) != 0;
        fives[q] = m[q] & ~kFlagBit & others[q];
    }
}

template <int G>
struct HashBlock {      // edges per workgroup of the kernels below: one wave, or 256 threads of narrower groups
    static constexpr int threads = G == 64 ? 64 : kBlock;
    static constexpr int edges = threads / G;
};

// `list` (optional): the edges to search, *n_list of them; else the edges 0..nr-1.  Edges that do not fit go to `spill`.
template <int G, int SLOTS>
__global__ __launch_bounds__(HashBlock<G>::threads) void k_count_cycles_hash(size_t nr, const uint32_t *list, const uint32_t *n_list,
                                                                           const int32_t *ri, const int32_t *rj, Adj g, int max_len,
                                                                           int shortest_only, ListPtrs<uint32_t, 3> cnt,
                                                                           uint32_t *spill, uint32_t *n_spill,
                                                                           WalkList walk)
{
    constexpr int kEdges = HashBlock<G>::edges;
    __shared__ HashStage<G, SLOTS> stage[kEdges];
    const int gl = (int)(threadIdx.x & (G - 1)), grp = (int)(threadIdx.x / G);
    HashStage<G, SLOTS> &S = stage[grp];
    const size_t n = list ? (size_t)*n_list : nr;
    for (size_t h = (size_t)blockIdx.x * kEdges + grp; h < n; h += (size_t)gridDim.x * kEdges) {
        const size_t r = list ? (size_t)list[h] : h;
        const HashEdge E = hash_stage(S, true, ri[r], rj[r], g, max_len);
        uint32_t n3 = 0, n4 = 0, n5 = 0;
        if (E.live) {
            n3 = E.three ? 1u : 0u;
            for (uint32_t base = 0; base < E.pairs; base += G * kHashBatch) {
                int32_t v1[kHashBatch], v2[kHashBatch];
                bool four[kHashBatch];
                uint64_t fives[kHashBatch];
                hash_pairs(S, E, g, base, v1, v2, four, fives);
#pragma unroll
                for (int q = 0; q < kHashBatch; ++q) { n4 += four[q] ? 1u : 0u; n5 += (uint32_t)__popcll(fives[q]); }
            }
        }
        n3 = lanes_sum<G>(n3); n4 = lanes_sum<G>(n4); n5 = lanes_sum<G>(n5);
        if (shortest_only) {   // only the shortest length that closes a cycle is kept
            if (n3) { n4 = 0; n5 = 0; }
            else if (n4) n5 = 0;
        }
        if (gl == 0) {
            cnt.p[0][r] = n3;
            if (max_len >= 4) cnt.p[1][r] = n4;
            if (max_len >= 5) cnt.p[2][r] = n5;
            // counted again by a kernel behind this one
            if (E.spilled && walk.n && E.dA <= kWalkRow) *(walk.last - atomicAdd(walk.n, 1u)) = (uint32_t)r;
            else if (E.spilled) spill[atomicAdd(n_spill, 1u)] = (uint32_t)r;
        }
    }
}

// writes the cycles of the edges that fit at the places the scans of the counts gave them
template <int G, int SLOTS>
__global__ __launch_bounds__(HashBlock<G>::threads) void k_fill_cycles_hash(size_t nh, const uint32_t *list, const uint32_t *n_list,
                                                                          const int32_t *ri, const int32_t *rj, Adj g, int max_len,
                                                                          int live, ListPtrs<uint32_t, 3> cnt,
                                                                          ListPtrs<uint64_t, 3> off, ListPtrs<int32_t, 3> out)
{
    constexpr int kEdges = HashBlock<G>::edges;
    __shared__ HashStage<G, SLOTS> stage[kEdges];
    const int gl = (int)(threadIdx.x & (G - 1)), grp = (int)(threadIdx.x / G);
    HashStage<G, SLOTS> &S = stage[grp];
    const uint64_t below = (1ull << gl) - 1ull;
    const size_t n = n_list ? (size_t)*n_list : nh;
    for (size_t h = (size_t)blockIdx.x * kEdges + grp; h < n; h += (size_t)gridDim.x * kEdges) {
        const uint32_t r = list ? list[h] : (uint32_t)h;
        // a list is written iff the count pass kept cycles of that length (with shortest_only: one length only);
        // `live`: bit k set iff list k holds any cycle at all
        const bool want3 = (live & 1) && cnt.p[0][r] != 0;
        const bool want4 = (live & 2) && cnt.p[1][r] != 0;
        const bool want5 = (live & 4) && cnt.p[2][r] != 0;
        const HashEdge E = hash_stage(S, want3 || want4 || want5, ri[r], rj[r], g, want5 ? max_len : 4);
        if (!E.live) continue;     // nothing to write, or written by the kernels behind this one; the whole group goes on
        if (want3) {
            const bool c3 = E.three;
            const uint64_t vote = lanes_ballot<G>(c3);
            if (c3) {
                int32_t *o = out.p[0] + 3 * (off.p[0][r] + (uint64_t)__popcll(vote & below));
                o[0] = E.v0; o[1] = E.my_v1; o[2] = E.vl;
            }
        }
        if (!want4 && !want5) continue;
        uint64_t at4 = want4 ? off.p[1][r] : 0, at5 = want5 ? off.p[2][r] : 0;
        for (uint32_t base = 0; base < E.pairs; base += G * kHashBatch) {   // the same number of turns for every lane of the group
            int32_t v1[kHashBatch], v2[kHashBatch];
            bool four[kHashBatch];
            uint64_t fives[kHashBatch];
            hash_pairs(S, E, g, base, v1, v2, four, fives);
#pragma unroll
            for (int q = 0; q < kHashBatch; ++q) {
                if (base + (uint32_t)(q * G) >= E.pairs) break;      // the same for every lane of the group
                if (want4) {
                    const uint64_t vote = lanes_ballot<G>(four[q]);
                    if (four[q]) {
                        int32_t *o = out.p[1] + 4 * (at4 + (uint64_t)__popcll(vote & below));
                        o[0] = E.v0; o[1] = v1[q]; o[2] = v2[q]; o[3] = E.vl;
                    }
                    at4 += (uint64_t)__popcll(vote);
                }
                if (want5) {
                    uint32_t total;
                    const uint32_t before = lanes_exclusive_scan<G>((uint32_t)__popcll(fives[q]), &total);
                    int32_t *o = out.p[2] + 5 * (at5 + before);
                    while (fives[q]) {
                        const int b = __ffsll((long long)fives[q]) - 1;
                        fives[q] &= fives[q] - 1;
                        o[0] = E.v0; o[1] = v1[q]; o[2] = v2[q]; o[3] = S.rowB[b]; o[4] = E.vl;
                        o += 5;
                    }
                    at5 += total;
                }
            }
        }
    }
}

// ---- triangles on graphs with long rows ----------------------------------------------------------
// The contracted graphs of later rounds can be dense (rows of 20-40 attractive neighbours and more).  One
// thread per repulsive edge then walks its shorter row alone, a dependent bisection of the longer row per
// entry.  Here sixteen lanes share the edge: they take the shorter row sixteen entries at a time, every lane
// bisects the longer row for its entry, and a ballot counts -- or, in the fill pass, places -- the common
// neighbours.  The shorter row is ascending, so the triangles (v0, v1, vL) come out in list order.
constexpr int kTriLanes = 16;                    // lanes per repulsive edge (one DPP row)
constexpr int kTriEdges = kBlock / kTriLanes;    // edges per workgroup
// The counting pass notes the common neighbours of an edge where there is room for them, up to kTriLanes of an edge, and the
// fill pass copies them instead of searching again: triangles of a 400x301 window graph, 2.4e6 of 2.9e5
// repulsive edges, count + fill 41 + 46 us without and 45 + 26 with it.  The room is what the pool has left of building the adjacency: spare blocks, in each of
// which every edge has `width` places.
constexpr int kRoomParts = 6;
struct TriRoom {
    int32_t *part[kRoomParts];
    int width, places;      // of an edge: in a part, in all
    __device__ __forceinline__ int32_t *place(int k) const      // k < places: place k of edge 0, `width` in front of that of edge 1
    {
        int32_t *p = part[0] + k;
#pragma unroll
        for (int q = 1; q < kRoomParts; ++q)
            if (k >= q * width) p = part[q] + (k - q * width);
        return p;
    }
};
// the room for mr edges that the cached blocks make up, as many places as can be, in the fewest parts
inline TriRoom tri_room(Ctx &ctx, size_t mr, Spares<kRoomParts> &blocks)
{
    TriRoom room = {};
    int parts = 0;
    if (ctx.active->is_arena()) return room;
    for (int w = kTriLanes; w >= 1; --w) {
        const int want = (kTriLanes + w - 1) / w, have = Spares<kRoomParts>::available(ctx, mr * (size_t)w * 4), p = have < want ? have : want;
        const int places = p * w < kTriLanes ? p * w : kTriLanes;
        if (places > room.places) { room.places = places; room.width = w; parts = p; }
    }
    blocks.take(ctx, parts, mr * (size_t)room.width * 4);
    return room;
}
// what is left of it: nothing, if a part was taken back
inline TriRoom tri_room_now(TriRoom room, const Spares<kRoomParts> &blocks)
{
    for (int q = 0; q * room.width < room.places; ++q) {
        room.part[q] = (int32_t *)blocks.get(q);
        if (!room.part[q]) room.places = 0;
    }
    return room;
}
template <bool FILL>
__global__ __launch_bounds__(kBlock) void k_triangles_group(size_t nr, const uint32_t *hit, const int32_t *ri,
                                                            const int32_t *rj, Adj g, uint32_t *cnt0, const uint64_t *off0,
                                                            int32_t *out0, TriRoom room)
{
    __shared__ int32_t s_note[kTriEdges][kTriLanes];      // found so far, so that a lane writes to one place of the room only
    const int gl = (int)(threadIdx.x & (kTriLanes - 1)), group = (int)threadIdx.x / kTriLanes;
    int32_t *const mine = gl < room.places ? room.place(gl) : nullptr;
    // strides (see grid_striding); a group of lanes has the same h throughout
    for (size_t h = (size_t)blockIdx.x * kTriEdges + group; h < nr; h += (size_t)gridDim.x * kTriEdges) {
        const uint32_t r = hit ? hit[h] : (uint32_t)h;
        uint32_t n = 0;
        if (FILL) n = cnt0[r];
        if (FILL && n == 0) continue;
        const int32_t v0 = ri[r], vl = rj[r];
        if (FILL && n <= (uint32_t)room.places) {
            if ((uint32_t)gl < n) {
                int32_t *o = out0 + 3 * (off0[r] + (uint64_t)gl);
                o[0] = v0; o[1] = mine[(size_t)r * (size_t)room.width]; o[2] = vl;
            }
            continue;
        }
        int32_t a0 = g.ptr[v0], a1 = g.ptr[v0 + 1], b0 = g.ptr[vl], b1 = g.ptr[vl + 1];
        if (a1 - a0 > b1 - b0) { int32_t t = a0; a0 = b0; b0 = t; t = a1; a1 = b1; b1 = t; }   // [a0,a1): the shorter row
        uint32_t found = 0;
        uint64_t at = FILL ? off0[r] : 0;
        if (b0 < b1)
            for (int32_t base = a0; base < a1; base += kTriLanes) {   // the same number of turns for every lane of the group
                const int32_t p = base + gl;
                bool common = false;
                int32_t x = 0;
                if (p < a1) {
                    x = g.nb[p];
                    int32_t lo = b0, hi = b1;
                    while (lo < hi) {
                        const int32_t mid = lo + ((hi - lo) >> 1);
                        if (g.nb[mid] < x) lo = mid + 1; else hi = mid;
                    }
                    common = lo < b1 && g.nb[lo] == x;
                }
                const uint32_t vote = (uint32_t)lanes_ballot<kTriLanes>(common);
                if (FILL) {
                    if (common) {
                        int32_t *o = out0 + 3 * (at + (uint64_t)__popc(vote & ((1u << gl) - 1u)));
                        o[0] = v0; o[1] = x; o[2] = vl;
                    }
                    at += (uint64_t)__popc(vote);
                } else {
                    const uint32_t k = found + (uint32_t)__popc(vote & ((1u << gl) - 1u));
                    if (common && k < (uint32_t)kTriLanes) s_note[group][k] = x;
                    found += (uint32_t)__popc(vote);
                }
            }
        if (!FILL) {
            wave_lds_fence();
            if (mine && (uint32_t)gl < found) mine[(size_t)r * (size_t)room.width] = s_note[group][gl];
            wave_lds_fence();
            if (gl == 0) cnt0[r] = found;
        }
    }
}

// cycles of the listed heavy edges: per round of 64 first hops every lane counts what its hop
// closes, a wave scan turns the counts into places, and the lane walks again and writes
template <int MAXL>
__global__ __launch_bounds__(kBlock) void k_fill_cycles_heavy(const uint32_t *heavy, const uint32_t *n_heavy, WalkList walk,
                                                              const int32_t *ri, const int32_t *rj, Adj g, int live,
                                                              ListPtrs<uint32_t, MAXL - 2> cnt,
                                                              ListPtrs<uint64_t, MAXL - 2> off,
                                                              ListPtrs<int32_t, MAXL - 2> out)
{
    const uint32_t n_own = *n_heavy, nh = n_own + walk.by_waves();
    const int lane = (int)(threadIdx.x & 63);
    for (uint32_t h = blockIdx.x * (kBlock / 64) + (threadIdx.x >> 6); h < nh; h += gridDim.x * (kBlock / 64)) {
        const uint32_t r = h < n_own ? heavy[h] : walk[h - n_own];
        int depth = 0;
        size_t place[MAXL - 2];   // cycles of this edge already written, per length
#pragma unroll
        for (int k = 0; k < MAXL - 2; ++k) {
            place[k] = 0;
            if (live & (1 << k)) {
                if (cnt.p[k][r]) depth = k + 3;
                place[k] = off.p[k][r];
            }
        }
        if (depth == 0) continue;
        const int32_t v0 = ri[r], vl = rj[r];
        EndRow end;
        end.load(g, vl);
        const int32_t r0 = g.ptr[v0], r1 = g.ptr[v0 + 1];
        for (int32_t p0 = r0; p0 < r1; p0 += 64) {
            const int32_t p = p0 + lane;
            const int32_t v1 = p < r1 ? g.nb[p] : -1;
            CountEmit<MAXL> em;
            em.clear();
            if (v1 >= 0) walk_from_first<MAXL>(g, end, v0, v1, vl, depth, em);
            FillEmit<MAXL> fe;
            fe.vl = vl;
#pragma unroll
            for (int k = 0; k < MAXL - 2; ++k) {
                fe.o[k] = nullptr;
                if (live & (1 << k)) {
                    const uint32_t inc = wave_inclusive_scan(em.n[k]);
                    fe.o[k] = out.p[k] + (size_t)(k + 3) * (place[k] + (inc - em.n[k]));
                    place[k] += wave_last(inc);
                }
            }
            if (v1 >= 0) walk_from_first<MAXL>(g, end, v0, v1, vl, depth, fe);
        }
    }
}

// count, scan, fill for walks of at most MAXL nodes
template <int MAXL>
rama_status count_and_fill(Ctx &ctx, size_t mr, const int32_t *ri, const int32_t *rj, Adj adj, int32_t n, size_t mp,
                           int max_len, bool shortest_only, CycleLists &out, const CycleSink &sink, uint32_t longest_row = 0xffffffffu)
{
    constexpr int NL = MAXL - 2;
    const int lists = max_len - 2;
    Buf<uint32_t> cnt[NL];
    Buf<uint64_t> off[NL];
    ListPtrs<uint32_t, NL> cp;
    ListPtrs<uint64_t, NL> op;
    ListPtrs<int32_t, NL> vp;
    for (int k = 0; k < NL; ++k) {
        cp.p[k] = nullptr; op.p[k] = nullptr; vp.p[k] = nullptr;
        if (k >= lists) continue;
        RAMA_TRY(cnt[k].alloc(ctx, mr));
        RAMA_TRY(off[k].alloc(ctx, mr + 1));
        cp.p[k] = cnt[k].get(); op.p[k] = off[k].get();
    }
    // heavy edges (only possible for max_len >= 4): listed by the kernels in front, counted by a wave each in a kernel
    // that ends at once when the list is empty
    const bool may_be_heavy = max_len >= 4;
    // Lengths 4 and 5.  If every attractive row has at most kRowRegs entries (3-D grids), the walk holds the rows it
    // needs in registers and is the fastest: 4.4 ms against 4.8 for the hashed search (eight lanes per edge) on the
    // 320^3 grid (rows <= 6, 3.1e7 repulsive edges); with whole rows in registers 2.2.  Otherwise the hashed search: sixteen lanes per edge while rows hold
    // up to twelve entries on average, a wave per edge beyond.  Measured (count pass, ms): 512^2 grid with long-range
    // edges (rows <= 12) 0.30 with sixteen lanes, 0.38 with 32, 0.75 with 64, 3.9 for the walk; 6-nearest-neighbour graph
    // of 10^6 points (rows of 3..15) 0.40, 0.56, 1.16, walk 1.27; a 180x181 long-range grid after one dual round
    // (rows of 16 on average, up to 43; 8e4 repulsive edges) 0.23 with 64 lanes, walk 21.
    bool hashed = false;
    const bool wide = 2 * mp > (size_t)12 * (size_t)n;
    if constexpr (MAXL == 5)
        hashed = max_len >= 4 && (ctx.cycle_search == 2 || (ctx.cycle_search == 0 && longest_row > (uint32_t)kRowRegs));
    // n_heavy[0]: length of the heavy list, [1]: a count saturated, [2]: length of the list of edges that take the large
    // hash table, [3]: length of the list of those that do not and are walked by a thread each (in heavy's array, from the back)
    Buf<uint32_t> heavy, spill, n_heavy;
    RAMA_TRY(heavy.alloc(ctx, may_be_heavy ? mr : 1));
    RAMA_TRY(spill.alloc(ctx, hashed ? mr : 1));
    RAMA_TRY(zeroed<uint32_t>(ctx, 4, n_heavy));
    const WalkList walk = hashed ? WalkList{heavy.get() + (mr - 1), n_heavy.get() + 3} : WalkList{};
    // mode 1 is the walk that fetches a row per path at its last level, kept for comparison; walks of at
    // most three nodes have no such level
    const bool meet = MAXL >= 5 && max_len >= 5 && ctx.cycle_search != 1;
    const int walk_flags = shortest_only ? 1 : 0;
    const double search_bytes = (double)(mr * (8 + 4 * (size_t)lists) + ((size_t)n + 1) * 4 + mp * 8);
    if constexpr (MAXL == 5) {
        if (hashed) {
            auto count = [&](auto lanes, auto slots, size_t edges, const uint32_t *list, const uint32_t *n_list, uint32_t *spill_to, uint32_t *n_spill,
                             WalkList walked) {
                constexpr int G = decltype(lanes)::value, S = decltype(slots)::value;
                ProfScope ps_(ctx, "k_count_cycles_hash", list ? 0.0 : search_bytes);
                k_count_cycles_hash<G, S><<<grid_striding(edges, HashBlock<G>::edges), HashBlock<G>::threads, 0, ctx.stream>>>(
                    mr, list, n_list, ri, rj, adj, max_len, shortest_only ? 1 : 0, cp, spill_to, n_spill, walked);
            };
            using std::integral_constant;
            if (wide) count(integral_constant<int, 64>{}, integral_constant<int, 1024>{}, mr, nullptr, nullptr, spill.get(), n_heavy.get() + 2, WalkList{});
            else count(integral_constant<int, 16>{}, integral_constant<int, 256>{}, mr, nullptr, nullptr, spill.get(), n_heavy.get() + 2, WalkList{});
            LAUNCH_TRY(ctx, "count_cycles_hash");
            count(integral_constant<int, 64>{}, integral_constant<int, kSpillSlots>{}, kSpillGroups, spill.get(), n_heavy.get() + 2, heavy.get(),
                  n_heavy.get(), walk);
            LAUNCH_TRY(ctx, "count_cycles_hash");
            ProfScope ps_(ctx, "k_count_cycles_listed", 0.0);
            k_count_cycles_listed<MAXL, true><<<kHeavyGroups, kBlock, 0, ctx.stream>>>(walk, ri, rj, adj, max_len, walk_flags, cp, n_heavy.get() + 1);
        }
    }
    // triangles only, rows of more than 12 attractive neighbours on average: sixteen lanes per repulsive edge
    bool wide3 = false;
    if constexpr (MAXL == 3)
        wide3 = ctx.cycle_search == 2 || (ctx.cycle_search == 0 && 2 * mp > (size_t)12 * (size_t)n);
    ScanPlan<uint64_t> places;      // of triangles
    if constexpr (MAXL == 3) RAMA_TRY((scan_plan_alloc<uint64_t>(ctx, mr, 0, places)));
    Spares<kRoomParts> blocks;
    TriRoom room = {};
    if (wide3) room = tri_room_now(tri_room(ctx, mr, blocks), blocks);
    if (wide3) {
        ProfScope ps_(ctx, "k_count_triangles_group", search_bytes);
        k_triangles_group<false><<<grid_striding(mr, kTriEdges), kBlock, 0, ctx.stream>>>(mr, (const uint32_t *)nullptr, ri, rj, adj, cp.p[0],
                                                                                   (const uint64_t *)nullptr, (int32_t *)nullptr, room);
    } else if (!hashed) {
        ProfScope ps_(ctx, MAXL == 3 ? "k_count_cycles<3>" : MAXL == 5 ? "k_count_cycles<5>" : "k_count_cycles<7>", search_bytes);
        bool short_rows = false;
        if constexpr (MAXL == 5) {
            short_rows = ctx.cycle_search == 0 && max_len == 5 && !shortest_only && longest_row <= 6;
            if (short_rows) k_count_cycles_short<6><<<grid_for(mr), kBlock, 0, ctx.stream>>>(mr, ri, rj, adj, cp);
        }
        if (short_rows) {
            // nothing heavy, nothing that could overflow a count
        } else if (meet)
            k_count_cycles<MAXL, (MAXL >= 5)><<<grid_for(mr), kBlock, 0, ctx.stream>>>(mr, ri, rj, adj, max_len, walk_flags, cp,
                                                                                      heavy.get(), n_heavy.get(), n_heavy.get() + 1);
        else
            k_count_cycles<MAXL, false><<<grid_for(mr), kBlock, 0, ctx.stream>>>(mr, ri, rj, adj, max_len, walk_flags, cp,
                                                                                heavy.get(), n_heavy.get(), n_heavy.get() + 1);
    }
    LAUNCH_TRY(ctx, "count_cycles");
    if (may_be_heavy) {
        ProfScope ps_(ctx, "k_count_cycles_heavy", 0.0);
        k_count_cycles_heavy<MAXL><<<kHeavyGroups, kBlock, 0, ctx.stream>>>(heavy.get(), n_heavy.get(), walk, ri, rj, adj, max_len,
                                                                          shortest_only ? 1 : 0, cp, n_heavy.get() + 1);
        LAUNCH_TRY(ctx, "count_cycles_heavy");
    }
    uint64_t tot[NL + 1], all = 0;
    if constexpr (MAXL == 3) {
        // one list, whose counts (common neighbours) cannot saturate: the total comes back from the scan of the tile sums,
        // and the places are only computed when there is a cycle
        RAMA_TRY((scan_totals<uint64_t>(ctx, PtrInput<uint32_t>{cnt[0].get()}, places)));
        tot[0] = places.total;
        if (tot[0]) RAMA_TRY((scan_store<uint64_t>(ctx, PtrInput<uint32_t>{cnt[0].get()}, places, off[0].get())));
        places.offs.reset(); places.sums.reset();
    } else {
        Buf<uint64_t> summary;
        RAMA_TRY(summary.alloc(ctx, NL + 1));
        const unsigned nb = grid_for(mr, kScanTile);
        if (nb <= kPlaceTiles) {
            Buf<uint64_t> sums;
            RAMA_TRY(sums.alloc(ctx, (size_t)nb * lists));
            if (nb > 1) {
                ProfScope ps_(ctx, "k_place_sums", (double)(mr * 4 * (size_t)lists));
                k_place_sums<NL><<<dim3(nb, (unsigned)lists), kBlock, 0, ctx.stream>>>(cp, mr, sums.get());
            }
            LAUNCH_TRY(ctx, "place_sums");
            {
                ProfScope ps_(ctx, "k_places", (double)(mr * 12 * (size_t)lists));
                k_places<NL><<<dim3(nb, (unsigned)lists), kBlock, 0, ctx.stream>>>(cp, op, mr, sums.get(), summary.get());
            }
            LAUNCH_TRY(ctx, "places");
            uint64_t back[NL + 1] = {};
            RAMA_TRY(read_back(ctx, back, summary.get(), (size_t)lists * 8, n_heavy.get() + 1, 4));
            for (int k = 0; k < NL; ++k) tot[k] = k < lists ? back[k] : 0;
            tot[NL] = (uint32_t)back[lists];
        } else {
            for (int k = 0; k < lists; ++k)
                RAMA_TRY((exclusive_scan<uint64_t>(ctx, PtrInput<uint32_t>{cnt[k].get()}, off[k].get(), mr)));
            k_cycle_totals<NL><<<1, 64, 0, ctx.stream>>>(op, mr, lists, n_heavy.get() + 1, summary.get());
            LAUNCH_TRY(ctx, "cycle_totals");
            RAMA_TRY(read_back(ctx, tot, summary.get(), sizeof(tot)));
        }
        if (tot[NL]) return fail(ctx, RAMA_ERR_CAPACITY, "a repulsive edge closes 2^32 - 1 or more cycles of one length");
    }
    for (int k = 0; k < lists; ++k) {
        out.n[k] = (int64_t)tot[k];
        all += tot[k];
    }
    int32_t *to[kCycleLists] = {};
    if (sink) RAMA_TRY(sink(out.n, to));
    double list_bytes = 0.0;
    for (int k = 0; k < lists; ++k) {
        RAMA_TRY(list_fits(ctx, k, out.n[k]));
        if (!sink) RAMA_TRY(out.v[k].alloc(ctx, (size_t)(k + 3) * tot[k]));
        vp.p[k] = sink ? to[k] : out.v[k].get();
        list_bytes += 4.0 * (k + 3) * (double)tot[k];
    }
    if (all == 0) return RAMA_OK;
    int live = 0;   // the lists that hold any cycle: the fill pass leaves the count and offset arrays of the others alone
    for (int k = 0; k < lists; ++k)
        if (tot[k]) live |= 1 << k;
    // The fill pass visits the repulsive edges that have cycles.  Listing them first pays on long lists; a
    // short one is visited whole (an edge without cycles costs its thread three loads) and the launches and
    // the count read-back of the listing are saved.
    const bool list_hits = mr > kListHitsFrom;
    Buf<uint32_t> hit;
    uint32_t nh = (uint32_t)mr;
    if (list_hits) {
        HasCycles<MAXL> has{cp, live};
        ScanPlan<uint32_t> hits;
        RAMA_TRY((scan_plan_alloc<uint32_t>(ctx, mr, 0, hits)));
        RAMA_TRY((scan_totals<uint32_t>(ctx, has, hits)));
        nh = hits.total;
        RAMA_TRY(hit.alloc(ctx, nh));
        RAMA_TRY((scan_emit<uint32_t>(ctx, has, CollectHitsEmit{hit.get()}, hits, (double)((size_t)nh * 4))));
    }
    const double fill_bytes = (double)((size_t)nh * (12 + 12 * (size_t)lists) + ((size_t)n + 1) * 4 + mp * 8) + list_bytes;
    bool long_cycles = false;   // is there any cycle of length 5 or more to write?
    for (int k = 2; k < lists; ++k) long_cycles |= tot[k] != 0;
    if constexpr (MAXL == 5) {
        if (hashed) {
            auto write = [&](auto lanes, auto slots, size_t edges, const uint32_t *list, const uint32_t *n_list) {
                constexpr int G = decltype(lanes)::value, S = decltype(slots)::value;
                ProfScope ps_(ctx, "k_fill_cycles_hash", n_list ? 0.0 : fill_bytes);
                k_fill_cycles_hash<G, S><<<grid_striding(edges, HashBlock<G>::edges), HashBlock<G>::threads, 0, ctx.stream>>>(
                    nh, list, n_list, ri, rj, adj, max_len, live, cp, op, vp);
            };
            using std::integral_constant;
            const uint32_t *hits = list_hits ? hit.get() : nullptr;
            if (wide) write(integral_constant<int, 64>{}, integral_constant<int, 1024>{}, nh, hits, nullptr);
            else write(integral_constant<int, 16>{}, integral_constant<int, 256>{}, nh, hits, nullptr);
            LAUNCH_TRY(ctx, "fill_cycles_hash");
            write(integral_constant<int, 64>{}, integral_constant<int, kSpillSlots>{}, kSpillGroups, spill.get(), n_heavy.get() + 2);
            LAUNCH_TRY(ctx, "fill_cycles_hash");
            ProfScope ps_(ctx, "k_fill_cycles_listed", 0.0);
            k_fill_cycles_listed<MAXL, true><<<kHeavyGroups, kBlock, 0, ctx.stream>>>(walk, ri, rj, adj, live, max_len, cp, op, vp);
        }
    }
    if (wide3) {
        ProfScope ps_(ctx, "k_fill_triangles_group", fill_bytes);
        k_triangles_group<true><<<grid_striding(nh, kTriEdges), kBlock, 0, ctx.stream>>>(nh, list_hits ? hit.get() : nullptr, ri, rj, adj, cp.p[0],
                                                                                  op.p[0], vp.p[0], tri_room_now(room, blocks));
    } else if (!hashed) {
        ProfScope ps_(ctx, MAXL == 3 ? "k_fill_cycles<3>" : MAXL == 5 ? "k_fill_cycles<5>" : "k_fill_cycles<7>", fill_bytes);
        if (meet && long_cycles)
            k_fill_cycles<MAXL, (MAXL >= 5)><<<grid_for(nh), kBlock, 0, ctx.stream>>>(nh, list_hits ? hit.get() : nullptr, ri, rj, adj, live, max_len, cp, op, vp);
        else
            k_fill_cycles<MAXL, false><<<grid_for(nh), kBlock, 0, ctx.stream>>>(nh, list_hits ? hit.get() : nullptr, ri, rj, adj, live, max_len, cp, op, vp);
    }
    LAUNCH_TRY(ctx, "fill_cycles");
    if (may_be_heavy) {
        ProfScope ps_(ctx, "k_fill_cycles_heavy", 0.0);
        k_fill_cycles_heavy<MAXL><<<kHeavyGroups, kBlock, 0, ctx.stream>>>(heavy.get(), n_heavy.get(), walk, ri, rj, adj, live, cp,
                                                                         op, vp);
        LAUNCH_TRY(ctx, "fill_cycles_heavy");
    }
    return RAMA_OK;
}

}  // namespace

rama_status find_cycles(Ctx &ctx, const Graph &g, int max_len, bool shortest_only, CycleLists &out, const CycleSink &sink)
{
    for (int k = 0; k < kCycleLists; ++k) { out.n[k] = 0; out.v[k].reset(); }
    out.n_attractive = 0; out.n_repulsive = 0;
    const size_t m = (size_t)g.m;
    if (m == 0 || max_len < 3) return RAMA_OK;
    RAMA_TRY(zero_page_recycle(ctx));
    if (max_len > kMaxCycleLen) return fail(ctx, RAMA_ERR_INVALID_ARG, "cycle length beyond the supported maximum");
    // sign partition
    ScanPlan<uint64_t> signs;
    RAMA_TRY((scan_plan_alloc<uint64_t>(ctx, m, 0, signs)));
    RAMA_TRY((scan_totals<uint64_t>(ctx, SignFlags{g.c.get()}, signs, g.sign_sums.get())));   // tile sums, if the graph brings them
    const uint32_t mp = (uint32_t)signs.total, mr = (uint32_t)(signs.total >> 32);
    out.n_attractive = mp; out.n_repulsive = mr;
    if (mp == 0 || mr == 0) return RAMA_OK;
    RAMA_TRY(adjacency_fits(ctx, mp, mr));
    Buf<int32_t> pi, pj, ri, rj;
    Buf<uint32_t> lkey, lval;
    RAMA_TRY(pi.alloc(ctx, mp));
    RAMA_TRY(pj.alloc(ctx, mp));
    RAMA_TRY(ri.alloc(ctx, mr));
    RAMA_TRY(rj.alloc(ctx, mr));
    RAMA_TRY((scan_emit<uint64_t>(ctx, SignFlags{g.c.get()},
                                  SplitSignEmit{g.i.get(), g.j.get(), pi.get(), pj.get(), ri.get(), rj.get()},
                                  signs, (double)(m * 8 + (size_t)mp * 8 + (size_t)mr * 8))));
    signs.offs.reset();
    // positive CSR
    const int32_t n = g.n;
    Buf<int32_t> up_ptr, low_ptr, rowptr, nb;
    RAMA_TRY(up_ptr.alloc(ctx, (size_t)n + 1));
    RAMA_TRY(low_ptr.alloc(ctx, (size_t)n + 1));
    RAMA_TRY(rowptr.alloc(ctx, (size_t)n + 1));
    RAMA_TRY(nb.alloc(ctx, (size_t)2 * mp + kWideRow));   // padded: short rows are read eight entries at a time
    // The choice between the two searches for lengths 4 and 5 needs the longest attractive row when the
    // rows are short on average (see count_and_fill).
    const bool want_longest = max_len >= 4 && max_len <= 5 && ctx.cycle_search == 0 && 2 * (size_t)mp <= (size_t)9 * (size_t)n / 2;
    Buf<uint32_t> longest;
    if (want_longest) {
        RAMA_TRY(zeroed<uint32_t>(ctx, 1, longest));
    }
    RAMA_TRY((row_bounds<int32_t, int32_t>(ctx, pi.get(), mp, n, up_ptr.get())));
    // lower neighbours: the attractive pairs read as (j, i), sorted by j (stable: i stays ascending)
    RAMA_TRY((radix_sort_pairs_from<uint32_t, uint32_t>(ctx, (const uint32_t *)pj.get(), (const uint32_t *)pi.get(), lkey, lval, mp,
                                                        bits_for((uint64_t)n), (uint64_t)n)));
    RAMA_TRY((row_bounds<uint32_t, int32_t>(ctx, lkey.get(), mp, n, low_ptr.get())));
    {
        ProfScope ps_(ctx, "k_add_ptr", (double)(((size_t)n + 1) * 12));
        k_add_ptr<<<grid_for((size_t)n + 1), kBlock, 0, ctx.stream>>>(n, up_ptr.get(), low_ptr.get(), rowptr.get(),
                                                                  want_longest ? longest.get() : nullptr);
    }
    LAUNCH_TRY(ctx, "add_ptr");
    {
        ProfScope ps_(ctx, "k_fill_adj", (double)((size_t)mp * 24 + ((size_t)n + 1) * 12));
        k_fill_adj<<<grid_for(mp), kBlock, 0, ctx.stream>>>(mp, pi.get(), pj.get(), lkey.get(), lval.get(), up_ptr.get(),
                                                        low_ptr.get(), rowptr.get(), nb.get());
    }
    LAUNCH_TRY(ctx, "fill_adj");
    pi.reset(); pj.reset(); lkey.reset(); lval.reset(); up_ptr.reset(); low_ptr.reset();
    Adj adj{rowptr.get(), nb.get()};
    uint32_t longest_row = 0xffffffffu;   // unknown
    if (want_longest) RAMA_TRY(read_back(ctx, &longest_row, longest.get(), 4));
    // one instantiation per depth class: triangles are row intersections and need no walk state
    if (max_len <= 3)
        return count_and_fill<3>(ctx, (size_t)mr, ri.get(), rj.get(), adj, n, (size_t)mp, max_len, shortest_only, out, sink);
    if (max_len <= 5)
        return count_and_fill<5>(ctx, (size_t)mr, ri.get(), rj.get(), adj, n, (size_t)mp, max_len, shortest_only, out, sink,
                                 longest_row);
    return count_and_fill<kMaxCycleLen>(ctx, (size_t)mr, ri.get(), rj.get(), adj, n, (size_t)mp, max_len, shortest_only, out, sink);
}

}  // namespace rama
