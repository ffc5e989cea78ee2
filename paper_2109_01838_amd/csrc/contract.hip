// Steps a4-a6: one primal update (paper Sec. 3.1: Lemma 1, Lemma 3, algorithm
// "Parallel-Edge-Contraction", "Maximum matching"; appendix algorithm "GPU Edge-Contraction").
//
//   S   : handshake matching on the edges with c > tau.  Edges are ranked by (cost, position in
//         the canonical list) packed into one 64-bit word, so "each node points at its best
//         incident candidate" is an integer atomicMax per endpoint -- order independent, hence
//         deterministic.  An edge both of whose endpoints point at it is matched; rounds repeat
//         on the shrinking list of edges whose endpoints are both still free (one kernel per round
//         on lists of up to 2^20: compaction of the survivors fused with their next proposals,
//         every candidate finding out itself whether its ends were matched; longer lists are
//         accepted by a kernel in front of it; the last 8192 on up to 16384 nodes, or 4096 on more, by
//         one workgroup); the list carries
//         endpoints and rank word, so a round streams it and touches no edge array.
//   f'  : connected components of (V,S) by min-label hooking + pointer jumping; a component is
//         represented by its smallest node; new ids are the ranks of the representatives.
//   S'  : when the matching joins fewer than forest_ratio*|V| pairs: maximum spanning forest of the
//         candidate edges (Boruvka rounds with the same atomicMax ranks) minus, for every
//         repulsive edge inside a tree, the lowest edge of its tree path (trees rooted breadth
//         first, paths walked up from both ends).
//   A'  : endpoints relabelled through f', re-oriented, sorted by (row, col) with the cost as
//         payload (stable), runs of equal pairs summed in order, loops dropped.
#include "prim.h"
#include "steps.h"

namespace rama {

namespace {

struct CandFlag {
    static constexpr int bytes = 4;   // bytes read per item
    static constexpr const char *tag = "CandFlag";
    const float *c;
    float tau;
    __device__ __forceinline__ uint32_t operator()(size_t e) const { return c[e] > tau ? 1u : 0u; }
};

// consumer of the scan over CandFlag: the list of candidate edges
struct CollectEmit {
    static constexpr const char *tag = "Collect";
    uint32_t *act;
    __device__ __forceinline__ void operator()(size_t e, uint32_t cand, uint32_t p) const
    {
        if (cand) act[p] = (uint32_t)e;
    }
};

// Both endpoints of a candidate edge learn its rank.  Edge lists are in canonical order, also where candidates were taken
// out of them, so neighbouring lanes often share the first endpoint: those lanes combine their ranks and only the last lane
// of a run issues the atomic.  (Combining any two lanes with the same node is valid whatever the list order; runs only make
// it pay.)  Lanes without a candidate take part with their node and no rank, so that they do not break up a run.
// Every step doubles the length of the stretch that is combined, and when no run of the wave is longer than that there is no
// further step: bounded by the shuffles (six steps of them, always taken, were 18 LDS exchanges per candidate, and rows of a
// volume have three entries) and by the atomics.  First lists of a 320^3 solve 6.5 -> 5.3 ms, of a 127x160x161 volume 122 ->
// 100 us.
__device__ __forceinline__ void propose_edge(bool valid, int32_t u, int32_t v, unsigned long long r,
                                             unsigned long long *best)
{
    if (!__ballot(valid)) return;      // uniform
    const int lane = lane_id();
    unsigned long long ru = valid ? r : 0ull;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const bool same = __shfl_up(u, off, 64) == u && lane >= off;
        if (!__ballot(same)) break;    // uniform
        const unsigned long long other = __shfl_up(ru, off, 64);
        if (same && other > ru) ru = other;
    }
    const int32_t next = __shfl_down(u, 1, 64);
    if (ru && (lane == 63 || next != u)) atomicMax(&best[u], ru);
    if (valid) atomicMax(&best[v], r);
}

// The matching keeps its candidates packed -- endpoints and rank word, 16 bytes per candidate in three
// arrays -- so that a handshake round reads its list contiguously instead of reaching through the edge
// id into i, j and c of an ever sparser subset of the edges.
struct Cands {
    int32_t *u, *v;
    unsigned long long *r;
};
// consumer of the scan over CandFlag: the packed candidate list; with `best` set, the candidates also make
// the proposals of the first handshake round on the way (the list is then not read once more just for that)
struct PackCandsEmit {
    static constexpr const char *tag = "PackCands";
    static constexpr bool whole_wave = true;
    const int32_t *i, *j;
    const float *c;
    Cands out;
    unsigned long long *best;
    struct Item { int32_t u, v; float c; };
    __device__ __forceinline__ Item load(size_t e) const { return {i[e], j[e], c[e]}; }
    __device__ __forceinline__ void operator()(size_t e, uint32_t cand, uint32_t p, const Item &x) const
    {
        unsigned long long r = 0ull;
        if (cand) {
            r = edge_rank(x.c, (uint32_t)e);
            out.u[p] = x.u; out.v[p] = x.v; out.r[p] = r;
        }
        if (best) propose_edge(cand != 0u, x.u, x.v, r, best);   // uniform
    }
};

// words that atomics of the same launch change are read where the atomics are carried out
template <typename T>
__device__ __forceinline__ T load_past_cache(const T *p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }

// Where a handshake round finds its candidates.  The first list is dense.  The survivors of a round go to kLists lists,
// workgroup b's to list b % kLists; each has as many places as the first round's workgroups of its number have candidates, and
// a counter in a cache line of its own: survivors | pairs made << 32.  With one counter for all, its two atomics took 15 ns each
// of every workgroup, one after the other, and that was what a round waited for: 4e5 candidates 23 us and 10 with the lists,
// 6.5e6 108 and 65; all rounds of a 320^3 solve 5.9 ms and 4.1.
// Lengths are read from device memory, so that several handshake rounds can be enqueued without the host looking at the counts
// in between; the grid is sized from an upper bound and surplus workgroups leave.
constexpr uint32_t kLists = 32, kListWords = 8;      // 64-bit words of a counter's line
struct ListPlaces {
    uint32_t each, more;      // places of a list, the first `more` of them one workgroup's more: `group`
    uint32_t group;
    __host__ __device__ __forceinline__ uint32_t begin(uint32_t l) const { return l * each + (l < more ? l : more) * group; }
};
struct CandList {
    Cands a;
    const uint32_t *n_dense;              // length of the dense list
    const unsigned long long *counts;     // of the lists; nullptr: the list is dense
    ListPlaces places;
};
// the workgroup's candidates: places [first, end) of the arrays, at most GROUP of them
template <uint32_t GROUP>
__device__ __forceinline__ bool group_of(const CandList &l, size_t &first, size_t &end)
{
    if (!l.counts) {
        first = (size_t)blockIdx.x * GROUP; end = *l.n_dense;
    } else {
        const uint32_t s = blockIdx.x % kLists;
        end = l.places.begin(s);
        first = end + (size_t)(blockIdx.x / kLists) * GROUP;
        end += (uint32_t)l.counts[(size_t)s * kListWords];
    }
    return first < end;
}

// matched edges fix their endpoints
__global__ __launch_bounds__(kBlock) void k_accept(CandList list, const unsigned long long *best, int32_t *mate)
{
    size_t first, end;
    if (!group_of<kBlock>(list, first, end)) return;
    const size_t k = first + threadIdx.x;
    if (k >= end) return;
    const int32_t u = list.a.u[k], v = list.a.v[k];
    const unsigned long long r = list.a.r[k];
    if (best[u] == r && best[v] == r) { mate[u] = v; mate[v] = u; }
}

// Survivors (both endpoints still free) move to the next list and at once propose for the next
// round.  Every workgroup compacts 2048 candidates locally and reserves its output range with a
// single atomicAdd, which notes the pairs as well; the order of the ranges varies from run to run, which is harmless: proposals
// (atomicMax) and the accept test do not depend on the order of the list.
// Three rank arrays rotate: this round's proposals were read by k_accept, the survivors propose into
// the second, and they clear their endpoints' words in the third, which takes the proposals of the
// round after next -- so only survivors pay for clearing, and nobody clears what somebody else
// is proposing into.
constexpr int kAdvItems = 8;
// Lists of up to 2^20 candidates give a workgroup 512 instead of 2048: with eight a thread they do not fill the chip, and a
// thread's eight combine-and-propose steps wait one after the other (contraction of a 300x301 long-range grid 3.06 ->
// 2.80 ms, 128^2 solve 3.90 -> 3.71, 512^2 8.82 -> 8.59, 6-NN graph of 10^6 points 14.44 -> 14.25).
constexpr size_t kAdvMedium = size_t(1) << 20;
constexpr uint32_t kMatchBatchMax = 1u << 20;   // candidate lists up to this length run their handshake rounds in batches
// The edge a node points at (its rank word names it) is matched iff its other end points at it as well: lists of up to 2^20
// candidates have each candidate find out for both of its ends by itself (ACCEPTS: four more gathers, no k_accept launch in
// front, and the pairs are noted here).  Contraction of a 300x301 long-range grid 2.68 ->
// 2.53 ms, 512^2 solve 8.38 -> 8.07, 6-NN graph of 10^6 points 14.28 -> 13.98; on longer lists the gathers cost more than the launch.
template <int ITEMS, bool ACCEPTS>
__global__ __launch_bounds__(kBlock) void k_advance(CandList list, int32_t *mate, Cands next,
                                                    const unsigned long long *best, const int32_t *gi, const int32_t *gj,
                                                    unsigned long long *best_next, unsigned long long *best_after,
                                                    unsigned long long *counters)
{
    __shared__ uint32_t s_base, s_wave[4], s_pairs[4];
    size_t group, na;
    if (!group_of<kBlock * ITEMS>(list, group, na)) return;   // the whole workgroup: nothing left of the list here
    const Cands &a = list.a;
    const int w = threadIdx.x >> 6, lane = lane_id();
    const size_t base = group + (size_t)w * (64 * ITEMS) + lane;
    int32_t u[ITEMS], v[ITEMS];
    unsigned long long r[ITEMS];
    uint32_t where[ITEMS];
    uint32_t live = 0, won = 0, cnt = 0, pairs = 0;     // bit q: candidate q
    // a thread's candidates take every step together (places behind the end read the last one): one after the other, each of
    // them would wait for its chain of gathers alone
#pragma unroll
    for (int q = 0; q < ITEMS; ++q) {
        const size_t k = base + (size_t)q * 64, at = k < na ? k : na - 1;
        u[q] = a.u[at]; v[q] = a.v[at];
        if (ACCEPTS) r[q] = a.r[at];
    }
    if constexpr (ACCEPTS) {
        unsigned long long wu[ITEMS], wv[ITEMS], pu[ITEMS], pv[ITEMS];
#pragma unroll
        for (int q = 0; q < ITEMS; ++q) { wu[q] = best[u[q]]; wv[q] = best[v[q]]; }
        int32_t xu[ITEMS], yu[ITEMS], xv[ITEMS], yv[ITEMS];
#pragma unroll
        for (int q = 0; q < ITEMS; ++q) {
            const uint32_t eu = 0xFFFFFFFFu - (uint32_t)wu[q], ev = 0xFFFFFFFFu - (uint32_t)wv[q];
            xu[q] = gi[eu]; yu[q] = gj[eu]; xv[q] = gi[ev]; yv[q] = gj[ev];
        }
#pragma unroll
        for (int q = 0; q < ITEMS; ++q) { pu[q] = best[xu[q] == u[q] ? yu[q] : xu[q]]; pv[q] = best[xv[q] == v[q] ? yv[q] : xv[q]]; }
#pragma unroll
        for (int q = 0; q < ITEMS; ++q) {
            const bool pair = wu[q] == r[q] && wv[q] == r[q], in = base + (size_t)q * 64 < na;
            if (in && pair) won |= 1u << q;
            if (in && !pair && pu[q] != wu[q] && pv[q] != wv[q]) live |= 1u << q;
        }
    } else {
        int32_t mu[ITEMS], mv[ITEMS];
#pragma unroll
        for (int q = 0; q < ITEMS; ++q) { mu[q] = mate[u[q]]; mv[q] = mate[v[q]]; }
#pragma unroll
        for (int q = 0; q < ITEMS; ++q) {
            const bool in = base + (size_t)q * 64 < na;
            if (in && mu[q] == v[q]) won |= 1u << q;               // this very edge was matched in the round that just ended
            if (in && mu[q] < 0 && mv[q] < 0) live |= 1u << q;
        }
#pragma unroll
        for (int q = 0; q < ITEMS; ++q) r[q] = a.r[(live & (1u << q)) ? base + (size_t)q * 64 : group];   // most do not survive
    }
#pragma unroll
    for (int q = 0; q < ITEMS; ++q) {
        const bool ok = (live & (1u << q)) != 0u, pair = (won & (1u << q)) != 0u;
        if (ACCEPTS && pair) { mate[u[q]] = v[q]; mate[v[q]] = u[q]; }
        pairs += (uint32_t)__popcll(__ballot(pair));
        const unsigned long long vote = __ballot(ok);
        where[q] = cnt + (uint32_t)__popcll(vote & ((1ull << lane) - 1ull));
        cnt += (uint32_t)__popcll(vote);
        if (ok) {
            best_after[u[q]] = 0ull;
            best_after[v[q]] = 0ull;
        }
        propose_edge(ok, u[q], v[q], r[q], best_next);
    }
    if (lane == 0) { s_wave[w] = cnt; s_pairs[w] = pairs; }
    __syncthreads();
    if (threadIdx.x == 0) {
        const uint32_t total = s_wave[0] + s_wave[1] + s_wave[2] + s_wave[3];
        const uint32_t made = s_pairs[0] + s_pairs[1] + s_pairs[2] + s_pairs[3], l = blockIdx.x % kLists;
        const unsigned long long both = (unsigned long long)total | (unsigned long long)made << 32;
        s_base = list.places.begin(l) + (both ? (uint32_t)atomicAdd(&counters[(size_t)l * kListWords], both) : 0u);
    }
    __syncthreads();
    uint32_t off = s_base;
#pragma unroll
    for (int k = 0; k < 3; ++k)
        if (k < w) off += s_wave[k];
#pragma unroll
    for (int q = 0; q < ITEMS; ++q)
        if (live & (1u << q)) {
            const uint32_t p = off + where[q];
            next.u[p] = u[q]; next.v[p] = v[q]; next.r[p] = r[q];
        }
}

// The rest of the matching for a list that one workgroup holds, and the host hears of it once; a longer list is left as it
// is.  Candidates stay in registers, the nodes' rank words in LDS: by the node's number where the graph has at most
// kFinishDirect nodes, else by its place in a hash table, which lists of half the length fill to four fifths at most.
// A handshake is three barriers that wait for LDS only, about 0.8 us (4 with the words in memory, whose four round trips a
// barrier waits for each).
// With the matching complete, the new nodes of a graph of up to kNumberMax nodes are numbered here as well (fmap; see
// NumberPairsEmit): all mates are read at once, and one scan numbers them (four turns of reading, scanning and storing took
// 22 us for 26000 nodes).  The message to the host goes out in front of that: mail[1] length of the first list | candidates left
// << 32, mail[2]: pairs made here and in the rounds enqueued with this launch, whose counters come along.
constexpr int kFinishThreads = 1024, kFinishItems = 8, kFinishWaves = kFinishThreads / 64;
constexpr int kFinishDirect = 1 << 14, kFinishSlots = 10240;
constexpr uint32_t kFinishMax = kFinishThreads * kFinishItems, kFinishMaxHashed = kFinishMax / 2;
static_assert(2 * kFinishMaxHashed <= kFinishSlots / 5 * 4 && kFinishSlots * 12 <= kFinishDirect * 8, "the table keeps room and takes the words' place");
__host__ __device__ constexpr uint32_t finish_max(int n_nodes) { return n_nodes <= kFinishDirect ? kFinishMax : kFinishMaxHashed; }
constexpr int kNumberMax = 1 << 15, kNumberRows = kNumberMax / kFinishThreads;
__global__ __launch_bounds__(kFinishThreads) void k_handshake_finish(const uint32_t *n_first, CandList list, int32_t *mate,
                                                                     int rounds_left, int n_nodes, int32_t *fmap,
                                                                     const unsigned long long *counters, int n_counters, MailWord *mail, uint64_t seq)
{
    constexpr unsigned long long kMatched = ~0ull;      // in a node's word: no candidate's rank
    __shared__ unsigned long long s_best[kFinishDirect];
    __shared__ uint32_t s_left, s_pairs, s_any[2], s_wave[kFinishWaves], s_before[kLists];
    const uint32_t tid = threadIdx.x;
    const int lane = lane_id(), w = (int)(tid >> 6);
    const Cands &a = list.a;
    // candidates, and those in the lists in front of a list
    uint32_t n, before = 0;
    if (!list.counts) {
        n = *list.n_dense;
    } else {
        const uint32_t x = lane < (int)kLists ? (uint32_t)list.counts[(size_t)lane * kListWords] : 0u;
        const uint32_t inc = wave_inclusive_scan(x);
        before = inc - x;
        n = wave_last(inc);
    }
    if (tid < kLists) s_before[tid] = before;
    if (tid == 0) { s_left = 0u; s_pairs = 0u; s_any[0] = 0u; s_any[1] = 0u; }
    lds_barrier();
    uint32_t pairs = 0;      // made in the rounds enqueued with this launch
    for (int k = (int)tid; k < n_counters * (int)kLists; k += kFinishThreads) pairs += (uint32_t)(counters[(size_t)k * kListWords] >> 32);
    auto tell = [&](uint32_t left, uint32_t made) {      // the first wave
        if (lane == 0) { mail_put(mail + 1, (uint64_t)*n_first | (uint64_t)left << 32); mail_put(mail + 2, (uint64_t)made); }
        mail_send_wave(mail, seq);
    };
    if (n > finish_max(n_nodes)) {      // uniform
        pairs = wave_sum(pairs);
        if (lane == 0 && pairs) atomicAdd(&s_pairs, pairs);
        __syncthreads();
        if (w == 0) tell(n, s_pairs);
        return;
    }
    int32_t u[kFinishItems], v[kFinishItems];
    unsigned long long r[kFinishItems];
    uint32_t alive = 0;
#pragma unroll
    for (int q = 0; q < kFinishItems; ++q) {
        const uint32_t k = tid + (uint32_t)q * kFinishThreads;
        u[q] = 0; v[q] = 0; r[q] = 0ull;
        if (k < n) {
            uint32_t at = k;
            if (list.counts) {      // the last list with at most k candidates in front of it
                uint32_t l = 0;
#pragma unroll
                for (uint32_t step = kLists / 2; step > 0; step >>= 1)
                    if (s_before[l + step] <= k) l += step;
                at = list.places.begin(l) + (k - s_before[l]);
            }
            u[q] = a.u[at]; v[q] = a.v[at]; r[q] = a.r[at];
            alive |= 1u << q;
        }
    }
    const bool direct = n_nodes <= kFinishDirect;
    int32_t *s_node = reinterpret_cast<int32_t *>(s_best + kFinishSlots);
    for (int k = (int)tid; k < (direct ? n_nodes : kFinishSlots); k += kFinishThreads) {
        s_best[k] = 0ull;
        if (!direct) s_node[k] = -1;
    }
    lds_barrier();
    auto place_of = [&](int32_t node) {
        if (direct) return node;
        uint32_t h = (uint32_t)(((uint64_t)((uint32_t)node * 0x9E3779B1u) * (uint32_t)kFinishSlots) >> 32);
        for (;;) {      // the table is never full: the walk ends
            const int32_t old = atomicCAS(&s_node[h], -1, node);
            if (old == -1 || old == node) return (int32_t)h;
            h = h + 1 == (uint32_t)kFinishSlots ? 0u : h + 1;
        }
    };
    int32_t su[kFinishItems], sv[kFinishItems];
#pragma unroll
    for (int q = 0; q < kFinishItems; ++q) {
        su[q] = 0; sv[q] = 0;
        if (alive & (1u << q)) {
            su[q] = place_of(u[q]); sv[q] = place_of(v[q]);
            atomicMax(&s_best[su[q]], r[q]); atomicMax(&s_best[sv[q]], r[q]);
        }
    }
    if (__ballot(alive != 0u) && lane == 0) s_any[0] = 1u;
    for (int round = 0; round < rounds_left; ++round) {
        lds_barrier();
        if (!s_any[round & 1]) break;      // uniform
        if (tid == 0) s_any[(round + 1) & 1] = 0u;
#pragma unroll
        for (int q = 0; q < kFinishItems; ++q)
            if ((alive & (1u << q)) && s_best[su[q]] == r[q] && s_best[sv[q]] == r[q]) {
                mate[u[q]] = v[q]; mate[v[q]] = u[q];
                s_best[su[q]] = kMatched; s_best[sv[q]] = kMatched;      // whoever reads it in this step has lost either way
                ++pairs;
            }
        lds_barrier();
#pragma unroll
        for (int q = 0; q < kFinishItems; ++q)
            if (alive & (1u << q)) {
                if (s_best[su[q]] == kMatched || s_best[sv[q]] == kMatched) alive &= ~(1u << q);
                else { s_best[su[q]] = 0ull; s_best[sv[q]] = 0ull; }
            }
        if (__ballot(alive != 0u) && lane == 0) s_any[(round + 1) & 1] = 1u;
        lds_barrier();
#pragma unroll
        for (int q = 0; q < kFinishItems; ++q)
            if (alive & (1u << q)) { atomicMax(&s_best[su[q]], r[q]); atomicMax(&s_best[sv[q]], r[q]); }
    }
    const uint32_t n_left = wave_sum((uint32_t)__popc(alive)), n_pairs = wave_sum(pairs);
    if (lane == 0) { atomicAdd(&s_left, n_left); atomicAdd(&s_pairs, n_pairs); }
    __syncthreads();      // the mates as well
    if (w == 0) tell(s_left, s_pairs);      // the host goes on; what it enqueues waits for the numbers
    if (fmap) {      // uniform; a wave takes `rows` rows of 64 nodes
        const int rows = (n_nodes + kFinishThreads - 1) / kFinishThreads, base = w * rows * 64 + lane;
        const uint64_t below = (1ull << lane) - 1ull;
        int32_t m[kNumberRows];
        uint32_t roots = 0, mine = 0;      // bit q: the node of row q
#pragma unroll
        for (int q = 0; q < kNumberRows; ++q)
            if (q < rows) {      // uniform, as below: a workgroup that works alone is bound by the instructions it issues
                const int node = base + q * 64;
                m[q] = node < n_nodes ? mate[node] : 0;
            }
#pragma unroll
        for (int q = 0; q < kNumberRows; ++q)
            if (q < rows) {
                const int node = base + q * 64;
                const bool root = node < n_nodes && (m[q] < 0 || m[q] > node);
                roots |= root ? 1u << q : 0u;
                mine += (uint32_t)__popcll(__ballot(root));
            }
        if (lane == 0) s_wave[w] = mine;
        __syncthreads();
        uint32_t number = 0;
#pragma unroll
        for (int k = 0; k < kFinishWaves - 1; ++k) number += k < w ? s_wave[k] : 0u;
#pragma unroll
        for (int q = 0; q < kNumberRows; ++q)
            if (q < rows) {
                const uint64_t row = __ballot((roots >> q) & 1u);
                if ((roots >> q) & 1u) {
                    const int32_t x = (int32_t)(number + (uint32_t)__popcll(row & below));
                    fmap[base + q * 64] = x;
                    if (m[q] >= 0) fmap[m[q]] = x;
                }
                number += (uint32_t)__popcll(row);
            }
    }
}

// mail[1]: candidates in a round's lists | in the longest of them << 32, mail[2]: pairs made in the round
__global__ __launch_bounds__(64) void k_look_at_lists(const unsigned long long *counts, MailWord *mail, uint64_t seq)
{
    const unsigned long long x = lane_id() < (int)kLists ? counts[(size_t)lane_id() * kListWords] : 0ull;
    const uint32_t n = wave_sum((uint32_t)x), pairs = wave_sum((uint32_t)(x >> 32));
    uint32_t longest = (uint32_t)x;
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) longest = max(longest, (uint32_t)__shfl_xor((int)longest, off, 64));
    if (lane_id() == 0) { mail_put(mail + 1, (uint64_t)n | (uint64_t)longest << 32); mail_put(mail + 2, (uint64_t)pairs); }
    mail_send_wave(mail, seq);
}

// The components of a matching are its pairs, represented by the smaller node: new numbers straight from the mates.
struct IsPairRoot {
    static constexpr int bytes = 4;   // bytes read per item
    static constexpr const char *tag = "IsPairRoot";
    const int32_t *mate;
    __device__ __forceinline__ uint32_t operator()(size_t v) const
    {
        const int32_t w = mate[v];
        return w < 0 || w > (int32_t)v ? 1u : 0u;
    }
};
// consumer of the scan over IsPairRoot: a representative numbers itself and its partner
struct NumberPairsEmit {
    static constexpr const char *tag = "NumberPairs";
    const int32_t *mate;
    int32_t *fmap;
    using Item = int32_t;
    __device__ __forceinline__ Item load(size_t v) const { return mate[v]; }
    __device__ __forceinline__ void operator()(size_t v, uint32_t root, uint32_t number, Item w) const
    {
        if (!root) return;
        fmap[v] = (int32_t)number;
        if (w >= 0) fmap[w] = (int32_t)number;
    }
};

// ---- connected components of (V,S) -------------------------------------------------------------
__global__ __launch_bounds__(kBlock) void k_iota(size_t n, int32_t *p)
{
    size_t v = (size_t)blockIdx.x * kBlock + threadIdx.x;
    if (v < n) p[v] = (int32_t)v;
}

__device__ __forceinline__ int32_t root_of(const int32_t *parent, int32_t v)
{
    int32_t p = parent[v];
    while (p != v) { v = p; p = parent[v]; }   // parents only ever decrease: the walk ends
    return v;
}

__global__ __launch_bounds__(kBlock) void k_hook(size_t ns, const int32_t *si, const int32_t *sj, int32_t *parent,
                                                 int32_t *changed)
{
    size_t e = (size_t)blockIdx.x * kBlock + threadIdx.x;
    if (e >= ns) return;
    int32_t a = root_of(parent, si[e]), b = root_of(parent, sj[e]);
    if (a == b) return;
    int32_t hi = max(a, b), lo = min(a, b);
    atomicMin(&parent[hi], lo);
    *changed = 1;
}

__global__ __launch_bounds__(kBlock) void k_flatten(size_t n, int32_t *parent)
{
    size_t v = (size_t)blockIdx.x * kBlock + threadIdx.x;
    if (v < n) parent[v] = root_of(parent, (int32_t)v);
}

struct IsRoot {
    static constexpr int bytes = 4;   // bytes read per item
    static constexpr const char *tag = "IsRoot";
    const int32_t *rep;
    __device__ __forceinline__ uint32_t operator()(size_t v) const { return rep[v] == (int32_t)v ? 1u : 0u; }
};

__global__ __launch_bounds__(kBlock) void k_number(size_t n, const int32_t *rep, const uint32_t *rank, int32_t *fmap)
{
    size_t v = (size_t)blockIdx.x * kBlock + threadIdx.x;
    if (v < n) fmap[v] = (int32_t)rank[rep[v]];
}

// ---- contraction ---------------------------------------------------------------------------------
struct InnerFlag {
    static constexpr int bytes = 16;   // bytes read per item
    static constexpr const char *tag = "InnerFlag";
    const int32_t *i, *j, *fmap;
    __device__ __forceinline__ uint32_t operator()(size_t e) const { return fmap[i[e]] == fmap[j[e]] ? 1u : 0u; }
};

// Relabelling gathers f' for both endpoints of every edge -- random 4-byte reads, the expensive
// part of the contraction -- so it is done exactly once: the packed pair of every edge is stored
// (a loop is seen by hi-lo = 0), what follows streams over the stored keys.
// raw[e] = (lo, hi-lo) in two 32-bit halves; *maxdiff collects the largest hi-lo.  A workgroup takes one tile of
// the scan that follows (kScanTile edges) and leaves the number of edges that are no loops in tile_sums: the scan
// over NotLoopKey then needs no pass of its own to count them.  It also clears its tile's word of sign_sums, where the sign
// counts of the contracted costs will go.
// diag (optional, behind a matching): a new node is a pair, and a canonical list has one edge between its nodes, whose cost is
// the diagonal's entry.  Collecting the inner edges, sorting them by their node and adding up runs of one were thirteen
// launches and a wait, 190 us for the 9.7e6 edges of a 127x160x161 grid; a pass of its own 44, here 12.
// With PARTS > 0 the sort's first digit (the top bits of lo, of which `shift` are left out) is counted on the way, for each of
// the PARTS tiles of the sort that the workgroup's edges make up: hist[digit][tile].
template <int PARTS>
__global__ __launch_bounds__(kBlock) void k_relabel_keys(size_t m, const int32_t *i, const int32_t *j,
                                                         const int32_t *fmap, uint64_t *raw, uint32_t *maxdiff,
                                                         uint32_t *tile_sums, uint64_t *sign_sums, uint32_t *hist, uint32_t nb, int shift, int bits,
                                                         const float *c, float *diag)
{
    constexpr int kParts = PARTS > 0 ? PARTS : 1, kPartItems = kScanItems / kParts;
    __shared__ uint32_t s_digits[kParts][kRadix];
    const size_t base = (size_t)blockIdx.x * kScanTile + threadIdx.x;
    uint32_t diff = 0, kept = 0;
    int32_t fa[kScanItems], fb[kScanItems];      // all gathers before the first store (behind the end: the last edge again)
#pragma unroll
    for (int q = 0; q < kScanItems; ++q) {
        const size_t e = base + (size_t)q * kBlock, at = e < m ? e : m - 1;
        fa[q] = i[at]; fb[q] = j[at];
    }
    if constexpr (PARTS > 0) {
#pragma unroll
        for (int p = 0; p < PARTS; ++p) s_digits[p][threadIdx.x] = 0u;
        __syncthreads();
    }
#pragma unroll
    for (int q = 0; q < kScanItems; ++q) { fa[q] = fmap[fa[q]]; fb[q] = fmap[fb[q]]; }
#pragma unroll
    for (int q = 0; q < kScanItems; ++q) {
        const size_t e = base + (size_t)q * kBlock;
        const int32_t a = fa[q], b = fb[q];
        const uint32_t d = (uint32_t)abs(a - b), lo = (uint32_t)min(a, b);
        if (e < m) {
            diff = d > diff ? d : diff;
            kept += a != b ? 1u : 0u;
            raw[e] = ((uint64_t)lo << 32) | d;
            if (diag && a == b) diag[a] = c[e];
        }
        if constexpr (PARTS > 0) {      // rows are nearly in order: most of a wave has the digit of its first lane
            uint64_t left = __ballot(e < m && a != b);
            if (left) {                 // uniform
                const uint32_t x = lo >> shift;
                const int first = __ffsll((long long)left) - 1;
                const uint32_t x0 = (uint32_t)__builtin_amdgcn_readlane((int)x, first);
                const uint64_t same = __ballot(x == x0) & left;
                if (lane_id() == first) atomicAdd(&s_digits[q / kPartItems][x0], (uint32_t)__popcll(same));
                left &= ~same;
                if (left & (1ull << lane_id())) atomicAdd(&s_digits[q / kPartItems][x], 1u);
            }
        }
    }
    kept = block_sum(kept);
    if (threadIdx.x == 0) { if (tile_sums) tile_sums[blockIdx.x] = kept; sign_sums[blockIdx.x] = 0ull; }
    if constexpr (PARTS > 0) {      // all have counted: the barriers of the sum
#pragma unroll
        for (int p = 0; p < PARTS; ++p) {
            const uint32_t tile = blockIdx.x * PARTS + p;
            if (threadIdx.x < (1u << bits) && tile < nb) hist[(size_t)threadIdx.x * nb + tile] = s_digits[p][threadIdx.x];
        }
    }
    block_max_into(diff, maxdiff);
}
struct NotLoopKey {
    static constexpr int bytes = 8;   // bytes read per item
    static constexpr const char *tag = "NotLoopKey";
    const uint64_t *raw;
    __device__ __forceinline__ uint32_t operator()(size_t e) const { return (uint32_t)raw[e] != 0u ? 1u : 0u; }
};
// The same as a source of the sort: its first pass reads the stored keys, and nothing is compacted in front of it (320^3 grid
// 93.9 -> 91.8 ms per solve, the compaction alone took 2.1; 61x97x131 8.11 -> 8.04, 512^2 long-range 7.63 -> 7.57).
struct RelabelledEdges {
    const uint64_t *raw;
    const float *c;
    int dbits;
    __device__ __forceinline__ uint64_t key(size_t e) const
    {
        const uint64_t x = raw[e];
        return ((x >> 32) << dbits) | (x & 0xFFFFFFFFull);
    }
    __device__ __forceinline__ bool takes_part(uint64_t k) const { return (k & ((uint64_t(1) << dbits) - 1u)) != 0u; }
    __device__ __forceinline__ uint32_t value(size_t e) const { return __float_as_uint(c[e]); }
};
// consumer of the scan over NotLoopKey: edge e that survives goes to place p
struct CompactKeysEmit {
    static constexpr const char *tag = "CompactKeys";
    const uint64_t *raw;
    const float *c;
    int dbits;
    uint64_t *key;
    uint32_t *val;
    struct Item { uint64_t k; float c; };
    __device__ __forceinline__ Item load(size_t e) const { return {raw[e], c[e]}; }
    __device__ __forceinline__ void operator()(size_t, uint32_t keep, uint32_t p, const Item &x) const
    {
        if (!keep) return;
        key[p] = ((x.k >> 32) << dbits) | (x.k & 0xFFFFFFFFull);
        val[p] = __float_as_uint(x.c);
    }
};

// consumer of the scan over InnerFlag: edge e inside a new node goes to place p.  (Positions of all edges, and a kernel that
// looks up both endpoints once more to use them, were two passes, 75 us on a 127x160x161
// grid, where this is one, 51.)
struct InnerEmit {
    static constexpr const char *tag = "Inner";
    const int32_t *i, *fmap;
    const float *c;
    uint32_t *key, *val;
    struct Item { int32_t a; float c; };
    __device__ __forceinline__ Item load(size_t e) const { return {fmap[i[e]], c[e]}; }
    __device__ __forceinline__ void operator()(size_t, uint32_t inner, uint32_t p, const Item &x) const
    {
        if (!inner) return;
        key[p] = (uint32_t)x.a;
        val[p] = __float_as_uint(x.c);
    }
};

struct HeadFlag {
    static constexpr int bytes = 8;   // bytes read per item
    static constexpr const char *tag = "HeadFlag";
    const uint64_t *key;
    __device__ __forceinline__ uint32_t operator()(size_t e) const { return ((e == 0) | (key[e] != key[e ? e - 1 : 0])) ? 1u : 0u; }
};

// Contraction of a middle-sized list behind one pass over the top bits of lo: a workgroup to a digit sorts the digit's edges in
// LDS, adds up the runs of equal pairs there, in order of appearance, and leaves its edges at the digit's place, not more than
// there were; counts[digit] tells how many.  The second field of the keys is as wide as a node's number; in LDS it gets
// the bits that the largest hi - lo needs, without which a row is one bucket of the in-LDS sort.
// Bounded by the instructions that one workgroup of sixteen waves issues (2600 edges: 3 us until they are there, 5 to sort, 2 to
// add up; a round's edges of a 300x301 long-range grid 14 us, where the in-LDS sort, the count of heads and the
// sums as launches of their own took 20 + 4 + 11).
__global__ __launch_bounds__(kLocalSortWaves * 64, 8) void k_sum_digit(const uint64_t *key, const uint32_t *val, const uint32_t *starts, int nbits, int low_bits,
                                                                      const uint32_t *maxdiff, uint32_t *counts, uint32_t *oversize,
                                                                      int32_t *ti, int32_t *tj, float *tc)
{
    using LS = LocalSort<uint32_t>;
    constexpr int kItems = LS::items;
    __shared__ LocalSortShared<uint32_t> S;
    __shared__ float s_val[LS::cap];
    __shared__ uint32_t s_runs[kLocalSortWaves];
    const uint32_t beg = starts[blockIdx.x], cnt = starts[blockIdx.x + 1] - beg;
    const int tid = (int)threadIdx.x, lane = lane_id(), w = tid >> 6;
    if (cnt == 0 || cnt > (uint32_t)LS::cap) {
        if (tid == 0) { counts[blockIdx.x] = 0u; if (cnt) *oversize = 1u; }
        return;
    }
    const int rows = (int)((cnt + LS::threads - 1) / LS::threads);
    const uint32_t first = (uint32_t)w * (uint32_t)rows * 64u + (uint32_t)lane;
    const uint32_t lo0 = (uint32_t)blockIdx.x << (low_bits - nbits), widest = *maxdiff;
    const int dbits = 32 - __clz((int)widest);      // at least one: there is an edge
    const uint32_t dmask = widest | ((1u << (dbits - 1)) - 1u);
    uint32_t k[kItems], v[kItems], rank[kItems];
#pragma unroll
    for (int r = 0; r < kItems; ++r) {
        k[r] = 0; v[r] = 0;
        const uint32_t p = first + (uint32_t)r * 64u;
        if (r < rows && p < cnt) {
            const uint64_t x = key[beg + p];
            k[r] = (((uint32_t)(x >> nbits) - lo0) << dbits) | ((uint32_t)x & dmask);
            v[r] = val[beg + p];
        }
    }
    local_sort<true>(S, k, v, rank, rows, cnt, low_bits - nbits + dbits);
#pragma unroll
    for (int r = 0; r < kItems; ++r)
        if (r < rows && first + (uint32_t)r * 64u < cnt) s_val[rank[r]] = __uint_as_float(v[r]);
    uint32_t heads = 0, mine = 0;
#pragma unroll
    for (int r = 0; r < kItems; ++r)
        if (r < rows) {
            const uint32_t p = first + (uint32_t)r * 64u;
            const bool head = p < cnt && (p == 0 || S.buf[p] != S.buf[p - 1]);
            heads |= head ? 1u << r : 0u;
            mine += (uint32_t)__popcll(__ballot(head));
        }
    if (lane == 0) s_runs[w] = mine;
    lds_barrier();
    uint32_t at = beg, all = 0;
#pragma unroll
    for (int q = 0; q < kLocalSortWaves; ++q) {
        const uint32_t x = s_runs[q];
        at += q < w ? x : 0u;
        all += x;
    }
    if (tid == 0) counts[blockIdx.x] = all;
#pragma unroll
    for (int r = 0; r < kItems; ++r)
        if (r < rows) {
            const uint64_t row = __ballot((heads >> r) & 1u);
            if ((heads >> r) & 1u) {
                uint32_t p = first + (uint32_t)r * 64u;
                const uint32_t x = S.buf[p], to = at + (uint32_t)__popcll(row & ((1ull << lane) - 1ull));
                float acc = s_val[p];
                for (++p; p < cnt && S.buf[p] == x; ++p) acc = acc + s_val[p];
                const uint32_t lo = lo0 + (x >> dbits);
                ti[to] = (int32_t)lo; tj[to] = (int32_t)(lo + (x & dmask)); tc[to] = acc;
            }
            at += (uint32_t)__popcll(row);
        }
}

// The digits' edges one behind the other, a workgroup to a digit; sign counts per kScanTile edges (see k_reduce_runs); the
// last workgroup tells the host: mail[1] number of edges, mail[2]: *oversize.
constexpr int kJoinThreads = 512;
__global__ __launch_bounds__(kJoinThreads) void k_join_digits(const uint32_t *starts, const uint32_t *counts, const int32_t *ti, const int32_t *tj, const float *tc,
                                                              int32_t *io, int32_t *jo, float *co, unsigned long long *sign_sums,
                                                              const uint32_t *oversize, MailWord *mail, uint64_t seq)
{
    constexpr int kTiles = LocalSort<uint32_t>::cap / kScanTile + 1;
    __shared__ uint32_t s_sum[kJoinThreads / 64], s_sign[kTiles];
    const int tid = (int)threadIdx.x;
    uint32_t x = 0;
    for (int d = tid; d < (int)blockIdx.x; d += kJoinThreads) x += counts[d];
    x = wave_sum(x);
    if (lane_id() == 0) s_sum[tid >> 6] = x;
    if (tid < kTiles) s_sign[tid] = 0u;
    __syncthreads();
    uint32_t at = 0;
#pragma unroll
    for (int w = 0; w < kJoinThreads / 64; ++w) at += s_sum[w];
    const uint32_t beg = starts[blockIdx.x], n = counts[blockIdx.x], tile0 = at / (uint32_t)kScanTile;
    if (blockIdx.x == gridDim.x - 1 && tid < 64) {
        if (tid == 0) {
            mail_put(mail + 1, (uint64_t)(at + n));
            mail_put(mail + 2, (uint64_t)*oversize);
        }
        mail_send_wave(mail, seq);
    }
    for (uint32_t k0 = 0; k0 < n; k0 += kJoinThreads) {      // uniform
        const uint32_t k = k0 + (uint32_t)tid;
        float c = 0.0f;
        if (k < n) {
            c = tc[beg + k];
            io[at + k] = ti[beg + k]; jo[at + k] = tj[beg + k]; co[at + k] = c;
        }
        // the wave's 64 places lie in one tile or in two
        const uint64_t pos = __ballot(c > 0.0f), neg = __ballot(c < 0.0f);
        const uint32_t p = at + k0 + (uint32_t)(tid & ~63), t = p / (uint32_t)kScanTile, lower = (t + 1) * (uint32_t)kScanTile - p;
        const uint64_t low = lower < 64u ? (1ull << lower) - 1ull : ~0ull;
        if (lane_id() == 0) {
            const uint32_t a = (uint32_t)__popcll(pos & low) | (uint32_t)__popcll(neg & low) << 16;
            const uint32_t b = (uint32_t)__popcll(pos & ~low) | (uint32_t)__popcll(neg & ~low) << 16;
            if (a) atomicAdd(&s_sign[t - tile0], a);
            if (b) atomicAdd(&s_sign[t - tile0 + 1], b);
        }
    }
    __syncthreads();
    if (tid < kTiles && s_sign[tid])
        atomicAdd(&sign_sums[tile0 + tid], (unsigned long long)(s_sign[tid] & 0xffffu) | (unsigned long long)(s_sign[tid] >> 16) << 32);
}

// diag[k] = sum of the values of run k of the sorted keys, in order of appearance (an ordered sum is a chain of adds, so
// what can be saved is the wait for its operands).  A wave takes 64 places; the runs that start there are added up from
// registers, all of them in step, and the one that goes on behind the 64 places is carried on by the whole wave: it
// fetches 64 values at a time, the next ones while these are added, and adds them lane by lane.
__global__ __launch_bounds__(kBlock) void k_diag_runs(size_t m, const uint32_t *key, const uint32_t *val, float *diag)
{
    const size_t base = (size_t)blockIdx.x * kBlock + (threadIdx.x & ~63u), e = base + lane_id();
    if (base >= m) return;      // the whole wave
    const int lane = lane_id();
    const uint32_t k = e < m ? key[e] : 0xffffffffu;      // no key: a node id is below 2^31
    const float v = e < m ? __uint_as_float(val[e]) : 0.0f;
    uint32_t left = (uint32_t)__shfl_up((int)k, 1, 64);
    if (lane == 0) left = base > 0 ? key[base - 1] : 0xffffffffu;
    const bool head = e < m && (k != left || e == 0);
    const uint64_t heads = __ballot(head);
    if (heads == 0ull) return;
    // places of the lane's run within the wave: up to the next head or the end
    const uint64_t later = lane == 63 ? 0ull : heads >> (lane + 1);
    const int in_wave = m - base < 64 ? (int)(m - base) : 64;
    const int len = !head ? 0 : later ? __ffsll((long long)later) : in_wave - lane;
    float acc = v;
    for (int d = 1; __ballot(d < len); ++d) {
        const float x = __shfl_down(v, d, 64);
        if (d < len) acc = acc + x;
    }
    const int last = 63 - __clzll((long long)heads);      // the run that may go on
    if (in_wave == 64 && base + 64 < m) {
        const uint32_t run = (uint32_t)__builtin_amdgcn_readlane((int)k, last);
        float sum = __uint_as_float((uint32_t)__builtin_amdgcn_readlane((int)__float_as_uint(acc), last));
        size_t p = base + 64;
        uint32_t nk = p + lane < m ? key[p + lane] : 0xffffffffu;
        float nv = p + lane < m ? __uint_as_float(val[p + lane]) : 0.0f;
        for (;;) {
            const uint64_t same = __ballot(nk == run);      // the keys ascend: the run's places come first
            const int cnt = same == ~0ull ? 64 : __ffsll((long long)~same) - 1;
            if (cnt == 0) break;
            const uint32_t x = __float_as_uint(nv);
            p += 64;
            if (cnt == 64) {
                nk = p + lane < m ? key[p + lane] : 0xffffffffu;
                nv = p + lane < m ? __uint_as_float(val[p + lane]) : 0.0f;
#pragma unroll
                for (int q = 0; q < 64; ++q) sum = sum + __uint_as_float((uint32_t)__builtin_amdgcn_readlane((int)x, q));
            } else {
                for (int q = 0; q < cnt; ++q) sum = sum + __uint_as_float((uint32_t)__builtin_amdgcn_readlane((int)x, q));
                break;
            }
        }
        if (lane == last) acc = sum;
    }
    if (head) diag[k] = acc;
}


// ---- maximum spanning forest without conflicts (second strategy for S, Sec. 3.1) ----------------
// Boruvka rounds on the candidate edges under the matching's edge order.  comp[] is kept flat
// (comp[v] = current component root of v).  Every component points at its best outgoing edge by
// atomicMax; the chosen edges join the forest; a component hooks onto the component across its
// edge, except that of two components choosing the same edge the smaller id stays a root.
// With a strict edge order the hook graph has no other cycles, and the forest is the unique
// maximum spanning forest whatever the execution order.
__global__ __launch_bounds__(kBlock) void k_bor_propose(size_t na, const uint32_t *act, const int32_t *i,
                                                        const int32_t *j, const float *c, const int32_t *comp,
                                                        unsigned long long *best)
{
    size_t a = (size_t)blockIdx.x * kBlock + threadIdx.x;
    if (a >= na) return;
    uint32_t e = act[a];
    int32_t cu = comp[i[e]], cv = comp[j[e]];
    if (cu == cv) return;
    unsigned long long r = edge_rank(c[e], e);
    atomicMax(&best[cu], r);
    atomicMax(&best[cv], r);
}

__global__ __launch_bounds__(kBlock) void k_bor_select(size_t na, const uint32_t *act, const int32_t *i,
                                                       const int32_t *j, const float *c, const int32_t *comp,
                                                       const unsigned long long *best, int32_t *hook,
                                                       uint8_t *in_forest)
{
    size_t a = (size_t)blockIdx.x * kBlock + threadIdx.x;
    if (a >= na) return;
    uint32_t e = act[a];
    int32_t cu = comp[i[e]], cv = comp[j[e]];
    if (cu == cv) return;
    unsigned long long r = edge_rank(c[e], e);
    const bool bu = best[cu] == r, bv = best[cv] == r;
    if (!(bu || bv)) return;
    in_forest[e] = 1;
    if (bu && !(bv && cu < cv)) hook[cu] = cv;
    if (bv && !(bu && cv < cu)) hook[cv] = cu;
}

// comp[v] <- root of comp[v] in the hook forest (roots have hook[r] == r)
__global__ __launch_bounds__(kBlock) void k_bor_flatten(size_t n, const int32_t *hook, int32_t *comp)
{
    size_t v = (size_t)blockIdx.x * kBlock + threadIdx.x;
    if (v >= n) return;
    int32_t r = comp[v], h = hook[r];
    while (h != r) { r = h; h = hook[r]; }   // every chain ends in a root: the hook graph is a forest
    comp[v] = r;
}

// edges still joining two components move on; best[] and hook[] of their components are reset
__global__ __launch_bounds__(kBlock) void k_bor_advance(size_t na, const uint32_t *act, const int32_t *i,
                                                        const int32_t *j, const int32_t *comp, uint32_t *act_next,
                                                        unsigned long long *best, int32_t *hook, uint32_t *counter)
{
    __shared__ uint32_t s_base;
    const size_t tile = (size_t)blockIdx.x * (kBlock * kAdvItems);
    uint32_t e[kAdvItems];
    uint32_t keep = 0, cnt = 0;
#pragma unroll
    for (int q = 0; q < kAdvItems; ++q) {
        size_t a = tile + (size_t)threadIdx.x * kAdvItems + q;
        e[q] = 0;
        if (a < na) {
            e[q] = act[a];
            int32_t cu = comp[i[e[q]]], cv = comp[j[e[q]]];
            if (cu != cv) {
                keep |= 1u << q;
                ++cnt;
                best[cu] = 0ull; best[cv] = 0ull;
                hook[cu] = cu; hook[cv] = cv;
            }
        }
    }
    uint32_t total;
    uint32_t off = block_inclusive_scan(cnt, &total) - cnt;
    if (threadIdx.x == 0) s_base = total ? atomicAdd(counter, total) : 0u;
    __syncthreads();
    off += s_base;
#pragma unroll
    for (int q = 0; q < kAdvItems; ++q)
        if (keep & (1u << q)) act_next[off++] = e[q];
}

struct ForestFlag {
    static constexpr int bytes = 1;   // bytes read per item
    static constexpr const char *tag = "ForestFlag";
    const uint8_t *in_forest;
    __device__ __forceinline__ uint32_t operator()(size_t e) const { return in_forest[e] ? 1u : 0u; }
};
struct KeptFlag {
    static constexpr int bytes = 2;   // bytes read per item
    static constexpr const char *tag = "KeptFlag";
    const uint8_t *in_forest, *removed;
    __device__ __forceinline__ uint32_t operator()(size_t e) const { return (in_forest[e] && !removed[e]) ? 1u : 0u; }
};

__global__ __launch_bounds__(kBlock) void k_collect_flagged(size_t m, const uint8_t *flag, const uint8_t *veto,
                                                            const uint32_t *pos, const int32_t *i, const int32_t *j,
                                                            uint32_t *ids, int32_t *si, int32_t *sj)
{
    size_t e = (size_t)blockIdx.x * kBlock + threadIdx.x;
    if (e >= m || !flag[e] || (veto && veto[e])) return;
    uint32_t p = pos[e];
    if (ids) ids[p] = (uint32_t)e;
    if (si) { si[p] = i[e]; sj[p] = j[e]; }
}

// rooting of the forest, one breadth-first level per launch: a node at depth `lvl` adopts its
// still unrooted forest neighbours.  up[v] = parent, up_edge[v] = edge to the parent.
__global__ __launch_bounds__(kBlock) void k_root_init(size_t n, const int32_t *comp, int32_t *depth, int32_t *up)
{
    size_t v = (size_t)blockIdx.x * kBlock + threadIdx.x;
    if (v >= n) return;
    bool root = comp[v] == (int32_t)v;
    depth[v] = root ? 0 : -1;
    up[v] = (int32_t)v;
}

__global__ __launch_bounds__(kBlock) void k_root_level(size_t nf, const uint32_t *fe, const int32_t *i, const int32_t *j,
                                                       int32_t lvl, int32_t *depth, int32_t *up, uint32_t *up_edge,
                                                       int32_t *changed)
{
    size_t q = (size_t)blockIdx.x * kBlock + threadIdx.x;
    if (q >= nf) return;
    uint32_t e = fe[q];
    int32_t a = i[e], b = j[e];
    int32_t da = depth[a], db = depth[b];
    if (da == lvl && db < 0) { depth[b] = lvl + 1; up[b] = a; up_edge[b] = e; *changed = 1; }
    else if (db == lvl && da < 0) { depth[a] = lvl + 1; up[a] = b; up_edge[a] = e; *changed = 1; }
}

// every repulsive edge whose endpoints share a tree walks the two ends up to their meeting
// point and marks the lowest-ranked edge of the path
__global__ __launch_bounds__(kBlock) void k_mark_conflicts(size_t m, const int32_t *i, const int32_t *j, const float *c,
                                                           const int32_t *comp, const int32_t *depth, const int32_t *up,
                                                           const uint32_t *up_edge, uint8_t *removed)
{
    size_t e = (size_t)blockIdx.x * kBlock + threadIdx.x;
    if (e >= m || !(c[e] < 0.0f)) return;
    int32_t a = i[e], b = j[e];
    if (comp[a] != comp[b]) return;
    int32_t da = depth[a], db = depth[b];
    unsigned long long low = ~0ull;
    uint32_t low_e = 0;
    while (a != b) {
        uint32_t pe;
        if (da >= db) { pe = up_edge[a]; a = up[a]; --da; } else { pe = up_edge[b]; b = up[b]; --db; }
        unsigned long long r = edge_rank(c[pe], pe);
        if (r < low) { low = r; low_e = pe; }
    }
    if (low != ~0ull) removed[low_e] = 1;
}

// ---- the same for a short candidate list: one workgroup ----------------------------------------------------------
// The rounds that fall back to the forest are late ones: few candidates are left, and the kernels above spend their time
// on launches (four per Boruvka round, one per level of the trees, one per sweep over the components) and on the counts
// the host looks at in between, 1.0 to 1.9 ms a forest.  One workgroup of 1024 threads walks through all of it between
// barriers, each thread with up to eight candidates; only nodes that have a candidate are touched (comp, hook, rep and best
// start out as v, v, v and 0 for all nodes).  A thread's candidates wait for their gathers one after the other, so longer
// lists are better off with the whole chip.  Contraction of 20000 nodes and 60000 edges with a forest, ms, level by level |
// here: 1000 candidates 0.44 | 0.30, 4000 0.51 | 0.39, 8000 0.60 | 0.58, 12000 1.09 | 1.27, 16000 1.40 | 2.21, 32000
// 1.34 | 3.46; a path of 8000 33 | 23, of 24000 118 | 151.  61x97x131 grid, three forests: 10.55 -> 10.16 ms a solve.
constexpr int kForestThreads = 1024, kForestItems = 8;
constexpr uint32_t kShortForest = kForestThreads * kForestItems;
static_assert(kForestItems <= 32, "a bit per candidate of a thread");

__global__ __launch_bounds__(kBlock) void k_forest_init(size_t n, int32_t *comp, int32_t *hook, int32_t *rep, unsigned long long *best)
{
    const size_t v = (size_t)blockIdx.x * kBlock + threadIdx.x;
    if (v >= n) return;
    comp[v] = (int32_t)v; hook[v] = (int32_t)v; rep[v] = (int32_t)v;
    best[v] = 0ull;
}

// forest and rooting; state[k] = 1 iff candidate k is in the forest, up_cand[v] = candidate that joins v to its parent
__global__ __launch_bounds__(kForestThreads) void k_forest_short(uint32_t na, Cands a, int32_t *comp, int32_t *hook, unsigned long long *best,
                                                                 int32_t *depth, int32_t *up, uint32_t *up_cand, uint8_t *state)
{
    const uint32_t tid = threadIdx.x;
    uint32_t own = 0, tree = 0;      // this thread's candidates tid, tid + 1024, ..; those in the forest
    for (uint32_t q = 0; q < (uint32_t)kForestItems && tid + q * kForestThreads < na; ++q) own |= 1u << q;
    uint32_t alive = own;
    for (int round = 0; round < 64; ++round) {      // the number of components with an outgoing candidate at least halves
        for (uint32_t left = alive; left; left &= left - 1) {
            const uint32_t k = tid + (uint32_t)(__ffs((int)left) - 1) * kForestThreads;
            const unsigned long long r = a.r[k];
            atomicMax(&best[comp[a.u[k]]], r);
            atomicMax(&best[comp[a.v[k]]], r);
        }
        if (!__syncthreads_or(alive != 0u)) break;
        for (uint32_t left = alive; left; left &= left - 1) {
            const int q = __ffs((int)left) - 1;
            const uint32_t k = tid + (uint32_t)q * kForestThreads;
            const int32_t cu = comp[a.u[k]], cv = comp[a.v[k]];
            const unsigned long long r = a.r[k];
            const bool bu = load_past_cache(&best[cu]) == r, bv = load_past_cache(&best[cv]) == r;
            if (!(bu || bv)) continue;
            tree |= 1u << q;
            if (bu && !(bv && cu < cv)) hook[cu] = cv;
            if (bv && !(bu && cv < cu)) hook[cv] = cu;
        }
        __syncthreads();
        // the hook graph is a forest and a root hooks onto itself: every chain ends
        uint32_t next = alive;
        for (uint32_t left = alive; left; left &= left - 1) {
            const int q = __ffs((int)left) - 1;
            const uint32_t k = tid + (uint32_t)q * kForestThreads;
            const int32_t u = a.u[k], v = a.v[k];
            int32_t ru = comp[u], rv = comp[v];
            for (int32_t h = hook[ru]; h != ru; h = hook[ru]) ru = h;
            for (int32_t h = hook[rv]; h != rv; h = hook[rv]) rv = h;
            comp[u] = ru; comp[v] = rv;      // several threads may write, all of them the same root
            if (ru == rv) next &= ~(1u << q);
            best[ru] = 0ull; best[rv] = 0ull;
        }
        alive = next;
        __syncthreads();
    }
    for (uint32_t left = own; left; left &= left - 1) {
        const uint32_t k = tid + (uint32_t)(__ffs((int)left) - 1) * kForestThreads;
        const int32_t e[2] = {a.u[k], a.v[k]};
#pragma unroll
        for (int s = 0; s < 2; ++s) {
            int32_t r = comp[e[s]];
            for (int32_t h = hook[r]; h != r; h = hook[r]) r = h;
            comp[e[s]] = r;
            depth[e[s]] = r == e[s] ? 0 : -1;
            up[e[s]] = e[s];
        }
        state[k] = (uint8_t)((tree >> ((k - tid) / kForestThreads)) & 1u);
    }
    __syncthreads();
    for (int32_t lvl = 0; lvl <= (int32_t)na; ++lvl) {      // a tree of na edges is at most na levels deep
        bool changed = false;
        for (uint32_t left = tree; left; left &= left - 1) {
            const int q = __ffs((int)left) - 1;
            const uint32_t k = tid + (uint32_t)q * kForestThreads;
            const int32_t u = a.u[k], v = a.v[k], du = depth[u], dv = depth[v];
            // a tree: nobody else reaches the child on this level
            if (du == lvl && dv < 0) { depth[v] = lvl + 1; up[v] = u; up_cand[v] = k; changed = true; }
            else if (dv == lvl && du < 0) { depth[u] = lvl + 1; up[u] = v; up_cand[u] = k; changed = true; }
            if (du >= 0 && dv >= 0) tree &= ~(1u << q);      // both ends rooted: done with this edge
        }
        if (!__syncthreads_or(changed)) break;
    }
}

// as k_mark_conflicts, on candidate numbers: state 2 = removed
__global__ __launch_bounds__(kBlock) void k_mark_conflicts_short(size_t m, const int32_t *i, const int32_t *j, const float *c, const int32_t *comp,
                                                                 const int32_t *depth, const int32_t *up, const uint32_t *up_cand,
                                                                 const unsigned long long *rank, uint8_t *state)
{
    const size_t e = (size_t)blockIdx.x * kBlock + threadIdx.x;
    if (e >= m || !(c[e] < 0.0f)) return;
    int32_t a = i[e], b = j[e];
    if (comp[a] != comp[b]) return;      // nodes without a candidate are alone in their component
    int32_t da = depth[a], db = depth[b];
    unsigned long long low = ~0ull;
    uint32_t low_k = 0;
    while (a != b) {
        uint32_t k;
        if (da >= db) { k = up_cand[a]; a = up[a]; --da; } else { k = up_cand[b]; b = up[b]; --db; }
        const unsigned long long r = rank[k];
        if (r < low) { low = r; low_k = k; }
    }
    if (low != ~0ull) state[low_k] = 2;
}

// components of the forest edges that were not removed; their number goes to the host
__global__ __launch_bounds__(kForestThreads) void k_forest_components(uint32_t na, Cands a, const uint8_t *state, int32_t *rep, MailWord *mail, uint64_t seq)
{
    __shared__ uint32_t s_kept;
    const uint32_t tid = threadIdx.x;
    if (tid == 0) s_kept = 0u;
    uint32_t kept = 0;
    for (uint32_t q = 0; q < (uint32_t)kForestItems; ++q) {
        const uint32_t k = tid + q * kForestThreads;
        if (k < na && state[k] == 1) kept |= 1u << q;
    }
    __syncthreads();
    const uint32_t n_wave = wave_sum((uint32_t)__popc(kept));
    if (lane_id() == 0 && n_wave) atomicAdd(&s_kept, n_wave);
    // Until nothing changes: pointers only ever decrease, and two sweeps leave at most half of the roots that are not done.  (A
    // root that has a smaller neighbour hooks.  One that has none keeps a neighbour's whole tree or meets a smaller root
    // through it in the next sweep.)
    for (;;) {
        bool changed = false;
        for (uint32_t left = kept; left; left &= left - 1) {
            const uint32_t k = tid + (uint32_t)(__ffs((int)left) - 1) * kForestThreads;
            int32_t p = a.u[k], q = a.v[k];      // parents only ever decrease: the walks end
            for (int32_t x = load_past_cache(&rep[p]); x != p; x = load_past_cache(&rep[p])) p = x;
            for (int32_t x = load_past_cache(&rep[q]); x != q; x = load_past_cache(&rep[q])) q = x;
            if (p != q) { atomicMin(&rep[max(p, q)], min(p, q)); changed = true; }
        }
        if (!__syncthreads_or(changed)) break;
    }
    for (uint32_t left = kept; left; left &= left - 1) {
        const uint32_t k = tid + (uint32_t)(__ffs((int)left) - 1) * kForestThreads;
        const int32_t u = a.u[k], v = a.v[k];
        int32_t p = u;      // both ends have the same root; a shorter way to it: no walk of another thread goes wrong
        for (int32_t x = load_past_cache(&rep[p]); x != p; x = load_past_cache(&rep[p])) p = x;
        rep[u] = p; rep[v] = p;
    }
    if (tid == 0) mail_put(mail + 1, (uint64_t)s_kept);
    mail_send(mail, seq);
}

}  // namespace

// The candidate edges of a graph: the scan that packs them and the arrays they were packed into (which the handshake
// rounds have used since).
struct Candidates {
    uint32_t n = 0;
    bool summed = false;      // the plan holds tile sums, not their scan
    ScanPlan<uint32_t> plan;
    Buf<int32_t> u, v;
    Buf<unsigned long long> r;
};

// handshake matching; mate[v] = partner or -1; returns |S| in n_matched.  fmap (optional): memory for the numbers of the new
// nodes; *numbered says whether they are there.
// On graphs of up to kBlindEdges edges nobody waits to hear how many candidates there are: arrays and grids are made for as
// many as there are edges, and the first look at the counts is the one behind the handshake rounds.
constexpr size_t kBlindEdges = size_t(1) << 20;
static_assert(kBlindEdges <= kMatchBatchMax && kBlindEdges <= kAdvMedium, "short lists");
static rama_status matching(Ctx &ctx, const Graph &g, float tau, int rounds_cap, Buf<int32_t> &mate, int64_t &n_matched, Candidates &list,
                            int32_t *fmap, bool *numbered)
{
    const size_t m = (size_t)g.m, n = (size_t)g.n;
    n_matched = 0;
    *numbered = false;
    RAMA_TRY(mate.alloc(ctx, n > 0 ? n : 1));
    MultiFill setup;   // mate = -1, rank words and counters = 0: one launch
    setup.add(mate.get(), 0xffffffffu, n);
    if (m == 0) return setup.run(ctx);
    Buf<int32_t> cu[2], cv[2];
    Buf<unsigned long long> cr[2];
    Cands cur{}, nxt{};
    ScanPlan<uint32_t> &cand = list.plan;   // its total -- the length of the first list -- stays on the device for the first round
    const CandFlag flag{g.c.get(), tau};
    const int cap = rounds_cap > 0 ? rounds_cap : 0;
    bool blind = m <= kBlindEdges && cap > 0 && !ctx.active->is_arena();
    list.summed = blind;
    RAMA_TRY((scan_plan_alloc<uint32_t>(ctx, m, 0, cand)));
    uint32_t na = (uint32_t)m;
    if (!blind) {
        RAMA_TRY((scan_totals<uint32_t>(ctx, flag, cand)));
        na = list.n = cand.total;
        if (na == 0) return setup.run(ctx);
    }
    const uint32_t group = na <= kAdvMedium ? kBlock * 2 : kBlock * kAdvItems, groups = grid_for(na, (int)group);
    const ListPlaces places{groups / kLists * group, groups % kLists, group};
    if ((uint64_t)groups * group > 0xFFFFFFFFull) return fail(ctx, RAMA_ERR_CAPACITY, "matching: more than 2^32 places");
    for (int k = 0; k < 2; ++k) {
        RAMA_TRY(cu[k].alloc(ctx, (size_t)groups * group));
        RAMA_TRY(cv[k].alloc(ctx, (size_t)groups * group));
        RAMA_TRY(cr[k].alloc(ctx, (size_t)groups * group));
    }
    cur = Cands{cu[0].get(), cv[0].get(), cr[0].get()};
    nxt = Cands{cu[1].get(), cv[1].get(), cr[1].get()};
    Buf<unsigned long long> best, best_next, best_after;   // rank words of this round, the next, the one after
    RAMA_TRY(best.alloc(ctx, n));
    RAMA_TRY(best_next.alloc(ctx, n));
    RAMA_TRY(best_after.alloc(ctx, n));
    // the counters of kRoundsAhead rounds; where there are more, the next ones get others (and the last one's are read once more)
    constexpr int kRoundsAhead = 8;
    constexpr size_t kRoundWords = (size_t)kLists * kListWords;
    const size_t counter_words = (size_t)(cap < kRoundsAhead ? cap : kRoundsAhead) * kRoundWords;
    Buf<unsigned long long> counters, counters_before;
    RAMA_TRY(counters.alloc(ctx, counter_words));
    setup.add(best.get(), 0u, n);
    setup.add(best_next.get(), 0u, n);
    setup.add(counters.get(), 0u, counter_words);
    // The list is packed and makes the first round's proposals on the way: it is not read once more just for that.
    const PackCandsEmit pack{g.i.get(), g.j.get(), g.c.get(), cur, cap > 0 ? best.get() : nullptr};
    const double pack_bytes = (double)((size_t)na * (cap > 0 ? 44 : 28));
    if (blind) {
        RAMA_TRY(setup.run_with_sums(ctx, flag, cand.offs.get(), m));
        RAMA_TRY((scan_emit_sums<uint32_t>(ctx, flag, pack, cand, pack_bytes)));
    } else {
        RAMA_TRY(setup.run(ctx));
        RAMA_TRY((scan_emit<uint32_t>(ctx, flag, pack, cand, pack_bytes)));
    }
    // Long lists: one round per look at the counts, so that every launch has its exact size.  Short lists (the launches
    // are empty anyway): as many rounds as should bring the list to what one workgroup finishes (a round keeps about two
    // candidates in five, and about half of the edges are candidates) are enqueued on the size of its first list, then the
    // kernel that finishes it, and the counts come back together; rounds behind one that emptied the list find a zero count
    // and do nothing.
    const uint32_t last_max = finish_max(g.n);
    uint32_t longest = places.begin(1);      // of the lists: a bound
    int first_round = 0, rounds_before = 0;      // of the counters; how many there were before them
    for (int r = 0; r < cap && na > 0;) {
        const bool finish = na <= kMatchBatchMax;
        int batch = finish ? 0 : 1;
        if (finish)
            for (uint32_t left = blind ? na / 2 + 1 : na; (left > last_max || (blind && batch == 0 && na > last_max)) && batch < cap - r; left = left / 5 * 2) ++batch;
        if (batch > kRoundsAhead) batch = kRoundsAhead;
        if (r + batch - first_round > kRoundsAhead) {
            counters_before = std::move(counters);
            RAMA_TRY(counters.alloc(ctx, counter_words));
            RAMA_TRY(fill<unsigned long long>(ctx, counters.get(), 0ull, counter_words));
            rounds_before = r - first_round;
            first_round = r;
        }
        auto counts = [&](int round) {
            return round >= first_round ? counters.get() + (size_t)(round - first_round) * kRoundWords
                                        : counters_before.get() + (size_t)(rounds_before - 1) * kRoundWords;
        };
        auto list_of = [&](int round) {
            return round == 0 ? CandList{cur, cand.offs.get() + cand.nb, nullptr, places} : CandList{cur, nullptr, counts(round - 1), places};
        };
        auto groups_of = [&](int round, uint32_t size) { return round == 0 ? grid_for(na, (int)size) : kLists * grid_for(longest, (int)size); };
        for (int b = 0; b < batch; ++b, ++r) {
            const bool accepts = na <= kAdvMedium;
            if (!accepts) {
                ProfScope ps_(ctx, "k_accept", (double)((size_t)na * 40));
                k_accept<<<groups_of(r, kBlock), kBlock, 0, ctx.stream>>>(list_of(r), best.get(), mate.get());
            }
            LAUNCH_TRY(ctx, "accept");
            {
                ProfScope ps_(ctx, "k_advance", (double)((size_t)na * (accepts ? 80 : 56)));
                if (accepts)
                    k_advance<2, true><<<groups_of(r, kBlock * 2), kBlock, 0, ctx.stream>>>(
                        list_of(r), mate.get(), nxt, best.get(), g.i.get(), g.j.get(), best_next.get(), best_after.get(), counts(r));
                else
                    k_advance<kAdvItems, false><<<groups_of(r, kBlock * kAdvItems), kBlock, 0, ctx.stream>>>(
                        list_of(r), mate.get(), nxt, best.get(), g.i.get(), g.j.get(), best_next.get(), best_after.get(), counts(r));
            }
            LAUNCH_TRY(ctx, "advance");
            Cands t = cur; cur = nxt; nxt = t;
            best.swap(best_next);          // (this, next, after) <- (next, after, this)
            best_next.swap(best_after);
        }
        const uint64_t seq = ++ctx.mail_seq;
        const volatile uint64_t *mail = mail_words(ctx);
        if (!finish) {
            {
                ProfScope ps_(ctx, "k_look_at_lists", (double)(kLists * 8));
                k_look_at_lists<<<1, 64, 0, ctx.stream>>>(counts(r - 1), mailbox(ctx), seq);
            }
            LAUNCH_TRY(ctx, "look_at_lists");
            RAMA_TRY(wait_mail(ctx, seq));
            const uint64_t lengths = mail[1];
            na = (uint32_t)lengths;
            longest = (uint32_t)(lengths >> 32);
            n_matched += (int64_t)mail[2];
            continue;
        }
        {
            ProfScope ps_(ctx, "k_handshake_finish", (double)(kFinishMax * 40));
            k_handshake_finish<<<1, kFinishThreads, 0, ctx.stream>>>(cand.offs.get() + cand.nb, list_of(r), mate.get(), cap - r, g.n, fmap,
                                                                    batch ? counts(r - batch) : nullptr, batch, mailbox(ctx), seq);
        }
        LAUNCH_TRY(ctx, "handshake_finish");
        RAMA_TRY(wait_mail(ctx, seq));
        const uint64_t lengths = mail[1];
        const uint32_t left = (uint32_t)(lengths >> 32);
        list.n = (uint32_t)lengths;
        n_matched += (int64_t)mail[2];
        blind = false;
        na = left;
        if (left <= last_max) {      // the rest was worked off, or the cap was reached
            *numbered = fmap != nullptr;
            break;
        }
    }
    list.u = std::move(cu[0]); list.v = std::move(cv[0]); list.r = std::move(cr[0]);
    return RAMA_OK;
}

// S by the spanning forest without conflicts, for a short candidate list: |S| and the components of (V,S)
static rama_status forest_short(Ctx &ctx, const Graph &g, float tau, Candidates &list, Buf<int32_t> &rep, int64_t &n_set)
{
    const size_t m = (size_t)g.m, n = (size_t)g.n;
    const Cands a{list.u.get(), list.v.get(), list.r.get()};
    const PackCandsEmit pack{g.i.get(), g.j.get(), g.c.get(), a, nullptr};
    const CandFlag flag{g.c.get(), tau};
    if (list.summed) RAMA_TRY((scan_emit_sums<uint32_t>(ctx, flag, pack, list.plan, (double)((size_t)list.n * 28))));
    else RAMA_TRY((scan_emit<uint32_t>(ctx, flag, pack, list.plan, (double)((size_t)list.n * 28))));
    Buf<int32_t> comp, hook, depth, up;
    Buf<uint32_t> up_cand;
    Buf<unsigned long long> best;
    Buf<uint8_t> state;
    RAMA_TRY(comp.alloc(ctx, n));
    RAMA_TRY(hook.alloc(ctx, n));
    RAMA_TRY(depth.alloc(ctx, n));
    RAMA_TRY(up.alloc(ctx, n));
    RAMA_TRY(up_cand.alloc(ctx, n));
    RAMA_TRY(rep.alloc(ctx, n));
    RAMA_TRY(best.alloc(ctx, n));
    RAMA_TRY(state.alloc(ctx, list.n));
    {
        ProfScope ps_(ctx, "k_forest_init", (double)(n * 20));
        k_forest_init<<<grid_for(n), kBlock, 0, ctx.stream>>>(n, comp.get(), hook.get(), rep.get(), best.get());
    }
    LAUNCH_TRY(ctx, "forest_init");
    {
        ProfScope ps_(ctx, "k_forest_short", (double)((size_t)list.n * 64));
        k_forest_short<<<1, kForestThreads, 0, ctx.stream>>>(list.n, a, comp.get(), hook.get(), best.get(), depth.get(), up.get(), up_cand.get(),
                                                             state.get());
    }
    LAUNCH_TRY(ctx, "forest_short");
    {
        ProfScope ps_(ctx, "k_mark_conflicts", (double)(m * 12));
        k_mark_conflicts_short<<<grid_for(m), kBlock, 0, ctx.stream>>>(m, g.i.get(), g.j.get(), g.c.get(), comp.get(), depth.get(), up.get(),
                                                                      up_cand.get(), a.r, state.get());
    }
    LAUNCH_TRY(ctx, "mark_conflicts");
    const uint64_t seq = ++ctx.mail_seq;
    {
        ProfScope ps_(ctx, "k_forest_components", (double)((size_t)list.n * 24));
        k_forest_components<<<1, kForestThreads, 0, ctx.stream>>>(list.n, a, state.get(), rep.get(), mailbox(ctx), seq);
    }
    LAUNCH_TRY(ctx, "forest_components");
    RAMA_TRY(wait_mail(ctx, seq));
    n_set = (int64_t)mail_words(ctx)[1];
    return RAMA_OK;
}

// S by the spanning forest without conflicts; writes the S edges to si/sj (allocated here)
static rama_status forest_set(Ctx &ctx, const Graph &g, float tau, Buf<int32_t> &si, Buf<int32_t> &sj, int64_t &n_set)
{
    const size_t m = (size_t)g.m, n = (size_t)g.n;
    n_set = 0;
    Buf<uint32_t> pos, act, act2, counters;
    RAMA_TRY(pos.alloc(ctx, m + 1));
    uint32_t na = 0;
    {
        ScanPlan<uint32_t> cand;
        RAMA_TRY((scan_plan_alloc<uint32_t>(ctx, m, 0, cand)));
        RAMA_TRY((scan_totals<uint32_t>(ctx, CandFlag{g.c.get(), tau}, cand)));
        na = cand.total;
        if (na == 0) return RAMA_OK;
        RAMA_TRY(act.alloc(ctx, na));
        RAMA_TRY(act2.alloc(ctx, na));
        RAMA_TRY((scan_emit<uint32_t>(ctx, CandFlag{g.c.get(), tau}, CollectEmit{act.get()}, cand, (double)((size_t)na * 4))));
    }
    Buf<unsigned long long> best;
    Buf<int32_t> comp, hook;
    Buf<uint8_t> in_forest, removed;
    RAMA_TRY(best.alloc(ctx, n));
    RAMA_TRY(comp.alloc(ctx, n));
    RAMA_TRY(hook.alloc(ctx, n));
    RAMA_TRY(in_forest.alloc(ctx, m));
    RAMA_TRY(removed.alloc(ctx, m));
    RAMA_TRY(fill<unsigned long long>(ctx, best.get(), 0ull, n));
    RAMA_TRY(fill<uint8_t>(ctx, in_forest.get(), (uint8_t)0, m));
    RAMA_TRY(fill<uint8_t>(ctx, removed.get(), (uint8_t)0, m));
    {
        ProfScope ps_(ctx, "k_iota", (double)(n * 8));
        k_iota<<<grid_for(n), kBlock, 0, ctx.stream>>>(n, comp.get());
        k_iota<<<grid_for(n), kBlock, 0, ctx.stream>>>(n, hook.get());
    }
    LAUNCH_TRY(ctx, "iota");
    const int max_rounds = 64;   // the number of components with an outgoing edge at least halves per round
    RAMA_TRY(zeroed<uint32_t>(ctx, max_rounds, counters));
    int round = 0;
    for (; round < max_rounds && na > 0; ++round) {
        {
            ProfScope ps_(ctx, "k_bor_propose", (double)((size_t)na * 40));
            k_bor_propose<<<grid_for(na), kBlock, 0, ctx.stream>>>(na, act.get(), g.i.get(), g.j.get(), g.c.get(), comp.get(),
                                                                  best.get());
        }
        LAUNCH_TRY(ctx, "bor_propose");
        {
            ProfScope ps_(ctx, "k_bor_select", (double)((size_t)na * 48));
            k_bor_select<<<grid_for(na), kBlock, 0, ctx.stream>>>(na, act.get(), g.i.get(), g.j.get(), g.c.get(), comp.get(),
                                                                 best.get(), hook.get(), in_forest.get());
        }
        LAUNCH_TRY(ctx, "bor_select");
        {
            ProfScope ps_(ctx, "k_bor_flatten", (double)(n * 12));
            k_bor_flatten<<<grid_for(n), kBlock, 0, ctx.stream>>>(n, hook.get(), comp.get());
        }
        LAUNCH_TRY(ctx, "bor_flatten");
        {
            ProfScope ps_(ctx, "k_bor_advance", (double)((size_t)na * 28));
            k_bor_advance<<<grid_for(na, kBlock * kAdvItems), kBlock, 0, ctx.stream>>>(
                na, act.get(), g.i.get(), g.j.get(), comp.get(), act2.get(), best.get(), hook.get(), counters.get() + round);
        }
        LAUNCH_TRY(ctx, "bor_advance");
        uint32_t nn = 0;
        RAMA_TRY(read_back(ctx, &nn, counters.get() + round, 4));
        act.swap(act2);
        na = nn;
    }
    if (na > 0) return fail(ctx, RAMA_ERR_HIP, "spanning forest did not converge");
    act.reset(); act2.reset(); best.reset();
    // forest edge list
    RAMA_TRY((exclusive_scan<uint32_t>(ctx, ForestFlag{in_forest.get()}, pos.get(), m)));
    uint32_t nf = 0;
    RAMA_TRY(read_back(ctx, &nf, pos.get() + m, 4));
    if (nf == 0) return RAMA_OK;
    Buf<uint32_t> fe, up_edge;
    Buf<int32_t> depth, up, changed;
    RAMA_TRY(fe.alloc(ctx, nf));
    {
        ProfScope ps_(ctx, "k_collect_flagged", (double)(m * 5 + (size_t)nf * 4));
        k_collect_flagged<<<grid_for(m), kBlock, 0, ctx.stream>>>(m, in_forest.get(), (const uint8_t *)nullptr, pos.get(),
                                                                 g.i.get(), g.j.get(), fe.get(), (int32_t *)nullptr,
                                                                 (int32_t *)nullptr);
    }
    LAUNCH_TRY(ctx, "collect_flagged");
    // root the trees at their component representative, level by level
    RAMA_TRY(depth.alloc(ctx, n));
    RAMA_TRY(up.alloc(ctx, n));
    RAMA_TRY(up_edge.alloc(ctx, n));
    {
        ProfScope ps_(ctx, "k_root_init", (double)(n * 12));
        k_root_init<<<grid_for(n), kBlock, 0, ctx.stream>>>(n, comp.get(), depth.get(), up.get());
    }
    LAUNCH_TRY(ctx, "root_init");
    const int levels_per_check = 8;
    for (int32_t lvl = 0;; lvl += levels_per_check) {
        // a tree is at most n-1 levels deep; the sweep after the deepest level reports no change
        if ((size_t)lvl > n + levels_per_check) return fail(ctx, RAMA_ERR_HIP, "forest rooting did not converge");
        RAMA_TRY(zeroed<int32_t>(ctx, 1, changed));   // a fresh word per look
        for (int q = 0; q < levels_per_check; ++q) {
            ProfScope ps_(ctx, "k_root_level", (double)((size_t)nf * 20));
            k_root_level<<<grid_for(nf), kBlock, 0, ctx.stream>>>(nf, fe.get(), g.i.get(), g.j.get(), lvl + q, depth.get(),
                                                                 up.get(), up_edge.get(), changed.get());
        }
        LAUNCH_TRY(ctx, "root_level");
        int32_t h = 0;
        RAMA_TRY(read_back(ctx, &h, changed.get(), 4));
        if (!h) break;
    }
    {
        ProfScope ps_(ctx, "k_mark_conflicts", (double)(m * 12));
        k_mark_conflicts<<<grid_for(m), kBlock, 0, ctx.stream>>>(m, g.i.get(), g.j.get(), g.c.get(), comp.get(), depth.get(),
                                                                up.get(), up_edge.get(), removed.get());
    }
    LAUNCH_TRY(ctx, "mark_conflicts");
    RAMA_TRY((exclusive_scan<uint32_t>(ctx, KeptFlag{in_forest.get(), removed.get()}, pos.get(), m)));
    uint32_t ns = 0;
    RAMA_TRY(read_back(ctx, &ns, pos.get() + m, 4));
    n_set = ns;
    if (ns == 0) return RAMA_OK;
    RAMA_TRY(si.alloc(ctx, ns));
    RAMA_TRY(sj.alloc(ctx, ns));
    {
        ProfScope ps_(ctx, "k_collect_flagged", (double)(m * 6 + (size_t)ns * 8));
        k_collect_flagged<<<grid_for(m), kBlock, 0, ctx.stream>>>(m, in_forest.get(), removed.get(), pos.get(), g.i.get(),
                                                                 g.j.get(), (uint32_t *)nullptr, si.get(), sj.get());
    }
    LAUNCH_TRY(ctx, "collect_flagged");
    return RAMA_OK;
}

// rep[v] = smallest node of v's component in (V,S)
static rama_status components(Ctx &ctx, size_t n, size_t ns, const int32_t *si, const int32_t *sj, Buf<int32_t> &rep)
{
    RAMA_TRY(rep.alloc(ctx, n > 0 ? n : 1));
    {
        ProfScope ps_(ctx, "k_iota", (double)(n * 4));
        k_iota<<<grid_for(n), kBlock, 0, ctx.stream>>>(n, rep.get());
    }
    LAUNCH_TRY(ctx, "iota");
    if (ns == 0) return RAMA_OK;
    Buf<int32_t> changed;
    for (int it = 0; it < 64; ++it) {   // two sweeps leave at most half of the roots that are not done (see k_forest_components)
        RAMA_TRY(zeroed<int32_t>(ctx, 1, changed));   // a fresh word per sweep
        {
            ProfScope ps_(ctx, "k_hook", (double)(ns * 24));
            k_hook<<<grid_for(ns), kBlock, 0, ctx.stream>>>(ns, si, sj, rep.get(), changed.get());
        }
        LAUNCH_TRY(ctx, "hook");
        {
            ProfScope ps_(ctx, "k_flatten", (double)(n * 12));
            k_flatten<<<grid_for(n), kBlock, 0, ctx.stream>>>(n, rep.get());
        }
        LAUNCH_TRY(ctx, "flatten");
        int32_t h = 0;
        RAMA_TRY(read_back(ctx, &h, changed.get(), 4));
        if (!h) return RAMA_OK;
    }
    return fail(ctx, RAMA_ERR_HIP, "connected components did not converge");
}

// contract_edges for a middle-sized list: five launches and a wait, where counting the digits, counting the heads and the sums
// as launches of their own were seven.  Contraction of a 300x301 long-range grid to the end 1.72 -> 1.54 ms, 128^2 static solve
// 2.07 -> 1.99, 512^2 5.46 -> 5.37, 6-NN graph of 10^6 points 9.35 -> 9.24, 61x97x131 volume 5.45 -> 5.29.  *done stays false if some digit holds more edges than a workgroup sorts.
static rama_status contract_by_digits(Ctx &ctx, const Graph &g, const int32_t *fmap, int nbits, int top_bits, Graph &out, float *diag, bool *done)
{
    const size_t m = (size_t)g.m;
    const int low_bits = 2 * nbits - top_bits;
    const bool short_tiles = m <= kSortShort;
    const uint32_t nb = grid_for(m, short_tiles ? kShortTile : kMediumTile), tiles = grid_for(m, kScanTile), digits = 1u << top_bits;
    static_assert(kScanTile == kMediumTile && kScanTile == 2 * kShortTile, "tiles of the sort per tile of k_relabel_keys");
    Buf<uint64_t> raw, key;
    Buf<uint32_t> val, val2, hist, starts, counts, words;      // words: largest hi - lo, a digit is too long
    RAMA_TRY(raw.alloc(ctx, m));
    RAMA_TRY(key.alloc(ctx, m));
    RAMA_TRY(val.alloc(ctx, m));
    RAMA_TRY(val2.alloc(ctx, m));
    RAMA_TRY(hist.alloc(ctx, ((size_t)nb + 1) << top_bits));
    RAMA_TRY(starts.alloc(ctx, (size_t)digits + 1));
    RAMA_TRY(counts.alloc(ctx, (size_t)digits));
    RAMA_TRY(zeroed<uint32_t>(ctx, 2, words));
    RAMA_TRY(out.sign_sums.alloc(ctx, tiles));
    {
        ProfScope ps_(ctx, "k_rs_hist<relabelled>", (double)(m * 24));      // makes the keys and counts for the sort's one pass
        auto relabel = [&](auto kernel) {
            kernel<<<tiles, kBlock, 0, ctx.stream>>>(m, g.i.get(), g.j.get(), fmap, raw.get(), words.get(), (uint32_t *)nullptr, out.sign_sums.get(),
                                                     hist.get(), nb, nbits - top_bits, top_bits, g.c.get(), diag);
        };
        if (short_tiles) relabel(k_relabel_keys<2>);
        else relabel(k_relabel_keys<1>);
    }
    LAUNCH_TRY(ctx, "relabel_keys");
    const RelabelledEdges source{raw.get(), g.c.get(), nbits};
    if (short_tiles)
        RAMA_TRY((radix_pass<uint64_t, uint32_t, true, kShortThreads, kShortTile / kShortThreads>(ctx, (const uint64_t *)nullptr, (const uint32_t *)nullptr, source, key.get(), val.get(),
                                                                                                 m, low_bits, top_bits, hist.get(), starts.get(), true)));
    else
        RAMA_TRY((radix_pass<uint64_t, uint32_t, true, kMediumThreads, kMediumTile / kMediumThreads>(ctx, (const uint64_t *)nullptr, (const uint32_t *)nullptr, source, key.get(), val.get(),
                                                                                                    m, low_bits, top_bits, hist.get(), starts.get(), true)));
    // the relabelled edges are no longer needed: the digits' edges take their place.  The timers book k_sum_digit, its sort
    // included, with the other kernel that adds up runs.
    int32_t *ti = reinterpret_cast<int32_t *>(raw.get()), *tj = ti + m;
    float *tc = reinterpret_cast<float *>(val2.get());
    {
        ProfScope ps_(ctx, "k_reduce_runs", (double)(m * 24));
        k_sum_digit<<<digits, LocalSort<uint32_t>::threads, 0, ctx.stream>>>(key.get(), val.get(), starts.get(), nbits, low_bits, words.get(), counts.get(),
                                                                          words.get() + 1, ti, tj, tc);
    }
    LAUNCH_TRY(ctx, "sum_digit");
    key.reset(); val.reset();      // the result may take their place
    RAMA_TRY(out.i.alloc(ctx, m));
    RAMA_TRY(out.j.alloc(ctx, m));
    RAMA_TRY(out.c.alloc(ctx, m));
    const uint64_t seq = ++ctx.mail_seq;
    {
        ProfScope ps_(ctx, "k_join_digits", (double)(m * 24));
        k_join_digits<<<digits, kJoinThreads, 0, ctx.stream>>>(starts.get(), counts.get(), ti, tj, tc, out.i.get(), out.j.get(), out.c.get(),
                                                            (unsigned long long *)out.sign_sums.get(), words.get() + 1, mailbox(ctx), seq);
    }
    LAUNCH_TRY(ctx, "join_digits");
    RAMA_TRY(wait_mail(ctx, seq));
    const volatile uint64_t *mail = mail_words(ctx);
    if (mail[2]) {
        ctx.sorts_unseen = false;
        out.i.reset(); out.j.reset(); out.c.reset(); out.sign_sums.reset();
        return RAMA_OK;
    }
    out.m = (int64_t)mail[1];
    out.i.shorten((size_t)out.m); out.j.shorten((size_t)out.m); out.c.shorten((size_t)out.m);
    *done = true;
    return RAMA_OK;
}

// contracted graph of canonical g under fmap (n_new new nodes)
static rama_status contract_edges(Ctx &ctx, const Graph &g, const int32_t *fmap, int32_t n_new, Graph &out, float *diag)
{
    const size_t m = (size_t)g.m;
    out.n = n_new;
    out.m = 0;
    const int nbits = bits_for((uint64_t)n_new);
    // A middle-sized list: one pass over the top bits of lo, whose digits are counted by the kernel that makes the keys, and a
    // workgroup to a digit does the rest.  Nobody waits to hear how many edges are left.
    bool narrow = false;
    const int top_bits = sort_takes_source(m, m) ? unseen_bits_now(ctx, m, 2 * nbits, (uint64_t)n_new << nbits, &narrow) : 0;
    if (top_bits > 0 && narrow && top_bits <= nbits) {
        bool done = false;
        RAMA_TRY(contract_by_digits(ctx, g, fmap, nbits, top_bits, out, diag, &done));
        if (done) return RAMA_OK;
    }
    ScanPlan<uint32_t> keep;   // the extra word behind the total: largest hi-lo
    Buf<uint64_t> raw;
    RAMA_TRY((scan_plan_alloc<uint32_t>(ctx, m, 1, keep)));
    RAMA_TRY(raw.alloc(ctx, m));
    RAMA_TRY(out.sign_sums.alloc(ctx, keep.nb > 0 ? keep.nb : 1));
    {
        ProfScope ps_(ctx, "k_relabel_keys", (double)(m * 24));
        k_relabel_keys<0><<<keep.nb, kBlock, 0, ctx.stream>>>(m, g.i.get(), g.j.get(), fmap, raw.get(), keep.extra_ptr(),
                                                           keep.sums.get(), out.sign_sums.get(), (uint32_t *)nullptr, 0u, 0, 0, g.c.get(), diag);
    }
    LAUNCH_TRY(ctx, "relabel_keys");
    RAMA_TRY((scan_totals<uint32_t>(ctx, NotLoopKey{raw.get()}, keep, keep.sums.get())));   // tile sums: left by k_relabel_keys
    const uint32_t kept = keep.total;
    const int dbits = bits_for((uint64_t)keep.extra_value[0] + 1);
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
    if (sort_takes_source(kept, m)) {
        // the sort's first pass reads the stored keys itself and leaves the loops out; they are no longer needed after it,
        // so their place serves as the second key array
        Buf<uint32_t> val2;
        RAMA_TRY(val2.alloc(ctx, kept));
        keep.offs.reset();
        RAMA_TRY((radix_sort_source<uint64_t, uint32_t>(ctx, RelabelledEdges{raw.get(), g.c.get(), dbits}, m, key, val, raw, val2, kept, nbits + dbits,
                                                        &head_sums, (uint64_t)n_new << dbits, &again)));
        raw.reset();
    } else {
        RAMA_TRY((scan_emit<uint32_t>(ctx, NotLoopKey{raw.get()}, CompactKeysEmit{raw.get(), g.c.get(), dbits, key.get(), val.get()},
                                      keep, (double)(m * 4 + (size_t)kept * 12))));
        keep.offs.reset();
        raw.reset();
        RAMA_TRY((radix_sort_pairs<uint64_t, uint32_t>(ctx, key, val, kept, nbits + dbits, false, &head_sums, (uint64_t)n_new << dbits, &again)));
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

rama_status contract_once(Ctx &ctx, const Graph &g, float tau, int rounds_cap, float forest_ratio, Buf<int32_t> &fmap,
                          int32_t &n_new, Graph &out, int64_t &n_matched, bool *used_forest, float *diag, bool *diag_made)
{
    const size_t n = (size_t)g.n;
    if (used_forest) *used_forest = false;
    n_new = g.n; n_matched = 0;
    // The rounds of a matching are enqueued without a look at the candidates; where it is known that there are none that costs
    // 35 us at the end of every solve, and 46 in a contraction of 10^6 repulsive edges, for nothing.
    if (g.none_attractive && tau >= 0.0f) return RAMA_OK;
    RAMA_TRY(zero_page_recycle(ctx));
    Buf<int32_t> mate;
    Candidates list;
    bool numbered = false;
    if (n <= (size_t)kNumberMax) RAMA_TRY(fmap.alloc(ctx, n > 0 ? n : 1));
    RAMA_TRY(matching(ctx, g, tau, rounds_cap, mate, n_matched, list, fmap.get(), &numbered));
    if (n_matched == 0) {
        fmap.reset();
        return RAMA_OK;
    }
    if (!fmap.get()) RAMA_TRY(fmap.alloc(ctx, n));
    // too few pairs: switch to the spanning forest without conflicts (Sec. 3.1, "fewer than 0.1|V|")
    const bool forest = forest_ratio > 0.0f && (double)n_matched < (double)forest_ratio * (double)g.n;
    if (!(forest && list.n <= kShortForest)) list = Candidates{};      // nobody else needs it, and what follows needs the memory
    if (forest) {
        Buf<uint32_t> npos;
        Buf<int32_t> si, sj, rep;
        mate.reset();
        if (used_forest) *used_forest = true;
        if (list.n > 0) {
            RAMA_TRY(forest_short(ctx, g, tau, list, rep, n_matched));
            list = Candidates{};
            if (n_matched == 0) return RAMA_OK;
        } else {
            RAMA_TRY(forest_set(ctx, g, tau, si, sj, n_matched));
            if (n_matched == 0) return RAMA_OK;
            RAMA_TRY(components(ctx, n, (size_t)n_matched, si.get(), sj.get(), rep));
        }
        RAMA_TRY(npos.alloc(ctx, n + 1));
        RAMA_TRY((exclusive_scan<uint32_t>(ctx, IsRoot{rep.get()}, npos.get(), n)));
        ProfScope ps_(ctx, "k_number", (double)(n * 12));
        k_number<<<grid_for(n), kBlock, 0, ctx.stream>>>(n, rep.get(), npos.get(), fmap.get());
        LAUNCH_TRY(ctx, "number");
    } else if (!numbered) {
        RAMA_TRY((scan_enumerate<uint32_t>(ctx, IsPairRoot{mate.get()}, NumberPairsEmit{mate.get(), fmap.get()}, n, (double)(n * 8))));
    }
    mate.reset();
    n_new = (int32_t)((int64_t)g.n - n_matched);   // S has no cycle: every edge of it removes one node, no need to ask the device
    if (forest) diag = nullptr;
    if (diag) {
        RAMA_TRY(fill<float>(ctx, diag, 0.0f, (size_t)n_new));
        *diag_made = true;
    }
    return contract_edges(ctx, g, fmap.get(), n_new, out, diag);
}

rama_status contraction_diagonal(Ctx &ctx, const Graph &g, const int32_t *fmap, int32_t n_new, float *diag)
{
    const size_t m = (size_t)g.m;
    RAMA_TRY(fill<float>(ctx, diag, 0.0f, (size_t)n_new));
    if (m == 0) return RAMA_OK;
    const InnerFlag inner{g.i.get(), g.j.get(), fmap};
    ScanPlan<uint32_t> plan;
    RAMA_TRY((scan_plan_alloc<uint32_t>(ctx, m, 0, plan)));
    RAMA_TRY((scan_totals<uint32_t>(ctx, inner, plan)));
    const uint32_t kept = plan.total;
    if (kept == 0) return RAMA_OK;
    Buf<uint32_t> key, val;
    RAMA_TRY(key.alloc(ctx, kept));
    RAMA_TRY(val.alloc(ctx, kept));
    RAMA_TRY((scan_emit<uint32_t>(ctx, inner, InnerEmit{g.i.get(), fmap, g.c.get(), key.get(), val.get()}, plan, (double)((size_t)kept * 16))));
    RAMA_TRY((radix_sort_pairs<uint32_t, uint32_t>(ctx, key, val, kept, bits_for((uint64_t)n_new), false, nullptr, (uint64_t)n_new)));
    {
        ProfScope ps_(ctx, "k_diag_runs", (double)((size_t)kept * 12));
        k_diag_runs<<<grid_for(kept), kBlock, 0, ctx.stream>>>(kept, key.get(), val.get(), diag);
    }
    LAUNCH_TRY(ctx, "diag_runs");
    return RAMA_OK;
}

}  // namespace rama
