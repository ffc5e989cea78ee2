// Device-wide primitives for gfx950, written for 64-wide wavefronts:
//   exclusive scan (reduce-then-scan, functor input), stable LSD radix sort (wave-level
//   match-any ranking), row boundaries of a sorted key array, deterministic sum reductions.
// Everything is integer-exact or uses a fixed reduction tree, so results do not depend on
// scheduling.
#pragma once

#include <list>

#include "common.h"
#include <type_traits>

namespace rama {

template <typename T>
rama_status fill(Ctx &ctx, T *p, T v, size_t n);   // defined with the reductions below

// `count` elements that are zero: from the ctx's page of zeroed words when they are few (no launch), else a block
// of their own plus a fill.  Page words are for use inside one stage (see zero_page_recycle).
template <typename T>
rama_status zeroed(Ctx &ctx, size_t count, Buf<T> &b)
{
    const size_t words = (count * sizeof(T) + 15) / 16 * 4;
    if (ctx.zero_page && words <= 1024 && ctx.zero_used + words <= rama_ctx::kZeroPageWords) {
        b.borrow((T *)(ctx.zero_page + ctx.zero_used), count);
        ctx.zero_used += words;
        return RAMA_OK;
    }
    RAMA_TRY(b.alloc(ctx, count > 0 ? count : 1));
    return fill<T>(ctx, b.get(), (T)0, count > 0 ? count : 1);
}
// At the start of a stage (nothing handed out from the page is needed any more): clear the page once half of it is used.
inline rama_status zero_page_recycle(Ctx &ctx)
{
    if (!ctx.zero_page || ctx.zero_used * 2 <= rama_ctx::kZeroPageWords) return RAMA_OK;
    RAMA_TRY(fill<uint32_t>(ctx, ctx.zero_page, 0u, rama_ctx::kZeroPageWords));
    ctx.zero_used = 0;
    return RAMA_OK;
}

// ------------------------------------------------------------------------------------------
// wave / block helpers
// ------------------------------------------------------------------------------------------
__device__ __forceinline__ int lane_id() { return (int)(threadIdx.x & 63); }

// A barrier that orders what the workgroup does in LDS and does not wait for its loads and stores elsewhere (__syncthreads
// does: up to a microsecond where any are under way).
__device__ __forceinline__ void lds_barrier()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// Consecutive workgroups of a launch go to the eight XCDs in turn, each with an L2 of its own.  A kernel whose
// neighbouring workgroups gather from the same stretch of an array then fetches that stretch into all eight L2s.
// Launched with xcd_grid(nb) workgroups and numbering its work by xcd_block(), a kernel gives every XCD one
// contiguous eighth of the work instead; numbers beyond nb - 1 come up for the padding and must leave at once.
// (The assignment of workgroups to XCDs only decides how well this works, not what is computed.)
inline uint32_t xcd_grid(uint32_t nb) { return ((nb + 7u) / 8u) * 8u; }
__device__ __forceinline__ uint32_t xcd_block()
{
    if (gridDim.x & 7u) return blockIdx.x;     // not launched with xcd_grid: plain numbering (every number still comes up once)
    return (blockIdx.x & 7u) * (gridDim.x >> 3) + (blockIdx.x >> 3);
}

template <typename T>
__device__ __forceinline__ T wave_inclusive_scan(T v)
{
    const int lane = lane_id();
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        T t = __shfl_up(v, off, 64);
        if (lane >= off) v += t;
    }
    return v;
}

// 32-bit integers: the same scan on the data-parallel-primitive path of the vector ALU instead of
// the LDS crossbar -- shifts by 1, 2, 4, 8 inside each row of 16 lanes, then lane 15 of rows 0 and
// 2 is broadcast into rows 1 and 3, then lane 31 into rows 2 and 3.  Lanes without a source add 0.
__device__ __forceinline__ uint32_t wave_inclusive_scan(uint32_t v)
{
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x111, 0xf, 0xf, false);   // row_shr:1
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x112, 0xf, 0xf, false);   // row_shr:2
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x114, 0xf, 0xf, false);   // row_shr:4
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x118, 0xf, 0xf, false);   // row_shr:8
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x142, 0xa, 0xf, false);   // row_bcast:15 -> rows 1, 3
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x143, 0xc, 0xf, false);   // row_bcast:31 -> rows 2, 3
    return v;
}
__device__ __forceinline__ int32_t wave_inclusive_scan(int32_t v) { return (int32_t)wave_inclusive_scan((uint32_t)v); }

// value of lane 63, the same in every lane
template <typename T>
__device__ __forceinline__ T wave_last(T v) { return __shfl(v, 63, 64); }
__device__ __forceinline__ uint32_t wave_last(uint32_t v) { return (uint32_t)__builtin_amdgcn_readlane((int)v, 63); }

template <typename T>
__device__ __forceinline__ T wave_sum(T v)
{
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
    return v;
}

// inclusive scan over the 256 threads of a block; *total gets the block sum
template <typename T>
__device__ __forceinline__ T block_inclusive_scan(T v, T *total)
{
    __shared__ T wave_tot[4];
    const int w = threadIdx.x >> 6;
    T inc = wave_inclusive_scan(v);
    if (lane_id() == 63) wave_tot[w] = inc;
    __syncthreads();
    T pre = 0, tot = 0;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        T x = wave_tot[k];
        if (k < w) pre += x;
        tot += x;
    }
    __syncthreads();
    *total = tot;
    return inc + pre;
}

// sum over the block in a fixed order (lane tree, then waves 0..3)
template <typename T>
__device__ __forceinline__ T block_sum(T v)
{
    __shared__ T wave_tot[4];
    T s = wave_sum(v);
    if (lane_id() == 0) wave_tot[threadIdx.x >> 6] = s;
    __syncthreads();
    T tot = ((wave_tot[0] + wave_tot[1]) + wave_tot[2]) + wave_tot[3];
    __syncthreads();
    return tot;
}

// ------------------------------------------------------------------------------------------
// scalars for the host: the mailbox
// ------------------------------------------------------------------------------------------
// The words of a message go to the host past the caches, and its number follows when they have arrived there: every wave
// waits for its own words.  A fence for the whole system would write the L2 back as well, of which the host sees nothing: with
// one in front of the number and one behind it a message of sixteen waves took 4 us.
__device__ __forceinline__ void mail_put(MailWord *to, uint64_t v) { __hip_atomic_store(&to->word_, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM); }
// 4-byte word k behind `to`
__device__ __forceinline__ void mail_put_half(MailWord *to, unsigned k, uint32_t v)
{
    __hip_atomic_store((uint32_t *)&to->word_ + k, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}
// closes message `seq`, all of whose words the calling wave has put into mail[1..]
__device__ __forceinline__ void mail_send_wave(MailWord *mail, uint64_t seq)
{
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    if (lane_id() == 0) mail_put(mail, seq);
}
// closes message `seq`: everything this workgroup put into mail[1..] before is visible to the host first
__device__ __forceinline__ void mail_send(MailWord *mail, uint64_t seq)
{
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (threadIdx.x == 0) mail_put(mail, seq);
}

// `words` 4-byte words from device memory into the mailbox, and `more` from another place behind them
static __global__ __launch_bounds__(kBlock) void k_publish(const uint32_t *src, unsigned words, const uint32_t *src2, unsigned more, MailWord *mail,
                                                           uint64_t seq)
{
    for (unsigned k = threadIdx.x; k < words; k += kBlock) mail_put_half(mail + 1, k, src[k]);
    for (unsigned k = threadIdx.x; k < more; k += kBlock) mail_put_half(mail + 1, words + k, src2[k]);
    mail_send(mail, seq);
}

// copy `bytes` (a multiple of 4, at most what a message holds with the `more` bytes from dev2 that go behind them) from
// device memory to the host and wait
inline rama_status read_back(Ctx &ctx, void *host, const void *dev, size_t bytes, const void *dev2 = nullptr, size_t more = 0)
{
    if (more == 0 && (bytes % 4 != 0 || bytes > (Ctx::kMailWords - 1) * 8)) return read_back_sync(ctx, host, dev, bytes);
    const uint64_t seq = ++ctx.mail_seq;
    k_publish<<<1, kBlock, 0, ctx.stream>>>((const uint32_t *)dev, (unsigned)(bytes / 4), (const uint32_t *)dev2, (unsigned)(more / 4), mailbox(ctx), seq);
    LAUNCH_TRY(ctx, "publish");
    RAMA_TRY(wait_mail(ctx, seq));
    memcpy(host, (const void *)(mail_words(ctx) + 1), bytes + more);
    return RAMA_OK;
}

// ------------------------------------------------------------------------------------------
// exclusive scan of f(0..n-1) into out[0..n] (out[n] = total)
// ------------------------------------------------------------------------------------------
// A workgroup owns a tile of 2048 consecutive items, each of its four waves 512 of them, taken
// 64 at a time: lane l of the wave reads item 64*q + l in step q, so every access is one
// contiguous 256-byte (or 512-byte) piece per wave.
constexpr int kScanItems = 8;
constexpr int kScanTile = kBlock * kScanItems;
constexpr int kScanWaveItems = 64 * kScanItems;

template <typename T>
struct PtrInput {
    static constexpr int bytes = (int)sizeof(T);   // bytes read per item
    static constexpr const char *tag = "PtrInput";
    const T *p;
    __device__ __forceinline__ T operator()(size_t k) const { return p[k]; }
};

// "<kernel><<functor tag>>", built once per (kernel, functor) pair
template <typename F>
inline const char *kernel_name(const char *kernel)
{
    static std::list<std::pair<std::string, std::string>> names;   // list: stable addresses
    for (auto &p : names) if (p.first == kernel) return p.second.c_str();
    names.emplace_back(std::string(kernel), std::string(kernel) + "<" + F::tag + ">");
    return names.back().second.c_str();
}

// exclusive scan of up to kScanMidMax tile sums by one workgroup, chunk after chunk; out[nb] = total
constexpr unsigned kScanMidMax = 1u << 13;
constexpr unsigned kScanFusedMax = 256;   // up to this many tiles (2^19 items) the reduce launch scans its own tile sums
template <typename TO, bool COHERENT>
__device__ __forceinline__ TO scan_tile_sums(const TO *in, TO *out, unsigned nb)
{
    TO carry = 0;
    for (unsigned c0 = 0; c0 < nb; c0 += kScanTile) {
        unsigned base = c0 + threadIdx.x * kScanItems;
        TO v[kScanItems];
        TO s = 0;
#pragma unroll
        for (int q = 0; q < kScanItems; ++q) {
            // sums written by other workgroups of the same launch are read past the local cache
            v[q] = (base + q < nb) ? (COHERENT ? __hip_atomic_load(in + base + q, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)
                                               : in[base + q])
                                   : (TO)0;
            s += v[q];
        }
        TO tot;
        TO run = block_inclusive_scan(s, &tot) - s + carry;
#pragma unroll
        for (int q = 0; q < kScanItems; ++q) {
            if (base + q < nb) out[base + q] = run;
            run += v[q];
        }
        carry += tot;
    }
    if (threadIdx.x == 0) out[nb] = carry;
    return carry;
}

// f(k), and 0 behind the end.  The last item is read there instead: a branch per item would end in the wait for its
// loads, and a thread's items would come one after the other.
template <typename TO, typename F>
__device__ __forceinline__ TO item_or_last(const F &f, size_t k, size_t n)
{
    const TO x = (TO)f(k < n ? k : n - 1);
    return k < n ? x : (TO)0;
}

// Tile sums.  With a ticket word the launch also scans them: every workgroup publishes its sum and draws
// a ticket; the one that draws the last ticket sees all sums, scans them into offs[0..nb] (offs[nb] = total),
// puts the ticket word back to zero and -- if a mailbox is given -- sends the total and the caller's
// `extra` words behind it (written by earlier launches) to the host.  One launch instead of two, and the
// total reaches the host without a copy.
template <typename TO, typename F>
__global__ __launch_bounds__(kBlock) void k_scan_reduce(F f, TO *block_sums, size_t n, TO *offs, uint32_t *ticket,
                                                        MailWord *mail, uint64_t seq, const TO *words, int extra)
{
    const size_t base = (size_t)blockIdx.x * kScanTile + threadIdx.x;
    TO s = 0, x[kScanItems];
#pragma unroll
    for (int q = 0; q < kScanItems; ++q) x[q] = item_or_last<TO>(f, base + (size_t)q * kBlock, n);
#pragma unroll
    for (int q = 0; q < kScanItems; ++q) s += x[q];
    TO tot = block_sum(s);
    if (!ticket) {
        if (threadIdx.x == 0) block_sums[blockIdx.x] = tot;
        return;
    }
    __shared__ bool last;
    if (threadIdx.x == 0) {
        __hip_atomic_store(block_sums + blockIdx.x, tot, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __threadfence();
        last = atomicAdd(ticket, 1u) == gridDim.x - 1;
    }
    __syncthreads();
    if (!last) return;
    __threadfence();
    const TO total = scan_tile_sums<TO, true>(block_sums, offs, gridDim.x);
    if (threadIdx.x == 0) *ticket = 0u;
    if (mail) {
        if (threadIdx.x == 0) {
            mail_put(mail + 1, (uint64_t)total);
            for (int e = 0; e < extra; ++e) mail_put(mail + 2 + e, (uint64_t)words[e]);
        }
        mail_send(mail, seq);
    }
}

// the scan of the tile sums as a launch of its own (long arrays: the election above would make every
// workgroup of the reduce launch wait for its sum to be visible, which costs more than a launch)
template <typename TO>
__global__ __launch_bounds__(kBlock) void k_scan_mid(const TO *in, TO *out, unsigned nb, MailWord *mail, uint64_t seq, const TO *words, int extra)
{
    const TO total = scan_tile_sums<TO, false>(in, out, nb);
    if (mail) {
        if (threadIdx.x == 0) {
            mail_put(mail + 1, (uint64_t)total);
            for (int e = 0; e < extra; ++e) mail_put(mail + 2 + e, (uint64_t)words[e]);
        }
        mail_send(mail, seq);
    }
}

template <typename TO, typename F>
__global__ __launch_bounds__(kBlock) void k_scan_apply(F f, TO *out, const TO *block_offsets, size_t n)
{
    __shared__ TO wave_tot[4];
    const int w = threadIdx.x >> 6;
    const size_t base = (size_t)blockIdx.x * kScanTile + (size_t)w * kScanWaveItems + lane_id();
    TO v[kScanItems];
#pragma unroll
    for (int q = 0; q < kScanItems; ++q) {
        const size_t k = base + (size_t)q * 64;
        v[q] = item_or_last<TO>(f, k, n);
    }
    TO carry = 0;   // sum of the wave's items before step q
#pragma unroll
    for (int q = 0; q < kScanItems; ++q) {
        const TO inc = wave_inclusive_scan(v[q]);
        v[q] = inc - v[q] + carry;
        carry += wave_last(inc);
    }
    if (lane_id() == 0) wave_tot[w] = carry;
    __syncthreads();
    TO pre = block_offsets ? block_offsets[blockIdx.x] : (TO)0;
#pragma unroll
    for (int k = 0; k < 3; ++k)
        if (k < w) pre += wave_tot[k];
#pragma unroll
    for (int q = 0; q < kScanItems; ++q) {
        const size_t k = base + (size_t)q * 64;
        if (k < n) out[k] = v[q] + pre;
    }
    if (blockIdx.x == gridDim.x - 1 && threadIdx.x == kBlock - 1) out[n] = pre + carry;
}

template <typename TO>
__global__ void k_store_zero(TO *p) { *p = 0; }

template <typename TO, typename F>
rama_status exclusive_scan(Ctx &ctx, F f, TO *out, size_t n);

// tile sums of f over n items (nb tiles) and their scan: offs[0..nb), offs[nb] = total
template <typename TO, typename F>
rama_status scan_offsets(Ctx &ctx, F f, TO *sums, TO *offs, size_t n, unsigned nb)
{
    const bool fused = nb <= kScanFusedMax;   // the last workgroup of the reduce launch scans the tile sums
    {
        ProfScope ps_(ctx, kernel_name<F>("k_scan_reduce"), (double)(n * F::bytes));
        k_scan_reduce<TO, F><<<nb, kBlock, 0, ctx.stream>>>(f, sums, n, offs, fused ? ctx.ticket : nullptr,
                                                           (MailWord *)nullptr, 0, (const TO *)nullptr, 0);
    }
    LAUNCH_TRY(ctx, "scan_reduce");
    if (!fused && nb <= kScanMidMax) {
        ProfScope ps_(ctx, "k_scan_mid", (double)((size_t)nb * 2 * sizeof(TO)));
        k_scan_mid<TO><<<1, kBlock, 0, ctx.stream>>>(sums, offs, nb, (MailWord *)nullptr, 0, (const TO *)nullptr, 0);
        LAUNCH_TRY(ctx, "scan_mid");
    } else if (!fused) {
        RAMA_TRY((exclusive_scan<TO, PtrInput<TO>>(ctx, PtrInput<TO>{sums}, offs, nb)));
    }
    return RAMA_OK;
}

template <typename TO, typename F>
rama_status exclusive_scan(Ctx &ctx, F f, TO *out, size_t n)
{
    if (n == 0) {
        {
            ProfScope ps_(ctx, "k_store_zero", (double)(0));
            k_store_zero<TO><<<1, 1, 0, ctx.stream>>>(out);
        }
        LAUNCH_TRY(ctx, "scan0");
        return RAMA_OK;
    }
    unsigned nb = grid_for(n, kScanTile);
    if (nb == 1) {
        {
            ProfScope ps_(ctx, kernel_name<F>("k_scan_apply"), (double)(n * (F::bytes + sizeof(TO))));
            k_scan_apply<TO, F><<<1, kBlock, 0, ctx.stream>>>(f, out, (const TO *)nullptr, n);
        }
        LAUNCH_TRY(ctx, "scan1");
        return RAMA_OK;
    }
    Buf<TO> sums, offs;
    RAMA_TRY(sums.alloc(ctx, nb));
    RAMA_TRY(offs.alloc(ctx, (size_t)nb + 1));
    RAMA_TRY((scan_offsets<TO, F>(ctx, f, sums.get(), offs.get(), n, nb)));
    {
        ProfScope ps_(ctx, kernel_name<F>("k_scan_apply"), (double)(n * (F::bytes + sizeof(TO))));
        k_scan_apply<TO, F><<<nb, kBlock, 0, ctx.stream>>>(f, out, offs.get(), n);
    }
    LAUNCH_TRY(ctx, "scan_apply");
    return RAMA_OK;
}

// ------------------------------------------------------------------------------------------
// Scan with a consumer instead of an output array.  scan_totals runs the reduce step and the scan of
// the tile sums and reads the total back (the caller sizes its outputs with it); scan_emit then
// recomputes f and hands every item k its value and exclusive prefix: emit(k, f(k), prefix).  The
// array of prefixes is never stored and the consumer does not re-read what the scan already had in
// registers.  `extra` words of the plan belong to the caller (e.g. a maximum a producer kernel left there); they start
// at zero and come back with the same read.
// ------------------------------------------------------------------------------------------
template <typename TO>
struct ScanPlan {
    Buf<TO> offs;   // [nb] tile offsets, [nb] total
    Buf<TO> sums;
    Buf<TO> words;  // the caller's extra words
    unsigned nb = 0;
    size_t n = 0;
    int extra = 0;
    TO total = 0;
    TO extra_value[2] = {0, 0};
    TO *extra_ptr() { return words.get(); }
};

template <typename TO>
rama_status scan_plan_alloc(Ctx &ctx, size_t n, int extra, ScanPlan<TO> &plan)
{
    plan.n = n;
    plan.nb = grid_for(n, kScanTile);
    plan.extra = extra;
    RAMA_TRY(plan.offs.alloc(ctx, (size_t)plan.nb + 1));
    RAMA_TRY(plan.sums.alloc(ctx, plan.nb > 0 ? plan.nb : 1));
    // the total is always written by the scan of the tile sums; only the caller's words start at zero
    if (extra > 0) return zeroed<TO>(ctx, (size_t)extra, plan.words);
    return RAMA_OK;
}

// `presums`: the tile sums exist already (the kernel that produced f's input left them, tile by tile of
// kScanTile items, in plan.sums or in an array of its own), so the counting launch is skipped
template <typename TO, typename F>
rama_status scan_totals(Ctx &ctx, F f, ScanPlan<TO> &plan, const TO *presums = nullptr)
{
    plan.total = 0;
    const unsigned nb = plan.nb;
    const bool presummed = presums != nullptr;
    const TO *sums = presummed ? presums : plan.sums.get();
    TO back[3] = {0, 0, 0};
    if (plan.n > 0 && nb <= kScanMidMax) {
        // short arrays, one launch: tile sums, their scan by the last workgroup, total and extra words into the
        // mailbox; longer arrays: the scan of the tile sums is a launch of its own
        const uint64_t seq = ++ctx.mail_seq;
        const bool fused = nb <= kScanFusedMax && !presummed;
        if (!presummed) {
            ProfScope ps_(ctx, kernel_name<F>("k_scan_reduce"), (double)(plan.n * F::bytes));
            k_scan_reduce<TO, F><<<nb, kBlock, 0, ctx.stream>>>(f, plan.sums.get(), plan.n, plan.offs.get(),
                                                               fused ? ctx.ticket : nullptr, mailbox(ctx), seq, plan.words.get(), plan.extra);
        }
        LAUNCH_TRY(ctx, "scan_reduce");
        if (!fused) {
            ProfScope ps_(ctx, "k_scan_mid", (double)((size_t)nb * 2 * sizeof(TO)));
            k_scan_mid<TO><<<1, kBlock, 0, ctx.stream>>>(sums, plan.offs.get(), nb, mailbox(ctx), seq, plan.words.get(), plan.extra);
            LAUNCH_TRY(ctx, "scan_mid");
        }
        RAMA_TRY(wait_mail(ctx, seq));
        const volatile uint64_t *m = mail_words(ctx);
        for (int k = 0; k < 1 + plan.extra; ++k) back[k] = (TO)m[1 + k];
    } else if (plan.n > 0) {
        if (!presummed) {
            ProfScope ps_(ctx, kernel_name<F>("k_scan_reduce"), (double)(plan.n * F::bytes));
            k_scan_reduce<TO, F><<<nb, kBlock, 0, ctx.stream>>>(f, plan.sums.get(), plan.n, (TO *)nullptr, (uint32_t *)nullptr,
                                                               (MailWord *)nullptr, 0, (const TO *)nullptr, 0);
        }
        LAUNCH_TRY(ctx, "scan_reduce");
        RAMA_TRY((exclusive_scan<TO, PtrInput<TO>>(ctx, PtrInput<TO>{sums}, plan.offs.get(), nb)));
        RAMA_TRY(read_back(ctx, back, plan.offs.get() + nb, sizeof(TO), plan.words.get(), (size_t)plan.extra * sizeof(TO)));
    } else if (plan.extra > 0) {
        RAMA_TRY(read_back(ctx, back + 1, plan.extra_ptr(), (size_t)plan.extra * sizeof(TO)));
    }
    plan.total = back[0];
    plan.extra_value[0] = back[1];
    plan.extra_value[1] = back[2];
    plan.sums.reset();
    return RAMA_OK;
}

// A consumer that works with whole waves (shuffles, ballots) declares `static constexpr bool whole_wave = true`:
// it is then also called for the places behind the end of the array, with value 0.
template <typename E, typename = void>
struct EmitWholeWave { static constexpr bool value = false; };
template <typename E>
struct EmitWholeWave<E, std::void_t<decltype(E::whole_wave)>> { static constexpr bool value = E::whole_wave; };

// A consumer that reads anything has a type `Item` and `Item load(k)`: its reads are made for all items of a thread before
// the scan, whether the item turns out to be taken or not, and operator() gets them.  Reads in operator() itself stand
// behind a branch and the stores of the item in front, so each item waits for its own.  With that, and the
// scanned values read the same way: 512^2 long-range solve 7.57 -> 7.35 ms, 6-NN graph of 10^6 points 12.35 -> 12.1, 320^3
// grid 91.8 -> 90.2, message passing on a 160^3 grid 3.59 -> 3.52.
struct NoItem {};
template <typename E, typename = void>
struct EmitItem { static constexpr bool value = false; using type = NoItem; };
template <typename E>
struct EmitItem<E, std::void_t<typename E::Item>> { static constexpr bool value = true; using type = typename E::Item; };

// A consumer that goes through a chain of dependent loads declares `static constexpr bool long_chain = true`: its items
// wait one after the other, so its tiles are worked on by 1024 threads with two items each (the list of triangles in the
// solve of a 128^2 long-range grid: 18.6 -> 9.3 us a launch; at 320^3, where there are waves enough, no difference).
template <typename E, typename = void>
struct EmitLongChain { static constexpr bool value = false; };
template <typename E>
struct EmitLongChain<E, std::void_t<decltype(E::long_chain)>> { static constexpr bool value = E::long_chain; };
constexpr int kChainThreads = 1024;

// SUMS: the tile sums have not been scanned; a workgroup adds up those in front of its tile, and the last one stores the total
// behind them (a few hundred tiles: less than a launch in between).
template <typename TO, typename F, typename E, int THREADS, bool SUMS>
__global__ __launch_bounds__(THREADS) void k_scan_emit(F f, E emit, std::conditional_t<SUMS, TO, const TO> *block_offsets, size_t n)
{
    constexpr int kItems = kScanTile / THREADS, kWaves = THREADS / 64;
    __shared__ TO wave_tot[kWaves];
    const int w = threadIdx.x >> 6;
    const size_t base = (size_t)blockIdx.x * kScanTile + (size_t)w * (64 * kItems) + lane_id();
    TO x[kItems], v[kItems];
    constexpr bool kLoads = EmitItem<E>::value;
    typename EmitItem<E>::type item[kLoads ? kItems : 1];
#pragma unroll
    for (int q = 0; q < kItems; ++q) {
        const size_t k = base + (size_t)q * 64;
        x[q] = item_or_last<TO>(f, k, n);
        if constexpr (kLoads) item[q] = emit.load(k < n ? k : n - 1);
    }
    TO carry = 0;
#pragma unroll
    for (int q = 0; q < kItems; ++q) {
        const TO inc = wave_inclusive_scan(x[q]);
        v[q] = inc - x[q] + carry;
        carry += wave_last(inc);
    }
    if (lane_id() == 0) wave_tot[w] = carry;
    TO pre = 0;
    if constexpr (SUMS) {
        static_assert(THREADS == kBlock, "block_sum");
        for (unsigned k = threadIdx.x; k < blockIdx.x; k += THREADS) pre += block_offsets[k];
        pre = block_sum(pre);      // its barriers are wave_tot's as well
        if (blockIdx.x == gridDim.x - 1 && threadIdx.x == 0) block_offsets[gridDim.x] = pre + block_offsets[blockIdx.x];
    } else {
        __syncthreads();
        pre = block_offsets[blockIdx.x];
    }
#pragma unroll
    for (int k = 0; k < kWaves - 1; ++k)
        if (k < w) pre += wave_tot[k];
#pragma unroll
    for (int q = 0; q < kItems; ++q) {
        const size_t k = base + (size_t)q * 64;
        if (EmitWholeWave<E>::value || k < n) {
            if constexpr (kLoads) emit(k, x[q], v[q] + pre, item[q]);
            else emit(k, x[q], v[q] + pre);
        }
    }
}

// `bytes`: what the consumer moves per launch beyond reading f's input (for the timers)
template <typename TO, typename F, typename E>
rama_status scan_emit(Ctx &ctx, F f, E emit, const ScanPlan<TO> &plan, double bytes)
{
    if (plan.n == 0) return RAMA_OK;
    {
        ProfScope ps_(ctx, kernel_name<E>("k_scan_emit"), (double)(plan.n * F::bytes) + bytes);
        constexpr int kThreads = EmitLongChain<E>::value ? kChainThreads : kBlock;
        k_scan_emit<TO, F, E, kThreads, false><<<plan.nb, kThreads, 0, ctx.stream>>>(f, emit, plan.offs.get(), plan.n);
    }
    LAUNCH_TRY(ctx, "scan_emit");
    return RAMA_OK;
}
// the same behind the tile sums alone (in plan.offs, which gets the total as well): a consumer whose total nobody on the host
// waits for
template <typename TO, typename F, typename E>
rama_status scan_emit_sums(Ctx &ctx, F f, E emit, const ScanPlan<TO> &plan, double bytes)
{
    if (plan.n == 0) return RAMA_OK;
    {
        ProfScope ps_(ctx, kernel_name<E>("k_scan_emit"), (double)(plan.n * F::bytes) + bytes);
        k_scan_emit<TO, F, E, kBlock, true><<<plan.nb, kBlock, 0, ctx.stream>>>(f, emit, plan.offs.get(), plan.n);
    }
    LAUNCH_TRY(ctx, "scan_emit");
    return RAMA_OK;
}

// scan_totals has run: the prefixes themselves, out[0..n]
template <typename TO, typename F>
rama_status scan_store(Ctx &ctx, F f, const ScanPlan<TO> &plan, TO *out)
{
    if (plan.n == 0) return RAMA_OK;
    {
        ProfScope ps_(ctx, kernel_name<F>("k_scan_apply"), (double)(plan.n * (F::bytes + sizeof(TO))));
        k_scan_apply<TO, F><<<plan.nb, kBlock, 0, ctx.stream>>>(f, out, plan.offs.get(), plan.n);
    }
    LAUNCH_TRY(ctx, "scan_apply");
    return RAMA_OK;
}

// scan_totals + scan_emit for a consumer that needs no total on the host: nobody waits
template <typename TO, typename F, typename E>
rama_status scan_enumerate(Ctx &ctx, F f, E emit, size_t n, double bytes)
{
    if (n == 0) return RAMA_OK;
    ScanPlan<TO> plan;
    RAMA_TRY((scan_plan_alloc<TO>(ctx, n, 0, plan)));
    RAMA_TRY((scan_offsets<TO, F>(ctx, f, plan.sums.get(), plan.offs.get(), n, plan.nb)));
    return scan_emit<TO>(ctx, f, emit, plan, bytes);
}

// ------------------------------------------------------------------------------------------
// row boundaries: keys[0..m) ascending with values in [0,n); ptr[v] = first position whose key
// is >= v, for v in [0,n]  (ptr[n] = m).  One launch, and every row is written exactly once:
//  - keys at least an eighth as many as rows: one thread per position fills the gap of rows before it when
//    the key changes there; a gap of more than kRowGapInline rows goes to a list in LDS that the whole
//    workgroup then fills side by side, so no thread ever loops over a long stretch alone;
//  - fewer keys than that (the empty stretches of a sparse key set are the rule): one thread per row,
//    binary search.
// ------------------------------------------------------------------------------------------
constexpr int kRowGapInline = 32;

// four positions per thread, read as one 16-byte vector (keys are 4 bytes wide)
template <typename K, typename P>
__global__ __launch_bounds__(kBlock) void k_row_bounds_fill(const K *keys, size_t m, int64_t n, P *ptr)
{
    static_assert(sizeof(K) == 4, "32-bit keys");
    __shared__ uint32_t s_count;
    __shared__ int64_t s_from[kBlock * 4], s_to[kBlock * 4];
    __shared__ P s_pos[kBlock * 4];
    if (threadIdx.x == 0) s_count = 0u;
    __syncthreads();
    const size_t e0 = ((size_t)blockIdx.x * kBlock + threadIdx.x) * 4;
    if (e0 <= m) {
        K k[4];
        if (e0 + 4 <= m) {
            const uint4 v = *reinterpret_cast<const uint4 *>(keys + e0);   // e0 is a multiple of 4, the array 16-byte aligned
            k[0] = (K)v.x; k[1] = (K)v.y; k[2] = (K)v.z; k[3] = (K)v.w;
        } else {
#pragma unroll
            for (int q = 0; q < 4; ++q) k[q] = e0 + q < m ? keys[e0 + q] : (K)0;
        }
        int64_t prev = (e0 == 0) ? -1 : (int64_t)keys[e0 - 1];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const size_t e = e0 + q;
            if (e > m) break;
            const int64_t cur = (e == m) ? n : (int64_t)k[q];
            if (cur != prev) {
                if (cur - prev <= kRowGapInline) {
                    for (int64_t v = prev + 1; v <= cur; ++v) ptr[v] = (P)e;
                } else {      // at most one entry per position: the list cannot overflow
                    const uint32_t slot = atomicAdd(&s_count, 1u);
                    s_from[slot] = prev + 1; s_to[slot] = cur; s_pos[slot] = (P)e;
                }
            }
            prev = cur;
        }
    }
    __syncthreads();
    const uint32_t n_long = s_count;
    for (uint32_t g = 0; g < n_long; ++g) {
        const int64_t to = s_to[g];
        const P e = s_pos[g];
        for (int64_t v = s_from[g] + threadIdx.x; v <= to; v += kBlock) ptr[v] = e;
    }
}

// four rows per thread; a row's search starts where the row before it ended
template <typename K, typename P>
__global__ __launch_bounds__(kBlock) void k_row_bounds_search(const K *keys, size_t m, int64_t n, P *ptr)
{
    const int64_t v0 = ((int64_t)blockIdx.x * kBlock + threadIdx.x) * 4;
    if (v0 > n) return;
    size_t from = 0;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int64_t v = v0 + q;
        if (v > n) break;
        size_t lo = from, hi = m;
        while (lo < hi) {
            size_t mid = lo + ((hi - lo) >> 1);
            if ((int64_t)keys[mid] < v) lo = mid + 1; else hi = mid;
        }
        ptr[v] = (P)lo;
        from = lo;
    }
}

// ------------------------------------------------------------------------------------------
// stable LSD radix sort, up to kRadixBits bits per pass, 6144 / 5120 keys per workgroup (fewer on
// arrays that would not fill the chip, see kSortShort and kSortMedium).
// Ranking inside a wave uses ballot-based match-any, so equal digits keep their order
// without any atomics in the scatter pass.
// ------------------------------------------------------------------------------------------
// Larger tiles give longer contiguous runs per digit on the way out; 6144 64-bit or 5120 32-bit keys measured best, beyond
// that the LDS footprint costs more than it gains.  A wave ranks its rows of 64 keys one after the other (see k_rs_scatter),
// so a tile is spread over eight waves: with four, two workgroups of 78 KB left two waves to a SIMD waiting for LDS.  One
// pass over 9.2e7 (64-bit key, value) pairs 0.68 -> 0.56 ms, over 1.9e8 32-bit pairs 0.77 -> 0.53 (4096-key rows of sixteen
// waves, 5120 and 6144 keys: 0.61 and 0.52).
template <typename K>
struct SortTile {
    static constexpr int threads = 512, items = sizeof(K) == 8 ? 12 : 10, tile = threads * items;
};
// Shorter arrays do not fill the chip with such tiles (10^6 keys: 163 workgroups for 256 CUs), so they get 2048 keys, and
// 1024 where even those tiles are fewer than the CUs.  Whole solves, ms, as the lines stand | kSortShort at 3 * 2^18 |
// kSortMedium at 6 * 2^20 | twice the keys a tile: 512^2 long-range grid 6.98 | 7.16 | 7.04 | 7.47, 6-NN graph of 10^6 points
// 11.4 | 11.7 | 11.7 | 11.9, 61x97x131 grid 7.2 | 7.4 | 7.2 | 7.9, 128^2 long-range grid 2.83 | 2.94 | 2.83 | 2.91; 256 threads
// instead of 512 for these tiles: 7.22, 11.8, 7.6, 3.00.
constexpr size_t kSortShort = size_t(3) << 16, kSortMedium = size_t(3) << 20;
constexpr int kShortTile = 1024, kShortThreads = 512, kMediumTile = 2048, kMediumThreads = 512;

constexpr int kRadixBits = 8;        // widest digit of a pass
constexpr int kRadix = 1 << kRadixBits;

// 16 bytes per lane and load: a plain copy with 4-byte accesses tops out near 3.8 TB/s on this
// chip, one with 16-byte accesses reaches 6 TB/s.  Only the histogram uses them: the scatter
// kernel gained nothing from 16-byte loads/stores, and a persistent variant that prefetches the
// next tile into registers was slower (its registers leave room for one workgroup per CU) -- it
// is bound by the latency of its load -> rank -> stage -> store chain at two tiles per CU.
// Chained passes (one histogram kernel for all digits, then per pass a single kernel whose tiles
// take tickets and read their predecessors' published digit counts instead of a scanned
// histogram) were also measured: the scatter kernels ran 25-50 % slower while they waited on the
// agent-scope status words, the all-digit histogram is bound by its LDS atomics, and the whole
// solve took 11 % longer than with histogram + scan + scatter per pass.
// Where one pass over 9.8e7 (64-bit key, value) pairs spent its time with tiles of four waves (one 8-bit pass, measured with
// keys built for the purpose; with eight waves it takes 0.56 ms, see SortTile): the scatter kernel took 0.78 ms on uniformly
// random digits, 0.57 ms when every key has the same digit (the output is then one sequential stream), and 0.47 ms for a
// 4-bit digit with sequential output -- so roughly 0.37 ms was moving the 24 bytes per key (6.3 TB/s),
// 0.2 ms the ballot ranking (about 26 us per digit bit) and 0.2 ms the cost of writing 256 separate
// pieces of ~24 keys per tile.  Computing all rows' ballots before touching the counters, or
// skipping the ballots for rows with a single digit, changed nothing measurable.
template <typename K>
struct alignas(16) KeyVec {
    K k[16 / sizeof(K)];
};

// The first pass of a sort may take its keys and values from a source instead of arrays: a functor that makes the key and
// the value of a place and tells by the key whether the place takes part (key 0 never does) or is left out.  What a
// compaction in front of the sort would write and the pass read again then never exists (both sides stand at
// RelabelledEdges).  All keys of a thread are made before the first is looked at: with a branch per place the loads
// wait one for the other, and the pass took 4.4 instead of 2.9 ms per solve of the 320^3 grid.
struct NoSource {};

// The [digit][tile] tables of a pass: a workgroup stores (and later fetches) one word in each of up to 256 rows.
// Workgroups take their tiles by xcd_block(): with tile = workgroup number, a cache line of a row collected the
// words of sixteen workgroups on eight XCDs, two words per L2, and went to memory in pieces (26 MB written for a
// 3.2 MB table); the runs the scatter kernel writes for neighbouring tiles meet in one L2 as well.
template <typename K, int ITEMS, typename SRC>
__global__ __launch_bounds__(kBlock) void k_rs_hist(const K *keys, SRC src, uint32_t *hist, size_t n, int shift, int bits,
                                                    uint32_t nb)
{
    constexpr bool kFromSource = !std::is_same<SRC, NoSource>::value;
    constexpr int kPer = 16 / (int)sizeof(K);                 // keys per vector
    constexpr int kVecs = ITEMS / kPer;                       // vectors per thread
    constexpr int kTile = kBlock * ITEMS;
    static_assert(ITEMS % kPer == 0, "tile must be a whole number of vectors per thread");
    __shared__ uint32_t h[kRadix];
    for (int k = threadIdx.x; k < kRadix; k += kBlock) h[k] = 0;
    __syncthreads();
    const uint32_t mask = (1u << bits) - 1u;
    const uint32_t tile_id = xcd_block();
    if (tile_id >= nb) return;      // the whole workgroup (padding of the grid)
    const size_t tile = (size_t)tile_id * kTile;
    // The top digits of nearly sorted keys (edge lists keyed by their first endpoint, the edges of
    // triangles listed triangle by triangle) take one, two or three values across a wave more often
    // than not, and atomics on one LDS word run one after the other: up to four times the lanes that
    // share the digit of the first lane left add their count once, as long as they are eight or more
    // (spread digits pay for one look only: on a neighbour graph's keys four looks per key made this
    // kernel 68 % slower); what is left then adds lane by lane.
    auto count = [&](K key, uint64_t left) {      // left: the lanes that hold a key, the same in all of them and not 0
        const uint32_t d = (uint32_t)(key >> shift) & mask;
#pragma unroll
        for (int round = 0; round < 4; ++round) {
            const int first = __ffsll((long long)left) - 1;
            const uint32_t d0 = (uint32_t)__builtin_amdgcn_readlane((int)d, first);
            const uint64_t same = __ballot(d == d0) & left;
            if (__popcll(same) < 8) break;                                     // uniform: digits are spread, no point
            if (lane_id() == first) atomicAdd(&h[d0], (uint32_t)__popcll(same));
            left &= ~same;
            if (left == 0ull) break;                                           // uniform
        }
        if (left & (1ull << lane_id())) atomicAdd(&h[d], 1u);
    };
    if constexpr (kFromSource) {
        K key[ITEMS];
#pragma unroll
        for (int r = 0; r < ITEMS; ++r) {
            const size_t idx = tile + (size_t)r * kBlock + threadIdx.x;
            const K k = src.key(idx < n ? idx : n - 1);
            key[r] = idx < n ? k : (K)0;
        }
#pragma unroll
        for (int r = 0; r < ITEMS; ++r) {
            const uint64_t lanes = __ballot(src.takes_part(key[r]));
            if (lanes) count(key[r], lanes);                                   // uniform
        }
    } else if (tile + kTile <= n) {               // full tile: vector loads (tile starts are 16-byte aligned)
        const KeyVec<K> *from = reinterpret_cast<const KeyVec<K> *>(keys + tile);
#pragma unroll
        for (int r = 0; r < kVecs; ++r) {
            KeyVec<K> v = from[(size_t)r * kBlock + threadIdx.x];
#pragma unroll
            for (int q = 0; q < kPer; ++q) count(v.k[q], ~0ull);
        }
    } else {
        for (size_t idx = tile + threadIdx.x; idx < n; idx += kBlock)
            atomicAdd(&h[(uint32_t)(keys[idx] >> shift) & mask], 1u);
    }
    __syncthreads();
    for (uint32_t d = threadIdx.x; d <= mask; d += kBlock) hist[(size_t)d * nb + tile_id] = h[d];
}

// Offsets of a pass from its [digit][tile] histogram: workgroup d scans row d (keys with digit d in
// earlier tiles) and stores the row's total behind the table; the scatter kernel adds the keys of
// smaller digits itself, from the 256 totals.  One launch instead of the three of a general scan.  In place: a thread
// reads its words before the barriers of the scan and writes the same ones behind them (with tiles of 1024 and 2048 keys
// a second table took more than the tiles of 6144 ever did).
static __global__ __launch_bounds__(kBlock) void k_rs_rowscan(uint32_t *hist, uint32_t nb, uint32_t *totals)
{
    uint32_t *row = hist + (size_t)blockIdx.x * nb;
    uint32_t carry = 0;
    for (uint32_t c0 = 0; c0 < nb; c0 += kScanTile) {
        const uint32_t base = c0 + threadIdx.x * kScanItems;
        uint32_t v[kScanItems], s = 0;
#pragma unroll
        for (int q = 0; q < kScanItems; ++q) {
            v[q] = (base + q < nb) ? row[base + q] : 0u;
            s += v[q];
        }
        uint32_t tot;
        uint32_t run = block_inclusive_scan(s, &tot) - s + carry;
#pragma unroll
        for (int q = 0; q < kScanItems; ++q) {
            if (base + q < nb) row[base + q] = run;
            run += v[q];
        }
        carry += tot;
    }
    if (threadIdx.x == 0) totals[blockIdx.x] = carry;
}

__device__ __forceinline__ uint64_t match_digit(uint32_t d, int bits, uint64_t valid)
{
    uint64_t m = valid;
    for (int b = 0; b < bits; ++b) {
        bool bit = (d >> b) & 1u;
        uint64_t bal = __ballot(bit);
        m &= bit ? bal : ~bal;
    }
    return m;
}

// One pass of the sort for one tile: (1) every wave ranks its items x 64 keys by digit with ballots,
// (2) per-digit prefix over the tile's waves and over the digits gives each key its place in the
// tile's digit-sorted order, (3) keys (and values) are staged in LDS in that order, (4) the tile
// is written out linearly -- neighbouring lanes hold neighbouring keys of the same digit, so the
// global stores fall into contiguous runs instead of 64 scattered lines per instruction.
// With LOCAL_SCAN (few tiles) `offs` is the raw [digit][tile] histogram and every workgroup derives
// its own global offsets from it, which saves the scan launch of the pass.
constexpr uint32_t kSortLocalScanTiles = 32;
// Waves per SIMD that the LDS of a workgroup leaves room for, which is what the registers have to allow as well (pairs; keys
// alone have LDS to spare and would spill).
template <bool HAS_V>
constexpr int rs_scatter_waves(int lds_bytes, int threads)
{
    const int waves = (160 * 1024 / lds_bytes) * (threads / 64) / 4;
    return !HAS_V ? 1 : waves > 8 ? 8 : waves;
}
template <typename K, typename V, bool HAS_V, bool LOCAL_SCAN, int THREADS, int ITEMS, typename SRC>
__global__ __launch_bounds__(THREADS, (rs_scatter_waves<HAS_V>(THREADS * ITEMS * ((int)sizeof(K) + 4) + THREADS * 8 + 1088, THREADS))) void k_rs_scatter(const K *kin, const V *vin, SRC src, K *kout, V *vout,
                                                        const uint32_t *offs, size_t n, int shift, int bits,
                                                        uint32_t nb, uint32_t *starts)
{
    constexpr bool kFromSource = !std::is_same<SRC, NoSource>::value;
    constexpr int kTile = THREADS * ITEMS, NW = THREADS / 64;
    static_assert(THREADS >= kRadix && kRadix == 256 && kTile < (1 << 16), "one digit per thread of the first four waves, 16-bit counts");
    __shared__ uint16_t whist[NW][kRadix];
    __shared__ uint32_t gdelta[kRadix];
    __shared__ uint32_t s_run[4], s_rows[4];
    __shared__ K skey[kTile];
    __shared__ uint32_t sval[HAS_V ? kTile : 1];
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const uint32_t mask = (1u << bits) - 1u;
    const uint32_t tile_id = xcd_block();
    if (tile_id >= nb) return;      // the whole workgroup (padding of the grid)
    for (int k = tid; k < NW * kRadix / 2; k += THREADS) reinterpret_cast<uint32_t *>(&whist[0][0])[k] = 0;
    __syncthreads();
    const size_t tile_base = (size_t)tile_id * kTile;
    const size_t wave_base = tile_base + (size_t)w * (64 * ITEMS);
    const uint64_t lt = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
    K key[ITEMS];
    uint32_t val[ITEMS];
    uint32_t rank[ITEMS];
#pragma unroll
    for (int r = 0; r < ITEMS; ++r) {
        size_t idx = wave_base + (size_t)r * 64 + lane;
        bool valid = idx < n;
        if constexpr (kFromSource) {
            const size_t at = valid ? idx : n - 1;
            const K k = src.key(at);
            key[r] = valid ? k : (K)0;
            if (HAS_V) val[r] = src.value(at);
        } else {
            key[r] = valid ? kin[idx] : (K)0;
            if (HAS_V) val[r] = valid ? (vin ? (uint32_t)vin[idx] : (uint32_t)idx) : 0u;   // no array of values: a key's value is its place
        }
    }
    auto takes_part = [&](int r) {
        if constexpr (kFromSource) return src.takes_part(key[r]);
        else return wave_base + (size_t)r * 64 + lane < n;
    };
#pragma unroll
    for (int r = 0; r < ITEMS; ++r) {
        bool valid = takes_part(r);
        uint32_t d = (uint32_t)(key[r] >> shift) & mask;
        uint64_t m = match_digit(d, bits, __ballot(valid));
        uint32_t before = whist[w][d];
        rank[r] = before + (uint32_t)__popcll(m & lt);
        __builtin_amdgcn_wave_barrier();
        if (valid && lane == (__ffsll((long long)m) - 1)) whist[w][d] = (uint16_t)(before + (uint32_t)__popcll(m));
        __builtin_amdgcn_wave_barrier();
    }
    // thread d < 256 owns digit d: the tile's keys with it, wave by wave, and where they go in the output
    uint32_t c[NW], tot = 0, in_tot = 0, in_rows = 0, rows = 0, before = 0;
    if (tid < kRadix && tid <= (int)mask) {
        if (LOCAL_SCAN) {      // keys with the digit in all tiles, and in earlier ones
            for (uint32_t b = 0; b < nb; ++b) {
                const uint32_t h = offs[(size_t)tid * nb + b];
                if (b < tile_id) before += h;
                rows += h;
            }
        } else {               // offs: per digit the keys in earlier tiles, and behind the table the digits' totals
            rows = offs[((size_t)nb << bits) + tid];
            before = offs[(size_t)tid * nb + tile_id];
        }
    }
    __syncthreads();
    if (tid < kRadix) {
#pragma unroll
        for (int k = 0; k < NW; ++k) { c[k] = whist[k][tid]; tot += c[k]; }
        in_tot = wave_inclusive_scan(tot);
        in_rows = wave_inclusive_scan(rows);
        if (lane == 63) { s_run[w] = in_tot; s_rows[w] = in_rows; }
    }
    __syncthreads();
    if (tid < kRadix) {
        uint32_t run = in_tot - tot, digit = in_rows - rows;
#pragma unroll
        for (int k = 0; k < 3; ++k)
            if (k < w) { run += s_run[k]; digit += s_rows[k]; }
        gdelta[tid] = digit + before - run;
        // where the digits' keys begin, and the end of the last one's; only arrays with small tiles are asked (the code alone
        // costs the large ones registers: 2.4e7 32-bit pairs 83 -> 105 us)
        if constexpr (kTile <= kMediumTile)
            if (starts && tile_id == 0 && tid <= (int)mask) {
                starts[tid] = digit;
                if (tid == (int)mask) starts[mask + 1u] = digit + rows;
            }
#pragma unroll
        for (int k = 0; k < NW; ++k) { whist[k][tid] = (uint16_t)run; run += c[k]; }
    }
    __syncthreads();
    const uint32_t cnt = s_run[0] + s_run[1] + s_run[2] + s_run[3];
#pragma unroll
    for (int r = 0; r < ITEMS; ++r) {
        if (takes_part(r)) {
            uint32_t d = (uint32_t)(key[r] >> shift) & mask;
            uint32_t lpos = whist[w][d] + rank[r];
            skey[lpos] = key[r];
            if (HAS_V) sval[lpos] = val[r];
        }
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < ITEMS; ++r) {
        uint32_t idx = (uint32_t)r * THREADS + tid;
        if (idx < cnt) {
            K k = skey[idx];
            uint32_t pos = gdelta[(uint32_t)(k >> shift) & mask] + idx;
            kout[pos] = k;
            if (HAS_V) vout[pos] = (V)sval[idx];
        }
    }
}

template <typename K, bool HAS_V>
inline const char *rs_scatter_name()
{
    if (HAS_V) return sizeof(K) == 8 ? "k_rs_scatter<u64,u32>" : "k_rs_scatter<u32,u32>";
    return sizeof(K) == 8 ? "k_rs_scatter<u64>" : "k_rs_scatter<u32>";
}

// ---- split sort: the top bits by LSD passes, the rest inside LDS ----------------------------------
// After stable passes over the top bits the array consists of segments of equal top bits, each of
// which only has to be sorted by its low bits -- and a segment that fits into LDS is sorted there in
// one read and one write of the data, however many digits its low bits have.  Workgroup b takes the
// segments that START inside window [b*W, (b+1)*W): bounds[b] is the first segment start at or
// behind b*W, so a workgroup holds fewer than W + (longest segment) elements.  `oversize` is raised
// when that exceeds what a workgroup can hold; the caller then sorts the classical way.
template <typename K>
__device__ __forceinline__ size_t first_segment_start_from(const K *keys, size_t n, int low_bits, size_t x)
{
    if (x == 0) return 0;
    if (x >= n) return n;
    const K p = keys[x] >> low_bits;
    if ((keys[x - 1] >> low_bits) != p) return x;
    // end of the segment that contains x: gallop, then bisect.  keys[lo] has top bits p, keys[hi] has not (or hi == n)
    size_t lo = x, hi, step = 1;
    for (;;) {
        hi = lo + step;
        if (hi >= n) { hi = n; break; }
        if ((keys[hi] >> low_bits) != p) break;
        lo = hi;
        step <<= 1;
    }
    while (hi - lo > 1) {
        const size_t mid = lo + (hi - lo) / 2;
        if ((keys[mid] >> low_bits) == p) lo = mid; else hi = mid;
    }
    return hi;
}

template <typename K>
__global__ __launch_bounds__(kBlock) void k_seg_bounds(const K *keys, size_t n, int low_bits, uint32_t window, uint32_t cap,
                                                       int local_key_bits, uint32_t nbk, uint32_t *bounds, uint32_t *oversize)
{
    const uint32_t b = blockIdx.x * kBlock + threadIdx.x;
    if (b > nbk) return;
    if (b == nbk) { bounds[b] = (uint32_t)n; return; }
    const size_t f0 = first_segment_start_from(keys, n, low_bits, (size_t)b * window);
    const size_t f1 = first_segment_start_from(keys, n, low_bits, (size_t)(b + 1) * window);
    bounds[b] = (uint32_t)f0;
    if (f1 - f0 > cap) *oversize = 1u;
    if (f1 > f0) {      // the workgroup's keys relative to its first segment must fit the local key type
        const uint64_t top_span = (uint64_t)((keys[f1 - 1] >> low_bits) - (keys[f0] >> low_bits));
        if (low_bits + (top_span ? 64 - __clzll((long long)top_span) : 0) > local_key_bits) *oversize = 1u;
    }
}

// Sorts the elements [bounds[b], bounds[b+1]) by their low bits (and by the few top bits in which
// the segments of one workgroup differ: the keys are taken relative to the first segment's top
// bits, so those cost digits only where a workgroup spans many sparse segments).  Waves hold
// consecutive chunks, the passes are those of k_rs_scatter with LDS as the destination; between
// passes the keys return to registers in the new order.
// LK is the type of the keys while they are being sorted: 32 bits whenever the low bits (plus the
// few top bits in which a workgroup's segments differ) fit, which halves the LDS a key takes.
// What counts is the number of waves a CU holds: 8 keys x 16 waves fill it with two workgroups (9.2e7 (64-bit key, value)
// pairs with 27 low bits 0.99 ms, 1.9e8 32-bit pairs 1.37); 16 keys x 8 waves, with keys and values side by side in LDS, left
// two waves to a SIMD free (1.24 and 1.63 ms), and with one of them after the other the registers did (1.13 and 1.56).
constexpr int kLocalSortWaves = 16;
constexpr int kBucketBits = 12, kBucketMax = 32, kAtATime = 4;
template <typename LK>
struct LocalSort {
    static constexpr int items = sizeof(LK) == 8 ? 4 : 8;
    static constexpr int threads = kLocalSortWaves * 64;
    static constexpr int cap = threads * items;
};
template <typename LK>
struct LocalSortShared {
    __align__(16) uint16_t whist[kLocalSortWaves][kRadix];
    uint32_t wave_tot[4], bucket_tot[kLocalSortWaves];
    LK buf[LocalSort<LK>::cap + kAtATime];      // the words that are compared (read a few at a time, beyond the last), then the keys, then the values
};
// Sorts cnt keys of sort_bits bits (stable): item r of lane l in wave w is number (w * rows + r) * 64 + l.  In the end the keys
// stand in S.buf in their order, rank[r] is the place of key r there (of the key that came last to this thread, if there
// were passes: val goes along), and everybody has passed a barrier.
template <bool HAS_V, typename LK>
__device__ __forceinline__ void local_sort(LocalSortShared<LK> &S, LK (&key)[LocalSort<LK>::items], uint32_t (&val)[LocalSort<LK>::items],
                                           uint32_t (&rank)[LocalSort<LK>::items], int rows, uint32_t cnt, int sort_bits)
{
    constexpr int NW = kLocalSortWaves, kItems = LocalSort<LK>::items, kThreads = LocalSort<LK>::threads, kCap = LocalSort<LK>::cap;
    static_assert(kRadix == 256 && kThreads >= kRadix, "one digit per thread of the first four waves");
    auto &whist = S.whist;
    auto &wave_tot = S.wave_tot;
    auto &bucket_tot = S.bucket_tot;
    LK *const sbuf = S.buf;
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int passes = (sort_bits + kRadixBits - 1) / kRadixBits;
    const uint32_t wave_base = (uint32_t)w * (uint32_t)rows * 64u;
    const uint64_t lt = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
    // Buckets first: the top kBucketBits of the keys' differing bits split the few thousand keys into buckets of one to
    // a few (an edge list: the edges of a node).  Count and place by LDS atomics -- in any order --, then every key
    // finds its place among its bucket's keys by comparing.  What is compared is one word: the bits below the bucket's
    // and, behind them, the place the key came from, so that equal keys keep their order and no second array is read.
    // Keys and values then go through the same LDS one after the other.
    // A bucket of more than kBucketMax keys, or bits that do not fit the word, send the workgroup through the passes.
    uint16_t *const s_end = &whist[0][0];
    constexpr int kMyWords = (1 << kBucketBits) / 2 / kThreads;      // words of two counters
    static_assert(NW * kRadix >= (1 << kBucketBits) && kThreads * kMyWords * 2 == (1 << kBucketBits), "bucket counters take the digit counters' place");
    const int bucket_shift = sort_bits > kBucketBits ? sort_bits - kBucketBits : 0;
    constexpr int kPlaceBits = 13;
    static_assert(kCap <= (1 << kPlaceBits), "a place fits its bits");
    const LK low_mask = (LK)(((LK)1 << bucket_shift) - 1);
    auto word_of = [&](LK k, uint32_t place) { return (LK)(((k & low_mask) << kPlaceBits) | (LK)place); };
    bool passes_needed = bucket_shift + kPlaceBits > 8 * (int)sizeof(LK);
    if (!passes_needed) {      // uniform
        uint32_t *words = reinterpret_cast<uint32_t *>(&whist[0][0]);
#pragma unroll
        for (int k = 0; k < kMyWords; ++k) words[tid * kMyWords + k] = 0;
        __syncthreads();
#pragma unroll
        for (int r = 0; r < kItems; ++r) {
            if (r < rows) {
                const uint32_t idx = wave_base + (uint32_t)r * 64u + lane;
                if (idx < cnt) {
                    const uint32_t b = (uint32_t)(key[r] >> bucket_shift);
                    rank[r] = (atomicAdd(&words[b >> 1], 1u << (16 * (b & 1))) >> (16 * (b & 1))) & 0xffffu;   // counts below 2^14: no carry
                }
            }
        }
        __syncthreads();
        uint32_t c[2 * kMyWords], mine = 0, longest = 0;
#pragma unroll
        for (int k = 0; k < kMyWords; ++k) {
            const uint32_t x = words[tid * kMyWords + k];
            c[2 * k] = x & 0xffffu; c[2 * k + 1] = x >> 16;
            mine += c[2 * k] + c[2 * k + 1];
            longest = max(longest, max(c[2 * k], c[2 * k + 1]));
        }
        const uint32_t inc = wave_inclusive_scan(mine);
        if (lane == 63) bucket_tot[w] = inc;
        passes_needed = __syncthreads_or(longest > (uint32_t)kBucketMax) != 0;
        if (!passes_needed) {      // uniform
            uint32_t run = inc - mine;
#pragma unroll
            for (int k = 0; k < NW - 1; ++k)
                if (k < w) run += bucket_tot[k];
#pragma unroll
            for (int k = 0; k < kMyWords; ++k) {      // ends of the buckets
                const uint32_t e0 = run + c[2 * k], e1 = e0 + c[2 * k + 1];
                words[tid * kMyWords + k] = e0 | e1 << 16;
                run = e1;
            }
            __syncthreads();
#pragma unroll
            for (int r = 0; r < kItems; ++r) {
                if (r < rows) {
                    const uint32_t idx = wave_base + (uint32_t)r * 64u + lane;
                    if (idx < cnt) {
                        const uint32_t b = (uint32_t)(key[r] >> bucket_shift);
                        sbuf[(b ? s_end[b - 1] : 0u) + rank[r]] = word_of(key[r], idx);
                    }
                }
            }
            __syncthreads();
#pragma unroll
            for (int r = 0; r < kItems; ++r) {
                if (r < rows) {
                    const uint32_t idx = wave_base + (uint32_t)r * 64u + lane;
                    if (idx < cnt) {
                        const uint32_t b = (uint32_t)(key[r] >> bucket_shift);
                        const uint32_t b0 = b ? s_end[b - 1] : 0u, b1 = s_end[b];
                        const LK self = word_of(key[r], idx);
                        uint32_t at = b0;
                        for (uint32_t p = b0; p < b1; p += kAtATime) {
                            LK x[kAtATime];
#pragma unroll
                            for (int k = 0; k < kAtATime; ++k) x[k] = sbuf[p + k];
#pragma unroll
                            for (int k = 0; k < kAtATime; ++k) at += p + k < b1 && x[k] < self ? 1u : 0u;
                        }
                        rank[r] = at;
                    }
                }
            }
            __syncthreads();
#pragma unroll
            for (int r = 0; r < kItems; ++r) {
                if (r < rows) {
                    const uint32_t idx = wave_base + (uint32_t)r * 64u + lane;
                    if (idx < cnt) sbuf[rank[r]] = key[r];
                }
            }
        }
        __syncthreads();
    }
    int shift = 0, remaining = sort_bits;
    for (int p = 0; passes_needed && p < passes; ++p) {
        const int bits = (remaining + (passes - p) - 1) / (passes - p);
        const uint32_t mask = (1u << bits) - 1u;
        for (int k = tid; k < NW * kRadix / 2; k += kThreads) reinterpret_cast<uint32_t *>(&whist[0][0])[k] = 0;
        __syncthreads();
#pragma unroll
        for (int r = 0; r < kItems; ++r) {
            if (r < rows) {
                const uint32_t idx = wave_base + (uint32_t)r * 64u + lane;
                const bool valid = idx < cnt;
                const uint32_t d = (uint32_t)(key[r] >> shift) & mask;
                const uint64_t m = match_digit(d, bits, __ballot(valid));
                const uint32_t before = whist[w][d];
                rank[r] = before + (uint32_t)__popcll(m & lt);
                __builtin_amdgcn_wave_barrier();
                if (valid && lane == (__ffsll((long long)m) - 1)) whist[w][d] = (uint16_t)(before + (uint32_t)__popcll(m));
                __builtin_amdgcn_wave_barrier();
            }
        }
        __syncthreads();
        {   // thread d < 256 owns digit d: places of the waves' keys with this digit in the sorted order
            uint32_t c[NW], tot = 0;
            if (tid < kRadix) {
#pragma unroll
                for (int k = 0; k < NW; ++k) { c[k] = whist[k][tid]; tot += c[k]; }
            }
            const uint32_t inc = wave_inclusive_scan(tot);
            if (tid < kRadix && lane == 63) wave_tot[w] = inc;
            __syncthreads();
            if (tid < kRadix) {
                uint32_t run = inc - tot;
#pragma unroll
                for (int k = 0; k < 3; ++k)
                    if (k < w) run += wave_tot[k];
#pragma unroll
                for (int k = 0; k < NW; ++k) { whist[k][tid] = (uint16_t)run; run += c[k]; }
            }
        }
        __syncthreads();
#pragma unroll
        for (int r = 0; r < kItems; ++r) {
            if (r < rows) {
                const uint32_t idx = wave_base + (uint32_t)r * 64u + lane;
                if (idx < cnt) {
                    const uint32_t d = (uint32_t)(key[r] >> shift) & mask;
                    rank[r] += whist[w][d];
                    sbuf[rank[r]] = key[r];
                }
            }
        }
        __syncthreads();
        if (p + 1 < passes) {      // keys, then values, come back in the new order; after the last pass they go out below
            auto take_turn = [&](auto &x, bool bring) {
                if (bring) {
                    __syncthreads();
#pragma unroll
                    for (int r = 0; r < kItems; ++r)
                        if (r < rows && wave_base + (uint32_t)r * 64u + lane < cnt) sbuf[rank[r]] = (LK)x[r];
                    __syncthreads();
                }
#pragma unroll
                for (int r = 0; r < kItems; ++r) {
                    const uint32_t idx = wave_base + (uint32_t)r * 64u + lane;
                    if (r < rows && idx < cnt) x[r] = (std::remove_reference_t<decltype(x[r])>)sbuf[idx];
                }
            };
            take_turn(key, false);
            if (HAS_V) take_turn(val, true);
            __syncthreads();
        }
        shift += bits;
        remaining -= bits;
    }
}

template <typename K, typename V, bool HAS_V, typename LK>
__global__ __launch_bounds__(kLocalSortWaves * 64, 8) void k_rs_local(const K *kin, const V *vin, K *kout, V *vout,
                                                                   const uint32_t *bounds, int low_bits, uint32_t n_all,
                                                                   uint32_t *head_sums, uint32_t *oversize)
{
    constexpr int kItems = LocalSort<LK>::items;
    constexpr int kThreads = LocalSort<LK>::threads;
    constexpr int kCap = LocalSort<LK>::cap;
    __shared__ LocalSortShared<LK> S;
    LK *const sbuf = S.buf;
    // without a bounds array the (single) workgroup takes the whole array of n_all keys
    const uint32_t beg = bounds ? bounds[blockIdx.x] : 0u, end = bounds ? bounds[blockIdx.x + 1] : n_all;
    const uint32_t cnt = end - beg;
    if (cnt == 0 || cnt > (uint32_t)kCap) {      // the second case: ruled out by the caller, or told to it
        if (cnt && oversize && threadIdx.x == 0) *oversize = 1u;
        return;
    }
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const K base = (kin[beg] >> low_bits) << low_bits;
    const uint64_t top_span = (uint64_t)((kin[end - 1] >> low_bits) - (kin[beg] >> low_bits));
    const int sort_bits = low_bits + (top_span ? 64 - __clzll((long long)top_span) : 0);
    const int rows = (int)((cnt + kThreads - 1) / kThreads);       // rows of 64 keys per wave
    const uint32_t wave_base = (uint32_t)w * (uint32_t)rows * 64u;
    LK key[kItems];
    uint32_t val[kItems];
    uint32_t rank[kItems];
#pragma unroll
    for (int r = 0; r < kItems; ++r) {
        const uint32_t idx = wave_base + (uint32_t)r * 64u + lane;
        const bool valid = r < rows && idx < cnt;
        key[r] = valid ? (LK)(kin[beg + idx] - base) : (LK)0;
        if (HAS_V) val[r] = valid ? (uint32_t)vin[beg + idx] : 0u;
    }
    local_sort<HAS_V>(S, key, val, rank, rows, cnt, sort_bits);
    auto values_out = [&]() {      // behind the keys, through the same LDS
        __syncthreads();
#pragma unroll
        for (int r = 0; r < kItems; ++r)
            if (r < rows && wave_base + (uint32_t)r * 64u + lane < cnt) sbuf[rank[r]] = (LK)val[r];
        __syncthreads();
        for (uint32_t idx = tid; idx < cnt; idx += kThreads) vout[beg + idx] = (V)sbuf[idx];
    };
    if (!head_sums) {   // uniform
        for (uint32_t idx = tid; idx < cnt; idx += kThreads) kout[beg + idx] = (K)((K)sbuf[idx] + base);
        if (HAS_V) values_out();
        return;
    }
    // The sorted keys are at hand: count the heads of runs of equal keys per tile of kScanTile places, for a scan
    // over the heads that follows the sort (it then needs no counting pass).  A workgroup's first key starts a
    // new segment of top bits, so it is a head; its places span at most kHeadTiles tiles.
    constexpr int kHeadTiles = kCap / kScanTile + 1;
    __shared__ uint32_t s_heads[kHeadTiles];
    if (tid < kHeadTiles) s_heads[tid] = 0;
    __syncthreads();
    const uint32_t tile0 = beg / (uint32_t)kScanTile;
    for (uint32_t idx0 = 0; idx0 < cnt; idx0 += kThreads) {
        const uint32_t idx = idx0 + tid;
        const bool valid = idx < cnt;
        bool head = false;
        if (valid) {
            const LK k = sbuf[idx];
            kout[beg + idx] = (K)((K)k + base);
            head = idx == 0 || k != sbuf[idx - 1];
        }
        // the wave's 64 places lie in one tile or in two
        const uint32_t first = beg + idx0 + (uint32_t)w * 64u;
        const uint32_t t_lo = first / (uint32_t)kScanTile, t_hi = (first + 63u) / (uint32_t)kScanTile;
        const uint64_t heads = __ballot(head);
        if (t_lo == t_hi) {
            if (lane == 0 && heads) atomicAdd(&s_heads[t_lo - tile0], (uint32_t)__popcll(heads));
        } else {
            const uint32_t n_lo = t_hi * (uint32_t)kScanTile - first;     // places of the wave that lie in the lower tile
            const uint64_t low = (~0ull) >> (64u - n_lo);
            if (lane == 0) {
                if (heads & low) atomicAdd(&s_heads[t_lo - tile0], (uint32_t)__popcll(heads & low));
                if (heads & ~low) atomicAdd(&s_heads[t_hi - tile0], (uint32_t)__popcll(heads & ~low));
            }
        }
    }
    __syncthreads();
    if (HAS_V) values_out();
    if (tid < kHeadTiles && s_heads[tid]) atomicAdd(&head_sums[tile0 + tid], s_heads[tid]);
}

template <typename K, bool HAS_V, typename LK>
inline const char *rs_local_name()
{
    if (sizeof(LK) == 8) {      // 64-bit keys inside LDS: the low bits did not fit 32
        if (HAS_V) return sizeof(K) == 8 ? "k_rs_local<u64,u32,wide>" : "k_rs_local<u32,u32,wide>";
        return sizeof(K) == 8 ? "k_rs_local<u64,wide>" : "k_rs_local<u32,wide>";
    }
    if (HAS_V) return sizeof(K) == 8 ? "k_rs_local<u64,u32>" : "k_rs_local<u32,u32>";
    return sizeof(K) == 8 ? "k_rs_local<u64>" : "k_rs_local<u32>";
}

// one pass: histogram (unless it is there: `counted`), offsets, scatter
template <typename K, typename V, bool HAS_V, int THREADS, int ITEMS, typename SRC>
rama_status radix_pass(Ctx &ctx, const K *ka, const V *va, const SRC &src, K *kb, V *vb, size_t n, int shift, int bits, uint32_t *hist, uint32_t *starts,
                       bool counted = false)
{
    const uint32_t nb = grid_for(n, THREADS * ITEMS);
    if (!counted) {
        ProfScope ps_(ctx, (sizeof(K) == 8 ? "k_rs_hist<u64>" : "k_rs_hist<u32>"), (double)(n * sizeof(K)));
        k_rs_hist<K, THREADS * ITEMS / kBlock, SRC><<<xcd_grid(nb), kBlock, 0, ctx.stream>>>(ka, src, hist, n, shift, bits, nb);
    }
    LAUNCH_TRY(ctx, "rs_hist");
    if (nb <= kSortLocalScanTiles) {
        ProfScope ps_(ctx, rs_scatter_name<K, HAS_V>(), (double)(n * (2 * sizeof(K) + (HAS_V ? 8 : 0))));
        k_rs_scatter<K, V, HAS_V, true, THREADS, ITEMS, SRC><<<xcd_grid(nb), THREADS, 0, ctx.stream>>>(ka, va, src, kb, vb, hist, n, shift, bits, nb, starts);
    } else {
        {
            ProfScope ps_(ctx, "k_rs_rowscan", (double)(((size_t)nb << bits) * 8));
            k_rs_rowscan<<<1u << bits, kBlock, 0, ctx.stream>>>(hist, nb, hist + ((size_t)nb << bits));
        }
        LAUNCH_TRY(ctx, "rs_rowscan");
        ProfScope ps_(ctx, rs_scatter_name<K, HAS_V>(), (double)(n * (2 * sizeof(K) + (HAS_V ? 8 : 0))));
        k_rs_scatter<K, V, HAS_V, false, THREADS, ITEMS, SRC><<<xcd_grid(nb), THREADS, 0, ctx.stream>>>(ka, va, src, kb, vb, hist, n, shift, bits, nb, starts);
    }
    LAUNCH_TRY(ctx, "rs_scatter");
    return RAMA_OK;
}
// the tile by the number of keys n; a pass over a source goes over its n_src >= n places in tiles of the same size
template <typename K, typename V, bool HAS_V, typename SRC>
rama_status radix_pass_sized(Ctx &ctx, const K *ka, const V *va, const SRC &src, K *kb, V *vb, size_t n, size_t places, int shift, int bits,
                             uint32_t *hist, uint32_t *starts)
{
    if (n <= kSortShort) return radix_pass<K, V, HAS_V, kShortThreads, kShortTile / kShortThreads, SRC>(ctx, ka, va, src, kb, vb, places, shift, bits, hist, starts);
    if (n <= kSortMedium) return radix_pass<K, V, HAS_V, kMediumThreads, kMediumTile / kMediumThreads, SRC>(ctx, ka, va, src, kb, vb, places, shift, bits, hist, starts);
    return radix_pass<K, V, HAS_V, SortTile<K>::threads, SortTile<K>::items, SRC>(ctx, ka, va, src, kb, vb, places, shift, bits, hist, starts);
}
// stable LSD passes over the key bits [shift, shift + total_bits); a/b swap with every pass.  starts (optional): where the
// keys of every digit of the last pass begin, and n.
template <typename K, typename V, bool HAS_V, typename SRC>
rama_status radix_passes(Ctx &ctx, K *&ka, V *&va, K *&kb, V *&vb, size_t n, int shift, int total_bits, uint32_t *hist,
                         bool *result_in_b, bool *iota, K *&kc, V *&vc, const SRC *&src, size_t n_src, uint32_t *starts = nullptr)
{
    const int passes = (total_bits + kRadixBits - 1) / kRadixBits;
    int remaining = total_bits;
    for (int p = 0; p < passes; ++p) {
        int bits = (remaining + (passes - p) - 1) / (passes - p);
        const V *vin = (HAS_V && *iota) ? (const V *)nullptr : va;   // the first pass of a sort whose values are the places 0..n-1
        *iota = false;
        if (src) {
            RAMA_TRY((radix_pass_sized<K, V, HAS_V, SRC>(ctx, ka, vin, *src, kb, vb, n, n_src, shift, bits, hist, starts)));
            src = nullptr;
        } else {
            RAMA_TRY((radix_pass_sized<K, V, HAS_V, NoSource>(ctx, ka, vin, NoSource{}, kb, vb, n, n, shift, bits, hist, starts)));
        }
        std::swap(ka, kb);
        std::swap(va, vb);
        if (kc) {   // the input must stay as it is: from now on the passes alternate between the two other buffers
            kb = kc; vb = vc;
            kc = nullptr; vc = nullptr;
        }
        *result_in_b = !*result_in_b;
        shift += bits;
        remaining -= bits;
    }
    return RAMA_OK;
}

// zeroed counters for the heads per scan tile of an array of n sorted keys (k_rs_local fills them)
inline rama_status head_sums_alloc(Ctx &ctx, size_t n, Buf<uint32_t> *head_sums)
{
    if (!head_sums) return RAMA_OK;
    const size_t tiles = (n + kScanTile - 1) / kScanTile + 1;
    return zeroed<uint32_t>(ctx, tiles, *head_sums);
}

// bounds + in-LDS sort of an array already sorted by its bits above low_bits; *done stays false
// when some workgroup could not hold its segments (nothing has been written then)
template <typename K, typename V, bool HAS_V, typename LK>
rama_status split_sort_tail(Ctx &ctx, K *ka, V *va, K *kb, V *vb, size_t n, int low_bits, bool *done, Buf<uint32_t> *head_sums)
{
    using LS = LocalSort<LK>;
    *done = false;
    const uint32_t window = LS::cap / 2;
    const uint32_t nbk = grid_for(n, (int)window);
    Buf<uint32_t> bounds, over_flag;
    RAMA_TRY(bounds.alloc(ctx, (size_t)nbk + 1));
    RAMA_TRY(zeroed<uint32_t>(ctx, 1, over_flag));
    uint32_t *oversize = over_flag.get();
    {
        ProfScope ps_(ctx, "k_seg_bounds", (double)((size_t)nbk * (4 + 32 * sizeof(K))));
        k_seg_bounds<K><<<grid_for((size_t)nbk + 1), kBlock, 0, ctx.stream>>>(ka, n, low_bits, window, (uint32_t)LS::cap,
                                                                             8 * (int)sizeof(LK), nbk, bounds.get(), oversize);
    }
    LAUNCH_TRY(ctx, "seg_bounds");
    uint32_t over = 0;
    RAMA_TRY(read_back(ctx, &over, oversize, 4));
    if (over) return RAMA_OK;
    RAMA_TRY(head_sums_alloc(ctx, n, head_sums));
    {
        ProfScope ps_(ctx, rs_local_name<K, HAS_V, LK>(), (double)(n * (2 * sizeof(K) + (HAS_V ? 8 : 0))));
        k_rs_local<K, V, HAS_V, LK><<<nbk, LS::threads, 0, ctx.stream>>>(ka, va, kb, vb, bounds.get(), low_bits, (uint32_t)n,
                                                                      head_sums ? head_sums->get() : nullptr, (uint32_t *)nullptr);
    }
    LAUNCH_TRY(ctx, "rs_local");
    *done = true;
    return RAMA_OK;
}

// A sort of a few hundred thousand keys is launches and nothing else, so it takes one pass over the top bits and one in-LDS
// sort, a workgroup to a digit, and nobody waits to hear whether every digit's keys fit: the in-LDS sort raises a flag if
// not, which comes to the host with the count that it waits for behind the sort anyway (count_heads), and the keys are sorted
// by passes then.  So is what comes after them in the same call: a node that crowds one digit does so in the contracted graphs
// as well (contraction to the end of 3.4e5 edges with one row of 40000, ms, switched off | tried at every sort 42.0 | 44.6, of
// 6e4 edges with one of 20000 3.88 | 4.14, of 8e5 edges with falling degrees 63.5 | 65.6).  Bits of that pass: digits of
// kUnseenSegment keys on average, a fifth of the 32-bit words that a workgroup holds and three eighths of the 64-bit ones, or
// of half as many as it holds at most where eight bits are too few for that.  0: no such sort.
// 1.3e5 64-bit pairs: four launches instead of nine; contraction of a 300x301 long-range grid 2.17 -> 1.95 ms, 128^2 long-range
// solve 2.36 -> 2.17, 512^2 5.87 -> 5.69, 6-NN graph of 10^6 points 9.95 -> 9.66, 61x97x131 volume 5.80 -> 5.55.  (The split sort,
// which waits to hear, measured the same as passes from 2^16 keys up to its line at 2^21.)
constexpr size_t kUnseenSegment = 1536;
inline int unseen_top_bits(size_t n, int total_bits, uint64_t key_limit, bool *narrow)
{
    for (int t = 1; t <= kRadixBits && t < total_bits; ++t) {
        const int low = total_bits - t;
        *narrow = low <= 32;
        const size_t cap = (size_t)(*narrow ? LocalSort<uint32_t>::cap : LocalSort<uint64_t>::cap);
        const uint64_t digits = key_limit ? ((key_limit - 1) >> low) + 1 : uint64_t(1) << t;
        const size_t seg = (size_t)(((uint64_t)n + digits - 1) / digits);
        if (seg <= cap / 2 && (seg <= kUnseenSegment || t == kRadixBits)) return t;
    }
    return 0;
}
inline int unseen_bits_now(const Ctx &ctx, size_t n, int total_bits, uint64_t key_limit, bool *narrow)
{
    if (!ctx.sorts_unseen || n >= ctx.sort_split_min || ctx.sort_split_min >= (size_t)INT64_MAX) return 0;
    return unseen_top_bits(n, total_bits, key_limit, narrow);
}
static_assert((LocalSort<uint32_t>::cap / 2) << kRadixBits <= kSortMedium, "tiles that tell where the digits begin");
struct SortUnseen {
    uint32_t *flag = nullptr;      // a zeroed word
    bool used = false;
};

// Sorts keys (and 32-bit values) by the low `total_bits` bits of the key.  a/b are two buffers
// of n elements each; input in a; on return *result_in_b says where the sorted data is.
// Long arrays are split when that replaces at least two passes: passes over the top bits until
// the segments of equal top bits are at most two fifths of a workgroup's capacity on average, then one
// in-LDS sort of the rest.  Should the keys be so uneven that some workgroup cannot hold its
// segments, the array (by then stably sorted by the top bits, which does no harm) is sorted by
// passes over all bits instead.
// `iota`: the values are the places 0..n-1 and va holds nothing yet -- the first pass makes them up instead of
// reading them (an array one workgroup sorts alone gets them from a fill first).
static __global__ __launch_bounds__(kBlock) void k_iota(size_t n, uint32_t *p)
{
    size_t k = (size_t)blockIdx.x * kBlock + threadIdx.x;
    if (k < n) p[k] = (uint32_t)k;
}
template <typename K, typename V, bool HAS_V, typename SRC = NoSource>
rama_status radix_sort_impl(Ctx &ctx, K *ka, V *va, K *kb, V *vb, size_t n, int total_bits, bool *result_in_b, bool iota = false,
                            Buf<uint32_t> *head_sums = nullptr, uint64_t key_limit = 0, K *kc = nullptr, V *vc = nullptr,
                            K **res_k = nullptr, V **res_v = nullptr, const SRC *src = nullptr, size_t n_src = 0, SortUnseen *unseen = nullptr)
{
    // src (optional): the keys and values come from a source of n_src places, n of which take part; there is no input a
    // then, and n is more than one workgroup sorts alone
    // kc, vc (optional): a third pair of buffers; the input a is then only read, and the sorted data ends up in b or
    // in c: *res_k, *res_v say where
    // key_limit (optional): all keys are below it (and it needs total_bits bits); 0 = nothing known
    // unseen (optional): the sort may be one that fails later (see unseen_top_bits); if so, unseen->used says it, and the
    // keys that the in-LDS sort read, in the other buffers, must stay until the flag is known
    if (key_limit && (total_bits >= 64 || key_limit > (uint64_t(1) << total_bits))) key_limit = 0;
    // head_sums (optional): comes back allocated and filled -- per tile of kScanTile places the number of keys that
    // differ from their left neighbour -- when the sort ends in the in-LDS kernel, and empty otherwise
    if (head_sums) head_sums->reset();
    *result_in_b = false;
    if (n <= 1 || total_bits <= 0) return RAMA_OK;
    if (n >= (size_t(1) << 32)) return fail(ctx, RAMA_ERR_CAPACITY, "radix sort: more than 2^32 keys");
    // an array that one workgroup can hold is sorted inside LDS by a single launch
    if (total_bits < 8 * (int)sizeof(K) && ctx.sort_split_min < (size_t)INT64_MAX) {
        const bool narrow = total_bits <= 32 && n <= (size_t)LocalSort<uint32_t>::cap;
        const bool wide = !narrow && n <= (size_t)LocalSort<uint64_t>::cap;
        if ((narrow || wide) && HAS_V && iota) {
            ProfScope ps_(ctx, "k_iota", (double)(n * 4));
            k_iota<<<grid_for(n), kBlock, 0, ctx.stream>>>(n, (uint32_t *)va);
            LAUNCH_TRY(ctx, "iota");
            iota = false;
        }
        if (narrow || wide) {
            RAMA_TRY(head_sums_alloc(ctx, n, head_sums));
            uint32_t *hs = head_sums ? head_sums->get() : nullptr;
            if (narrow) {
                ProfScope ps_(ctx, rs_local_name<K, HAS_V, uint32_t>(), (double)(n * (2 * sizeof(K) + (HAS_V ? 8 : 0))));
                k_rs_local<K, V, HAS_V, uint32_t><<<1, LocalSort<uint32_t>::threads, 0, ctx.stream>>>(ka, va, kb, vb, (const uint32_t *)nullptr,
                                                                                                  total_bits, (uint32_t)n, hs, (uint32_t *)nullptr);
            } else {
                ProfScope ps_(ctx, rs_local_name<K, HAS_V, uint64_t>(), (double)(n * (2 * sizeof(K) + (HAS_V ? 8 : 0))));
                k_rs_local<K, V, HAS_V, uint64_t><<<1, LocalSort<uint64_t>::threads, 0, ctx.stream>>>(ka, va, kb, vb, (const uint32_t *)nullptr,
                                                                                                  total_bits, (uint32_t)n, hs, (uint32_t *)nullptr);
            }
            LAUNCH_TRY(ctx, "rs_local");
            *result_in_b = true;
            if (res_k) { *res_k = kb; *res_v = vb; }
            return RAMA_OK;
        }
    }
    bool unseen_narrow = false;
    const int unseen_bits = unseen ? unseen_bits_now(ctx, n, total_bits, key_limit, &unseen_narrow) : 0;
    const uint32_t nb = grid_for(src ? n_src : n, n <= kSortShort ? kShortTile : n <= kSortMedium ? kMediumTile : SortTile<K>::tile);
    const int all_passes = (total_bits + kRadixBits - 1) / kRadixBits;
    // [digit][tile] and the digits' totals, for the widest digit of a pass (the top bits of a split sort: whole digits)
    const int digit_bits = unseen_bits ? unseen_bits : n >= ctx.sort_split_min ? kRadixBits : (total_bits + all_passes - 1) / all_passes;
    Buf<uint32_t> hist;
    RAMA_TRY(hist.alloc(ctx, ((size_t)nb + 1) << digit_bits));
    if (unseen_bits) {
        Buf<uint32_t> starts;
        RAMA_TRY(starts.alloc(ctx, ((size_t)1 << unseen_bits) + 1));
        const int low_bits = total_bits - unseen_bits;
        RAMA_TRY((radix_passes<K, V, HAS_V, SRC>(ctx, ka, va, kb, vb, n, low_bits, unseen_bits, hist.get(), result_in_b, &iota, kc, vc, src, n_src, starts.get())));
        RAMA_TRY(head_sums_alloc(ctx, n, head_sums));
        uint32_t *hs = head_sums ? head_sums->get() : nullptr;
        if (unseen_narrow) {
            ProfScope ps_(ctx, rs_local_name<K, HAS_V, uint32_t>(), (double)(n * (2 * sizeof(K) + (HAS_V ? 8 : 0))));
            k_rs_local<K, V, HAS_V, uint32_t><<<1u << unseen_bits, LocalSort<uint32_t>::threads, 0, ctx.stream>>>(ka, va, kb, vb, starts.get(), low_bits,
                                                                                                             (uint32_t)n, hs, unseen->flag);
        } else {
            ProfScope ps_(ctx, rs_local_name<K, HAS_V, uint64_t>(), (double)(n * (2 * sizeof(K) + (HAS_V ? 8 : 0))));
            k_rs_local<K, V, HAS_V, uint64_t><<<1u << unseen_bits, LocalSort<uint64_t>::threads, 0, ctx.stream>>>(ka, va, kb, vb, starts.get(), low_bits,
                                                                                                             (uint32_t)n, hs, unseen->flag);
        }
        LAUNCH_TRY(ctx, "rs_local");
        unseen->used = true;
        *result_in_b = !*result_in_b;
        if (res_k) { *res_k = kb; *res_v = vb; }
        return RAMA_OK;
    }
    if (n >= ctx.sort_split_min) {
        // top bits: whole passes, enough of them for segments that a workgroup can hold.  A workgroup takes the
        // segments that start in half a capacity of places, so what it gets stays below the capacity as long as no
        // segment is longer than half the capacity.  Without knowledge of the keys the segments are assumed to be a
        // quarter of the capacity on average at most (the keys seldom fill the whole range of their bits: fewer,
        // longer segments).  With a bound on the keys (`key_limit`) the number of segments is known and two fifths of
        // the capacity are allowed (the incidence sort of the 320^3 grid, 1.9e8 keys below 1.3e8: two top-bit passes
        // and one in-LDS sort instead of four passes, -0.6 ms).  A few spare low bits leave room for the top bits in
        // which a workgroup's segments differ.
        auto plan = [&](int cap, int *top_bits) {
            const uint64_t seg = key_limit ? (uint64_t)cap * 2 / 5 : (uint64_t)cap / 4;
            int t = kRadixBits;
            for (; t < total_bits; t += kRadixBits) {
                const uint64_t nseg = key_limit ? ((key_limit - 1) >> (total_bits - t)) + 1 : (uint64_t(1) << t);
                if (((uint64_t)n + nseg - 1) / nseg <= seg) break;
            }
            *top_bits = t;
            return t < total_bits && all_passes - t / kRadixBits >= ctx.sort_split_gain;
        };
        int top_bits = 0;
        bool narrow = plan(LocalSort<uint32_t>::cap, &top_bits) && total_bits - top_bits + 6 <= 32;
        const bool split = narrow || plan(LocalSort<uint64_t>::cap, &top_bits);
        if (split) {
            const int low_bits = total_bits - top_bits;
            RAMA_TRY((radix_passes<K, V, HAS_V, SRC>(ctx, ka, va, kb, vb, n, low_bits, top_bits, hist.get(), result_in_b, &iota, kc, vc, src, n_src)));
            bool done = false;
            if (narrow) RAMA_TRY((split_sort_tail<K, V, HAS_V, uint32_t>(ctx, ka, va, kb, vb, n, low_bits, &done, head_sums)));
            else RAMA_TRY((split_sort_tail<K, V, HAS_V, uint64_t>(ctx, ka, va, kb, vb, n, low_bits, &done, head_sums)));
            if (done) {
                *result_in_b = !*result_in_b;
                if (res_k) { *res_k = kb; *res_v = vb; }
                return RAMA_OK;
            }
        }
    }
    RAMA_TRY((radix_passes<K, V, HAS_V, SRC>(ctx, ka, va, kb, vb, n, 0, total_bits, hist.get(), result_in_b, &iota, kc, vc, src, n_src)));
    if (res_k) { *res_k = ka; *res_v = va; }
    return RAMA_OK;
}

// The other pair of buffers of a sort that may turn out to have failed, and the flag that tells.
template <typename K, typename V>
struct SortAgain : SortUnseen {
    Buf<K> k;
    Buf<V> v;
    SortUnseen *unseen() { return flag ? this : nullptr; }
};

// Convenience wrappers working on Buf pairs: after the call `k`/`v` hold the sorted data.
// `iota`: v comes in unset and stands for the values 0..n-1
template <typename K, typename V>
rama_status radix_sort_pairs(Ctx &ctx, Buf<K> &k, Buf<V> &v, size_t n, int total_bits, bool iota = false,
                             Buf<uint32_t> *head_sums = nullptr, uint64_t key_limit = 0, SortAgain<K, V> *again = nullptr)
{
    static_assert(sizeof(V) == 4, "32-bit payload");
    if (head_sums) head_sums->reset();
    if (n <= 1 || total_bits <= 0) {
        if (iota && n >= 1) {
            k_iota<<<grid_for(n), kBlock, 0, ctx.stream>>>(n, (uint32_t *)v.get());
            LAUNCH_TRY(ctx, "iota");
        }
        return RAMA_OK;
    }
    Buf<K> k2;
    Buf<V> v2;
    RAMA_TRY(k2.alloc(ctx, n));
    RAMA_TRY(v2.alloc(ctx, n));
    bool in_b = false;
    RAMA_TRY((radix_sort_impl<K, V, true>(ctx, k.get(), v.get(), k2.get(), v2.get(), n, total_bits, &in_b, iota, head_sums, key_limit,
                                                 (K *)nullptr, (V *)nullptr, (K **)nullptr, (V **)nullptr, (const NoSource *)nullptr, 0,
                                                 again ? again->unseen() : nullptr)));
    if (in_b) { k.swap(k2); v.swap(v2); }
    if (again && again->used) { again->k = std::move(k2); again->v = std::move(v2); }
    return RAMA_OK;
}

// The same sort for the places of a source (see NoSource), n of whose n_src places take part.  k, v and the second pair
// k2, v2 come in allocated for n each; k2 may hold what the source reads (the first pass writes k and v only).
// For what one workgroup sorts alone there is no first pass; and the pass goes twice over the places that take no part and
// keeps its table for them, so where they are more than half the list is compacted first.
inline bool sort_takes_source(size_t n, size_t n_src)
{
    static_assert(LocalSort<uint64_t>::cap <= LocalSort<uint32_t>::cap, "no longer array is sorted by one workgroup");
    return n > (size_t)LocalSort<uint32_t>::cap && n >= n_src / 2;
}
template <typename K, typename V, typename SRC>
rama_status radix_sort_source(Ctx &ctx, const SRC &source, size_t n_src, Buf<K> &k, Buf<V> &v, Buf<K> &k2, Buf<V> &v2, size_t n, int total_bits,
                              Buf<uint32_t> *head_sums, uint64_t key_limit, SortAgain<K, V> *again = nullptr)
{
    static_assert(sizeof(V) == 4, "32-bit payload");
    bool in_b = false;
    K *rk = nullptr;
    V *rv = nullptr;
    RAMA_TRY((radix_sort_impl<K, V, true, SRC>(ctx, (K *)nullptr, (V *)nullptr, k.get(), v.get(), n, total_bits, &in_b, false, head_sums, key_limit,
                                               k2.get(), v2.get(), &rk, &rv, &source, n_src, again ? again->unseen() : nullptr)));
    if (rk == k2.get()) { k.swap(k2); v.swap(v2); }
    if (again && again->used) { again->k = std::move(k2); again->v = std::move(v2); }
    return RAMA_OK;
}

// The same sort for pairs that must stay where they are (kin, vin are only read): k, v are allocated here and hold
// the sorted pairs on return.
template <typename K, typename V>
rama_status radix_sort_pairs_from(Ctx &ctx, const K *kin, const V *vin, Buf<K> &k, Buf<V> &v, size_t n, int total_bits,
                                  uint64_t key_limit = 0)
{
    static_assert(sizeof(V) == 4, "32-bit payload");
    RAMA_TRY(k.alloc(ctx, n > 0 ? n : 1));
    RAMA_TRY(v.alloc(ctx, n > 0 ? n : 1));
    if (n <= 1 || total_bits <= 0) {
        if (n > 0) {
            HIP_TRY(ctx, hipMemcpyAsync(k.get(), kin, n * sizeof(K), hipMemcpyDeviceToDevice, ctx.stream));
            HIP_TRY(ctx, hipMemcpyAsync(v.get(), vin, n * sizeof(V), hipMemcpyDeviceToDevice, ctx.stream));
        }
        return RAMA_OK;
    }
    Buf<K> k2;
    Buf<V> v2;
    RAMA_TRY(k2.alloc(ctx, n));
    RAMA_TRY(v2.alloc(ctx, n));
    bool in_b = false;
    K *rk = nullptr;
    V *rv = nullptr;
    RAMA_TRY((radix_sort_impl<K, V, true>(ctx, const_cast<K *>(kin), const_cast<V *>(vin), k.get(), v.get(), n, total_bits, &in_b, false,
                                          nullptr, key_limit, k2.get(), v2.get(), &rk, &rv)));
    if (rk == k2.get()) { k.swap(k2); v.swap(v2); }
    return RAMA_OK;
}

template <typename K>
rama_status radix_sort_keys(Ctx &ctx, Buf<K> &k, size_t n, int total_bits, Buf<uint32_t> *head_sums = nullptr, uint64_t key_limit = 0,
                            SortAgain<K, uint32_t> *again = nullptr)
{
    if (head_sums) head_sums->reset();
    if (n <= 1) return RAMA_OK;
    Buf<K> k2;
    RAMA_TRY(k2.alloc(ctx, n));
    bool in_b = false;
    RAMA_TRY((radix_sort_impl<K, uint32_t, false>(ctx, k.get(), (uint32_t *)nullptr, k2.get(), (uint32_t *)nullptr, n,
                                                  total_bits, &in_b, false, head_sums, key_limit, (K *)nullptr, (uint32_t *)nullptr,
                                                  (K **)nullptr, (uint32_t **)nullptr, (const NoSource *)nullptr, 0, again ? again->unseen() : nullptr)));
    if (in_b) k.swap(k2);
    if (again && again->used) again->k = std::move(k2);
    return RAMA_OK;
}

// What follows a sort whose flag is the word `word` of `plan`: the heads of the sorted keys are counted (scan_totals) and the
// count comes to the host with the flag.  If it is raised, the keys are sorted once more, from the buffers that the
// in-LDS sort read (in the order of their top bits, which does no harm), and counted again.  flags(k): the scan's input.
template <typename K, typename V, typename FLAGS>
rama_status count_heads(Ctx &ctx, Buf<K> &k, Buf<V> *v, size_t n, int total_bits, const FLAGS &flags, ScanPlan<uint32_t> &plan, int word,
                        Buf<uint32_t> &head_sums, SortAgain<K, V> &again)
{
    RAMA_TRY((scan_totals<uint32_t>(ctx, flags(k.get()), plan, head_sums.get())));
    head_sums.reset();
    if (!again.used || !plan.extra_value[word]) {
        again.k.reset(); again.v.reset();
        return RAMA_OK;
    }
    ctx.sorts_unseen = false;
    const uint32_t nb = grid_for(n, n <= kSortShort ? kShortTile : n <= kSortMedium ? kMediumTile : SortTile<K>::tile);
    Buf<uint32_t> hist;
    RAMA_TRY(hist.alloc(ctx, ((size_t)nb + 1) << kRadixBits));
    K *ka = again.k.get(), *kb = k.get(), *kc = nullptr;
    V *va = again.v.get(), *vb = v ? v->get() : nullptr, *vc = nullptr;
    bool in_b = false, iota = false;
    const NoSource *src = nullptr;
    if (v) RAMA_TRY((radix_passes<K, V, true, NoSource>(ctx, ka, va, kb, vb, n, 0, total_bits, hist.get(), &in_b, &iota, kc, vc, src, 0)));
    else RAMA_TRY((radix_passes<K, V, false, NoSource>(ctx, ka, va, kb, vb, n, 0, total_bits, hist.get(), &in_b, &iota, kc, vc, src, 0)));
    if (!in_b) {
        k.swap(again.k);
        if (v) v->swap(again.v);
    }
    again.k.reset(); again.v.reset();
    RAMA_TRY(plan.sums.alloc(ctx, plan.nb));
    return scan_totals<uint32_t>(ctx, flags(k.get()), plan);
}

// ------------------------------------------------------------------------------------------
// deterministic sum of f(0..n-1) in double: per-block partials, then one block adds them in order
// ------------------------------------------------------------------------------------------
constexpr int kSumItems = 32;

template <typename F>
__global__ __launch_bounds__(kBlock) void k_sum_partial(F f, double *partial, size_t n)
{
    size_t base = (size_t)blockIdx.x * (kBlock * kSumItems) + threadIdx.x;
    double s = 0.0;
    // eight items at a time read, then added in order (a branch per item would make each wait for its own reads)
#pragma unroll
    for (int g = 0; g < kSumItems && n > 0; g += 8) {
        double x[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            const size_t idx = base + (size_t)(g + q) * kBlock;
            x[q] = f(idx < n ? idx : n - 1);
        }
#pragma unroll
        for (int q = 0; q < 8; ++q)
            if (base + (size_t)(g + q) * kBlock < n) s += x[q];
    }
    double tot = block_sum(s);
    if (threadIdx.x == 0) partial[blockIdx.x] = tot;
}

static __global__ __launch_bounds__(kBlock) void k_sum_final(const double *partial, size_t nb, double *out, int accumulate)
{
    // thread t adds partial[t], partial[t+256], ... in order; then the fixed block tree
    double s = 0.0;
    for (size_t k = threadIdx.x; k < nb; k += kBlock) s += partial[k];
    double tot = block_sum(s);
    if (threadIdx.x == 0) *out = accumulate ? (*out + tot) : tot;
}

template <typename F>
rama_status device_sum(Ctx &ctx, F f, size_t n, double *out_dev, bool accumulate)
{
    unsigned nb = grid_for(n, kBlock * kSumItems);
    if (nb == 0) nb = 1;
    Buf<double> partial;
    RAMA_TRY(partial.alloc(ctx, nb));
    {
        ProfScope ps_(ctx, kernel_name<F>("k_sum_partial"), (double)(n * F::bytes));
        k_sum_partial<F><<<nb, kBlock, 0, ctx.stream>>>(f, partial.get(), n);
    }
    LAUNCH_TRY(ctx, "sum_partial");
    {
        ProfScope ps_(ctx, "k_sum_final", (double)(nb * 8));
        k_sum_final<<<1, kBlock, 0, ctx.stream>>>(partial.get(), nb, out_dev, accumulate ? 1 : 0);
    }
    LAUNCH_TRY(ctx, "sum_final");
    return RAMA_OK;
}

// ------------------------------------------------------------------------------------------
// small fill / iota kernels
// ------------------------------------------------------------------------------------------
template <typename T>
__global__ __launch_bounds__(kBlock) void k_fill(T *p, T v, size_t n)
{
    size_t k = (size_t)blockIdx.x * kBlock + threadIdx.x;
    if (k < n) p[k] = v;
}
// 16 bytes per thread; p must be 16-byte aligned
template <typename T>
__global__ __launch_bounds__(kBlock) void k_fill_wide(T *p, T v, size_t n)
{
    constexpr int kPer = 16 / (int)sizeof(T);
    struct alignas(16) Vec { T x[kPer]; };
    size_t k = ((size_t)blockIdx.x * kBlock + threadIdx.x) * kPer;
    if (k + kPer <= n) {
        Vec w;
#pragma unroll
        for (int q = 0; q < kPer; ++q) w.x[q] = v;
        *reinterpret_cast<Vec *>(p + k) = w;
    } else {
        for (; k < n; ++k) p[k] = v;
    }
}
// up to four arrays of 32-bit words filled by one launch (arrays that one step sets up together);
// every array is 16-byte aligned (pool blocks are) and is written 16 bytes per thread
struct FillJobs {
    uint32_t *p[4];
    uint32_t v[4];
    size_t end[4];   // running totals of the arrays' lengths in 16-byte pieces
    size_t words[4];
};
__device__ __forceinline__ void fill_piece(const FillJobs &jobs, size_t k)
{
#pragma unroll
    for (int a = 0; a < 4; ++a) {
        const size_t first = a ? jobs.end[a - 1] : 0;
        if (k >= first && k < jobs.end[a]) {
            const size_t w = (k - first) * 4;
            uint32_t *p = jobs.p[a] + w;
            const uint32_t v = jobs.v[a];
            if (w + 4 <= jobs.words[a]) *reinterpret_cast<uint4 *>(p) = make_uint4(v, v, v, v);
            else for (size_t q = w; q < jobs.words[a]; ++q) jobs.p[a][q] = v;
        }
    }
}
static __global__ __launch_bounds__(kBlock) void k_fill_multi(FillJobs jobs)
{
    fill_piece(jobs, (size_t)blockIdx.x * kBlock + threadIdx.x);
}
// tile sums of f over n items, and the arrays of a MultiFill on the way
template <typename F>
__global__ __launch_bounds__(kBlock) void k_fill_and_sum(FillJobs jobs, F f, uint32_t *sums, unsigned nb, size_t n)
{
    for (size_t k = (size_t)blockIdx.x * kBlock + threadIdx.x; k < jobs.end[3]; k += (size_t)gridDim.x * kBlock) fill_piece(jobs, k);
    if (blockIdx.x >= nb) return;      // the whole workgroup
    const size_t base = (size_t)blockIdx.x * kScanTile + threadIdx.x;
    uint32_t x[kScanItems], s = 0;
#pragma unroll
    for (int q = 0; q < kScanItems; ++q) x[q] = item_or_last<uint32_t>(f, base + (size_t)q * kBlock, n);
#pragma unroll
    for (int q = 0; q < kScanItems; ++q) s += x[q];
    s = block_sum(s);
    if (threadIdx.x == 0) sums[blockIdx.x] = s;
}
class MultiFill {
public:
    template <typename T>
    void add(T *p, uint32_t pattern, size_t count)   // `count` elements of T, every 32-bit word of which becomes `pattern`
    {
        static_assert(sizeof(T) % 4 == 0, "whole words");
        if (count == 0 || n_ >= 4) { overflow_ |= (count != 0); return; }
        jobs_.p[n_] = reinterpret_cast<uint32_t *>(p);
        jobs_.v[n_] = pattern;
        jobs_.words[n_] = count * (sizeof(T) / 4);
        total_ += (jobs_.words[n_] + 3) / 4;
        jobs_.end[n_] = total_;
        bytes_ += (double)(count * sizeof(T));
        ++n_;
    }
    rama_status run(Ctx &ctx)
    {
        if (overflow_) return fail(ctx, RAMA_ERR_INVALID_ARG, "more than four arrays in one fill");
        if (n_ == 0) return RAMA_OK;
        for (int a = n_; a < 4; ++a) { jobs_.p[a] = nullptr; jobs_.v[a] = 0; jobs_.end[a] = total_; jobs_.words[a] = 0; }
        {
            ProfScope ps_(ctx, "k_fill", bytes_);
            k_fill_multi<<<grid_for(total_), kBlock, 0, ctx.stream>>>(jobs_);
        }
        LAUNCH_TRY(ctx, "fill_multi");
        return RAMA_OK;
    }
    // the fills by the launch that adds up f tile by tile
    template <typename F>
    rama_status run_with_sums(Ctx &ctx, const F &f, uint32_t *sums, size_t n)
    {
        if (overflow_) return fail(ctx, RAMA_ERR_INVALID_ARG, "more than four arrays in one fill");
        for (int a = n_; a < 4; ++a) { jobs_.p[a] = nullptr; jobs_.v[a] = 0; jobs_.end[a] = total_; jobs_.words[a] = 0; }
        {
            ProfScope ps_(ctx, "k_fill_and_sum", bytes_ + (double)(n * F::bytes));
            const unsigned nb = grid_for(n, kScanTile), fill_groups = grid_for(total_, 4 * kBlock);
            k_fill_and_sum<F><<<nb > fill_groups ? nb : fill_groups, kBlock, 0, ctx.stream>>>(jobs_, f, sums, nb, n);
        }
        LAUNCH_TRY(ctx, "fill_and_sum");
        return RAMA_OK;
    }

private:
    FillJobs jobs_{};
    int n_ = 0;
    size_t total_ = 0;
    double bytes_ = 0.0;
    bool overflow_ = false;
};

template <typename T>
rama_status fill(Ctx &ctx, T *p, T v, size_t n)
{
    if (n == 0) return RAMA_OK;
    constexpr int kPer = 16 / (int)sizeof(T);
    const bool wide = sizeof(T) < 16 && n >= 1024 && (reinterpret_cast<uintptr_t>(p) & 15u) == 0;
    {
        ProfScope ps_(ctx, "k_fill", (double)(n * sizeof(T)));
        if (wide) k_fill_wide<T><<<grid_for((n + kPer - 1) / kPer), kBlock, 0, ctx.stream>>>(p, v, n);
        else k_fill<T><<<grid_for(n), kBlock, 0, ctx.stream>>>(p, v, n);
    }
    LAUNCH_TRY(ctx, "fill");
    return RAMA_OK;
}

template <typename K, typename P>
rama_status row_bounds(Ctx &ctx, const K *keys, size_t m, int64_t n, P *ptr)
{
    if (m >= (size_t)n / 8) {
        ProfScope ps_(ctx, "k_row_bounds_fill", (double)(m * sizeof(K) + ((size_t)n + 1) * sizeof(P)));
        k_row_bounds_fill<K, P><<<grid_for(m / 4 + 1), kBlock, 0, ctx.stream>>>(keys, m, n, ptr);
    } else {
        ProfScope ps_(ctx, "k_row_bounds_search", (double)(m * sizeof(K) + ((size_t)n + 1) * sizeof(P)));
        k_row_bounds_search<K, P><<<grid_for((size_t)n / 4 + 1), kBlock, 0, ctx.stream>>>(keys, m, n, ptr);
    }
    LAUNCH_TRY(ctx, "row_bounds");
    return RAMA_OK;
}

// Edge keys.  An undirected edge (lo,hi), lo<hi, sorts as the pair (lo, hi-lo): same order as
// (lo,hi), but the second field only needs bits(max hi-lo) bits -- on grid-like graphs that saves
// a radix pass.  key = lo << dbits | (hi-lo).
__device__ __forceinline__ uint64_t edge_key(uint32_t lo, uint32_t hi, int dbits) { return ((uint64_t)lo << dbits) | (hi - lo); }

// maximum over the workgroup folded into *out (which only ever grows, so a stale read can only
// cause a redundant atomic)
__device__ __forceinline__ void block_max_into(uint32_t v, uint32_t *out)
{
    __shared__ uint32_t wmax[4];
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v = max(v, (uint32_t)__shfl_xor((int)v, off, 64));
    if (lane_id() == 0) wmax[threadIdx.x >> 6] = v;
    __syncthreads();
    if (threadIdx.x == 0) {
        v = max(max(wmax[0], wmax[1]), max(wmax[2], wmax[3]));
        if (v > *(volatile uint32_t *)out) atomicMax(out, v);
    }
}

// Sums runs of equal keys in order of appearance (one thread per run, sequential adds) and writes run number p
// -- endpoint pair and cost -- at place p.  The tiling is that of the scan over the run heads (HeadFlag), whose
// tile offsets come in through `block_offsets`.  A workgroup keeps its 2048 values and head marks in LDS:
// the heads are found from the keys in registers (the left neighbour's key by a shuffle), and a run is
// added up from LDS instead of by a chain of dependent fetches of keys and values; only a run that
// crosses the end of the tile goes on in memory.
// `sign_sums` (optional, zero on entry): per tile of kScanTile *outputs* the number of positive costs (low half)
// and of negative costs (high half) -- the tile sums of the scan that splits the new graph by sign, which then
// needs no counting pass.  A workgroup's outputs are contiguous and at most a tile long: two atomic adds.
static __global__ __launch_bounds__(kBlock) void k_reduce_runs(size_t m, const uint64_t *key, const uint32_t *val, int dbits,
                                                        const uint32_t *block_offsets, int32_t *io, int32_t *jo, float *co,
                                                        unsigned long long *sign_sums)
{
    __shared__ float s_val[kScanTile];
    __shared__ uint8_t s_head[kScanTile];
    __shared__ uint32_t wave_tot[4];
    const int w = threadIdx.x >> 6, lane = lane_id();
    const size_t tile0 = (size_t)blockIdx.x * kScanTile;
    const int local0 = w * kScanWaveItems + lane;
    uint64_t k[kScanItems];
    uint32_t x[kScanItems], v[kScanItems];
    uint64_t before[kScanItems];      // the key in front of the wave's stretch
    uint32_t value[kScanItems];
#pragma unroll
    for (int q = 0; q < kScanItems; ++q) {
        const size_t first = tile0 + (size_t)(w * kScanWaveItems + q * 64), e = first + (size_t)lane, at = e < m ? e : m - 1;
        k[q] = key[at];
        value[q] = val[at];
        before[q] = key[first == 0 ? 0 : (first < m ? first : m) - 1];
    }
#pragma unroll
    for (int q = 0; q < kScanItems; ++q) {
        const int local = local0 + q * 64;
        const size_t e = tile0 + (size_t)local;
        uint64_t left = __shfl_up(k[q], 1, 64);
        if (lane == 0) left = before[q];
        x[q] = (e < m && (e == 0 || k[q] != left)) ? 1u : 0u;
        s_val[local] = e < m ? __uint_as_float(value[q]) : 0.0f;
        s_head[local] = (uint8_t)(e < m ? x[q] : 1u);   // what lies behind the array ends every run
    }
    uint32_t carry = 0;
#pragma unroll
    for (int q = 0; q < kScanItems; ++q) {
        const uint32_t inc = wave_inclusive_scan(x[q]);
        v[q] = inc - x[q] + carry;
        carry += wave_last(inc);
    }
    if (lane == 0) wave_tot[w] = carry;
    __syncthreads();
    const uint32_t pre0 = block_offsets[blockIdx.x];
    uint32_t pre = pre0;
#pragma unroll
    for (int j = 0; j < 3; ++j)
        if (j < w) pre += wave_tot[j];
    const uint32_t tile_a = pre0 / (uint32_t)kScanTile;
    unsigned long long sa = 0ull, sb = 0ull;   // sign counts of the outputs in tile_a and in the tile behind it
#pragma unroll
    for (int q = 0; q < kScanItems; ++q) {
        if (!x[q]) continue;
        int pos = local0 + q * 64;
        float acc = s_val[pos];
        for (++pos; pos < kScanTile && !s_head[pos]; ++pos) acc = acc + s_val[pos];
        if (pos == kScanTile)
            for (size_t f = tile0 + kScanTile; f < m && key[f] == k[q]; ++f) acc = acc + __uint_as_float(val[f]);
        const uint32_t p = v[q] + pre;
        const uint32_t lo = (uint32_t)(k[q] >> dbits);
        io[p] = (int32_t)lo;
        jo[p] = (int32_t)(lo + (uint32_t)(k[q] & ((1ull << dbits) - 1ull)));
        co[p] = acc;
        const unsigned long long sgn = acc > 0.0f ? 1ull : (acc < 0.0f ? (1ull << 32) : 0ull);
        if (p / (uint32_t)kScanTile == tile_a) sa += sgn;
        else sb += sgn;
    }
    if (sign_sums) {   // uniform
        sa = block_sum(sa);
        sb = block_sum(sb);
        if (threadIdx.x == 0) {
            if (sa) atomicAdd(&sign_sums[tile_a], sa);
            if (sb) atomicAdd(&sign_sums[tile_a + 1], sb);
        }
    }
}

// `plan`: the scan over HeadFlag{key} (scan_totals has run); uniq = its total.  `sign_sums` (optional): an array of
// ceil(uniq / kScanTile) words that gets the sign counts of the output costs per tile; if it has memory already, the words are
// there and zero.
inline rama_status reduce_runs(Ctx &ctx, const ScanPlan<uint32_t> &plan, const uint64_t *key, const uint32_t *val, int dbits,
                               int32_t *io, int32_t *jo, float *co, Buf<uint64_t> *sign_sums = nullptr)
{
    if (plan.n == 0) return RAMA_OK;
    unsigned long long *ss = nullptr;
    if (sign_sums) {
        const size_t tiles = ((size_t)plan.total + kScanTile - 1) / kScanTile;
        if (!sign_sums->get()) {
            RAMA_TRY(sign_sums->alloc(ctx, tiles > 0 ? tiles : 1));
            RAMA_TRY(fill<uint64_t>(ctx, sign_sums->get(), 0ull, tiles > 0 ? tiles : 1));
        }
        ss = (unsigned long long *)sign_sums->get();
    }
    {
        ProfScope ps_(ctx, "k_reduce_runs", (double)(plan.n * 12 + (size_t)plan.total * 12));
        k_reduce_runs<<<plan.nb, kBlock, 0, ctx.stream>>>(plan.n, key, val, dbits, plan.offs.get(), io, jo, co, ss);
    }
    LAUNCH_TRY(ctx, "reduce_runs");
    return RAMA_OK;
}

// position of the canonical edge (u,v), u<v, in rows given by rowptr over i (upper CSR) or -1
__device__ __forceinline__ int32_t find_edge_between(const int32_t *j, int32_t lo, int32_t hi, int32_t v)
{
    if (hi - lo <= 8) {
        // a short row: eight entries with two 16-byte loads (one wait instead of a chain of probes);
        // what lies behind the row's end is read but not looked at (device arrays end with slack)
        int32_t row[8];
        __builtin_memcpy(row, j + lo, sizeof(row));
        int32_t pos = -1;
#pragma unroll
        for (int k = 0; k < 8; ++k)
            if (lo + k < hi && row[k] == v) pos = lo + k;
        return pos;
    }
    const int32_t end = hi;
    while (lo < hi) {
        int32_t mid = lo + ((hi - lo) >> 1);
        if (j[mid] < v) lo = mid + 1; else hi = mid;
    }
    return (lo < end && j[lo] == v) ? lo : -1;
}
__device__ __forceinline__ int32_t find_edge_in_row(const int32_t *rowptr, const int32_t *j, int32_t u, int32_t v)
{
    return find_edge_between(j, rowptr[u], rowptr[u + 1], v);
}
// two edges of one row, v < w: one fetch of a short row, and the probes of a long one side by side
__device__ __forceinline__ void find_two_in_row(const int32_t *rowptr, const int32_t *j, int32_t u, int32_t v, int32_t w, int32_t &ev, int32_t &ew)
{
    const int32_t begin = rowptr[u], end = rowptr[u + 1];
    ev = -1; ew = -1;
    if (end - begin <= 8) {
        int32_t row[8];
        __builtin_memcpy(row, j + begin, sizeof(row));
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            if (begin + k < end && row[k] == v) ev = begin + k;
            if (begin + k < end && row[k] == w) ew = begin + k;
        }
        return;
    }
    int32_t lo = begin, hi = end, lo2 = begin, hi2 = end;
    while (lo < hi || lo2 < hi2) {      // a search that is over probes its last place again and stays
        const int32_t mid = min(lo + ((hi - lo) >> 1), end - 1), mid2 = min(lo2 + ((hi2 - lo2) >> 1), end - 1);
        const int32_t x = j[mid], y = j[mid2];
        if (lo < hi) { if (x < v) lo = mid + 1; else hi = mid; }
        if (lo2 < hi2) { if (y < w) lo2 = mid2 + 1; else hi2 = mid2; }
    }
    const int32_t x = j[min(lo, end - 1)], y = j[min(lo2, end - 1)];
    if (lo < end && x == v) ev = lo;
    if (lo2 < end && y == w) ew = lo2;
}

}  // namespace rama
