// The enumeration kernel shared by the single-group searches (every ordering
// of one group), its reduction and its launch.
//
// A Rule says which model the lanes simulate: the lane state and its window
// and tail functions (BaseRule: the temporal model alone; the memory limit,
// concurrent kernels and dependent tasks bring their own, rule_dev.h), how a
// subtree's prefix is placed, the tables the block keeps in LDS beside the
// tasks', and the registers the 32-bit kernel may use.
//
// Each lane walks subtrees (see enum_dev.h), striding over the grid in the
// set-major order of prefix_by_set; every merge prefers the lower rank on
// equal times, so the reduction keeps the lowest rank on ties.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdlib>
#include <type_traits>

#include "enum_dev.h"
#include "tables_dev.h"
#include "tgo_internal.h"

namespace tgo {

constexpr int EX_THREADS = 256;

// Per-lane accumulators over all ranks the lane owns.
template <typename TT>
struct Acc {
    TT min_t;        // smallest T seen
    TT max_t1;       // largest T seen, plus one (0 = none yet)
    uint64_t min_r, max_r;
    uint64_t sum_lo, sum_hi;
    uint64_t fp;
};

template <typename TT>
__device__ __forceinline__ void acc_init(Acc<TT> &a) {
    a.min_t = inf_time<TT>();
    a.max_t1 = 0;
    a.min_r = ~0ull;
    a.max_r = ~0ull;
    a.sum_lo = 0;
    a.sum_hi = 0;
    a.fp = 0;
}

// Fold a finished subtree (first rank r0) into the lane accumulators.  The
// lane meets its subtrees in set-major order, not in rank order, so ties
// between subtrees go to the lower rank explicitly (inside a subtree the
// leaves come in rank order).  fingerprint: sum of (2r+1) T with r = r0 + l
// is 2 (r0 sum T + sum l T) + sum T.
// On the 32-bit time path every T is below 2^31 and a group has at most
// 13! < 2^33 orderings, so even the sum over all of them stays below 2^64:
// the lane keeps no carry word there (two fewer live registers).
template <typename TT>
__device__ __forceinline__ void fold(Acc<TT> &a, const Sub<TT> &u, uint64_t r0) {
    const uint64_t rmin = r0 + u.min_l, rmax = r0 + u.max_l;
    if (u.min_t < a.min_t || (u.min_t == a.min_t && rmin < a.min_r)) { a.min_t = u.min_t; a.min_r = rmin; }
    if (u.max_t1 > a.max_t1 || (u.max_t1 == a.max_t1 && rmax < a.max_r)) { a.max_t1 = u.max_t1; a.max_r = rmax; }
    const uint64_t lo = a.sum_lo + u.sum;
    if constexpr (sizeof(TT) == 8) a.sum_hi += lo < a.sum_lo ? 1ull : 0ull;
    a.sum_lo = lo;
    a.fp += 2ull * (r0 * u.sum + u.s2) + u.sum;
}

// Reduce a block's lane accumulators into one Partial, returned to thread 0.
// wsum: LDS for one Partial per wave; it may alias memory the block used
// before (every thread has left its loop once the barrier below is passed).
__device__ inline Partial block_reduce(Partial p, Partial *wsum) {
    for (int m = 32; m >= 1; m >>= 1) {
        const uint64_t mt = shfl_xor64(p.min_t, m), mr = shfl_xor64(p.min_r, m);
        const uint64_t xt = shfl_xor64(p.max_t, m), xr = shfl_xor64(p.max_r, m);
        const uint64_t sl = shfl_xor64(p.sum_lo, m), sh = shfl_xor64(p.sum_hi, m);
        const uint64_t f = shfl_xor64(p.fp, m);
        merge_min(p.min_t, p.min_r, mt, mr);
        merge_max(p.max_t, p.max_r, xt, xr);
        add128(p.sum_lo, p.sum_hi, sl, sh);
        p.fp += f;
    }
    const int w = threadIdx.x / 64;
    __syncthreads();
    if ((threadIdx.x & 63) == 0) wsum[w] = p;
    __syncthreads();
    Partial o = wsum[0];
    if (threadIdx.x == 0) {
        for (int i = 1; i < (int)(blockDim.x / 64); ++i) {
            merge_min(o.min_t, o.min_r, wsum[i].min_t, wsum[i].min_r);
            merge_max(o.max_t, o.max_r, wsum[i].max_t, wsum[i].max_r);
            add128(o.sum_lo, o.sum_hi, wsum[i].sum_lo, wsum[i].sum_hi);
            o.fp += wsum[i].fp;
        }
        o.status = 0;
        o.pad = 0;
    }
    return o;
}

// Whole-group accumulators of the 32-bit time path, folded into by every
// block with 64-bit atomics.  There T < 2^31 and a rank < 13! < 2^33, so
// (T << 33) | rank orders by time and then by rank: the smallest key is the
// best ordering with the lowest rank, and with the rank complemented the
// largest key is the worst ordering with the lowest rank.  The sum over all
// orderings stays below 13! * 2^31 < 2^64; the fingerprint wraps.
// Device-scope atomics on one address are served one after another (about
// 15 ns each here), so blocks spread over EX_ACCS accumulators, a cache line
// each, and the finalize merges them.
struct alignas(128) ExAcc {
    unsigned long long minkey, maxkey, sum, fp;
};
constexpr int EX_ACCS = 64;
constexpr uint64_t EX_RANK_MASK = (1ull << 33) - 1;

// One lane per accumulator.
__device__ __forceinline__ void exacc_init(ExAcc *acc, int lane) {
    ExAcc a;
    a.minkey = ~0ull;
    a.maxkey = 0;
    a.sum = 0;
    a.fp = 0;
    acc[lane] = a;
}
static_assert(EX_ACCS == 64, "one wave initialises and merges the accumulators");

// A block's result (one lane): into an accumulator (32-bit time) or as a partial.
template <typename TT>
__device__ __forceinline__ void block_out(const Partial &o, uint32_t block, Partial *partials, ExAcc *acc) {
    if constexpr (sizeof(TT) == 4) {
        // every block owns at least one subtree, so o holds an ordering
        acc += block % EX_ACCS;
        atomicMin(&acc->minkey, (unsigned long long)((o.min_t << 33) | o.min_r));
        atomicMax(&acc->maxkey, (unsigned long long)(((o.max_t - 1) << 33) | (EX_RANK_MASK - o.max_r)));
        atomicAdd(&acc->sum, (unsigned long long)o.sum_lo);
        atomicAdd(&acc->fp, (unsigned long long)o.fp);
    } else {
        partials[block] = o;
    }
}

// ------------------------------------------------------------------ summary

// Rank -> ordering, one task per nibble.  Only the first digit of n = 13
// needs more than 32 bits of the rank (12! < 2^32 < 13!).
__device__ __forceinline__ uint64_t unrank_nibbles(int n, uint64_t rank) {
    uint64_t list = 0, o = 0;
    for (int i = n - 1; i >= 0; --i) list = (list << 4) | (uint64_t)i;
    uint64_t top = 0;
    while (n == 13 && rank >= factorial(12)) {
        rank -= factorial(12);
        ++top;
    }
    uint32_t r = (uint32_t)rank, f = 1;
    for (int i = 2; i <= n - 1 && i <= 12; ++i) f *= (uint32_t)i;
    for (int i = 0; i < n; ++i) {
        uint32_t cd;
        if (n == 13 && i == 0) {
            cd = (uint32_t)top;
        } else {
            cd = r / f;
            r -= cd * f;
        }
        if (n - 1 - i > 0) f /= (uint32_t)(n - 1 - i);
        o |= ((list >> (4 * cd)) & 15u) << (4 * i);
        const uint64_t lo = list & ((1ull << (4 * cd)) - 1ull);
        const uint64_t hi = (list >> (4 * cd + 4)) << (4 * cd);
        list = lo | hi;
    }
    return o;
}

// Nibbles lo .. lo + 7 of an ordering of n tasks as 8 bytes (0xff past n).
__device__ __forceinline__ uint64_t order_bytes(uint64_t o, int n, int lo) {
    uint64_t b = 0;
#pragma unroll
    for (int i = 0; i < 8; ++i)
        b |= (uint64_t)(lo + i < n ? (uint32_t)(o >> (4 * (lo + i))) & 15u : 0xffu) << (8 * i);
    return b;
}
__device__ __forceinline__ void put_order(uint8_t *dst, uint64_t o, int n) {
    reinterpret_cast<uint64_t *>(dst)[0] = order_bytes(o, n, 0);  // the three orderings of a
    reinterpret_cast<uint64_t *>(dst)[1] = order_bytes(o, n, 8);  // summary lie at multiples of 8
}
static_assert(offsetof(tgo_summary, best) % 8 == 0 && offsetof(tgo_summary, worst) % 8 == 0 &&
                  offsetof(tgo_summary, heur) % 8 == 0,
              "orderings are written as 8-byte words");

// sum / count: whole part exactly, then the fraction
__device__ __forceinline__ double mean_of(uint64_t sum_lo, uint64_t sum_hi, uint64_t count) {
    if (sum_hi == 0) {
        const uint64_t qt = sum_lo / count, rm = sum_lo % count;
        return (double)qt + (double)rm / (double)count;
    }
    return ((double)sum_hi * 18446744073709551616.0 + (double)sum_lo) / (double)count;
}

// The fields of *out that the enumeration fills, from its reduced result
// (thread 0 the numbers and the best ordering, thread 64 the worst).
template <typename Decode>
__device__ __forceinline__ void write_summary(const Partial &o, int status, int n, uint64_t count, Decode decode,
                                              tgo_summary *out) {
    if (threadIdx.x == 0) {
        out->n = n;
        out->status = status;
        out->count = count;
        out->min_ns = status ? 0 : (int64_t)o.min_t;
        out->max_ns = status ? 0 : (int64_t)(o.max_t - 1);
        out->argmin_rank = status ? 0 : o.min_r;
        out->argmax_rank = status ? 0 : o.max_r;
        out->sum_lo = status ? 0 : o.sum_lo;
        out->sum_hi = status ? 0 : o.sum_hi;
        out->fingerprint = status ? 0 : o.fp;
        out->mean_ns = status ? 0.0 : mean_of(o.sum_lo, o.sum_hi, count);
        put_order(out->best, status ? 0 : decode(o.min_r), status ? 0 : n);
    } else if (threadIdx.x == 64) {
        put_order(out->worst, status ? 0 : decode(o.max_r), status ? 0 : n);
    }
}

// -------------------------------------------------------------- enumeration

// Dynamic LDS of the enumeration kernel: the task tables (n entries each),
// the rule's own tables, then the per-lane queue, n - 1 slots (the last
// position's slot is never read; none when the lanes need no queue).  The
// block reduction reuses the queue's memory at the end.
template <class Rule, typename TT>
__host__ __device__ constexpr size_t enum_tables_bytes(int n) {
    return ((size_t)n * (sizeof(Quad<TT>) + sizeof(DRec<TT>)) + Rule::lds_bytes(n) + 15) & ~size_t(15);
}
// The queue's slots and the reduction's partials lie at their alignment for every n.
template <class Rule, typename TT>
constexpr bool enum_queue_aligned() {
    for (int n = 1; n <= MAXN; ++n)
        if (enum_tables_bytes<Rule, TT>(n) % alignof(Slot<TT>) || enum_tables_bytes<Rule, TT>(n) % alignof(Partial))
            return false;
    return true;
}
template <class Rule, typename TT>
inline size_t enum_shm_bytes(int n, bool one_dma) {
    static_assert(enum_queue_aligned<Rule, TT>(), "queue alignment");
    const size_t q = Rule::queue(one_dma) ? EX_THREADS * Rule::template lane_bytes<TT>(n) : 0;
    const size_t red = sizeof(Partial) * (EX_THREADS / 64);
    return enum_tables_bytes<Rule, TT>(n) + (q > red ? q : red);
}

// Ranks of one group's orderings: subtrees in set-major order for the large
// groups, lexicographic order for the small ones.
struct GroupRule {
    // Mode word for which a kernel of this width runs.
    template <typename TT>
    static constexpr int mode() { return sizeof(TT) == 4 ? 0 : 1; }
    // Queue of one lane, and the view's pointers into the block's.
    template <typename TT>
    static __host__ __device__ constexpr size_t lane_bytes(int n) {
        return sizeof(Slot<TT>) * (size_t)(n > 1 ? n - 1 : 1);
    }
    template <typename TT, typename ViewT>
    static __device__ __forceinline__ void bind(ViewT &v, unsigned char *queue, int) {
        v.Q = reinterpret_cast<Slot<TT> *>(queue) + threadIdx.x;
    }
    template <typename TT>
    static __device__ __forceinline__ void entry(const tgo_task &t, const Rates &r, Quad<TT> *H, DRec<TT> *D) {
        table_entry<TT>(t, r, H, D);
    }
    template <int DMA, typename LaneT, typename ViewT, typename ArgsT>
    static __device__ __forceinline__ uint64_t prefix(LaneT &st, uint32_t s, int n, int m, ViewT &v, const Rates &r,
                                                      const ArgsT &, uint32_t *lex) {
        return prefix_by_set<DMA>(st, s, n, m, v, r, lex);
    }
    template <int DMA, typename LaneT, typename ViewT, typename ArgsT>
    static __device__ __forceinline__ uint64_t small_prefix(LaneT &st, uint32_t rank, int n, ViewT &v, const Rates &r,
                                                            const ArgsT &) {
        return tgo::prefix<DMA>(st, rank, n, 1, v, r);
    }
    template <typename ArgsT>
    static __device__ __forceinline__ uint64_t decode(uint64_t rank, int n, const ArgsT &) {
        return unrank_nibbles(n, rank);
    }
    // Other outputs of a group in error.
    template <typename ArgsT>
    static __device__ __forceinline__ void on_error(const ArgsT &) {}
    // Time path or error code of the group, by one wave (lane i: task i).
    template <typename ArgsT>
    static __device__ __forceinline__ int status(const tgo_task *tasks, int n, const Rates &r, const ArgsT &,
                                                 int lane) {
        return classify_group_wave(tasks, n, r, lane);
    }
};

// The temporal model alone.  32-bit time path: at most 72 VGPRs so that 7
// waves fit per SIMD (with the n - 1 slot queue, 7 blocks also fit in LDS at
// n = 12).
struct BaseRule : GroupRule {
    struct Args {};
    static constexpr bool SIDE = false;
    template <typename TT>
    using View = tgo::View<TT, 1, EX_THREADS>;
    // two DMA engines: the chain form; one engine: windows without DtH events
    template <typename TT, int DMA>
    using Lane = std::conditional_t<DMA == DMA_TWO, CLane<TT>, tgo::Lane<TT>>;
    template <typename TT, int DMA>
    static constexpr int min_waves() { return sizeof(TT) == 4 ? 7 : 1; }
    static constexpr bool queue(bool one_dma) { return !one_dma; }
    static __host__ __device__ constexpr size_t lds_bytes(int) { return 0; }
    // SMALL: the rule's tables straight from the call's inputs (small_kernel)
    template <bool SMALL, typename ViewT>
    static __device__ __forceinline__ void load(ViewT &, unsigned char *, const Args &, int, uint64_t *) {}
};

// Every ordering of one group.  modep: the group's time path, decided by the
// launch before (0 = 32-bit, 1 = 64-bit, or a negative error code); both
// widths are launched, and every block of the one that does not match the
// group's path (or of both, on an error) returns after reading one word.  DMA
// is the launch scheme (DMA_TWO or DMA_ONE, fixed per instantiation).
template <class Rule, typename TT, int M, bool STORE, int DMA>
__global__ __launch_bounds__(EX_THREADS) __attribute__((amdgpu_waves_per_eu(Rule::template min_waves<TT, DMA>())))
void enum_kernel(const tgo_task *__restrict__ tasks, int n, Rates r, typename Rule::Args args, uint32_t n_sub,
                 int64_t *out, Partial *partials, ExAcc *acc, const int *__restrict__ modep) {
    extern __shared__ __align__(16) unsigned char smem[];
    if (*modep != Rule::template mode<TT>()) return;
    Quad<TT> *Ht = reinterpret_cast<Quad<TT> *>(smem);
    DRec<TT> *Dt = reinterpret_cast<DRec<TT> *>(smem + (size_t)n * sizeof(Quad<TT>));
    unsigned char *qbase = smem + enum_tables_bytes<Rule, TT>(n);
    if ((int)threadIdx.x < n)
        Rule::template entry<TT>(tasks[threadIdx.x], r, &Ht[threadIdx.x], &Dt[threadIdx.x]);

    typename Rule::template View<TT> v;
    v.H = Ht;
    v.D = Dt;
    Rule::template bind<TT>(v, qbase, n);
    uint64_t seq = 0;  // task at each placed position, one per nibble (rules that ask for it)
    Rule::template load<false>(v, smem + (size_t)n * (sizeof(Quad<TT>) + sizeof(DRec<TT>)), args, n, &seq);
    __syncthreads();
    // the rule's heuristic runs on one wave of block 0, beside the enumeration
    // (its latency is that of a small group's whole enumeration)
    if constexpr (Rule::SIDE) {
        if (blockIdx.x == 0) {
            if (threadIdx.x < 64) Rule::template side<TT, DMA>(v, n, r, args);
            return;
        }
    }
    const uint32_t blocks = gridDim.x - (Rule::SIDE ? 1u : 0u), block = blockIdx.x - (Rule::SIDE ? 1u : 0u);
    Ctx c;
    c.n = n;
    c.r = r;
    c.out_sub = nullptr;

    Acc<TT> a;
    acc_init(a);
    const uint32_t stride = blocks * blockDim.x;
    using LaneT = typename Rule::template Lane<TT, DMA>;
    for (uint32_t s = block * blockDim.x + threadIdx.x; s < n_sub; s += stride) {
        LaneT st;
        uint32_t lex;
        const uint64_t list = Rule::template prefix<DMA>(st, s, n, M, v, r, args, &lex);
        const uint64_t r0 = (uint64_t)lex * factorial(M);
        if constexpr (STORE) c.out_sub = out + r0;
        Sub<TT> u;
        sub_init(u);
        level<TT, M, STORE, DMA>(c, v, st, (uint32_t)list, 0u, u);
        fold(a, u, r0);
    }
    Partial p;
    p.min_t = (uint64_t)a.min_t;
    p.min_r = a.min_r;
    if constexpr (sizeof(TT) == 4) {
        p.min_t = a.min_t == inf_time<TT>() ? ~0ull : (uint64_t)a.min_t;
    }
    p.max_t = (uint64_t)a.max_t1;
    p.max_r = a.max_r;
    p.sum_lo = a.sum_lo;
    p.sum_hi = a.sum_hi;
    p.fp = a.fp;
    p.status = 0;
    p.pad = 0;
    const Partial o = block_reduce(p, reinterpret_cast<Partial *>(qbase));
    if (threadIdx.x == 0) block_out<TT>(o, block, partials, acc);
}

constexpr int EX_FIN_THREADS = 1024;

// One block: the group's result from the accumulators (32-bit path) or from the
// block partials (64-bit path).  decode(rank) gives an ordering, one task per
// nibble.
template <typename Decode>
__device__ __forceinline__ void finalize_block(const Partial *__restrict__ parts, int nparts, int n, uint64_t count,
                                               const ExAcc *__restrict__ acc, int mode, Decode decode,
                                               tgo_summary *out) {
    __shared__ Partial red[EX_FIN_THREADS / 64];
    Partial p;
    p.min_t = ~0ull; p.min_r = ~0ull; p.max_t = 0; p.max_r = ~0ull;
    p.sum_lo = 0; p.sum_hi = 0; p.fp = 0; p.status = 0; p.pad = 0;
    if (mode == 1) {
        auto take = [&p](const Partial &q) {
            merge_min(p.min_t, p.min_r, q.min_t, q.min_r);
            merge_max(p.max_t, p.max_r, q.max_t, q.max_r);
            add128(p.sum_lo, p.sum_hi, q.sum_lo, q.sum_hi);
            p.fp += q.fp;
        };
        // four partials in flight per thread: the loads, not the merges, set the time
        const int b = (int)blockDim.x;
        int i = (int)threadIdx.x;
        for (; i + 3 * b < nparts; i += 4 * b) {
            const Partial q0 = parts[i], q1 = parts[i + b], q2 = parts[i + 2 * b], q3 = parts[i + 3 * b];
            take(q0);
            take(q1);
            take(q2);
            take(q3);
        }
        for (; i < nparts; i += b) take(parts[i]);
        p = block_reduce(p, red);
        if (threadIdx.x == 0) red[0] = p;
        __syncthreads();
        p = red[0];
    } else if (mode >= 0) {
        // every wave merges the accumulators (waves 0 and 1 use the result)
        if (threadIdx.x >= 128) return;
        const ExAcc mine = acc[threadIdx.x & 63];
        uint64_t mn = mine.minkey, mx = mine.maxkey, sum = mine.sum, fp = mine.fp;
        for (int m = 32; m >= 1; m >>= 1) {
            const uint64_t a = shfl_xor64(mn, m), b = shfl_xor64(mx, m);
            mn = a < mn ? a : mn;
            mx = b > mx ? b : mx;
            sum += shfl_xor64(sum, m);
            fp += shfl_xor64(fp, m);
        }
        p.min_t = mn >> 33;
        p.min_r = mn & EX_RANK_MASK;
        p.max_t = (mx >> 33) + 1;
        p.max_r = EX_RANK_MASK - (mx & EX_RANK_MASK);
        p.sum_lo = sum;
        p.sum_hi = 0;
        p.fp = fp;
    }
    write_summary(p, mode < 0 ? mode : 0, n, count, decode, out);
}
__device__ __forceinline__ void finalize_block(const Partial *__restrict__ parts, int nparts, int n, uint64_t count,
                                               const ExAcc *__restrict__ acc, int mode, tgo_summary *out) {
    finalize_block(parts, nparts, n, count, acc, mode, [n](uint64_t rk) { return unrank_nibbles(n, rk); }, out);
}

// The summary's heuristic ordering and its total time (one lane writes).
__device__ __forceinline__ void put_heuristic(tgo_summary *out, uint64_t ord, int n, int64_t T) {
    if (threadIdx.x == 0) {
        put_order(out->heur, ord, n);
        out->heur_ns = T;
    }
}

// The finalize of a search under a rule; the heuristic's fields are the side
// block's unless the group is in error.
static __global__ __launch_bounds__(EX_FIN_THREADS) void rule_finalize(const Partial *__restrict__ parts, int nparts,
                                                                       int n, uint64_t count,
                                                                       const ExAcc *__restrict__ acc,
                                                                       const int *__restrict__ modep,
                                                                       tgo_summary *out) {
    const int mode = *modep;
    if (mode < 0) put_heuristic(out, 0, 0, mode);
    finalize_block(parts, nparts, n, count, acc, mode, out);
}

// -------------------------------------------------------------- small groups

// Up to SMALL_COUNT orderings: one lane per ordering, every window of it in a
// short loop, both time widths in one kernel.  Such a call is launches, cold
// instruction fetch and latency, not work: the general path's three launches
// before the finalize (time path, enumeration, its idle twin) and its unrolled
// walk took 25 of a four-task group's 27 us here.  One block (at most
// SMALL_ONE orderings) also writes the summary; several leave partials.
constexpr int SMALL_THREADS = EX_THREADS;  // the views' queue stride
constexpr uint32_t SMALL_ONE = 1024;
constexpr uint32_t SMALL_COUNT = 65536;

struct SmallOut {
    int64_t *times;  // T by rank, or null
    Partial *parts;
    tgo_summary *summary;
};

// The heuristic's fields when no side block writes them.
template <class Rule>
__device__ __forceinline__ void no_heuristic(int status, const typename Rule::Args &args, tgo_summary *out) {
    if (threadIdx.x == 128 && (!Rule::SIDE || status != 0)) {
        put_order(out->heur, 0, 0);
        out->heur_ns = Rule::SIDE ? status : -1;
        if (status != 0) Rule::on_error(args);
    }
}

__device__ __forceinline__ uint64_t wave_min_u64(uint64_t x) {
    for (int m = 32; m >= 1; m >>= 1) {
        const uint64_t y = shfl_xor64(x, m);
        x = y < x ? y : x;
    }
    return x;
}

template <class Rule, typename TT, int DMA>
__device__ __forceinline__ void small_run(const tgo_task *__restrict__ tasks, int n, const Rates &r,
                                          const typename Rule::Args &args, uint32_t count, int nblocks, bool side,
                                          unsigned char *smem, const SmallOut &o) {
    Quad<TT> *Ht = reinterpret_cast<Quad<TT> *>(smem);
    DRec<TT> *Dt = reinterpret_cast<DRec<TT> *>(smem + (size_t)n * sizeof(Quad<TT>));
    unsigned char *qbase = smem + enum_tables_bytes<Rule, TT>(n);
    if ((int)threadIdx.x < n) table_entry<TT>(tasks[threadIdx.x], r, &Ht[threadIdx.x], &Dt[threadIdx.x]);
    typename Rule::template View<TT> v;
    v.H = Ht;
    v.D = Dt;
    v.Q = reinterpret_cast<Slot<TT> *>(qbase) + threadIdx.x;
    uint64_t seq = 0;
    Rule::template load<true>(v, smem + (size_t)n * (sizeof(Quad<TT>) + sizeof(DRec<TT>)), args, n, &seq);
    __syncthreads();
    if constexpr (Rule::SIDE) {
        if (side) {
            if (threadIdx.x < 64) Rule::template side<TT, DMA>(v, n, r, args);
            return;
        }
    }
    using LaneT = typename Rule::template Lane<TT, DMA>;
    Partial p;
    p.min_t = ~0ull; p.min_r = ~0ull; p.max_t = 0; p.max_r = ~0ull;
    p.sum_lo = 0; p.sum_hi = 0; p.fp = 0; p.status = 0; p.pad = 0;
    // a lane meets its ranks in increasing order
#pragma unroll 1
    for (uint32_t rk = blockIdx.x * SMALL_THREADS + threadIdx.x; rk < count; rk += (uint32_t)nblocks * SMALL_THREADS) {
        LaneT st;
        const uint32_t x = (uint32_t)Rule::template small_prefix<DMA>(st, rk, n, v, r, args);
        window<DMA, false>(st, n - 1, x, v, r);
        const uint64_t T = (uint64_t)tail<DMA>(st, r);
        if (o.times) o.times[rk] = (int64_t)T;
        if (T < p.min_t) { p.min_t = T; p.min_r = rk; }
        if (T + 1 > p.max_t) { p.max_t = T + 1; p.max_r = rk; }
        p.sum_lo += (uint32_t)T;  // halves of the sum: 2^16 terms below 2^32 each
        p.sum_hi += T >> 32;
        p.fp += (2ull * rk + 1ull) * T;
    }
    // wave: the extreme time, then the lowest rank that has it
    const uint64_t mn = wave_min_u64(p.min_t), mx = ~wave_min_u64(~p.max_t);
    const uint64_t mr = wave_min_u64(p.min_t == mn ? p.min_r : ~0ull);
    const uint64_t xr = wave_min_u64(p.max_t == mx ? p.max_r : ~0ull);
    for (int m = 32; m >= 1; m >>= 1) {
        p.sum_lo += shfl_xor64(p.sum_lo, m);
        p.sum_hi += shfl_xor64(p.sum_hi, m);
        p.fp += shfl_xor64(p.fp, m);
    }
    p.min_t = mn; p.min_r = mr; p.max_t = mx; p.max_r = xr;
    // whole sum = sum_hi 2^32 + sum_lo
    const uint64_t lo = p.sum_lo + (p.sum_hi << 32);
    p.sum_hi = (p.sum_hi >> 32) + (lo < p.sum_lo ? 1ull : 0ull);
    p.sum_lo = lo;
    __syncthreads();  // the queue's memory is free
    Partial *wsum = reinterpret_cast<Partial *>(qbase);
    if ((threadIdx.x & 63) == 0) wsum[threadIdx.x / 64] = p;
    __syncthreads();
    if ((threadIdx.x & 63) != 0 || threadIdx.x > 64) return;
    Partial t = wsum[0];
#pragma unroll 1
    for (int i = 1; i < SMALL_THREADS / 64; ++i) {
        merge_min(t.min_t, t.min_r, wsum[i].min_t, wsum[i].min_r);
        merge_max(t.max_t, t.max_r, wsum[i].max_t, wsum[i].max_r);
        add128(t.sum_lo, t.sum_hi, wsum[i].sum_lo, wsum[i].sum_hi);
        t.fp += wsum[i].fp;
    }
    if (nblocks > 1) {
        if (threadIdx.x == 0) o.parts[blockIdx.x] = t;
        return;
    }
    write_summary(t, 0, n, count, [&](uint64_t rk) { return Rule::decode(rk, n, args); }, o.summary);
}

template <class Rule, int DMA>
__global__ __launch_bounds__(SMALL_THREADS) void small_kernel(const tgo_task *__restrict__ tasks, int n, Rates r,
                                                              typename Rule::Args args, uint32_t count, int nblocks,
                                                              SmallOut o) {
    extern __shared__ __align__(16) unsigned char smem[];
    const int cls = __builtin_amdgcn_readfirstlane(Rule::status(tasks, n, r, args, threadIdx.x & 63));
    const bool side = (int)blockIdx.x == nblocks;
    if (cls >= 0) {
        if (!side && nblocks == 1) no_heuristic<Rule>(0, args, o.summary);
        if (cls == 0) small_run<Rule, uint32_t, DMA>(tasks, n, r, args, count, nblocks, side, smem, o);
        else small_run<Rule, uint64_t, DMA>(tasks, n, r, args, count, nblocks, side, smem, o);
        return;
    }
    if (side) return;
    Partial p = {};
    p.status = cls;
    if (nblocks > 1) {
        if (threadIdx.x == 0) o.parts[blockIdx.x] = p;
        return;
    }
    no_heuristic<Rule>(cls, args, o.summary);
    write_summary(p, cls, n, count, [](uint64_t) { return 0ull; }, o.summary);
}

template <class Rule>
__global__ __launch_bounds__(SMALL_THREADS) void small_finalize(const Partial *__restrict__ parts, int nparts, int n,
                                                                uint32_t count, typename Rule::Args args,
                                                                tgo_summary *out) {
    __shared__ Partial red[SMALL_THREADS / 64];
    const int status = parts[0].status;
    Partial p;
    p.min_t = ~0ull; p.min_r = ~0ull; p.max_t = 0; p.max_r = ~0ull;
    p.sum_lo = 0; p.sum_hi = 0; p.fp = 0; p.status = 0; p.pad = 0;
    static_assert(SMALL_COUNT <= SMALL_THREADS * SMALL_THREADS, "one partial per thread");
    if ((int)threadIdx.x < nparts) p = parts[threadIdx.x];
    p = block_reduce(p, red);
    if (threadIdx.x == 0) red[0] = p;
    __syncthreads();
    no_heuristic<Rule>(status, args, out);
    write_summary(red[0], status, n, count, [&](uint64_t rk) { return Rule::decode(rk, n, args); }, out);
}

// ------------------------------------------------------------------- launch

// Blocks per launch, in units of the blocks the 32-bit kernel keeps resident
// at once.  A subtree's cost varies with its DtH events, so blocks finish at
// different times: one resident round leaves SIMDs idle at the end, many
// short blocks let the dispatcher fill them.  Measured at N = 12 on MI355X
// with 6 waves per SIMD (1,536 resident blocks) and block partials: 8 rounds
// gave 3.06-3.11 ms per launch against 3.82 ms for one round and 3.30 ms for
// 20 subtrees per lane.  With 7 waves (1,792 resident blocks) and the
// accumulator atomics: 6 / 8 / 10 / 12 / 14 / 16 / 20 rounds took 2.85-2.87 /
// 2.80 / 2.81-2.82 / 2.78-2.80 / 2.80-2.82 / 2.77-2.78 / 2.83 ms, and grids
// that are not a multiple of the resident count were slower; 12 rounds,
// 21,504 blocks.
constexpr uint32_t EX_ROUNDS = 12;

// Scratch of one call: caller-provided (ptr, bytes), or the library's
// per-(device, stream) workspace when ptr is NULL.
struct ExScratch {
    void *ptr = nullptr;
    size_t bytes = 0;
};

// Device scratch of an enumeration: block partials (64-bit path), the 32-bit
// path's accumulators, the group's time path, then `extra` bytes of the rule.
struct EnumScratch {
    Partial *parts;
    ExAcc *acc;
    int *mode;
    unsigned char *extra;
};
constexpr size_t ENUM_FIXED = sizeof(ExAcc) * EX_ACCS + 256;  // accumulators and time path

// Blocks of an enumeration of n_sub subtrees and the scratch it needs.  The
// grid is sized from the 32-bit kernel (the fast path), capped at one subtree
// per lane; TGO_EXHAUSTIVE_BLOCKS overrides it for tuning experiments.  A
// fixed scratch bounds the grid instead (any grid gives the same result:
// lanes stride over the subtrees).
inline int enum_grid(const void *k32, size_t shm32, uint32_t n_sub, size_t extra, ExScratch ws, hipStream_t st,
                     uint32_t *blocks_out, EnumScratch *sc) {
    const uint64_t want = ((uint64_t)n_sub + EX_THREADS - 1) / EX_THREADS;
    uint32_t blocks = resident_blocks(k32, EX_THREADS, shm32);
    blocks = blocks == 0 ? 8192u : blocks * EX_ROUNDS;
    if (const char *e = std::getenv("TGO_EXHAUSTIVE_BLOCKS")) {
        const long v = std::atol(e);
        if (v >= 1 && v <= (1l << 20)) blocks = (uint32_t)v;
    }
    if ((uint64_t)blocks > want) blocks = (uint32_t)want;
    const size_t fixed = ENUM_FIXED + ((extra + 255) & ~size_t(255));
    unsigned char *base = nullptr;
    if (ws.ptr) {
        if (ws.bytes < fixed + sizeof(Partial)) return fail(TGO_ENOMEM, "scratch too small for one block");
        const size_t fit = (ws.bytes - fixed) / sizeof(Partial);
        if ((size_t)blocks > fit) blocks = (uint32_t)fit;
        base = reinterpret_cast<unsigned char *>(ws.ptr);
    } else {
        int rc = workspace(fixed + sizeof(Partial) * blocks, (void **)&base, st);
        if (rc) return rc;
    }
    sc->acc = reinterpret_cast<ExAcc *>(base);
    sc->mode = reinterpret_cast<int *>(base + sizeof(ExAcc) * EX_ACCS);
    sc->extra = base + ENUM_FIXED;
    sc->parts = reinterpret_cast<Partial *>(base + fixed);
    *blocks_out = blocks;
    return TGO_OK;
}

// Launch one instantiation.
template <class Rule, typename TT, int M, bool STORE, int DMA>
inline void enum_launch_one(hipStream_t st, const tgo_task *t, int n, const Rates &r, const typename Rule::Args &args,
                            uint32_t n_sub, int64_t *out, uint32_t blocks, const EnumScratch &sc) {
    hipLaunchKernelGGL((enum_kernel<Rule, TT, M, STORE, DMA>), dim3(blocks + (Rule::SIDE ? 1u : 0u)), dim3(EX_THREADS),
                       (enum_shm_bytes<Rule, TT>(n, DMA == DMA_ONE)), st, t, n, r, args, n_sub, out, sc.parts, sc.acc,
                       sc.mode);
}

// Launch the 32-bit and 64-bit instantiations (the one that does not match
// the group's time path returns at once).
template <class Rule, int M, bool STORE, int DMA>
inline int enum_launch(hipStream_t st, const tgo_task *t, int n, const Rates &r, const typename Rule::Args &args,
                       uint32_t n_sub, int64_t *out, uint32_t blocks, const EnumScratch &sc) {
    enum_launch_one<Rule, uint32_t, M, STORE, DMA>(st, t, n, r, args, n_sub, out, blocks, sc);
    enum_launch_one<Rule, uint64_t, M, STORE, DMA>(st, t, n, r, args, n_sub, out, blocks, sc);
    TGO_HIP(hipGetLastError());
    return TGO_OK;
}

// A small search (count <= SMALL_COUNT) in one launch, or two.
template <class Rule, int DMA>
inline int small_launch(hipStream_t st, const tgo_task *t, int n, const Rates &r, const typename Rule::Args &args,
                        uint32_t count, int64_t *out, tgo_summary *d_out, ExScratch ws) {
    SmallOut o;
    o.times = out;
    o.summary = d_out;
    o.parts = nullptr;
    const int nblocks = count <= SMALL_ONE ? 1 : (int)((count + SMALL_THREADS - 1) / SMALL_THREADS);
    if (nblocks > 1) {
        const size_t need = sizeof(Partial) * nblocks;
        if (!ws.ptr) {
            int rc = workspace(need, &ws.ptr, st);
            if (rc) return rc;
        } else if (ws.bytes < need) {
            return fail(TGO_ENOMEM, "scratch too small for a small group");
        }
        o.parts = reinterpret_cast<Partial *>(ws.ptr);
    }
    const dim3 grid((uint32_t)nblocks + (Rule::SIDE ? 1u : 0u));
    hipLaunchKernelGGL((small_kernel<Rule, DMA>), grid, dim3(SMALL_THREADS),
                       (enum_shm_bytes<Rule, uint64_t>(n, DMA == DMA_ONE)), st, t, n, r, args, count, nblocks, o);
    TGO_HIP(hipGetLastError());
    if (nblocks > 1) {
        hipLaunchKernelGGL(small_finalize<Rule>, dim3(1), dim3(SMALL_THREADS), 0, st, o.parts, nblocks, n, count, args,
                           d_out);
        TGO_HIP(hipGetLastError());
    }
    return TGO_OK;
}

// Depth of the walk under a rule: the deepest of 1 .. top that leaves 32,768
// subtrees, one lane each (half a wave per SIMD; fewer would leave SIMDs idle).
inline int rule_depth(int n, int top) {
    for (int m = top; m > 1; --m)
        if (m <= n && factorial(n) / factorial(m) >= 32768) return m;
    return 1;
}

}  // namespace tgo
