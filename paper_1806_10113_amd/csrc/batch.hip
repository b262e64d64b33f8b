// Batched exhaustive evaluation: thousands of task groups of uneven size in
// one persistent launch, replayed from a HIP graph, with an autotuned work
// decomposition.  Per group the result is the same summary as for a single
// group (best / worst / mean over every ordering) plus the ordering of the
// heuristic of Section 5.1.
//
// Work decomposition.  Group g of size n is split into n!/m(n) subtrees
// (enum_dev.h), one lane per subtree; a wave-sized tile holds
// 64 * lane_mult consecutive subtrees of one group, so the four waves of a
// block work on up to four different groups, each with its own task table in
// LDS.  Waves pull tiles from a device counter until the batch is drained (a
// persistent grid), which balances groups whose work differs by a factor of
// 10!/4! without any host-side schedule.  Per-group results are combined with
// 64-bit atomics on packed (time, rank) keys, so they do not depend on the
// order in which tiles finish.
#include <type_traits>
#include <hip/hip_runtime.h>

#include <algorithm>
#include <chrono>
#include <cstdio>
#include <string>
#include <vector>

#include "enum_kernel.h"
#include "potential_dev.h"
#include "tables_dev.h"
#include "tgo_internal.h"

namespace tgo {

constexpr int BT_THREADS = 256;
constexpr int BT_WAVES = BT_THREADS / 64;
constexpr int BT_MAX_N = 12;  // 12! < 2^29 keeps a rank in the low word of a key
constexpr int BT_MAX_M = 5;

struct BatchCfg {
    int8_t m[BT_MAX_N + 1];  // positions enumerated per lane, by group size
    int32_t lane_mult;       // subtrees per lane in one tile
    int32_t blocks;          // persistent grid size
};

// Largest group whose potential form fits the queue of the chain form: 8 bytes and,
// but for the last slot, a slack byte per slot.
constexpr int BT_POT_N = 10;
// The queues of a wave's lanes are a region of their own, slots and slack bytes in
// columns of 64: the waves of a block are on different groups, each in its group's
// form, so what one form keeps in a wave's region is nothing in the other's place.
constexpr int BT_LANES = 64;
constexpr size_t BT_WAVE_QUEUE = sizeof(Slot<uint32_t>) * BT_LANES * BT_MAX_N;
static_assert(PotRule::lane_bytes<uint32_t>(BT_POT_N) * BT_LANES <= BT_WAVE_QUEUE, "slots, then slack bytes");

struct GroupAcc {
    unsigned long long minkey;  // (T << 32) | rank, smallest
    unsigned long long maxkey;  // (T << 32) | (2^32 - 1 - rank), largest
    unsigned long long sum;     // sum of T (n <= 12 and T < 2^31: no overflow)
    unsigned long long fp;      // sum of (2 rank + 1) T mod 2^64
    int32_t status, n;
    int32_t wide;               // 1: the group runs the 64-bit path (per-tile partials)
    int32_t pad;
};

struct BatchHdr {
    unsigned int next_tile;
    unsigned int total_tiles;
    unsigned int next_wide;     // 64-bit path: tiles handed out / in total
    unsigned int total_wide;
};

// Groups whose times could reach 2^31 ns take the 64-bit path: a group of S
// subtrees is cut into W = min(S, wide_tiles) tiles of consecutive subtrees,
// one wave each, and every tile writes a partial summary of its own; the
// finalize reduces a group's partials.  No packed keys: T may need 46 bits.
constexpr int BT_WIDE_M = 3;              // positions enumerated per lane (64-bit path)
constexpr size_t BT_WIDE_BUDGET = 64u << 20;  // bytes of partials per plan
constexpr int BT_WIDE_TILES_MAX = 256;

// The wide tile offsets carry in their top bit whether the group's walk takes the
// potential form.  (The accumulators would be the natural place, but a load from the
// line that every tile's atomics go to makes them twice as slow: two groups of 12,
// 124,740 tiles, 12.1 ms where 5.3 suffice.)
constexpr uint32_t BT_POTENTIAL = 1u << 31;
static_assert(BT_WIDE_BUDGET / sizeof(Partial) < BT_POTENTIAL, "wide tiles of a plan");
__device__ __forceinline__ uint32_t wide_off(const uint32_t *__restrict__ wtile_off, int g) {
    return wtile_off[g] & ~BT_POTENTIAL;
}

__device__ __forceinline__ uint32_t subtrees_of(int n, int m) {
    return (uint32_t)(fact_c(n) / fact_c(m));
}

__device__ __forceinline__ uint32_t wide_tiles_of(int n, int wide_tiles) {
    const uint32_t S = subtrees_of(n, n < BT_WIDE_M ? n : BT_WIDE_M);
    return S < (uint32_t)wide_tiles ? S : (uint32_t)wide_tiles;
}

// Exclusive scans of v and w over a block of 1024 threads, and their totals.
__device__ __forceinline__ void block_exscan2(uint32_t v, uint32_t w, uint2 *wave_sum, uint2 *ex, uint2 *total) {
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    uint32_t a = v, b = w;
    for (int off = 1; off < 64; off <<= 1) {
        const uint32_t x = __shfl_up(a, off), y = __shfl_up(b, off);
        a += lane >= off ? x : 0u;
        b += lane >= off ? y : 0u;
    }
    if (lane == 63) wave_sum[wid] = make_uint2(a, b);
    __syncthreads();
    uint2 before = make_uint2(0, 0), all = make_uint2(0, 0);
    for (int i = 0; i < 16; ++i) {
        const uint2 t = wave_sum[i];
        before.x += i < wid ? t.x : 0u;
        before.y += i < wid ? t.y : 0u;
        all.x += t.x;
        all.y += t.y;
    }
    __syncthreads();
    *ex = make_uint2(before.x + a - v, before.y + b - w);
    *total = all;
}

// One block: per-group status and tile counts, exclusive scan into tile_off,
// accumulators reset, tile counters reset.  waves: the batch kernel's, which take
// the first `waves` tiles by their own number; the counter hands out the rest.
__global__ __launch_bounds__(1024) void batch_prepare(const tgo_task *__restrict__ tasks,
                                                      const int32_t *__restrict__ offs, int G,
                                                      Rates r, BatchCfg cfg, int wide_tiles, int max_n, GroupAcc *acc,
                                                      uint32_t *tile_off, uint32_t *wtile_off, BatchHdr *hdr,
                                                      uint32_t waves, uint32_t wide_waves) {
    __shared__ uint2 wave_sum[16];
    uint2 carry = make_uint2(0, 0);
    const uint32_t per_tile = 64u * (uint32_t)cfg.lane_mult;
    for (int base = 0; base < G; base += 1024) {
        const int g = base + threadIdx.x;
        uint32_t tiles = 0, wtiles = 0, potential = 0;
        if (g < G) {
            const int n = offs[g + 1] - offs[g];
            int st = 0, wide = 0;
            if (n < 1 || n > max_n) {
                st = TGO_EINVAL;
            } else {
                uint64_t bound;
                const int c = classify_group(tasks + offs[g], n, r, &bound);
                st = c < 0 ? c : 0;
                wide = c == 1;
                if (c == 0 && n <= BT_POT_N && pot_rates(r, n) && potential_fits<uint32_t>(bound, r))
                    potential = BT_POTENTIAL;
            }
            GroupAcc a;
            a.minkey = ~0ull;
            a.maxkey = 0;
            a.sum = 0;
            a.fp = 0;
            a.status = st;
            a.n = n;
            a.wide = wide;
            a.pad = 0;
            acc[g] = a;
            if (st == 0 && !wide) tiles = (subtrees_of(n, cfg.m[n]) + per_tile - 1) / per_tile;
            if (st == 0 && wide) wtiles = wide_tiles_of(n, wide_tiles);
        }
        uint2 ex, total;
        block_exscan2(tiles, wtiles, wave_sum, &ex, &total);
        if (g < G) {
            tile_off[g] = carry.x + ex.x;
            wtile_off[g] = (carry.y + ex.y) | potential;
        }
        carry.x += total.x;
        carry.y += total.y;
    }
    if (threadIdx.x == 0) {
        tile_off[G] = carry.x;
        wtile_off[G] = carry.y;
        hdr->next_tile = waves;
        hdr->total_tiles = carry.x;
        hdr->next_wide = wide_waves;
        hdr->total_wide = carry.y;
    }
}

// The wave's next tile after `tile` (first: its own number), wave-uniform.
// Same-address atomics are served one after another (about 15 ns each here): a
// launch of 8,192 waves that each asked once took 100 us to find a small
// batch empty.
__device__ __forceinline__ uint32_t next_tile(unsigned int *counter, uint32_t total, uint32_t waves, int lane) {
    if (total <= waves) return total;  // one tile per wave covers the batch
    uint32_t tile = 0;
    if (lane == 0) tile = atomicAdd(counter, 1u);
    return __builtin_amdgcn_readfirstlane(tile);
}

// Simulation state of a lane: the chain form with two DMA engines, windows
// without DtHs with one.
template <typename TT, int DMA>
using BatchLane = std::conditional_t<DMA == DMA_TWO, CLane<TT>, Lane<TT>>;

__device__ __forceinline__ unsigned long long wave_min(unsigned long long x) {
    for (int m = 32; m >= 1; m >>= 1) {
        const unsigned long long y = shfl_xor64(x, m);
        x = y < x ? y : x;
    }
    return x;
}
__device__ __forceinline__ unsigned long long wave_max(unsigned long long x) {
    for (int m = 32; m >= 1; m >>= 1) {
        const unsigned long long y = shfl_xor64(x, m);
        x = y > x ? y : x;
    }
    return x;
}
__device__ __forceinline__ unsigned long long wave_sum(unsigned long long x) {
    for (int m = 32; m >= 1; m >>= 1) x += shfl_xor64(x, m);
    return x;
}

struct TileKeys {
    unsigned long long min, max, sum, fp;
};

// One lane's subtree s of a group of n (m positions walked) into the tile's keys.
template <int MMAX, int DMA, typename LaneT, typename ViewT>
__device__ __forceinline__ void walk_subtree(const Ctx &c, const ViewT &v, uint32_t s, int m, TileKeys &k) {
    LaneT st;
    uint32_t lex;
    const uint32_t list = (uint32_t)prefix_by_set<DMA>(st, s, c.n, m, v, c.r, &lex);
    Sub<uint32_t> u;
    sub_init(u);
    switch (m) {
        case 1: level<uint32_t, 1, false, DMA>(c, v, st, list, 0u, u); break;
        case 2: level<uint32_t, 2, false, DMA>(c, v, st, list, 0u, u); break;
        case 3: level<uint32_t, 3, false, DMA>(c, v, st, list, 0u, u); break;
        case 4:
            if constexpr (MMAX >= 4) level<uint32_t, 4, false, DMA>(c, v, st, list, 0u, u);
            break;
        default:
            if constexpr (MMAX >= 5) level<uint32_t, 5, false, DMA>(c, v, st, list, 0u, u);
            break;
    }
    const uint64_t r0 = (uint64_t)lex * fact_c(m);
    const unsigned long long a = ((unsigned long long)u.min_t << 32) | (r0 + u.min_l);
    const unsigned long long b = ((unsigned long long)(u.max_t1 - 1u) << 32) | (0xffffffffull - (r0 + u.max_l));
    k.min = a < k.min ? a : k.min;
    k.max = b > k.max ? b : k.max;
    k.sum += u.sum;
    k.fp += 2ull * (r0 * u.sum + u.s2) + u.sum;
}

// MMAX: deepest per-lane walk compiled in (the plan's largest m); a smaller
// bound lets the compiler keep fewer level snapshots live, so more waves fit.
// Two DMA engines: at most 80 VGPRs, so 6 waves fit per SIMD (the 26 KB of
// LDS per block allows 6 per CU); the walk of 5 levels then spills registers that
// are mostly read once per tile or subtree (5 waves: the same within 0.5%).
// Subtrees in set-major order, as in the single-group kernel: the lanes of a wave
// walk the same remaining tasks.  Groups that allow it take the potential form, a
// tile at a time, so that one launch serves all.  4,096 groups of 4 to 10 tasks,
// one label per task: 13.3 ms in rank order, 10.1 in set-major order, 7.7 in the
// potential form.
template <int DMA, int MMAX>
__global__ __launch_bounds__(BT_THREADS) __attribute__((amdgpu_waves_per_eu(DMA == DMA_TWO ? 6 : 1))) void batch_kernel(const tgo_task *__restrict__ tasks,
                                                           const int32_t *__restrict__ offs, int G,
                                                           Rates r, BatchCfg cfg, GroupAcc *acc,
                                                           const uint32_t *__restrict__ tile_off,
                                                           const uint32_t *__restrict__ wtile_off, BatchHdr *hdr) {
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ Quad<uint32_t> Ht[BT_WAVES][MAXN];
    __shared__ DRec<uint32_t> Dt[BT_WAVES][MAXN];
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    unsigned char *const region = smem + BT_WAVE_QUEUE * w;
    View<uint32_t, 1, BT_LANES> v;
    v.H = Ht[w];
    v.D = Dt[w];
    v.Q = reinterpret_cast<Slot<uint32_t> *>(region) + lane;
    __shared__ PotSlot origin;
    PotView<BT_LANES> pv;
    pv.H = Ht[w];
    pv.D = Dt[w];
    pv.Q = reinterpret_cast<PotSlot *>(region) + lane;
    pv.S = region + sizeof(PotSlot) * BT_LANES * BT_POT_N + lane;
    pv.zero = &origin;
    if constexpr (DMA == DMA_TWO) {
        if (threadIdx.x == 0) origin.g = origin.e = 0;
        __syncthreads();
    }
    const uint32_t total = hdr->total_tiles, waves = gridDim.x * BT_WAVES;
    const uint32_t per_tile = 64u * (uint32_t)cfg.lane_mult;
    for (uint32_t tile = blockIdx.x * BT_WAVES + w; tile < total; tile = next_tile(&hdr->next_tile, total, waves, lane)) {
        // group of this tile: largest g with tile_off[g] <= tile
        int lo = 0, hi = G;  // tile_off[lo] <= tile < tile_off[hi]
        while (hi - lo > 1) {
            const int mid = (lo + hi) >> 1;
            if (tile_off[mid] <= tile) lo = mid; else hi = mid;
        }
        const int g = lo;
        const int base = offs[g];
        const int n = offs[g + 1] - base;
        const int m = cfg.m[n];
        const bool potential = DMA == DMA_TWO && (wtile_off[g] & BT_POTENTIAL) != 0;
        if (lane < n) {
            if (potential) PotRule::entry<uint32_t>(tasks[base + lane], r, &Ht[w][lane], &Dt[w][lane]);
            else table_entry<uint32_t>(tasks[base + lane], r, &Ht[w][lane], &Dt[w][lane]);
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        if (potential) pv.Q[(n - 1) * BT_LANES].g = POT_INF;
        const uint32_t S = subtrees_of(n, m);
        const uint32_t s0 = (tile - tile_off[g]) * per_tile;
        Ctx c;
        c.n = n;
        c.r = r;
        c.out_sub = nullptr;
        TileKeys key = {~0ull, 0, 0, 0};
        for (int k = 0; k < cfg.lane_mult; ++k) {
            const uint32_t s = s0 + (uint32_t)k * 64u + (uint32_t)lane;
            if (s < S) {
                if constexpr (DMA == DMA_TWO) {
                    if (potential) {
                        walk_subtree<MMAX, DMA, PotLane>(c, pv, s, m, key);
                        continue;
                    }
                }
                walk_subtree<MMAX, DMA, BatchLane<uint32_t, DMA>>(c, v, s, m, key);
            }
        }
        const unsigned long long kmin = wave_min(key.min), kmax = wave_max(key.max);
        const unsigned long long ksum = wave_sum(key.sum), kfp = wave_sum(key.fp);
        if (lane == 0) {
            atomicMin(&acc[g].minkey, kmin);
            atomicMax(&acc[g].maxkey, kmax);
            atomicAdd(&acc[g].sum, ksum);
            atomicAdd(&acc[g].fp, kfp);
        }
        __builtin_amdgcn_wave_barrier();
    }
}

// 64-bit path: wave-sized tiles of the groups flagged wide, each a range of
// consecutive subtrees (BT_WIDE_M positions walked per lane); every tile
// writes the Partial of its range to parts[tile].
template <int DMA>
__global__ __launch_bounds__(BT_THREADS) void batch_wide_kernel(const tgo_task *__restrict__ tasks,
                                                                const int32_t *__restrict__ offs, int G, Rates r,
                                                                int wide_tiles, const uint32_t *__restrict__ wtile_off,
                                                                BatchHdr *hdr, Partial *parts) {
    using TT = uint64_t;
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ Quad<TT> Ht[BT_WAVES][MAXN];
    __shared__ DRec<TT> Dt[BT_WAVES][MAXN];
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    View<TT, 1, BT_THREADS> v;
    v.H = Ht[w];
    v.D = Dt[w];
    v.Q = reinterpret_cast<Slot<TT> *>(smem) + threadIdx.x;
    const uint32_t total = hdr->total_wide, waves = gridDim.x * BT_WAVES;
    for (uint32_t tile = blockIdx.x * BT_WAVES + w; tile < total; tile = next_tile(&hdr->next_wide, total, waves, lane)) {
        int lo = 0, hi = G;  // wide_off(lo) <= tile < wide_off(hi)
        while (hi - lo > 1) {
            const int mid = (lo + hi) >> 1;
            if (wide_off(wtile_off, mid) <= tile) lo = mid; else hi = mid;
        }
        const int g = lo;
        const int base = offs[g];
        const int n = offs[g + 1] - base;
        const int m = n < BT_WIDE_M ? n : BT_WIDE_M;
        if (lane < n) table_entry<TT>(tasks[base + lane], r, &Ht[w][lane], &Dt[w][lane]);
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        const uint32_t S = subtrees_of(n, m);
        const uint32_t W = wide_tiles_of(n, wide_tiles);
        const uint32_t t = tile - wide_off(wtile_off, g);
        const uint32_t s0 = (uint32_t)((uint64_t)S * t / W), s1 = (uint32_t)((uint64_t)S * (t + 1) / W);
        Ctx c;
        c.n = n;
        c.r = r;
        c.out_sub = nullptr;
        Partial p;
        p.min_t = ~0ull; p.min_r = ~0ull; p.max_t = 0; p.max_r = ~0ull;
        p.sum_lo = 0; p.sum_hi = 0; p.fp = 0; p.status = 0; p.pad = 0;
        for (uint32_t sb = s0 + (uint32_t)lane; sb < s1; sb += 64u) {
            BatchLane<TT, DMA> st;
            const uint32_t list = (uint32_t)prefix<DMA>(st, sb, n, m, v, r);
            Sub<TT> u;
            sub_init(u);
            switch (m) {
                case 1: level<TT, 1, false, DMA>(c, v, st, list, 0u, u); break;
                case 2: level<TT, 2, false, DMA>(c, v, st, list, 0u, u); break;
                default: level<TT, 3, false, DMA>(c, v, st, list, 0u, u); break;
            }
            const uint64_t r0 = (uint64_t)sb * fact_c(m);
            // the lane meets its subtrees in increasing rank: strict comparisons keep the lowest rank
            if (u.min_t < p.min_t) { p.min_t = u.min_t; p.min_r = r0 + u.min_l; }
            if (u.max_t1 > p.max_t) { p.max_t = u.max_t1; p.max_r = r0 + u.max_l; }
            add128(p.sum_lo, p.sum_hi, u.sum, 0);
            p.fp += 2ull * (r0 * u.sum + u.s2) + u.sum;
        }
        for (int k = 32; k >= 1; k >>= 1) {
            const uint64_t mt = shfl_xor64(p.min_t, k), mr = shfl_xor64(p.min_r, k);
            const uint64_t xt = shfl_xor64(p.max_t, k), xr = shfl_xor64(p.max_r, k);
            const uint64_t sl = shfl_xor64(p.sum_lo, k), sh = shfl_xor64(p.sum_hi, k);
            const uint64_t f = shfl_xor64(p.fp, k);
            merge_min(p.min_t, p.min_r, mt, mr);
            merge_max(p.max_t, p.max_r, xt, xr);
            add128(p.sum_lo, p.sum_hi, sl, sh);
            p.fp += f;
        }
        if (lane == 0) parts[tile] = p;
        __builtin_amdgcn_wave_barrier();
    }
}

// One thread per group: its summary, written field by field.
__global__ __launch_bounds__(256) void batch_finalize(const GroupAcc *__restrict__ acc, int G,
                                                      const uint32_t *__restrict__ wtile_off,
                                                      const Partial *__restrict__ parts, tgo_summary *out) {
    const int g = blockIdx.x * blockDim.x + threadIdx.x;
    if (g >= G) return;
    const GroupAcc a = acc[g];
    Partial p = {};
    if (a.status == 0 && a.wide) {
        const uint32_t end = wide_off(wtile_off, g + 1);
        uint32_t i = wide_off(wtile_off, g);
        p = parts[i];
        for (++i; i < end; ++i) {
            const Partial q = parts[i];
            merge_min(p.min_t, p.min_r, q.min_t, q.min_r);
            merge_max(p.max_t, p.max_r, q.max_t, q.max_r);
            add128(p.sum_lo, p.sum_hi, q.sum_lo, q.sum_hi);
            p.fp += q.fp;
        }
    } else if (a.status == 0) {
        p.min_t = a.minkey >> 32;
        p.min_r = a.minkey & 0xffffffffull;
        p.max_t = (a.maxkey >> 32) + 1;
        p.max_r = 0xffffffffull - (a.maxkey & 0xffffffffull);
        p.sum_lo = a.sum;
        p.fp = a.fp;
    }
    const bool ok = a.status == 0;
    const uint64_t count = ok ? fact_c(a.n) : 0;
    tgo_summary *s = out + g;
    s->n = a.n;
    s->status = a.status;
    s->count = count;
    s->min_ns = ok ? (int64_t)p.min_t : 0;
    s->max_ns = ok ? (int64_t)(p.max_t - 1) : 0;
    s->argmin_rank = ok ? p.min_r : 0;
    s->argmax_rank = ok ? p.max_r : 0;
    s->sum_lo = p.sum_lo;
    s->sum_hi = p.sum_hi;
    s->fingerprint = p.fp;
    s->mean_ns = ok ? mean_of(p.sum_lo, p.sum_hi, count) : 0.0;
    put_order(s->best, ok ? unrank_nibbles(a.n, p.min_r) : 0, ok ? a.n : 0);
    put_order(s->worst, ok ? unrank_nibbles(a.n, p.max_r) : 0, ok ? a.n : 0);
    put_order(s->heur, 0, 0);
    s->heur_ns = -1;
}

// ------------------------------------------------------------------- host side

static int default_m(int n) {
    // smallest per-lane depth that still gives at least one full wave of
    // subtrees, capped at 5
    int m = 1;
    for (int c = std::min(n, 5); c >= 1; --c) {
        if (factorial(n) / factorial(c) >= 64) { m = c; break; }
    }
    return m;
}

static BatchCfg default_cfg(int cus) {
    BatchCfg c;
    for (int n = 0; n <= BT_MAX_N; ++n) c.m[n] = (int8_t)(n < 1 ? 1 : default_m(n));
    c.lane_mult = 1;
    c.blocks = cus * 8;
    return c;
}

}  // namespace tgo

struct tgo_plan {
    tgo::Rates r;
    int max_groups = 0;
    int device = 0;
    int cus = 256;
    void *ws = nullptr;
    tgo::GroupAcc *acc = nullptr;
    uint32_t *tile_off = nullptr;
    tgo::BatchHdr *hdr = nullptr;
    uint32_t *wtile_off = nullptr;
    tgo::Partial *wparts = nullptr;
    int wide_tiles = 1;
    int max_n = 12;
    size_t bytes = 0;
    tgo::BatchCfg cfg;
    bool tuned = false;
    double tuned_ms = 0.0;
    hipStream_t cap = nullptr;
    hipGraph_t graph = nullptr;
    hipGraphExec_t exec = nullptr;
    const void *k_tasks = nullptr, *k_offs = nullptr;
    void *k_out = nullptr;
    int k_groups = -1;
};

namespace tgo {

static int enqueue_batch(tgo_plan *p, const BatchCfg &cfg, const tgo_task *d_tasks,
                         const int32_t *d_offs, int G, tgo_summary *d_out, hipStream_t st) {
    const dim3 wgrid(p->cus * 2);
    hipLaunchKernelGGL(batch_prepare, dim3(1), dim3(1024), 0, st, d_tasks, d_offs, G, p->r, cfg, p->wide_tiles,
                       p->max_n, p->acc, p->tile_off, p->wtile_off, p->hdr, (uint32_t)cfg.blocks * BT_WAVES,
                       wgrid.x * BT_WAVES);
    int mmax = 1;
    for (int n = 1; n <= BT_MAX_N; ++n) mmax = std::max(mmax, (int)cfg.m[n]);
    // no kernel-completion queue with one DMA engine
    const size_t shm = p->r.one_dma ? 0 : BT_WAVE_QUEUE * BT_WAVES;
    const dim3 grid(cfg.blocks), block(BT_THREADS);
    if (p->r.one_dma) {
        if (mmax <= 3)
            hipLaunchKernelGGL((batch_kernel<DMA_ONE, 3>), grid, block, shm, st, d_tasks, d_offs, G, p->r, cfg,
                               p->acc, p->tile_off, p->wtile_off, p->hdr);
        else if (mmax == 4)
            hipLaunchKernelGGL((batch_kernel<DMA_ONE, 4>), grid, block, shm, st, d_tasks, d_offs, G, p->r, cfg,
                               p->acc, p->tile_off, p->wtile_off, p->hdr);
        else
            hipLaunchKernelGGL((batch_kernel<DMA_ONE, 5>), grid, block, shm, st, d_tasks, d_offs, G, p->r, cfg,
                               p->acc, p->tile_off, p->wtile_off, p->hdr);
    } else {
        if (mmax <= 3)
            hipLaunchKernelGGL((batch_kernel<DMA_TWO, 3>), grid, block, shm, st, d_tasks, d_offs, G, p->r, cfg,
                               p->acc, p->tile_off, p->wtile_off, p->hdr);
        else if (mmax == 4)
            hipLaunchKernelGGL((batch_kernel<DMA_TWO, 4>), grid, block, shm, st, d_tasks, d_offs, G, p->r, cfg,
                               p->acc, p->tile_off, p->wtile_off, p->hdr);
        else
            hipLaunchKernelGGL((batch_kernel<DMA_TWO, 5>), grid, block, shm, st, d_tasks, d_offs, G, p->r, cfg,
                               p->acc, p->tile_off, p->wtile_off, p->hdr);
    }
    // the 64-bit path (its blocks return at once when no group needs it)
    const size_t wshm = sizeof(Slot<uint64_t>) * BT_THREADS * BT_MAX_N;
    if (p->r.one_dma)
        hipLaunchKernelGGL(batch_wide_kernel<DMA_ONE>, wgrid, block, 0, st, d_tasks, d_offs, G, p->r, p->wide_tiles,
                           p->wtile_off, p->hdr, p->wparts);
    else
        hipLaunchKernelGGL(batch_wide_kernel<DMA_TWO>, wgrid, block, wshm, st, d_tasks, d_offs, G, p->r,
                           p->wide_tiles, p->wtile_off, p->hdr, p->wparts);
    hipLaunchKernelGGL(batch_finalize, dim3((G + 255) / 256), dim3(256), 0, st, p->acc, G, p->wtile_off, p->wparts,
                       d_out);
    int rc = launch_heuristic(p->r, d_tasks, d_offs, G, &d_out[0].heur[0], (int)sizeof(tgo_summary),
                              &d_out[0].heur_ns, (int)(sizeof(tgo_summary) / sizeof(int64_t)), st);
    if (rc) return rc;
    TGO_HIP(hipGetLastError());
    return TGO_OK;
}

size_t plan_device_bytes(const tgo_plan *p) { return p ? p->bytes : 0; }

static void drop_graph(tgo_plan *p) {
    if (p->exec) (void)hipGraphExecDestroy(p->exec);
    if (p->graph) (void)hipGraphDestroy(p->graph);
    p->exec = nullptr;
    p->graph = nullptr;
    p->k_groups = -1;
}

}  // namespace tgo

using namespace tgo;

extern "C" {

int tgo_plan_create(const tgo_model *model, int max_groups, int max_n, size_t mem_budget, tgo_plan **out) {
    if (!out) return fail(TGO_EINVAL, "out is NULL");
    *out = nullptr;
    Rates r;
    int rc = make_rates(model, &r);
    if (rc) return rc;
    if (max_groups < 1 || max_groups > (1 << 24)) return fail(TGO_EINVAL, "max_groups must be in 1..2^24");
    if (max_n < 1 || max_n > BT_MAX_N) return fail(TGO_EINVAL, "max_n must be in 1..12");
    tgo_plan *p = new (std::nothrow) tgo_plan();
    if (!p) return fail(TGO_ENOMEM, "plan");
    p->r = r;
    p->max_groups = max_groups;
    hipError_t e = hipGetDevice(&p->device);
    if (e == hipSuccess) e = hipDeviceGetAttribute(&p->cus, hipDeviceAttributeMultiprocessorCount, p->device);
    if (e != hipSuccess) {
        delete p;
        return hip_fail(e, "device query");
    }
    const size_t acc_b = (sizeof(GroupAcc) * (size_t)max_groups + 255) & ~size_t(255);
    const size_t off_b = (sizeof(uint32_t) * ((size_t)max_groups + 1) + 255) & ~size_t(255);
    // partials of the 64-bit path: up to BT_WIDE_TILES_MAX tiles per group
    // within BT_WIDE_BUDGET bytes (at least one tile per group)
    const size_t base_b = acc_b + 2 * off_b + 256;
    size_t budget = mem_budget ? mem_budget : base_b + BT_WIDE_BUDGET;
    if (budget > base_b + BT_WIDE_BUDGET) budget = base_b + BT_WIDE_BUDGET;
    if (base_b + sizeof(Partial) * (size_t)max_groups > budget) {
        delete p;
        return fail(TGO_ENOMEM, "mem_budget below the plan's minimum (" +
                                    std::to_string(base_b + sizeof(Partial) * (size_t)max_groups) + " bytes)");
    }
    size_t wt = (budget - base_b) / (sizeof(Partial) * (size_t)max_groups);
    wt = wt < 1 ? 1 : (wt > (size_t)BT_WIDE_TILES_MAX ? (size_t)BT_WIDE_TILES_MAX : wt);
    p->wide_tiles = (int)wt;
    p->max_n = max_n;
    const size_t wp_b = sizeof(Partial) * wt * (size_t)max_groups;
    p->bytes = base_b + wp_b;
    e = hipMalloc(&p->ws, base_b + wp_b);
    if (e != hipSuccess) {
        delete p;
        return fail(TGO_ENOMEM, std::string("plan workspace: ") + hipGetErrorString(e));
    }
    p->acc = (GroupAcc *)p->ws;
    p->tile_off = (uint32_t *)((char *)p->ws + acc_b);
    p->wtile_off = (uint32_t *)((char *)p->ws + acc_b + off_b);
    p->hdr = (BatchHdr *)((char *)p->ws + acc_b + 2 * off_b);
    p->wparts = (Partial *)((char *)p->ws + acc_b + 2 * off_b + 256);
    e = hipStreamCreateWithFlags(&p->cap, hipStreamNonBlocking);
    if (e != hipSuccess) {
        (void)hipFree(p->ws);
        delete p;
        return hip_fail(e, "plan stream");
    }
    p->cfg = default_cfg(p->cus);
    *out = p;
    return TGO_OK;
}

void tgo_plan_destroy(tgo_plan *p) {
    if (!p) return;
    (void)hipStreamSynchronize(p->cap);
    drop_graph(p);
    (void)hipStreamDestroy(p->cap);
    (void)hipFree(p->ws);
    delete p;
}

static int check_batch_args(tgo_plan *p, const tgo_task *d_tasks, const int32_t *d_offs, int G,
                            tgo_summary *d_out) {
    if (!p) return fail(TGO_EINVAL, "plan is NULL");
    if (G < 1 || G > p->max_groups) return fail(TGO_EINVAL, "n_groups must be in 1..max_groups");
    if (!d_tasks || !d_offs || !d_out) return fail(TGO_EINVAL, "NULL buffer");
    int dev = 0;
    TGO_HIP(hipGetDevice(&dev));
    if (dev != p->device) return fail(TGO_EINVAL, "plan belongs to another device");
    return TGO_OK;
}

int tgo_batch(tgo_plan *p, const tgo_task *d_tasks, const int32_t *d_offs, int G,
              tgo_summary *d_out, tgo_stream stream) {
    int rc = check_batch_args(p, d_tasks, d_offs, G, d_out);
    if (rc) return rc;
    if (!(p->exec && p->k_tasks == d_tasks && p->k_offs == d_offs && p->k_groups == G && p->k_out == d_out)) {
        drop_graph(p);
        TGO_HIP(hipStreamBeginCapture(p->cap, hipStreamCaptureModeThreadLocal));
        rc = enqueue_batch(p, p->cfg, d_tasks, d_offs, G, d_out, p->cap);
        hipGraph_t g = nullptr;
        hipError_t e = hipStreamEndCapture(p->cap, &g);
        if (rc) {
            if (g) (void)hipGraphDestroy(g);
            return rc;
        }
        if (e != hipSuccess) return hip_fail(e, "hipStreamEndCapture");
        p->graph = g;
        e = hipGraphInstantiate(&p->exec, g, nullptr, nullptr, 0);
        if (e != hipSuccess) {
            drop_graph(p);
            return hip_fail(e, "hipGraphInstantiate");
        }
        p->k_tasks = d_tasks;
        p->k_offs = d_offs;
        p->k_groups = G;
        p->k_out = d_out;
    }
    TGO_HIP(hipGraphLaunch(p->exec, (hipStream_t)stream));
    return TGO_OK;
}

int tgo_plan_autotune(tgo_plan *p, const tgo_task *d_tasks, const int32_t *d_offs, int G,
                      tgo_summary *d_out, tgo_stream stream) {
    int rc = check_batch_args(p, d_tasks, d_offs, G, d_out);
    if (rc) return rc;
    hipStream_t st = (hipStream_t)stream;
    hipEvent_t e0, e1;
    TGO_HIP(hipEventCreate(&e0));
    TGO_HIP(hipEventCreate(&e1));
    std::vector<BatchCfg> cands;
    for (int mbig = 4; mbig <= BT_MAX_M; ++mbig)
        for (int mult : {1, 2, 4})
            for (int bpc : {4, 6, 8}) {
                BatchCfg c = default_cfg(p->cus);
                for (int n = 1; n <= BT_MAX_N; ++n) c.m[n] = (int8_t)std::min((int)c.m[n], mbig);
                for (int n = 8; n <= BT_MAX_N; ++n) c.m[n] = (int8_t)std::min(n, mbig);
                c.lane_mult = mult;
                c.blocks = p->cus * bpc;
                cands.push_back(c);
            }
    double best = 1e30;
    BatchCfg bestc = p->cfg;
    for (const BatchCfg &c : cands) {
        rc = enqueue_batch(p, c, d_tasks, d_offs, G, d_out, st);  // warm-up
        if (rc) break;
        float tot = 0.f;
        for (int rep = 0; rep < 2; ++rep) {
            (void)hipEventRecord(e0, st);
            rc = enqueue_batch(p, c, d_tasks, d_offs, G, d_out, st);
            (void)hipEventRecord(e1, st);
            if (rc) break;
            hipError_t e = hipEventSynchronize(e1);
            if (e != hipSuccess) { rc = hip_fail(e, "autotune"); break; }
            float ms = 0.f;
            (void)hipEventElapsedTime(&ms, e0, e1);
            tot += ms;
        }
        if (rc) break;
        if (tot / 2 < best) {
            best = tot / 2;
            bestc = c;
        }
    }
    (void)hipEventDestroy(e0);
    (void)hipEventDestroy(e1);
    if (rc) return rc;
    p->cfg = bestc;
    p->tuned = true;
    p->tuned_ms = best;
    drop_graph(p);
    return TGO_OK;
}

int tgo_plan_set_decomposition(tgo_plan *p, const int32_t *m_by_n, int lane_mult, int blocks) {
    if (!p || !m_by_n) return fail(TGO_EINVAL, "NULL argument");
    if (lane_mult < 1 || lane_mult > 64) return fail(TGO_EINVAL, "lane_mult must be in 1..64");
    if (blocks < 1 || blocks > 65536) return fail(TGO_EINVAL, "blocks must be in 1..65536");
    BatchCfg c = p->cfg;
    for (int n = 1; n <= BT_MAX_N; ++n) {
        const int m = m_by_n[n - 1];
        if (m < 1 || m > std::min(n, BT_MAX_M)) return fail(TGO_EINVAL, "m_by_n[n-1] must be in 1..min(n, 5)");
        c.m[n] = (int8_t)m;
    }
    c.lane_mult = lane_mult;
    c.blocks = blocks;
    p->cfg = c;
    drop_graph(p);
    return TGO_OK;
}

int tgo_plan_describe(const tgo_plan *p, char *buf, size_t len) {
    if (!p || !buf || len == 0) return fail(TGO_EINVAL, "bad argument");
    std::string s = "{\"m_by_n\": [";
    for (int n = 1; n <= BT_MAX_N; ++n) s += std::to_string((int)p->cfg.m[n]) + (n < BT_MAX_N ? ", " : "");
    s += "], \"lane_mult\": " + std::to_string(p->cfg.lane_mult);
    s += ", \"blocks\": " + std::to_string(p->cfg.blocks);
    s += ", \"block_threads\": " + std::to_string(BT_THREADS);
    s += ", \"max_n\": " + std::to_string(p->max_n);
    s += ", \"wide_tiles\": " + std::to_string(p->wide_tiles);
    s += ", \"device_bytes\": " + std::to_string(p->bytes);
    s += ", \"tuned\": " + std::string(p->tuned ? "true" : "false");
    char tmp[64];
    std::snprintf(tmp, sizeof(tmp), "%.4f", p->tuned_ms);
    s += ", \"tuned_ms\": " + std::string(tmp) + "}";
    if (s.size() + 1 > len) return fail(TGO_ERANGE, "buffer too small");
    std::copy(s.begin(), s.end(), buf);
    buf[s.size()] = 0;
    return TGO_OK;
}

}  // extern "C"
