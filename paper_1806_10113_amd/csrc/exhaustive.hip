// Exhaustive evaluation of every launch ordering of one task group.
//
// Brute force over all n! orderings (the search that Section 1 and
// Section 5.1 rule out at runtime on a CPU), reduced to the best, worst and
// average ordering (the quantities plotted in Section 6).
// The kernel and its reduction are in enum_kernel.h.
#include <hip/hip_runtime.h>

#include <cstdlib>
#include <mutex>

#include "enum_kernel.h"
#include "one_dev.h"
#include "potential_dev.h"

namespace tgo {

// Whether a group that fits the potential form also gains by it (32-bit time, one
// wave, lane i: task i).  The chain form's cost is the DtHs that end before the
// last HtD.  From 12 tasks on (five waves of the potential form per SIMD, seven of
// the chain form) it is the faster one where the DtHs (at the overlapped rate) take
// longer together than the HtDs and the kernels, which precede them.  960 groups of
// 12 timed in both forms (eight pairs of rates, durations of three spreads): the
// line at 1.0 to 1.07 gives the least mean, 0.8995 of the chain form's time.  384
// groups of 12, D / (H + K) and the time without the potential form over that with
// it, mean and least: up to 0.4 1.28 (1.00), 0.6 1.16 (0.95), 0.8 1.09 (0.96), 0.85
// 1.04 (0.94), 0.9 1.03 (1.00), 0.95 1.01 (1.00), 1.0 1.02 (0.91); above (chain
// form) 1.00 (1.00).  So 9 of 384 lose, 8 of them more than 2%: the chain
// form's time also follows how often the lanes of a wave part, which no sum over the
// tasks that was tried shows.  D <= 1.24 H as well would leave 3 of 960 that lose
// more than 2%, for a mean of 0.908.
// Groups of 11, always on: 1.08 and more on average in each of those ranges, least
// 0.99; of 13: 1.08 to 1.29, least 0.995.
__device__ __forceinline__ bool potential_gains(const tgo_task *__restrict__ tasks, int n, const Rates &r, int lane) {
    if (n < 12) return true;
    uint32_t lead = 0, d = 0;
    if (lane < n) {
        Quad<uint32_t> H;
        DRec<uint32_t> D;
        table_entry<uint32_t>(tasks[lane], r, &H, &D);
        lead = H.hp + H.k;
        d = D.dp;
    }
    for (int m = 8; m >= 1; m >>= 1) {  // lanes 0 to 15 hold the tasks; both sums are below 2^31
        lead += __shfl_xor(lead, m);
        d += __shfl_xor(d, m);
    }
    return d <= lead;
}

// The group's time path, decided once before the enumeration: 0 = 32-bit,
// 1 = 64-bit, 2 = 32-bit in the potential form (if `potential`, and the group's
// potentials fit), or a negative error code (classify_group).
__global__ __launch_bounds__(64) void exhaustive_classify(const tgo_task *__restrict__ tasks, int n, Rates r,
                                                          bool potential, int *mode, ExAcc *acc) {
    uint64_t bound;
    int m = classify_group_wave(tasks, n, r, threadIdx.x, &bound);
    if (potential && m == 0 && potential_fits<uint32_t>(bound, r) && potential_gains(tasks, n, r, threadIdx.x)) m = 2;
    if (threadIdx.x == 0) *mode = m;
    exacc_init(acc, threadIdx.x);
}

__global__ __launch_bounds__(EX_FIN_THREADS) void exhaustive_finalize(const Partial *__restrict__ parts,
                                                                      int nparts, int n, uint64_t count,
                                                                      const ExAcc *__restrict__ acc,
                                                                      const int *__restrict__ modep,
                                                                      tgo_summary *out) {
    finalize_block(parts, nparts, n, count, acc, *modep, out);
    if (threadIdx.x == 128) {  // no heuristic in this call
        put_order(out->heur, 0, 0);
        out->heur_ns = -1;
    }
}

// Last positions that one lane enumerates (two engines, a walk) or whose orders
// a block's prefixes share (one engine).  TGO_EXHAUSTIVE_M overrides the choice
// for tuning experiments (1..5, or 1..6 with one DMA engine).
static int choose_m(int n, bool one_dma) {
    const int cap = one_dma ? ONE_MAX_M : 5;
    if (const char *e = std::getenv("TGO_EXHAUSTIVE_M")) {
        const int m = std::atoi(e);
        if (m >= 1 && m <= cap && m <= n) return m;
    }
    // one engine: 720 prefixes per set, two tiles that fill their lanes.  Groups of
    // 9 / 10 / 11 in us, with 3 to 6 positions shared: 28 28 36 79 / 43 32 37 81 /
    // 249 85 50 84 (fewer: the block computes (B, C) for nothing; more: idle lanes)
    if (one_dma) return n < 7 ? 1 : (n - 6 < cap ? n - 6 : cap);
    // enough subtrees to fill the GPU.  With the three innermost levels
    // unrolled, 5 levels beat 4 at n = 12 on MI355X (1.81 vs 1.99 ms: fewer
    // windows per ordering, 2.77 vs 3.0).
    int m = 1;
    for (int c = cap; c >= 1; --c) {
        if (c > n) continue;
        const uint64_t sub = factorial(n) / factorial(c);
        if (sub >= 32768 || c == 1) { m = c; break; }
    }
    if (n <= 5) m = n < 1 ? 1 : n;
    return m;
}

// Blocks that fit on the device at once for a kernel and its dynamic LDS.
uint32_t resident_blocks(const void *kern, int threads, size_t shm) {
    struct Entry { int dev; const void *k; size_t shm; uint32_t blocks; };
    static std::mutex mu;
    static Entry cache[256];
    static int used = 0;
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) return 0;
    std::lock_guard<std::mutex> lk(mu);
    for (int i = 0; i < used; ++i)
        if (cache[i].dev == dev && cache[i].k == kern && cache[i].shm == shm) return cache[i].blocks;
    int cus = 0, per_cu = 0;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus <= 0)
        return 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kern, threads, shm) != hipSuccess || per_cu <= 0)
        per_cu = 1;
    const uint32_t b = (uint32_t)cus * (uint32_t)per_cu;
    if (used < 256) cache[used++] = Entry{dev, kern, shm, b};
    return b;
}

// The walk that also has the potential form (PotRule): the deepest, which the
// groups of 11 and more take, where it gains (potential_gains): 1782 / 1712 / 1744
// us where the chain form takes 2165 / 2011 / 2551 (three groups of 12).  At depth
// 4 it gained nothing, and the groups below 11, done in 60 us and less, would pay the launch
// that finds nothing to do, 4.5 us, when theirs does not fit.  Both forms take one
// grid, 12 rounds of the chain form's resident blocks (EX_ROUNDS, seven waves per
// SIMD): 16.8 rounds of the potential form's, with five; twice the grid was slower
// (1803 us against 1684).
constexpr int POT_M = 5;
template <int M, bool STORE>
static int launch_two(hipStream_t st, const tgo_task *t, int n, const Rates &r, uint32_t n_sub, int64_t *out,
                      tgo_summary *d_out, ExScratch ws) {
    const void *k32 = reinterpret_cast<const void *>(&enum_kernel<BaseRule, uint32_t, M, STORE, DMA_TWO>);
    uint32_t blocks = 0;
    EnumScratch sc;
    int rc = enum_grid(k32, enum_shm_bytes<BaseRule, uint32_t>(n, false), n_sub, 0, ws, st, &blocks, &sc);
    if (rc) return rc;
    const bool potential = M == POT_M && pot_rates(r, n);
    hipLaunchKernelGGL(exhaustive_classify, dim3(1), dim3(64), 0, st, t, n, r, potential, sc.mode, sc.acc);
    if constexpr (M == POT_M) {
        if (potential) {
            enum_launch_one<PotRule, uint32_t, M, STORE, DMA_TWO>(st, t, n, r, PotRule::Args{}, n_sub, out, blocks, sc);
            TGO_HIP(hipGetLastError());
        }
    }
    rc = enum_launch<BaseRule, M, STORE, DMA_TWO>(st, t, n, r, BaseRule::Args{}, n_sub, out, blocks, sc);
    if (rc) return rc;
    hipLaunchKernelGGL(exhaustive_finalize, dim3(1), dim3(EX_FIN_THREADS), 0, st, sc.parts, (int)blocks, n,
                       factorial(n), sc.acc, sc.mode, d_out);
    TGO_HIP(hipGetLastError());
    return TGO_OK;
}

template <bool STORE>
static int launch_two_m(int m, hipStream_t st, const tgo_task *t, int n,
                        const Rates &r, uint32_t n_sub, int64_t *out, tgo_summary *d_out, ExScratch ws) {
    switch (m) {
        case 1: return launch_two<1, STORE>(st, t, n, r, n_sub, out, d_out, ws);
        case 2: return launch_two<2, STORE>(st, t, n, r, n_sub, out, d_out, ws);
        case 3: return launch_two<3, STORE>(st, t, n, r, n_sub, out, d_out, ws);
        case 4: return launch_two<4, STORE>(st, t, n, r, n_sub, out, d_out, ws);
        default: return launch_two<5, STORE>(st, t, n, r, n_sub, out, d_out, ws);
    }
}

template <bool STORE>
static int launch_one(int m, hipStream_t st, const tgo_task *t, int n, const Rates &r, int64_t *out,
                      tgo_summary *d_out, ExScratch ws) {
    const OneShape sh = one_shape(n, m);
    const size_t lds = one_lds<uint64_t, STORE>(n, sh.orders);
    uint32_t blocks = 0;
    EnumScratch sc;
    int rc = enum_grid(reinterpret_cast<const void *>(&one_kernel<STORE>), lds, sh.tiles * EX_THREADS, 0, ws, st,
                       &blocks, &sc);
    if (rc) return rc;
    hipLaunchKernelGGL(exhaustive_classify, dim3(1), dim3(64), 0, st, t, n, r, false, sc.mode, sc.acc);
    hipLaunchKernelGGL(one_kernel<STORE>, dim3(blocks), dim3(EX_THREADS), lds, st, t, n, m, r, sh, out, sc.parts,
                       sc.acc, sc.mode);
    hipLaunchKernelGGL(exhaustive_finalize, dim3(1), dim3(EX_FIN_THREADS), 0, st, sc.parts, (int)blocks, n,
                       factorial(n), sc.acc, sc.mode, d_out);
    TGO_HIP(hipGetLastError());
    return TGO_OK;
}

static int launch_exhaustive_ws(const Rates &r, const tgo_task *d_tasks, int n, int64_t *d_per_order,
                                tgo_summary *d_out, hipStream_t st, ExScratch ws) {
    const bool one = r.one_dma != 0;
    // small groups: unless a tuning override asks for the general path
    if (factorial(n) <= SMALL_COUNT && !std::getenv("TGO_EXHAUSTIVE_M") && !std::getenv("TGO_EXHAUSTIVE_BLOCKS")) {
        const uint32_t count = (uint32_t)factorial(n);
        return one ? small_launch<BaseRule, DMA_ONE>(st, d_tasks, n, r, BaseRule::Args{}, count, d_per_order, d_out, ws)
                   : small_launch<BaseRule, DMA_TWO>(st, d_tasks, n, r, BaseRule::Args{}, count, d_per_order, d_out, ws);
    }
    const int m = choose_m(n, one);
    const uint64_t n_sub64 = factorial(n) / factorial(m);
    if (n_sub64 >= (1ull << 32)) return fail(TGO_EINVAL, "group too large to enumerate");
    const uint32_t n_sub = (uint32_t)n_sub64;
    if (one)
        return d_per_order ? launch_one<true>(m, st, d_tasks, n, r, d_per_order, d_out, ws)
                           : launch_one<false>(m, st, d_tasks, n, r, nullptr, d_out, ws);
    return d_per_order ? launch_two_m<true>(m, st, d_tasks, n, r, n_sub, d_per_order, d_out, ws)
                       : launch_two_m<false>(m, st, d_tasks, n, r, n_sub, nullptr, d_out, ws);
}

int launch_exhaustive(const Rates &r, const tgo_task *d_tasks, int n, int64_t *d_per_order,
                      tgo_summary *d_out, hipStream_t st) {
    return launch_exhaustive_ws(r, d_tasks, n, d_per_order, d_out, st, ExScratch{});
}

// Fixed scratch of the allocation-free enumeration: block partials, the
// 32-bit accumulator and the time-path word of one call.  Each device holds
// its own copy for the life of the process.  On the host the array's name is
// only a stand-in: its device address comes from hipGetSymbolAddress, taken
// once per device with that device current.
static __device__ __align__(256) unsigned char scratch[TGO_NOALLOC_SCRATCH_BYTES];

constexpr int EX_MAX_DEVICES = 64;

static int scratch_address(void **ptr) {
    static std::mutex mu;
    static void *addr[EX_MAX_DEVICES] = {};
    int dev = 0;
    TGO_HIP(hipGetDevice(&dev));
    if (dev < 0 || dev >= EX_MAX_DEVICES) return fail(TGO_EDEVICE, "device index above 63");
    std::lock_guard<std::mutex> lk(mu);
    if (!addr[dev]) {
        void *p = nullptr;
        const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return hip_fail(e, "hipGetSymbolAddress(scratch)");
        if (!p) return fail(TGO_EDEVICE, "hipGetSymbolAddress(scratch) returned NULL");
        addr[dev] = p;
    }
    *ptr = addr[dev];
    return TGO_OK;
}

int launch_exhaustive_noalloc(const Rates &r, const tgo_task *d_tasks, int n, int64_t *d_per_order,
                              tgo_summary *d_out, hipStream_t st) {
    ExScratch ws;
    int rc = scratch_address(&ws.ptr);
    if (rc) return rc;
    ws.bytes = TGO_NOALLOC_SCRATCH_BYTES;
    return launch_exhaustive_ws(r, d_tasks, n, d_per_order, d_out, st, ws);
}

}  // namespace tgo
