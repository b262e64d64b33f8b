// Task groups whose kernels may run concurrently (CKE).
//
// The paper's model keeps one kernel queue (Section 4.1, last paragraph): a
// kernel that exhausts the device overlaps the next one only at its tail, and
// devices do not disclose how they run concurrent kernels.  Its NoReorder
// experiments do use one command queue per kernel (Section 6.2), Section 3.2
// states when kernels from different queues can overlap (while the device's
// resources are not exhausted), and the conclusion leaves concurrent kernels
// to future work.  Reading used here:
//   * the device has `capacity` units of computing resources; kernel x holds
//     units[x] of them (1 .. capacity) from its start to its end;
//   * kernels are dispatched in launch order: K at position j starts once its
//     HtD has ended, the kernel at position j - 1 has started, and its units
//     fit beside those of the running kernels; it takes its solo time;
//   * transfers follow the launch schemes of Section 3.2 as everywhere else
//     (two DMA engines: HtD and DtH FIFO queues; one engine: every HtD, then
//     every DtH, on one queue), with the Section 4.2.1 overlap rates.
// With every kernel holding the whole capacity this is the one-queue model.
//
// The enumeration and Algorithm 1 run the window formulation (rule_dev.h,
// RULE_CONCURRENT): transfers do not feel how kernels are dispatched, and the
// end of a kernel is fixed once its HtD has ended.  tgo_evaluate_cke steps the
// events of each given ordering (64-bit time): at each instant every finished
// command retires, then every ready head starts and the kernel dispatcher
// takes what fits, until nothing changes; time then advances to the earliest
// completion.
#include <hip/hip_runtime.h>

#include "enum_kernel.h"
#include "heur_dev.h"
#include "rule_dev.h"
#include "tables_dev.h"
#include "tgo_internal.h"

namespace tgo {

constexpr int CK_THREADS = 256;
constexpr int32_t CK_MAX_CAPACITY = 1 << 30;

struct CTab {
    int64_t h[MAXN], k[MAXN], d[MAXN];
    int32_t u[MAXN];
};

// Block-wide load of the task table; 0, TGO_ERANGE (a duration outside
// [0, 2^40)) or TGO_EINVAL (a unit count outside 1..cap).
__device__ int ctab_load(const tgo_task *__restrict__ tasks, const int32_t *__restrict__ units, int n, int cap,
                         CTab &tb, int *flag) {
    if (threadIdx.x == 0) *flag = 0;
    __syncthreads();
    if ((int)threadIdx.x < n) {
        const tgo_task t = tasks[threadIdx.x];
        const int32_t u = units[threadIdx.x];
        if (t.htd_ns < 0 || t.kern_ns < 0 || t.dth_ns < 0 || t.htd_ns >= MAX_DURATION ||
            t.kern_ns >= MAX_DURATION || t.dth_ns >= MAX_DURATION)
            atomicOr(flag, 1);
        if (u < 1 || u > cap) atomicOr(flag, 2);
        tb.h[threadIdx.x] = t.htd_ns;
        tb.k[threadIdx.x] = t.kern_ns;
        tb.d[threadIdx.x] = t.dth_ns;
        tb.u[threadIdx.x] = u;
    }
    __syncthreads();
    const int f = *flag;
    return (f & 1) ? TGO_ERANGE : (f & 2) ? TGO_EINVAL : 0;
}

// T of one ordering (seq: task at position j in nibble j, n positions).  kend:
// this lane's kernel end times by position (stride kst).
template <bool ONE>
__device__ int64_t cke_sim(uint64_t seq, int n, const CTab &tb, int cap, const Rates &r, int64_t *kend, int kst) {
    const int64_t q = int64_t(1) << r.q_log2;
    int64_t t = 0;
    int hc = 0, dc = 0, xo = 0;  // next queue entry: HtD, DtH (two engines); transfer queue (one)
    bool hrun = false, drun = false;
    int hpos = 0, dpos = 0, hdone = 0;
    int64_t uh = 0, ud = 0;
    int kc = 0, held = 0;
    uint32_t krun = 0, kdone = 0;
    for (;;) {
        bool changed = true;
        while (changed) {
            changed = false;
            if (hrun && uh == 0) {
                hrun = false;
                ++hdone;
                changed = true;
            }
            if (drun && ud == 0) {
                drun = false;
                changed = true;
            }
            for (uint32_t m = krun; m; m &= m - 1) {
                const int p = __ffs(m) - 1;
                if (kend[p * kst] == t) {
                    krun &= ~(1u << p);
                    kdone |= 1u << p;
                    held -= tb.u[nibble(seq, p)];
                    changed = true;
                }
            }
            if constexpr (!ONE) {
                if (!hrun && hc < n) {
                    hpos = hc++;
                    uh = q * tb.h[nibble(seq, hpos)];
                    hrun = true;
                    changed = true;
                }
                if (!drun && dc < n && ((kdone >> dc) & 1u)) {
                    dpos = dc++;
                    ud = q * tb.d[nibble(seq, dpos)];
                    drun = true;
                    changed = true;
                }
            } else {
                if (!hrun && !drun) {
                    if (xo < n) {
                        hpos = xo++;
                        uh = q * tb.h[nibble(seq, hpos)];
                        hrun = true;
                        changed = true;
                    } else if (xo < 2 * n && ((kdone >> (xo - n)) & 1u)) {
                        dpos = xo - n;
                        ++xo;
                        ud = q * tb.d[nibble(seq, dpos)];
                        drun = true;
                        changed = true;
                    }
                }
            }
            // in-order dispatch of the kernels whose HtD has ended and that fit
            while (kc < n && kc < hdone && held + tb.u[nibble(seq, kc)] <= cap) {
                const uint32_t x = nibble(seq, kc);
                kend[kc * kst] = t + tb.k[x];
                krun |= 1u << kc;
                held += tb.u[x];
                ++kc;
                changed = true;
            }
        }
        if (!hrun && !drun && !krun) break;
        const bool both = !ONE && hrun && drun;
        const int64_t rh = both ? (int64_t)r.p_h : q, rd = both ? (int64_t)r.p_d : q;
        const int64_t INF = INT64_MAX;
        const int64_t eh = hrun ? (uh + rh - 1) / rh : INF;
        const int64_t ed = drun ? (ud + rd - 1) / rd : INF;
        int64_t dt = eh < ed ? eh : ed;
        for (uint32_t m = krun; m; m &= m - 1) {
            const int p = __ffs(m) - 1;
            const int64_t e = kend[p * kst] - t;
            dt = e < dt ? e : dt;
        }
        if (hrun) uh = eh == dt ? 0 : uh - rh * dt;
        if (drun) ud = ed == dt ? 0 : ud - rd * dt;
        t += dt;
    }
    return t;
}

// Concurrent kernels under the enumeration kernel (enum_kernel.h).  Bound by
// VALU issue over divergent window loops, like the plain enumeration, plus the
// scan of running kernels where a kernel does not fit at once.  As a lane per
// ordering stepping all of its events in 64-bit time, n = 12 took 123.5 ms
// (479M orderings); with shared prefixes, windows and 32-bit time 4.6 ms.
struct CkeRule : GroupRule {
    struct Args {
        const int32_t *units;
        int32_t cap;
        tgo_summary *out;  // the heuristic's fields
    };
    static constexpr bool SIDE = true;
    template <typename TT>
    using View = RView<TT, 1, EX_THREADS, RULE_CONCURRENT>;
    template <typename TT, int DMA>
    using Lane = RLane<TT, RULE_CONCURRENT>;
    // 6 waves per SIMD (80 VGPRs; 160 B of saved walk state per lane spill): 4.15 /
    // 4.22 / 4.49 ms on three n = 12 groups, against 4.32 / 4.53 / 4.77 at 5 waves,
    // 4.24 / 4.12 / 4.43 at 7 and 4.89 / 4.87 / 5.09 at 8
    template <typename TT, int DMA>
    static constexpr int min_waves() { return sizeof(TT) == 4 ? 6 : 1; }
    static constexpr bool queue(bool) { return true; }
    static __host__ __device__ constexpr size_t lds_bytes(int) { return sizeof(int32_t) * MAXN; }
    static __device__ __forceinline__ int status(const tgo_task *tasks, int n, const Rates &r, const Args &a,
                                                 int lane) {
        const int m = classify_group_wave(tasks, n, r, lane);
        const int32_t u = lane < n ? a.units[lane] : 1;
        const bool bad = __any(u < 1 || u > a.cap);
        return m < 0 ? m : bad ? TGO_EINVAL : m;
    }
    template <bool SMALL, typename ViewT>
    static __device__ __forceinline__ void load(ViewT &v, unsigned char *lds, const Args &a, int n, uint64_t *seq) {
        int32_t *u = reinterpret_cast<int32_t *>(lds);
        if ((int)threadIdx.x < n) u[threadIdx.x] = a.units[threadIdx.x];
        v.units = u;
        v.cap = a.cap;
        v.seq = seq;
    }
    // Algorithm 1 (Section 5.1) with `update` simulating the ordered set under
    // the same rule.
    template <typename TT, int DMA, typename ViewT>
    static __device__ __forceinline__ void side(const ViewT &v, int n, const Rates &r, const Args &a) {
        uint64_t ord;
        const int64_t T = heuristic_wave<DMA, Lane<TT, DMA>>((1u << n) - 1u, v, r, &ord);
        put_heuristic(a.out, ord, n, T);
    }
};

// Time path of the group (as classify_group), or TGO_ERANGE / TGO_EINVAL (a
// unit count outside 1..cap); clears the accumulators.
__global__ __launch_bounds__(64) void cke_prepare_kernel(const tgo_task *__restrict__ tasks, CkeRule::Args args, int n,
                                                         Rates r, int *mode, ExAcc *acc) {
    const int m = CkeRule::status(tasks, n, r, args, threadIdx.x);
    if (threadIdx.x == 0) *mode = m;
    exacc_init(acc, threadIdx.x);
}

template <int M, bool STORE, int DMA>
static int launch_cke(hipStream_t st, const tgo_task *t, const CkeRule::Args &args, int n, const Rates &r,
                      int64_t *out, tgo_summary *d_out) {
    const void *k32 = reinterpret_cast<const void *>(&enum_kernel<CkeRule, uint32_t, M, STORE, DMA>);
    const uint32_t n_sub = (uint32_t)(factorial(n) / factorial(M));
    uint32_t blocks = 0;
    EnumScratch sc;
    int rc = enum_grid(k32, enum_shm_bytes<CkeRule, uint32_t>(n, DMA == DMA_ONE), n_sub, 0, ExScratch{}, st, &blocks,
                       &sc);
    if (rc) return rc;
    hipLaunchKernelGGL(cke_prepare_kernel, dim3(1), dim3(64), 0, st, t, args, n, r, sc.mode, sc.acc);
    rc = enum_launch<CkeRule, M, STORE, DMA>(st, t, n, r, args, n_sub, out, blocks, sc);
    if (rc) return rc;
    hipLaunchKernelGGL(rule_finalize, dim3(1), dim3(EX_FIN_THREADS), 0, st, sc.parts, (int)blocks, n, factorial(n),
                       sc.acc, sc.mode, d_out);
    TGO_HIP(hipGetLastError());
    return TGO_OK;
}

// Positions walked depth first per lane (TGO_CKE_M, 1..5, overrides it): at
// n = 12, 14.9 / 7.6 / 4.9 / 4.1 ms with 2 / 3 / 4 / 5.
static int choose_cke_m(int n) {
    if (const char *e = std::getenv("TGO_CKE_M")) {
        const int m = std::atoi(e);
        if (m >= 1 && m <= 5 && m <= n) return m;
    }
    return rule_depth(n, 5);
}

template <bool STORE, int DMA>
static int launch_cke_m(hipStream_t st, const tgo_task *t, const int32_t *units, int n, int cap, const Rates &r,
                        int64_t *out, tgo_summary *d_out) {
    const CkeRule::Args a{units, cap, d_out};
    if (factorial(n) <= SMALL_COUNT && !std::getenv("TGO_CKE_M"))
        return small_launch<CkeRule, DMA>(st, t, n, r, a, (uint32_t)factorial(n), out, d_out, ExScratch{});
    switch (choose_cke_m(n)) {
        case 1: return launch_cke<1, STORE, DMA>(st, t, a, n, r, out, d_out);
        case 2: return launch_cke<2, STORE, DMA>(st, t, a, n, r, out, d_out);
        case 3: return launch_cke<3, STORE, DMA>(st, t, a, n, r, out, d_out);
        case 4: return launch_cke<4, STORE, DMA>(st, t, a, n, r, out, d_out);
        default: return launch_cke<5, STORE, DMA>(st, t, a, n, r, out, d_out);
    }
}

// T of given orderings (rows of n bytes), or a negative TGO_E*.
template <bool ONE>
__global__ __launch_bounds__(CK_THREADS) void cke_evaluate_kernel(const tgo_task *__restrict__ tasks,
                                                                 const int32_t *__restrict__ units, int n, int cap,
                                                                 Rates r, const uint8_t *__restrict__ orders,
                                                                 int64_t m, int64_t *out) {
    __shared__ CTab tb;
    __shared__ int flag;
    __shared__ int64_t kq[MAXN * CK_THREADS];
    const int st = ctab_load(tasks, units, n, cap, tb, &flag);
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= m) return;
    if (st != 0) {
        out[i] = st;
        return;
    }
    uint64_t seq = 0;
    uint32_t seen = 0;
    for (int j = 0; j < n; ++j) {
        const uint32_t x = orders[i * n + j];
        if (x < (uint32_t)n) seen |= 1u << x;
        seq |= (uint64_t)(x & 15u) << (4 * j);
    }
    if (seen != (1u << n) - 1u) {
        out[i] = TGO_EINVAL;
        return;
    }
    out[i] = cke_sim<ONE>(seq, n, tb, cap, r, kq + threadIdx.x, CK_THREADS);
}

static int check_cke(const tgo_model *model, Rates *r, int n, int max_n, int32_t cap) {
    int rc = make_rates(model, r);
    if (rc) return rc;
    if (n < 1 || n > max_n) return fail(TGO_EINVAL, "n out of range");
    if (cap < 1 || cap > CK_MAX_CAPACITY) return fail(TGO_EINVAL, "capacity must be in 1..2^30");
    return TGO_OK;
}

}  // namespace tgo

using namespace tgo;

extern "C" {

int tgo_exhaustive_cke(const tgo_model *model, const tgo_task *d_tasks, const int32_t *d_units, int n,
                       int32_t capacity, int64_t *d_per_order, tgo_summary *d_summary, tgo_stream stream) {
    Rates r;
    int rc = check_cke(model, &r, n, TGO_MAX_CKE_N, capacity);
    if (rc) return rc;
    if (!d_tasks || !d_units || !d_summary) return fail(TGO_EINVAL, "NULL buffer");
    hipStream_t st = (hipStream_t)stream;
    if (r.one_dma)
        return d_per_order ? launch_cke_m<true, DMA_ONE>(st, d_tasks, d_units, n, capacity, r, d_per_order, d_summary)
                           : launch_cke_m<false, DMA_ONE>(st, d_tasks, d_units, n, capacity, r, nullptr, d_summary);
    return d_per_order ? launch_cke_m<true, DMA_TWO>(st, d_tasks, d_units, n, capacity, r, d_per_order, d_summary)
                       : launch_cke_m<false, DMA_TWO>(st, d_tasks, d_units, n, capacity, r, nullptr, d_summary);
}

int tgo_evaluate_cke(const tgo_model *model, const tgo_task *d_tasks, const int32_t *d_units, int n,
                     int32_t capacity, const uint8_t *d_orders, int64_t m, int64_t *d_out, tgo_stream stream) {
    Rates r;
    int rc = check_cke(model, &r, n, TGO_MAX_N, capacity);
    if (rc) return rc;
    if (m < 0 || m > ((int64_t)1 << 40)) return fail(TGO_EINVAL, "m must be in 0..2^40");
    if (m == 0) return TGO_OK;
    if (!d_tasks || !d_units || !d_orders || !d_out) return fail(TGO_EINVAL, "NULL buffer");
    hipStream_t st = (hipStream_t)stream;
    const int64_t blocks = (m + CK_THREADS - 1) / CK_THREADS;
    if (r.one_dma)
        hipLaunchKernelGGL(cke_evaluate_kernel<true>, dim3((uint32_t)blocks), dim3(CK_THREADS), 0, st, d_tasks,
                           d_units, n, capacity, r, d_orders, m, d_out);
    else
        hipLaunchKernelGGL(cke_evaluate_kernel<false>, dim3((uint32_t)blocks), dim3(CK_THREADS), 0, st, d_tasks,
                           d_units, n, capacity, r, d_orders, m, d_out);
    TGO_HIP(hipGetLastError());
    return TGO_OK;
}

}  // extern "C"
