// Multi-round task groups (Section 6.2): T workers, each offloading R
// dependent tasks; a worker hands over its next task only when the previous
// one has completely finished (its DtH has ended).
//
// Task (w, r) is index w * R + r of the task table.  Two setups:
//   NoReorder: all T*R tasks queued at t = 0, round by round, round r in a
//     worker order pi_r; every (pi_0, ..., pi_{R-1}) is an ordering, ranked
//     with pi_0 most significant and each pi_r lexicographic.  The HtD of
//     (w, r) waits for the DtH of (w, r - 1), and the in-order queue behind it
//     waits too.  One lane per ordering, reduced like the single-group
//     enumeration.
//   Heuristic: a proxy takes every task waiting in the shared buffer as a
//     task group, orders it with Algorithm 1 and queues it; it looks at the
//     buffer again when the HtD of the group's last task starts (HtDs handed
//     to the engine just in time), or at the next arrival if the buffer is
//     empty then.  One lane per experiment.
//
// NoReorder runs the window formulation (rule_dev.h, RULE_ROUNDS): an HtD that
// depends on a DtH waits at a gate, in launch order like everything else.  The
// proxy's groups depend on when commands start and end, so the Heuristic setup
// steps events: at each instant every finished command retires, then every ready
// queue head starts, then the proxy looks, until nothing changes; time then
// advances to the earliest completion estimate (remaining transfer work is
// exact in 1/q solo-ns, estimates rounded up to whole ns, overlapped HtD and
// DtH at p_htd/q and p_dth/q).  Launch schemes of Section 3.2: two DMA
// engines = three FIFO queues in submission order; one DMA engine = one
// transfer queue holding, per submitted group, its HtDs then its DtHs.
#include <hip/hip_runtime.h>

#include "enum_kernel.h"
#include "heur_dev.h"
#include "rule_dev.h"
#include "tables_dev.h"
#include "tgo_internal.h"

namespace tgo {

// Event-stepping state of one simulation (the proxy's), the same on every lane.
template <typename TT>
struct RSim {
    TT t;
    uint64_t seq;    // nibble j: task at submitted position j
    uint64_t posof;  // nibble x: position of task x (once submitted)
    uint32_t gend;   // bit j: position j closes a submitted group
    int nsub;        // positions submitted so far
    // completed commands: positions < *_done have finished (every queue is
    // served in position order)
    int h_done, k_done, d_done;
    // two engines: next position to start per queue; one engine: the
    // transfer queue's current group [xb, xe) and offset xo in [0, 2 (xe - xb))
    int hc, kc, dc;
    int xb, xe, xo;
    bool hrun, krun, drun;  // one engine: hrun/drun say which transfer runs
    int hpos, dpos;         // position of the running transfer(s)
    TT uh, ud, kend;        // remaining transfer work (1/q ns), kernel end
};

template <typename TT>
__device__ __forceinline__ void rsim_init(RSim<TT> &s) {
    s.t = 0;
    s.seq = 0;
    s.posof = 0;
    s.gend = 0;
    s.nsub = 0;
    s.h_done = s.k_done = s.d_done = 0;
    s.hc = s.kc = s.dc = 0;
    s.xb = s.xe = s.xo = 0;
    s.hrun = s.krun = s.drun = false;
    s.hpos = s.dpos = 0;
    s.uh = s.ud = s.kend = 0;
}

// Append a group of g tasks (in launch order, one nibble each) at the current instant.
template <typename TT>
__device__ __forceinline__ void rsim_submit(RSim<TT> &s, uint64_t order, int g) {
    s.seq |= order << (4 * s.nsub);
    for (int i = 0; i < g; ++i) s.posof |= (uint64_t)(s.nsub + i) << (4 * nibble(order, i));
    s.nsub += g;
    s.gend |= 1u << (s.nsub - 1);
}

// The HtD at position j may start once the DtH of the same worker's previous
// task has ended (dep: bit x = task x depends on task x - 1).
template <typename TT>
__device__ __forceinline__ bool dep_ok(const RSim<TT> &s, int j, uint32_t dep) {
    const uint32_t x = nibble(s.seq, j);
    if (!((dep >> x) & 1u)) return true;
    return (uint32_t)s.d_done > nibble(s.posof, x - 1);
}

// One pass at the current instant: retire finished commands, then start every
// ready head.  Starts depend only on what has finished and been submitted, so
// another pass is needed only after a command of no length started (returned)
// or a submission; finished DtHs are reported
// in *arrived (bit x: the worker's next task x became available), the start
// of the HtD at position trig in *trig_started.
template <bool ONE, typename TT, typename ViewT>
__device__ __forceinline__ bool rsim_pass(RSim<TT> &s, const ViewT &v, const Rates &r, int trig,
                                          uint32_t *arrived, bool *trig_started) {
    bool again = false;
    // retire
    if (s.hrun && s.uh == 0) { s.hrun = false; ++s.h_done; }
    if (s.krun && s.kend == s.t) { s.krun = false; ++s.k_done; }
    if (s.drun && s.ud == 0) {
        s.drun = false;
        ++s.d_done;
        *arrived |= (2u << nibble(s.seq, s.dpos)) & v.dep;
    }
    // start ready heads
    if constexpr (!ONE) {
        if (!s.hrun && s.hc < s.nsub && dep_ok(s, s.hc, v.dep)) {
            s.hpos = s.hc++;
            s.uh = v.task(nibble(s.seq, s.hpos)).h << r.q_log2;
            s.hrun = true;
            again = again || s.uh == 0;
            if (s.hpos == trig) *trig_started = true;
        }
        if (!s.drun && s.dc < s.nsub && s.dc < s.k_done) {
            s.dpos = s.dc++;
            s.ud = v.task(nibble(s.seq, s.dpos)).d << r.q_log2;
            s.drun = true;
            again = again || s.ud == 0;
        }
    } else {
        if (!s.hrun && !s.drun) {
            if (s.xo == 2 * (s.xe - s.xb) && s.xe < s.nsub) {
                // next submitted group: [xe, end of that group)
                s.xb = s.xe;
                const uint32_t rest = s.gend >> s.xb;
                s.xe = s.xb + __ffs(rest);
                s.xo = 0;
            }
            const int len = s.xe - s.xb;
            if (s.xo < len) {
                const int j = s.xb + s.xo;
                if (dep_ok(s, j, v.dep)) {
                    s.hpos = j;
                    s.uh = v.task(nibble(s.seq, j)).h << r.q_log2;
                    s.hrun = true;
                    ++s.xo;
                    again = again || s.uh == 0;
                    if (j == trig) *trig_started = true;
                }
            } else if (s.xo < 2 * len) {
                const int j = s.xb + s.xo - len;
                if (s.k_done > j) {
                    s.dpos = j;
                    s.ud = v.task(nibble(s.seq, j)).d << r.q_log2;
                    s.drun = true;
                    ++s.xo;
                    again = again || s.ud == 0;
                }
            }
        }
    }
    if (!s.krun && s.kc < s.nsub && s.kc < s.h_done) {
        const int j = s.kc++;
        s.kend = s.t + v.task(nibble(s.seq, j)).k;
        s.krun = true;
        again = again || s.kend == s.t;
    }
    return again;
}

// Advance to the earliest completion estimate.  Returns false when nothing runs.
template <bool ONE, typename TT>
__device__ __forceinline__ bool rsim_advance(RSim<TT> &s, const Rates &r) {
    if (!s.hrun && !s.krun && !s.drun) return false;
    const bool both = !ONE && s.hrun && s.drun;
    const TT q = TT(1) << r.q_log2;
    constexpr TT INF = ~TT(0);
    const TT eh = s.hrun ? (both ? (TT)ceil_p(s.uh, r.p_h, r.inv_ph, r.c_ph) : ceil_q(s.uh, r.q_log2)) : INF;
    const TT ed = s.drun ? (both ? (TT)ceil_p(s.ud, r.p_d, r.inv_pd, r.c_pd) : ceil_q(s.ud, r.q_log2)) : INF;
    const TT ek = s.krun ? s.kend - s.t : INF;
    TT dt = eh < ed ? eh : ed;
    dt = ek < dt ? ek : dt;
    if (s.hrun) s.uh = eh == dt ? TT(0) : s.uh - (both ? TT(r.p_h) : q) * dt;
    if (s.drun) s.ud = ed == dt ? TT(0) : s.ud - (both ? TT(r.p_d) : q) * dt;
    s.t += dt;
    return true;
}

// Heuristic setup: one wave drives the proxy and the device model.  v: the
// tables of all tasks; first: the tasks waiting at t = 0.
template <bool ONE, typename TT, typename ViewT>
__device__ __forceinline__ void rounds_proxy(const ViewT &v, uint32_t first, int n, const Rates &r, tgo_summary *out,
                                             uint16_t *groups) {
    RSim<TT> s;
    rsim_init(s);
    uint32_t buffer = first;
    bool armed = true;
    int trig = -1;
    for (;;) {
        bool again = true;
        while (again) {
            uint32_t arrived = 0;
            bool started = false;
            again = rsim_pass<ONE>(s, v, r, trig, &arrived, &started);
            buffer |= arrived;
            armed = armed || started;
            if (armed && buffer) {
                // the group: the waiting tasks, ordered by Algorithm 1
                uint64_t ord;
                if constexpr (ONE) heuristic_wave<DMA_ONE, Lane<TT>, false>(buffer, v, r, &ord);
                else heuristic_wave<DMA_TWO, CLane<TT>, false>(buffer, v, r, &ord);
                rsim_submit(s, ord, __popc(buffer));
                trig = s.nsub - 1;
                buffer = 0;
                armed = false;
                again = true;
            }
        }
        if (!rsim_advance<ONE>(s, r)) break;
    }
    put_heuristic(out, s.seq, n, (int64_t)s.t);
    if (groups && threadIdx.x == 0) *groups = (uint16_t)s.gend;
}

// Launch sequence (task per position, one nibble each) of NoReorder rank rk.
__device__ __forceinline__ uint64_t rounds_unrank(int T, int R, uint64_t rk, uint32_t tfact) {
    uint32_t rem = (uint32_t)rk;  // (T!)^R < 2^32
    uint64_t out = 0;
    for (int rr = R - 1; rr >= 0; --rr) {
        uint32_t d = rem % tfact;
        rem /= tfact;
        uint64_t list = 0;
        for (int i = T - 1; i >= 0; --i) list = (list << 4) | (uint64_t)i;
        uint32_t f = tfact;
        for (int i = 0; i < T; ++i) {
            f /= (uint32_t)(T - i);
            const uint32_t c = d / f;
            d -= c * f;
            const uint64_t w = (list >> (4 * c)) & 15u;
            const uint64_t lo = list & ((1ull << (4 * c)) - 1ull);
            list = lo | ((list >> (4 * c + 4)) << (4 * c));
            out |= (w * (uint64_t)R + (uint64_t)rr) << (4 * (rr * T + i));
        }
    }
    return out;
}

// Dependent tasks under the enumeration kernel (enum_kernel.h): a subtree
// holds the orderings that share every earlier round and the last round's
// first T - M positions; subtrees are taken in rank order.  Bound by the
// latency of one lane's windows: four workers with four tasks each are 331,776
// orderings, 55,296 lanes of 28 windows.  Stepping the events of every
// ordering in 64-bit time took 198 us for them and the Heuristic setup, on one
// thread after it, 115 us; together, side by side, 313 -> 48 us per call, 40 with
// the proxies' single pass per instant.
struct RoundsRule : GroupRule {
    struct Args {
        int T, R;
        uint32_t tfact;  // T!
        tgo_summary *out;  // the Heuristic setup's fields
        uint16_t *groups;
    };
    static constexpr bool SIDE = true;
    template <typename TT>
    using View = RView<TT, 1, EX_THREADS, RULE_ROUNDS>;
    template <typename TT, int DMA>
    using Lane = std::conditional_t<DMA == DMA_TWO, RLane<TT, RULE_ROUNDS>, SubChain<TT, RULE_ROUNDS>>;
    template <typename TT, int DMA>
    static constexpr int min_waves() { return sizeof(TT) == 4 ? 4 : 1; }
    static constexpr bool queue(bool one_dma) { return !one_dma; }
    static __host__ __device__ constexpr size_t lds_bytes(int) { return 0; }
    static __device__ __forceinline__ int status(const tgo_task *tasks, int n, const Rates &r, const Args &,
                                                 int lane) {
        return classify_group_wave(tasks, n, r, lane);
    }
    static __device__ __forceinline__ void on_error(const Args &a) {
        if (a.groups) *a.groups = 0;
    }
    template <int DMA, typename LaneT, typename ViewT>
    static __device__ __forceinline__ uint64_t small_prefix(LaneT &st, uint32_t rank, int n, ViewT &v, const Rates &r,
                                                            const Args &a) {
        uint32_t lex;
        return prefix<DMA>(st, rank, n, 1, v, r, a, &lex);
    }
    static __device__ __forceinline__ uint64_t decode(uint64_t rk, int, const Args &a) {
        return rounds_unrank(a.T, a.R, rk, a.tfact);
    }
    template <bool SMALL, typename ViewT>
    static __device__ __forceinline__ void load(ViewT &v, unsigned char *, const Args &a, int n, uint64_t *seq) {
        v.seq = seq;
        v.pos = 0;
        v.dep = v.opens = 0;
        for (int x = 0; x < n; ++x) v.dep |= (x % a.R != 0 ? 1u : 0u) << x;
        for (int j = a.T; j < n; j += a.T) v.opens |= 1u << j;
    }
    template <typename TT, int DMA, typename ViewT>
    static __device__ __forceinline__ void side(const ViewT &v, int n, const Rates &r, const Args &a) {
        rounds_proxy<DMA == DMA_ONE, TT>(v, ((1u << n) - 1u) & ~v.dep, n, r, a.out, a.groups);
    }
    template <int DMA, typename LaneT, typename ViewT>
    static __device__ __forceinline__ uint64_t prefix(LaneT &st, uint32_t s, int n, int m, ViewT &v, const Rates &r,
                                                      const Args &a, uint32_t *lex) {
        lane_reset(st);
        *lex = s;
        uint64_t workers = 0;
        for (int i = a.T - 1; i >= 0; --i) workers = (workers << 4) | (uint64_t)i;
        uint32_t mf = 1;
        for (int i = 2; i <= m; ++i) mf *= (uint32_t)i;
        // weight of a round's digit, in subtrees; the last round's are its
        // blocks of m! orderings
        uint32_t weight = a.tfact / mf;
        for (int i = 2; i < a.R; ++i) weight *= a.tfact;  // below n_sub < 2^32
        uint32_t rem = s;
        uint64_t pos = 0, list = 0;
        for (int rr = 0; rr < a.R; ++rr) {
            const bool last = rr == a.R - 1;
            uint32_t d = rem;
            if (!last) {
                d = rem / weight;
                rem -= d * weight;
                weight = rr == a.R - 2 ? weight : weight / a.tfact;
            }
            list = workers;
            uint32_t f = last ? a.tfact / mf : a.tfact;
            const int np = last ? a.T - m : a.T;
            for (int i = 0; i < np; ++i) {
                f /= (uint32_t)(a.T - i);
                const uint32_t c = d / f;
                d -= c * f;
                const uint32_t w = (uint32_t)(list >> (4 * c)) & 15u;
                const uint64_t lo = list & ((1ull << (4 * c)) - 1ull);
                list = lo | ((list >> (4 * c + 4)) << (4 * c));
                const uint32_t x = w * (uint32_t)a.R + (uint32_t)rr;
                const int j = rr * a.T + i;
                v.pos = pos;
                window<DMA>(st, j, x, v, r);
                pos |= (uint64_t)j << (4 * x);
            }
        }
        v.pos = pos;
        // the workers left in the last round as tasks, ascending
        uint64_t left = 0;
        for (int i = 0; i < m; ++i)
            left |= (uint64_t)(((uint32_t)(list >> (4 * i)) & 15u) * (uint32_t)a.R + (uint32_t)a.R - 1u) << (4 * i);
        return left;
    }
};

// Time path of the group, or TGO_ERANGE; clears the accumulators.
__global__ __launch_bounds__(64) void rounds_prepare_kernel(const tgo_task *__restrict__ tasks, int n, Rates r,
                                                            int *mode, ExAcc *acc) {
    const int m = classify_group_wave(tasks, n, r, threadIdx.x);
    if (threadIdx.x == 0) *mode = m;
    exacc_init(acc, threadIdx.x);
}

__global__ __launch_bounds__(EX_FIN_THREADS) void rounds_finalize_kernel(
    const Partial *__restrict__ parts, int nparts, int T, int R, uint64_t count, uint32_t tfact,
    const ExAcc *__restrict__ acc, const int *__restrict__ modep, tgo_summary *out, uint16_t *groups) {
    const int mode = *modep;
    if (mode < 0) {
        put_heuristic(out, 0, 0, mode);
        if (groups && threadIdx.x == 0) *groups = 0;
    }
    finalize_block(parts, nparts, T * R, count, acc, mode,
                   [=](uint64_t rk) { return rounds_unrank(T, R, rk, tfact); }, out);
}

template <int M, bool STORE, int DMA>
static int launch_rounds_m(hipStream_t st, const tgo_task *t, int T, int R, const Rates &r, uint64_t count,
                           uint32_t tf, int64_t *out, tgo_summary *d_out, uint16_t *d_groups) {
    const void *k32 = reinterpret_cast<const void *>(&enum_kernel<RoundsRule, uint32_t, M, STORE, DMA>);
    const uint32_t n_sub = (uint32_t)(count / factorial(M));
    const int n = T * R;
    uint32_t blocks = 0;
    EnumScratch sc;
    int rc = enum_grid(k32, enum_shm_bytes<RoundsRule, uint32_t>(n, DMA == DMA_ONE), n_sub, 0, ExScratch{}, st,
                       &blocks, &sc);
    if (rc) return rc;
    hipLaunchKernelGGL(rounds_prepare_kernel, dim3(1), dim3(64), 0, st, t, n, r, sc.mode, sc.acc);
    rc = enum_launch<RoundsRule, M, STORE, DMA>(st, t, n, r, RoundsRule::Args{T, R, tf, d_out, d_groups}, n_sub, out, blocks, sc);
    if (rc) return rc;
    hipLaunchKernelGGL(rounds_finalize_kernel, dim3(1), dim3(EX_FIN_THREADS), 0, st, sc.parts, (int)blocks, T, R,
                       count, tf, sc.acc, sc.mode, d_out, d_groups);
    TGO_HIP(hipGetLastError());
    return TGO_OK;
}

// Positions of the last round walked depth first per lane (TGO_ROUNDS_M, 1..4,
// overrides it): the deepest that leaves 32,768 subtrees, as in rule_depth.
// Four workers with four tasks: 62 / 51 / 48 us per call with 1 / 2 / 3 (before the
// proxies took one pass per instant: 40 with 3).
static int choose_rounds_m(int T, uint64_t count) {
    int top = T < 4 ? T : 4;
    if (const char *e = std::getenv("TGO_ROUNDS_M")) {
        const int m = std::atoi(e);
        if (m >= 1 && m <= top) return m;
    }
    while (top > 1 && count / factorial(top) < 32768) --top;
    return top;
}

template <bool STORE, int DMA>
static int launch_rounds_dma(hipStream_t st, const tgo_task *t, int T, int R, const Rates &r, uint64_t count,
                             uint32_t tf, int64_t *out, tgo_summary *d_out, uint16_t *d_groups) {
    switch (choose_rounds_m(T, count)) {
        case 1: return launch_rounds_m<1, STORE, DMA>(st, t, T, R, r, count, tf, out, d_out, d_groups);
        case 2: return launch_rounds_m<2, STORE, DMA>(st, t, T, R, r, count, tf, out, d_out, d_groups);
        case 3: return launch_rounds_m<3, STORE, DMA>(st, t, T, R, r, count, tf, out, d_out, d_groups);
        default: return launch_rounds_m<4, STORE, DMA>(st, t, T, R, r, count, tf, out, d_out, d_groups);
    }
}

int launch_rounds(const Rates &r, const tgo_task *d_tasks, int T, int R, int64_t *d_per_order,
                  tgo_summary *d_out, uint16_t *d_groups, hipStream_t st) {
    const uint32_t tf = (uint32_t)factorial(T);
    uint64_t count = 1;
    for (int i = 0; i < R; ++i) count *= tf;
    if (count <= SMALL_COUNT && !std::getenv("TGO_ROUNDS_M")) {
        const RoundsRule::Args a{T, R, tf, d_out, d_groups};
        const uint32_t c = (uint32_t)count;
        return r.one_dma
                   ? small_launch<RoundsRule, DMA_ONE>(st, d_tasks, T * R, r, a, c, d_per_order, d_out, ExScratch{})
                   : small_launch<RoundsRule, DMA_TWO>(st, d_tasks, T * R, r, a, c, d_per_order, d_out, ExScratch{});
    }
    if (r.one_dma)
        return d_per_order ? launch_rounds_dma<true, DMA_ONE>(st, d_tasks, T, R, r, count, tf, d_per_order, d_out, d_groups)
                           : launch_rounds_dma<false, DMA_ONE>(st, d_tasks, T, R, r, count, tf, nullptr, d_out, d_groups);
    return d_per_order ? launch_rounds_dma<true, DMA_TWO>(st, d_tasks, T, R, r, count, tf, d_per_order, d_out, d_groups)
                       : launch_rounds_dma<false, DMA_TWO>(st, d_tasks, T, R, r, count, tf, nullptr, d_out, d_groups);
}

}  // namespace tgo
