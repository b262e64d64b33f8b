// Device-side temporal execution model (gfx950).
//
// The model is the FIFO simulator of Section 4.1 for a two-DMA device
// (launch scheme of Section 3.2 with three command queues), with the
// overlapped-transfer slowdown of Section 4.2.1 read as constant rates p/q.
// Integer nanoseconds; remaining transfer work exact in 1/q solo-ns units; a
// completion estimate is rounded up to a whole nanosecond.
//
// GPU formulation (same results as stepping every event):
//   * The HtD engine is busy without a gap from t = 0 until the last HtD
//     completes, so the DtH rate is p_dth/q for every DtH that starts before
//     that instant and q/q afterwards.  The HtD rate changes only when the
//     DtH engine goes idle or starts from idle.
//   * Between rate changes an end estimate stays valid, because
//     ceil((U - r*D)/r) = ceil(U/r) - D for a whole number of ns D.  So each
//     running transfer carries its absolute end time, and the remaining work is
//     recomputed (one multiply) only when its rate changes.
//   * The kernel engine needs no events of its own: K_j = max(HtD_j end,
//     K_{j-1} end) + k.
//   * The simulation is cut into "windows": window j runs from the start to
//     the end of HtD at position j and processes the DtHs inside it.
//     The state at the start of window j depends only on positions < j, which
//     lets an enumeration share the windows of a common prefix.
//   * After the last HtD every DtH runs at full speed, so the rest is the
//     two-machine recurrence D = max(D, K_p end) + d_p over the remaining
//     positions, whose value is
//       max(end of the running DtH + sum of the solo DtH left after it,
//           max_p (K_p end + sum_{s >= p} d_s)).
//     Terms of positions whose DtH already started are lower bounds of the total
//     (every DtH takes at least its solo time after its kernel), so the second
//     max may run over every placed position: it is emax + dpre, kept per window.
//   * Chain form (CLane below): since every DtH that starts before the last
//     HtD ends runs at the overlapped rate, its start and end follow from the
//     previous DtH's end and its own kernel's end alone:
//     S_j = max(E_{j-1}, K_j), E_j = S_j + ceil(q d_j / p_dth).  Window j
//     appends DtH j to this chain once K_j is known, and a window only walks
//     the DtHs that end inside it; a start from idle is handled in the same
//     step as the completion before it, and a DtH that follows the previous
//     one without a gap leaves the HtD estimate as it is.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace tgo {

constexpr int MAXN = 16;

// Host-prepared model constants.
struct Rates {
    int32_t q_log2;
    uint32_t p_h, p_d;
    int32_t one_dma;  // 1: device with one DMA engine (launch scheme of Section 3.2)
    // ceil(u / p) for u < 2^32 as trunc(fma(u, 1/p, (p - 1/2)/p)).  The exact
    // value (u + p - 1/2)/p lies at least 1/(2p) away from the integers that
    // bound ceil(u/p); the double rounding error is below 2^-19 for u < 2^32,
    // so for p <= 1024 the truncation is exact.
    double inv_ph, c_ph;
    double inv_pd, c_pd;
    // exact quotients by q - p_h (p_h < q): it is odd << dsh, odd * dinv = 1 mod 2^32
    uint32_t dinv;
    int32_t dsh;
    // floor(x / p_h) = umulhi(x, phm) >> phs for x < 2^31 (p_h > 1)
    uint32_t phm;
    int32_t phs;
};

template <typename TT>
struct alignas(4 * sizeof(TT)) DRec {
    TT d;      // DtH solo duration
    TT dp;     // duration when fully overlapped: ceil(q d / p_dth)
    TT slack;  // p_dth dp - q d, in [0, p_dth)
    TT pad;
};

template <typename TT>
struct alignas(4 * sizeof(TT)) Quad {
    TT h, hp, k, d;  // HtD solo, HtD fully overlapped, kernel, DtH solo
};

template <typename TT>
struct alignas(2 * sizeof(TT)) Slot {
    TT ck;  // completion time of the kernel at this position
    TT dp;  // its DtH while overlapped: ceil(q d / p_dth).  p_dth dp = q d + slack
            // with slack < p_dth <= q, so d and slack follow from p_dth dp
};

// Chain entry of DtH j: start and end while the HtD engine is busy.
template <typename TT>
struct alignas(2 * sizeof(TT)) Span {
    TT s, e;
};
static_assert(sizeof(Span<uint32_t>) == sizeof(Slot<uint32_t>), "chain entries reuse the queue slots");
static_assert(sizeof(Span<uint64_t>) == sizeof(Slot<uint64_t>), "chain entries reuse the queue slots");

template <typename TT> struct Signed;
template <> struct Signed<uint32_t> { using type = int32_t; };
template <> struct Signed<uint64_t> { using type = int64_t; };

template <typename TT>
__device__ __forceinline__ TT ceil_q(TT u, int q_log2) {
    return (u + ((TT(1) << q_log2) - 1)) >> q_log2;
}

__device__ __forceinline__ uint32_t ceil_p(uint32_t u, uint32_t, double inv, double c) {
    return (uint32_t)__builtin_fma((double)u, inv, c);
}
// 64-bit: u < 2^51 is exact as a double, and u / p there is off by less than
// 1/2, so the truncated quotient is off by at most one; the exact remainder
// says which way.  (A 64-bit integer division is a sequence of over a hundred
// instructions.)  Taken as signed: windows also pass work left at an instant that
// they then do not choose, above -2^61, for which the conversion has to be defined.
__device__ __forceinline__ uint64_t ceil_p(uint64_t u, uint32_t p, double inv, double) {
    const uint64_t est = (uint64_t)(int64_t)((double)(int64_t)u * inv);
    const int64_t rem = (int64_t)(u - est * p);
    return est + (rem > 0 ? 1u : 0u) + (rem > (int64_t)p ? 1u : 0u);
}

template <typename TT>
__device__ __forceinline__ TT tmax(TT a, TT b) { return a > b ? a : b; }
template <typename TT>
__device__ __forceinline__ TT tmin(TT a, TT b) { return a < b ? a : b; }

template <typename TT>
__device__ __forceinline__ TT inf_time() { return ~TT(0); }

// Launch scheme a function is compiled for.
enum DmaMode : int { DMA_ONE = 1, DMA_TWO = 2 };

// Task tables and the per-lane kernel-completion queue.  Entry x of a table
// is at [x * TS], slot j of the queue at [j * QS] (compile-time strides);
// shared tables use TS = 1, per-lane tables interleave lanes so that a
// wave's accesses fall into distinct banks.
template <typename TT, int TS, int QS>
struct View {
    const Quad<TT> *H;  // (h, ceil(q h / p_h), k, d)
    const DRec<TT> *D;  // (d, ceil(q d / p_d), slack)
    Slot<TT> *Q;
    __device__ __forceinline__ Quad<TT> task(uint32_t x) const { return H[x * TS]; }
    __device__ __forceinline__ DRec<TT> d(uint32_t x) const { return D[x * TS]; }
    __device__ __forceinline__ Slot<TT> q(int j) const { return Q[j * QS]; }
    __device__ __forceinline__ void put(int j, Slot<TT> s) const { Q[j * QS] = s; }
    // the same queue memory holding chain entries (start, end) of DtH j
    __device__ __forceinline__ Span<TT> span(int j) const { return reinterpret_cast<const Span<TT> *>(Q)[j * QS]; }
    __device__ __forceinline__ void put_span(int j, Span<TT> e) const { reinterpret_cast<Span<TT> *>(Q)[j * QS] = e; }
};

// One DMA engine (Section 3.2, scheme for such devices): every HtD is queued
// on the one transfer engine before every DtH, so the HtDs run back to back
// at solo speed (two transfers never move data at the same time), kernels
// follow K_j = max(HtD_j end, K_{j-1} end) + k, and every DtH waits for the
// last HtD.  A window is the HtD alone; the DtHs are left to the tail.
template <typename TT>
struct Lane {
    using ST = typename Signed<TT>::type;
    TT t;     // end of the previous HtD (0 before the first)
    TT ck;    // end of the previous kernel
    TT dpre;  // sum of solo DtH durations of the positions placed so far
    ST emax;  // max over placed positions p of (K_p end - sum_{s<p} d_s)
};

template <typename TT>
__device__ __forceinline__ void lane_reset(Lane<TT> &s) {
    using ST = typename Signed<TT>::type;
    s.t = 0; s.ck = 0; s.dpre = 0;
    s.emax = (ST)(((TT)1) << (8 * sizeof(TT) - 1));  // most negative
}

template <int DMA = DMA_ONE, bool PUT = true, typename TT, typename ViewT>
__device__ __forceinline__ void window(Lane<TT> &s, int, uint32_t x, const ViewT &v, const Rates &) {
    static_assert(DMA == DMA_ONE, "a lane of the one-engine scheme");
    using ST = typename Signed<TT>::type;
    const Quad<TT> tx = v.task(x);
    s.t += tx.h;
    s.ck = tmax(s.t, s.ck) + tx.k;
    const ST e = (ST)s.ck - (ST)s.dpre;
    s.emax = e > s.emax ? e : s.emax;
    s.dpre += tx.d;
}

// Total time: the DtHs start when the last HtD ends (the engine is busy with
// HtDs until s.t), so it is
// max(s.t + sum d, max_p (K_p end + sum_{s >= p} d_s)) = max(s.t, emax) + dpre.
template <int DMA = DMA_ONE, typename TT>
__device__ __forceinline__ TT tail(const Lane<TT> &s, const Rates &) {
    static_assert(DMA == DMA_ONE, "a lane of the one-engine scheme");
    using ST = typename Signed<TT>::type;
    const ST e = (ST)s.t > s.emax ? (ST)s.t : s.emax;
    return (TT)(e + (ST)s.dpre);
}

// ------------------------------------------------------------ chain form
// Simulation state at the start of a window, two DMA engines.  The DtHs of
// positions < j are on the chain (entries in the queue); c is the first of
// them that may still run at t, and its entry is kept in registers.
template <typename TT>
struct CLane {
    using ST = typename Signed<TT>::type;
    TT t;       // now: end of the previous HtD (0 before the first)
    TT ck;      // end of the previous kernel
    ST emax;    // max over placed positions p of (K_p end - sum_{s<p} d_s)
    TT dpre;    // sum of solo DtH durations of the positions placed so far
    TT elast;   // end of the last DtH on the chain (0 while it is empty)
    TT cs, ce;  // start and end of DtH c (when c is on the chain)
    TT dcross;  // sum of solo DtH durations of the DtHs before c
    int c;      // chain cursor: every DtH before c ends by t
    bool run;   // the last window's HtD ended while DtH c ran
};

template <typename TT>
__device__ __forceinline__ void lane_reset(CLane<TT> &s) {
    using ST = typename Signed<TT>::type;
    s.t = 0; s.ck = 0;
    s.emax = (ST)(((TT)1) << (8 * sizeof(TT) - 1));  // most negative
    s.dpre = 0; s.elast = 0; s.cs = 0; s.ce = 0; s.dcross = 0;
    s.c = 0; s.run = false;
}

// Window j of the chain form: HtD of task x from s.t, against the DtHs on the
// chain.  The loop visits only DtHs that end before the HtD: in the busy state
// the HtD end estimate stays valid while DtHs follow each other without a gap;
// at a gap the exact remaining work gives the idle estimate, and a DtH that
// starts before it gives a new busy estimate.  Event order and roundings are
// those of stepping every event (an event at ev is processed when ev is
// before the current estimate).  PUT = false skips appending DtH j (the last
// position: no later window reads it).
template <int DMA = DMA_TWO, bool PUT = true, typename TT, int TS, int QS>
__device__ __forceinline__ void window(CLane<TT> &s, int j, uint32_t x, const View<TT, TS, QS> &v,
                                       const Rates &r) {
    static_assert(DMA == DMA_TWO, "the chain form models two DMA engines");
    using ST = typename Signed<TT>::type;
    const Quad<TT> tx = v.task(x);
    int i = s.c;
    TT S = s.cs, E = s.ce, dsum = s.dcross;
    TT rc = s.t;                  // last rate change
    TT u = tx.h << r.q_log2;      // HtD work left at rc, 1/q solo-ns
    TT eb;                        // HtD end estimate
    TT ecmp = E;                  // end of the running DtH; inf once the HtD end is final
    if (!(i < j)) {
        eb = s.t + tx.h;          // no DtH on the chain (first position)
        ecmp = inf_time<TT>();
    } else if (S < s.t) {
        eb = s.t + tx.hp;         // DtH c runs at t
    } else {
        const TT ei = s.t + tx.h;
        if (S < ei) {             // DtH c starts inside the window
            u -= (S - s.t) << r.q_log2;
            rc = S;
            eb = S + (TT)ceil_p(u, r.p_h, r.inv_ph, r.c_ph);
        } else {
            eb = ei;
            ecmp = inf_time<TT>();
        }
    }
    // One exit: while the running DtH ends before the estimate, it completes
    // and the next one on the chain follows, after a gap or without one.
    while (ecmp < eb) {
        // its solo time joins the crossed sum (p_dth dp = q d + slack, slack < q)
        dsum += (TT(r.p_d) * (E - S)) >> r.q_log2;
        const TT ep = E;
        ++i;
        const Span<TT> nx = v.span(i < j ? i : j - 1);  // slot j - 1 exists: i >= 1
        S = nx.s;
        E = nx.e;
        ecmp = E;
        if (!(i < j) || S != ep) {
            // the DtH engine goes idle at ep: exact work left, idle estimate;
            // the next DtH starts from idle if it begins before that estimate
            u -= TT(r.p_h) * (ep - rc);
            rc = ep;
            const TT ei = rc + ceil_q(u, r.q_log2);
            const bool start = i < j && S < ei;
            const TT us = u - ((S - rc) << r.q_log2);
            const TT ebs = S + (TT)ceil_p(us, r.p_h, r.inv_ph, r.c_ph);
            u = start ? us : u;
            rc = start ? S : rc;
            eb = start ? ebs : ei;
            ecmp = start ? ecmp : inf_time<TT>();
        }
    }
    const TT eh = eb;
    const bool run = ecmp != inf_time<TT>();
    s.c = i;
    s.cs = S;
    s.ce = E;
    s.dcross = dsum;
    s.run = run;
    s.t = eh;
    s.ck = tmax(eh, s.ck) + tx.k;
    const ST e = (ST)s.ck - (ST)s.dpre;
    s.emax = e > s.emax ? e : s.emax;
    s.dpre += tx.d;
    if constexpr (PUT) {
        // DtH j joins the chain: it starts once the engine and its kernel are done
        Span<TT> sp;
        sp.s = tmax(s.elast, s.ck);
        sp.e = sp.s + v.d(x).dp;
        v.put_span(j, sp);
        s.elast = sp.e;
        if (s.c == j) {
            s.cs = sp.s;
            s.ce = sp.e;
        }
    }
}

// Total time of the chain form once the last HtD has ended at s.t.  A DtH running at s.t has
// moved p_dth (s.t - start) of its q d work, so it needs
// d - floor(p_dth (s.t - start) / q) more ns at full speed, followed by the
// solo times of the DtHs after it.
template <int DMA = DMA_TWO, typename TT>
__device__ __forceinline__ TT tail(const CLane<TT> &s, const Rates &r) {
    static_assert(DMA == DMA_TWO, "the chain form models two DMA engines");
    using ST = typename Signed<TT>::type;
    TT T = (TT)(s.emax + (ST)s.dpre);
    if (s.run) {
        const TT dend = s.t + (s.dpre - s.dcross) - ((TT(r.p_d) * (s.t - s.cs)) >> r.q_log2);
        T = tmax(T, dend);
    }
    return T;
}

// ------------------------------------------------------- whole orderings
// Potential form: how far the HtD engine has come.  Let W(t) be the work it
// has done by t, in 1/q solo-ns, if it is never idle: W grows by q per ns while
// the DtH engine is idle and by p_htd while it runs, and the DtH of position i
// ends at E_i with W(E_i) = G_i.  Both follow when the position is placed:
// S = max(E_{i-1}, K_i), E_i = S + dp_i, G_i = G_{i-1} + q (S - E_{i-1}) + p_htd dp_i.
// An HtD of h ns that starts at t ends at the first instant with
// W >= X = W(t) + q h.  So a window only has to find the first DtH with
// G_i >= X: between E_{i-1} and E_i, W is the smaller of the line of slope q
// through (E_{i-1}, G_{i-1}) and the line of slope p_htd through (E_i, G_i)
// (q >= p_htd), so the HtD ends at the later of the two lines' crossings of X,
// rounded up -- the event windows' roundings, since every rate change falls on
// a whole ns.  No branch but the search, whose step is one LDS read and one
// comparison, where the chain form's loop divides at every gap: on random
// orderings the lanes of a wave disagree about nearly every branch (35 % of
// them active in the chain form, 196 VALU instructions per window).
//
// The potentials are below q T: the 32-bit form needs q times the group's time
// bound below 2^31, the 64-bit one below 2^51 (its quotients are taken in
// double); other groups take the chain form.

// Task x of the potential form: q h, k, d, dp, and p_htd dp beside it.
template <typename TT>
struct alignas(4 * sizeof(TT)) PRec {
    TT qh, k, d, dp;
};

// Tables of a lane that evaluates whole orderings, one after another, and its
// queue: G of n positions (the last only ever a sentinel) and E of n - 1 in the
// potential form; the kernel ends alone in the chain form.
template <typename TT, int QS>
struct OrderView {
    const Quad<TT> *H;
    const DRec<TT> *D;
    const PRec<TT> *P;
    const TT *gain;
    TT *Q;
    __device__ __forceinline__ Quad<TT> task(uint32_t x) const { return H[x]; }
};
template <typename TT>
__host__ __device__ constexpr size_t order_queue_bytes(int n, int threads) {
    return sizeof(TT) * (size_t)threads * (size_t)(2 * n - 1);
}

// The tables of up to MAXN tasks in LDS: a group takes one of the two forms.
template <typename TT>
struct OrderTables {
    union {
        struct {
            Quad<TT> H[MAXN];
            DRec<TT> D[MAXN];
        };
        struct {
            PRec<TT> P[MAXN];
            TT gain[MAXN];
        };
    };
    template <int QS>
    __device__ __forceinline__ OrderView<TT, QS> view(TT *q) const {
        return OrderView<TT, QS>{H, D, P, gain, q};
    }
};

// Whether a group with this time bound may take the potential form.
template <typename TT>
__device__ __forceinline__ bool potential_fits(uint64_t bound, const Rates &r) {
    return bound < (1ull << ((sizeof(TT) == 4 ? 31 : 51) - r.q_log2));
}

// floor(u / p): u < 2^32 as trunc(fma(u, 1/p, 1/(2p))) (as ceil_p); u < 2^51 by
// the exact remainder.
__device__ __forceinline__ uint32_t floor_p(uint32_t u, uint32_t, double inv) {
    return (uint32_t)__builtin_fma((double)u, inv, 0.5 * inv);
}
__device__ __forceinline__ uint64_t floor_p(uint64_t u, uint32_t p, double inv) {
    const uint64_t est = (uint64_t)((double)u * inv);
    const int64_t rem = (int64_t)(u - est * p);
    return est + (rem >= (int64_t)p ? 1u : 0u) - (rem < 0 ? 1u : 0u);
}

template <typename TT, int QS>
__device__ __forceinline__ TT simulate_potential(int n, uint64_t perm, const OrderView<TT, QS> &v, const Rates &r) {
    using ST = typename Signed<TT>::type;
    constexpr TT INF = ~TT(0) >> 1;  // above every potential
    const TT q1 = (TT(1) << r.q_log2) - 1;
    TT t = 0, w = 0, ck = 0, dpre = 0;
    ST emax = (ST)(((TT)1) << (8 * sizeof(TT) - 1));  // most negative
    TT gl = 0, el = 0;            // the last DtH placed
    TT gp = 0, ep = 0;            // the DtH before the cursor (none: the start)
    TT gc = INF, ec = 0;          // DtH i, the first that ends at t or later (INF: none placed)
    int i = 0;
    TT *const G = v.Q, *const E = v.Q + n * QS;
    uint64_t seq = perm;
    for (int j = 0; j < n; ++j, seq >>= 4) {
        const uint32_t x = (uint32_t)seq & 15u;
        const PRec<TT> tx = v.P[x];
        const TT X = w + tx.qh;
        while (gc < X) {
            gp = gc;
            ep = ec;
            ++i;
            gc = G[i * QS];  // slot j holds INF
            ec = E[(i < j ? i : j - 1) * QS];
        }
        const TT eq = ep + ((X - gp + q1) >> r.q_log2);
        const TT ek = ec - (TT)floor_p((TT)(gc - X), r.p_h, r.inv_ph);
        const bool live = gc != INF;
        t = live && (ST)ek > (ST)eq ? ek : eq;
        w = gp + ((t - ep) << r.q_log2);
        const TT wp = gc - TT(r.p_h) * (ec - t);
        w = live && wp < w ? wp : w;
        ck = tmax(t, ck) + tx.k;
        const ST e = (ST)ck - (ST)dpre;
        emax = e > emax ? e : emax;
        dpre += tx.d;
        if (j + 1 < n) {
            const TT S = tmax(el, ck);
            gl += ((S - el) << r.q_log2) + v.gain[x];
            el = S + tx.dp;
            G[j * QS] = gl;
            E[j * QS] = el;
            G[(j + 1) * QS] = INF;
            gc = live ? gc : gl;  // every earlier DtH has ended: DtH j is the cursor's
            ec = live ? ec : el;
        }
    }
    TT T = (TT)(emax + (ST)dpre);
    if (gc != INF) {
        // DtH i may run at t: its solo time less what it has moved, then the
        // solo times of the DtHs after it
        uint64_t cur = perm >> (4 * i);
        const TT S = ec - v.P[(uint32_t)cur & 15u].dp;
        if (S < t) {
            TT rest = 0;
            for (int s = i; s < n; ++s, cur >>= 4) rest += v.P[(uint32_t)cur & 15u].d;
            T = tmax(T, t + rest - ((TT(r.p_d) * (t - S)) >> r.q_log2));
        }
    }
    return T;
}

// T of one whole ordering (perm: the task at position j in nibble j): with one
// DMA engine its windows; with two the potential form, or
// (potential false: the group's potentials do not fit) the chain form's windows
// (CLane), the chain entries computed when the cursor reaches them.
template <typename TT, int QS>
__device__ __forceinline__ TT simulate_order(int n, uint64_t perm, const OrderView<TT, QS> &v, const Rates &r,
                                             bool potential) {
    using ST = typename Signed<TT>::type;
    if (potential) return simulate_potential(n, perm, v, r);
    if (r.one_dma) {
        Lane<TT> st;
        lane_reset(st);
        for (int j = 0; j < n; ++j) window(st, j, (uint32_t)(perm >> (4 * j)) & 15u, v, r);
        return tail(st, r);
    }
    TT t = 0, ck = 0, dpre = 0, dcross = 0;
    ST emax = (ST)(((TT)1) << (8 * sizeof(TT) - 1));  // most negative
    // the cursor: DtH i of solo time dc, from S to E while the HtD engine is busy
    int i = 0;
    TT S = 0, E = 0, dc = 0;
    bool run = false;
    uint64_t seq = perm;
    for (int j = 0; j < n; ++j, seq >>= 4) {
        const uint32_t x = (uint32_t)seq & 15u;
        const Quad<TT> tx = v.task(x);
        TT rc = t;
        TT u = tx.h << r.q_log2;
        TT eb, ecmp = E;
        if (!(i < j)) {
            eb = t + tx.h;
            ecmp = inf_time<TT>();
        } else if (S < t) {
            eb = t + tx.hp;
        } else {
            const TT ei = t + tx.h;
            if (S < ei) {
                u -= (S - t) << r.q_log2;
                rc = S;
                eb = S + (TT)ceil_p(u, r.p_h, r.inv_ph, r.c_ph);
            } else {
                eb = ei;
                ecmp = inf_time<TT>();
            }
        }
        while (ecmp < eb) {
            dcross += dc;
            const TT ep = E;
            ++i;
            const DRec<TT> y = v.D[(uint32_t)(perm >> (4 * i)) & 15u];
            S = tmax(ep, v.Q[(i < j ? i : j - 1) * QS]);  // slot j - 1 exists: i >= 1
            E = S + y.dp;
            dc = y.d;
            ecmp = E;
            if (!(i < j) || S != ep) {
                u -= TT(r.p_h) * (ep - rc);
                rc = ep;
                const TT ei = rc + ceil_q(u, r.q_log2);
                const bool start = i < j && S < ei;
                const TT us = u - ((S - rc) << r.q_log2);
                const TT ebs = S + (TT)ceil_p(us, r.p_h, r.inv_ph, r.c_ph);
                u = start ? us : u;
                rc = start ? S : rc;
                eb = start ? ebs : ei;
                ecmp = start ? ecmp : inf_time<TT>();
            }
        }
        run = ecmp != inf_time<TT>();
        t = eb;
        ck = tmax(eb, ck) + tx.k;
        const ST e = (ST)ck - (ST)dpre;
        emax = e > emax ? e : emax;
        dpre += tx.d;
        if (j + 1 < n) v.Q[j * QS] = ck;
        if (i == j) {  // every earlier DtH has ended: DtH j starts when its kernel ends
            S = ck;
            E = ck + v.D[x].dp;
            dc = tx.d;
        }
    }
    TT T = (TT)(emax + (ST)dpre);
    if (run) {
        const TT dend = t + (dpre - dcross) - ((TT(r.p_d) * (t - S)) >> r.q_log2);
        T = tmax(T, dend);
    }
    return T;
}

// Host-side validity bound for the 32-bit time path (checked on the device
// from the task table): every work amount fits 31 bits and every instant of
// the simulation fits 31 bits.  T never exceeds the sum of each command's
// slowest duration plus one ns of rounding per rate change per command.
__host__ __device__ inline uint64_t time_bound_slack(int n) { return 3ull * n * (2ull * n + 2ull); }

}  // namespace tgo
