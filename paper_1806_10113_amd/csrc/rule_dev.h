// Lanes under a start rule: the temporal model (model_dev.h) where a command
// may have to wait for more than its engine and its own task.
//
//   GATED (two DMA engines): the HtD of position j starts only once the DtHs
//     of the first g_j positions have ended (device memory: the buffers that
//     must be free again; dependent tasks: the worker's previous task).  The
//     gate depends on the ordering alone, not on times.
//   CONCURRENT: the kernel of position j starts once its HtD has ended, the
//     kernel before it has started and its units fit beside those of the
//     kernels still running (model of csrc/cke.hip).
//
// Both keep the window formulation.  DtHs still run in launch order, each
// once its kernel has ended, so DtH i starts at S_i = max(E_{i-1}, K_i) and,
// while the HtD engine is busy, ends at E_i = S_i + ceil(q d_i / p_dth).
// Unlike the chain form (CLane) the entries are not computed when a position
// is placed but when the cursor reaches them, from slot i = (end of K_i,
// overlapped duration): a gate leaves the HtD engine idle, DtHs then run at
// full speed, and every later entry moves.  While an HtD waits at its gate,
// only the DtH that runs at that instant has moved at two rates: it has
// p_dth (E - t) - slack work left and ends ceil(that / q) later; the others
// up to the gate take their solo time, and the HtD starts exactly when one of
// them ends, so no DtH runs then.  Kernel ends need no events either way: they
// are fixed when their HtD has ended.
#pragma once

#include "model_dev.h"

namespace tgo {

enum RuleKind : int { RULE_MEMORY, RULE_CONCURRENT, RULE_ROUNDS };

__device__ __forceinline__ uint32_t nibble(uint64_t v, int i) { return (uint32_t)(v >> (4 * i)) & 15u; }

// Tables of a lane under a rule: the tasks', the queue, the task at each
// placed position (one nibble each; nibbles at and past the position being
// placed are stale), and what the rule reads.
template <typename TT, int TS, int QS, int KIND>
struct RView : View<TT, TS, QS> {
    uint64_t *seq;
    const int32_t *units;  // CONCURRENT: units per task, and the device's
    int32_t cap;
    const uint32_t *fits;  // MEMORY: bit s = the tasks of set s fit together
    uint64_t pos;          // ROUNDS: position of each placed task of an earlier round (one nibble each)
    uint32_t dep;          // ROUNDS: bit x = task x waits for the end of task x - 1
    uint32_t opens;        // ROUNDS, one engine: bit j = position j opens a round's sub-group
};

template <typename TT, int KIND>
struct RLane {
    using ST = typename Signed<TT>::type;
    TT t;       // now: end of the previous HtD (0 before the first)
    TT ck;      // end of the previous kernel (CONCURRENT: its start)
    TT ke;      // end of the previous kernel
    ST emax;    // max over placed positions p of (K_p end - sum_{s<p} d_s)
    TT dpre;    // sum of solo DtH durations of the positions placed so far
    TT cs, ce;  // DtH c: start, end while the HtD engine is busy (c placed)
    TT dcross;  // sum of solo DtH durations of the DtHs before c
    int c;      // cursor: every DtH before c ends by t
    bool run;   // the last window's HtD ended while DtH c ran or as it started
    // MEMORY: positions a .. hold their buffers, as a set of tasks;
    // CONCURRENT: positions whose kernels may still run, and their units
    uint32_t held;
    int32_t a;
};

template <typename TT, int KIND>
__device__ __forceinline__ void lane_reset(RLane<TT, KIND> &s) {
    using ST = typename Signed<TT>::type;
    s.t = 0; s.ck = 0; s.ke = 0;
    s.emax = (ST)(((TT)1) << (8 * sizeof(TT) - 1));  // most negative
    s.dpre = 0; s.cs = 0; s.ce = 0; s.dcross = 0;
    s.c = 0; s.run = false;
    s.held = 0; s.a = 0;
}

// The positions whose DtHs must have ended before the HtD of task x may start
// at position j: [0, returned).
template <int KIND, typename TT, typename ViewT>
__device__ __forceinline__ int gate(RLane<TT, KIND> &s, int j, uint32_t x, const ViewT &v) {
    if constexpr (KIND == RULE_MEMORY) {
        // drop the oldest holders until the set with x fits (x alone does)
        uint32_t set = s.held | (1u << x);
        while (s.a < j && !((v.fits[set >> 5] >> (set & 31u)) & 1u)) {
            set &= ~(1u << nibble(*v.seq, s.a));
            ++s.a;
        }
        s.held = set;
        return s.a;
    } else if constexpr (KIND == RULE_ROUNDS) {
        return (v.dep >> x) & 1u ? (int)nibble(v.pos, (int)x - 1) + 1 : 0;
    } else {
        return 0;
    }
}

// The HtD engine waits from s.t until DtH g - 1 has ended (s.c < g <= j).
template <int KIND, typename TT, typename ViewT>
__device__ __forceinline__ void wait_gate(RLane<TT, KIND> &s, int g, int j, const ViewT &v, const Rates &r) {
    const TT q = TT(1) << r.q_log2;
    int i = s.c;
    // p_dth dp = q d + slack with slack < q
    TT w = TT(r.p_d) * v.q(i).dp;
    TT e;
    if (s.cs < s.t) {
        const TT pw = TT(r.p_d) * (s.ce - s.t), slack = w & (q - 1);
        e = s.t + ceil_q(pw > slack ? pw - slack : TT(0), r.q_log2);
    } else {
        e = s.cs + (w >> r.q_log2);
    }
    TT dsum = s.dcross + (w >> r.q_log2);
    for (++i; i < g; ++i) {
        const Slot<TT> sl = v.q(i);
        const TT d = (TT(r.p_d) * sl.dp) >> r.q_log2;
        e = tmax(e, sl.ck) + d;
        dsum += d;
    }
    s.t = e;
    s.dcross = dsum;
    s.c = i;
    const Slot<TT> nx = v.q(i < j ? i : j - 1);
    s.cs = tmax(e, nx.ck);
    s.ce = s.cs + nx.dp;
}

// Start of the kernel of position j (task x) no earlier than `from`: the
// first instant its units fit beside those of the kernels still running.
// s.held keeps positions whose kernels may still run and s.a their units;
// kernels that have ended are dropped only when that is needed to fit.
template <typename TT, typename ViewT>
__device__ __forceinline__ TT dispatch(RLane<TT, RULE_CONCURRENT> &s, TT from, int32_t ux, const ViewT &v) {
    TT at = from;
    if (s.a > v.cap - ux) {
        for (;;) {
            TT next = inf_time<TT>();
            for (uint32_t m = s.held; m; m &= m - 1) {
                const int p = __ffs(m) - 1;
                const TT e = v.q(p).ck;
                if (e <= at) {
                    s.held &= ~(1u << p);
                    s.a -= v.units[nibble(*v.seq, p)];
                } else {
                    next = e < next ? e : next;
                }
            }
            if (s.a <= v.cap - ux) break;
            at = next;  // every round drops at least one kernel, and ux <= cap
        }
    }
    return at;
}

// The kernel of position j (its HtD ends at s.t): its end, kept for the
// reduction terms and, with PUT, for later positions.
template <bool PUT, int KIND, typename TT, typename ViewT>
__device__ __forceinline__ void place_kernel(RLane<TT, KIND> &s, int j, uint32_t x, const Quad<TT> &tx,
                                             const ViewT &v) {
    using ST = typename Signed<TT>::type;
    if constexpr (KIND == RULE_CONCURRENT) {
        const int32_t ux = v.units[x];
        s.ck = dispatch(s, tmax(s.t, s.ck), ux, v);
        s.ke = s.ck + tx.k;
        if constexpr (PUT) {
            s.held |= 1u << j;
            s.a += ux;
        }
    } else {
        s.ck = tmax(s.t, s.ck) + tx.k;
        s.ke = s.ck;
    }
    const ST e = (ST)s.ke - (ST)s.dpre;
    s.emax = e > s.emax ? e : s.emax;
    s.dpre += tx.d;
    if constexpr (PUT && KIND != RULE_ROUNDS) *v.seq = (*v.seq & ~(15ull << (4 * j))) | ((uint64_t)x << (4 * j));
}

// Window j: HtD of task x, started from s.t or from its gate, against the
// DtHs placed before; the event order and roundings of CLane's window.
// PUT = false: the last position, nothing is kept for later ones.
template <int DMA, bool PUT = true, typename TT, int KIND, typename ViewT>
__device__ __forceinline__ void window(RLane<TT, KIND> &s, int j, uint32_t x, const ViewT &v, const Rates &r) {
    const Quad<TT> tx = v.task(x);
    if constexpr (DMA == DMA_ONE) {
        // every HtD before every DtH on the one engine: no overlap
        static_assert(KIND == RULE_CONCURRENT || DMA != DMA_ONE, "one engine: sub-groups, not gates");
        s.t += tx.h;
        place_kernel<PUT>(s, j, x, tx, v);
        if constexpr (PUT) {
            Slot<TT> sl;
            sl.ck = s.ke;
            sl.dp = 0;
            v.put(j, sl);
        }
    } else {
        if constexpr (KIND != RULE_CONCURRENT) {
            const int g = gate<KIND>(s, j, x, v);
            if (s.c < g) wait_gate(s, g, j, v, r);
        }
        int i = s.c;
        TT S = s.cs, E = s.ce, dsum = s.dcross;
        TT rc = s.t;              // last rate change
        TT u = tx.h << r.q_log2;  // HtD work left at rc, 1/q solo-ns
        TT eb;                    // HtD end estimate
        TT ecmp = E;              // end of the running DtH; inf once the HtD end is final
        if (!(i < j)) {
            eb = s.t + tx.h;      // no DtH left among the placed positions
            ecmp = inf_time<TT>();
        } else if (S < s.t) {
            eb = s.t + tx.hp;     // DtH c runs at t
        } else {
            const TT ei = s.t + tx.h;
            if (S < ei) {         // DtH c starts inside the window
                u -= (S - s.t) << r.q_log2;
                rc = S;
                eb = S + (TT)ceil_p(u, r.p_h, r.inv_ph, r.c_ph);
            } else {
                eb = ei;
                ecmp = inf_time<TT>();
            }
        }
        while (ecmp < eb) {
            dsum += (TT(r.p_d) * (E - S)) >> r.q_log2;
            const TT ep = E;
            ++i;
            const Slot<TT> nx = v.q(i < j ? i : j - 1);  // slot j - 1 exists: i >= 1
            S = tmax(ep, nx.ck);
            E = S + nx.dp;
            ecmp = E;
            if (!(i < j) || S != ep) {
                // the DtH engine goes idle at ep (CLane's window)
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
        s.run = ecmp != inf_time<TT>();
        // an HtD without length right behind its gate: DtH c takes the engine
        // at that same instant
        if constexpr (KIND != RULE_CONCURRENT) s.run = s.run || (i < j && S <= eb);
        s.c = i;
        s.cs = S;
        s.ce = E;
        s.dcross = dsum;
        s.t = eb;
        place_kernel<PUT>(s, j, x, tx, v);
        if constexpr (PUT) {
            Slot<TT> sl;
            sl.ck = s.ke;
            sl.dp = v.d(x).dp;
            v.put(j, sl);
            if (s.c == j) {  // every earlier DtH has ended: DtH j starts when its kernel ends
                s.cs = sl.ck;
                s.ce = sl.ck + sl.dp;
            }
        }
    }
}

// Total time once the last placed HtD has ended (CLane's and the one-engine
// tail: from then on every DtH takes its solo time, in launch order).
template <int DMA, typename TT, int KIND>
__device__ __forceinline__ TT tail(const RLane<TT, KIND> &s, const Rates &r) {
    using ST = typename Signed<TT>::type;
    if constexpr (DMA == DMA_ONE) {
        const ST e = (ST)s.t > s.emax ? (ST)s.t : s.emax;
        return (TT)(e + (ST)s.dpre);
    } else {
        TT T = (TT)(s.emax + (ST)s.dpre);
        if (s.run) {
            const TT dend = s.t + (s.dpre - s.dcross) - ((TT(r.p_d) * (s.t - s.cs)) >> r.q_log2);
            T = tmax(T, dend);
        }
        return T;
    }
}

// One DMA engine, the ordering cut into consecutive sub-groups, each launched
// as its HtDs, then its DtHs, behind the previous one (MEMORY: as long as its
// buffers fit together; ROUNDS: one per round, whose DtHs all end before the
// next round's HtDs, so no dependency ever waits).  Transfers never overlap:
// HtDs back to back, K_i = max(HtD_i end, K_{i-1} end) + k_i, and the
// sub-group's DtHs end at max(last HtD end, max_p (K_p - sum_{s<p} d_s)) + sum d.
template <typename TT, int KIND>
struct SubChain {
    using ST = typename Signed<TT>::type;
    TT x;          // end of the open sub-group's last HtD (none open: of the last DtH)
    TT kp;         // end of the last kernel
    ST emax;       // open sub-group: max of (K_p end - its DtH time before p)
    TT dsum;       // open sub-group: its DtH time so far
    uint32_t set;  // MEMORY: the open sub-group's tasks
};
template <typename TT, int KIND>
__device__ __forceinline__ void lane_reset(SubChain<TT, KIND> &s) {
    using ST = typename Signed<TT>::type;
    s.x = s.kp = s.dsum = 0;
    s.emax = (ST)(((TT)1) << (8 * sizeof(TT) - 1));  // most negative
    s.set = 0;
}
template <int DMA, typename TT, int KIND>
__device__ __forceinline__ TT tail(const SubChain<TT, KIND> &s, const Rates &) {
    using ST = typename Signed<TT>::type;
    const ST e = (ST)s.x > s.emax ? (ST)s.x : s.emax;
    return (TT)(e + (ST)s.dsum);
}
template <int DMA, bool PUT = true, typename TT, int KIND, typename ViewT>
__device__ __forceinline__ void window(SubChain<TT, KIND> &s, int j, uint32_t x, const ViewT &v, const Rates &r) {
    using ST = typename Signed<TT>::type;
    const Quad<TT> tx = v.task(x);
    bool close;
    if constexpr (KIND == RULE_MEMORY) {
        // x alone fits, so the first task of a sub-group never closes one
        const uint32_t set = s.set | (1u << x);
        close = !((v.fits[set >> 5] >> (set & 31u)) & 1u);
        s.set = close ? 1u << x : set;
    } else {
        close = (v.opens >> j) & 1u;
    }
    s.x = (close ? tail<DMA>(s, r) : s.x) + tx.h;
    s.kp = tmax(s.x, s.kp) + tx.k;
    const TT before = close ? TT(0) : s.dsum;
    const ST e = (ST)s.kp - (ST)before;
    s.emax = close ? e : (e > s.emax ? e : s.emax);
    s.dsum = before + tx.d;
}

}  // namespace tgo
