// The potential form (model_dev.h, simulate_potential) for the enumeration
// kernel: the windows of a walk, 32-bit time.
//
// A lane's queue holds, per placed position, G_i and E_i of its DtH and, in a
// byte, the rounding slack of the DtHs before it.  What a window needs of the DtH
// before its cursor it reads after the search, so the state saved at each level of
// the walk is seven words (the chain form's is ten) and the search itself is one
// LDS read and one comparison per DtH.
//
// A DtH that runs when the last HtD ends at t has moved p_dth (t - S_i) of its
// work.  With P_i = sum_{s<=i} dp_s, the time the DtH engine has stood idle
// before E_i is E_i - P_i, and q times the solo time of the DtHs before i is
// p_dth P_{i-1} less their slack (p_dth dp = q d + slack), so the total time is
//   t + sum d - floor((p_dth (t - E_i + P_i) - slack before i) / q),
// and P_i = (q E_i - G_i) / (q - p_htd), exactly: a shift and a multiplication by
// the inverse of the odd part modulo 2^32.  (If DtH i has not started by t, this
// is a lower bound that another term of the maximum already reaches.)  The form
// therefore needs p_htd < q, slack sums below 256 and, as everywhere, q times
// the group's time bound below 2^31.
//
// What bounds it: instruction issue and the chain of LDS reads of the search,
// about evenly.  Three groups of 12 (479 M orderings each), five tasks left at the
// root of a walk: chain form 2165 / 2011 / 2551 us (a group's time follows the
// length of its searches and, there, how often the lanes of a wave part), potential
// form 1782 / 1712 / 1744 us.  Slots of 8 bytes hold five waves per SIMD at 12
// tasks; potentials and ends in arrays of their own, without the last end, hold six
// but read twice as often and select the origin: 1855 / 1823 / 1842.  The slack
// bytes in the last slot's spare word hold six, too, and spill: 1960 / 1826 / 1845.
// The DtH before taken along in the search: 1845 / 1777 / 1817 (it spills).
#pragma once

#include "enum_kernel.h"

namespace tgo {

constexpr uint32_t POT_INF = 0x7fffffffu;  // above every potential

// A placed DtH: its potential and its end, one 8-byte LDS access.
struct PotSlot {
    uint32_t g, e;
};

template <int QS>
struct PotView {
    const Quad<uint32_t> *H;  // (q h, k, d, dp) of a task
    const DRec<uint32_t> *D;  // (p_htd dp, slack)
    PotSlot *Q;               // slot i at [i * QS]
    const PotSlot *zero;      // the slot before the first: the origin (one for the block)
    uint8_t *S;               // at [i * QS]
};

struct PotLane {
    uint32_t t;     // now: end of the previous HtD
    uint32_t w;     // HtD potential at t
    uint32_t ck;    // end of the previous kernel
    int32_t emax;   // max over placed positions p of (K_p end - sum_{s<p} d_s)
    uint32_t dpre;  // sum of solo DtH durations of the positions placed so far
    uint32_t sig;   // sum of their slacks
    int i;          // cursor times QS: the first DtH that ends at t or later
    // the last position's window: DtH i (g = POT_INF: none), its slack byte
    uint32_t g, e, s;
};

__device__ __forceinline__ void lane_reset(PotLane &s) {
    s.t = s.w = s.ck = s.dpre = s.sig = 0;
    s.emax = INT32_MIN;
    s.i = 0;
    s.g = POT_INF;
    s.e = s.s = 0;
}

template <int DMA, bool PUT = true, int QS>
__device__ __forceinline__ void window(PotLane &s, int j, uint32_t x, const PotView<QS> &v, const Rates &r) {
    const Quad<uint32_t> tx = v.H[x];  // (q h, k, d, dp)
    const uint32_t X = s.w + tx.h;
    int i = s.i;
    // the search stops at slot j: what a sibling of this position left there is
    // cleared (the last position's slot never holds anything else)
    if constexpr (PUT) v.Q[j * QS].g = POT_INF;
    PotSlot c = v.Q[i];
    while (c.g < X) c = v.Q[i += QS];
    // the lines of slope q through the DtH before and of slope p_htd through
    // DtH i; the origin before the first one
    const PotSlot p = *(i > 0 ? v.Q + (i - QS) : v.zero);
    const uint32_t eq = p.e + ((X + ((1u << r.q_log2) - 1u) - p.g) >> r.q_log2);
    const uint32_t ek = c.e - (__umulhi(c.g - X, r.phm) >> r.phs);
    const bool live = c.g != POT_INF;
    const uint32_t t = live && (int32_t)ek > (int32_t)eq ? ek : eq;
    s.ck = tmax(t, s.ck) + tx.hp;
    const int32_t e = (int32_t)s.ck - (int32_t)s.dpre;
    s.emax = e > s.emax ? e : s.emax;
    s.dpre += tx.k;
    s.t = t;
    if constexpr (PUT) {
        const uint32_t wq = p.g + ((t - p.e) << r.q_log2), wp = c.g - r.p_h * (c.e - t);
        s.w = live && wp < wq ? wp : wq;
        s.i = i;
        const DRec<uint32_t> dx = v.D[x];
        const PotSlot l = *(j > 0 ? v.Q + (j - 1) * QS : v.zero);
        const uint32_t S = tmax(l.e, s.ck);
        PotSlot o;
        o.g = l.g + ((S - l.e) << r.q_log2) + dx.d;
        o.e = S + tx.d;
        v.Q[j * QS] = o;
        v.S[j * QS] = (uint8_t)s.sig;
        s.sig += dx.dp;
    } else {
        s.g = c.g;
        s.e = c.e;
        s.s = v.S[live ? i : 0];
    }
}

// Total time (only the last position's window leaves what it needs).
template <int DMA>
__device__ __forceinline__ uint32_t tail(const PotLane &s, const Rates &r) {
    uint32_t T = (uint32_t)(s.emax + (int32_t)s.dpre);
    const uint32_t P = (((s.e << r.q_log2) - s.g) >> r.dsh) * r.dinv;
    const int32_t moved = (int32_t)(r.p_d * (s.t - s.e + P) - s.s) >> r.q_log2;
    const uint32_t run = s.t + s.dpre - (uint32_t)moved;
    return s.g != POT_INF ? tmax(T, run) : T;
}

// The temporal model alone in the potential form (host: pot_rates).
struct PotRule : GroupRule {
    struct Args {};
    static constexpr bool SIDE = false;
    template <typename TT>
    using View = PotView<EX_THREADS>;
    template <typename TT, int DMA>
    using Lane = PotLane;
    template <typename TT, int DMA>
    static constexpr int min_waves() { return 5; }
    template <typename TT>
    static constexpr int mode() { return 2; }
    static constexpr bool queue(bool) { return true; }
    static __host__ __device__ constexpr size_t lds_bytes(int) { return sizeof(Quad<uint32_t>); }  // the origin
    template <typename TT>
    static __host__ __device__ constexpr size_t lane_bytes(int n) {
        return sizeof(PotSlot) * n + (size_t)(n > 1 ? n - 1 : 1);
    }
    template <typename TT>
    static __device__ __forceinline__ void bind(PotView<EX_THREADS> &v, unsigned char *queue, int n) {
        PotSlot *q = reinterpret_cast<PotSlot *>(queue), *zero = reinterpret_cast<PotSlot *>(queue - sizeof(Quad<TT>));
        v.Q = q + threadIdx.x;
        v.S = queue + sizeof(PotSlot) * EX_THREADS * n + threadIdx.x;
        v.Q[(n - 1) * EX_THREADS].g = POT_INF;
        v.zero = zero;
        if (threadIdx.x == 0) zero->g = zero->e = 0;
    }
    template <typename TT>
    static __device__ __forceinline__ void entry(const tgo_task &t, const Rates &r, Quad<TT> *H, DRec<TT> *D) {
        Quad<TT> h;
        DRec<TT> d;
        table_entry<TT>(t, r, &h, &d);
        H->h = h.h << r.q_log2;
        H->hp = h.k;
        H->k = h.d;
        H->d = d.dp;
        D->d = r.p_h * d.dp;
        D->dp = d.slack;
        D->slack = D->pad = 0;
    }
    template <bool SMALL, typename ViewT>
    static __device__ __forceinline__ void load(ViewT &, unsigned char *, const Args &, int, uint64_t *) {}
};

// Whether the rates allow the form for groups of n tasks.
__host__ __device__ inline bool pot_rates(const Rates &r, int n) {
    return !r.one_dma && r.p_h > 1 && r.p_h < (1u << r.q_log2) && (uint64_t)(n > 2 ? n - 2 : 0) * (r.p_d - 1) < 256;
}

}  // namespace tgo
