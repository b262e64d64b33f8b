// The potential form (model_dev.h, simulate_potential) for the enumeration
// kernel: the windows of a walk, 32-bit time.
//
// A lane's queue holds, per placed position, G_i and E_i of its DtH and, in a
// byte, the rounding slack of the DtHs before it.  What a window needs of them
// it reads after the search, so the state saved at each level of the walk is
// seven words (the chain form's is ten) and the search itself is one LDS read
// and one comparison per DtH.
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
// about evenly (171 vector instructions and 33 LDS accesses per ordering; the
// vector units issue in 59% of the cycles).  Three groups of 12 (479 M orderings
// each), five tasks left at the root of a walk: chain form 2165 / 2011 / 2551 us
// (a group's time follows the length of its searches and, there, how often the
// lanes of a wave part), potential form 1855 / 1823 / 1842 us at 6 waves per
// SIMD, 1959 / 1933 / 1959 at 5, 1914 / 1864 / 1887 at 7 (spills).
#pragma once

#include "enum_kernel.h"

namespace tgo {

constexpr uint32_t POT_INF = 0x7fffffffu;  // above every potential

template <int QS>
struct PotView {
    const Quad<uint32_t> *H;  // (q h, k, d, dp) of a task
    const DRec<uint32_t> *D;  // (p_htd dp, slack)
    uint32_t *G, *E;          // slot i at [i * QS]
    uint8_t *S;
};

struct PotLane {
    uint32_t t;     // now: end of the previous HtD
    uint32_t w;     // HtD potential at t
    uint32_t ck;    // end of the previous kernel
    int32_t emax;   // max over placed positions p of (K_p end - sum_{s<p} d_s)
    uint32_t dpre;  // sum of solo DtH durations of the positions placed so far
    uint32_t sig;   // sum of their slacks
    int i;          // cursor: the first DtH that ends at t or later
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
    if constexpr (PUT) v.G[j * QS] = POT_INF;
    uint32_t gc = v.G[i * QS];
    while (gc < X) gc = v.G[++i * QS];
    // the lines of slope q through the DtH before and of slope p_htd through
    // DtH i; the origin before the first one
    const bool live = gc != POT_INF;
    const int b = i > 0 ? i - 1 : 0;
    uint32_t gp = v.G[b * QS], ep = v.E[b * QS];
    const int ci = live ? i : b;
    const uint32_t ec = v.E[ci * QS];
    gp = i > 0 ? gp : 0;
    ep = i > 0 ? ep : 0;
    const uint32_t eq = ep + ((X - gp + ((1u << r.q_log2) - 1u)) >> r.q_log2);
    const uint32_t ek = ec - floor_p(gc - X, r.p_h, r.inv_ph);
    const uint32_t t = live && (int32_t)ek > (int32_t)eq ? ek : eq;
    s.ck = tmax(t, s.ck) + tx.hp;
    const int32_t e = (int32_t)s.ck - (int32_t)s.dpre;
    s.emax = e > s.emax ? e : s.emax;
    s.dpre += tx.k;
    s.t = t;
    if constexpr (PUT) {
        const uint32_t wq = gp + ((t - ep) << r.q_log2), wp = gc - r.p_h * (ec - t);
        s.w = live && wp < wq ? wp : wq;
        s.i = i;
        const DRec<uint32_t> dx = v.D[x];
        const uint32_t gl = j > 0 ? v.G[(j - 1) * QS] : 0u, el = j > 0 ? v.E[(j - 1) * QS] : 0u;
        const uint32_t S = tmax(el, s.ck);
        v.G[j * QS] = gl + ((S - el) << r.q_log2) + dx.d;
        v.E[j * QS] = S + tx.d;
        v.S[j * QS] = (uint8_t)s.sig;
        s.sig += dx.dp;
    } else {
        s.g = gc;
        s.e = ec;
        s.s = v.S[ci * QS];
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
    static constexpr int min_waves() { return 6; }
    template <typename TT>
    static constexpr int mode() { return 2; }
    static constexpr bool queue(bool) { return true; }
    static __host__ __device__ constexpr size_t lds_bytes(int) { return 0; }
    template <typename TT>
    static __host__ __device__ constexpr size_t lane_bytes(int n) {
        return (size_t)(4 * n + 5 * (n > 1 ? n - 1 : 1));
    }
    template <typename TT>
    static __device__ __forceinline__ void bind(PotView<EX_THREADS> &v, unsigned char *queue, int n) {
        const int m = n > 1 ? n - 1 : 1;
        v.G = reinterpret_cast<uint32_t *>(queue) + threadIdx.x;
        v.E = v.G + n * EX_THREADS;
        v.S = queue + (size_t)4 * EX_THREADS * (n + m) + threadIdx.x;
        v.G[(n - 1) * EX_THREADS] = POT_INF;
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
inline bool pot_rates(const Rates &r, int n) {
    return !r.one_dma && r.p_h < (1u << r.q_log2) && (uint64_t)(n > 2 ? n - 2 : 0) * (r.p_d - 1) < 256;
}

}  // namespace tgo
