// Task-table loading and validation on the device.
#pragma once

#include "../../include/tgo.h"
#include "enum_dev.h"
#include "model_dev.h"

namespace tgo {

// 0 = every instant and work amount fits the 32-bit path, 1 = 64-bit path,
// TGO_ERANGE = a duration is negative or >= 2^40 ns.
__device__ inline int classify_group(const tgo_task *t, int n, const Rates &r, uint64_t *bound = nullptr) {
    const uint64_t q = 1ull << r.q_log2;
    uint64_t mx = 0, sum = 0;
    for (int i = 0; i < n; ++i) {
        const int64_t h = t[i].htd_ns, k = t[i].kern_ns, d = t[i].dth_ns;
        const int64_t lim = int64_t(1) << 40;
        if (h < 0 || k < 0 || d < 0 || h >= lim || k >= lim || d >= lim) return TGO_ERANGE;
        const uint64_t qh = q * (uint64_t)h, qd = q * (uint64_t)d;
        mx = qh > mx ? qh : mx;
        mx = qd > mx ? qd : mx;
        sum += ceil_p(qh, r.p_h, r.inv_ph, r.c_ph) + (uint64_t)k + ceil_p(qd, r.p_d, r.inv_pd, r.c_pd);
    }
    if (bound) *bound = sum + time_bound_slack(n);
    const uint64_t lim32 = 1ull << 31;
    return (mx < lim32 && sum + time_bound_slack(n) < lim32) ? 0 : 1;
}

// The group's status as classify_group computes it, with one lane per task
// (the per-task terms are combined by wave reductions; same result).
__device__ inline int classify_group_wave(const tgo_task *t, int n, const Rates &r, int lane,
                                          uint64_t *bound = nullptr) {
    const uint64_t q = 1ull << r.q_log2;
    int bad = 0;
    uint64_t mx = 0, sum = 0;
    if (lane < n) {
        const int64_t h = t[lane].htd_ns, k = t[lane].kern_ns, d = t[lane].dth_ns;
        const int64_t lim = int64_t(1) << 40;
        if (h < 0 || k < 0 || d < 0 || h >= lim || k >= lim || d >= lim) {
            bad = 1;
        } else {
            const uint64_t qh = q * (uint64_t)h, qd = q * (uint64_t)d;
            mx = qh > qd ? qh : qd;
            sum = ceil_p(qh, r.p_h, r.inv_ph, r.c_ph) + (uint64_t)k + ceil_p(qd, r.p_d, r.inv_pd, r.c_pd);
        }
    }
    for (int m = 32; m >= 1; m >>= 1) {
        bad |= __shfl_xor(bad, m);
        const uint64_t mx2 = shfl_xor64(mx, m);
        mx = mx2 > mx ? mx2 : mx;
        sum += shfl_xor64(sum, m);
    }
    if (bound) *bound = sum + time_bound_slack(n);
    if (bad) return TGO_ERANGE;
    const uint64_t lim32 = 1ull << 31;
    return (mx < lim32 && sum + time_bound_slack(n) < lim32) ? 0 : 1;
}

// Entry x of the tables from task t: (h, ceil(q h/p_h), k, d) and
// (d, ceil(q d/p_d), p_d ceil(q d/p_d) - q d).
template <typename TT>
__device__ inline void table_entry(const tgo_task &t, const Rates &r, Quad<TT> *H, DRec<TT> *D) {
    const uint64_t q = 1ull << r.q_log2;
    const uint64_t h = (uint64_t)t.htd_ns, k = (uint64_t)t.kern_ns, d = (uint64_t)t.dth_ns;
    Quad<TT> e;
    e.h = (TT)h;
    e.hp = (TT)ceil_p(q * h, r.p_h, r.inv_ph, r.c_ph);
    e.k = (TT)k;
    e.d = (TT)d;
    DRec<TT> pd;
    const uint64_t dp = ceil_p(q * d, r.p_d, r.inv_pd, r.c_pd);
    pd.d = (TT)d;
    pd.dp = (TT)dp;
    pd.slack = (TT)(r.p_d * dp - q * d);
    pd.pad = 0;
    *H = e;
    *D = pd;
}

// Entry `lane` of a wave's or block's tables (every lane of the wave active):
// the tasks' and, where the group takes the potential form, that form's.
// Returns whether it does, as a scalar: two DMA engines, and the time bound
// that classify_group tests is small enough.
template <typename TT>
__device__ __forceinline__ bool order_tables(OrderTables<TT> &o, const tgo_task *t, int n, const Rates &r) {
    const int lane = threadIdx.x & 63;
    Quad<TT> h = {};
    DRec<TT> d = {};
    if (lane < n) table_entry<TT>(t[lane], r, &h, &d);
    uint64_t sum = (uint64_t)h.hp + (uint64_t)h.k + (uint64_t)d.dp;
    for (int m = 8; m >= 1; m >>= 1) sum += shfl_xor64(sum, m);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)sum);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(sum >> 32));
    const bool potential = !r.one_dma && potential_fits<TT>((((uint64_t)hi << 32) | lo) + time_bound_slack(n), r);
    if (lane < n) {
        if (potential) {
            o.P[lane] = PRec<TT>{(TT)(h.h << r.q_log2), h.k, h.d, d.dp};
            o.gain[lane] = TT(r.p_h) * d.dp;
        } else {
            o.H[lane] = h;
            o.D[lane] = d;
        }
    }
    return potential;
}

}  // namespace tgo
