// The ordering heuristic of Section 5.1 (Algorithm 1) as a device function of
// one wave, shared by the per-group heuristic kernel, the enumerations under a
// rule and the proxy of the multi-round evaluator.
//
// The three selection functions are described in words only; the readings:
//   select_first: largest K - HtD (short HtD, long kernel); ties to the longer
//                 DtH, then the lower index.
//   select_next:  smallest |h_c - (t_K - t_HtD)| + |k_c - (t_DtH - max(t_HtD + h_c, t_K))|,
//                 i.e. the HtD that best fills the kernel engine's remaining
//                 busy time and the kernel that best fills the DtH engine's;
//                 ties to the lower index.
//   select_last:  both orders (x, y) of the last two tasks scored
//                 fit(x | OT) + fit(y | OT + x) + d_y; ties to the shorter
//                 final DtH, then to x with the lower index.
// t_HtD, t_K, t_DtH come from simulating the ordered set OT alone (update).
#pragma once

#include "../../include/tgo.h"
#include "enum_dev.h"
#include "model_dev.h"
#include "rule_dev.h"

namespace tgo {

struct Fit3 {
    int64_t th, tk, td;
};

// |h_c - (t_K - t_HtD)| + |k_c - (t_DtH - max(t_HtD + h_c, t_K))|
__device__ __forceinline__ int64_t fit(int64_t h, int64_t k, const Fit3 &u) {
    const int64_t a = h - (u.tk - u.th);
    const int64_t kstart = (u.th + h) > u.tk ? (u.th + h) : u.tk;
    const int64_t b = k - (u.td - kstart);
    return (a < 0 ? -a : a) + (b < 0 ? -b : b);
}

// Ends of the last HtD, kernel and DtH of the ordered set simulated alone.
template <int DMA, typename TT>
__device__ __forceinline__ Fit3 fit_ends(const Lane<TT> &s, const Rates &r) {
    return Fit3{(int64_t)s.t, (int64_t)s.ck, (int64_t)tail<DMA>(s, r)};
}
template <int DMA, typename TT>
__device__ __forceinline__ Fit3 fit_ends(const CLane<TT> &s, const Rates &r) {
    return Fit3{(int64_t)s.t, (int64_t)s.ck, (int64_t)tail<DMA>(s, r)};
}
template <int DMA, typename TT, int KIND>
__device__ __forceinline__ Fit3 fit_ends(const RLane<TT, KIND> &s, const Rates &r) {
    return Fit3{(int64_t)s.t, (int64_t)s.ke, (int64_t)tail<DMA>(s, r)};
}
template <int DMA, typename TT, int KIND>
__device__ __forceinline__ Fit3 fit_ends(const SubChain<TT, KIND> &s, const Rates &r) {
    return Fit3{(int64_t)s.x, (int64_t)s.kp, (int64_t)tail<DMA>(s, r)};
}

// The smallest key of lanes 0..15, as a scalar.  Every lane must be active.
__device__ __forceinline__ uint64_t row0_min(uint64_t k) {
    uint64_t o = row_ror_u64<8>(k);
    k = o < k ? o : k;
    o = row_ror_u64<4>(k);
    k = o < k ? o : k;
    o = row_ror_u64<2>(k);
    k = o < k ? o : k;
    o = row_ror_u64<1>(k);
    k = o < k ? o : k;
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)k);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(k >> 32));
    return ((uint64_t)hi << 32) | lo;
}

// Orders this wave's LDS writes before its later LDS reads.
__device__ __forceinline__ void wave_lds_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Algorithm 1 by one wave (all 64 lanes active) on the tasks in `set` (bits
// 0..15, at least one).  The simulation of the ordered set is the same on
// every lane (each with its own queue column, or one they share); each
// selection step scores the remaining tasks on their own lanes and takes the
// smallest key of a row of 16 lanes (DPP moves: a shuffle over the wave per
// step was half of the time), with the tie rules above.  Every instant stays
// below 2^56 (16 tasks, work below 2^50 each), so a score and a lane index
// share one key.  *ord_out receives the ordering, one task per nibble.  Returns
// the total time (TIME = false: 0, and the windows only the time needs are
// left out, all of them for one or two tasks).
template <int DMA, typename LaneT, bool TIME = true, typename ViewT>
__device__ __forceinline__ int64_t heuristic_wave(uint32_t set, const ViewT &v, const Rates &r, uint64_t *ord_out) {
    constexpr uint64_t NONE = ~0ull;
    const int lane = threadIdx.x & 63;
    uint32_t rt = set;
    uint64_t ord = 0;
    // this lane's task as a candidate
    int64_t ch = 0, ckn = 0, cd = 0;
    if (lane < MAXN && ((set >> lane) & 1u)) {
        const auto q = v.task((uint32_t)lane);
        ch = (int64_t)q.h;
        ckn = (int64_t)q.k;
        cd = (int64_t)q.d;
    }
    auto cand = [&] { return lane < MAXN && ((rt >> lane) & 1u); };
    // largest K - HtD, then longest DtH, then lowest index
    const uint64_t kh = (uint64_t)((int64_t(1) << 41) + ch - ckn);
    const uint64_t lowest = row0_min(cand() ? kh : NONE);
    const uint64_t longest = row0_min(cand() && kh == lowest
                                          ? ((uint64_t)((int64_t(1) << 41) - cd) << 4) | (uint64_t)lane : NONE);
    const uint32_t first = (uint32_t)longest & 15u;
    ord = first;
    rt &= ~(1u << first);
    if constexpr (!TIME) {
        if (__popc(rt) < 2) {
            *ord_out = ord | (rt ? (uint64_t)(__ffs(rt) - 1) << 4 : 0);
            return 0;
        }
    }
    LaneT st;
    lane_reset(st);
    window<DMA>(st, 0, first, v, r);
    int pos = 1;
    while (__popc(rt) > 2) {
        const Fit3 u = fit_ends<DMA>(st, r);
        const uint64_t key = cand() ? ((uint64_t)fit(ch, ckn, u) << 4) | (uint64_t)lane : NONE;
        const uint32_t best = (uint32_t)row0_min(key) & 15u;
        ord |= (uint64_t)best << (4 * pos);
        rt &= ~(1u << best);
        window<DMA>(st, pos, best, v, r);
        ++pos;
    }
    if (__popc(rt) == 2) {
        // select_last: both orders of the last two, scored on every lane
        const int a = __ffs(rt) - 1;
        const int b = 31 - __clz(rt);
        const Fit3 u = fit_ends<DMA>(st, r);
        int bx = -1, by = -1;
        int64_t bs = 0, bdy = 0;
#pragma unroll 1
        for (int o = 0; o < 2; ++o) {
            const int x = o == 0 ? a : b, y = o == 0 ? b : a;
            const auto tx = v.task((uint32_t)x), ty = v.task((uint32_t)y);
            const int64_t s1 = fit((int64_t)tx.h, (int64_t)tx.k, u);
            LaneT s2 = st;
            window<DMA>(s2, pos, (uint32_t)x, v, r);
            const Fit3 wf = fit_ends<DMA>(s2, r);
            const int64_t sc = s1 + fit((int64_t)ty.h, (int64_t)ty.k, wf) + (int64_t)ty.d;
            const int64_t dy = (int64_t)ty.d;
            if (bx < 0 || sc < bs || (sc == bs && dy < bdy)) { bx = x; by = y; bs = sc; bdy = dy; }
        }
        bx = __builtin_amdgcn_readfirstlane(bx);
        by = __builtin_amdgcn_readfirstlane(by);
        ord |= ((uint64_t)bx << (4 * pos)) | ((uint64_t)by << (4 * pos + 4));
        if constexpr (!TIME) {
            *ord_out = ord;
            return 0;
        }
        window<DMA>(st, pos, (uint32_t)bx, v, r);
        window<DMA, false>(st, pos + 1, (uint32_t)by, v, r);
    } else if (__popc(rt) == 1) {
        const int x = __ffs(rt) - 1;
        ord |= (uint64_t)x << (4 * pos);
        window<DMA, false>(st, pos, (uint32_t)x, v, r);
    }
    *ord_out = ord;
    return fit_ends<DMA>(st, r).td;
}

}  // namespace tgo
