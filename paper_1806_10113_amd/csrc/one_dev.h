// Every ordering of one group on a device with one DMA engine.
//
// There the HtDs run back to back and the DtHs wait for the last of them, so the
// total time is a maximum of sums: with t and ck the ends of the HtDs and kernels
// of a prefix, emax and dpre as the windows keep them (model_dev.h), D the solo
// DtH time of the tasks that are left and H their HtD time,
//   T = max(X, ck + D + B, t + D + C),  X = max(emax, t + H) + dpre + D,
//   B = max_p (sum_{s<=p} k_s - sum_{s<p} d_s),
//   C = max_p (A_p - sum_{s<p} d_s),  A_p = max(A_{p-1}, sum_{s<=p} h_s) + k_p,
// p and s over the order of the remaining tasks.  X, Y = ck + D and Z = t + D
// belong to the prefix alone, B and C to the order of the rest alone.  A block
// takes one set of remaining tasks, computes B and C of its m! orders once, and
// its lanes, two prefixes each, add and compare: no window is walked twice, and
// an ordering is two additions, two comparisons and its statistics.
//
// What bounds it: the vector units.  The inner loop is 29 instructions for two
// orders of two prefixes, 9 of them of the kind that issues twice as fast, and
// the units are busy 70% of the time.  A group of 13: 1320 us, of 12 200, of 10
// 32; walked window by window (35 instructions per ordering) 3960, 400 and 68.
#pragma once

#include "enum_kernel.h"

namespace tgo {

constexpr int ONE_PP = 2;  // prefixes per lane: one read of (B, C) serves both
constexpr uint32_t ONE_TILE = ONE_PP * EX_THREADS;
constexpr int ONE_MAX_M = 6;

// A tile is a part of the prefixes of one set; the parts of a set are alike.
struct OneShape {
    uint32_t prefixes, orders;  // (n - m)!, m!
    uint32_t parts, per;        // tiles of a set, prefixes of a tile
    uint32_t tiles;
};
inline OneShape one_shape(int n, int m) {
    OneShape s;
    s.prefixes = (uint32_t)factorial(n - m);
    s.orders = (uint32_t)factorial(m);
    s.parts = (s.prefixes + ONE_TILE - 1) / ONE_TILE;
    s.per = (s.prefixes + s.parts - 1) / s.parts;
    s.tiles = (uint32_t)(factorial(n) / factorial(n - m) / factorial(m)) * s.parts;
    return s;
}

// Dynamic LDS: the task tables, (B, C) of every order, and with STORE the
// prefixes' X, Y, Z and first ranks.
template <typename TT, bool STORE>
__host__ __device__ constexpr size_t one_lds(int n, uint32_t orders) {
    return (size_t)n * (sizeof(Quad<TT>) + sizeof(DRec<TT>)) + ((2 * sizeof(TT) * orders + 15) & ~size_t(15)) +
           (STORE ? ONE_TILE * (3 * sizeof(TT) + sizeof(uint64_t)) : 0);
}

template <typename TT>
struct OnePrefix {
    TT x, y, z;
    uint64_t r0;  // first rank
    __device__ __forceinline__ TT total(TT b, TT c) const { return tmax(x, tmax(y + b, z + c)); }
};

// B and C of the l-th order of the tasks in list (ascending, one per nibble).
template <typename TT, typename ViewT>
__device__ __forceinline__ void one_order(uint32_t l, int m, uint32_t list, const ViewT &v, TT *B, TT *C) {
    using ST = typename Signed<TT>::type;
    uint32_t dig = 0;  // factorial digits of l, position p at nibble p
#pragma unroll
    for (int i = 2; i <= ONE_MAX_M; ++i)
        if (i <= m) {
            dig |= (l % (uint32_t)i) << (4 * (m - i));
            l /= (uint32_t)i;
        }
    TT h = 0, k = 0, a = 0;
    ST d = 0, b = 0, c = 0;  // both maxima start at the first position's, which is not negative
#pragma unroll 1
    for (int p = 0; p < m; ++p) {
        const uint32_t sh = 4 * ((dig >> (4 * p)) & 15u);
        const Quad<TT> t = v.task((list >> sh) & 15u);
        list = (list & ((1u << sh) - 1u)) | ((list >> sh >> 4) << sh);
        h += t.h;
        k += t.k;
        a = tmax(a, h) + t.k;
        b = (ST)k - d > b ? (ST)k - d : b;
        c = (ST)a - d > c ? (ST)a - d : c;
        d += (ST)t.d;
    }
    *B = (TT)b;
    *C = (TT)c;
}

template <typename TT, bool STORE>
__device__ __forceinline__ void one_run(const tgo_task *__restrict__ tasks, int n, int m, const Rates &r,
                                        const OneShape &sh, int64_t *out, Partial *partials, ExAcc *acc,
                                        unsigned char *smem) {
    __shared__ Partial red[EX_THREADS / 64];
    __shared__ Partial best, all;  // the tile's result; thread 0's: the block's tiles together
    __shared__ OnePrefix<TT> win[2];  // the prefixes of the tile's smallest and largest time
    __shared__ uint32_t at[2];        // and the orders
    Quad<TT> *Ht = reinterpret_cast<Quad<TT> *>(smem);
    DRec<TT> *Dt = reinterpret_cast<DRec<TT> *>(smem + (size_t)n * sizeof(Quad<TT>));
    TT *tab = reinterpret_cast<TT *>(Dt + n);
    const int tid = threadIdx.x;
    if (tid < n) table_entry<TT>(tasks[tid], r, &Ht[tid], &Dt[tid]);
    View<TT, 1, EX_THREADS> v;
    v.H = Ht;
    v.D = Dt;
    v.Q = nullptr;
    if (tid == 0) {
        all.min_t = ~0ull; all.min_r = ~0ull; all.max_t = 0; all.max_r = ~0ull;
        all.sum_lo = 0; all.sum_hi = 0; all.fp = 0; all.status = 0; all.pad = 0;
    }
    const uint32_t L = sh.orders;
    for (uint32_t tile = blockIdx.x; tile < sh.tiles; tile += gridDim.x) {
        __syncthreads();  // the tables; the last tile's reads
        const uint32_t set = tile / sh.parts, base = (tile - set * sh.parts) * sh.per;
        const uint32_t cnt = base + sh.per <= sh.prefixes ? sh.per : sh.prefixes - base;
        const uint32_t half = (cnt + ONE_PP - 1) / ONE_PP;
        OnePrefix<TT> px[ONE_PP];
        uint32_t list = 0;
        // lane i: prefixes i and half + i of the tile (past the end: the first again, not counted)
#pragma unroll
        for (int q = 0; q < ONE_PP; ++q) {
            const uint32_t i = q * half + tid;
            Lane<TT> st;
            uint32_t lex;
            const uint64_t rest = prefix_by_set<DMA_ONE>(st, set * sh.prefixes + base + (i < cnt ? i : 0), n, m, v, r, &lex);
            list = (uint32_t)rest;
            TT H = 0, D = 0;
            for (int p = 0; p < m; ++p) {
                const Quad<TT> t = v.task((list >> (4 * p)) & 15u);
                H += t.h;
                D += t.d;
            }
            using ST = typename Signed<TT>::type;
            const ST e = (ST)(st.t + H) > st.emax ? (ST)(st.t + H) : st.emax;
            px[q].x = (TT)(e + (ST)(st.dpre + D));
            px[q].y = st.ck + D;
            px[q].z = st.t + D;
            px[q].r0 = (uint64_t)lex * L;
        }
        for (uint32_t l = tid; l < L; l += EX_THREADS) one_order<TT>(l, m, list, v, &tab[2 * l], &tab[2 * l + 1]);
        if (tid < 2) at[tid] = ~0u;
        __syncthreads();
        // all orders, the last pair first: with S_k the sum of pair k, S over all
        // of them so far and Q the sum of these, sum l T = 2 (Q - S) + the odd ones.
        // In 64-bit time one prefix after the other (registers).
        constexpr int W = sizeof(TT) == 4 ? ONE_PP : 1;
        Partial p;
        p.min_t = ~0ull; p.min_r = ~0ull; p.max_t = 0; p.max_r = ~0ull;
        p.sum_lo = 0; p.sum_hi = 0; p.fp = 0; p.status = 0; p.pad = 0;
#pragma unroll
        for (int q0 = 0; q0 < ONE_PP; q0 += W) {
            TT mn[W], mx[W];
            uint64_t S[W], Q[W], odd[W];
#pragma unroll
            for (int q = 0; q < W; ++q) {
                mn[q] = inf_time<TT>();
                mx[q] = 0;
                S[q] = Q[q] = odd[q] = 0;
                if (L == 1) {
                    mn[q] = mx[q] = px[q0 + q].total(tab[0], tab[1]);
                    S[q] = Q[q] = (uint64_t)mn[q];
                }
            }
            const Quad<TT> *pair = reinterpret_cast<const Quad<TT> *>(tab);
            for (int k = (int)(L / 2) - 1; k >= 0; --k) {
                const Quad<TT> e = pair[k];  // (B, C) of orders 2k and 2k + 1
#pragma unroll
                for (int q = 0; q < W; ++q) {
                    const TT t0 = px[q0 + q].total(e.h, e.hp), t1 = px[q0 + q].total(e.k, e.d);
                    mn[q] = tmin(mn[q], tmin(t0, t1));
                    mx[q] = tmax(mx[q], tmax(t0, t1));
                    S[q] += (uint64_t)(TT)(t0 + t1);  // 32 bits: each is below 2^31
                    Q[q] += S[q];
                    odd[q] += (uint64_t)t1;
                }
            }
#pragma unroll
            for (int q = 0; q < W; ++q)
                if ((uint32_t)tid < half && (q0 + q) * half + tid < cnt) {
                    const uint64_t r0 = px[q0 + q].r0;
                    merge_min(p.min_t, p.min_r, (uint64_t)mn[q], r0);
                    merge_max(p.max_t, p.max_r, (uint64_t)mx[q] + 1, r0);
                    add128(p.sum_lo, p.sum_hi, S[q], 0);
                    p.fp += 2ull * (r0 * S[q] + 2ull * (Q[q] - S[q]) + odd[q]) + S[q];
                }
        }
        const Partial o = block_reduce(p, red);
        if (tid == 0) best = o;
        __syncthreads();
#pragma unroll
        for (int q = 0; q < ONE_PP; ++q)
            if ((uint32_t)tid < half && q * half + tid < cnt) {
                if (px[q].r0 == best.min_r) win[0] = px[q];
                if (px[q].r0 == best.max_r) win[1] = px[q];
                if constexpr (STORE) {
                    TT *xyz = reinterpret_cast<TT *>(reinterpret_cast<unsigned char *>(tab) +
                                                     ((2 * sizeof(TT) * L + 15) & ~size_t(15)));
                    uint64_t *r0 = reinterpret_cast<uint64_t *>(xyz + 3 * ONE_TILE);
                    const uint32_t i = q * half + tid;
                    xyz[i] = px[q].x;
                    xyz[ONE_TILE + i] = px[q].y;
                    xyz[2 * ONE_TILE + i] = px[q].z;
                    r0[i] = px[q].r0;
                }
            }
        __syncthreads();
        // the lowest order with either time
        const OnePrefix<TT> lo = win[0], hi = win[1];
        for (uint32_t l = tid; l < L; l += EX_THREADS) {
            const TT b = tab[2 * l], c = tab[2 * l + 1];
            if ((uint64_t)lo.total(b, c) == best.min_t) atomicMin(&at[0], l);
            if ((uint64_t)hi.total(b, c) + 1 == best.max_t) atomicMin(&at[1], l);
        }
        if constexpr (STORE) {
            // a prefix's times lie together: neighbouring lanes take neighbouring orders
            const TT *xyz = reinterpret_cast<const TT *>(reinterpret_cast<const unsigned char *>(tab) +
                                                         ((2 * sizeof(TT) * L + 15) & ~size_t(15)));
            const uint64_t *r0 = reinterpret_cast<const uint64_t *>(xyz + 3 * ONE_TILE);
            uint32_t i = (uint32_t)tid / L, l = (uint32_t)tid % L;
            while (i < cnt) {
                OnePrefix<TT> x;
                x.x = xyz[i];
                x.y = xyz[ONE_TILE + i];
                x.z = xyz[2 * ONE_TILE + i];
                out[r0[i] + l] = (int64_t)x.total(tab[2 * l], tab[2 * l + 1]);
                i += EX_THREADS / L;
                l += EX_THREADS % L;
                if (l >= L) {
                    l -= L;
                    ++i;
                }
            }
        }
        __syncthreads();
        if (tid == 0) {
            merge_min(all.min_t, all.min_r, best.min_t, best.min_r + at[0]);
            merge_max(all.max_t, all.max_r, best.max_t, best.max_r + at[1]);
            add128(all.sum_lo, all.sum_hi, best.sum_lo, best.sum_hi);
            all.fp += best.fp;
        }
    }
    if (tid == 0) block_out<TT>(all, blockIdx.x, partials, acc);
}

// Both time widths in one launch (modep: the group's, or an error code): the
// second one's idle launch costs 4.5 us, its registers (5 waves per SIMD where the
// 32-bit code alone fits 7) 2% of the largest group.
template <bool STORE>
__global__ __launch_bounds__(EX_THREADS) void one_kernel(const tgo_task *__restrict__ tasks, int n, int m, Rates r,
                                                         OneShape sh, int64_t *out, Partial *partials, ExAcc *acc,
                                                         const int *__restrict__ modep) {
    extern __shared__ __align__(16) unsigned char smem[];
    const int mode = *modep;
    if (mode == 0) one_run<uint32_t, STORE>(tasks, n, m, r, sh, out, partials, acc, smem);
    else if (mode == 1) one_run<uint64_t, STORE>(tasks, n, m, r, sh, out, partials, acc, smem);
}

}  // namespace tgo
