// Per-ordering evaluation (one lane per given ordering) and the ordering
// heuristic of Section 5.1 (Algorithm 1, one wave per group).
#include <hip/hip_runtime.h>

#include <algorithm>

#include "enum_dev.h"
#include "heur_dev.h"
#include "tables_dev.h"
#include "tgo_internal.h"

namespace tgo {

constexpr int EV_THREADS = 256;
// Blocks per launch, in units of the resident ones.  A block's tables cost what some
// rows do: groups of up to EV_FEW tasks take one round of blocks with the same number
// of rows each, larger ones two rounds, whose blocks finish at different times.
// 1,000,003 / 2,000,000 rows in us, one even round, one round, two rounds: 3 tasks
// 16.4 / 24.9, 17.6 / 23.7, 22.3 / 28.0; 5 tasks 20.9 / 34.4, 22.0 / 32.0, 26.1 / 35.0;
// 12 tasks 39 / 70, 33 / 61, 38 / 61; 16 tasks 50 / 127, 61 / 114, 54 / 98 (a kernel per
// width, NARROW).
constexpr uint32_t EV_ROUNDS = 2;
constexpr int EV_FEW = 5;
constexpr int HEU_WAVES = 4;  // groups per block of the heuristic, one wave each

// A row of n <= N bytes, as nibbles: N loads (past the row its last byte again), in
// flight together.  seen: bit of every value, high: all of their bits.
template <int N>
__device__ __forceinline__ void read_row(const uint8_t *o, int n, uint64_t *perm, uint32_t *seen, uint32_t *high) {
    uint32_t b[N];
#pragma unroll
    for (int j = 0; j < N; ++j) b[j] = o[j < n ? j : n - 1];
#pragma unroll
    for (int j = 0; j < N; ++j) {
        *perm |= (uint64_t)(b[j] & 15u) << (4 * j);
        *seen |= j < n ? 1u << (b[j] & 15u) : 0u;
        *high |= b[j];
    }
}

// One lane per given ordering.  Bound by VALU issue over divergent windows.
// The row is read once, all of its bytes in flight together, checked and kept
// as nibbles; blocks stride over the rows so that the time path and the tables
// are set up by few blocks (a block per 256 rows, each with the time path
// decided by one thread, and as many idle ones of the other width: 1,000,003
// orderings of 16 tasks in 146 us; now 81, and 57 in the potential form).  NARROW: short
// rows are read by fewer loads (3 tasks, 1,000,003 rows: 25.9 us with 16 loads and two
// rounds of blocks in two launches, 13.7 as now).
template <typename TT, bool NARROW>
__device__ __forceinline__ void evaluate_rows(const tgo_task *__restrict__ tasks, int n, const Rates &r,
                                              const uint8_t *__restrict__ orders, int64_t m, int64_t *out,
                                              unsigned char *smem) {
    __shared__ OrderTables<TT> ot;
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    const bool potential = order_tables(ot, tasks, n, r);  // every wave writes the same
    __syncthreads();
    const auto v = ot.template view<EV_THREADS>(reinterpret_cast<TT *>(smem) + threadIdx.x);
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < m; i += stride) {
        const uint8_t *o = orders + i * n;
        uint64_t perm = 0;
        uint32_t seen = 0, high = 0;
        if constexpr (NARROW) {
            if (n <= 4) read_row<4>(o, n, &perm, &seen, &high);
            else if (n <= 8) read_row<8>(o, n, &perm, &seen, &high);
            else read_row<MAXN>(o, n, &perm, &seen, &high);
        } else {  // read_row<MAXN>, written out: called, 64-bit time took 2 % more
            uint32_t b[MAXN];
#pragma unroll
            for (int j = 0; j < MAXN; ++j) b[j] = o[j < n ? j : n - 1];
#pragma unroll
            for (int j = 0; j < MAXN; ++j) {
                perm |= (uint64_t)(b[j] & 15u) << (4 * j);
                seen |= j < n ? 1u << (b[j] & 15u) : 0u;
                high |= b[j];
            }
        }
        // a permutation: no value above 15 and every one of the n below
        if (high > 15u || seen != (1u << n) - 1u) {
            out[i] = TGO_EINVAL;
            continue;
        }
        out[i] = (int64_t)simulate_order(n, perm, v, r, potential);
    }
}

// ONLY: the time width it runs for (0: 32 bits, 1: 64; errors go with 0), or -1: both.
template <int ONLY>
__global__ __launch_bounds__(EV_THREADS) void evaluate_kernel(const tgo_task *__restrict__ tasks,
                                                              int n, Rates r,
                                                              const uint8_t *__restrict__ orders,
                                                              int64_t m, int64_t *out) {
    extern __shared__ __align__(16) unsigned char smem[];
    const int mode = __builtin_amdgcn_readfirstlane(classify_group_wave(tasks, n, r, threadIdx.x & 63));
    if (mode < 0) {
        if (ONLY != 1)
            for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < m;
                 i += (int64_t)gridDim.x * blockDim.x)
                out[i] = mode;
        return;
    }
    if constexpr (ONLY != 1)
        if (mode == 0) evaluate_rows<uint32_t, ONLY == -1>(tasks, n, r, orders, m, out, smem);
    if constexpr (ONLY != 0)
        if (mode == 1) evaluate_rows<uint64_t, ONLY == -1>(tasks, n, r, orders, m, out, smem);
}

// Rows up to which both widths share a launch: the second width's idle launch
// costs 3 us, its code a part of the resident blocks, which two blocks per CU do
// not miss.  One launch against two in us, 16 tasks: 500 rows 13.4 / 14.8, 65,536
// 13.9 / 15.7, 131,072 14.8 / 17.0, 262,144 27.6 / 21.5 (64-bit time, 131,072:
// 17.5 / 19.6, 262,144: 32.8 / 35.0); 5 tasks, 3 rows: 10.7 / 13.4.  Groups of up to
// EV_FEW tasks, whose queues leave seven blocks per CU in either width, share it
// whatever the rows.
constexpr int64_t EV_BOTH = 131072;

// What a block may take without asking for more: both widths' tables and the 64-bit
// queue of the largest group.
static_assert(sizeof(OrderTables<uint32_t>) + sizeof(OrderTables<uint64_t>) +
                      order_queue_bytes<uint64_t>(MAXN, EV_THREADS) <= 64 * 1024,
              "LDS of a block");

int launch_evaluate(const Rates &r, const tgo_task *d_tasks, int n, const uint8_t *d_orders,
                    int64_t m, int64_t *d_out, hipStream_t st) {
    if (m == 0) return TGO_OK;
    const int64_t want = (m + EV_THREADS - 1) / EV_THREADS;
    const size_t shm32 = order_queue_bytes<uint32_t>(n, EV_THREADS);
    const size_t shm64 = order_queue_bytes<uint64_t>(n, EV_THREADS);
    auto grid = [want, n](const void *k, size_t shm) {
        const int64_t b = resident_blocks(k, EV_THREADS, shm);
        if (b == 0) return dim3((uint32_t)std::min<int64_t>(want, 8192));
        if (n > EV_FEW) return dim3((uint32_t)std::min<int64_t>(want, b * EV_ROUNDS));
        const int64_t rows = (want + b - 1) / b;  // per thread
        return dim3((uint32_t)((want + rows - 1) / rows));
    };
    auto launch = [&](auto *kernel, size_t shm) {
        hipLaunchKernelGGL(kernel, grid(reinterpret_cast<const void *>(kernel), shm), dim3(EV_THREADS), shm, st,
                           d_tasks, n, r, d_orders, m, d_out);
    };
    if (m <= EV_BOTH || n <= EV_FEW) {
        launch(&evaluate_kernel<-1>, shm64);
    } else {
        launch(&evaluate_kernel<0>, shm32);
        launch(&evaluate_kernel<1>, shm64);
    }
    TGO_HIP(hipGetLastError());
    return TGO_OK;
}

// ---------------------------------------------------------------- heuristic

// Tables and queue of one wave, in either time width.
template <typename TT>
struct HeurLds {
    Quad<TT> H[MAXN];
    DRec<TT> D[MAXN];
    Slot<TT> Q[MAXN];
};

template <typename TT>
__device__ __forceinline__ int64_t heuristic_group(const tgo_task *t, int n, const Rates &r, int lane,
                                                   HeurLds<TT> &l, uint64_t *ord) {
    if (lane < n) table_entry<TT>(t[lane], r, &l.H[lane], &l.D[lane]);
    wave_lds_sync();
    View<TT, 1, 1> v;
    v.H = l.H;
    v.D = l.D;
    v.Q = l.Q;
    const uint32_t set = (1u << n) - 1u;
    return r.one_dma ? heuristic_wave<DMA_ONE, Lane<TT>>(set, v, r, ord)
                     : heuristic_wave<DMA_TWO, CLane<TT>>(set, v, r, ord);
}

// One wave per group (heuristic_wave), in 32-bit time where the group allows
// it.  Bound by the latency of one wave's dependent instructions.
__global__ __launch_bounds__(HEU_WAVES * 64) void heuristic_kernel(const tgo_task *__restrict__ tasks,
                                                                   const int32_t *__restrict__ offs,
                                                                   int n_groups, Rates r,
                                                                   uint8_t *orders, int order_stride,
                                                                   int64_t *ns, int ns_stride) {
    __shared__ union {
        HeurLds<uint32_t> w32;
        HeurLds<uint64_t> w64;
    } lds[HEU_WAVES];
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    const int g = blockIdx.x * HEU_WAVES + w;
    if (g >= n_groups) return;
    const int base = offs[g];
    const int n = offs[g + 1] - base;
    uint8_t *orow = orders + (size_t)g * order_stride;
    int64_t *nsg = ns + (size_t)g * ns_stride;
    if (n < 1 || n > MAXN) {
        if (lane < 16) orow[lane] = 0xff;
        if (lane == 0) *nsg = TGO_EINVAL;
        return;
    }
    const tgo_task *t = tasks + base;
    const int cls = __builtin_amdgcn_readfirstlane(classify_group_wave(t, n, r, lane));
    if (cls < 0) {
        if (lane < 16) orow[lane] = 0xff;
        if (lane == 0) *nsg = cls;
        return;
    }
    uint64_t ord;
    const int64_t T = cls == 0 ? heuristic_group<uint32_t>(t, n, r, lane, lds[w].w32, &ord)
                               : heuristic_group<uint64_t>(t, n, r, lane, lds[w].w64, &ord);
    if (lane < 16) orow[lane] = lane < n ? (uint8_t)((ord >> (4 * lane)) & 15u) : (uint8_t)0xff;
    if (lane == 0) *nsg = T;
}

int launch_heuristic(const Rates &r, const tgo_task *d_tasks, const int32_t *d_offs, int n_groups,
                     uint8_t *d_orders, int order_stride, int64_t *d_ns, int ns_stride,
                     hipStream_t st) {
    if (n_groups == 0) return TGO_OK;
    const int blocks = (n_groups + HEU_WAVES - 1) / HEU_WAVES;
    hipLaunchKernelGGL(heuristic_kernel, dim3(blocks), dim3(HEU_WAVES * 64), 0, st, d_tasks, d_offs,
                       n_groups, r, d_orders, order_stride, d_ns, ns_stride);
    TGO_HIP(hipGetLastError());
    return TGO_OK;
}

}  // namespace tgo
