// One lane of every walk and of the whole-ordering evaluation, compiled for the CPU:
// every ordering of random groups of 5 to 7 tasks in both time widths (durations from
// a few ns, with empty stages, to just below 2^40) against the C oracle.  The queue is
// heap memory of its exact size, not initialised.
#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <functional>
#include <random>
#include <vector>

#include "../../paper_1806_10113_amd/csrc/enum_dev.h"
#include "../../paper_1806_10113_amd/csrc/rule_dev.h"

extern "C" {
int64_t oracle_simulate(const int64_t *, int, const int *, int, int, int, int, int64_t *);
int oracle_mem_times(const int64_t *, const int64_t *, int, int64_t, int, int, int, int, uint64_t, uint64_t, int, int64_t *);
int oracle_cke_times(const int64_t *, const int *, int, int, int, int, int, int, uint64_t, uint64_t, int, int64_t *);
}

using namespace tgo;

struct Case {
    int n;
    Rates r;
    std::vector<int64_t> t, mem;
    std::vector<int32_t> units;
    std::vector<uint32_t> fits;
    int64_t cap;
    int ucap;
};

static Rates rates(int q_log2, int p_h, int p_d, int one) {
    Rates r = {};
    r.q_log2 = q_log2;
    r.p_h = (uint32_t)p_h;
    r.p_d = (uint32_t)p_d;
    r.one_dma = one;
    r.inv_ph = 1.0 / p_h;
    r.c_ph = (p_h - 0.5) * r.inv_ph;
    r.inv_pd = 1.0 / p_d;
    r.c_pd = (p_d - 0.5) * r.inv_pd;
    return r;
}

template <typename TT, int DMA, typename LaneT, typename ViewT>
static void walk(ViewT &v, const Case &c, std::vector<int64_t> &out) {
    constexpr int M = DMA == DMA_ONE ? 4 : 5;
    Ctx x;
    x.n = c.n;
    x.r = c.r;
    for (uint32_t s = 0; s < fact_c(c.n) / fact_c(M); ++s) {
        LaneT st;
        uint32_t lex;
        const uint64_t list = prefix_by_set<DMA>(st, s, c.n, M, v, c.r, &lex);
        x.out_sub = out.data() + (size_t)lex * fact_c(M);
        Sub<TT> u;
        sub_init(u);
        level<TT, M, true, DMA>(x, v, st, (uint32_t)list, 0u, u);
    }
}

template <typename TT>
static int check(const Case &c) {
    const int n = c.n, q = 1 << c.r.q_log2;
    const uint64_t f = fact_c(n);
    std::vector<int64_t> out(f), want(f);
    std::vector<Quad<TT>> H(n);
    std::vector<DRec<TT>> D(n);
    std::vector<PRec<TT>> P(n);
    std::vector<TT> gain(n);
    uint64_t bound = time_bound_slack(n);
    for (int i = 0; i < n; ++i) {
        const uint64_t h = c.t[3 * i], k = c.t[3 * i + 1], d = c.t[3 * i + 2];
        const uint64_t hp = (q * h + c.r.p_h - 1) / c.r.p_h, dp = (q * d + c.r.p_d - 1) / c.r.p_d;
        H[i] = Quad<TT>{(TT)h, (TT)hp, (TT)k, (TT)d};
        D[i] = DRec<TT>{(TT)d, (TT)dp, (TT)(c.r.p_d * dp - q * d), 0};
        P[i] = PRec<TT>{(TT)(h << c.r.q_log2), (TT)k, (TT)d, (TT)dp};
        gain[i] = (TT)(c.r.p_h * dp);
        bound += hp + k + dp;
    }
    Slot<TT> *Q = static_cast<Slot<TT> *>(std::malloc(sizeof(Slot<TT>) * (n - 1)));
    int bad = 0;
    auto same = [&](const char *what) {
        if (out == want) return;
        std::printf("%s: %zu-bit time, n %d, rates %d %u %u\n", what, 8 * sizeof(TT), n, q, c.r.p_h, c.r.p_d);
        ++bad;
    };
    std::vector<int> p(n);
    auto each = [&](const std::function<int64_t()> &T, std::vector<int64_t> &to) {
        for (int i = 0; i < n; ++i) p[i] = i;
        for (uint64_t rk = 0; rk < f; ++rk, std::next_permutation(p.begin(), p.end())) to[rk] = T();
    };
    const int dma = c.r.one_dma ? 1 : 2;
    each([&] { return oracle_simulate(c.t.data(), n, p.data(), q, c.r.p_h, c.r.p_d, dma, nullptr); }, want);
    View<TT, 1, 1> v;
    v.H = H.data();
    v.D = D.data();
    v.Q = Q;
    if (c.r.one_dma) walk<TT, DMA_ONE, Lane<TT>>(v, c, out);
    else walk<TT, DMA_TWO, CLane<TT>>(v, c, out);
    same("walk");
    for (bool potential : {false, true}) {
        if (potential && (c.r.one_dma || !potential_fits<TT>(bound, c.r))) continue;
        std::vector<TT> queue(2 * n - 1);
        const OrderView<TT, 1> o{H.data(), D.data(), P.data(), gain.data(), queue.data()};
        each([&] {
            uint64_t perm = 0;
            for (int j = 0; j < 16; ++j) perm |= (uint64_t)p[j < n ? j : n - 1] << (4 * j);
            return (int64_t)simulate_order(n, perm, o, c.r, potential);
        }, out);
        same(potential ? "orderings, potential form" : "orderings");
    }
    uint64_t seq = 0;
    auto rule = [&](auto &w) {
        w.H = H.data();
        w.D = D.data();
        w.Q = Q;
        w.seq = &seq;
        w.units = c.units.data();
        w.cap = c.ucap;
        w.fits = c.fits.data();
        w.pos = 0;
        w.dep = w.opens = 0;
    };
    RView<TT, 1, 1, RULE_MEMORY> m;
    rule(m);
    oracle_mem_times(c.t.data(), c.mem.data(), n, c.cap, q, c.r.p_h, c.r.p_d, dma, 0, f, 1, want.data());
    if (c.r.one_dma) walk<TT, DMA_ONE, SubChain<TT, RULE_MEMORY>>(m, c, out);
    else walk<TT, DMA_TWO, RLane<TT, RULE_MEMORY>>(m, c, out);
    same("memory limit");
    RView<TT, 1, 1, RULE_CONCURRENT> k;
    rule(k);
    oracle_cke_times(c.t.data(), c.units.data(), n, c.ucap, q, c.r.p_h, c.r.p_d, dma, 0, f, 1, want.data());
    if (c.r.one_dma) walk<TT, DMA_ONE, RLane<TT, RULE_CONCURRENT>>(k, c, out);
    else walk<TT, DMA_TWO, RLane<TT, RULE_CONCURRENT>>(k, c, out);
    same("concurrent kernels");
    std::free(Q);
    return bad;
}

int main(int argc, char **argv) {
    std::mt19937_64 g(std::strtoull(argv[2], nullptr, 0));
    int bad = 0;
    for (int it = 0; it < std::atoi(argv[1]); ++it) {
        Case c;
        c.n = 5 + (int)(g() % 3);
        const int ql = (int)(g() % 11), q = 1 << ql;
        c.r = rates(ql, g() % 6 ? 1 + (int)(g() % q) : q, g() % 6 ? 1 + (int)(g() % q) : q, it % 3 == 2);
        const int64_t top[] = {4, 50, 3000000 >> (ql / 2), 20000000 >> ql, (int64_t(1) << 40) - 1};
        const int64_t mx = top[g() % 5];
        for (int i = 0; i < 3 * c.n; ++i) c.t.push_back(g() % 8 ? (int64_t)(g() % (uint64_t)(mx + 1)) : 0);
        int64_t sum = 0, most = 1;
        for (int i = 0; i < c.n; ++i) {
            c.mem.push_back((int64_t)(g() % 100));
            sum += c.mem[i];
            most = std::max(most, c.mem[i]);
        }
        c.cap = most + (int64_t)(g() % (uint64_t)(sum + 1));
        c.ucap = 1 + (int)(g() % 16);
        for (int i = 0; i < c.n; ++i) c.units.push_back(1 + (int)(g() % c.ucap));
        c.fits.assign(4, 0);
        uint64_t bound = time_bound_slack(c.n), work = 0;
        for (uint32_t s = 0; s < (1u << c.n); ++s) {
            int64_t held = 0;
            for (int i = 0; i < c.n; ++i) held += (s >> i) & 1u ? c.mem[i] : 0;
            if (held <= c.cap) c.fits[s >> 5] |= 1u << (s & 31u);
        }
        for (int i = 0; i < c.n; ++i) {
            const uint64_t h = (uint64_t)c.t[3 * i] << ql, d = (uint64_t)c.t[3 * i + 2] << ql;
            bound += (h + c.r.p_h - 1) / c.r.p_h + (uint64_t)c.t[3 * i + 1] + (d + c.r.p_d - 1) / c.r.p_d;
            work = std::max(work, std::max(h, d));
        }
        if (work < (1ull << 31) && bound < (1ull << 31)) bad += check<uint32_t>(c);
        bad += check<uint64_t>(c);
    }
    std::printf("walks done, %d differ\n", bad);
    return bad != 0;
}
