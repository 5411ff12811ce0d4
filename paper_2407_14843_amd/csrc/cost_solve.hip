// The whole solve of an instance by one wavefront, with the recurrence over the
// total cost instead of the latency budget.
//
// Section 4.4 splits the latency budget between the models, f[s][t] = least cost
// of models s.. within t ticks.  The same recurrence can be written the other way
// round, g[s][x] = least ticks of models s.. for at most x cores more than the
// least they can be run with at all:
//
//     base[s]  = least cost of model s over its feasible candidates
//     g[S][x]  = 0
//     g[s][x]  = min over candidates k with cost[s][k] - base[s] <= x of
//                lt[s][k] + g[s+1][x - (cost[s][k] - base[s])]
//
// The least total cost is sum(base) + x* with x* the first x for which
// g[0][x] <= T, and g[0][x*] is the least number of ticks at that cost.  The
// answer is the same one (the smallest assignment by cost, ticks, then the
// choices of model 0, 1, ...), but a row has as many cells as the answer costs
// more than sum(base), while a row over the budget has T + 1: on pipelines like
// those of the numbered workloads x* is 0 for 65-100 % of the instances and
// below 64 for nearly all, against budgets of 300 to 16000 ticks.
//
// Exactness.  An assignment of total cost sum(base) + x* within T ticks exists
// and none is cheaper, so every assignment that attains (cost, ticks) spends
// exactly x* over base and exactly g[0][x*] ticks; reading the choices out
// forward, a candidate of model s continues such an assignment if and only if
// lt + g[s+1][x - d] equals the ticks that are left, and the smallest index among
// those is taken.  A candidate that another one of its model beats or ties on
// both cost and latency (ties: smaller index) cannot do so: put in its place, the
// other one would give a smaller assignment.  So it is enough to keep, per model
// and cost, the least (lt, index), and only those costs where the latency drops
// below that of everything cheaper.
//
// Steps per instance, all of them within one wavefront:
//   0  input check, budget; the fastest candidate of every (model, batch size),
//      which is the one at the core cap (latency never grows with the cores).  The
//      instance is infeasible exactly when the fastest candidates of all models
//      together exceed the budget.
//   A  base[s], with the least (lt, index) at that cost.  Lane = (model, batch
//      size); a lane walks the cores upward from the first that can be feasible and
//      stops where a lower bound of everything beyond exceeds the model's best.
//      When these candidates fit the budget together, x* = 0 and they are the
//      answer.
//   B  else the recurrence over the first `window` cells: one table of (lt, index)
//      by model and cost over base, rows in LDS, lane = cell.
//   C  else a wider window, as far as LDS goes; and past that
//   D  the recurrence over the budget with rows in HBM, which is bounded by T
//      whatever the costs are (costs spread over thousands of cores in one model).
//
// What bounds it: vector issue.  An instance is some hundreds of instructions,
// mostly the double-precision evaluation of candidates (candidate_eval.h, shared
// with the candidate tables and the rate search, so that all agree bit for bit),
// against 0.3 KB of inputs and outputs; nothing but those touches HBM.  Whole solves
// by the three stages (dense / with dominated candidates pruned) against this one, in
// microseconds: 65536 x 8 models 25900 / 3890 -> 173, 16384 x 8 with replicas given
// 3360 -> 37, 86400 x 6 2790 -> 86, 4096 x 5 178 -> 21, 64 x 3 27.5 -> 9.7.
#include "candidate_eval.h"
#include "instance_queue.h"
#include "themis_internal.h"
#include "wave_ops.h"

#include <type_traits>

namespace themis {
namespace {

constexpr int RC_TABLE = 128;                // reciprocals of core counts kept in LDS
constexpr uint32_t LT_NONE = 1u << 20;       // "no candidate": above any budget
constexpr uint32_t EMPTY = 0xFFFFFFFFu;      // empty cell of the (lt, index) table
constexpr int INDEX_BITS = 13;               // candidate indices are below 8192
constexpr uint32_t G_INF = 0x8000u;          // row cell beyond any budget
constexpr int RAW = 8;                       // words per model: coefficients, replicas, cores

struct CostArgs {
    const int32_t *coef, *lambda, *slo_us, *r_fixed, *c_fixed;
    int32_t *status, *cost, *ticks, *cfg;
    int32_t* tmeta;     // budgets, for calls that inspect the workspace afterwards
    int32_t* hard;      // per instance: left to the launch with the large window
    int32_t* ctrl;
    uint16_t* frow;     // rows of step D
    int32_t* keep;      // inputs and results for such calls, or null
    KeepLayout kept;
    BatchList bl;
    int32_t N, S, cs, c_max, r_max, tick, slo_max, coef_shared, c_all, sparse, row_stride;
    int32_t window;     // cells of the largest window, a multiple of 64
    uint32_t nb_magic;  // ceil(2^16 / n_batch): x / n_batch = x * nb_magic >> 16 for x < 1024
    uint32_t k_magic;   // ceil(2^20 / n_batch): the same with 20 for x < 8192
    double rtick;
};

// LDS words of one wavefront
struct CostLds {
    int raw, best, key, fast, tab, rows, words;
};
__host__ __device__ inline CostLds cost_lds(int S, int window)
{
    CostLds l;
    l.raw = 0;
    l.best = l.raw + RAW * S;  // two words per model
    l.key = l.best + 2 * S;
    l.fast = l.key + S;
    l.tab = (l.fast + S + 3) & ~3;
    l.rows = l.tab + S * window;
    l.words = (l.rows + S * window / 2 + 3) & ~3;
    return l;
}

__device__ __forceinline__ int in_range(int32_t v, int32_t lo, int32_t hi)
{
    return (int)(v >= lo) & (int)(v <= hi);
}

// One wavefront's view of the instance it works on.
template <int QUEUE, bool DERIVE>
struct Solver {
    const CostArgs& a;
    uint32_t* const lds;   // this wavefront's words
    const double* const rc;  // reciprocals of 1 .. RC_TABLE cores (at most c_max of them)
    const CostLds L;
    const int lane;

    // the instance
    int i, T;
    int32_t lam, slo;
    bool small;

    __device__ Solver(const CostArgs& args, uint32_t* mine, const double* r, const CostLds& l)
        : a(args), lds(mine), rc(r), L(l), lane(threadIdx.x & 63)
    {
    }

    // What a lane works on: one model and one batch size, cores lo .. last.
    struct Pair {
        RowHdr h;
        BatchHdr bh;
        double num, o2;    // numerator of the division by the cores; what the cores do not shrink
        double lam_per_M;  // at most lambda / (b 1e6)
        uint32_t s, j, lo, last, pcap;
        bool there;
    };

    __device__ __forceinline__ Pair pair_of(uint32_t s, uint32_t j, bool there) const
    {
        Pair p;
        p.there = there;
        p.s = there ? s : 0u;
        p.j = there ? j : 0u;
        const int32_t* raw = reinterpret_cast<const int32_t*>(lds + L.raw) + RAW * p.s;
        p.h = make_row_hdr(raw, 6u, lam, slo, T, (uint32_t)a.tick, DERIVE ? 0 : raw[6]);
        p.bh = make_batch_hdr(a.bl.b[p.j]);
        p.pcap = (uint32_t)raw[3];
        const uint32_t only = (uint32_t)raw[7];
        p.lo = only ? only : 1u;
        const uint32_t hi = only ? only : (uint32_t)a.c_max;
        // beyond the cap a candidate has the cap's latency and costs more
        const uint32_t reach = p.pcap > p.lo ? p.pcap : p.lo;
        p.last = hi < reach ? hi : reach;
        p.num = __builtin_fma(p.h.q, p.bh.b2, __builtin_fma(p.h.k, p.bh.b, p.h.a));
        p.o2 = __builtin_fma(p.h.d, p.bh.b, p.h.o);
        p.lam_per_M = p.h.lam * p.bh.rM * (1.0 - 0x1p-40);
        return p;
    }

    template <bool SMALL>
    __device__ __forceinline__ Eval eval(const Pair& p, uint32_t c) const
    {
        const uint32_t d = c < p.pcap ? c : p.pcap;
        const double dd = (double)d;
        const double rd = a.c_max <= RC_TABLE ? rc[d - 1u] : recip_below(dd);
        return eval_candidate_rd<QUEUE, SMALL, DERIVE ? N_DERIVED : N_GIVEN>(
            p.h, p.bh, dd, rd, (double)a.r_max, (double)a.tick, a.rtick);
    }

    // No candidate of the pair with fewer cores than this is feasible: its processing
    // time alone, num / c + o2, would exceed what the budget, less the least queueing
    // delay that goes with it, and the throughput with the most replicas leave.
    // Single precision, rounded down by far more than its error.
    __device__ __forceinline__ uint32_t first_core(const Pair& p) const
    {
        const double room = (double)T * (double)a.tick;
        const double n_max = DERIVE ? (double)a.r_max : p.h.n_given;
        double most = n_max * p.bh.M * p.h.rlam;
        const double wait = p.bh.w * p.h.rlam;
        const double least = QUEUE == THEMIS_QUEUE_PER_REPLICA && !DERIVE ? wait * n_max : wait;
        most = room - least < most ? room - least : most;
        if (QUEUE == THEMIS_QUEUE_PER_REPLICA && DERIVE) {
            // n >= lambda proc / (b 1e6), so the queue is at least (b - 1) / b proc
            const double both = room * p.bh.b * recip_below(2.0 * p.bh.b - 1.0) * (1.0 + 0x1p-40);
            most = both < most ? both : most;
        }
        const float left = (float)(most - p.o2) * 1.0001f;
        const float c = (float)p.num * __builtin_amdgcn_rcpf(left > 1.0f ? left : 1.0f) * 0.999f;
        uint32_t c0 = (uint32_t)__builtin_ceilf(c < 65536.0f ? c : 65536.0f);
        c0 = c0 > p.lo ? c0 : p.lo;
        return c0 < p.last ? c0 : p.last;
    }

    // At most the cost of every candidate of the pair with c cores or more, c up to
    // the cap: n >= 1 and n >= lambda (num / c + o2) / (b 1e6).
    __device__ __forceinline__ bool may_cost(const Pair& p, uint32_t c, uint32_t limit) const
    {
        if (!DERIVE) return (double)c * p.h.n_given <= (double)limit;
        return c <= limit && __builtin_fma((double)c, p.o2, p.num) * p.lam_per_M <= (double)limit;
    }

    // per model: cost << 15 | lt of the best candidate met so far; the same with the
    // index below it, complete after step A; lt of the fastest candidate
    __device__ __forceinline__ uint32_t* keys() const { return lds + L.key; }
    __device__ __forceinline__ unsigned long long* bests() const
    {
        return reinterpret_cast<unsigned long long*>(lds + L.best);
    }
    __device__ __forceinline__ uint32_t* fastest() const { return lds + L.fast; }

    __device__ __forceinline__ uint32_t pairs() const { return (uint32_t)(a.S * a.bl.n); }

    // Calls f(pair) for this lane's pair of every round of 64; lanes without one get a
    // pair with `there` unset.
    template <typename F>
    __device__ __forceinline__ void for_pairs(F f) const
    {
        const uint32_t P = pairs();
        for (uint32_t r = 0; r < P; r += 64u) {
            const uint32_t x = r + (uint32_t)lane;
            const uint32_t s = (x * a.nb_magic) >> 16;
            f(pair_of(s, x - s * (uint32_t)a.bl.n, x < P));
        }
    }

    // ---- results -----------------------------------------------------------------
    __device__ __forceinline__ void put(int32_t status, int32_t cost, int32_t ticks) const
    {
        if (lane != 0) return;
        a.status[i] = status;
        a.cost[i] = cost;
        a.ticks[i] = ticks;
        if (a.keep) {
            a.keep[a.kept.status + i] = status;
            a.keep[a.kept.cost + i] = cost;
            a.keep[a.kept.ticks + i] = ticks;
        }
    }

    __device__ __forceinline__ void put_none(int32_t status) const
    {
        put(status, -1, -1);
        const int words = 3 * a.S;
        for (int x = lane; x < words; x += 64) {
            a.cfg[(size_t)i * words + x] = 0;
            if (a.keep) a.keep[a.kept.cfg + (size_t)i * words + x] = 0;
        }
    }

    // lane s < S: index and cost of model s's candidate
    __device__ __forceinline__ void put_choice(uint32_t k, uint32_t cost) const
    {
        if (lane >= a.S) return;
        const uint32_t q = (k * a.k_magic) >> 20;
        const uint32_t c = q + 1u;
        const int32_t b = a.bl.b[k - q * (uint32_t)a.bl.n];
        // cost / c: the exact quotient is a whole number up to 32767, half of 1 / c away
        // from where the truncation would go wrong
        const uint32_t n = (uint32_t)(((float)cost + 0.5f) * __builtin_amdgcn_rcpf((float)c));
        int32_t* const out = a.cfg + ((size_t)i * a.S + lane) * 3;
        out[0] = (int32_t)c;
        out[1] = b;
        out[2] = (int32_t)n;
        if (a.keep) {
            int32_t* const kp = a.keep + a.kept.cfg + ((size_t)i * a.S + lane) * 3;
            kp[0] = (int32_t)c;
            kp[1] = b;
            kp[2] = (int32_t)n;
        }
    }

    // ---- step 0 ------------------------------------------------------------------
    // Inputs into LDS, input check.
    __device__ __forceinline__ bool load()
    {
        lam = a.lambda[i];
        slo = a.slo_us[i];
        int ok = in_range(lam, 1, THEMIS_VALUE_MAX) & in_range(slo, 0, a.slo_max);
        if (lane < a.S) {
            const size_t row = (size_t)i * a.S + lane;
            const int32_t* cf = a.coef + (a.coef_shared ? (size_t)lane : row) * a.cs;
            int32_t v[RAW];
#pragma unroll
            for (int x = 0; x < 5; ++x) v[x] = cf[x];
            v[5] = a.cs == 6 ? cf[5] : 0;
            v[6] = a.r_fixed ? a.r_fixed[row] : 0;
            v[7] = a.c_fixed ? a.c_fixed[row] : a.c_all;
            ok &= in_range(v[0], 0, THEMIS_VALUE_MAX) & in_range(v[1], 0, THEMIS_VALUE_MAX) &
                  in_range(v[2], 0, THEMIS_VALUE_MAX) & (int)(v[3] >= 1) &
                  in_range(v[4], 1, THEMIS_VALUE_MAX) & in_range(v[5], 0, THEMIS_VALUE_MAX);
            if (a.r_fixed) ok &= in_range(v[6], 1, a.r_max);
            if (a.c_fixed) ok &= in_range(v[7], 1, a.c_max);
            uint32_t* const raw = lds + L.raw + RAW * lane;
#pragma unroll
            for (int x = 0; x < RAW; ++x) raw[x] = (uint32_t)v[x];
            keys()[lane] = EMPTY;
            bests()[lane] = ~0ull;
            fastest()[lane] = LT_NONE;
            if (a.keep) {
                int32_t* const kc = a.keep + a.kept.coef + row * a.cs;
#pragma unroll
                for (int x = 0; x < 5; ++x) kc[x] = v[x];
                if (a.cs == 6) kc[5] = v[5];
                a.keep[a.kept.given + row] = v[6];
                a.keep[a.kept.only + row] = v[7];
            }
        }
        const bool valid = __ballot(!ok) == 0ull;
        // floor(slo / tick): the quotient lies at least half of 1 / tick above any whole
        // number below it, which the reciprocal's error (2^-44 relative) does not reach
        T = valid ? (int)(((double)slo + 0.5) * a.rtick) : -1;
        T = __builtin_amdgcn_readfirstlane(T);
        if (lane == 0) {
            a.tmeta[i] = T;
            if (a.keep) {
                a.keep[a.kept.lam + i] = valid ? lam : 0;
                a.keep[a.kept.slo + i] = slo;
            }
        }
        // row_is_small(), which is the same for all models of an instance
        small = (double)lam * (double)slo <= 0x1p42;
        wave_lds_fence();
        return valid;
    }

    // ---- steps 0 and A: returns false when x* > 0 ---------------------------------
    template <bool SMALL>
    __device__ __forceinline__ void least_costs() const
    {
        for_pairs([&](const Pair& p) {
            // fastest first: where the cap's candidate is infeasible the whole pair is
            uint32_t best = EMPTY, best_c = 0;
            if (p.there) {
                const Eval ev = eval<SMALL>(p, p.last);
                if (ev.lt >= 0) {
                    atomicMin(&fastest()[p.s], (uint32_t)ev.lt);
                    best = (__umul24((uint32_t)ev.n, p.last) << 15) | (uint32_t)ev.lt;
                    best_c = p.last;
                    atomicMin(&keys()[p.s], best);
                }
            }
            bool go = best != EMPTY;
            uint32_t c = go ? first_core(p) : 0u;
            wave_lds_fence();
            for (;;) {
                go = go && c < p.last && may_cost(p, c, keys()[p.s] >> 15);
                if (__ballot(go) == 0ull) break;
                if (go) {
                    const Eval ev = eval<SMALL>(p, c);
                    if (ev.lt >= 0) {
                        const uint32_t key = (__umul24((uint32_t)ev.n, c) << 15) | (uint32_t)ev.lt;
                        // (cores ascend, so of equal keys the first one met has the smaller
                        // index; the cap's, met first, has the largest)
                        if (key < best || (key == best && best_c == p.last)) best = key, best_c = c;
                        atomicMin(&keys()[p.s], key);
                    }
                    ++c;
                }
                wave_lds_fence();
            }
            if (best != EMPTY)
                atomicMin(&bests()[p.s],
                          ((unsigned long long)best << INDEX_BITS) |
                              ((best_c - 1u) * (uint32_t)a.bl.n + p.j));
            wave_lds_fence();
        });
    }

    // ---- step B / C ----------------------------------------------------------------
    // The table of (lt, index) by cost over base, W cells per model.
    template <bool SMALL>
    __device__ __forceinline__ void fill_table(int W) const
    {
        uint32_t* const tab = lds + L.tab;
        for (int x = lane; x < a.S * W; x += 64) tab[x] = EMPTY;
        wave_lds_fence();
        for_pairs([&](const Pair& p) {
            if (!p.there) return;
            const uint32_t base = keys()[p.s] >> 15;
            const uint32_t top = base + (uint32_t)W - 1u;
            for (uint32_t c = first_core(p); c <= p.last && may_cost(p, c, top); ++c) {
                const Eval ev = eval<SMALL>(p, c);
                const uint32_t cost = __umul24((uint32_t)ev.n, c);
                if (ev.lt >= 0 && cost <= top)
                    atomicMin(&tab[p.s * (uint32_t)W + (cost - base)],
                              ((uint32_t)ev.lt << INDEX_BITS) |
                                  ((c - 1u) * (uint32_t)a.bl.n + p.j));
            }
        });
        wave_lds_fence();
    }

    // The recurrence over W cells and, where it ends within the budget, the answer.
    __device__ __forceinline__ bool solve_window(int W) const
    {
        uint32_t* const tab = lds + L.tab;
        uint16_t* const rows = reinterpret_cast<uint16_t*>(lds + L.rows);  // row s at s * W
        int x_star = -1;
        uint32_t t_star = 0;
        for (int s = a.S - 1; s >= 0; --s) {
            uint32_t* const mine = tab + s * W;
            uint16_t* const row = rows + s * W;
            const uint16_t* const next = row + W;
            // drop what does not beat everything cheaper
            uint32_t low = LT_NONE;
            for (int x0 = 0; x0 < W; x0 += 64) {
                const int x = x0 + lane;
                const uint32_t e = mine[x];
                const uint32_t lt = e >> INDEX_BITS;  // EMPTY: above any budget too
                uint32_t incl = wave_scan<true>(lt);
                incl = incl < low ? incl : low;
                const uint32_t before = from_lane_below(incl, low);
                if (lt >= before) mine[x] = EMPTY;
                low = lane_value(incl, 63);
                if (s == a.S - 1) row[x] = (uint16_t)(incl < G_INF ? incl : G_INF);
            }
            wave_lds_fence();
            if (s < a.S - 1) {
                for (int x0 = 0; x0 < W; x0 += 64) {
                    const int x = x0 + lane;
                    uint32_t acc = G_INF;
                    for (int d0 = 0; d0 <= x0; d0 += 64) {
                        const uint32_t e = mine[d0 + lane];
                        unsigned long long m = __ballot(e != EMPTY);
                        while (m) {
                            const int l = __builtin_ctzll(m);
                            m &= m - 1ull;
                            const uint32_t lt = lane_value(e, l) >> INDEX_BITS;
                            const int y = x - d0 - l;
                            const uint32_t v = (uint32_t)next[y < 0 ? 0 : y] + lt;
                            acc = y >= 0 && v < acc ? v : acc;
                        }
                    }
                    row[x] = (uint16_t)acc;
                }
                wave_lds_fence();
            }
        }
        for (int x0 = 0; x0 < W; x0 += 64) {
            const uint32_t v = rows[x0 + lane];
            const unsigned long long m = __ballot(v <= (uint32_t)T);
            if (m) {
                const int l = __builtin_ctzll(m);
                x_star = x0 + l;
                t_star = lane_value(v, l);
                break;
            }
        }
        if (x_star < 0) return false;

        // forward: the smallest index among the candidates that continue an optimum
        uint32_t my_k = 0, my_cost = 0;
        uint32_t total = (uint32_t)x_star;
        uint32_t t = t_star;
        int x_left = x_star;
        for (int s = 0; s < a.S; ++s) {
            const uint32_t* const mine = tab + s * W;
            const uint16_t* const next = rows + (s + 1) * W;
            uint32_t key = EMPTY, key_lt = 0;
            int key_d = 0;
            for (int d0 = 0; d0 <= x_left; d0 += 64) {
                const int d = d0 + lane;
                uint32_t e = EMPTY, rest = 0;
                if (d <= x_left) {
                    e = mine[d];
                    rest = s + 1 < a.S ? (uint32_t)next[x_left - d] : 0u;
                }
                unsigned long long m = __ballot(e != EMPTY && (e >> INDEX_BITS) + rest == t);
                while (m) {
                    const int l = __builtin_ctzll(m);
                    m &= m - 1ull;
                    const uint32_t el = lane_value(e, l);
                    const uint32_t k = el & ((1u << INDEX_BITS) - 1u);
                    if (k < key) key = k, key_lt = el >> INDEX_BITS, key_d = d0 + l;
                }
            }
            if (key == EMPTY) {  // never expected
                put_none(THEMIS_INTERNAL);
                return true;
            }
            const uint32_t base = keys()[s] >> 15;
            total += base;
            if (lane == s) my_k = key, my_cost = base + (uint32_t)key_d;
            t -= key_lt;
            x_left -= key_d;
        }
        put(THEMIS_SOLVED, (int32_t)total, (int32_t)t_star);
        put_choice(my_k, my_cost);
        return true;
    }

    // ---- step D ---------------------------------------------------------------------
    // Candidate number x of model s in index order (64 at a time, one per lane).
    template <bool SMALL>
    __device__ __forceinline__ Eval candidate(int s, uint32_t x, uint32_t count, uint32_t& cost,
                                              uint32_t& k) const
    {
        const uint32_t q = (x * a.k_magic) >> 20;
        const Pair p = pair_of((uint32_t)s, x - q * (uint32_t)a.bl.n, true);
        const uint32_t c = p.lo + (x < count ? q : 0u);
        Eval ev = eval<SMALL>(p, c);
        if (x >= count) ev.lt = -1;
        cost = __umul24((uint32_t)ev.n, c);
        k = (c - 1u) * (uint32_t)a.bl.n + p.j;
        return ev;
    }

    // Rows over the budget, in this instance's part of the row region.  Candidates are
    // first entered into a table of least latencies by cost (as many costs per bin as
    // it takes) so that only those faster than everything in a cheaper bin are swept.
    template <bool SMALL>
    __device__ __forceinline__ void solve_by_budget(int W) const
    {
        const int bins = a.S * W;
        uint32_t* const tab = lds + L.tab;
        uint32_t* const list = lds + L.rows;  // lt | cost << 16
        const int cap = a.S * W / 2;          // entries of the list, a multiple of 32
        uint16_t* const rows = a.frow + (size_t)i * a.S * a.row_stride;
        const uint32_t nbat = (uint32_t)a.bl.n;
        for (int s = a.S - 1; s >= 0; --s) {
            uint16_t* const out = rows + (size_t)s * a.row_stride;
            const uint16_t* const next = out + a.row_stride;
            const bool first_model = s == a.S - 1;
            const Pair p0 = pair_of((uint32_t)s, 0u, true);
            const uint32_t count = (p0.last - p0.lo + 1u) * nbat;
            const uint32_t base = keys()[s] >> 15;
            int sh = 0;
            while ((a.r_max * a.c_max >> sh) >= bins) ++sh;
            for (int x = lane; x < bins; x += 64) tab[x] = LT_NONE;
            wave_lds_fence();
            for (uint32_t x0 = 0; x0 < count; x0 += 64u) {
                const uint32_t x = x0 + (uint32_t)lane;
                uint32_t cost, k;
                const Eval ev = candidate<SMALL>(s, x, count, cost, k);
                if (ev.lt >= 0) atomicMin(&tab[(cost - base) >> sh], (uint32_t)ev.lt);
            }
            wave_lds_fence();
            uint32_t low = LT_NONE;
            for (int x0 = 0; x0 < bins; x0 += 64) {
                const int x = x0 + lane;
                uint32_t incl = wave_scan<true>(tab[x]);
                incl = incl < low ? incl : low;
                tab[x] = from_lane_below(incl, low);  // least of all cheaper bins
                low = lane_value(incl, 63);
            }
            wave_lds_fence();
            for (int t = lane; t <= T; t += 64) out[t] = (uint16_t)F_INF;
            int n = 0;
            auto sweep = [&]() {
                wave_lds_fence();
                for (int t = lane; t - lane <= T; t += 64) {
                    uint32_t acc = t <= T ? (uint32_t)out[t] : F_INF;
                    for (int e = 0; e < n; ++e) {
                        const uint32_t w = list[e];
                        const int y = t - (int)(w & 0xFFFFu);
                        uint32_t v = F_INF;
                        if (y >= 0 && t <= T) v = (w >> 16) + (first_model ? 0u : (uint32_t)next[y]);
                        acc = v < acc ? v : acc;
                    }
                    if (t <= T) out[t] = (uint16_t)acc;
                }
                n = 0;
                wave_lds_fence();
            };
            for (uint32_t x0 = 0; x0 < count; x0 += 64u) {
                const uint32_t x = x0 + (uint32_t)lane;
                uint32_t cost, k;
                const Eval ev = candidate<SMALL>(s, x, count, cost, k);
                const bool use =
                    ev.lt >= 0 && tab[(cost - base) >> sh] > (uint32_t)ev.lt;
                const unsigned long long m = __ballot(use);
                if (n + (int)__builtin_popcountll(m) > cap) sweep();
                // (a list shorter than a wavefront takes its lanes in portions)
                unsigned long long todo = m;
                while (todo) {
                    const int rank = (int)__builtin_popcountll(todo & ((1ull << lane) - 1ull));
                    const bool in = ((todo >> lane) & 1ull) && n + rank < cap;
                    if (in) list[n + rank] = (uint32_t)ev.lt | (cost << 16);
                    const unsigned long long took = __ballot(in);
                    n += (int)__builtin_popcountll(took);
                    todo &= ~took;
                    if (todo) sweep();
                }
            }
            sweep();
            // the next model reads what other lanes wrote
            __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "workgroup");
        }
        const uint32_t best = rows[T];
        int t = T;
        for (int t0 = 0; t0 <= T; t0 += 64) {
            const unsigned long long m = __ballot(t0 + lane <= T && rows[t0 + lane <= T ? t0 + lane : T] == best);
            if (m) {
                t = t0 + __builtin_ctzll(m);
                break;
            }
        }
        const int t_star = t;
        uint32_t my_k = 0, my_cost = 0, target = best;
        for (int s = 0; s < a.S; ++s) {
            const uint16_t* const next = rows + (size_t)(s + 1) * a.row_stride;
            const Pair p0 = pair_of((uint32_t)s, 0u, true);
            const uint32_t count = (p0.last - p0.lo + 1u) * nbat;
            bool found = false;
            for (uint32_t x0 = 0; x0 < count && !found; x0 += 64u) {
                const uint32_t x = x0 + (uint32_t)lane;
                uint32_t cost, k;
                const Eval ev = candidate<SMALL>(s, x, count, cost, k);
                uint32_t rest = F_INF;
                if (ev.lt >= 0 && ev.lt <= t) rest = s + 1 < a.S ? (uint32_t)next[t - ev.lt] : 0u;
                const unsigned long long m = __ballot(rest < F_INF && cost + rest == target);
                if (m) {  // candidates are in index order: the first is the smallest
                    const int l = __builtin_ctzll(m);
                    const uint32_t ck = lane_value(k, l), cc = lane_value(cost, l);
                    if (lane == s) my_k = ck, my_cost = cc;
                    target -= cc;
                    t -= (int)lane_value((uint32_t)ev.lt, l);
                    found = true;
                }
            }
            if (!found) {  // never expected
                put_none(THEMIS_INTERNAL);
                return;
            }
        }
        put(THEMIS_SOLVED, (int32_t)best, t_star);
        put_choice(my_k, my_cost);
    }

    // Solves instance i.  LAST: whatever it takes; else false when the first window
    // does not suffice.
    template <bool LAST>
    __device__ __forceinline__ bool solve(int inst)
    {
        i = inst;
        if (!load()) {
            if (!a.sparse) put_none(THEMIS_INVALID);
            return true;
        }
        if (small)
            least_costs<true>();
        else
            least_costs<false>();
        uint32_t key = 0, k = 0, fast = 0;
        if (lane < a.S) {
            const unsigned long long best = bests()[lane];
            key = (uint32_t)(best >> INDEX_BITS);
            k = (uint32_t)best & ((1u << INDEX_BITS) - 1u);
            fast = fastest()[lane];
        }
        if (wave_sum(fast) > (uint32_t)T) {
            put_none(THEMIS_INFEASIBLE);
            return true;
        }
        const uint32_t ticks = wave_sum(key & 0x7FFFu);
        if (ticks <= (uint32_t)T) {
            put(THEMIS_SOLVED, (int32_t)wave_sum(key >> 15), (int32_t)ticks);
            put_choice(k, key >> 15);
            return true;
        }
        // (a marked instance has been through the first window)
        for (int W = LAST && a.hard ? 256 : 64;; W *= 4) {
            W = W < a.window ? W : a.window;
            if (small)
                fill_table<true>(W);
            else
                fill_table<false>(W);
            if (solve_window(W)) return true;
            if (!LAST) return false;
            if (W >= a.window) break;
        }
        if (LAST) {
            if (small)
                solve_by_budget<true>(a.window);
            else
                solve_by_budget<false>(a.window);
        }
        return true;
    }
};

// LAST: this launch finishes every instance it takes; the instances are those
// marked in `hard` by the launch before it, or all of them when `hard` is null.
template <int QUEUE, bool DERIVE, bool LAST>
__global__ __launch_bounds__(256) void kc_solve(CostArgs a)
{
    extern __shared__ uint32_t cost_smem[];
    double* const rc = reinterpret_cast<double*>(cost_smem);
    const int rc_n = a.c_max <= RC_TABLE ? a.c_max : 0;
    for (int c = (int)threadIdx.x; c < rc_n; c += (int)blockDim.x) rc[c] = recip_below((double)(c + 1));
    const CostLds L = cost_lds(a.S, a.window);
    const int nw = (int)blockDim.x >> 6;
    const int w = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    uint32_t* const mine = cost_smem + ((2 * rc_n + 3) & ~3) + w * L.words;
    // what the class lists and the state word say about this workspace from now on:
    // no tables, the inputs and results in the table region
    if ((!LAST || !a.hard) && blockIdx.x == 0 && (int)threadIdx.x <= STATE_WORD)
        a.ctrl[threadIdx.x] =
            (int)threadIdx.x < STATE_WORD || !a.keep ? 0 : STATE_KEPT_IN_TABLE | (DERIVE ? 0 : STATE_GIVEN);
    __syncthreads();
    Solver<QUEUE, DERIVE> sv(a, mine, rc, L);
    const int me = (int)blockIdx.x * nw + w, all = (int)gridDim.x * nw;
    if (!LAST) {
        if (me >= a.N) return;
        const bool done = sv.template solve<false>(me);
        if (sv.lane == 0) a.hard[me] = done ? 0 : 1;
    } else {
        // lane l of a wavefront looks at every all-th instance: the marked ones spread
        // over the wavefronts whatever their order
        for (long long i0 = me; i0 < a.N; i0 += 64ll * all) {
            const long long mine_i = i0 + (long long)sv.lane * all;
            const bool take = mine_i < a.N && (!a.hard || a.hard[mine_i] != 0);
            unsigned long long m = __ballot(take);
            while (m) {
                const int l = __builtin_ctzll(m);
                m &= m - 1ull;
                sv.template solve<true>((int)(i0 + (long long)l * all));
                wave_lds_fence();
            }
        }
    }
}

constexpr size_t LDS_PER_CU = 160 * 1024;

}  // namespace

bool cost_solve_serves(const Layout& L) { return L.S <= COST_MAX_STAGES; }

hipError_t launch_cost_solve(const themis_problem_t& p, const Layout& L, const int32_t* d_coef,
                             const int32_t* d_lambda, const int32_t* d_slo_us,
                             const int32_t* d_r_fixed, int32_t* d_status, int32_t* d_cost,
                             int32_t* d_ticks, int32_t* d_cfg, char* ws, hipStream_t st,
                             const PassOpts& opts)
{
    CostArgs a{};
    a.coef = d_coef;
    a.lambda = d_lambda;
    a.slo_us = d_slo_us;
    a.r_fixed = d_r_fixed;
    a.c_fixed = opts.c_fixed;
    a.status = d_status;
    a.cost = d_cost;
    a.ticks = d_ticks;
    a.cfg = d_cfg;
    a.tmeta = (int32_t*)(ws + L.tmeta_off);
    a.hard = (int32_t*)(ws + L.ans_off);
    a.ctrl = (int32_t*)(ws + L.ctrl_off);
    a.frow = (uint16_t*)(ws + L.frow_off);
    a.kept = make_keep_layout(p, L);
    a.keep = opts.inspectable ? (int32_t*)(ws + L.step_off) : nullptr;
    a.bl.n = p.n_batch;
    for (int j = 0; j < p.n_batch; ++j) a.bl.b[j] = p.batch_sizes[j];
    a.N = L.N;
    a.S = L.S;
    a.cs = p.profile_form == THEMIS_PROFILE_EQ1 ? 6 : 5;
    a.c_max = p.c_max;
    a.r_max = p.r_max;
    a.tick = p.tick_us;
    a.slo_max = p.slo_max_us;
    a.coef_shared = p.coef_shared;
    a.c_all = opts.c_all;
    a.sparse = opts.sparse;
    a.row_stride = L.row_stride;
    a.nb_magic = (65536u + (uint32_t)p.n_batch - 1u) / (uint32_t)p.n_batch;
    a.k_magic = ((1u << 20) + (uint32_t)p.n_batch - 1u) / (uint32_t)p.n_batch;
    a.rtick = (1.0 / (double)p.tick_us) * (1.0 - 0x1p-45);

    const size_t rc_bytes = p.c_max <= RC_TABLE ? ((2 * (size_t)p.c_max + 3) & ~(size_t)3) * 4 : 0;
    auto lds_for = [&](int waves, int window) {
        return rc_bytes + (size_t)waves * cost_lds(L.S, window).words * sizeof(uint32_t);
    };
    // the largest window that leaves `per_cu` workgroups of a wavefront on a compute
    // unit, no larger than the costs of a pipeline can spread
    auto widest = [&](size_t per_cu) {
        int w = 64;
        while (w + 64 <= 8192 && w < L.S * p.r_max * p.c_max &&
               lds_for(1, w + 64) <= LDS_PER_CU / per_cu - 512)
            w += 64;
        return w;
    };
    auto launch = [&](auto kernel, int grid, int waves, size_t lds) -> hipError_t {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kernel),
                                           hipFuncAttributeMaxDynamicSharedMemorySize,
                                           (int)(LDS_PER_CU - 1024));
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(kernel, dim3((unsigned)grid), dim3(64 * waves), lds, st, a);
        return hipGetLastError();
    };
    const int cus = compute_units();
    auto run = [&](auto q_tag, auto d_tag) -> hipError_t {
        constexpr int Q = decltype(q_tag)::value;
        constexpr bool D = decltype(d_tag)::value;
        if (L.N <= 4 * cus) {
            // one launch, a workgroup per instance, whatever window four of them leave
            // each other on a compute unit
            a.hard = nullptr;
            a.window = widest(4);
            return launch(&kc_solve<Q, D, true>, L.N, 1, lds_for(1, a.window));
        }
        constexpr int WAVES = 4;
        a.window = 64;
        hipError_t e = launch(&kc_solve<Q, D, false>, (L.N + WAVES - 1) / WAVES, WAVES,
                              lds_for(WAVES, a.window));
        if (e != hipSuccess) return e;
        a.window = widest(4);
        return launch(&kc_solve<Q, D, true>, 4 * cus, 1, lds_for(1, a.window));
    };
    auto by_replicas = [&](auto q_tag) -> hipError_t {
        return d_r_fixed ? run(q_tag, std::false_type{}) : run(q_tag, std::true_type{});
    };
    switch (p.queue_model) {
    case THEMIS_QUEUE_SHARED:
        return by_replicas(std::integral_constant<int, THEMIS_QUEUE_SHARED>{});
    case THEMIS_QUEUE_WORST_CASE:
        return by_replicas(std::integral_constant<int, THEMIS_QUEUE_WORST_CASE>{});
    default: return by_replicas(std::integral_constant<int, THEMIS_QUEUE_PER_REPLICA>{});
    }
}

}  // namespace themis
