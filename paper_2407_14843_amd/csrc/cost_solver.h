// One wavefront's solve of one instance, for the kernels of cost_solve.hip and
// cost_multi.hip; the method is described in cost_solve.hip.
#pragma once

#include "candidate_eval.h"
#include "instance_queue.h"
#include "themis_internal.h"
#include "wave_ops.h"

#include <type_traits>

namespace themis {
namespace {

constexpr uint32_t LT_NONE = 1u << 22;       // "no candidate": above any sum of 64 budgets
constexpr uint32_t EMPTY = 0xFFFFFFFFu;      // empty cell of the (lt, index) table
constexpr int INDEX_BITS = 13;               // candidate indices are below 8192
constexpr uint32_t G_INF = 0x8000u;          // row cell beyond any budget

// a batch size b, and recip_below(b * 1e6)
struct __attribute__((aligned(16))) BatchConst {
    double b, rM;
};

struct CostArgs {
    const int32_t *coef, *lambda, *slo_us, *r_fixed, *c_fixed;
    const int32_t* lambda2;  // stability test: the predicted rates
    int32_t *status, *cost, *ticks, *cfg;
    int32_t *status2, *cost2, *ticks2, *cfg2;  // results of the second kind, see ROLE
    int32_t *lambda_v, *stable;
    int32_t* tmeta;     // budgets, for calls that inspect the workspace afterwards
    const int32_t* list;  // the instances to solve (LISTED)
    int32_t* ctrl;
    uint16_t* frow;     // rows of steps W and D
    int32_t* keep;      // inputs and results for such calls, or null
    KeepLayout kept;
    BatchConst bc[THEMIS_MAX_BATCH];
    int32_t n_batch;
    int32_t S, cs, c_max, r_max, tick, slo_max, coef_shared, c_all, row_stride;
    int32_t window;     // cells of the largest window with rows in LDS, a multiple of 64
    int32_t window_hbm; // and in HBM (no larger than the other: none)
    uint32_t magic;     // index_magic() of n_batch
    double rtick;
};

// LDS words of one wavefront.  From `tab` on, step B takes 32 words per model, a table
// and rows of sixteen words; the window of 64 cells a table of 64 words per model and
// S + 1 rows of 16-bit cells, each with a guard cell (and one of padding) in front; wider
// windows a table of one model and such rows.
struct CostLds {
    int best, key, fast, pin, tab, rows, words;
};
__host__ __device__ inline CostLds cost_lds(int S, int window)
{
    CostLds l;
    l.best = 0;  // two words per model
    l.key = 2 * S;
    l.fast = l.key + S;
    l.pin = l.fast + S;
    l.tab = (l.pin + S + 3) & ~3;
    l.rows = l.tab + window;
    const int c = l.rows + (S + 1) * (window + 2) / 2, b = l.tab + 64 * S + (S + 1) * 33;
    l.words = ((c > b ? c : b) + 3) & ~3;
    return l;
}

// lo <= v <= hi, 0 <= lo
__device__ __forceinline__ bool in_range(int32_t v, int32_t lo, int32_t hi)
{
    return (uint32_t)v - (uint32_t)lo <= (uint32_t)(hi - lo);
}

// four consecutive words on a word boundary
typedef int32_t words4 __attribute__((ext_vector_type(4), aligned(4)));

// The launch's arguments where they lie, for code that takes them by address: in the
// constant address space, so that uniform reads stay scalar loads.
typedef const __attribute__((address_space(4))) CostArgs* ArgsPtr;

extern __shared__ uint32_t cost_smem[];

// The value D lanes down within the rows of sixteen that `ROWS` names; `fill` where
// there is none, x itself in the other rows.
template <int D, int ROWS = 0xF>
__device__ __forceinline__ uint32_t row_shifted(uint32_t x, uint32_t fill)
{
    const uint32_t old = ROWS == 0xF ? fill : x;
    return (uint32_t)__builtin_amdgcn_update_dpp((int)old, (int)x, 0x110 | D, ROWS, 0xF, false);
}

__device__ __forceinline__ uint32_t least(uint32_t a, uint32_t b) { return a < b ? a : b; }

// The least of the four lanes that have the same place in the rows of sixteen, in all
// of them.
__device__ __forceinline__ uint32_t least_of_rows(uint32_t x)
{
    typedef uint32_t two __attribute__((ext_vector_type(2)));
    const two h = __builtin_amdgcn_permlane32_swap(x, x, false, false);
    x = least(h.x, h.y);
    const two q = __builtin_amdgcn_permlane16_swap(x, x, false, false);
    return least(q.x, q.y);
}

// What a solve is for, which says where its results go: PLAIN, the caller's results and
// the record; QUIET, the same without the record; SECOND, the second set of results;
// PINNED, the second set and the record, with the cores of every model taken from LDS.
enum { PLAIN, QUIET, SECOND, PINNED };
// Besides the status of an instance: the steps so far did not suffice.
constexpr int UNFINISHED = -1;

template <int QUEUE, bool DERIVE, int ROLE>
__device__ __attribute__((noinline)) int solve_further(uint64_t args, int i, int T, int32_t lam,
                                                       int32_t slo);

// One wavefront's view of the instance it works on.  ONE: its (model, batch size)
// pairs fit the lanes, so every lane keeps its own from step A on.
template <int QUEUE, bool DERIVE, bool ONE, int ROLE = PLAIN>
struct Solver {
    const __attribute__((address_space(4))) CostArgs& a;
    uint32_t* const lds;  // the wavefront's words: a workgroup is one wavefront
    const CostLds L;
    const int lane;

    // the instance
    int i, T;
    int32_t lam, slo;
    int32_t lane_b;  // lane j: batch size j

    __device__ __forceinline__ explicit Solver(ArgsPtr args)
        : a(*args), lds(cost_smem), L(cost_lds(args->S, args->window)),
          lane(threadIdx.x)
    {
    }

    // What a lane works on: one model and one batch size, cores lo .. last.
    struct Pair {
        RowHdr h;
        BatchHdr bh;
        double num, fixed;  // numerator of the division by the cores; what they do not shrink
        double lam_per_M;   // at most lambda / (b 1e6)
        uint32_t s, j, lo, last, pcap;
        bool there, valid;
    };

    __device__ __forceinline__ Pair pair_of(uint32_t s, uint32_t j, bool there) const
    {
        Pair p;
        p.there = there;
        p.s = there ? s : 0u;
        p.j = there ? j : 0u;
        const double b = a.bc[p.j].b;
        const double rM = a.bc[p.j].rM;
        const size_t row0 = (size_t)i * a.S;
        const int32_t* const cf = a.coef + (a.coef_shared ? 0 : row0 * a.cs) + p.s * (uint32_t)a.cs;
        const words4 c4 = *reinterpret_cast<const words4*>(cf);
        int32_t v[6] = {c4.x, c4.y, c4.z, c4.w, cf[4], 0};
        if (a.cs == 6) v[5] = cf[5];
        const int32_t given = DERIVE ? 0 : (a.r_fixed + row0)[p.s];
        const int32_t only = ROLE == PINNED ? (int32_t)lds[L.pin + p.s]
                             : a.c_fixed    ? (a.c_fixed + row0)[p.s]
                                            : a.c_all;
        // a, k, q, d in 0 .. max, p >= 1, o in 1 .. max
        uint32_t top = (uint32_t)v[0] > (uint32_t)v[1] ? (uint32_t)v[0] : (uint32_t)v[1];
        top = (uint32_t)v[2] > top ? (uint32_t)v[2] : top;
        top = (uint32_t)v[5] > top ? (uint32_t)v[5] : top;
        p.valid = top <= (uint32_t)THEMIS_VALUE_MAX && v[3] >= 1 && in_range(v[4], 1, THEMIS_VALUE_MAX);
        if (!DERIVE) p.valid = p.valid && in_range(given, 1, a.r_max);
        if (ROLE != PINNED && a.c_fixed) p.valid = p.valid && in_range(only, 1, a.c_max);
        p.h = make_row_hdr(v, 6u, lam, slo, T, (uint32_t)a.tick, given);
        p.bh.b = b;
        p.bh.b2 = b * b;
        p.bh.M = b * 1.0e6;
        p.bh.rM = rM;
        p.bh.w = p.bh.M - 1.0e6;
        p.pcap = (uint32_t)v[3];
        p.lo = only > 0 ? (uint32_t)only : 1u;
        const uint32_t hi = only > 0 ? (uint32_t)only : (uint32_t)a.c_max;
        // beyond the cap a candidate has the cap's latency and costs more
        const uint32_t reach = p.pcap > p.lo ? p.pcap : p.lo;
        p.last = hi < reach ? hi : reach;
        p.num = __builtin_fma(p.h.q, p.bh.b2, __builtin_fma(p.h.k, p.bh.b, p.h.a));
        p.fixed = __builtin_fma(p.h.d, p.bh.b, p.h.o);
        p.lam_per_M = p.h.lam * p.bh.rM * (1.0 - 0x1p-40);
        return p;
    }

    // The pair kept from another rate at the rate `lam` (where pairs are not kept they are
    // formed at that rate anyway).
    __device__ __forceinline__ Pair at_rate(Pair p) const
    {
        if (ONE) {
            p.h.lam = (double)lam;
            p.h.rlam = recip_below(p.h.lam);
            p.h.lt_den = p.h.lam * (double)a.tick;
            p.h.rlt_den = recip_below(p.h.lt_den);
            p.lam_per_M = p.h.lam * p.bh.rM * (1.0 - 0x1p-40);
        }
        return p;
    }

    // this lane's pair of the round that starts with pair r
    __device__ __forceinline__ Pair pair_of_round(uint32_t r) const
    {
        const uint32_t x = r + (uint32_t)lane;
        const uint32_t s = index_quotient(x, a.magic);  // x < 64 * 16 + 64
        return pair_of(s, x - s * (uint32_t)a.n_batch, x < (uint32_t)(a.S * a.n_batch));
    }

    // Calls f(pair) for this lane's pair of every round of 64; lanes without one get a
    // pair with `there` unset.  `mine`: the pair, where there is one round only.
    template <typename F>
    __device__ __forceinline__ void for_pairs(const Pair& mine, F f) const
    {
        if constexpr (ONE) {
            f(mine);
        } else {
            for (uint32_t r = 0; r < (uint32_t)(a.S * a.n_batch); r += 64u) f(pair_of_round(r));
        }
    }

    // Reciprocals of the core counts, for loops over them: lane l holds that of l + 1, a
    // lane fetches the one it needs (three instructions instead of nine).
    struct Recips {
        double mine;
        bool held;
    };
    __device__ __forceinline__ Recips recips() const
    {
        return Recips{recip_below((double)(lane + 1)), a.c_max <= 64};
    }
    __device__ __forceinline__ double recip(const Recips& r, uint32_t d) const
    {
        return r.held ? __shfl(r.mine, (int)d - 1, 64) : recip_below((double)d);
    }

    // rd: recip_below() of the cores, or of the cap beyond it
    template <bool SMALL>
    __device__ __forceinline__ Eval eval(const Pair& p, double rd) const
    {
        return eval_parts<QUEUE, SMALL, DERIVE ? N_DERIVED : N_GIVEN>(
            p.h, p.bh, p.num, p.fixed, rd, (double)a.r_max, (double)a.tick, a.rtick);
    }

    static __device__ __forceinline__ uint32_t speed(const Pair& p, uint32_t c)
    {
        return c < p.pcap ? c : p.pcap;
    }

    // No candidate of the pair with fewer cores than this is feasible (last + 1: none
    // is): its processing time alone, num / c + fixed, would exceed what the budget,
    // less the least queueing delay that goes with it, and the throughput with the
    // most replicas leave.  Single precision; every term is rounded to the safe side
    // by more than its error (some units in 2^-24).
    __device__ __forceinline__ uint32_t first_core(const Pair& p) const
    {
        constexpr float UP = 1.00001f, DOWN = 0.99999f;
        const float room = (float)((double)T * (double)a.tick) * UP;
        const float rl = __builtin_amdgcn_rcpf((float)lam);
        const float b = (float)p.bh.b;
        const float n_max = DERIVE ? (float)a.r_max : (float)p.h.n_given;
        float most = n_max * (float)p.bh.M * rl * UP;
        float wait = (float)p.bh.w * rl * DOWN;
        if (QUEUE == THEMIS_QUEUE_PER_REPLICA && !DERIVE) wait *= n_max;
        most = room - wait < most ? room - wait : most;
        if (QUEUE == THEMIS_QUEUE_PER_REPLICA && DERIVE) {
            // n >= lambda proc / (b 1e6), so the queue is at least (b - 1) / b proc
            const float both = room * b * __builtin_amdgcn_rcpf(2.0f * b - 1.0f) * UP;
            most = both < most ? both : most;
        }
        const float left = most - (float)p.fixed * DOWN;
        const float c = (float)p.num * __builtin_amdgcn_rcpf(left) * DOWN;
        if (!(left > 0.0f) || c > (float)p.last) return p.last + 1u;
        const uint32_t c0 = (uint32_t)__builtin_ceilf(c);
        return c0 > p.lo ? c0 : p.lo;
    }

    // Whether a candidate of the pair with c cores or more can cost as little as
    // `limit`: n >= 1 and n >= lambda (num / c + fixed) / (b 1e6).
    __device__ __forceinline__ bool may_cost(const Pair& p, uint32_t c, uint32_t limit) const
    {
        if (!DERIVE) return (double)c * p.h.n_given <= (double)limit;
        return c <= limit &&
               __builtin_fma((double)c, p.fixed, p.num) * p.lam_per_M <= (double)limit;
    }

    // per model: cost << 15 | lt of the best candidate met so far; the same with the
    // index below it, complete after step A; lt << 15 | cost of the fastest candidate at
    // the cap
    __device__ __forceinline__ uint32_t* keys() const { return lds + L.key; }
    __device__ __forceinline__ unsigned long long* bests() const
    {
        return reinterpret_cast<unsigned long long*>(lds + L.best);
    }
    __device__ __forceinline__ uint32_t* fastest() const { return lds + L.fast; }

    // Sum over the lanes below S of values that are zero elsewhere, as a uniform value.
    __device__ __forceinline__ uint32_t sum_models(uint32_t x) const
    {
        if (a.S <= 16) return lane_value(segmented_scan<false>(x, 0u, 16u), 15);
        return wave_sum(x);
    }

    // ---- results -----------------------------------------------------------------
    // this instance's record for the calls that look at the workspace afterwards
    __device__ __forceinline__ int32_t* record() const { return a.keep + (size_t)i * a.kept.words; }
    __device__ __forceinline__ bool records() const
    {
        return (ROLE == PLAIN || ROLE == PINNED) && a.keep;
    }
    // where configurations go
    __device__ __forceinline__ int32_t* config() const
    {
        return (ROLE == SECOND || ROLE == PINNED ? a.cfg2 : a.cfg) + (size_t)i * a.S * 3;
    }

    __device__ __forceinline__ void record_result(int32_t status, int32_t cost, int32_t ticks,
                                                  SolveStep step) const
    {
        if (!records() || lane != 0) return;
        int32_t* const kp = record();
        kp[KEEP_STATUS] = status | step << KEEP_STEP;
        kp[KEEP_COST] = cost;
        kp[KEEP_TICKS] = ticks;
    }

    __device__ __forceinline__ void put(int32_t status, int32_t cost, int32_t ticks,
                                        SolveStep step = BY_A) const
    {
        constexpr bool TWO = ROLE == SECOND || ROLE == PINNED;
        if (lane == 0) {
            (TWO ? a.status2 : a.status)[i] = status;
            (TWO ? a.cost2 : a.cost)[i] = cost;
            (TWO ? a.ticks2 : a.ticks)[i] = ticks;
        }
        record_result(status, cost, ticks, step);
    }

    // `amount`: what the result says for cost and ticks
    __device__ __forceinline__ void put_none(int32_t status, int32_t amount = -1) const
    {
        put(status, amount, amount);
        int32_t* const out = config();
        for (int x = lane; x < 3 * a.S; x += 64) {
            out[x] = 0;
            if (records()) record()[a.kept.cfg + x] = 0;
        }
    }

    // lane s < S: index and cost of model s's candidate
    __device__ __forceinline__ void put_choice(uint32_t k, uint32_t cost) const
    {
        const uint32_t q = index_quotient(k, a.magic);
        const uint32_t c = q + 1u;
        const int32_t b = __shfl(lane_b, (int)(k - q * (uint32_t)a.n_batch), 64);
        if (lane >= a.S) return;
        // cost / c: the exact quotient is a whole number up to 32767, half of 1 / c away
        // from where the truncation would go wrong
        const uint32_t n = (uint32_t)(((float)cost + 0.5f) * __builtin_amdgcn_rcpf((float)c));
        const uint32_t off = 3u * (uint32_t)lane;
        int32_t* const out = config();
        out[off] = (int32_t)c;
        out[off + 1u] = b;
        out[off + 2u] = (int32_t)n;
        if (records()) {
            int32_t* const kp = record() + a.kept.cfg;
            kp[off] = (int32_t)c;
            kp[off + 1u] = b;
            kp[off + 2u] = (int32_t)n;
        }
    }

    // The instance's inputs into its record, see STATE_WORD.  `word`: word `lane` of the
    // coefficients, loaded with the rest of the inputs.
    __device__ __forceinline__ bool keeps_coef() const
    {
        return records() && !a.coef_shared;  // shared: see mark_workspace()
    }
    __device__ __forceinline__ void keep_inputs(bool valid, int32_t word) const
    {
        if (!records()) return;
        int32_t* const kp = record();
        if (keeps_coef()) {
            const int words = a.S * a.cs;
            if (lane < words) (kp + a.kept.coef)[lane] = word;
            for (int x = lane + 64; x < words; x += 64)
                (kp + a.kept.coef)[x] = (a.coef + (size_t)i * words)[x];
        }
        if (!DERIVE && lane < a.S)
            (kp + a.kept.given)[lane] = (a.r_fixed + (size_t)i * a.S)[lane];
        if (ROLE == PINNED && lane < a.S) (kp + a.kept.only)[lane] = (int32_t)lds[L.pin + lane];
        if (ROLE != PINNED && a.c_fixed && lane < a.S)
            (kp + a.kept.only)[lane] = (a.c_fixed + (size_t)i * a.S)[lane];
        if (lane == 0) {
            kp[KEEP_LAM] = valid ? lam : 0;
            kp[KEEP_SLO] = slo;
        }
    }

    // ---- step A ------------------------------------------------------------------
    template <bool SMALL>
    __device__ __forceinline__ void least_costs(const Pair& first) const
    {
        for_pairs(first, [&](const Pair& p) {
            uint32_t best = EMPTY, best_c = 0;
            auto meet = [&](uint32_t c, double rd) {
                const Eval ev = eval<SMALL>(p, rd);
                if (ev.lt >= 0) {
                    const uint32_t key = (__umul24((uint32_t)ev.n, c) << 15) | (uint32_t)ev.lt;
                    // (cores ascend: of equal keys the first one met has the smaller index)
                    if (key < best) best = key, best_c = c;
                    atomicMin(&keys()[p.s], key);
                }
            };
            auto goes_on = [&](uint32_t c) {
                return c <= p.last && may_cost(p, c, keys()[p.s] >> 15);
            };
            // most pipelines at low rates are done with the first core count
            uint32_t c = p.lo;
            if (p.there) meet(c, recip_below((double)speed(p, c)));
            wave_lds_fence();
            ++c;
            bool go = p.there && goes_on(c);
            if (__ballot(go) != 0ull) {
                const uint32_t c0 = first_core(p);
                c = c0 > c ? c0 : c;
                const Recips rc = recips();
                for (;;) {
                    go = go && goes_on(c);
                    if (__ballot(go) == 0ull) break;
                    const double rd = recip(rc, go ? speed(p, c) : 1u);
                    if (go) meet(c++, rd);
                    wave_lds_fence();
                }
            }
            if (best != EMPTY)
                atomicMin(&bests()[p.s],
                          ((unsigned long long)best << INDEX_BITS) |
                              ((best_c - 1u) * (uint32_t)a.n_batch + p.j));
        });
        wave_lds_fence();
    }

    // ---- step F ------------------------------------------------------------------
    template <bool SMALL>
    __device__ __forceinline__ uint32_t fastest_ticks(const Pair& first) const
    {
        if (lane < a.S) fastest()[lane] = EMPTY;
        wave_lds_fence();
        for_pairs(first, [&](const Pair& p) {
            if (!p.there) return;
            const Eval ev = eval<SMALL>(p, recip_below((double)speed(p, p.last)));
            if (ev.lt >= 0)
                atomicMin(&fastest()[p.s],
                          (uint32_t)ev.lt << 15 | __umul24((uint32_t)ev.n, p.last));
        });
        wave_lds_fence();
        return sum_models(lane < a.S ? fastest()[lane] >> 15 : 0u);  // none: beyond any budget
    }

    // ---- step B ------------------------------------------------------------------
    static __device__ __forceinline__ uint32_t entry(const Eval& ev, uint32_t k)
    {
        return ((uint32_t)ev.lt << INDEX_BITS) | k;
    }

    // The table of (lt, index) by cost over base, W cells per model.
    template <bool SMALL, int W>
    __device__ __forceinline__ void fill_all(const Pair& first) const
    {
        uint32_t* const tab = lds + L.tab;
        for (int x = lane; x < a.S * W; x += 64) tab[x] = EMPTY;
        const Recips rc = recips();
        wave_lds_fence();
        for_pairs(first, [&](const Pair& p) {
            const uint32_t base = keys()[p.s] >> 15;
            const uint32_t top = base + (uint32_t)W - 1u;
            uint32_t* const mine = tab + p.s * (uint32_t)W;
            auto enter = [&](const Eval& ev, uint32_t c) {
                const uint32_t cost = __umul24((uint32_t)ev.n, c);
                if (ev.lt >= 0 && cost <= top)
                    atomicMin(&mine[cost - base], entry(ev, (c - 1u) * (uint32_t)a.n_batch + p.j));
            };
            // two at a time: their chains of dependent operations fill each other's waits
            uint32_t c = first_core(p);
            for (;;) {
                const bool go = p.there && c <= p.last && may_cost(p, c, top);
                if (__ballot(go) == 0ull) break;
                const uint32_t c1 = c < p.last ? c + 1u : c;
                const double r0 = recip(rc, go ? speed(p, c) : 1u);
                const double r1 = recip(rc, go ? speed(p, c1) : 1u);
                if (go) {
                    const Eval e0 = eval<SMALL>(p, r0), e1 = eval<SMALL>(p, r1);
                    enter(e0, c);
                    enter(e1, c1);
                    c += 2u;
                }
            }
        });
        wave_lds_fence();
    }

    // Forward over the models, with the table of W <= 64 cells per model: the smallest
    // index among the candidates that continue an optimum of x cells over base and
    // `ticks`.  rest(s, y): cell y of row s + 1; lane s: base of model s.
    template <int W, typename F>
    __device__ __forceinline__ int read_out(uint32_t total, uint32_t ticks, int x,
                                            uint32_t my_base, F rest) const
    {
        constexpr uint32_t INDEX = (1u << INDEX_BITS) - 1u;
        const uint32_t* const tab = lds + L.tab;
        uint32_t t = ticks, my_k = 0, my_cost = my_base;
        const int d = lane & (W - 1);
        uint32_t e = tab[d];
        for (int s = 0; s < a.S; ++s) {
            const bool more_models = s + 1 < a.S;
            const uint32_t r = more_models ? rest(s, x >= d ? x - d : 0) : 0u;
            const uint32_t e_next = more_models ? tab[(s + 1) * W + d] : 0u;
            unsigned long long who = __ballot(d <= x && (e >> INDEX_BITS) + r == t);
            if (W < 64) who &= (1ull << (W & 63)) - 1ull;
            if (who == 0ull) {  // never expected
                put_none(THEMIS_INTERNAL);
                return THEMIS_INTERNAL;
            }
            int l = __builtin_ctzll(who);
            uint32_t el = lane_value(e, l);
            for (unsigned long long more = who & (who - 1ull); more; more &= more - 1ull) {
                const int l2 = __builtin_ctzll(more);
                const uint32_t e2 = lane_value(e, l2);
                if ((e2 & INDEX) < (el & INDEX)) l = l2, el = e2;
            }
            if (lane == s) my_k = el & INDEX, my_cost += (uint32_t)l;
            t -= el >> INDEX_BITS;
            x -= l;
            e = e_next;
        }
        put(THEMIS_SOLVED, (int32_t)total, (int32_t)ticks, W == 16 ? BY_B : BY_C);
        put_choice(my_k, my_cost);
        return THEMIS_SOLVED;
    }

    // The recurrence over 16 cells.  Every row of sixteen lanes holds g[s+1][0..15]; row r
    // takes the table's costs 4 q + r, so its copy is first shifted by r and then by 4 q,
    // both operand modifiers, and the four rows' minima are combined.  (What does not beat
    // everything cheaper does no harm.)  `base_sum`: the sum of the models' least costs.
    __device__ __forceinline__ int solve_sixteen(uint32_t base_sum, uint32_t my_base) const
    {
        const uint32_t* const tab = lds + L.tab;
        uint32_t* const rows = lds + L.tab + 16 * a.S;
        uint32_t g = 0u;  // g[S]: nothing left to run
        const int at = lane >> 4;
        for (int s = a.S - 1; s >= 0; --s) {
            const uint32_t* const mine = tab + s * 16 + at;
            uint32_t v[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) v[q] = mine[4 * q] >> INDEX_BITS;  // EMPTY: 2^19 - 1
            uint32_t h = row_shifted<1, 0x2>(g, LT_NONE);
            // the lanes a shift leaves without a source keep their own value: mark them
            h = row_shifted<2, 0x4>(h, LT_NONE);
            h = row_shifted<3, 0x8>(h, LT_NONE);
            h = (lane & 15) < at ? LT_NONE : h;
            uint32_t acc = h + v[0];
            acc = least(acc, row_shifted<4>(h, LT_NONE) + v[1]);
            acc = least(acc, row_shifted<8>(h, LT_NONE) + v[2]);
            acc = least(acc, row_shifted<12>(h, LT_NONE) + v[3]);
            g = least_of_rows(acc);
            if (lane < 16) rows[s * 16 + lane] = g;
        }
        const uint32_t m = (uint32_t)__ballot(g <= (uint32_t)T) & 0xFFFFu;
        if (m == 0u) return UNFINISHED;
        const int x = __builtin_ctz(m);
        const uint32_t ticks = lane_value(g, x);
        const uint32_t total = base_sum + (uint32_t)x;
        wave_lds_fence();
        return read_out<16>(total, ticks, x, my_base,
                            [&](int s, int y) { return rows[(s + 1) * 16 + y]; });
    }

    // ---- step G ------------------------------------------------------------------
    // Entries of lists: lt | cost << 16, and the index beside it.
    struct Lists {
        uint32_t* bins;   // 64 words per model; later the survivors, KEPT of each kind
        uint32_t* lists;  // 2 * len words per model; later the rows
        uint32_t* kept;   // per model: entries listed, later survivors
        uint32_t* floor;  // per model: the least cost among them
        int len;          // entries a list has room for
    };
    static constexpr int KEPT = 32;

    __device__ __forceinline__ Lists lists_of() const
    {
        Lists l;
        l.bins = lds + L.tab;
        l.lists = l.bins + 64 * a.S;
        l.kept = lds + L.best;
        l.floor = l.kept + a.S;
        l.len = (L.words - L.tab - 64 * a.S) / (2 * a.S);
        l.len = l.len < 64 ? l.len : 64;
        return l;
    }

    // Lists, per model, the candidates that nothing in a cheaper bin of costs is as fast
    // as (a bin is as many costs as it takes for 64 bins to reach the fastest candidate's).
    // False when one does not fit its list.
    __device__ __forceinline__ bool list_candidates(const Lists& l) const
    {
        for (int x = lane; x < 64 * a.S; x += 64) l.bins[x] = LT_NONE;
        wave_lds_fence();
        const Recips rc = recips();
        auto each = [&](auto use) {
            for_pairs(Pair(), [&](const Pair& p) {
                const uint32_t base = keys()[p.s] >> 15;
                const uint32_t top = fastest()[p.s] & 0x7FFFu;
                const uint32_t range = top - base;  // its bits beyond six are cut
                const int sh = range < 64u ? 0 : 26 - __builtin_clz(range);
                auto one = [&](const Eval& ev, uint32_t c) {
                    const uint32_t cost = __umul24((uint32_t)ev.n, c);
                    if (ev.lt >= 0 && cost <= top)
                        use(p, c, (uint32_t)ev.lt, cost, p.s * 64u + ((cost - base) >> sh));
                };
                uint32_t c = first_core(p);
                for (;;) {
                    const bool go = p.there && c <= p.last && may_cost(p, c, top);
                    if (__ballot(go) == 0ull) break;
                    const bool both = c < p.last;
                    const double r0 = recip(rc, go ? speed(p, c) : 1u);
                    const double r1 = recip(rc, go && both ? speed(p, c + 1u) : 1u);
                    if (go) {
                        const Eval e0 = eval<false>(p, r0), e1 = eval<false>(p, r1);
                        one(e0, c);
                        if (both) one(e1, c + 1u);
                        c += 2u;
                    }
                }
            });
        };
        each([&](const Pair&, uint32_t, uint32_t lt, uint32_t, uint32_t bin) {
            atomicMin(&l.bins[bin], lt);
        });
        wave_lds_fence();
        for (int s = 0; s < a.S; ++s) {
            const uint32_t incl = wave_scan<true>(l.bins[64 * s + lane]);
            l.bins[64 * s + lane] = from_lane_below(incl, LT_NONE);  // least of all cheaper bins
        }
        if (lane < a.S) l.kept[lane] = 0u;
        wave_lds_fence();
        each([&](const Pair& p, uint32_t c, uint32_t lt, uint32_t cost, uint32_t bin) {
            if (lt >= l.bins[bin]) return;
            const uint32_t at = atomicAdd(&l.kept[p.s], 1u);
            if (at < (uint32_t)l.len) {
                uint32_t* const e = l.lists + 2 * ((int)p.s * l.len + (int)at);
                e[0] = lt | cost << 16;
                e[1] = (c - 1u) * (uint32_t)a.n_batch + p.j;
            }
        });
        wave_lds_fence();
        const bool fits = lane >= a.S || l.kept[lane] <= (uint32_t)l.len;
        return __ballot(!fits) == 0ull;
    }

    // Candidates that can be part of an answer at all, by Lagrangian bounds.  For any
    // price mu >= 0 of a tick, sum over the models of min(cost + mu lt) less mu T is at
    // most the optimum, and an assignment that uses a candidate whose cost + mu lt
    // exceeds its model's least by r costs at least r more than that bound.  With the
    // cost `ub` of some assignment within the budget, candidates with r > ub - bound are
    // in no optimum.  mu is found by walking the lower hull of (ticks, cost) between the
    // cheapest and the fastest assignment to where the budget lies.  Single precision;
    // `slack` covers its error, so a candidate is kept rather than dropped.
    // What is left is two or three candidates per model whose costs span some tens of
    // cells, where the window would have to span hundreds.
    __device__ __forceinline__ int solve_gap()
    {
        const Lists l = lists_of();
        if (l.len < 16) return UNFINISHED;
        // the cheapest assignment (too slow) and the fastest (within the budget)
        uint32_t my_lt = 0, my_cost = 0, my_fast = 0;
        if (lane < a.S) {
            const uint32_t key = keys()[lane];
            my_lt = key & 0x7FFFu, my_cost = key >> 15;
            my_fast = fastest()[lane];
        }
        int64_t c0 = sum_models(my_cost), l0 = sum_models(my_lt);
        int64_t c1 = sum_models(my_fast & 0x7FFFu), l1 = sum_models(my_fast >> 15);
        if (!list_candidates(l)) return UNFINISHED;

        // lanes: `width` of them per model, entries dealt in turn
        int width = 1;
        while (2 * width * a.S <= 64) width *= 2;
        const int s = lane / width, sub = lane & (width - 1);
        const bool there = s < a.S;
        const int n = there ? (int)l.kept[s] : 0;
        const uint32_t* const mine = l.lists + 2 * (there ? s : 0) * l.len;
        auto lt_of = [](uint32_t w) { return w & 0xFFFFu; };
        auto cost_of = [](uint32_t w) { return w >> 16; };
        // the model's choice at a price, in all of its lanes, and its cost + mu lt
        auto choose = [&](float mu, float& v) {
            uint32_t w = 0u;
            v = 3.0e38f;
            for (int e = sub; e < n; e += width) {
                const uint32_t x = mine[2 * e];
                const float y = __builtin_fmaf(mu, (float)lt_of(x), (float)cost_of(x));
                if (y < v) v = y, w = x;
            }
            for (int d = 1; d < width; d <<= 1) {
                const float ov = __shfl_xor(v, d, 64);
                const uint32_t ow = (uint32_t)__shfl_xor((int)w, d, 64);
                if (ov < v || (ov == v && ow < w)) v = ov, w = ow;
            }
            return w;
        };
        auto total = [&](uint32_t x) { return (int64_t)wave_sum(there && sub == 0 ? x : 0u); };
        float mu = 0.0f, v = 0.0f;
        // the fastest assignment as choices: cost and lt of the caps' candidates
        uint32_t chosen = there ? (fastest()[s] >> 15) | (fastest()[s] & 0x7FFFu) << 16 : 0u;
        for (int turn = 0; turn < 16; ++turn) {
            mu = (float)(c1 - c0) / (float)(l0 - l1);
            const uint32_t w = choose(mu, v);
            const int64_t c = total(cost_of(w)), t = total(lt_of(w));
            // on the line between the two, or above it: the walk has ended
            if (c * (l0 - l1) + (c1 - c0) * t >= c1 * (l0 - l1) + (c1 - c0) * l1) break;
            if (t <= T)
                c1 = c, l1 = t, chosen = w;
            else
                c0 = c, l0 = t;
            if (c0 >= c1 || l0 <= l1) break;
        }
        // (the prices at which the walk stopped)
        choose(mu, v);
        // one change of a choice that the ticks left over allow, for a better `ub`
        const int64_t left = T - l1;
        uint32_t gain = 0u;
        for (int e = sub; e < n; e += width) {
            const uint32_t x = mine[2 * e];
            if ((int64_t)lt_of(x) - (int64_t)lt_of(chosen) <= left && cost_of(x) < cost_of(chosen)) {
                const uint32_t g = cost_of(chosen) - cost_of(x);
                gain = g > gain ? g : gain;
            }
        }
        for (int d = 32; d >= 1; d >>= 1) {
            const uint32_t o = (uint32_t)__shfl_xor((int)gain, d, 64);
            gain = o > gain ? o : gain;
        }
        const int ub = (int)c1 - (int)__builtin_amdgcn_readfirstlane((int)gain);
        float bound = there && sub == 0 ? v : 0.0f;
        for (int d = 32; d >= 1; d >>= 1) bound += __shfl_xor(bound, d, 64);
        bound -= mu * (float)T;
        const float slack = ((float)c1 + mu * (float)(T + l0)) * 0x1p-16f + 0x1p-10f;
        const float gap = (float)ub - bound + slack;
        wave_lds_fence();
        if (lane < a.S) l.kept[lane] = 0u, l.floor[lane] = EMPTY;
        wave_lds_fence();
        for (int e = sub; e < n; e += width) {
            const uint32_t x = mine[2 * e];
            const float y = __builtin_fmaf(mu, (float)lt_of(x), (float)cost_of(x));
            if (y - v <= gap) {
                const uint32_t at = atomicAdd(&l.kept[s], 1u);
                atomicMin(&l.floor[s], cost_of(x));
                if (at < (uint32_t)KEPT) {
                    l.bins[64 * s + (int)at] = x;
                    l.bins[64 * s + KEPT + (int)at] = mine[2 * e + 1];
                }
            }
        }
        wave_lds_fence();
        const uint32_t my_kept = lane < a.S ? l.kept[lane] : 1u;
        if (__ballot(my_kept > (uint32_t)KEPT || my_kept == 0u) != 0ull) return UNFINISHED;
        const int floor = (int)sum_models(lane < a.S ? l.floor[lane] : 0u);
        const int span = ub - floor;  // cells above the first that can be needed
        if (span < 0) return UNFINISHED;
        const int W = (span + 64) & ~63;
        // the rows in LDS where they fit; few combinations are tried one by one before rows
        // in HBM are taken, many only where those do not fit either
        const int cells = (a.S + 1) * (W + 2);
        if (cells / 2 <= 2 * l.len * a.S) return solve_listed<false>(l, W, floor);
        int status = solve_by_trial(l, my_kept, 1u << 10);
        if (status == UNFINISHED && cells <= a.S * a.row_stride)
            status = solve_listed<true>(l, W, floor);
        return status == UNFINISHED ? solve_by_trial(l, my_kept, TRIALS) : status;
    }

    // The recurrence over the survivors: W cells over the sum of their least costs.
    // HBM: the rows are in this instance's part of the row region.
    template <bool HBM>
    __device__ __forceinline__ int solve_listed(const Lists& l, int W, int floor) const
    {
        uint16_t* const rows = HBM ? a.frow + (size_t)i * a.S * a.row_stride
                                   : reinterpret_cast<uint16_t*>(l.lists);
        auto rows_fence = [] {  // a row's lanes read what others wrote
            if (HBM)
                __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "workgroup");
            else
                wave_lds_fence();
        };
        auto row_of = [&](int s) { return rows + s * (W + 2) + 2; };  // cell -1 is the guard
        for (int x = lane; x <= a.S; x += 64) row_of(x)[-1] = (uint16_t)G_INF;
        for (int x = lane; x < W; x += 64) row_of(a.S)[x] = 0;
        rows_fence();
        for (int s = a.S - 1; s >= 0; --s) {
            const uint16_t* const next = row_of(s + 1);
            uint16_t* const row = row_of(s);
            const int n = __builtin_amdgcn_readfirstlane((int)l.kept[s]);
            const uint32_t base = l.floor[s];
            const uint32_t* const ent = l.bins + 64 * s;
            for (int x0 = 0; x0 < W; x0 += 64) {
                uint32_t acc = G_INF;
                for (int e = 0; e < n; e += 2) {
                    const uint32_t w0 = ent[e], w1 = ent[e + 1 < n ? e + 1 : e];
                    const int y0 = x0 + lane - (int)((w0 >> 16) - base);
                    const int y1 = x0 + lane - (int)((w1 >> 16) - base);
                    const uint32_t v0 = next[y0 < -1 ? -1 : y0] + (w0 & 0xFFFFu);
                    const uint32_t v1 = next[y1 < -1 ? -1 : y1] + (w1 & 0xFFFFu);
                    acc = least(acc, least(v0, v1));
                }
                row[x0 + lane] = (uint16_t)acc;
            }
            rows_fence();
        }
        int x = -1;
        uint32_t ticks = 0;
        for (int x0 = 0; x0 < W && x < 0; x0 += 64) {
            const uint32_t v = row_of(0)[x0 + lane];
            const unsigned long long m = __ballot(v <= (uint32_t)T);
            if (m) {
                const int q = __builtin_ctzll(m);
                x = x0 + q;
                ticks = lane_value(v, q);
            }
        }
        if (x < 0) return UNFINISHED;  // never expected: the assignment of cost ub is in reach
        const uint32_t total = (uint32_t)(floor + x);
        uint32_t t = ticks, my_k = 0, my_cost = 0;
        for (int s = 0; s < a.S; ++s) {
            const int n = (int)l.kept[s];
            const uint32_t w = l.bins[64 * s + (lane & (KEPT - 1))];
            const uint32_t k = l.bins[64 * s + KEPT + (lane & (KEPT - 1))];
            const int d = (int)((w >> 16) - l.floor[s]);
            const bool in = lane < n && d <= x;
            const uint32_t rest = row_of(s + 1)[in ? x - d : 0];
            unsigned long long m = __ballot(in && (w & 0xFFFFu) + rest == t);
            uint32_t key = EMPTY, key_w = 0u;
            int key_d = 0;
            while (m) {
                const int q = __builtin_ctzll(m);
                m &= m - 1ull;
                const uint32_t kq = lane_value(k, q);
                if (kq < key) key = kq, key_w = lane_value(w, q), key_d = (int)lane_value((uint32_t)d, q);
            }
            if (key == EMPTY) {  // never expected
                put_none(THEMIS_INTERNAL);
                return THEMIS_INTERNAL;
            }
            if (lane == s) my_k = key, my_cost = key_w >> 16;
            t -= key_w & 0xFFFFu;
            x -= key_d;
        }
        put(THEMIS_SOLVED, (int32_t)total, (int32_t)ticks, HBM ? BY_G_HBM : BY_G_LDS);
        put_choice(my_k, my_cost);
        return THEMIS_SOLVED;
    }

    // Every combination of the survivors, where there are few of them and their costs span
    // more cells than the rows have room for.  The survivors of a model are put in index
    // order first, so that of equal combinations the first one met is the smallest.
    static constexpr uint32_t TRIALS = 1u << 14;
    __device__ __forceinline__ int solve_by_trial(const Lists& l, uint32_t my_kept,
                                                  uint32_t most) const
    {
        uint32_t count = 1u;
        for (int s = 0; s < a.S; ++s) {
            count *= lane_value(my_kept, s);
            if (count > most) return UNFINISHED;
        }
        for (int s = 0; s < a.S; ++s) {
            const int n = (int)l.kept[s];
            const int e = lane & (KEPT - 1);
            const uint32_t w = l.bins[64 * s + e], k = l.bins[64 * s + KEPT + e];
            int rank = 0;
            for (int o = 0; o < n; ++o) rank += l.bins[64 * s + KEPT + o] < k ? 1 : 0;
            wave_lds_fence();
            if (lane < n) {
                l.bins[64 * s + rank] = w;
                l.bins[64 * s + KEPT + rank] = k;
            }
            wave_lds_fence();
        }
        unsigned long long best = ~0ull;
        for (uint32_t x0 = 0; x0 < count; x0 += 64u) {
            const uint32_t x = x0 + (uint32_t)lane;
            if (x < count) {
                uint32_t rest = x, c = 0, t = 0;
                for (int s = a.S - 1; s >= 0; --s) {  // model 0 is the most significant digit
                    const uint32_t n = l.kept[s];
                    const uint32_t q = rest / n;
                    const uint32_t w = l.bins[64 * s + (int)(rest - q * n)];
                    rest = q;
                    c += w >> 16;
                    t += w & 0xFFFFu;
                }
                if (t <= (uint32_t)T) {
                    const unsigned long long key =
                        ((unsigned long long)c << 32) | ((unsigned long long)t << 14) | x;
                    best = key < best ? key : best;
                }
            }
        }
        for (int d = 32; d >= 1; d >>= 1) {
            const unsigned long long o = __shfl_xor(best, d, 64);
            best = o < best ? o : best;
        }
        if (best == ~0ull) return UNFINISHED;  // never expected
        uint32_t rest = (uint32_t)best & (TRIALS - 1u), my_k = 0, my_cost = 0;
        for (int s = a.S - 1; s >= 0; --s) {
            const uint32_t n = l.kept[s];
            const uint32_t q = rest / n;
            if (lane == s) {
                my_cost = l.bins[64 * s + (int)(rest - q * n)] >> 16;
                my_k = l.bins[64 * s + KEPT + (int)(rest - q * n)];
            }
            rest = q;
        }
        put(THEMIS_SOLVED, (int32_t)(best >> 32), (int32_t)((best >> 14) & 0x3FFFFull), BY_G_TRIAL);
        put_choice(my_k, my_cost);
        return THEMIS_SOLVED;
    }

    // ---- steps C and W -------------------------------------------------------------
    // The recurrence over 64 cells, lane = cell, the table of all models in LDS.
    __device__ __forceinline__ int solve_sixtyfour() const
    {
        const uint32_t* const tab = lds + L.tab;
        // rows of 16-bit cells, a guard cell (and one of padding) in front of each
        uint16_t* const rows = reinterpret_cast<uint16_t*>(lds + L.tab + 64 * a.S);
        auto row_of = [&](int s) { return rows + s * 66 + 2; };
        for (int x = lane; x <= a.S; x += 64) row_of(x)[-1] = (uint16_t)G_INF;
        row_of(a.S)[lane] = 0;
        uint32_t acc = 0;
        uint32_t lt = tab[(a.S - 1) * 64 + lane] >> INDEX_BITS;
        wave_lds_fence();
        for (int s = a.S - 1; s >= 0; --s) {
            const uint16_t* const next = row_of(s + 1);
            // what beats everything cheaper
            const bool on = lt < from_lane_below(wave_scan<true>(lt), LT_NONE) && lt < G_INF;
            const uint32_t lt_next = s > 0 ? tab[(s - 1) * 64 + lane] >> INDEX_BITS : 0u;
            acc = G_INF;
            unsigned long long m = __ballot(on);
            while (m) {  // four entries at a time: independent reads
                uint32_t v[4];
#pragma unroll
                for (int z = 0; z < 4; ++z) {
                    const int d = m ? __builtin_ctzll(m) : 64;
                    const uint32_t l = m ? lane_value(lt, d & 63) : 0u;
                    m &= m - 1ull;
                    const int y = lane - d;
                    v[z] = (uint32_t)next[y < -1 ? -1 : y] + l;
                }
                acc = least(least(acc, v[0]), least(v[1], least(v[2], v[3])));
            }
            row_of(s)[lane] = (uint16_t)acc;
            wave_lds_fence();
            lt = lt_next;
        }
        const unsigned long long m = __ballot(acc <= (uint32_t)T);
        if (m == 0ull) return UNFINISHED;
        const int x = __builtin_ctzll(m);
        const uint32_t my_base = lane < a.S ? keys()[lane] >> 15 : 0u;
        return read_out<64>(sum_models(my_base) + (uint32_t)x, lane_value(acc, x), x, my_base,
                            [&](int s, int y) { return (uint32_t)row_of(s + 1)[y]; });
    }

    // The table of one model, W cells.  All lanes work on it: lane = (part, batch size),
    // the parts take the cores in turn.
    __device__ __forceinline__ void fill_model(int s, int W) const
    {
        uint32_t* const tab = lds + L.tab;
        for (int x = lane; x < W; x += 64) tab[x] = EMPTY;
        const uint32_t nb = (uint32_t)a.n_batch;
        const uint32_t parts = index_quotient(64u, a.magic);
        const uint32_t part = index_quotient((uint32_t)lane, a.magic);
        const Pair p = pair_of((uint32_t)s, (uint32_t)lane - part * nb, part < parts);
        const uint32_t base = keys()[s] >> 15;
        const uint32_t top = base + (uint32_t)W - 1u;
        wave_lds_fence();
        if (part < parts) {
            for (uint32_t c = first_core(p) + part; c <= p.last && may_cost(p, c, top); c += parts) {
                const Eval ev = eval<false>(p, recip_below((double)speed(p, c)));
                const uint32_t cost = __umul24((uint32_t)ev.n, c);
                if (ev.lt >= 0 && cost <= top)
                    atomicMin(&tab[cost - base], entry(ev, (c - 1u) * nb + (uint32_t)(lane - part * nb)));
            }
        }
        wave_lds_fence();
    }

    // The recurrence over W cells (a multiple of 64) and, where it ends within the budget,
    // the answer.  HBM: the rows are in this instance's part of the row region.
    template <bool HBM>
    __device__ __forceinline__ int solve_window(int W) const
    {
        uint32_t* const tab = lds + L.tab;
        uint16_t* const rows = HBM ? a.frow + (size_t)i * a.S * a.row_stride
                                   : reinterpret_cast<uint16_t*>(lds + L.rows);
        // a row's lanes read what others wrote
        auto rows_fence = [] {
            if (HBM)
                __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "workgroup");
            else
                wave_lds_fence();
        };
        auto row_of = [&](int s) { return rows + s * (W + 2) + 2; };  // cell -1 is the guard
        for (int x = lane; x <= a.S; x += 64) row_of(x)[-1] = (uint16_t)G_INF;
        for (int x = lane; x < W; x += 64) row_of(a.S)[x] = 0;
        rows_fence();
        for (int s = a.S - 1; s >= 0; --s) {
            fill_model(s, W);
            // what beats everything cheaper, as a list in the table's own place: cost over
            // base and lt of entry n at n, never beyond the cells already read
            uint32_t low = LT_NONE;
            int n = 0;
            for (int x0 = 0; x0 < W; x0 += 64) {
                const uint32_t lt = tab[x0 + lane] >> INDEX_BITS;
                const uint32_t incl = least(wave_scan<true>(lt), low);
                const bool on = lt < from_lane_below(incl, low) && lt < G_INF;
                low = lane_value(incl, 63);
                const unsigned long long m = __ballot(on);
                if (on)
                    tab[n + (int)__builtin_popcountll(m & ((1ull << lane) - 1ull))] =
                        (uint32_t)(x0 + lane) << 16 | lt;
                n += (int)__builtin_popcountll(m);
                wave_lds_fence();
            }
            // entries beyond the list that never apply, so that it can be read in pairs
            if (lane < 2 && n + lane < W) tab[n + lane] = 0xFFFFu << 16;
            wave_lds_fence();
            const uint16_t* const next = row_of(s + 1);
            uint16_t* const row = row_of(s);
            for (int x0 = 0; x0 < W; x0 += 256) {
                uint32_t acc[4];
#pragma unroll
                for (int q = 0; q < 4; ++q) acc[q] = G_INF;
                const int end = x0 + 255;
                for (int e = 0; e < n; e += 2) {
                    const uint32_t w0 = tab[e], w1 = tab[e + 1 < W ? e + 1 : e];
                    if (__builtin_amdgcn_readfirstlane((int)(w0 >> 16)) > end) break;
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        const int x = x0 + 64 * q + lane;
                        if (x0 + 64 * q < W) {
                            const int y0 = x - (int)(w0 >> 16), y1 = x - (int)(w1 >> 16);
                            const uint32_t a0 = next[y0 < -1 ? -1 : y0] + (w0 & 0xFFFFu);
                            const uint32_t a1 = next[y1 < -1 ? -1 : y1] + (w1 & 0xFFFFu);
                            acc[q] = least(acc[q], least(a0, a1));
                        }
                    }
                }
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    if (x0 + 64 * q < W) row[x0 + 64 * q + lane] = (uint16_t)acc[q];
            }
            rows_fence();
        }
        int x = -1;
        uint32_t ticks = 0;
        for (int x0 = 0; x0 < W && x < 0; x0 += 64) {
            const uint32_t v = row_of(0)[x0 + lane];
            const unsigned long long m = __ballot(v <= (uint32_t)T);
            if (m) {
                const int l = __builtin_ctzll(m);
                x = x0 + l;
                ticks = lane_value(v, l);
            }
        }
        if (x < 0) return UNFINISHED;

        // forward: the smallest index among the candidates that continue an optimum
        uint32_t total = (uint32_t)x, t = ticks, my_k = 0, my_cost = 0;
        for (int s = 0; s < a.S; ++s) {
            fill_model(s, W);
            const uint16_t* const next = row_of(s + 1);
            uint32_t key = EMPTY, key_lt = 0;
            int key_d = 0;
            for (int d0 = 0; d0 <= x; d0 += 64) {
                const int d = d0 + lane;
                const uint32_t e = d <= x ? tab[d] : EMPTY;
                const uint32_t rest = next[d <= x ? x - d : 0];
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
                return THEMIS_INTERNAL;
            }
            const uint32_t base = keys()[s] >> 15;
            total += base;
            if (lane == s) my_k = key, my_cost = base + (uint32_t)key_d;
            t -= key_lt;
            x -= key_d;
            wave_lds_fence();
        }
        put(THEMIS_SOLVED, (int32_t)total, (int32_t)ticks, HBM ? BY_W_HBM : BY_W_LDS);
        put_choice(my_k, my_cost);
        return THEMIS_SOLVED;
    }

    // ---- step D ---------------------------------------------------------------------
    // Candidate number x of model s in index order (64 at a time, one per lane).
    __device__ __forceinline__ Eval candidate(int s, uint32_t x, uint32_t count, uint32_t& cost,
                                              uint32_t& k) const
    {
        const uint32_t q = index_quotient(x, a.magic);  // x < MAX_CAND: a multiple of 64
        const Pair p = pair_of((uint32_t)s, x - q * (uint32_t)a.n_batch, true);
        const uint32_t c = p.lo + (x < count ? q : 0u);
        Eval ev = eval<false>(p, recip_below((double)speed(p, c)));
        if (x >= count) ev.lt = -1;
        cost = __umul24((uint32_t)ev.n, c);
        k = (c - 1u) * (uint32_t)a.n_batch + p.j;
        return ev;
    }

    // Rows over the budget, in this instance's part of the row region.  Candidates are
    // first entered into a table of least latencies by cost (as many costs per bin as
    // it takes) so that only those faster than everything in a cheaper bin are swept.
    __device__ __forceinline__ int solve_by_budget(int W) const
    {
        const int bins = W;
        uint32_t* const tab = lds + L.tab;
        uint32_t* const list = lds + L.rows;  // lt | cost << 16
        const int cap = a.S * W / 2;          // entries of the list (the rows have room)
        uint16_t* const rows = a.frow + (size_t)i * a.S * a.row_stride;
        const uint32_t nbat = (uint32_t)a.n_batch;
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
                const Eval ev = candidate(s, x, count, cost, k);
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
                const Eval ev = candidate(s, x, count, cost, k);
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
                const Eval ev = candidate(s, x, count, cost, k);
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
                return THEMIS_INTERNAL;
            }
        }
        put(THEMIS_SOLVED, (int32_t)best, t_star, BY_D);
        put_choice(my_k, my_cost);
        return THEMIS_SOLVED;
    }

    // Steps A, F and B.
    template <bool SMALL>
    __device__ __forceinline__ int solve_valid(const Pair& first) const
    {
        least_costs<SMALL>(first);
        uint32_t key = 0, k = 0, lt = 0;
        if (lane < a.S) {
            const unsigned long long best = bests()[lane];
            key = (uint32_t)(best >> INDEX_BITS);
            k = (uint32_t)best & ((1u << INDEX_BITS) - 1u);
            lt = key == EMPTY ? LT_NONE : key & 0x7FFFu;
        }
        const uint32_t ticks = sum_models(lt);
        if (ticks <= (uint32_t)T) {
            put(THEMIS_SOLVED, (int32_t)sum_models(key >> 15), (int32_t)ticks);
            put_choice(k, key >> 15);
            return THEMIS_SOLVED;
        }
        if (ticks >= LT_NONE || fastest_ticks<SMALL>(first) > (uint32_t)T) return THEMIS_INFEASIBLE;
        fill_all<SMALL, 16>(first);
        const int status = solve_sixteen(sum_models(key >> 15), key >> 15);
        wave_lds_fence();
        return status;
    }

    // Steps C, G and D.
    __device__ __forceinline__ int further(int inst, int budget, int32_t rate, int32_t objective)
    {
        i = inst, T = budget, lam = rate, slo = objective;
        lane_b = lane < a.n_batch ? (int32_t)a.bc[lane].b : 0;
        fill_all<false, 64>(Pair());
        int status = solve_sixtyfour();
        wave_lds_fence();
        if (status == UNFINISHED) status = solve_gap();
        int W = 64;
        while (status == UNFINISHED && W < a.window) {
            wave_lds_fence();
            W = 2 * W < a.window ? 2 * W : a.window;
            status = solve_window<false>(W);
        }
        while (status == UNFINISHED && W < a.window_hbm) {
            wave_lds_fence();
            W = 2 * W < a.window_hbm ? 2 * W : a.window_hbm;
            status = solve_window<true>(W);
        }
        wave_lds_fence();
        return status == UNFINISHED ? solve_by_budget(a.window) : status;
    }

    // The inputs of instance `inst` at `rate`; valid: the input check's result.
    __device__ __forceinline__ Pair begin(int inst, int32_t rate, bool& valid)
    {
        i = inst;
        lam = rate;
        slo = a.slo_us[i];
        const bool rates = in_range(lam, 1, THEMIS_VALUE_MAX) && in_range(slo, 0, a.slo_max);
        // floor(slo / tick): the quotient lies at least half of 1 / tick above any whole
        // number below it, which the reciprocal's error (2^-44 relative) does not reach
        T = __builtin_amdgcn_readfirstlane((int)(((double)slo + 0.5) * a.rtick));
        int32_t word = 0;
        if (keeps_coef() && lane < a.S * a.cs) word = (a.coef + (size_t)i * (a.S * a.cs))[lane];
        const Pair first = pair_of_round(0u);
        lane_b = (int32_t)first.bh.b;  // the first n_batch lanes have the first model's pairs
        bool fine = rates;
        for_pairs(first, [&](const Pair& p) { fine = fine && (!p.there || p.valid); });
        valid = __ballot(!fine) == 0ull;
        keep_inputs(valid, word);
        if (records() && lane == 0) a.tmeta[i] = valid ? T : -1;
        return first;
    }

    // Solves the instance that was begun, and is valid, at the rate `lam`; writes the
    // results unless it is infeasible.
    __device__ __forceinline__ int solve(const Pair& first) const
    {
        if (lane < a.S) {
            keys()[lane] = EMPTY;
            bests()[lane] = ~0ull;
        }
        wave_lds_fence();
        int status;
        // row_is_small(), which is the same for all models of an instance
        if (__builtin_amdgcn_readfirstlane((int)((double)lam * (double)slo <= 0x1p42)))
            status = solve_valid<true>(first);
        else
            status = solve_valid<false>(first);
        status = __builtin_amdgcn_readfirstlane(status);
        if (status == UNFINISHED)
            status = solve_further<QUEUE, DERIVE, ROLE>((uint64_t)(uintptr_t)&a, i, T, lam, slo);
        return status;
    }
};

// Out of line, so that its registers do not weigh on the allocation of the steps
// that nearly every instance ends with.
template <int QUEUE, bool DERIVE, int ROLE>
__device__ __attribute__((noinline)) int solve_further(uint64_t args, int i, int T, int32_t lam,
                                                       int32_t slo)
{
    auto uniform = [](int v) { return __builtin_amdgcn_readfirstlane(v); };
    const uint64_t lo = (uint32_t)uniform((int)(uint32_t)args);
    const uint64_t hi = (uint32_t)uniform((int)(uint32_t)(args >> 32));
    Solver<QUEUE, DERIVE, false, ROLE> sv((ArgsPtr)(uintptr_t)(hi << 32 | lo));
    return uniform(sv.further(uniform(i), uniform(T), uniform(lam), uniform(slo)));
}

// One whole solve of instance `inst` at `rate`.
template <int QUEUE, bool DERIVE, bool ONE, int ROLE>
__device__ __forceinline__ int solve_instance(ArgsPtr args, int inst, int32_t rate)
{
    Solver<QUEUE, DERIVE, ONE, ROLE> sv(args);
    bool valid;
    const auto first = sv.begin(inst, rate, valid);
    int status = THEMIS_INVALID;
    if (valid) status = sv.solve(first);
    if (status == THEMIS_INVALID || status == THEMIS_INFEASIBLE) sv.put_none(status);
    return status;
}

// What the class lists and the state word say about the workspace after a solve: no
// tables, the inputs and results in the table region.  Shared coefficients are in the
// first record, whether or not that instance is solved.
__device__ __forceinline__ void mark_workspace(ArgsPtr args, int state)
{
    if (blockIdx.x != 0) return;
    if ((int)threadIdx.x <= STATE_WORD)
        args->ctrl[threadIdx.x] = (int)threadIdx.x < STATE_WORD || !args->keep ? 0 : state;
    if (args->keep && args->coef_shared)
        for (int x = (int)threadIdx.x; x < args->S * args->cs; x += 64)
            (args->keep + args->kept.coef)[x] = args->coef[x];
}

// (Kernels read their arguments where they lie, see ArgsPtr.)
__device__ __forceinline__ ArgsPtr kernel_args()
{
    return (ArgsPtr)__builtin_amdgcn_kernarg_segment_ptr();
}

}  // namespace

// ---- launching ---------------------------------------------------------------------
namespace {

typedef void (*CostKernel)(CostArgs);

constexpr size_t LDS_PER_CU = 160 * 1024;
constexpr int MAX_WINDOW = 8192;
// Wavefronts whose LDS a compute unit has room for.  Registers allow 32, but some twenty
// are in flight on average, and the room of the others lets step G list more candidates:
// at 16384 x 8 with a twelfth of the objectives 32 / 28 / 24 / 20 take 579 / 122 / 121 /
// 129 us, at 86400 x 6 51 / 51 / 55 / 60.
constexpr int RESIDENT_PER_CU = 28;

// What does not depend on the entry point.
inline CostArgs cost_args(const themis_problem_t& p, const Layout& L, const int32_t* d_coef,
                          const int32_t* d_lambda, const int32_t* d_slo_us,
                          const int32_t* d_r_fixed, int32_t* d_status, int32_t* d_cost,
                          int32_t* d_ticks, int32_t* d_cfg, char* ws, const PassOpts& opts)
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
    a.ctrl = (int32_t*)(ws + L.ctrl_off);
    a.frow = (uint16_t*)(ws + L.frow_off);
    a.kept = make_keep_layout(p);
    a.keep = opts.inspectable ? (int32_t*)(ws + L.step_off) : nullptr;
    a.n_batch = p.n_batch;
    for (int j = 0; j < p.n_batch; ++j)
        a.bc[j] = {(double)p.batch_sizes[j], (1.0 / (1.0e6 * p.batch_sizes[j])) * (1.0 - 0x1p-45)};
    a.S = L.S;
    a.cs = p.profile_form == THEMIS_PROFILE_EQ1 ? 6 : 5;
    a.c_max = p.c_max;
    a.r_max = p.r_max;
    a.tick = p.tick_us;
    a.slo_max = p.slo_max_us;
    a.coef_shared = p.coef_shared;
    a.c_all = opts.c_all;
    a.list = opts.list;
    a.row_stride = L.row_stride;
    a.magic = index_magic((uint32_t)p.n_batch);
    a.rtick = (1.0 / (double)p.tick_us) * (1.0 - 0x1p-45);
    return a;
}

// The arguments with the arrays of all instances but the first n, for the launches after
// the first one of a large batch: offsets in the kernels would cost every solve (the
// fallback at 16384 x 8 62.8 us instead of 61.8, 65536 x 8 99.5 instead of 98.8).  (Each
// of these launches marks the workspace again, with the same words.)
inline CostArgs past(CostArgs a, size_t n)
{
    auto skip = [](auto*& array, size_t elements) {
        if (array) array += elements;
    };
    const size_t rows = n * (size_t)a.S;
    if (!a.coef_shared) skip(a.coef, rows * a.cs);
    for (const int32_t** in : {&a.lambda, &a.slo_us, &a.lambda2}) skip(*in, n);
    for (const int32_t** in : {&a.r_fixed, &a.c_fixed}) skip(*in, rows);
    for (int32_t** out : {&a.status, &a.cost, &a.ticks, &a.status2, &a.cost2, &a.ticks2, &a.lambda_v,
                          &a.stable, &a.tmeta})
        skip(*out, n);
    for (int32_t** out : {&a.cfg, &a.cfg2}) skip(*out, 3 * rows);
    skip(a.frow, rows * a.row_stride);
    skip(a.keep, n * a.kept.words);
    return a;
}

// A workgroup per instance, or where `listed` as many as stay resident (the host does
// not know how long the list is).  `one` in kernel(one): the (model, batch size) pairs
// fit a wavefront's lanes.
//
// One launch (of up to MAX_PER_LAUNCH instances), whatever the instances need: a second one with room for wider windows,
// for the instances the first one could not solve, took 4.5 us to find that there are
// none (of 24 at 16384 x 8, 55 at 86400 x 6); windows wider than the LDS of a full
// compute unit allows have their rows in HBM instead.
template <typename K>
hipError_t launch_per_instance(const themis_problem_t& p, const Layout& L, CostArgs& a,
                               hipStream_t st, bool listed, K kernel)
{
    const int cus = compute_units();
    const int grid = listed && L.N > RESIDENT_PER_CU * cus ? RESIDENT_PER_CU * cus : L.N;
    // the largest window that leaves the wavefronts that can be resident their LDS, no
    // larger than the costs of a pipeline can spread
    int per_cu = (int)(((long long)grid + cus - 1) / cus);
    per_cu = per_cu < 4 ? 4 : per_cu > RESIDENT_PER_CU ? RESIDENT_PER_CU : per_cu;
    auto lds_for = [&](int window) {
        return (size_t)cost_lds(L.S, window).words * sizeof(uint32_t);
    };
    const int spread = L.S * p.r_max * p.c_max;
    a.window = 64;
    while (a.window + 64 <= MAX_WINDOW && a.window < spread &&
           lds_for(a.window + 64) <= LDS_PER_CU / per_cu)
        a.window += 64;
    // rows in HBM: S + 1 of them in the S that an instance has of the row region, and the
    // table of a model still in LDS
    const CostLds lds = cost_lds(L.S, a.window);
    const int fit = (int)((long long)L.S * L.row_stride / (L.S + 1)) - 2;
    const int room = lds.words - lds.tab;
    a.window_hbm = (fit < room ? fit : room) & ~63;
    // (at most 40 KB of LDS, which a kernel may have without asking)
    const CostKernel k = kernel(L.S * p.n_batch <= 64);
    hipError_t e = hipSuccess;
    in_launches(grid, [&](int first, int count) {
        if (e != hipSuccess) return;
        hipLaunchKernelGGL(k, dim3((unsigned)count), dim3(64), lds_for(a.window), st,
                           past(a, (size_t)first));
        e = hipGetLastError();
    });
    return e;
}

}  // namespace
}  // namespace themis
