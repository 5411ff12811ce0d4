// The start of one wavefront's solve of one instance: inputs, steps A, F and B of
// cost_solve.hip, and the table of step C; what they do not settle goes on in the functions
// of cost_solver.h.
//
// What bounds it: for large batches vector issue (86400 x 6: the vector ALUs are busy 93 %
// of the time), for small ones the chain of dependent instructions of the slowest wavefront, at
// eight cycles each where four would issue and 40 to 60 for a branch, an LDS read or a value
// that goes through a scalar register.  So: minima per model in registers, bounds in
// single precision ahead of evaluations, no loop over the models in step B, one call at the
// very end.  Against evaluating every core count that the real-valued bound allows, with
// LDS atomics per model and sixteen cells for every instance, in microseconds:
// 512 x 5 9.5 -> 7.0, 4096 x 5 13.3 -> 10.8, 3001 x 7 17.3 -> 12.8, stability 4099 x 5
// 23.4 -> 17.4, 16384 x 8 with replicas given 26.3 -> 22.5, 86400 x 6 51.8 -> 39.7,
// 65536 x 8 98.1 -> 76.3, fallback 16384 x 8 65 -> 28.5.
#pragma once

#include <type_traits>

#include "cost_solver.h"

namespace themis {
namespace {

// A model's (model, batch size) pairs are neighbouring lanes, `width` of them, a power of
// two, so what is sought per model is found between neighbours in registers, by
// data-parallel primitives: a minimum over eight lanes is three instructions, where LDS
// atomics took an initial value, a wait for each atomic and a read (some 200 cycles).
// WIDTH: that width, where all models fit the wavefront that way (every lane keeps its pair
// from step A on); PACKED: where they fit it only without gaps between the models, and
// minima go through LDS; TURNS: where there are more pairs than lanes, the lanes of a model with
// its batch sizes in turns (a power of two of lanes, or where that takes fewer turns as many as
// all models leave room for, with minima through LDS).  A lane then keeps its model, and is done
// with all of its batch sizes before minima and sums are formed.  ROUNDS: where that leaves too
// many lanes idle (front_layout() has the rule; single solves only), the models in rounds of
// args->per_round, in lanes for all of their batch sizes (round_log below zero: without gaps),
// with their inputs asked for again, minima and sums formed in each, and what is found about
// them in LDS.  (That way 3001 x 7 models with twelve batch sizes take 11.8 us and in turns 10.4,
// 59755 x 7 with fourteen and replicas given 246 and 203, fallback 13320 x 9 with fifteen 105 and
// 59, 186 x 10 with seven 30.6 and 32.4, on other inputs 6.48 and 6.53; 43 shapes of five to ten
// models, four calls and three batches each, are in turns done in 0.84 of the time in the mean
// and 1.02 at most.)
// (One kernel for the widths 4, 8 and 16, with the width an argument:
// 86400 x 6 43.6 us instead of 39.8, fallback 16384 x 8 30.8 instead of 28.5, 65536 x 8 79.5
// instead of 76.4, 512 x 5 7.4 instead of 7.0.)
constexpr int TURNS = WIDTH_TURNS, PACKED = WIDTH_PACKED, ROUNDS = WIDTH_ROUNDS;
// MANY: TURNS or, where the instance's steps are taken that way, ROUNDS
template <int QUEUE, bool DERIVE, int ROLE, int MANY>
__device__ __attribute__((noinline)) int solve_rest(uint64_t args, int i, int T, int32_t lam,
                                                    int32_t slo);

template <int QUEUE, bool DERIVE, int WIDTH, int ROLE = PLAIN>
struct Front : Solver<QUEUE, DERIVE, ROLE> {
    using Base = Solver<QUEUE, DERIVE, ROLE>;
    using typename Base::Model;
    using typename Base::Pair;
    using Base::a, Base::args, Base::i, Base::L, Base::lam, Base::lane, Base::lds, Base::slo, Base::T;
    // a pair, or a model, for every lane from the start
    static constexpr bool ONE = WIDTH != TURNS && WIDTH != ROUNDS, OWN = WIDTH == TURNS;
    static constexpr int MANY = WIDTH == ROUNDS ? ROUNDS : TURNS;

    __device__ __forceinline__ explicit Front(ArgsPtr p, int l = (int)threadIdx.x, uint32_t offset = 0u)
        : Base(p, l, offset)
    {
    }
    static __device__ __forceinline__ Front of_wave(ArgsPtr p)
    {
        return Front(p, (int)threadIdx.x & 63, wave_number() * p->wave_words);
    }

    __device__ __forceinline__ int width_log() const
    {
        return WIDTH == 16 ? 4 : WIDTH == 8 ? 3 : WIDTH == 4 ? 2 : WIDTH == ROUNDS ? args->round_log : a.width_log;
    }
    // this lane's pair (ROUNDS: of the round that starts with model s0)
    __device__ __forceinline__ Pair lanes_pair(int s0 = 0) const
    {
        uint32_t s, j;
        if (packed()) {
            s = index_quotient((uint32_t)lane, a.magic);
            j = (uint32_t)lane - s * (uint32_t)a.n_batch;
        } else {
            s = (uint32_t)lane >> width_log();
            j = (uint32_t)lane & ((1u << width_log()) - 1u);
        }
        if (WIDTH == ROUNDS) s = s < (uint32_t)args->per_round ? s + (uint32_t)s0 : (uint32_t)a.S;
        const bool in = s < (uint32_t)a.S;
        Pair p = this->pair_of(s, j, (int)in & (int)(j < (uint32_t)a.n_batch));
        p.in = in, p.first = j == 0u;
        return p;
    }
    // What a lane starts from: its pair, or (OWN) its model and which of its lanes it is.
    struct Own {
        Model m;
        uint32_t s, part;
        bool there, valid, in;
        int32_t size;
    };
    typedef typename std::conditional<OWN, Own, Pair>::type Start;
    __device__ __forceinline__ Start start() const
    {
        if constexpr (!OWN) {
            return lanes_pair();
        } else {
            Own o;
            const uint32_t lanes = (uint32_t)args->lanes;
            o.s = index_quotient((uint32_t)lane, args->lane_magic);
            o.part = (uint32_t)lane - o.s * lanes;
            o.in = o.there = o.s < (uint32_t)a.S;
            o.s = o.there ? o.s : 0u;
            o.m = this->model_of(o.s);
            o.valid = o.m.valid;
            o.size = args->bc[lane < a.n_batch ? lane : 0].size;
            return o;
        }
    }
    // Calls f(pair) for this lane's pair, or each of its pairs; lanes without one get a pair
    // with `there` unset.  The lanes of a model take batch sizes next to one another, so that
    // they have about the same work; SPREAD: each from its own part of the list, so that the first
    // ones met are of all sizes.
    template <bool SPREAD = false, typename F>
    __device__ __forceinline__ void for_pairs(const Start& mine, F f) const
    {
        if constexpr (ONE) {
            f(mine);
        } else if constexpr (!OWN) {
            for (int s0 = 0; s0 < a.S; s0 += args->per_round) f(lanes_pair(s0));
        } else {
            const uint32_t nb = (uint32_t)a.n_batch, turns = (uint32_t)args->turns;
            const uint32_t first = SPREAD ? mine.part * turns : mine.part;
            const uint32_t step = SPREAD ? 1u : (uint32_t)args->lanes;
            for (uint32_t t = 0u, j = first; t < turns; ++t, j += step) {
                const bool there = mine.there && j < nb;
                Pair p;
                this->batch_size(p, there ? j : 0u);
                this->of_model(p, mine.m, mine.s);
                p.there = there, p.in = mine.in, p.first = mine.part == 0u;
                f(p);
            }
        }
    }
    // whether this lane is the first of its model's
    static __device__ __forceinline__ bool leads(const Pair& p) { return (int)p.in & (int)p.first; }
    static __device__ __forceinline__ bool leads(const Own& o) { return (int)o.in & (int)(o.part == 0u); }
    __device__ __forceinline__ bool packed() const
    {
        return WIDTH == PACKED || (!ONE && width_log() < 0);
    }
    static __device__ __forceinline__ bool any(bool x) { return __builtin_amdgcn_ballot_w64(x) != 0ull; }

    // The least of a model's lanes, in all of them.
    template <int CTRL>
    static __device__ __forceinline__ uint32_t least_step(uint32_t x)
    {
        return least(x, (uint32_t)__builtin_amdgcn_update_dpp(-1, (int)x, CTRL, 0xF, 0xF, false));
    }
    template <typename P>
    __device__ __forceinline__ uint32_t model_least(const P& p, uint32_t x) const
    {
        if (packed()) {
            // (a wavefront's LDS operations complete in order)
            uint32_t* const slot = this->fastest() + p.s;
            if (leads(p)) *slot = EMPTY;
            wave_lds_fence();
            if (p.there) atomicMin(slot, x);
            wave_lds_fence();
            const uint32_t least_x = *slot;
            wave_lds_fence();
            return p.there ? least_x : EMPTY;
        }
        const int w = width_log();
        if (w > 0) x = least_step<0xB1 /* quad_perm:[1,0,3,2] */>(x);
        if (w > 1) x = least_step<0x4E /* quad_perm:[2,3,0,1] */>(x);
        if (w > 2) x = least_step<0x141 /* row_half_mirror */>(x);
        if (w > 3) x = least_step<0x140 /* row_mirror */>(x);
        return x;
    }
    // The sum over all models of a value that their lanes share.
    template <int CTRL>
    static __device__ __forceinline__ uint32_t add_step(uint32_t x)
    {
        return x + (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, CTRL, 0xF, 0xF, false);
    }
    template <typename P>
    __device__ __forceinline__ uint32_t sum_of_models(const P& p, uint32_t x) const
    {
        if constexpr (ONE && WIDTH != PACKED) {
            x = p.in ? x : 0u;
            if (WIDTH <= 4) x = add_step<0x124 /* row_ror:4 */>(x);
            if (WIDTH <= 8) x = add_step<0x128 /* row_ror:8 */>(x);
            return lane_value(x, 0) + lane_value(x, 16) + lane_value(x, 32) + lane_value(x, 48);
        } else {
            return wave_sum(leads(p) ? x : 0u);
        }
    }

    // What step A finds about a model, the same in all its lanes: cost << 15 | lt of the best
    // candidate (EMPTY: none is feasible) and its index.  c0: the lane's first_core().
    // mine: this lane's own best is the one, with that many cores and that batch size.
    // own: the lane's own best's.
    struct Best {
        uint32_t key, k, c0, c, own;
        int32_t size;
        bool mine;
    };

    // Cost << 15 | lt of the pair's candidate with c cores, EMPTY where it is infeasible.
    // rd: recip_below() of what they do to its speed.
    template <bool SMALL>
    __device__ __forceinline__ uint32_t meet(const Pair& p, uint32_t c, double rd) const
    {
        if (!SMALL || QUEUE == THEMIS_QUEUE_WORST_CASE) {
            const Eval ev = this->template eval<SMALL>(p, rd);
            return ev.lt >= 0 ? __umul24((uint32_t)ev.n, c) << 15 | (uint32_t)ev.lt : EMPTY;
        }
        // eval_parts() with the division by b 1e6 of lambda as a factor that all candidates of
        // the pair share.  p.ratio is lambda / (b 1e6) less at most 2^-44 of it, so
        // ceil_div_small()'s argument holds for proc * ratio as it does for
        // (lambda proc) * rM.  (A candidate for which lambda proc exceeds 2^42 is slower than
        // the objective and fails the last test whatever its replica count comes out as.)
        const double proc = ceil_div_small(p.num, rd) + p.fixed;
        const double need = proc * p.ratio;
        const double n = DERIVE ? __builtin_ceil(need) : p.h.n_given;
        // the given replicas carry lambda exactly when the least number that does is no larger
        bool ok = DERIVE ? n <= a.r_max_d : need <= n;
        const double top =
            __builtin_fma(proc, p.h.lam, QUEUE == THEMIS_QUEUE_PER_REPLICA ? p.bh.w * n : p.bh.w);
        const double lt = ceil_div_small(top, p.h.rlt_den);
        ok = ok && lt <= p.h.T;
        const double key = __builtin_fma(n * (double)c, 32768.0, lt);
        return ok ? (uint32_t)key : EMPTY;
    }
    template <bool SMALL>
    __device__ __forceinline__ uint32_t meet(const Pair& p, uint32_t c) const
    {
        return meet<SMALL>(p, c, recip_below((double)this->speed(p, c)));
    }

    // ---- step A ------------------------------------------------------------------
    // What the cost and the latency of a pair's candidates are at least, in single precision
    // with every term moved to the safe side by more than its error (2^-22 or so): with c
    // cores n = ceil(rn / c + rf) replicas, and td / c + tf + n tw ticks.  (With the replicas
    // given a cost says which core count it is, and every one is worth its evaluation.)
    struct Bounds {
        float rn, rf, td, tf, tw;
    };
    __device__ __forceinline__ Bounds bounds_of(const Pair& p) const
    {
        constexpr float DOWN = 0.999998f;
        Bounds b;
        const float num = (float)p.num, fixed = (float)p.fixed, rate = (float)p.ratio;
        b.rn = rate * num * DOWN, b.rf = rate * fixed * DOWN;
        const float per_us = (float)a.rtick * DOWN;
        b.td = num * per_us, b.tf = fixed * per_us;
        b.tw = p.w * __builtin_amdgcn_rcpf((float)lam) * per_us * DOWN;
        if (QUEUE != THEMIS_QUEUE_PER_REPLICA) b.tf += b.tw, b.tw = 0.0f;
        return b;
    }
    // The most cores with which candidates of the pair can cost as little as `limit`.
    __device__ __forceinline__ float most_cores(const Pair& p, const Bounds& b, float limit) const
    {
        const float most =
            __builtin_fminf((limit - b.rn) * __builtin_amdgcn_rcpf(b.rf) * 1.00001f, limit);
        return __builtin_fminf(most, (float)p.last);
    }
    // Which of the 32 core counts from c0 on, and up to `most`, can cost as little as `limit`
    // and (LATE) take fewer than `before` ticks: bit 31 is c0's.  Nine instructions a
    // count, four counts at a time, against thirty for an evaluation.
    template <bool LATE>
    __device__ __forceinline__ uint32_t promising(const Bounds& b, uint32_t c0, float most,
                                                  float limit, float before) const
    {
        uint32_t mask = 0u;
        const float over = most - (float)c0;
        float c = (float)c0;
        int n = 0;
#pragma unroll 1
        for (; n < 32 && any((float)n <= over); n += 4) {
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const float r = __builtin_amdgcn_rcpf(c);
                // negative where the count is promising
                const float reps = __builtin_ceilf(__builtin_fmaf(b.rn, r, b.rf));
                uint32_t sign = __float_as_uint(__builtin_fmaf(reps, c, -0.5f - limit));
                float y = b.tf;
                if (QUEUE == THEMIS_QUEUE_PER_REPLICA) y = __builtin_fmaf(reps, b.tw, y);
                if (LATE) sign &= __float_as_uint(__builtin_fmaf(b.td, r, y) + (0.9f - before));
                mask = __builtin_amdgcn_alignbit(mask, sign, 31);
                c += 1.0f;
            }
        }
        if (n == 0 || over < 0.0f) return 0u;
        const uint32_t counts = (uint32_t)(over < 31.0f ? over : 31.0f);
        return mask << (32 - n) & ~(0x7FFFFFFFu >> counts);
    }

    // The best candidate of the lanes' models.
    //
    // A lane evaluates the first core count that can be feasible, and then those that can
    // cost as little as the model's best: of 31 per instance at 65536 x 8 that lambda (num /
    // c + fixed) / (b 1e6) allows some two are left where that is rounded up.
    template <bool SMALL>
    __device__ __forceinline__ Best best_of(const Pair& p) const
    {
        const uint32_t c0 = this->first_core(p);
        bool go = p.there && c0 <= p.last;
        uint32_t c = go ? c0 : p.lo;
        uint32_t best = meet<SMALL>(p, c), best_c = c;
        best = go ? best : EMPTY;
        uint32_t model = model_least(p, best);
        if (DERIVE) {
            go = go && c < p.last;
            if (any(go)) {
                const Bounds b = bounds_of(p);
                for (;;) {
                    const float limit = (float)(model >> 15);
                    const float most = go ? most_cores(p, b, limit) : -1.0f;
                    go = go && (float)(c + 1u) <= most;
                    if (!any(go)) break;
                    uint32_t mask = promising<false>(b, c + 1u, most, limit, 0.0f);
                    const uint32_t from = c + 1u;
                    while (any(mask != 0u)) {
                        const bool is = mask != 0u;
                        const uint32_t z = (uint32_t)__builtin_clz(mask | 1u);
                        mask &= ~(0x80000000u >> z);
                        c = is ? from + z : p.lo;
                        const uint32_t key = meet<SMALL>(p, c);
                        // (cores ascend: of equal keys the first one met has the smaller index)
                        if (is && key < best) best = key, best_c = c;
                    }
                    model = model_least(p, best);
                    c = from + 31u;
                }
            }
        } else {
            // the cost grows with every core: a lane is done with its first feasible count
            go = go && best == EMPTY;
            while (any(go)) {
                go = go && ++c <= p.last && (double)c * p.h.n_given <= (double)(model >> 15);
                const uint32_t key = meet<SMALL>(p, c);
                if (go && key != EMPTY) best = key, best_c = c, go = false;
                model = model_least(p, best);
            }
        }
        Best b;
        b.key = model;
        b.c0 = c0;
        const uint32_t mine = __umul24(best_c - 1u, (uint32_t)a.n_batch) + p.j;
        b.k = model_least(p, best == model ? mine : EMPTY);
        b.c = best_c, b.own = best, b.size = p.size;
        b.mine = p.there && best == model && mine == b.k;
        return b;
    }
    // The same where a lane has several pairs, one after the other: of a pair only what can
    // still matter after those before it is evaluated.  (own, c, size, k: of the lane's own best;
    // key: the model's, in all of its lanes.)
    template <bool SMALL>
    __device__ __forceinline__ void improve(Best& b, const Pair& p) const
    {
        const uint32_t c0 = this->first_core(p);
        bool go = p.there && c0 <= p.last;
        auto offer = [&](uint32_t c, bool is) {
            const uint32_t key = meet<SMALL>(p, c);
            const uint32_t k = __umul24(c - 1u, (uint32_t)a.n_batch) + p.j;
            if (is && key != EMPTY && (key < b.own || (key == b.own && k < b.k)))
                b.own = key, b.k = k, b.c = c, b.size = p.size;
            return key;
        };
        if (DERIVE && this->one_each()) {
            if (any(go)) offer(go ? c0 : p.lo, go);
        } else if (DERIVE) {
            uint32_t from = c0;
            if (any(go && b.key == EMPTY)) {
                const bool is = go && b.key == EMPTY;
                offer(is ? c0 : p.lo, is);
                from = is ? c0 + 1u : c0;
                b.key = model_least(p, b.own);
            }
            if (!any(go)) return;
            const Bounds bound = bounds_of(p);
            for (;;) {
                const float limit = (float)(b.key >> 15);
                const float most = go ? most_cores(p, bound, limit) : -1.0f;
                go = go && (float)from <= most;
                if (!any(go)) break;
                uint32_t mask = promising<false>(bound, from, go ? most : -1.0f, limit, 0.0f);
                while (any(mask != 0u)) {
                    const bool is = mask != 0u;
                    const uint32_t z = (uint32_t)__builtin_clz(mask | 1u);
                    mask &= ~(0x80000000u >> z);
                    offer(is ? from + z : p.lo, is);
                }
                b.key = model_least(p, b.own);
                from += 32u;
            }
        } else {
            // the cost grows with every core: a lane is done with its first feasible count
            for (uint32_t c = c0;; ++c) {
                go = go && c <= p.last && (double)c * p.h.n_given <= (double)(b.key >> 15);
                if (!any(go)) break;
                const uint32_t key = offer(go ? c : p.lo, go);
                go = go && key == EMPTY;
                b.key = model_least(p, b.own);
            }
        }
    }

    // ---- step F ------------------------------------------------------------------
    // lt << 15 | cost of a candidate, EMPTY where there is none (of equal latencies any cost
    // will do).
    static __device__ __forceinline__ uint32_t turned(const Pair& p, uint32_t key)
    {
        return key == EMPTY || !p.there ? EMPTY : (key & 0x7FFFu) << 15 | key >> 15;
    }
    // That of the fastest candidate of the lanes' models.
    template <bool SMALL>
    __device__ __forceinline__ uint32_t fastest_of(const Start& first) const
    {
        static_assert(WIDTH != ROUNDS, "a lane has several models");
        uint32_t fast = EMPTY;
        for_pairs(first, [&](const Pair& p) { fast = least(fast, turned(p, meet<SMALL>(p, p.last))); });
        return model_least(first, fast);
    }
    // Sum of the models' least latencies, beyond any budget where one has no candidate.
    template <bool SMALL>
    __device__ __forceinline__ uint32_t fastest_ticks(const Start& first) const
    {
        return sum_of_models(first, fastest_of<SMALL>(first) >> 15);
    }

    // ---- the tables of steps B and C ----------------------------------------------
    // (lt, index) by cost over base, `cells` cells per model, of the candidates that are
    // dearer (by less than `span`) and faster than the model's best (`best`: its cost << 15 | lt).
    template <bool SMALL>
    __device__ __forceinline__ void enter(const Pair& p, uint32_t c0, uint32_t best, uint32_t cells,
                                          uint32_t span) const
    {
        uint32_t* const tab = lds + L.tab;
        const uint32_t base = best >> 15, before = best & 0x7FFFu;
        const float limit = (float)(base + span - 1u);
        // two at a time: their chains of dependent operations fill each other's waits
        auto enter_two = [&](const bool (&is)[2], const uint32_t (&c)[2]) {
            uint32_t at[2], what[2];
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                const uint32_t key = meet<SMALL>(p, c[q]);
                const uint32_t d = (key >> 15) - base, lt = key & 0x7FFFu;
                // (EMPTY is beyond any cell)
                const bool use = (int)is[q] & (int)(d - 1u < span - 1u) & (int)(lt < before);
                at[q] = use ? p.s * cells + d : (uint32_t)lane;
                what[q] = use ? lt << INDEX_BITS | (__umul24(c[q] - 1u, (uint32_t)a.n_batch) + p.j) : EMPTY;
            }
            // EMPTY changes nothing, in a word of the lane's own: where all lanes without an
            // entry had the first word, one after the other, the atomics of a compute unit's
            // wavefronts took most of the time of a table (24000 x 6 with answers of 8 to 15
            // cells and replicas given 80 us instead of 48; under a branch 49.4, and small
            // batches up to half a microsecond longer)
            atomicMin(&tab[at[0]], what[0]);
            atomicMin(&tab[at[1]], what[1]);
        };
        if constexpr (DERIVE) {
            const Bounds b = bounds_of(p);
            const float most = p.there ? most_cores(p, b, limit) : -1.0f;
            for (uint32_t from = c0; any((float)from <= most); from += 32u) {
                uint32_t mask = promising<true>(b, from, most, limit, (float)before);
                while (any(mask != 0u)) {
                    bool is[2];
                    uint32_t c[2];
#pragma unroll
                    for (int q = 0; q < 2; ++q) {
                        is[q] = mask != 0u;
                        const uint32_t z = (uint32_t)__builtin_clz(mask | 1u);
                        mask &= ~(0x80000000u >> z);
                        c[q] = is[q] ? from + z : p.lo;
                    }
                    enter_two(is, c);
                }
            }
        } else {
            const float r = __builtin_amdgcn_rcpf((float)p.h.n_given);
            const float most =
                p.there ? __builtin_fminf(limit * r * 1.00001f, (float)p.last) : -1.0f;
            const uint32_t least_c = (uint32_t)((float)base * r * 0.9999f);
            for (uint32_t from = least_c > c0 ? least_c : c0; any((float)from <= most); from += 2u) {
                const bool is[2] = {(float)from <= most, (float)(from + 1u) <= most};
                const uint32_t c[2] = {is[0] ? from : p.lo, is[1] ? from + 1u : p.lo};
                enter_two(is, c);
            }
        }
    }

    // ---- step B ------------------------------------------------------------------
    // The recurrence over eight cells for eight models at a time, lane = (model, cell): rows of
    // neighbouring models are combined, then of two and two, of four and four (and with the
    // row of the models behind those), so that three or four dependent steps take the place of
    // one per model.  The choices of all models at all cells are read out together, and what
    // is left per model is one lane index.  (With the results' way out: 2.0 us for five models
    // and 3.3 for eight as sixteen cells a model after the other, 1.6 and 1.9 this way.  Sixteen
    // cells this way, two per lane, hold 32 values at once, with twenty registers spilled in
    // every kernel: 512 x 5 7.5 us instead of 7.2, stability 4099 x 5 19.4 instead of 18.8,
    // 22473 x 9 with replicas given 58.9 instead of 55.2.)
    // `span`: the cells over base up to which the table is complete; shift: its words per model,
    // as a power of two.
    __device__ __forceinline__ int solve_eight(uint32_t base_sum, int span, uint32_t shift) const
    {
        typedef uint32_t four __attribute__((ext_vector_type(4), aligned(16)));
        constexpr uint32_t INDEX = (1u << INDEX_BITS) - 1u;
        constexpr int CELLS = 8, STRIDE = 16, BITS = 3;
        const uint32_t* const tab = lds + L.tab;
        // rows of eight cells, as many guard cells in front of each
        uint32_t* const rows = lds + L.tab + 64 * a.S + 8;
        const int S = a.S, x = lane & 7, g = lane >> 3;
        for (int y = g; y <= S; y += 8) rows[STRIDE * y + x - 8] = LT_NONE;
        if (lane < CELLS) rows[STRIDE * S + lane] = 0u;  // nothing left to run
        // cells x, x - 1, .. x - 7 of a row that starts at `row`, and cells 0 .. 7
        auto backwards = [&](const uint32_t* row, uint32_t (&v)[8]) {
#pragma unroll
            for (int q = 0; q < 8; ++q) v[q] = (row + x - 7)[7 - q];
        };
        auto forwards = [](const uint32_t* row, uint32_t (&v)[8]) {
            const four a = *reinterpret_cast<const four*>(row);
            const four b = *reinterpret_cast<const four*>(row + 4);
            v[0] = a.x, v[1] = a.y, v[2] = a.z, v[3] = a.w, v[4] = b.x, v[5] = b.y, v[6] = b.z, v[7] = b.w;
        };
        uint32_t h = 0u;
        for (int s0 = (S - 1) & ~7; s0 >= 0; s0 -= 8) {
            const int end = s0 + 8 < S ? s0 + 8 : S;
            const bool is = s0 + g < end;
            const int s = is ? s0 + g : end - 1;
            uint32_t* const mine = rows + STRIDE * s;
            // (of at most x cells: with nothing behind them the models are done)
            h = segmented_scan<true>(tab[(s << shift) + x] >> INDEX_BITS, (uint32_t)x, 8u);
            if (is) mine[x] = h;
            wave_lds_fence();
            const int to = end < S ? end + 1 : end;
            for (int l = 1; l < to - s0; l *= 2) {
                const bool on = is && s + l < to;
                uint32_t f[8], o[8], all = LT_NONE;
                forwards(mine, f);
                backwards(rows + STRIDE * (on ? s + l : end), o);
#pragma unroll
                for (int q = 0; q < 8; ++q) all = least(all, f[q] + o[q]);
                wave_lds_fence();
                if (on) mine[x] = h = all;
                wave_lds_fence();
            }
        }
        uint32_t m = (uint32_t)__builtin_amdgcn_ballot_w64(h <= (uint32_t)T) & ((1u << span) - 1u);
        if (m == 0u) return UNFINISHED;
        int left = __builtin_ctz(m);
        this->put(THEMIS_SOLVED, (int32_t)(base_sum + (uint32_t)left), (int32_t)lane_value(h, left), BY_B8);
        for (int s0 = 0; s0 < S; s0 += 8) {
            const int s = s0 + g < S ? s0 + g : S - 1;
            const uint32_t* const mine = rows + STRIDE * s;
            // the smallest index among the candidates that continue an optimum, and its cell
            uint32_t pick = EMPTY, w[8], o[8];
            const uint32_t t = mine[x];
            forwards(tab + (s << shift), w);
            backwards(mine + STRIDE, o);
#pragma unroll
            for (int q = 0; q < 8; ++q) {
                const bool hit = (w[q] >> INDEX_BITS) + o[q] == t;
                pick = least(pick, hit ? (w[q] & INDEX) << BITS | (uint32_t)q : EMPTY);
            }
            const int n = S - s0 < 8 ? S - s0 : 8;
            unsigned long long chosen = 0ull;
            uint32_t none = 0u;
            for (int q = 0; q < n; ++q) {
                const int at = 8 * q + (left & 7);
                const uint32_t p = lane_value(pick, at);
                none |= p;
                chosen |= 1ull << at;
                left -= (int)(p & (uint32_t)(CELLS - 1));
            }
            if (none == EMPTY) {  // never expected
                this->put_none(THEMIS_INTERNAL);
                return THEMIS_INTERNAL;
            }
            this->put_row((int)((chosen >> lane) & 1ull), (uint32_t)s, pick >> BITS,
                          (this->keys()[s] >> 15) + (pick & (uint32_t)(CELLS - 1)));
        }
        return THEMIS_SOLVED;
    }

    // The largest rate for which the given replicas are known to do, by halves between 1 and
    // lambda, at which they do not.  A midpoint needs no recurrence: a configuration within
    // the budget exists exactly when the fastest candidates of all models fit it together, and
    // with the replicas given those are the ones at the core cap, whatever the rate.
    template <bool SMALL>
    __device__ __forceinline__ int32_t search_rate(const Start& first)
    {
        constexpr bool KEPT = ONE && SMALL && QUEUE != THEMIS_QUEUE_WORST_CASE;
        const int32_t lambda = lam;
        int32_t lo = 1, hi = lambda;
        double proc = 0.0, wait = 0.0;
        if constexpr (KEPT) {
            proc = ceil_div_small(first.num, recip_below((double)this->speed(first, first.last))) + first.fixed;
            wait = QUEUE == THEMIS_QUEUE_PER_REPLICA ? first.bh.w * first.h.n_given : first.bh.w;
        }
        while (hi - lo > 1) {
            lam = lo + ((hi - lo) >> 1);
            uint32_t ticks;
            if constexpr (KEPT) {
                // what meet() makes of it
                const double rate = (double)lam;
                const double lt = ceil_div_small(__builtin_fma(proc, rate, wait),
                                                 recip_below(rate * a.tick_d));
                const bool ok = (int)first.there & (int)(proc * (rate * first.bh.rM) <= first.h.n_given) &
                                (int)(lt <= first.h.T);
                const uint32_t fast = model_least(first, ok ? (uint32_t)lt : LT_NONE);
                ticks = sum_of_models(first, fast);
            } else {
                ticks = fastest_ticks<SMALL>(at_rate(first));
            }
            if (ticks <= (uint32_t)T)
                lo = lam;
            else
                hi = lam;
        }
        lam = lambda;
        return lo;
    }

    // Steps A, F and B of a valid instance.
    template <bool SMALL>
    __device__ __forceinline__ int solve_valid(const Start& first) const
    {
        Best mine{EMPTY, EMPTY, 0u, 1u, EMPTY, 0, false};
        uint32_t ticks = 0u, base_sum;
        bool vain = false;
        if constexpr (WIDTH == ROUNDS) {
            for_pairs(first, [&](const Pair& p) {
                const Best b = best_of<SMALL>(p);
                ticks += sum_of_models(p, b.key == EMPTY ? LT_NONE : b.key & 0x7FFFu);
                if (leads(p)) {
                    this->keys()[p.s] = b.key;
                    this->bests()[p.s] = (unsigned long long)b.key << INDEX_BITS | b.k;
                }
            });
        } else {
            if constexpr (ONE) {
                mine = best_of<SMALL>(first);
            } else {
                for_pairs<DERIVE>(first, [&](const Pair& p) {
                    vain = vain || this->in_vain();
                    if (!vain) improve<SMALL>(mine, p);
                });
                mine.key = model_least(first, mine.own);
                const uint32_t k = mine.own == mine.key ? mine.k : EMPTY;
                mine.k = model_least(first, k);
                mine.mine = first.there && mine.own != EMPTY && k == mine.k;
            }
            ticks = sum_of_models(first, mine.key == EMPTY ? LT_NONE : mine.key & 0x7FFFu);
        }
        if (ticks >= LT_NONE || vain) return THEMIS_INFEASIBLE;
        if constexpr (WIDTH == ROUNDS) {
            // from here on lane s has what was found about model s
            wave_lds_fence();
            const unsigned long long best = lane < a.S ? this->bests()[lane] : 0ull;
            mine.key = (uint32_t)(best >> INDEX_BITS);
            mine.k = (uint32_t)best & ((1u << INDEX_BITS) - 1u);
            base_sum = this->sum_models(mine.key >> 15);
        } else {
            base_sum = sum_of_models(first, mine.key >> 15);
        }
        if (ticks <= (uint32_t)T) {
            this->put(THEMIS_SOLVED, (int32_t)base_sum, (int32_t)ticks);
            if constexpr (WIDTH == ROUNDS)
                this->put_choice(mine.k, mine.key >> 15);
            else
                this->put_row(mine.mine, first.s, mine.c, ONE ? first.size : mine.size, mine.k, mine.key >> 15);
            return THEMIS_SOLVED;
        }
        const uint32_t word = this->vain_word();
        const bool one = this->one_each();
        uint32_t fast = 0u, least_ticks = 0u;
        if constexpr (WIDTH == ROUNDS) {
            for_pairs(first, [&](const Pair& p) {
                const uint32_t f = model_least(p, turned(p, meet<SMALL>(p, p.last)));
                least_ticks += sum_of_models(p, f >> 15);
                if (leads(p)) this->fastest()[p.s] = f;
            });
            wave_lds_fence();
            fast = lane < a.S ? this->fastest()[lane] : 0u;
        } else {
            // (where it is the lane's only candidate step A has met it)
            if constexpr (ONE)
                fast = one ? model_least(first, turned(first, mine.own)) : fastest_of<SMALL>(first);
            else
                fast = fastest_of<SMALL>(first);
            least_ticks = sum_of_models(first, fast >> 15);
            if (leads(first)) this->fastest()[first.s] = fast, this->keys()[first.s] = mine.key;
        }
        if (least_ticks > (uint32_t)T || vain || this->in_vain(word)) return THEMIS_INFEASIBLE;
        const int reach = reach_of(ticks, least_ticks, one, [&] {
            return (WIDTH == ROUNDS ? this->sum_models(fast & 0x7FFFu) : sum_of_models(first, fast & 0x7FFFu)) -
                   base_sum;
        });
        // (one candidate each: what there is to enter is at hand, for all windows at once)
        if (one) fill_one_each<SMALL>(first, mine);
        if (reach <= 8) {
            if (!one) fill<SMALL>(first, mine, 8, reach);
            const int status = solve_eight(base_sum, one ? 8 : reach, one ? 6u : 3u);
            if (status != UNFINISHED) return status;
            wave_lds_fence();
        }
        if (this->in_vain()) return THEMIS_INFEASIBLE;
        if (reach <= 16) {
            if (!one) fill<SMALL>(first, mine, 16, 16);
            const int status = this->solve_sixteen(base_sum, one ? 64 : 16);
            if (status != UNFINISHED) return status;
            wave_lds_fence();
        }
        if (!one && !this->shares_pairs()) fill<SMALL>(first, mine, 64, 64);
        return UNFINISHED;
    }
    // How many cells it takes, by how late the cheapest assignment is (`late`), what the fastest
    // gains on it (`gain`) and how much more that one costs (span()).  The answers' cells over
    // base grow as late / (1.1 gain - late) times the fourth root of the span: of the answers of
    // 700 shapes drawn over 1 to 10 models, 4 to 32 cores, every list of batch sizes and
    // objective, and of 6000 instances each of the numbered workloads, it is what a fit gives,
    // and the bounds are where a step too small costs what a step too large does (24000
    // instances of one class: eight cells 28 us, sixteen 47, sixty-four 69 beyond steps A and
    // F; a single wavefront 1.6, 3.4 and 6.4).  Where the replicas are derived and up to three
    // tenths of the gain is needed, four cells do, with next to no exception.  Where every pair
    // has one candidate a table serves all windows, and sixteen cells are always asked first:
    // in vain they cost 1 us of 12 to 17, left out in vain 2.5 of 10.  (By late / gain alone, at 26 and 31 of 40, or 14 and 26 with the replicas given, 43
    // and 24 % of those sent to sixty-four had fewer than sixteen: 134 x 10 11.7 us instead of
    // 9.6, 2 x 10 12.5 instead of 10.9, 13359 x 5 17.7 instead of 16.4; 16193 x 7 81.2 instead
    // of 82.5.)
    template <typename F>
    __device__ __forceinline__ int reach_of(uint32_t ticks, uint32_t least_ticks, bool one, F span) const
    {
        const float late = (float)(ticks - (uint32_t)T), gain = (float)(ticks - least_ticks);
        if (DERIVE && late <= 0.3f * gain) return 4;
        const float have = late * __builtin_amdgcn_sqrtf(__builtin_amdgcn_sqrtf((float)span()));
        const float need = 1.1f * gain - late;
        if (have <= need * (DERIVE && !one ? 4.5f : 2.6f)) return 8;
        return one || have <= need * (DERIVE ? 11.0f : 7.0f) ? 16 : 64;
    }
    // The table of `cells` cells per model.  mine: what step A found.
    template <bool SMALL>
    __device__ __forceinline__ void fill(const Start& first, const Best& mine, int cells, int span) const
    {
        uint32_t* const tab = lds + L.tab;
        for (int y = lane; y < cells * a.S; y += 64) tab[y] = EMPTY;
        wave_lds_fence();
        if (WIDTH == ROUNDS ? lane < a.S : leads(first))
            tab[(WIDTH == ROUNDS ? (uint32_t)lane : first.s) * cells] = (mine.key & 0x7FFFu) << INDEX_BITS | mine.k;
        wave_lds_fence();
        for_pairs(first, [&](const Pair& p) {
            enter<SMALL>(p, ONE ? mine.c0 : this->first_core(p), WIDTH == ROUNDS ? this->keys()[p.s] : mine.key,
                         (uint32_t)cells, (uint32_t)span);
        });
        wave_lds_fence();
    }
    // The table of 64 cells per model where every pair has one candidate.
    template <bool SMALL>
    __device__ __forceinline__ void fill_one_each(const Start& first, const Best& mine) const
    {
        uint32_t* const tab = lds + L.tab;
        for (int y = lane; y < 64 * a.S; y += 64) tab[y] = EMPTY;
        wave_lds_fence();
        for_pairs(first, [&](const Pair& p) {
            const uint32_t key = ONE ? mine.own : meet<SMALL>(p, p.last);
            const uint32_t d = (key >> 15) - ((WIDTH == ROUNDS ? this->keys()[p.s] : mine.key) >> 15);
            // (EMPTY is beyond any cell)
            const bool use = (int)p.there & (int)(d < 64u);
            atomicMin(&tab[use ? 64u * p.s + d : (uint32_t)lane],
                      use ? (key & 0x7FFFu) << INDEX_BITS | (__umul24(p.last - 1u, (uint32_t)a.n_batch) + p.j)
                          : EMPTY);
        });
        wave_lds_fence();
    }
    // The inputs of instance `inst` at the rate rates[inst], or at `rate`; valid: the input
    // check's result.
    //
    // The arguments this takes are held in scalar registers from the start: where the
    // compiler is free to load each where it is used, there are a dozen waits of 50 to 200
    // cycles, and the coefficients are asked for only after the rate has come.
    __device__ __forceinline__ Start begin(int inst, const int32_t* rates, bool& valid)
    {
        asm volatile("" ::"s"(rates));
        return begin(inst, constant(rates)[inst], valid);
    }
    __device__ __forceinline__ Start begin(int inst, int32_t rate, bool& valid)
    {
        i = inst;
        // (asked for, and not changed, here)
        asm volatile("" ::"s"(a.coef), "s"(a.slo_us), "s"(a.S), "s"(a.cs), "s"(a.n_batch), "s"(a.c_max),
                     "s"(a.r_max), "s"(a.tick), "s"(a.slo_max), "s"(a.coef_stride), "s"(a.c_all),
                     "s"(a.keep), "s"(a.c_fixed), "s"(a.r_fixed), "s"(a.kept.coef),
                     "s"(a.kept.cfg), "s"(a.kept.words), "s"(a.tmeta), "s"(a.tick_magic));
        lam = rate;
        slo = constant(a.slo_us)[inst];
        // floor(slo / tick), from below by at most one
        T = (int)__umulhi((uint32_t)slo, a.tick_magic);
        T += (uint32_t)(slo - T * a.tick) >= (uint32_t)a.tick ? 1 : 0;
        int32_t word = 0;
        const bool keeps = (ROLE == PLAIN || ROLE == PINNED) && a.keep && a.coef_stride;
        if (keeps && lane < a.S * a.cs) word = (a.coef + (size_t)i * (uint32_t)a.coef_stride)[lane];
        const Start first = start();
        this->lane_b = first.size;  // (the first lanes have the first model's pairs)
        int fine = (int)in_range(lam, 1, THEMIS_VALUE_MAX) & (int)in_range(slo, 0, a.slo_max);
        if constexpr (WIDTH == ROUNDS)
            for_pairs(first, [&](const Pair& p) { fine &= (int)!p.there | (int)p.valid; });
        else
            fine &= (int)!first.there | (int)first.valid;
        valid = !any(!fine);
        this->keep_inputs(valid, word);
        if (this->records() && lane == 0) a.tmeta[i] = valid ? T : -1;
        return first;
    }
    // The pair kept from another rate at the rate `lam` (where pairs are not kept they are
    // formed at that rate anyway).
    __device__ __forceinline__ Start at_rate(Start p) const
    {
        if constexpr (ONE) this->set_rate(p);
        return p;
    }

    // row_is_small(), which is the same for all models of an instance
    __device__ __forceinline__ bool is_small() const
    {
        return __umulhi((uint32_t)lam, (uint32_t)slo) < 1u << 10;
    }
    // Steps A, F and B of the instance that was begun, at the rate `lam`, with the results
    // where these suffice.
    __device__ __forceinline__ int solve(const Start& first, bool valid) const
    {
        int status = valid ? LARGE : THEMIS_INVALID;
        if (valid && is_small())
            status = solve_valid<true>(first);
        return __builtin_amdgcn_readfirstlane(status);
    }
    // What is left to do after that, and the results of an instance without an answer.
    __device__ __forceinline__ int finish(int status) const
    {
        if (status == THEMIS_SOLVED) return status;
        if (status != UNFINISHED && status != LARGE) {
            this->put_none(status);
            return status;
        }
        return __builtin_amdgcn_readfirstlane(solve_rest<QUEUE, DERIVE, ROLE, MANY>(
            (uint64_t)(uintptr_t)afresh(args), i, T, lam, slo));
    }
    // The same pointer, to arguments that the compiler hasn't loaded yet.
    static __device__ __forceinline__ ArgsPtr afresh(ArgsPtr p)
    {
        asm volatile("" : "+s"(p));
        return p;
    }
};

// The rate the given replicas of an instance are solved at (see Front::search_rate()), where
// products exceed 2^42.
template <int QUEUE>
__device__ __attribute__((noinline)) int32_t rate_of_large(uint64_t args, int i, int T, int32_t lam,
                                                           int32_t slo)
{
    auto uniform = [](int v) { return __builtin_amdgcn_readfirstlane(v); };
    const uint64_t lo = (uint32_t)uniform((int)(uint32_t)args);
    const uint64_t hi = (uint32_t)uniform((int)(uint32_t)(args >> 32));
    Front<QUEUE, false, TURNS, QUIET> sv((ArgsPtr)(uintptr_t)(hi << 32 | lo));
    sv.instance(uniform(i), uniform(T), uniform(lam), uniform(slo));
    const auto first = sv.start();
    return uniform(sv.template fastest_ticks<false>(first) <= (uint32_t)sv.T
                       ? sv.lam
                       : sv.template search_rate<false>(first));
}

// What an instance needs that most of them do not, out of their way: with calls between the
// steps instead of one behind them all, what the steps keep in registers went to scratch
// memory around them (86400 x 6: 99 us instead of 45 at the time).  That includes steps A, F
// and B where products exceed 2^42, with rates times objectives beyond those of any of the
// numbered workloads by a factor of 200.  (Step B's sixteen cells stay with the others:
// from here 4096 x 5 took 12.4 us instead of 11.2.)
template <int QUEUE, bool DERIVE, int ROLE, int MANY>
__device__ __attribute__((noinline)) int solve_rest(uint64_t args, int i, int T, int32_t lam,
                                                    int32_t slo)
{
    auto uniform = [](int v) { return __builtin_amdgcn_readfirstlane(v); };
    const uint64_t lo = (uint32_t)uniform((int)(uint32_t)args);
    const uint64_t hi = (uint32_t)uniform((int)(uint32_t)(args >> 32));
    auto sv = Front<QUEUE, DERIVE, MANY, ROLE>::of_wave((ArgsPtr)(uintptr_t)(hi << 32 | lo));
    sv.instance(uniform(i), uniform(T), uniform(lam), uniform(slo));
    int status;
    if (sv.is_small() ||
        (status = uniform(sv.template solve_valid<false>(sv.start()))) == UNFINISHED) {
        if (sv.shares_pairs() && !sv.one_each()) sv.fill_sixtyfour();
        status = sv.solve_further();
    }
    status = uniform(status);
    if (status == THEMIS_INVALID || status == THEMIS_INFEASIBLE) sv.put_none(status);
    return status;
}

// One whole solve of instance `inst` at the rate rates[inst].
template <int QUEUE, bool DERIVE, int WIDTH, int ROLE>
__device__ __forceinline__ int solve_instance(ArgsPtr args, int inst, const int32_t* rates,
                                              int lane = (int)threadIdx.x, uint32_t offset = 0u)
{
    Front<QUEUE, DERIVE, WIDTH, ROLE> sv(args, lane, offset);
    bool valid;
    const auto first = sv.begin(inst, rates, valid);
    return sv.finish(sv.solve(first, valid));
}

}  // namespace
}  // namespace themis
