// One wavefront's solve of one instance, for the kernels of cost_solve.hip and
// cost_multi.hip; the method is described in cost_solve.hip.
#pragma once

#include "candidate_eval.h"
#include "cost_plan.h"
#include "themis_internal.h"
#include "wave_ops.h"

namespace themis {
namespace {

constexpr uint32_t LT_NONE = 1u << 22;       // "no candidate": above any sum of 64 budgets
constexpr uint32_t EMPTY = 0xFFFFFFFFu;      // empty cell of the (lt, index) table
constexpr int INDEX_BITS = 13;               // candidate indices are below 8192
constexpr uint32_t G_INF = 0x8000u;          // row cell beyond any budget
constexpr uint32_t SAME = 0xFFFFFFFFu;       // for a choice: the one of the solve before

// A batch size b: recip_below(b 1e6), (b - 1) 1e6, and in single precision b 1e6 and
// b / (2 b - 1).  (What takes one instruction to form from these is not here: a launch
// takes the longer the larger its arguments are.)
struct __attribute__((aligned(16))) BatchConst {
    double rM, w;
    float M, both;
    int32_t size;
};

// What every instance needs.
struct HotArgs {
    const int32_t *coef, *lambda, *slo_us, *r_fixed, *c_fixed;
    int32_t S, cs, n_batch, width_log;  // see Front
    int32_t c_max, r_max, tick, slo_max;
    int32_t coef_stride;  // words of an instance's coefficients (shared: 0)
    int32_t c_all;
    uint32_t magic;       // index_magic() of n_batch
    int32_t window;       // cells of the largest window with rows in LDS, a multiple of 64
    double rtick, tick_d, r_max_d;
    uint32_t tick_magic;  // floor(2^32 / tick)
    float r_max_f;
    int32_t* keep;        // inputs and results for calls that inspect the workspace, or null
    KeepLayout kept;
    int32_t* tmeta;       // budgets, for such calls
    int32_t *status, *cost, *ticks, *cfg;
};
struct CostArgs : HotArgs {
    const int32_t* lambda2;  // stability test: the predicted rates
    int32_t *status2, *cost2, *ticks2, *cfg2;  // results of the second kind, see ROLE
    int32_t *lambda_v, *stable;
    const int32_t* list;  // the instances to solve (LISTED)
    int32_t* ctrl;
    uint16_t* frow;       // rows of step D, by budget
    uint16_t* hrow;       // rows of steps G and W, by cost, where LDS has no room
    int32_t hrow_stride;  // cells of hrow per instance
    int32_t row_stride;
    int32_t window_hbm;   // like `window`, in HBM (no larger than the other: none)
    int32_t lds_words;    // of one wavefront, see CostLds
    uint32_t wave_words;  // LDS words of each wavefront of a workgroup (0: there is one)
    uint32_t parts, pair_magic;  // lanes per (model, batch size) pair of a sweep, see sweep()
    int32_t width;         // how the pairs lie in the wavefront, see Front
    int32_t lanes, turns;  // lanes per model, and the batch sizes of each, see Front
    uint32_t lane_magic;   // index_magic() of them
    int32_t round_log, per_round;  // see FrontLayout
    BatchConst bc[THEMIS_MAX_BATCH];
};

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

// Inputs that no kernel of the solve writes: uniform reads as scalar loads.
template <typename T>
__device__ __forceinline__ const __attribute__((address_space(4))) T* constant(const T* p)
{
    return (const __attribute__((address_space(4))) T*)(uintptr_t)p;
}

extern __shared__ uint32_t cost_smem[];

// which of its workgroup's wavefronts this is
__device__ __forceinline__ uint32_t wave_number()
{
    return (uint32_t)__builtin_amdgcn_readfirstlane((int)threadIdx.x) >> 6;
}

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
// Besides the status of an instance: the steps so far did not suffice; the lists are made;
// the lists are to be made by narrowing; products exceed 2^42.
constexpr int UNFINISHED = -1, ARE_LISTED = -2, TOO_MANY = -3, LARGE = -4;

// What follows on step C is in functions of their own, called one after the other: LIST, the lists
// of step G where all candidates fit them; NARROW, those lists where they do not, by way of
// PRICE; GAP, step G up to its end, which is TRIAL, ROWS or ROWS_HBM; WD, steps W and D.
enum { PART_LIST, PART_PRICE, PART_NARROW, PART_GAP, PART_TRIAL, PART_ROWS, PART_ROWS_HBM, PART_WD };
template <int QUEUE, bool DERIVE, int ROLE, int PART>
__device__ __attribute__((noinline)) int solve_part(uint64_t args, int i, int T, int32_t lam,
                                                    int32_t slo, int x);

// One wavefront's view of the instance it works on.
template <int QUEUE, bool DERIVE, int ROLE>
struct Solver {
    const ArgsPtr args;
    HotArgs a;
    uint32_t* const lds;  // the wavefront's words
    const CostLds L;
    const int lane;

    // the instance
    int i, T;
    int32_t lam, slo;
    int32_t lane_b;  // lane j: batch size j

    // `offset`: of the wavefront's words
    __device__ __forceinline__ explicit Solver(ArgsPtr p, int l = (int)threadIdx.x, uint32_t offset = 0u)
        : args(p), a(hot_args(p)), lds(cost_smem + offset), L(cost_lds(p->S, p->window, p->lds_words)), lane(l)
    {
    }
    // (out of line, where a workgroup may have several wavefronts)
    static __device__ __forceinline__ Solver of_wave(ArgsPtr p)
    {
        return Solver(p, (int)threadIdx.x & 63, wave_number() * p->wave_words);
    }
    // (member by member: the address space has no copies of whole structures)
    static __device__ __forceinline__ HotArgs hot_args(ArgsPtr p)
    {
        static_assert(sizeof(HotArgs) == 192, "a member was added: copy it below");
        HotArgs h;
        h.coef = p->coef, h.lambda = p->lambda, h.slo_us = p->slo_us;
        h.r_fixed = p->r_fixed, h.c_fixed = p->c_fixed;
        h.S = p->S, h.cs = p->cs, h.n_batch = p->n_batch, h.width_log = p->width_log;
        h.c_max = p->c_max, h.r_max = p->r_max, h.tick = p->tick, h.slo_max = p->slo_max;
        h.coef_stride = p->coef_stride, h.c_all = p->c_all, h.magic = p->magic;
        h.window = p->window, h.rtick = p->rtick, h.tick_d = p->tick_d, h.r_max_d = p->r_max_d;
        h.tick_magic = p->tick_magic, h.r_max_f = p->r_max_f;
        h.keep = p->keep;
        h.kept.coef = p->kept.coef, h.kept.given = p->kept.given, h.kept.only = p->kept.only;
        h.kept.cfg = p->kept.cfg, h.kept.words = p->kept.words;
        h.tmeta = p->tmeta;
        h.status = p->status, h.cost = p->cost, h.ticks = p->ticks, h.cfg = p->cfg;
        return h;
    }

    // What a lane works on: one model and one batch size, cores lo .. last.
    struct Pair {
        RowHdr h;
        BatchHdr bh;
        double num, fixed;  // numerator of the division by the cores; what they do not shrink
        double ratio;       // at most lambda / (b 1e6), by 2^-44 of it or less
        float M, w, both;   // b 1e6, (b - 1) 1e6, see BatchConst
        int32_t size;
        uint32_t s, j, lo, last, pcap;
        bool there, valid;  // there: the lane has a pair
        bool in, first;     // its model exists; the lane is the model's first (see Front)
    };

    // One model as the caller's arrays have it.
    struct Model {
        words4 c4;
        int32_t v4, v5, given;
        uint32_t lo, hi;  // the cores: all, or one count for all models, or one for each
        bool valid;
    };
    __device__ __forceinline__ Model model_of(uint32_t s) const
    {
        Model m;
        const size_t row0 = (size_t)i * a.S;
        const int32_t* const cf = a.coef + (size_t)i * (uint32_t)a.coef_stride + s * (uint32_t)a.cs;
        m.c4 = *reinterpret_cast<const words4*>(cf);
        m.v4 = cf[4];
        m.v5 = 0;
        if (a.cs == 6) m.v5 = cf[5];
        m.given = DERIVE ? 0 : (a.r_fixed + row0)[s];
        // a, k, q, d in 0 .. max, p >= 1, o in 1 .. max
        uint32_t top = (uint32_t)m.c4.x > (uint32_t)m.c4.y ? (uint32_t)m.c4.x : (uint32_t)m.c4.y;
        top = (uint32_t)m.c4.z > top ? (uint32_t)m.c4.z : top;
        top = (uint32_t)m.v5 > top ? (uint32_t)m.v5 : top;
        m.valid = (int)(top <= (uint32_t)THEMIS_VALUE_MAX) & (int)(m.c4.w >= 1) &
                  (int)in_range(m.v4, 1, THEMIS_VALUE_MAX);
        if (!DERIVE) m.valid &= (int)in_range(m.given, 1, a.r_max);
        m.lo = a.c_all > 0 ? (uint32_t)a.c_all : 1u;
        m.hi = a.c_all > 0 ? (uint32_t)a.c_all : (uint32_t)a.c_max;
        if (ROLE == PINNED) {
            m.lo = m.hi = lds[L.pin + s];
        } else if (a.c_fixed) {
            const int32_t only = (a.c_fixed + row0)[s];
            m.valid &= (int)in_range(only, 1, a.c_max);
            m.lo = m.hi = only > 0 ? (uint32_t)only : 1u;
        }
        return m;
    }
    // A pair's parts.
    __device__ __forceinline__ void batch_size(Pair& p, uint32_t j) const
    {
        const auto& bc = args->bc[j];
        p.j = j;
        p.bh.rM = bc.rM, p.bh.w = bc.w;
        p.M = bc.M, p.both = bc.both, p.size = bc.size;
        p.bh.b = (double)p.size;
        p.bh.b2 = p.bh.b * p.bh.b;
        p.bh.M = p.bh.b * 1.0e6;
        p.w = (float)p.bh.w;
    }
    __device__ __forceinline__ void of_model(Pair& p, const Model& m, uint32_t s) const
    {
        p.s = s;
        p.valid = m.valid;
        p.lo = m.lo;
        p.pcap = (uint32_t)m.c4.w;
        // beyond the cap a candidate has the cap's latency and costs more
        const uint32_t reach = p.pcap > p.lo ? p.pcap : p.lo;
        p.last = m.hi < reach ? m.hi : reach;
        p.h.a = (double)m.c4.x, p.h.k = (double)m.c4.y, p.h.q = (double)m.c4.z, p.h.o = (double)m.v4;
        p.h.d = (double)m.v5;
        p.h.p = (double)m.c4.w;
        p.h.slo = (double)slo, p.h.T = (double)T;
        p.h.n_given = (double)m.given;
        p.num = __builtin_fma(p.h.q, p.bh.b2, __builtin_fma(p.h.k, p.bh.b, p.h.a));
        p.fixed = p.h.o;
        if (a.cs == 6) p.fixed = __builtin_fma(p.h.d, p.bh.b, p.fixed);
        set_rate(p);
    }
    __device__ __forceinline__ Pair pair_of(uint32_t s, uint32_t j, bool there) const
    {
        s = there ? s : 0u, j = there ? j : 0u;
        Pair p;
        batch_size(p, j);
        of_model(p, model_of(s), s);
        p.there = there;
        return p;
    }

    // What depends on the rate.
    __device__ __forceinline__ void set_rate(Pair& p) const
    {
        p.h.lam = (double)lam;
        p.h.rlam = recip_below(p.h.lam);
        p.h.lt_den = p.h.lam * a.tick_d;
        p.h.rlt_den = recip_below(p.h.lt_den);
        p.ratio = p.h.lam * p.bh.rM;
    }

    // Whether every pair has one core count, and with it one candidate.
    __device__ __forceinline__ bool one_each() const
    {
        return ROLE == PINNED || a.c_fixed || a.c_all || a.c_max == 1;
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
            p.h, p.bh, p.num, p.fixed, rd, a.r_max_d, a.tick_d, a.rtick);
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
        const float room = (float)(T * a.tick) * UP;
        const float rl = __builtin_amdgcn_rcpf((float)lam);
        const float n_max = DERIVE ? a.r_max_f : (float)p.h.n_given;
        float wait = rl * DOWN * p.w;
        if (QUEUE == THEMIS_QUEUE_PER_REPLICA && !DERIVE) wait *= n_max;
        float most = __builtin_fminf(n_max * rl * UP * p.M, room - wait);
        // n >= lambda proc / (b 1e6), so the queue is at least (b - 1) / b proc
        if (QUEUE == THEMIS_QUEUE_PER_REPLICA && DERIVE)
            most = __builtin_fminf(most, room * UP * p.both);
        const float left = most - (float)p.fixed * DOWN;
        const float c = (float)p.num * __builtin_amdgcn_rcpf(left) * DOWN;
        const uint32_t c0 = (uint32_t)__builtin_ceilf(__builtin_fminf(c, 1.0e6f));
        // (c >= 0: num is)
        return !(left > 0.0f) || c0 > p.last ? p.last + 1u : c0 > p.lo ? c0 : p.lo;
    }

    // Whether a candidate of the pair with c cores or more can cost as little as
    // `limit`: n >= 1 and n >= lambda (num / c + fixed) / (b 1e6).
    __device__ __forceinline__ bool may_cost(const Pair& p, uint32_t c, uint32_t limit) const
    {
        if (!DERIVE) return (double)c * p.h.n_given <= (double)limit;
        return c <= limit &&
               __builtin_fma((double)c, p.fixed, p.num) * p.ratio <= (double)limit * (1.0 + 0x1p-40);
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
        return (ROLE == SECOND || ROLE == PINNED ? args->cfg2 : a.cfg) + (size_t)i * a.S * 3;
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
            (TWO ? args->status2 : a.status)[i] = status;
            (TWO ? args->cost2 : a.cost)[i] = cost;
            (TWO ? args->ticks2 : a.ticks)[i] = ticks;
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

    // Model s's candidate into the configuration, of the lanes with `who`: its cores, batch
    // size, index and cost.
    __device__ __forceinline__ void put_row(bool who, uint32_t s, uint32_t c, int32_t b, uint32_t k,
                                            uint32_t cost) const
    {
        if (!who) return;
        // cost / c: the exact quotient is a whole number up to 32767, half of 1 / c away
        // from where the truncation would go wrong
        const uint32_t n = (uint32_t)(((float)cost + 0.5f) * __builtin_amdgcn_rcpf((float)c));
        const uint32_t off = 3u * s;
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
        // for what the entry point does with it next
        if (ROLE != PINNED) {
            uint32_t* const at = lds + L.pin + s;
            const uint32_t choice = n << INDEX_BITS | k;
            *at = ROLE == SECOND && *at == choice ? SAME : choice;
        }
    }
    // ... by its index and cost (of all lanes together)
    __device__ __forceinline__ void put_row(bool who, uint32_t s, uint32_t k, uint32_t cost) const
    {
        const uint32_t q = index_quotient(k, a.magic);
        const int32_t b = __shfl(lane_b, (int)(k - q * (uint32_t)a.n_batch), 64);
        put_row(who, s, q + 1u, b, k, cost);
    }

    // lane s < S: index and cost of model s's candidate
    __device__ __forceinline__ void put_choice(uint32_t k, uint32_t cost) const
    {
        put_row(lane < a.S, (uint32_t)lane, k, cost);
    }

    // The instance's inputs into its record, see STATE_WORD.  `word`: word `lane` of the
    // coefficients, loaded with the rest of the inputs.
    __device__ __forceinline__ bool keeps_coef() const
    {
        return records() && a.coef_stride;  // shared: see mark_workspace()
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

    // ---- step B ------------------------------------------------------------------
    static __device__ __forceinline__ uint32_t entry(const Eval& ev, uint32_t k)
    {
        return ((uint32_t)ev.lt << INDEX_BITS) | k;
    }

    // Forward over the models, with the table of W <= 64 cells per model, `stride` from one
    // model to the next: the smallest index among the candidates that continue an optimum of
    // x cells over base and `ticks`.  rows: W cells each, of models 0 to S - 1 and of nothing
    // left to run.
    //
    // What bounds it is the chain from one model to the next: a read of LDS, a comparison, a
    // scan of its bits and a lane's value.  So nothing else is in it: a lane whose cost is
    // beyond x reads of the row before and is masked.
    template <int W, typename R>
    __device__ __forceinline__ int read_out(uint32_t total, uint32_t ticks, int x, int stride,
                                            const R* rows) const
    {
        constexpr uint32_t INDEX = (1u << INDEX_BITS) - 1u;
        const uint32_t* const tab = lds + L.tab;
        uint32_t t = ticks, my_k = 0, my_over = 0;
        const int d = lane & (W - 1);
        const R* row = rows + W - d;
        uint32_t e = tab[d];
        for (int s = 0; s < a.S; ++s) {
            const uint32_t r = (uint32_t)row[x];
            const uint32_t e_next = tab[(s + 1) * stride + d];  // (behind the last: of the rows)
            const unsigned long long who =
                __ballot((e >> INDEX_BITS) + r == t) & ((2ull << x) - 1ull);
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
            my_k = lane == s ? el & INDEX : my_k;
            my_over = lane == s ? (uint32_t)l : my_over;
            t -= el >> INDEX_BITS;
            x -= l;
            e = e_next;
            row += W;
        }
        put(THEMIS_SOLVED, (int32_t)total, (int32_t)ticks, W == 16 ? BY_B16 : BY_C);
        put_choice(my_k, my_over + (lane < a.S ? keys()[lane] >> 15 : 0u));
        return THEMIS_SOLVED;
    }

    // The recurrence over 16 cells.  Every row of sixteen lanes holds g[s+1][0..15]; row r
    // takes the table's costs 4 q + r, so its copy is first shifted by r and then by 4 q,
    // both operand modifiers, and the four rows' minima are combined.  (What does not beat
    // everything cheaper does no harm.)  `base_sum`: the sum of the models' least costs;
    // `stride`: words of the table per model.
    __device__ __forceinline__ int solve_sixteen(uint32_t base_sum, int stride) const
    {
        const uint32_t* const tab = lds + L.tab;
        uint32_t* const rows = lds + L.tab + 64 * a.S;
        uint32_t g = 0u;  // g[S]: nothing left to run
        const int at = lane >> 4;
        if (lane < 16) rows[a.S * 16 + lane] = 0u;
        for (int s = a.S - 1; s >= 0; --s) {
            const uint32_t* const mine = tab + s * stride + at;
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
        wave_lds_fence();
        return read_out<16>(base_sum + (uint32_t)x, ticks, x, stride, rows);
    }

    // ---- sweeps over the candidates, for steps C and G -----------------------------
    struct Cores {
        uint32_t lo, hi;  // lo > hi: none
    };

    // The cores with which candidates of the pair can cost as little as `limit`: the cost is
    // at least c (given replicas: n c) and at least lambda (num + fixed c) / (b 1e6).  Here
    // and below in single precision, with every term moved to the safe side by far more than
    // its error (2^-22 or so).
    __device__ __forceinline__ Cores cores_up_to(const Pair& p, uint32_t limit) const
    {
        const float most = (float)limit * 1.0001f;
        float hi;
        if (DERIVE) {
            hi = ((float)limit * __builtin_amdgcn_rcpf((float)p.ratio) * 1.0001f -
                  (float)p.num * 0.9999f) *
                     __builtin_amdgcn_rcpf((float)p.fixed) * 1.0001f + 1.0f;
            hi = most < hi ? most : hi;
        } else {
            hi = most * __builtin_amdgcn_rcpf((float)p.h.n_given) + 1.0f;
        }
        hi = hi < (float)p.last ? hi : (float)p.last;
        return Cores{first_core(p), hi > 0.0f ? (uint32_t)hi : 0u};
    }

    // The cores with which candidates of the pair can have cost + mu lt <= limit.  The cost
    // is as above, the latency at least (num / c + fixed + wait) / tick and, where the replica
    // count is derived and each one queues by itself, n >= lambda proc / (b 1e6) makes it
    // (2 - 1 / b) (num / c + fixed) / tick: with either of both, k0 + k1 c + latency + M / c
    // <= limit, so c lies between the roots of a quadratic.
    __device__ __forceinline__ Cores cores_within(const Pair& p, float mu, float limit) const
    {
        const float per_us = mu * (float)a.rtick;
        const float num = (float)p.num, fixed = (float)p.fixed;
        float wait = (float)p.bh.w * __builtin_amdgcn_rcpf((float)lam);
        if (QUEUE == THEMIS_QUEUE_PER_REPLICA && !DERIVE) wait *= (float)p.h.n_given;
        float lo = (float)first_core(p), hi = (float)p.last;
        auto cut = [&](float k0, float k1, float M, float latency) {
            const float R =
                limit - k0 - latency + 1.0e-4f * (limit + k0 + latency) + 1.0e-3f;
            const float D = R * R - 4.0f * k1 * (M * 0.9999f);
            if (!(R > 0.0f) || !(D >= 0.0f)) {
                hi = 0.0f;
                return;
            }
            const float q = R + __builtin_amdgcn_sqrtf(D);
            const float top = q * __builtin_amdgcn_rcpf(2.0f * k1) * 1.0001f + 1.0f;
            const float bottom = 2.0f * M * __builtin_amdgcn_rcpf(q) * 0.9998f - 1.0f;
            hi = top < hi ? top : hi;
            lo = bottom > lo ? bottom : lo;
        };
        const float M = per_us * num, latency = per_us * (fixed + wait);
        if (DERIVE) {
            const float rate = (float)p.ratio;
            const bool each_queues = QUEUE == THEMIS_QUEUE_PER_REPLICA;
            const float both = 2.0f - __builtin_amdgcn_rcpf((float)p.bh.b) * 1.0001f;
            auto cuts = [&](float k0, float k1) {
                cut(k0, k1, M, latency);
                if (each_queues) cut(k0, k1, both * M, both * per_us * fixed);
            };
            cuts(0.0f, 1.0f);
            cuts(rate * num, rate * fixed);
            // no fewer replicas than with the most cores left, in turn
            for (int turn = 0; turn < 2; ++turn) {
                const float n = rate * (num * __builtin_amdgcn_rcpf(hi) + fixed) * 0.9999f;
                if (hi >= lo) cuts(0.0f, __builtin_ceilf(n));
            }
        } else {
            cut(0.0f, (float)p.h.n_given, M, latency);
        }
        return Cores{(uint32_t)lo, (uint32_t)hi};
    }

    // The cores of the pair with about the least cost + mu lt at the least replica count (or
    // `more` above it): as few as that count allows, or where another one saves less in
    // latency than it costs.
    __device__ __forceinline__ uint32_t likely_core(const Pair& p, float mu, uint32_t more) const
    {
        const float num = (float)p.num, fixed = (float)p.fixed, rate = (float)p.ratio;
        const float last = (float)p.last;
        float n = (float)p.h.n_given, least_c = 0.0f;
        if (DERIVE) {
            n = __builtin_ceilf(rate * (num * __builtin_amdgcn_rcpf(last) + fixed)) + (float)more;
            least_c = rate * num * __builtin_amdgcn_rcpf(n - rate * fixed);
        }
        float c = __builtin_amdgcn_sqrtf(mu * (float)a.rtick * num * __builtin_amdgcn_rcpf(n));
        c = c > least_c ? c : least_c;
        c = __builtin_ceilf(c);
        c = c < last ? c : last;
        return c > (float)p.lo ? (uint32_t)c : p.lo;
    }

    // Calls use(pair)(cores, lt, cost) for the feasible candidates among range(pair).  Lanes
    // are pairs, 64 at a time; where all pairs fit half of the lanes, several lanes share a
    // pair's cores.  DEALT: where one lane would have far more of them than the others, all
    // are dealt out, 64 at a time (1400 cycles, against 650 for two of every lane's own; with
    // the replicas given the lanes' shares differ too little to look for that).
    // SAMPLE: the more cores, the fewer of them (every eighth of their number).
    // One or two core counts are evaluated whatever range() would say, which takes longer.
    enum How { DEALT, SAMPLE };
    template <How HOW, typename R, typename F>
    __device__ __forceinline__ void sweep(R range, F use) const
    {
        const Recips rc = recips();
        const bool few = ROLE == PINNED || a.c_fixed || a.c_all || a.c_max <= 2;
        const uint32_t pairs = (uint32_t)(a.S * a.n_batch), parts = args->parts;
        const uint32_t part = parts > 1u ? index_quotient((uint32_t)lane, args->pair_magic) : 0u;
        auto after = [&](uint32_t c) {
            return c + (HOW == SAMPLE && (c >> 3) > parts ? c >> 3 : parts);
        };
        for (uint32_t r = 0; r < pairs; r += 64u) {
            const uint32_t x = r + (uint32_t)lane - part * pairs;
            const uint32_t s = index_quotient(x, a.magic);
            const Pair p = pair_of(s, x - s * (uint32_t)a.n_batch, x < pairs && part < parts);
            Cores c = few ? Cores{p.lo, p.last} : range(p);
            if (!p.there) c.hi = 0u;
            if (HOW == DEALT && DERIVE && !few && (uint32_t)a.c_max > 8u * parts) {
                const uint32_t mine = part == 0u && c.lo <= c.hi ? c.hi - c.lo + 1u : 0u;
                const uint32_t end = wave_scan<false>(mine), all = lane_value(end, 63);
                const uint32_t most = ~lane_value(wave_scan<true>(~mine), 63);
                if (most > 5u * parts * ((all + 63u) / 64u)) {
                    deal_out(p, rc, c.lo, end - mine, all, use);
                    continue;
                }
            }
            const auto meet = use(p);
            c.lo += part;
            for (;;) {
                // two at a time: their chains of dependent operations fill each other's waits
                const bool go = c.lo <= c.hi;
                if (__ballot(go) == 0ull) break;
                const uint32_t c1 = after(c.lo);
                const bool both = go && c1 <= c.hi;
                const double r0 = recip(rc, go ? speed(p, c.lo) : 1u);
                const double r1 = recip(rc, both ? speed(p, c1) : 1u);
                if (go) {
                    const Eval e0 = eval<false>(p, r0), e1 = eval<false>(p, r1);
                    if (e0.lt >= 0) meet(c.lo, (uint32_t)e0.lt, __umul24((uint32_t)e0.n, c.lo));
                    if (both && e1.lt >= 0) meet(c1, (uint32_t)e1.lt, __umul24((uint32_t)e1.n, c1));
                    c.lo = after(c1);
                }
            }
        }
        wave_lds_fence();
    }

    // The candidates of all lanes' pairs p, `all` of them: a lane's first one is number
    // `start` of all and has `lo` cores.
    template <typename F>
    __device__ __forceinline__ void deal_out(const Pair& p, const Recips& rc, uint32_t lo,
                                             uint32_t start, uint32_t all, F use) const
    {
        auto fetch = [](uint32_t v, int from) { return (uint32_t)__shfl((int)v, from, 64); };
        const uint32_t what = p.s << 4 | p.j;
        for (uint32_t x0 = 0; x0 < all; x0 += 64u) {
            const uint32_t x = x0 + (uint32_t)lane;
            // whose it is: the last lane that starts at or before it
            int of = 0;
            for (int d = 32; d >= 1; d >>= 1)
                if (fetch(start, of + d) <= x) of += d;
            Pair q = p;
            const uint32_t sj = fetch(what, of);
            q.s = sj >> 4, q.j = sj & 15u;
            q.num = __shfl(p.num, of, 64);
            q.fixed = __shfl(p.fixed, of, 64);
            q.pcap = fetch(p.pcap, of);
            q.bh.M = __shfl(p.bh.M, of, 64);
            q.bh.rM = __shfl(p.bh.rM, of, 64);
            q.bh.w = q.bh.M - 1.0e6;
            const uint32_t c = fetch(lo, of) + (x - fetch(start, of));
            const bool go = x < all;
            const double rd = recip(rc, go ? speed(q, c) : 1u);
            if (go) {
                const Eval ev = eval<false>(q, rd);
                if (ev.lt >= 0) use(q)(c, (uint32_t)ev.lt, __umul24((uint32_t)ev.n, c));
            }
        }
    }

    // ---- step G ------------------------------------------------------------------
    // A candidate as lt << 15 | cost; in lists the index is in the next word.
    static __device__ __forceinline__ uint32_t lt_of(uint32_t w) { return w >> 15; }
    static __device__ __forceinline__ uint32_t cost_of(uint32_t w) { return w & 0x7FFFu; }
    static __device__ __forceinline__ float priced(float mu, uint32_t w)
    {
        return __builtin_fmaf(mu, (float)lt_of(w), (float)cost_of(w));
    }

    // Two words per candidate in lists: the above, and its index.
    struct Lists {
        uint32_t* bins;   // 64 words per model
        uint32_t* kept;   // per model: entries listed, later survivors
        uint32_t* floor;  // per model: entries its list has room for, later the least cost of
                          // its survivors
        uint32_t* first;  // per model: where its list starts, later its survivors, in words
                          // from `bins` on
        uint32_t* plan;   // cells of the survivors' rows, combinations worth trying
        uint32_t* lists;
        int room;         // words from `lists` on
    };

    __device__ __forceinline__ Lists lists_of() const
    {
        Lists l;
        l.bins = lds + L.tab;
        l.kept = l.bins + 64 * a.S;
        l.floor = l.kept + a.S;
        l.first = l.floor + a.S;
        l.plan = l.first + a.S;
        l.lists = l.plan + 2;
        l.room = L.words - L.tab - 67 * a.S - 2;
        return l;
    }
    // The room for lists divided evenly (at least fourteen entries each, see cost_lds()).
    __device__ __forceinline__ void divide_evenly(const Lists& l) const
    {
        const uint32_t len = (uint32_t)(l.room / (2 * a.S));
        if (lane < a.S) {
            l.first[lane] = (uint32_t)(l.lists - l.bins) + 2u * (uint32_t)lane * len;
            l.floor[lane] = len;
        }
        wave_lds_fence();
    }
    // ... or as the numbers in `kept` need it; false where there is not enough.
    __device__ __forceinline__ bool divide_by_need(const Lists& l) const
    {
        const uint32_t need = lane < a.S ? l.kept[lane] : 0u;
        const uint32_t end = wave_scan<false>(need);
        if (2u * lane_value(end, 63) > (uint32_t)l.room) return false;
        if (lane < a.S) {
            l.first[lane] = (uint32_t)(l.lists - l.bins) + 2u * (end - need);
            l.floor[lane] = need;
        }
        wave_lds_fence();
        return true;
    }

    // The survivors are packed in the place of the bins, in the order of their indices, or
    // still in the lists.  `free`: the other of the two places.
    struct Survivors : Lists {
        bool packed;
        uint32_t* free;
        int free_words;
    };
    __device__ __forceinline__ Survivors survivors() const
    {
        Survivors l{lists_of()};
        l.packed = __builtin_amdgcn_readfirstlane((int)l.first[0]) == 0;
        l.free = l.packed ? l.lists : l.bins;
        l.free_words = l.packed ? l.room : 64 * a.S;
        return l;
    }

    // A model's bins: as many costs in each as it takes for 64 of them to reach the fastest
    // candidate's.
    struct Bins {
        uint32_t* words;
        uint32_t base, top;  // least cost, fastest candidate's
        int shift;
        __device__ __forceinline__ bool reach(uint32_t cost) const { return cost <= top; }
        __device__ __forceinline__ uint32_t at(uint32_t cost) const { return (cost - base) >> shift; }
    };
    __device__ __forceinline__ Bins bins_of(const Lists& l, uint32_t s) const
    {
        Bins b;
        b.words = l.bins + 64u * s;
        b.base = keys()[s] >> 15;
        b.top = cost_of(fastest()[s]);
        const uint32_t range = b.top - b.base;  // its bits beyond six are cut
        b.shift = range < 64u ? 0 : 26 - __builtin_clz(range);
        return b;
    }
    // The fastest candidate of every bin, of all or of a sample of the candidates.
    template <How HOW>
    __device__ __forceinline__ void fill_bins(const Lists& l) const
    {
        for (int x = lane; x < 64 * a.S; x += 64) l.bins[x] = EMPTY;
        wave_lds_fence();
        if (lane < a.S) {
            const uint32_t cheapest = keys()[lane], fast = fastest()[lane];
            l.bins[64 * lane] = (cheapest & 0x7FFFu) << 15 | cheapest >> 15;
            const Bins b = bins_of(l, (uint32_t)lane);
            uint32_t* const last = &b.words[b.at(b.top)];
            *last = least(*last, fast);
        }
        wave_lds_fence();
        sweep<HOW>(
            [&](const Pair& p) { return cores_up_to(p, cost_of(fastest()[p.s])); },
            [&](const Pair& p) {
                return [b = bins_of(l, p.s)](uint32_t, uint32_t lt, uint32_t cost) {
                    if (b.reach(cost)) atomicMin(&b.words[b.at(cost)], lt << 15 | cost);
                };
            });
    }
    // Lists the candidates among range(pair) that pass(pair)(candidate) and that the fastest
    // candidate of their own and all cheaper bins, which the bins are turned into, does not
    // beat, nor that of the cheaper ones alone.  False when there are more of a model than its
    // list has room for.
    template <typename R, typename F>
    __device__ __forceinline__ bool list_candidates(const Lists& l, R range, F pass) const
    {
        for (int m = 0; m < a.S; m += 4) {
            uint32_t fast[4];
#pragma unroll
            for (int q = 0; q < 4; ++q)
                fast[q] = m + q < a.S ? l.bins[64 * (m + q) + lane] : 0u;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                fast[q] = wave_scan<true>(fast[q]);
                if (m + q < a.S) l.bins[64 * (m + q) + lane] = fast[q];
            }
        }
        if (lane < a.S) l.kept[lane] = 0u;
        wave_lds_fence();
        sweep<DEALT>(range, [&](const Pair& p) {
            return [=, passes = pass(p), b = bins_of(l, p.s), list = l.bins + l.first[p.s],
                    room = l.floor[p.s], s = p.s, j = p.j](uint32_t c, uint32_t lt, uint32_t cost) {
                const uint32_t x = lt << 15 | cost;
                if (!b.reach(cost) || !passes(x)) return;
                const uint32_t bin = b.at(cost);
                const uint32_t y = b.words[bin], z = bin > 0u ? b.words[bin - 1u] : EMPTY;
                if ((x != y && cost_of(y) <= cost && lt_of(y) <= lt) || lt_of(z) <= lt) return;
                const uint32_t at = atomicAdd(&l.kept[s], 1u);
                if (at < room) {
                    list[2u * at] = x;
                    list[2u * at + 1u] = (c - 1u) * (uint32_t)a.n_batch + j;
                }
            };
        });
        return __ballot(lane < a.S && l.kept[lane] > l.floor[lane]) == 0ull;
    }

    // The walk along the lower hull of (ticks, cost) between the cheapest assignment (too
    // slow) and the fastest (within the budget) to where the budget lies.
    struct Source {
        const uint32_t* words;  // this lane's model's candidates
        int n, step;
    };
    struct Hull {
        const Solver& sv;
        int width, s, sub;  // lanes per model; this lane's model, and which of its lanes it is
        bool there;
        int64_t c0, l0, c1, l1;  // cost and ticks of the assignments at both ends
        uint32_t cheap, fast;    // their choices of this lane's model
        float mu, v;             // the price of a tick; the model's least cost + mu lt
        uint32_t held[4];        // this lane's first entries of what the walk goes over

        __device__ __forceinline__ explicit Hull(const Solver& solver) : sv(solver), mu(0.0f), v(0.0f)
        {
            const int S = sv.a.S;
            width = 1;
            while (2 * width * S <= 64) width *= 2;
            s = sv.lane / width, sub = sv.lane & (width - 1);
            there = s < S;
            if (!there) s = 0;
            const uint32_t key = sv.keys()[s];
            cheap = (key & 0x7FFFu) << 15 | key >> 15, fast = sv.fastest()[s];
            c0 = total(cost_of(cheap)), l0 = total(lt_of(cheap));
            c1 = total(cost_of(fast)), l1 = total(lt_of(fast));
        }

        __device__ __forceinline__ int total(uint32_t x) const
        {
            return (int)wave_sum(there && sub == 0 ? x : 0u);
        }
        // (any price gives a bound, so its last bits do not matter)
        __device__ __forceinline__ float price() const
        {
            return (float)(int)(c1 - c0) * __builtin_amdgcn_rcpf((float)(int)(l0 - l1));
        }
        // Has choose() and changed() go over these candidates.
        __device__ __forceinline__ void hold(const Source& from)
        {
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int e = sub + q * width;
                held[q] = e < from.n ? from.words[from.step * e] : EMPTY;
            }
        }
        // calls f(candidate) for this lane's entries (EMPTY reads as a candidate slower and
        // dearer than any)
        template <typename F>
        __device__ __forceinline__ void each(const Source& from, F f) const
        {
#pragma unroll
            for (int q = 0; q < 4; ++q) f(held[q]);
            for (int e = sub + 4 * width; e < from.n; e += width) f(from.words[from.step * e]);
        }
        // The model's choice at the price, in all of its lanes, and its cost + mu lt.
        __device__ __forceinline__ uint32_t choose(const Source& from)
        {
            uint32_t w = EMPTY;
            v = 3.0e38f;
            each(from, [&](uint32_t x) {
                const float y = priced(mu, x);
                if (y < v) v = y, w = x;
            });
            with_partners(width, [&](auto of) {
                const float ov = __uint_as_float(of(__float_as_uint(v)));
                const uint32_t ow = of(w);
                if (ov < v || (ov == v && ow < w)) v = ov, w = ow;
            });
            return w;
        }
        // The assignment of the choices w becomes an end; true where the walk is over: on the
        // line between the ends, or above it.
        __device__ __forceinline__ bool ends(uint32_t w)
        {
            const int64_t c = total(cost_of(w)), t = total(lt_of(w));
            if (c * (l0 - l1) + (c1 - c0) * t >= c1 * (l0 - l1) + (c1 - c0) * l1) return true;
            if (t <= sv.T)
                c1 = c, l1 = t, fast = w;
            else
                c0 = c, l0 = t, cheap = w;
            return c0 >= c1 || l0 <= l1;
        }
        __device__ __forceinline__ void walk(const Source& from)
        {
            // (c0 >= c1: the price at hand is the last that means anything)
            for (int turn = 0; turn < 16 && c0 < c1; ++turn) {
                mu = price();
                if (ends(choose(from))) break;
            }
        }

        // The least cost after a change of one choice that leaves an assignment (cost c, t
        // ticks) within the budget; 2^30: there is none.
        __device__ __forceinline__ int changed(const Source& from, uint32_t choice) const
        {
            const int c = total(cost_of(choice)), t = total(lt_of(choice));
            uint32_t best = 0u;  // 2^16 less the change of the cost
            each(from, [&](uint32_t x) {
                const uint32_t gain = 0x10000u + cost_of(choice) - cost_of(x);
                if (t + (int)lt_of(x) - (int)lt_of(choice) <= sv.T && gain > best) best = gain;
            });
            const int b = (int)~lane_value(wave_scan<true>(~best), 63);  // the most of all lanes
            return b ? c + 0x10000 - b : 1 << 30;
        }
        // The cost of some assignment within the budget: from the choices of the faster end,
        // as many models as the ticks left over allow go over to those of the cheaper end,
        // then one choice changes; or one model more goes over, or all, and then one choice
        // changes that takes it back into the budget.
        __device__ __forceinline__ int upper(const Source& from) const
        {
            const int left = sv.T - (int)l1;
            const int d = there ? (int)lt_of(cheap) - (int)lt_of(fast) : 0;
            // (the first lane of a model counts, so its lanes have the same sum)
            const int sum = (int)wave_scan<false>(sub == 0 && d > 0 ? (uint32_t)d : 0u);
            uint32_t choice[3];
            choice[0] = d > 0 && sum <= left ? cheap : fast;
            choice[1] = d > 0 && sum - d <= left ? cheap : fast;
            choice[2] = cheap;
            int ub = (int)c1;
#pragma unroll 1
            for (int x = 0; x < 3; ++x) {
                const int u = changed(from, x == 0 ? choice[0] : x == 1 ? choice[1] : choice[2]);
                ub = u < ub ? u : ub;
            }
            return ub;
        }
        // How much more than its model's least a candidate of an answer can have at the price,
        // in the light of an assignment of cost `ub`.
        __device__ __forceinline__ float gap_to(int ub) const
        {
            float bound = there && sub == 0 ? v : 0.0f;
            with_partners(64, [&](auto of) { bound += __uint_as_float(of(__float_as_uint(bound))); });
            bound -= mu * (float)sv.T;
            const float slack =
                ((float)(int)c1 + mu * (float)(sv.T + (int)l0)) * 0x1p-16f + 0x1p-10f;
            return (float)ub - bound + slack;
        }
    };

    // The price, and the gap at it, where there are too many candidates for a list of all: the
    // walk goes over a sample of them first and then over all, of which only those are
    // evaluated that can beat the sample's best at that price (cores_within()).
    __device__ __forceinline__ int find_price() const
    {
        const Lists l = lists_of();
        fill_bins<SAMPLE>(l);
        Hull h(*this);
        const Source bins{l.bins + 64 * h.s, h.there ? 64 : 0, 1};
        h.hold(bins);
        h.walk(bins);
        // over all candidates: per model the least cost + mu lt, and whose it is, from the
        // sample's on
        uint32_t w = 0u;
        for (int turn = 0;; ++turn) {
            h.hold(bins);
            const uint32_t sampled = h.choose(bins);
            if (turn > 0 && priced(h.mu, w) < h.v)
                h.v = priced(h.mu, w);
            else
                w = sampled;
            if (h.there && h.sub == 0)
                bests()[h.s] = (unsigned long long)__float_as_uint(h.v) << 32 | w;
            wave_lds_fence();
            auto offer = [&](const Pair& p) {
                return [mine = bests() + p.s, mu = h.mu](uint32_t, uint32_t lt, uint32_t cost) {
                    const uint32_t x = lt << 15 | cost;
                    atomicMin(mine, (unsigned long long)__float_as_uint(priced(mu, x)) << 32 | x);
                };
            };
            sweep<DEALT>(
                [&](const Pair& p) {
                    // the likeliest first: what they offer leaves the others less room
#pragma unroll 1
                    for (uint32_t more = 0u; more < 2u; ++more) {
                        const uint32_t c = likely_core(p, h.mu, more);
                        const Eval ev = eval<false>(p, recip_below((double)speed(p, c)));
                        if (p.there && ev.lt >= 0)
                            offer(p)(c, (uint32_t)ev.lt, __umul24((uint32_t)ev.n, c));
                    }
                    wave_lds_fence();
                    return cores_within(p, h.mu, __uint_as_float((uint32_t)(bests()[p.s] >> 32)));
                },
                offer);
            const unsigned long long best = bests()[h.s];
            h.v = __uint_as_float((uint32_t)(best >> 32));
            w = (uint32_t)best;
            if (h.ends(w) || turn == 7) break;
            h.mu = h.price();
        }
        h.hold(bins);
        const float gap = h.gap_to(h.upper(bins));
        if (lane == 0) l.plan[0] = __float_as_uint(h.mu), l.plan[1] = __float_as_uint(gap);
        wave_lds_fence();
        return TOO_MANY;
    }

    // Lists those within the gap at the price; false when they do not fit either.
    __device__ __forceinline__ bool list_narrowed() const
    {
        const Lists l = lists_of();
        const float mu = __uint_as_float(__builtin_amdgcn_readfirstlane(l.plan[0]));
        const float gap = __uint_as_float(__builtin_amdgcn_readfirstlane(l.plan[1]));
        auto least_priced = [&](const Pair& p) {
            return __uint_as_float((uint32_t)(bests()[p.s] >> 32));
        };
        auto range = [&](const Pair& p) { return cores_within(p, mu, least_priced(p) + gap); };
        auto near = [&](const Pair& p) {
            return [mu, gap, v = least_priced(p)](uint32_t x) { return priced(mu, x) - v <= gap; };
        };
        uint32_t key = 0, fast = 0;
        if (lane < a.S) key = keys()[lane], fast = fastest()[lane];
        bool fits = false;
        for (int turn = 0; turn < 4 && !fits; ++turn) {
            if (turn == 2) {
                // bins of the costs that those within the gap have
                if (lane < a.S) l.floor[lane] = EMPTY, l.first[lane] = 0u;
                wave_lds_fence();
                sweep<DEALT>(range, [&](const Pair& p) {
                    return [is_near = near(p), lo = l.floor + p.s, hi = l.first + p.s](
                               uint32_t, uint32_t lt, uint32_t cost) {
                        if (!is_near(lt << 15 | cost)) return;
                        atomicMin(lo, cost);
                        atomicMax(hi, cost);
                    };
                });
                for (int x = lane; x < 64 * a.S; x += 64) l.bins[x] = EMPTY;
                wave_lds_fence();
                // (in the place of what bins_of() goes by)
                if (lane < a.S) keys()[lane] = l.floor[lane] << 15, fastest()[lane] = l.first[lane];
                wave_lds_fence();
                sweep<DEALT>(range, [&](const Pair& p) {
                    return [is_near = near(p), b = bins_of(l, p.s)](uint32_t, uint32_t lt, uint32_t cost) {
                        const uint32_t x = lt << 15 | cost;
                        if (is_near(x)) atomicMin(&b.words[b.at(cost)], x);
                    };
                });
            }
            if (turn & 1) {
                if (!divide_by_need(l)) continue;
            } else {
                divide_evenly(l);
            }
            fits = list_candidates(l, range, near);
        }
        wave_lds_fence();
        if (lane < a.S) keys()[lane] = key, fastest()[lane] = fast;
        wave_lds_fence();
        return fits;
    }

    // Candidates that can be part of an answer at all, by Lagrangian bounds.  For any
    // price mu >= 0 of a tick, sum over the models of min(cost + mu lt) less mu T is at
    // most the optimum, and an assignment that uses a candidate whose cost + mu lt
    // exceeds its model's least by r costs at least r more than that bound.  With the
    // cost `ub` of some assignment within the budget, candidates with r > ub - bound are
    // in no optimum.  mu is found by walking the lower hull to where the budget lies.  Single
    // precision; `slack` covers its error, so a candidate is kept rather than dropped.
    // What is left is two or three candidates per model whose costs span some tens of
    // cells, where the window would have to span hundreds.
    //
    // What bounds it: latency, a chain of one wavefront's sweeps (300 cycles an evaluation),
    // walks (1200 a turn) and instruction fetches.  One instance of 8 models with 256
    // candidates takes 43 us (steps A to C 23 of them), of 3 models with 8192 75 to 96.
    // Before the narrowing and the trial by halves, where lists overflowed and the wide
    // windows and step D took over, batches of 4096 took, in microseconds, then and now (in
    // brackets by the three stages, dense / pruned): 64 models 8320 -> 407 (1240 / 647), 32
    // models 1980 -> 137 (626 / 334), 3 models of 8192 candidates with tight objectives
    // 5100 -> 1980 (3850 / 2280); 240 of 8 models with 2000 replicas 104 -> 41 (51 / 47).
    __device__ __forceinline__ int list_all() const
    {
        if (a.c_max * a.n_batch > FEW) return TOO_MANY;
        const Lists l = lists_of();
        fill_bins<DEALT>(l);
        divide_evenly(l);
        for (int turn = 0; turn < 2; ++turn) {
            if (turn > 0 && !divide_by_need(l)) break;
            if (list_candidates(
                    l, [&](const Pair& p) { return cores_up_to(p, cost_of(fastest()[p.s])); },
                    [](const Pair&) { return [](uint32_t) { return true; }; }))
                return ARE_LISTED;
        }
        return TOO_MANY;
    }

    // The survivors of the listed candidates, and what to do with them.
    __device__ __forceinline__ int find_survivors() const
    {
        const Lists l = lists_of();
        Hull h(*this);
        uint32_t* const mine = l.bins + l.first[h.s];
        const Source listed{mine, h.there ? (int)l.kept[h.s] : 0, 2};
        h.hold(listed);
        h.walk(listed);
        h.choose(listed);  // (the prices at which the walk stopped)
        const int ub = h.upper(listed);
        const float gap = h.gap_to(ub);
        // Those of this model's n entries that stay(entry, index), to the front of its list.
        auto keep = [&](int n, auto stay) {
            wave_lds_fence();
            if (lane < a.S) l.kept[lane] = 0u;
            wave_lds_fence();
            // (`width` entries at a time; their places are not behind those read so far)
            for (int e0 = 0; __ballot(e0 < n) != 0ull; e0 += h.width) {
                const int e = e0 + h.sub;
                const uint32_t x = e < n ? mine[2 * e] : 0u, k = e < n ? mine[2 * e + 1] : 0u;
                const bool stays = e < n && stay(x, k);
                wave_lds_fence();
                if (stays) {
                    const uint32_t at = atomicAdd(&l.kept[h.s], 1u);
                    mine[2 * at] = x, mine[2 * at + 1] = k;
                }
                wave_lds_fence();
            }
            return h.there ? (int)l.kept[h.s] : 0;
        };
        const int near =
            keep(listed.n, [&](uint32_t x, uint32_t) { return priced(h.mu, x) - h.v <= gap; });
        // no other one beats or ties it on cost and ticks (ties: smaller index)
        const int n = keep(near, [&](uint32_t x, uint32_t k) {
            bool beaten = false;
            for (int o0 = 0; o0 < near; o0 += 4) {
                uint32_t y[4], ky[4];
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const int o = o0 + q < near ? o0 + q : o0;
                    y[q] = mine[2 * o], ky[q] = mine[2 * o + 1];
                }
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    beaten |= cost_of(y[q]) <= cost_of(x) && lt_of(y[q]) <= lt_of(x) &&
                              (y[q] != x || ky[q] < k);
            }
            return !beaten;
        });
        const uint32_t my_kept = lane < a.S ? l.kept[lane] : 1u;
        if (__ballot(my_kept == 0u) != 0ull) return UNFINISHED;
        // the survivors of all models one after the other in the place of the bins, where that
        // has room for them
        const int entries = (int)sum_models(lane < a.S ? my_kept : 0u);
        const bool packed = entries <= 32 * a.S;
        const uint32_t before = wave_scan<false>(lane < a.S ? my_kept : 0u) - my_kept;
        if (lane < a.S) {
            l.floor[lane] = EMPTY;
            if (packed) l.first[lane] = 2u * before;
        }
        wave_lds_fence();
        for (int e = h.sub; e < n; e += h.width) {
            const uint32_t x = mine[2 * e], k = mine[2 * e + 1];
            atomicMin(&l.floor[h.s], cost_of(x));
            if (packed) {
                uint32_t rank = 0u;
                for (int o = 0; o < n; ++o) rank += mine[2 * o + 1] < k ? 1u : 0u;
                uint32_t* const to = l.bins + l.first[h.s] + 2u * rank;
                to[0] = x, to[1] = k;
            }
        }
        wave_lds_fence();
        const int span = ub - (int)sum_models(lane < a.S ? l.floor[lane] : 0u);
        if (span < 0) return UNFINISHED;
        const int W = (span + 64) & ~63;  // cells above the first that can be needed
        // Rows over W cells, or every combination.  By instructions: some 60 for every 256
        // cells and pair of entries (three times that with rows in HBM), 8 for every 64
        // combinations.
        const bool in_lds = (a.S + 1) * (W + 2) / 2 <= (packed ? l.room : 64 * a.S);
        const int rows = (W + 255) / 256 * entries * (in_lds ? 240 : 720);
        const int most = rows < TRIALS ? rows : TRIALS;
        // (the number of combinations by its logarithm, rounded down)
        auto log_of = [](uint32_t n) { return __builtin_amdgcn_logf((float)n) * 256.0f; };
        const bool few = (float)sum_models(lane < a.S ? (uint32_t)log_of(my_kept) : 0u) <= log_of((uint32_t)most);
        if (lane == 0) l.plan[0] = (uint32_t)W, l.plan[1] = few ? (uint32_t)most : 0u;
        wave_lds_fence();
        return ARE_LISTED;
    }
    // Candidates per model up to which all of them are listed if they fit: two evaluations of
    // each, against one of a sample and four or five of a few per pair otherwise (one
    // instance of 8 models with 256: 43 us this way, 52 the other).
    static constexpr int FEW = 512;
    // Combinations that are tried at all, and where nothing but step D is left.
    static constexpr int TRIALS = 1 << 18, MOST_TRIALS = 1 << 22;

    // The recurrence over the survivors: W cells over the sum of their least costs.
    // HBM: the rows are in this instance's part of the row region.
    template <bool HBM>
    __device__ __forceinline__ int solve_listed(int W) const
    {
        const Survivors l = survivors();
        const bool there = lane < a.S;
        const uint32_t my_floor = there ? l.floor[lane] : 0u, my_kept = there ? l.kept[lane] : 1u;
        const uint32_t my_first = there ? l.first[lane] : 0u;
        const int floor = (int)sum_models(my_floor);
        uint16_t* const rows = HBM ? args->hrow + (size_t)i * args->hrow_stride
                                   : reinterpret_cast<uint16_t*>(l.free);
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
        // entry e of model s, one of the lane's in advance
        auto entry_of = [&](int s, int e) {
            const int n = (int)lane_value(my_kept, s);
            return (l.bins + lane_value(my_first, s))[2 * (e < n ? e : 0)];
        };
        uint32_t w = entry_of(a.S - 1, lane);
        for (int s = a.S - 1; s >= 0; --s) {
            const uint16_t* const next = row_of(s + 1);
            uint16_t* const row = row_of(s);
            const int n = (int)lane_value(my_kept, s);
            const uint32_t base = lane_value(my_floor, s);
            // (four stretches of 64 and four entries at a time: reads that do not wait for
            // one another)
            for (int x0 = 0; x0 < W; x0 += 256) {
                uint32_t acc[4] = {G_INF, G_INF, G_INF, G_INF};
                for (int e = 0; e < n; e += 4) {
                    if (n > 64 && (e & 63) == 0) w = entry_of(s, e + lane);
                    uint32_t lt[4];
                    int d[4];
#pragma unroll
                    for (int z = 0; z < 4; ++z) {
                        const uint32_t wz = lane_value(w, (e + z < n ? e + z : e) & 63);
                        lt[z] = lt_of(wz), d[z] = (int)(cost_of(wz) - base);
                    }
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        if (x0 + 64 * q >= W) break;
                        uint32_t v[4];
#pragma unroll
                        for (int z = 0; z < 4; ++z) {
                            const int y = x0 + 64 * q + lane - d[z];
                            v[z] = next[y < -1 ? -1 : y] + lt[z];
                        }
                        acc[q] = least(least(acc[q], v[0]), least(v[1], least(v[2], v[3])));
                    }
                }
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    if (x0 + 64 * q < W) row[x0 + 64 * q + lane] = (uint16_t)acc[q];
            }
            if (s > 0) w = entry_of(s - 1, lane);
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
            const int n = (int)lane_value(my_kept, s), base = (int)lane_value(my_floor, s);
            const uint32_t* const ent = l.bins + lane_value(my_first, s);
            uint32_t key = EMPTY, key_w = 0u;
            for (int e0 = 0; e0 < n; e0 += 64) {
                const int e = e0 + lane;
                const uint32_t w = e < n ? ent[2 * e] : 0u, k = e < n ? ent[2 * e + 1] : 0u;
                const int d = (int)cost_of(w) - base;
                const bool in = e < n && d <= x;
                const uint32_t rest = row_of(s + 1)[in ? x - d : 0];
                unsigned long long m = __ballot(in && lt_of(w) + rest == t);
                while (m) {
                    const int q = __builtin_ctzll(m);
                    m &= m - 1ull;
                    const uint32_t kq = lane_value(k, q);
                    if (kq < key) key = kq, key_w = lane_value(w, q);
                }
            }
            if (key == EMPTY) {  // never expected
                put_none(THEMIS_INTERNAL);
                return THEMIS_INTERNAL;
            }
            if (lane == s) my_k = key, my_cost = cost_of(key_w);
            t -= lt_of(key_w);
            x -= (int)cost_of(key_w) - base;
        }
        put(THEMIS_SOLVED, (int32_t)total, (int32_t)ticks, HBM ? BY_G_HBM : BY_G_LDS);
        put_choice(my_k, my_cost);
        return THEMIS_SOLVED;
    }

    // Every combination of the survivors, if there are no more than `most`: every pair of a
    // combination of the first models, a lane each, and one of the others, in a list.  Both
    // are ticks << 15 | cost, beyond any budget where the ticks are.  (Costs add up to 32767
    // at most, so they do not carry into the ticks.)
    __device__ __forceinline__ int solve_by_trial(uint32_t most) const
    {
        const Survivors l = survivors();
        const uint32_t my_kept = lane < a.S ? l.kept[lane] : 1u;
        constexpr uint32_t LATE = 0xFFFFu << 15;
        uint32_t count = 1u;
        for (int s = 0; s < a.S; ++s) {
            count *= lane_value(my_kept, s);
            if (count > most) return UNFINISHED;
        }
        // the first models: as many as it takes to have work for all lanes and at least half of
        // the combinations' digits
        int half = 0;
        uint32_t n0 = 1u;
        while (half < a.S && (n0 < 64u || n0 * n0 < count)) n0 *= lane_value(my_kept, half++);
        const uint32_t n1 = count / n0;
        if (n1 + 3u > (uint32_t)l.free_words || n0 > 0xFFFFu) return UNFINISHED;
        uint32_t* const list = l.free;
        // Model s's digit of combination x as that survivor's words; x is left to the models
        // before it.  x / n: half of 1 / n from where the truncation would go wrong.
        const float my_recip = __builtin_amdgcn_rcpf((float)my_kept);
        const uint32_t my_first = lane < a.S ? l.first[lane] : 0u;
        auto digit = [&](uint32_t& x, int s) {
            const uint32_t n = lane_value(my_kept, s);
            const float r = __uint_as_float(lane_value(__float_as_uint(my_recip), s));
            const uint32_t q = (uint32_t)(((float)x + 0.5f) * r);
            const uint32_t* const e = l.bins + lane_value(my_first, s) + 2u * (x - q * n);
            x = q;
            return e;
        };
        // the models of either part, and its part of a pair x << 16 | y
        auto from = [&](int part) { return part ? half : 0; };
        auto to = [&](int part) { return part ? a.S : half; };
        auto of_pair = [](uint32_t pair, int part) { return part ? pair & 0xFFFFu : pair >> 16; };
        // an entry: combination x of one part's models
        auto entry_of = [&](int part, uint32_t x) {
            uint32_t c = 0, t = 0;
            // (four models at a time: reads that do not wait for one another)
            for (int s = to(part) - 1; s >= from(part); s -= 4) {
                uint32_t e[4];
#pragma unroll
                for (int q = 0; q < 4; ++q) e[q] = s - q >= from(part) ? *digit(x, s - q) : 0u;
#pragma unroll
                for (int q = 0; q < 4; ++q) c += cost_of(e[q]), t += lt_of(e[q]);
            }
            return t <= (uint32_t)T ? t << 15 | c : LATE;
        };
        wave_lds_fence();
        for (uint32_t x = (uint32_t)lane; x < n1 + 3u; x += 64u)  // read in fours
            list[x] = x < n1 ? entry_of(1, x) : LATE;
        wave_lds_fence();
        // whether one pair comes before another, by the indices of model 0, 1, ..
        auto precedes = [&](uint32_t p, uint32_t o) {
            if (l.packed) return p < o;
            bool is = false;  // the more significant a digit, the later it has its say
            for (int part = 1; part >= 0; --part) {
                uint32_t x = of_pair(p, part), y = of_pair(o, part);
                for (int s = to(part) - 1; s >= from(part); --s) {
                    const uint32_t kx = digit(x, s)[1], ky = digit(y, s)[1];
                    is = kx == ky ? is : kx < ky;
                }
            }
            return is;
        };
        const uint32_t late = ((uint32_t)T + 1u) << 15;
        uint32_t best = EMPTY, at = 0u;  // cost << 17 | ticks; which pair
        for (uint32_t x0 = 0; x0 < n0; x0 += 64u) {
            const uint32_t x = x0 + (uint32_t)lane;
            const uint32_t mine = x < n0 ? entry_of(0, x) : LATE;
            for (uint32_t y = 0; y < n1; y += 4u) {
                uint32_t v[4];
#pragma unroll
                for (uint32_t q = 0; q < 4u; ++q) v[q] = list[y + q];
#pragma unroll
                for (uint32_t q = 0; q < 4u; ++q) {
                    const uint32_t sum = mine + v[q];
                    const uint32_t key = sum < late ? sum << 17 | sum >> 15 : EMPTY;
                    if (key < best || (key == best && key != EMPTY && !l.packed)) {
                        const uint32_t now = x << 16 | (y + q);  // (ascending)
                        if (key < best || precedes(now, at)) at = now;
                        best = key;
                    }
                }
            }
        }
        const uint32_t key = lane_value(wave_scan<true>(best), 63);
        if (key == EMPTY) return UNFINISHED;  // never expected
        unsigned long long m = __ballot(best == key);
        uint32_t found = lane_value(at, __builtin_ctzll(m));
        for (m &= m - 1ull; m; m &= m - 1ull) {
            const uint32_t other = lane_value(at, __builtin_ctzll(m));
            if (__builtin_amdgcn_readfirstlane((int)precedes(other, found))) found = other;
        }
        // lane s: model s's digit of its part
        uint32_t below = 1u;  // combinations of the models after this one in its list
        for (int s = 1; s < a.S; ++s) {
            const uint32_t n = lane_value(my_kept, s);
            if (lane < s && s < to(lane >= half)) below *= n;
        }
        uint32_t my_k = 0, my_cost = 0;
        if (lane < a.S) {
            const uint32_t x = of_pair(found, lane >= half) / below;
            const uint32_t* const e = l.bins + my_first + 2u * (x % my_kept);
            my_cost = cost_of(e[0]), my_k = e[1];
        }
        put(THEMIS_SOLVED, (int32_t)(key >> 17), (int32_t)(key & 0x1FFFFu), BY_G_TRIAL);
        put_choice(my_k, my_cost);
        return THEMIS_SOLVED;
    }

    // ---- steps C and W -------------------------------------------------------------
    // The recurrence over 64 cells, the table of all models in LDS.
    //
    // Lane = two neighbouring cells, 16 bits each, the lower half of the wavefront for the
    // table's even costs over base, the upper for the odd ones: for an even cost the two cells
    // it leads from are a word of the row, for an odd one a word of a copy that is shifted by a
    // cell.  So 64 of the 64 x 64 pairs take a packed addition and a packed minimum, with operands
    // at fixed distances from a lane's first: no scan for the candidates worth a look, no address
    // of an entry's own.  Sums saturate, so "none" (all ones) stays above any budget.
    //
    // What bounds it: latency.  A model is one wait for the row written last, 32 costs at a
    // time, up to that of its fastest candidate.  A cell per lane, with every candidate that is
    // faster than all cheaper ones in turn, four at a time, took 5.0 us for eight models of
    // 65536 x 8, and the read-out 3.4; this takes 3.0 and 2.0.  The batches whose last wavefronts
    // end here: 16384 x 8 with replicas given 22.6 -> 20.4 us, stability 4099 x 5 17.4 -> 16.3,
    // 65536 x 8 76.2 -> 74.7.
    __device__ __forceinline__ int solve_sixtyfour() const
    {
        typedef uint32_t four __attribute__((ext_vector_type(4), aligned(16)));
        typedef uint16_t pair __attribute__((ext_vector_type(2)));
        constexpr uint32_t NONE = 0xFFFFu, BOTH = 0xFFFFFFFFu;
        const uint32_t* const tab = lds + L.tab;
        const StepCLds at = step_c_lds(a.S, L.tab);
        // 32 words per model; row s is "none" for the model before it until it is formed
        uint32_t* const rows = lds + at.rows;
        uint16_t* const cells = reinterpret_cast<uint16_t*>(rows);
        uint32_t* const odd = lds + at.copy;
        const bool upper = lane >= 32;
        const int m = lane & 31;
        for (int x = lane; x < 8 * (a.S - 1); x += 64)
            reinterpret_cast<four*>(rows)[x] = four{BOTH, BOTH, BOTH, BOTH};
        odd[m - 32] = BOTH;
        const uint32_t my_fast = lane < a.S ? fastest()[lane] >> 15 : 0u;
        auto latency = [](uint32_t e) { return least(e >> INDEX_BITS, NONE); };
        auto pair_of = [](uint32_t x) { return __builtin_bit_cast(pair, x); };
        auto faster = [&](uint32_t x, uint32_t y) {
            return __builtin_bit_cast(uint32_t, __builtin_elementwise_min(pair_of(x), pair_of(y)));
        };
        // Where a lane's words of a row are, in words from `rows` on: the lower half's of model 0
        // and their distance to the next model's; the upper half's are in the copy, a cell to
        // the left of which is the last of the word before it (none: of word 0).
        const int step = upper ? 0 : 32;
        const int place = upper ? (int)(odd - rows) + m : m;
        const uint32_t shift = !upper ? 0x07060504u : m > 0 ? 0x05040302u : 0x05040D0Du;
        // (w: the lower half's and the upper's are the same)
        auto put_words = [&](int s, uint32_t w) {
            rows[place + step * s] = __builtin_amdgcn_perm(w, from_lane_below(w, 0u), shift);
        };
        // a model's latencies, each in both halves of its word
        uint32_t* const my_entry = lds + (lane & 1 ? at.odd : at.even) + (lane >> 1);
        auto enter = [&](uint32_t lt) { *my_entry = lt << 16 | lt; };
        const four* const ent = reinterpret_cast<const four*>(lds + (upper ? at.odd : at.even));
        // the last model: the least of what costs no more
        cells[(a.S - 1) * 64 + lane] = (uint16_t)wave_scan<true>(latency(tab[(a.S - 1) * 64 + lane]));
        uint32_t lt = latency(tab[(a.S > 1 ? a.S - 2 : 0) * 64 + lane]);
        enter(lt);
        wave_lds_fence();
        put_words(a.S - 1, rows[32 * (a.S - 1) + m]);
        wave_lds_fence();
        for (int s = a.S - 2; s >= 0; --s) {
            // a lane's words of the row, from the last one on that it reads (the others are at
            // distances that fit the instruction)
            int last = place + step * (s + 1) - 31;
            asm("" : "+v"(last));
            const uint32_t* const from = rows + last;
            const uint32_t next = tab[(s > 0 ? s - 1 : 0) * 64 + lane];
            // nothing dearer than the fastest candidate is of use
            const uint32_t fast = (uint32_t)__ballot(lt <= lane_value(my_fast, s));
            uint32_t acc[2] = {BOTH, BOTH};
            auto costs = [&](int q0) {
                uint32_t v[16];
                four e[4];
#pragma unroll
                for (int q = 0; q < 4; ++q) e[q] = ent[q0 / 4 + q];
#pragma unroll
                for (int q = 0; q < 16; ++q) v[q] = from[31 - q0 - q];
#pragma unroll
                for (int q = 0; q < 16; ++q)
                    acc[q & 1] = faster(acc[q & 1], __builtin_bit_cast(uint32_t, __builtin_elementwise_add_sat(
                                                        pair_of(v[q]), pair_of(e[q / 4][q % 4]))));
            };
            costs(0);
            if (fast == 0u) costs(16);
            const uint32_t mine = faster(acc[0], acc[1]);
            const auto h = __builtin_amdgcn_permlane32_swap(mine, mine, false, false);
            lt = latency(next);
            wave_lds_fence();
            put_words(s, faster(h[0], h[1]));
            enter(lt);
            wave_lds_fence();
        }
        rows[32 * a.S + m] = 0u;  // nothing left to run
        wave_lds_fence();
        const uint32_t g = cells[lane];
        const unsigned long long within = __ballot(g <= (uint32_t)T);
        if (within == 0ull) return UNFINISHED;
        const int x = __builtin_ctzll(within);
        const uint32_t my_base = lane < a.S ? keys()[lane] >> 15 : 0u;
        return read_out<64>(sum_models(my_base) + (uint32_t)x, lane_value(g, x), x, 64, cells);
    }

    // Whether several lanes share a pair's cores in sweeps.
    __device__ __forceinline__ bool shares_pairs() const { return args->parts > 1u; }
    // The table of 64 cells per model, where they do: with a lane per pair half of the lanes
    // or more would have no part in it (16193 x 7 with three batch sizes 118 us instead of
    // 84, 25925 x 6 with four, replicas given, 73 instead of 60).  With more pairs than half
    // the lanes, those of step A, kept in registers, are the faster way (16384 x 8 with
    // replicas given 23.9 us instead of 25.2, 65536 x 8 76.0 instead of 77.4).
    __device__ __forceinline__ void fill_sixtyfour() const
    {
        uint32_t* const tab = lds + L.tab;
        for (int x = lane; x < a.S * 64; x += 64) tab[x] = EMPTY;
        wave_lds_fence();
        sweep<DEALT>(
            [&](const Pair& p) {
                const uint32_t base = keys()[p.s] >> 15;
                Cores c = cores_up_to(p, base + 63u);
                if (!DERIVE) {
                    const float least_c =
                        (float)base * __builtin_amdgcn_rcpf((float)p.h.n_given) * 0.9999f;
                    c.lo = least_c > (float)c.lo ? (uint32_t)least_c : c.lo;
                }
                return c;
            },
            [&](const Pair& p) {
                return [=, base = keys()[p.s] >> 15, mine = tab + 64u * p.s, j = p.j](
                           uint32_t c, uint32_t lt, uint32_t cost) {
                    if (cost - base < 64u)
                        atomicMin(&mine[cost - base],
                                  (lt << INDEX_BITS) | ((c - 1u) * (uint32_t)a.n_batch + j));
                };
            });
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
        uint16_t* const rows = HBM ? args->hrow + (size_t)i * args->hrow_stride
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
        uint16_t* const rows = args->frow + (size_t)i * a.S * args->row_stride;
        const uint32_t nbat = (uint32_t)a.n_batch;
        for (int s = a.S - 1; s >= 0; --s) {
            uint16_t* const out = rows + (size_t)s * args->row_stride;
            const uint16_t* const next = out + args->row_stride;
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
            const uint16_t* const next = rows + (size_t)(s + 1) * args->row_stride;
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

    template <int PART>
    __device__ __forceinline__ int out_of_line(int x = 0) const
    {
        return __builtin_amdgcn_readfirstlane(
            solve_part<QUEUE, DERIVE, ROLE, PART>((uint64_t)(uintptr_t)args, i, T, lam, slo, x));
    }

    // Step C, and if it does not suffice the lists of step G.
    __device__ __forceinline__ int solve_c() const
    {
        const int status = solve_sixtyfour();
        wave_lds_fence();
        return status == UNFINISHED ? out_of_line<PART_LIST>() : status;
    }

    // Whether the first of an instance's two wavefronts has found that there is no solution, and
    // what the second one is still about to find is not asked for: the second word behind its
    // others.  It looks between its steps (vain_word() ahead of one, in_vain() of it behind).
    __device__ __forceinline__ uint32_t vain_word() const
    {
        if (ROLE != SECOND || !args->wave_words) return 0u;
        return __hip_atomic_load(lds + L.words + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    }
    __device__ __forceinline__ bool in_vain(uint32_t word) const
    {
        return ROLE == SECOND && __builtin_amdgcn_readfirstlane((int)word) != 0;
    }
    __device__ __forceinline__ bool in_vain() const { return in_vain(vain_word()); }

    // Rows in HBM are the instance's.  Where both of its solves have a wavefront, the second one
    // waits with them until the first is done (which it says with a barrier as its last step).
    // The word behind its others tells whether it has.
    __device__ __forceinline__ void wait_for_rows() const
    {
        if (ROLE != SECOND || !args->wave_words) return;
        uint32_t* const waited = lds + L.words;
        if (__builtin_amdgcn_readfirstlane((int)*waited)) return;
        __syncthreads();
        if (lane == 0) *waited = 1u;
        wave_lds_fence();
    }

    // Steps C, G, W and D.
    __device__ __forceinline__ int solve_further() const
    {
        if (in_vain()) return THEMIS_INFEASIBLE;
        int status = solve_c();
        if (status == TOO_MANY) {
            if (in_vain()) return THEMIS_INFEASIBLE;
            out_of_line<PART_PRICE>();
            status = out_of_line<PART_NARROW>();
        }
        if (status == ARE_LISTED) {
            if (in_vain()) return THEMIS_INFEASIBLE;
            status = out_of_line<PART_GAP>();
        }
        if (status == ARE_LISTED) {
            if (in_vain()) return THEMIS_INFEASIBLE;
            const Survivors l = survivors();
            const int W = __builtin_amdgcn_readfirstlane((int)l.plan[0]);
            const int most = __builtin_amdgcn_readfirstlane((int)l.plan[1]);
            const int cells = (a.S + 1) * (W + 2);
            const bool in_lds = cells / 2 <= l.free_words;
            status = most ? out_of_line<PART_TRIAL>(most) : UNFINISHED;
            if (status == UNFINISHED && in_lds) status = out_of_line<PART_ROWS>(W);
            else if (status == UNFINISHED && cells <= args->hrow_stride) {
                wait_for_rows();
                if (in_vain()) return THEMIS_INFEASIBLE;
                status = out_of_line<PART_ROWS_HBM>(W);
            }
            if (status == UNFINISHED) status = out_of_line<PART_TRIAL>(MOST_TRIALS);
        }
        if (status != UNFINISHED) return status;
        wait_for_rows();
        if (in_vain()) return THEMIS_INFEASIBLE;
        return out_of_line<PART_WD>();
    }

    // Steps W and D.
    __device__ __forceinline__ int solve_wide() const
    {
        int status = UNFINISHED;
        int W = 64;
        while (status == UNFINISHED && W < a.window) {
            wave_lds_fence();
            W = 2 * W < a.window ? 2 * W : a.window;
            status = solve_window<false>(W);
        }
        while (status == UNFINISHED && W < args->window_hbm) {
            wave_lds_fence();
            W = 2 * W < args->window_hbm ? 2 * W : args->window_hbm;
            status = solve_window<true>(W);
        }
        wave_lds_fence();
        return status == UNFINISHED ? solve_by_budget(a.window) : status;
    }

    // An instance that was begun elsewhere.
    __device__ __forceinline__ void instance(int inst, int budget, int32_t rate, int32_t objective)
    {
        i = inst, T = budget, lam = rate, slo = objective;
        lane_b = lane < a.n_batch ? args->bc[lane].size : 0;
    }

    // A part of the solve of the instance, in a function of its own.
    template <int PART>
    __device__ __forceinline__ int part(int inst, int budget, int32_t rate, int32_t objective, int x)
    {
        instance(inst, budget, rate, objective);
        if constexpr (PART == PART_LIST) return list_all();
        if constexpr (PART == PART_PRICE) return find_price();
        if constexpr (PART == PART_NARROW) return list_narrowed() ? ARE_LISTED : UNFINISHED;
        if constexpr (PART == PART_GAP) return find_survivors();
        if constexpr (PART == PART_TRIAL) return solve_by_trial((uint32_t)x);
        if constexpr (PART == PART_ROWS) return solve_listed<false>(x);
        if constexpr (PART == PART_ROWS_HBM) return solve_listed<true>(x);
        if constexpr (PART == PART_WD) return solve_wide();
    }

};

// Out of line, so that their registers do not weigh on the allocation of the steps that
// nearly every instance ends with, nor on one another's.
template <int QUEUE, bool DERIVE, int ROLE, int PART>
__device__ __attribute__((noinline)) int solve_part(uint64_t args, int i, int T, int32_t lam,
                                                    int32_t slo, int x)
{
    auto uniform = [](int v) { return __builtin_amdgcn_readfirstlane(v); };
    const uint64_t lo = (uint32_t)uniform((int)(uint32_t)args);
    const uint64_t hi = (uint32_t)uniform((int)(uint32_t)(args >> 32));
    auto sv = Solver<QUEUE, DERIVE, ROLE>::of_wave((ArgsPtr)(uintptr_t)(hi << 32 | lo));
    return uniform(
        sv.template part<PART>(uniform(i), uniform(T), uniform(lam), uniform(slo), uniform(x)));
}

// What the class lists and the state word say about the workspace after a solve: no
// tables, the inputs and results in the table region.  Shared coefficients are in the
// first record, whether or not that instance is solved.
__device__ __forceinline__ void mark_workspace(ArgsPtr args, int state)
{
    if (blockIdx.x != 0) return;
    if ((int)threadIdx.x <= STATE_WORD)
        args->ctrl[threadIdx.x] = (int)threadIdx.x < STATE_WORD || !args->keep ? 0 : state;
    if (args->keep && !args->coef_stride)
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

// What does not depend on the entry point.
inline CostArgs cost_args(const themis_problem_t& p, const Layout& L, const int32_t* d_coef,
                          const int32_t* d_lambda, const int32_t* d_slo_us,
                          const int32_t* d_r_fixed, int32_t* d_status, int32_t* d_cost,
                          int32_t* d_ticks, int32_t* d_cfg, char* ws, const PassOpts& opts,
                          FrontWork work)
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
    // Rows by cost go where an instance has more of: of the row region, or of what the
    // records (at most sixteen words per model) leave of the table region.
    a.hrow = a.frow;
    a.hrow_stride = L.S * L.row_stride;
    const int left = L.S * (L.Kp - 8) * (int)(sizeof(StepEntry) / sizeof(uint16_t));
    if (left > a.hrow_stride) {
        a.hrow = (uint16_t*)(ws + L.step_off + (size_t)L.N * L.S * 8 * sizeof(StepEntry));
        a.hrow_stride = left;
    }
    a.keep = opts.inspectable ? (int32_t*)(ws + L.step_off) : nullptr;
    a.n_batch = p.n_batch;
    for (int j = 0; j < p.n_batch; ++j) {
        const double b = (double)p.batch_sizes[j];
        a.bc[j] = {(1.0 / (1.0e6 * b)) * (1.0 - 0x1p-45), 1.0e6 * (b - 1.0), (float)(1.0e6 * b),
                   (float)(b / (2.0 * b - 1.0)), p.batch_sizes[j]};
    }
    const FrontLayout front = front_layout(L.S, p.n_batch, work);
    a.width = front.width;
    a.width_log = front.width_log;
    a.lanes = front.lanes;
    a.turns = front.turns;
    a.round_log = front.round_log;
    a.per_round = front.per_round;
    a.lane_magic = index_magic((uint32_t)a.lanes);
    a.S = L.S;
    a.cs = p.profile_form == THEMIS_PROFILE_EQ1 ? 6 : 5;
    a.c_max = p.c_max;
    a.r_max = p.r_max;
    a.tick = p.tick_us;
    a.slo_max = p.slo_max_us;
    a.coef_stride = p.coef_shared ? 0 : L.S * a.cs;
    a.c_all = opts.c_all;
    a.list = opts.list;
    a.row_stride = L.row_stride;
    a.magic = index_magic((uint32_t)p.n_batch);
    const uint32_t pairs = (uint32_t)(L.S * p.n_batch);
    a.parts = pairs < 64u ? 64u / pairs : 1u;
    a.pair_magic = index_magic(pairs < 64u ? pairs : 64u);
    a.rtick = (1.0 / (double)p.tick_us) * (1.0 - 0x1p-45);
    a.tick_d = (double)p.tick_us;
    a.r_max_d = (double)p.r_max;
    a.r_max_f = (float)p.r_max;
    a.tick_magic = p.tick_us > 1 ? (uint32_t)((1ull << 32) / (uint32_t)p.tick_us) : 0xFFFFFFFFu;
    return a;
}

// The arguments with the arrays of all instances but the first n, for the launches after
// the first one of a large batch: offsets in the kernels would cost every solve (when it was
// measured, the fallback at 16384 x 8 62.8 us instead of 61.8, 65536 x 8 99.5 instead of
// 98.8).  (Each of these launches marks the workspace again, with the same words.)
inline CostArgs past(CostArgs a, size_t n)
{
    auto skip = [](auto*& array, size_t elements) {
        if (array) array += elements;
    };
    const size_t rows = n * (size_t)a.S;
    if (a.coef_stride) skip(a.coef, rows * a.cs);
    for (const int32_t** in : {&a.lambda, &a.slo_us, &a.lambda2}) skip(*in, n);
    for (const int32_t** in : {&a.r_fixed, &a.c_fixed}) skip(*in, rows);
    for (int32_t** out : {&a.status, &a.cost, &a.ticks, &a.status2, &a.cost2, &a.ticks2, &a.lambda_v,
                          &a.stable, &a.tmeta})
        skip(*out, n);
    for (int32_t** out : {&a.cfg, &a.cfg2}) skip(*out, 3 * rows);
    skip(a.frow, rows * a.row_stride);
    skip(a.hrow, n * a.hrow_stride);
    skip(a.keep, n * a.kept.words);
    return a;
}

// A workgroup per instance, or where `listed` as many as stay resident (the host does
// not know how long the list is).  `width` in kernel(width): see Front.
//
// One launch (of up to MAX_PER_LAUNCH instances), whatever the instances need: a second one with room for wider windows,
// for the instances the first one could not solve, took 4.5 us to find that there are
// none (of 24 at 16384 x 8, 55 at 86400 x 6); windows wider than the LDS of a full
// compute unit allows have their rows in HBM instead.
template <typename K>
hipError_t launch_per_instance(const themis_problem_t& p, const Layout& L, CostArgs& a,
                               hipStream_t st, bool listed, K kernel, int waves = 1)
{
    const int cus = compute_units();
    const int grid = listed && L.N > SHARED_PER_CU * cus ? SHARED_PER_CU * cus : L.N;
    const LdsPlan lds = lds_plan(L.S, L.S * p.r_max * p.c_max, grid, waves, cus);
    a.window = lds.window;
    a.lds_words = lds.words;
    // rows in HBM: S + 1 of them, and the table of a model still in LDS
    const int fit = a.hrow_stride / (L.S + 1) - 2;
    const int room = lds.words - cost_lds(L.S, a.window).tab;
    a.window_hbm = (fit < room ? fit : room) & ~63;
    a.wave_words = waves > 1 ? (uint32_t)(lds.words + WAVE_FLAGS) : 0u;
    const CostKernel k = kernel(a.width);
    hipError_t e = hipSuccess;
    if (lds.bytes > LDS_UNASKED)
        e = hipFuncSetAttribute(reinterpret_cast<const void*>(k), hipFuncAttributeMaxDynamicSharedMemorySize, LDS_MOST);
    in_launches(grid, [&](int first, int count) {
        if (e != hipSuccess) return;
        const dim3 groups((unsigned)count), lanes(64 * waves);
        if (first == 0)
            hipLaunchKernelGGL(k, groups, lanes, lds.bytes, st, a);
        else
            hipLaunchKernelGGL(k, groups, lanes, lds.bytes, st, past(a, (size_t)first));
        e = hipGetLastError();
    });
    return e;
}

}  // namespace
}  // namespace themis
