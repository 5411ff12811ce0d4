// The entry points that solve an instance more than once, each with all of an
// instance's solves in one launch (cost_solver.h), one after the other but for kc_stability:
//
//   kc_fallback   Algorithm 1 with its fallback (Section 4.4): whether the replicas given
//                 can meet the SLO at lambda; where they cannot, the binary search on the
//                 rate; the vertical solve at lambda or the rate found, and the horizontal
//                 solve of the rest with the cores just chosen.
//   kc_stability  the stability test of Section 5.1.3: the horizontal solve at the
//                 current and, where the rate differs, at the predicted rate, and whether
//                 the configurations agree; by a wavefront each where the batch leaves
//                 room for that, else (where the first succeeds) one after the other.
//
// The search needs no recurrence: a configuration within the budget exists exactly
// when the fastest feasible candidates of all models fit it together, and with the
// replicas given the fastest candidate of a (model, batch size) is the one at the
// core cap, since a candidate's latency never grows with the cores.  So a midpoint is
// one evaluation per lane, a minimum per model and a sum.
//
// What bounds them is what bounds a single solve.  As passes over all instances with
// the search by one thread per instance (170 us of it at 16384 x 8) and a compare
// kernel around one-wavefront solves, eight launches and three, they took 250 and 28 us
// at 16384 x 8 and 4099 x 5; as one launch each 65 and 23, with a solve at lambda ahead of
// the search, an evaluation from the start for each of its midpoints and some sixty registers
// spilled; now 27 and 12.  Pipelines of more than 64 models still go the other way, over the
// three stages.
#include "cost_front.h"

namespace themis {
namespace {

// (Every solve starts from the arguments again: what could be kept of them from one to the
// next, and over the calls behind it, would cost registers that the steps need.)
template <int QUEUE, int WIDTH>
__device__ __forceinline__ void fallback_instance(ArgsPtr args, int i)
{
    const int32_t lambda = constant(args->lambda)[i];
    int32_t rate = lambda;  // what the running replicas are solved at
    int status;
    {
        Front<QUEUE, false, WIDTH, QUIET> sv(args);
        bool valid;
        auto first = sv.begin(i, lambda, valid);
        // Whether they can carry lambda is asked before anything is solved for it: it takes a
        // third of what step A does, which then is taken at one rate only.
        if (valid && sv.is_small()) {
            if (sv.template fastest_ticks<true>(first) > (uint32_t)sv.T) {
                sv.lam = rate = sv.template search_rate<true>(first);
                first = sv.at_rate(first);
            }
        } else if (valid) {
            rate = rate_of_large<QUEUE>((uint64_t)(uintptr_t)args, i, sv.T, lambda, sv.slo);
            sv.lam = rate = __builtin_amdgcn_readfirstlane(rate);
            first = sv.at_rate(first);
        }
        status = sv.finish(sv.solve(first, valid));
    }
    const bool solved = status == THEMIS_SOLVED;
    args = Front<QUEUE, false, WIDTH, QUIET>::afresh(args);
    if (threadIdx.x == 0) args->lambda_v[i] = solved ? rate : 0;

    // new instances for what is left, with the cores of the configuration
    Front<QUEUE, true, WIDTH, PINNED> nw(args);
    wave_lds_fence();  // (other lanes wrote what a lane reads here)
    const int32_t rest = solved ? lambda - rate : 0;
    nw.i = i;
    if (nw.lane < nw.a.S) {
        // what put_row() left there
        const uint32_t k = nw.lds[nw.L.pin + nw.lane] & ((1u << INDEX_BITS) - 1u);
        nw.lds[nw.L.pin + nw.lane] = solved ? index_quotient(k, nw.a.magic) + 1u : 1u;
    }
    wave_lds_fence();
    if (rest == 0) {
        // nothing to solve; for calls that look at the workspace afterwards the instance
        // is one that the last solve was not given
        nw.put_none(solved ? THEMIS_SOLVED : THEMIS_INVALID, solved ? 0 : -1);
        if (nw.lane == 0) nw.a.tmeta[i] = -1;
        return;
    }
    bool valid;
    const auto first = nw.begin(i, rest, valid);
    nw.finish(nw.solve(first, valid));
}

template <int QUEUE, int WIDTH>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(6, 6))) void kc_fallback(CostArgs)
{
    const ArgsPtr args = kernel_args();
    fallback_instance<QUEUE, WIDTH>(args, (int)blockIdx.x);
    mark_workspace(Front<QUEUE, false, WIDTH>::afresh(args), STATE_KEPT | STATE_ONLY);
}

template <int QUEUE, int WIDTH>
__device__ __forceinline__ void stability_instance(ArgsPtr args, int i)
{
    const int32_t now = constant(args->lambda)[i], pred = constant(args->lambda2)[i];
    bool stable = solve_instance<QUEUE, true, WIDTH, PLAIN>(args, i, args->lambda) == THEMIS_SOLVED;
    wave_lds_fence();
    args = Front<QUEUE, true, WIDTH>::afresh(args);
    if (stable && pred != now) {
        stable = solve_instance<QUEUE, true, WIDTH, SECOND>(args, i, args->lambda2) == THEMIS_SOLVED;
        args = Front<QUEUE, true, WIDTH>::afresh(args);
        if (stable) {
            wave_lds_fence();
            const CostLds L = cost_lds(args->S, args->window, args->lds_words);
            // what put_row() made of the choices of both
            const bool same =
                (int)threadIdx.x >= args->S || cost_smem[L.pin + threadIdx.x] == SAME;
            stable = __ballot(!same) == 0ull;
        }
    }
    if (threadIdx.x == 0) args->stable[i] = stable ? 1 : 0;
}

// The same with a wavefront for each of the two rates.  Two barriers each: the first one's first
// is when its solve is done, the second one's before it uses the instance's rows in HBM or, if
// it has no use for them, after its solve; then both have their results.  A first one without a
// solution says so ahead of its barrier, for the second to end its solve early (in_vain()).
template <int QUEUE, int WIDTH>
__device__ __forceinline__ void stability_pair(ArgsPtr args, int i)
{
    const uint32_t lane = threadIdx.x & 63u;
    const bool later = wave_number() == 1u;
    const bool moves = constant(args->lambda)[i] != constant(args->lambda2)[i];
    int status = THEMIS_SOLVED;
    if (!later) {
        status = solve_instance<QUEUE, true, WIDTH, PLAIN>(args, i, args->lambda, (int)lane);
        if (status != THEMIS_SOLVED) {
            // (where that is before the other one has made its words ready, it isn't told)
            args = Front<QUEUE, true, WIDTH>::afresh(args);
            const CostLds L = cost_lds(args->S, args->window, args->lds_words);
            if (lane == 0u)
                __hip_atomic_store(cost_smem + args->wave_words + L.words + 1, 1u, __ATOMIC_RELAXED,
                                   __HIP_MEMORY_SCOPE_WORKGROUP);
        }
        __syncthreads();
    } else {
        {
            const CostLds L = cost_lds(args->S, args->window, args->lds_words);
            uint32_t* const mine = cost_smem + args->wave_words;
            // (there is no choice of a solve before for put_row() to find)
            if (lane < (uint32_t)args->S) mine[L.pin + lane] = SAME;
            if (lane < 2u) mine[L.words + lane] = 0u;
            wave_lds_fence();
        }
        if (moves)
            status = solve_instance<QUEUE, true, WIDTH, SECOND>(args, i, args->lambda2, (int)lane,
                                                                args->wave_words);
        args = Front<QUEUE, true, WIDTH>::afresh(args);
        const CostLds L = cost_lds(args->S, args->window, args->lds_words);
        uint32_t* const mine = cost_smem + args->wave_words;
        wave_lds_fence();
        if (__builtin_amdgcn_readfirstlane((int)mine[L.words]) == 0) __syncthreads();
        if (lane == 0u) mine[L.words] = status == THEMIS_SOLVED ? 1u : 0u;
    }
    __syncthreads();
    if (later) return;
    args = Front<QUEUE, true, WIDTH>::afresh(args);
    const CostLds L = cost_lds(args->S, args->window, args->lds_words);
    // what put_row() left of the choices of both
    const uint32_t *const first = cost_smem, *const second = cost_smem + args->wave_words;
    const bool same = !moves || lane >= (uint32_t)args->S || first[L.pin + lane] == second[L.pin + lane];
    const bool stable = status == THEMIS_SOLVED && second[L.words] && __ballot(!same) == 0ull;
    if (lane == 0u) args->stable[i] = stable ? 1 : 0;
}

// TWO: a workgroup of two wavefronts per instance.
template <int QUEUE, int WIDTH, bool TWO>
__global__ __launch_bounds__(TWO ? 128 : 64) __attribute__((amdgpu_waves_per_eu(6, 6))) void kc_stability(CostArgs)
{
    const ArgsPtr args = kernel_args();
    if (TWO)
        stability_pair<QUEUE, WIDTH>(args, (int)blockIdx.x);
    else
        stability_instance<QUEUE, WIDTH>(args, (int)blockIdx.x);
    mark_workspace(args, STATE_KEPT | (args->c_fixed ? STATE_ONLY : 0) |
                             args->c_all << STATE_C_ALL);
}

template <int QUEUE>
CostKernel fallback_kernel(int width)
{
    switch (width) {
    case WIDTH_PACKED: return &kc_fallback<QUEUE, PACKED>;
    case 4: return &kc_fallback<QUEUE, 4>;
    case 8: return &kc_fallback<QUEUE, 8>;
    case 16: return &kc_fallback<QUEUE, 16>;
    default: return &kc_fallback<QUEUE, TURNS>;
    }
}

template <int QUEUE, bool TWO>
CostKernel stability_kernel(int width)
{
    switch (width) {
    case WIDTH_PACKED: return &kc_stability<QUEUE, PACKED, TWO>;
    case 4: return &kc_stability<QUEUE, 4, TWO>;
    case 8: return &kc_stability<QUEUE, 8, TWO>;
    case 16: return &kc_stability<QUEUE, 16, TWO>;
    default: return &kc_stability<QUEUE, TURNS, TWO>;
    }
}
template <int QUEUE>
CostKernel stability_kernel(int width, bool two)
{
    return two ? stability_kernel<QUEUE, true>(width) : stability_kernel<QUEUE, false>(width);
}

}  // namespace

hipError_t launch_cost_fallback(const themis_problem_t& p, const Layout& L, const int32_t* d_coef,
                                const int32_t* d_lambda, const int32_t* d_slo_us,
                                const int32_t* d_r_fixed, const FallbackOut& out, char* ws,
                                hipStream_t st)
{
    CostArgs a = cost_args(p, L, d_coef, d_lambda, d_slo_us, d_r_fixed, out.status, out.cost,
                           out.ticks, out.cfg, ws, PassOpts(), WORK_FEW);
    a.status2 = out.status_h;
    a.cost2 = out.cost_h;
    a.ticks2 = out.ticks_h;
    a.cfg2 = out.cfg_h;
    a.lambda_v = out.lambda_v;
    return launch_per_instance(p, L, a, st, false, [&](int width) {
        switch (p.queue_model) {
        case THEMIS_QUEUE_SHARED: return fallback_kernel<THEMIS_QUEUE_SHARED>(width);
        case THEMIS_QUEUE_WORST_CASE: return fallback_kernel<THEMIS_QUEUE_WORST_CASE>(width);
        default: return fallback_kernel<THEMIS_QUEUE_PER_REPLICA>(width);
        }
    });
}

hipError_t launch_cost_stability(const themis_problem_t& p, const Layout& L,
                                 const StabilityLayout& B, const int32_t* d_coef,
                                 const int32_t* d_lambda_now, const int32_t* d_lambda_pred,
                                 const int32_t* d_slo_us, int32_t* d_stable, int32_t* d_status,
                                 int32_t* d_cost, int32_t* d_ticks, int32_t* d_cfg, char* ws,
                                 hipStream_t st, const PassOpts& opts)
{
    CostArgs a = cost_args(p, L, d_coef, d_lambda_now, d_slo_us, nullptr, d_status, d_cost, d_ticks,
                           d_cfg, ws, opts, WORK_FEW);
    a.lambda2 = d_lambda_pred;
    a.stable = d_stable;
    a.status2 = (int32_t*)(ws + B.status_off);
    a.cost2 = (int32_t*)(ws + B.cost_off);
    a.ticks2 = (int32_t*)(ws + B.ticks_off);
    a.cfg2 = (int32_t*)(ws + B.cfg_off);
    const bool two = stability_in_pairs(L.S, L.N, compute_units());
    return launch_per_instance(p, L, a, st, false, [&](int width) {
        switch (p.queue_model) {
        case THEMIS_QUEUE_SHARED: return stability_kernel<THEMIS_QUEUE_SHARED>(width, two);
        case THEMIS_QUEUE_WORST_CASE: return stability_kernel<THEMIS_QUEUE_WORST_CASE>(width, two);
        default: return stability_kernel<THEMIS_QUEUE_PER_REPLICA>(width, two);
        }
    }, two ? 2 : 1);
}

}  // namespace themis
