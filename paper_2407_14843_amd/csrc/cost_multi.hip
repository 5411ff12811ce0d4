// The entry points that solve an instance more than once, each with all of an
// instance's solves in one wavefront (cost_solver.h), one after the other:
//
//   kc_fallback   Algorithm 1 with its fallback (Section 4.4): the vertical solve at
//                 lambda; where the replicas given cannot meet the SLO, the binary
//                 search on the rate, the vertical solve at the rate it settles on, and
//                 the horizontal solve of the rest with the cores just chosen.
//   kc_stability  the stability test of Section 5.1.3: the horizontal solve at the
//                 current and, where that succeeds and the rate differs, at the
//                 predicted rate, and whether the configurations agree.
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
// at 16384 x 8 and 4099 x 5; now one launch each, 62 and 23.  Pipelines of more than 64
// models still go that way, over the three stages.
#include "cost_solver.h"

namespace themis {
namespace {

// The largest rate the search finds; `first`: the pair at lambda, which is infeasible.
template <int QUEUE, bool ONE, bool SMALL>
__device__ __forceinline__ int32_t search_rate(Solver<QUEUE, false, ONE, QUIET>& sv,
                                               const typename Solver<QUEUE, false, ONE, QUIET>::Pair& first)
{
    int32_t lo = 1, hi = sv.lam;
    while (hi - lo > 1) {
        const int32_t mid = lo + ((hi - lo) >> 1);
        sv.lam = mid;
        const bool fits = sv.template fastest_ticks<SMALL>(sv.at_rate(first)) <= (uint32_t)sv.T;
        if (fits)
            lo = mid;
        else
            hi = mid;
    }
    return lo;
}

template <int QUEUE, bool ONE>
__device__ __forceinline__ void fallback_instance(ArgsPtr args, int i)
{
    Solver<QUEUE, false, ONE, QUIET> sv(args);
    const int32_t lambda = args->lambda[i];
    int32_t rate = lambda;  // what the running replicas are solved at
    int status;
    {
        bool valid;
        auto first = sv.begin(i, lambda, valid);
        status = valid ? THEMIS_INFEASIBLE : THEMIS_INVALID;
        for (bool searched = false; valid; searched = true) {
            status = sv.solve(first);
            if (searched || status != THEMIS_INFEASIBLE) break;
            // (lambda is the largest rate met, so the short divisions stay allowed)
            if (__builtin_amdgcn_readfirstlane((int)((double)lambda * (double)sv.slo <= 0x1p42)))
                rate = search_rate<QUEUE, ONE, true>(sv, first);
            else
                rate = search_rate<QUEUE, ONE, false>(sv, first);
            sv.lam = rate;
            first = sv.at_rate(first);
        }
    }
    const bool solved = status == THEMIS_SOLVED;
    if (!solved) sv.put_none(status);
    if (sv.lane == 0) args->lambda_v[i] = solved ? rate : 0;

    // new instances for what is left, with the cores of the configuration
    Solver<QUEUE, true, ONE, PINNED> nw(args);
    const int32_t rest = solved ? lambda - rate : 0;
    nw.i = i;
    if (nw.lane < nw.a.S) {
        // (this lane wrote the configuration's row)
        const int32_t c = solved ? (sv.config() + 3 * nw.lane)[0] : 1;
        nw.lds[nw.L.pin + nw.lane] = (uint32_t)c;
    }
    wave_lds_fence();
    if (rest == 0) {
        // nothing to solve; for calls that look at the workspace afterwards the instance
        // is one that the last solve was not given
        nw.put_none(solved ? THEMIS_SOLVED : THEMIS_INVALID, solved ? 0 : -1);
        if (nw.lane == 0) args->tmeta[i] = -1;
        return;
    }
    bool valid;
    const auto first = nw.begin(i, rest, valid);
    if (nw.solve(first) == THEMIS_INFEASIBLE) nw.put_none(THEMIS_INFEASIBLE);
}

template <int QUEUE, bool ONE>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(6, 8))) void kc_fallback(CostArgs)
{
    const ArgsPtr args = kernel_args();
    mark_workspace(args, STATE_KEPT | STATE_ONLY);
    fallback_instance<QUEUE, ONE>(args, (int)blockIdx.x);
}

template <int QUEUE, bool ONE>
__device__ __forceinline__ void stability_instance(ArgsPtr args, int i)
{
    const int32_t now = args->lambda[i], pred = args->lambda2[i];
    bool stable = solve_instance<QUEUE, true, ONE, PLAIN>(args, i, now) == THEMIS_SOLVED;
    wave_lds_fence();
    if (stable && pred != now) {
        stable = solve_instance<QUEUE, true, ONE, SECOND>(args, i, pred) == THEMIS_SOLVED;
        if (stable) {
            bool same = true;
            if ((int)threadIdx.x < args->S) {
                // (this lane wrote both rows)
                const size_t at = ((size_t)i * args->S + threadIdx.x) * 3;
                const int32_t *const x = args->cfg + at, *const y = args->cfg2 + at;
                same = x[0] == y[0] && x[1] == y[1] && x[2] == y[2];
            }
            stable = __ballot(!same) == 0ull;
        }
    }
    if (threadIdx.x == 0) args->stable[i] = stable ? 1 : 0;
}

template <int QUEUE, bool ONE>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(8, 8))) void kc_stability(CostArgs)
{
    const ArgsPtr args = kernel_args();
    mark_workspace(args, STATE_KEPT | (args->c_fixed ? STATE_ONLY : 0) |
                             args->c_all << STATE_C_ALL);
    stability_instance<QUEUE, ONE>(args, (int)blockIdx.x);
}

template <int QUEUE>
CostKernel fallback_kernel(bool one)
{
    return one ? &kc_fallback<QUEUE, true> : &kc_fallback<QUEUE, false>;
}

template <int QUEUE>
CostKernel stability_kernel(bool one)
{
    return one ? &kc_stability<QUEUE, true> : &kc_stability<QUEUE, false>;
}

}  // namespace

hipError_t launch_cost_fallback(const themis_problem_t& p, const Layout& L, const int32_t* d_coef,
                                const int32_t* d_lambda, const int32_t* d_slo_us,
                                const int32_t* d_r_fixed, const FallbackOut& out, char* ws,
                                hipStream_t st)
{
    CostArgs a = cost_args(p, L, d_coef, d_lambda, d_slo_us, d_r_fixed, out.status, out.cost,
                           out.ticks, out.cfg, ws, PassOpts());
    a.status2 = out.status_h;
    a.cost2 = out.cost_h;
    a.ticks2 = out.ticks_h;
    a.cfg2 = out.cfg_h;
    a.lambda_v = out.lambda_v;
    return launch_per_instance(p, L, a, st, false, [&](bool one) {
        switch (p.queue_model) {
        case THEMIS_QUEUE_SHARED: return fallback_kernel<THEMIS_QUEUE_SHARED>(one);
        case THEMIS_QUEUE_WORST_CASE: return fallback_kernel<THEMIS_QUEUE_WORST_CASE>(one);
        default: return fallback_kernel<THEMIS_QUEUE_PER_REPLICA>(one);
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
                           d_cfg, ws, opts);
    a.lambda2 = d_lambda_pred;
    a.stable = d_stable;
    a.status2 = (int32_t*)(ws + B.status_off);
    a.cost2 = (int32_t*)(ws + B.cost_off);
    a.ticks2 = (int32_t*)(ws + B.ticks_off);
    a.cfg2 = (int32_t*)(ws + B.cfg_off);
    return launch_per_instance(p, L, a, st, false, [&](bool one) {
        switch (p.queue_model) {
        case THEMIS_QUEUE_SHARED: return stability_kernel<THEMIS_QUEUE_SHARED>(one);
        case THEMIS_QUEUE_WORST_CASE: return stability_kernel<THEMIS_QUEUE_WORST_CASE>(one);
        default: return stability_kernel<THEMIS_QUEUE_PER_REPLICA>(one);
        }
    });
}

}  // namespace themis
