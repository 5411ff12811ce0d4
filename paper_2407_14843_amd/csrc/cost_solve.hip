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
//   A  input check, budget; base[s], with the least (lt, index) at that cost.
//      Lane = (model, batch size); a lane evaluates the first core count that can be
//      feasible, and of the others those that can cost as little as the model's best.
//      When these candidates fit the budget together, x* = 0 and they are the answer.
//   F  else the fastest candidate of every (model, batch size), which is the one at
//      the core cap (latency never grows with the cores): the instance is infeasible
//      exactly when the fastest candidates of all models together exceed the budget.
//   B  else the recurrence over the first 8 or 16 cells: one table of (lt, index) by
//      model and cost over base in LDS, lane = (model, cell), rows of neighbouring models
//      combined in turns.  How late the candidates of step A are says which it takes.
//   C  else over 64 cells, rows in LDS, lane = two cells, the halves of the wavefront for the even
//      and the odd costs over base;
//   G  else lists of the candidates (of all, or where those do not fit of those that
//      Lagrangian bounds leave), those that the bounds show to be in no answer dropped, and
//      every combination of what is left, a few candidates per model; or the recurrence
//      over them, if there are many combinations and their costs span few cells;
//   W  else (a list too long even so, one instance in thousands of the densest) the
//      recurrence over wider windows, with the table of one model at a time and the rows
//      in LDS, then in HBM; and past that
//   D  the recurrence over the budget with rows in HBM, which is bounded by T
//      whatever the costs are.
//
// What bounds it: vector issue.  An instance is some hundreds of instructions,
// mostly the double-precision evaluation of candidates (candidate_eval.h, shared
// with the candidate tables and the rate search, so that all agree bit for bit),
// against 0.3 KB of inputs and outputs; nothing but those touches HBM.  Whole solves
// by the three stages (dense / with dominated candidates pruned) against this one, in
// microseconds: 65536 x 8 models 25800 / 3880 -> 72, 16384 x 8 with replicas given
// 3370 -> 20, 86400 x 6 2790 -> 39, 4096 x 5 177 -> 10.0, 64 x 3 27.2 -> 6.3.
#include "cost_front.h"

namespace themis {
namespace {

// LISTED: the instances of a list, each workgroup some of them; else one per workgroup.
// Seven wavefronts per SIMD, as LDS has room for: eight, with 64 registers, have to spill in the
// steps that every instance takes (86400 x 6: 52 us instead of 42; six: 43.5).
template <int QUEUE, bool DERIVE, int WIDTH, bool LISTED>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(7, 7))) void kc_solve(CostArgs)
{
    const ArgsPtr args = kernel_args();
    auto mark = [](ArgsPtr p) {
        p = Front<QUEUE, DERIVE, WIDTH>::afresh(p);
        mark_workspace(p, STATE_KEPT | (DERIVE ? 0 : STATE_GIVEN) | (p->c_fixed ? STATE_ONLY : 0) |
                              p->c_all << STATE_C_ALL);
    };
    if (!LISTED) {
        const int i = (int)blockIdx.x;
        solve_instance<QUEUE, DERIVE, WIDTH, PLAIN>(args, i, args->lambda);
        mark(args);
        return;
    }
    const int n = args->ctrl[LIST_WORD];
    for (int k = (int)blockIdx.x; k < n; k += (int)gridDim.x) {
        // every instance starts from the arguments and the lane's number again: what could
        // be kept of them from one to the next would cost registers that the steps need
        ArgsPtr again = args;
        int lane = (int)threadIdx.x;
        asm volatile("" : "+s"(again), "+v"(lane));
        const int i = __builtin_amdgcn_readfirstlane(again->list[k]);
        solve_instance<QUEUE, DERIVE, WIDTH, PLAIN>(again, i, again->lambda, lane);
        wave_lds_fence();
    }
    mark(args);
}

template <int QUEUE, bool DERIVE, bool LISTED>
CostKernel solve_kernel(int width)
{
    switch (width) {
    case WIDTH_PACKED: return &kc_solve<QUEUE, DERIVE, PACKED, LISTED>;
    case WIDTH_ROUNDS: return &kc_solve<QUEUE, DERIVE, ROUNDS, LISTED>;
    case 4: return &kc_solve<QUEUE, DERIVE, 4, LISTED>;
    case 8: return &kc_solve<QUEUE, DERIVE, 8, LISTED>;
    case 16: return &kc_solve<QUEUE, DERIVE, 16, LISTED>;
    default: return &kc_solve<QUEUE, DERIVE, TURNS, LISTED>;
    }
}

template <int QUEUE, bool DERIVE>
CostKernel solve_kernel(bool listed, int width)
{
    return listed ? solve_kernel<QUEUE, DERIVE, true>(width) : solve_kernel<QUEUE, DERIVE, false>(width);
}

}  // namespace

bool cost_solve_serves(const Layout& L) { return L.S <= COST_MAX_STAGES; }
bool cost_solve_side_by_side(const Layout& L)
{
    return cost_solve_serves(L) && L.N <= SIMDS_PER_CU * compute_units();
}

hipError_t launch_cost_solve(const themis_problem_t& p, const Layout& L, const int32_t* d_coef,
                             const int32_t* d_lambda, const int32_t* d_slo_us,
                             const int32_t* d_r_fixed, int32_t* d_status, int32_t* d_cost,
                             int32_t* d_ticks, int32_t* d_cfg, char* ws, hipStream_t st,
                             const PassOpts& opts)
{
    CostArgs a = cost_args(p, L, d_coef, d_lambda, d_slo_us, d_r_fixed, d_status, d_cost, d_ticks,
                           d_cfg, ws, opts,
                           d_r_fixed                                           ? WORK_GIVEN
                           : opts.c_fixed || opts.c_all > 0 || p.c_max == 1 ? WORK_FEW
                                                                               : WORK_DERIVED);
    const bool listed = opts.list != nullptr;
    return launch_per_instance(p, L, a, st, listed, [&](int width) {
        switch (p.queue_model) {
        case THEMIS_QUEUE_SHARED:
            return d_r_fixed ? solve_kernel<THEMIS_QUEUE_SHARED, false>(listed, width)
                             : solve_kernel<THEMIS_QUEUE_SHARED, true>(listed, width);
        case THEMIS_QUEUE_WORST_CASE:
            return d_r_fixed ? solve_kernel<THEMIS_QUEUE_WORST_CASE, false>(listed, width)
                             : solve_kernel<THEMIS_QUEUE_WORST_CASE, true>(listed, width);
        default:
            return d_r_fixed ? solve_kernel<THEMIS_QUEUE_PER_REPLICA, false>(listed, width)
                             : solve_kernel<THEMIS_QUEUE_PER_REPLICA, true>(listed, width);
        }
    });
}

}  // namespace themis
