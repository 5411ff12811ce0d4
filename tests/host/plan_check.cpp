// Host-side check of how the one-wavefront solve lies in lanes and in LDS.  Built and run by
// tests/test_host_plan.py (no GPU needed).  The properties are stated from what the kernels do
// with the layout, not from the formulas under test:
//   every (model, batch size) pair is taken once, by a lane of the wavefront;
//   where there are more pairs than lanes, no more of them one after the other than whole
//   models side by side would take, with or without gaps between them, if there is a choice
//   among many candidates, or the lane has no other's to go by;
//   what step C has in LDS at one time lies apart and inside the wavefront's words, and takes
//   no more of them than its table, rows and the copy of one, or below 16 models 32 more;
//   the lists of step G have room for fourteen candidates of a model;
//   a launch asks for what its wavefronts have, with room for those that a compute unit has at a
//   time, and for all of what that leaves each of them.
#include <cstdio>
#include <vector>

#include "cost_plan.h"

using namespace themis;

static int failures = 0;
#define CHECK(cond, ...)                                  \
    do {                                                  \
        if (!(cond)) {                                    \
            if (failures < 20) {                          \
                std::printf("FAIL %s: ", #cond);          \
                std::printf(__VA_ARGS__);                 \
                std::printf("\n");                        \
            }                                             \
            ++failures;                                   \
        }                                                 \
    } while (0)

static int up(int a, int b) { return (a + b - 1) / b; }

static void check_lanes(int S, int nb, FrontWork work)
{
    const FrontLayout f = front_layout(S, nb, work);
    for (int spread = 0; spread < 2; ++spread) {
        std::vector<int> taken(S * nb, 0);
        int steps = 0;
        auto take = [&](int s, int j) {
            if (s < S && j < nb) ++taken[s * nb + j];
        };
        if (f.width == WIDTH_TURNS) {
            steps = f.turns;
            CHECK(f.width_log < 0 || f.lanes == 1 << f.width_log, "%d x %d", S, nb);
            for (int lane = 0; lane < 64; ++lane)
                for (int t = 0; t < f.turns; ++t) {
                    const int part = lane % f.lanes;
                    take(lane / f.lanes, spread ? part * f.turns + t : part + t * f.lanes);
                }
            CHECK(S * f.lanes <= 64, "%d x %d", S, nb);
        } else if (f.width == WIDTH_ROUNDS) {
            const int width = f.round_log < 0 ? nb : 1 << f.round_log;
            CHECK(f.per_round >= 1 && f.per_round * width <= 64 && nb <= width, "%d x %d", S, nb);
            for (int s0 = 0; s0 < S; s0 += f.per_round, ++steps)
                for (int lane = 0; lane < 64; ++lane)
                    if (lane / width < f.per_round) take(s0 + lane / width, lane % width);
        } else {
            const int width = f.width == WIDTH_PACKED ? nb : f.width;
            steps = 1;
            CHECK(f.turns == 1, "%d x %d", S, nb);
            CHECK(f.width == WIDTH_PACKED || f.width == 4 || f.width == 8 || f.width == 16, "%d x %d", S, nb);
            for (int lane = 0; lane < 64; ++lane) take(lane / width, lane % width);
        }
        for (int t : taken) CHECK(t == 1, "%d x %d, width %d: taken %d times", S, nb, f.width, t);
        int width = S <= 16 ? 4 : 1;
        while (width < nb) width *= 2;
        const int with_gaps = up(S, 64 / width), without = up(S, 64 / nb);
        const int rounds = with_gaps < without ? with_gaps : without;
        // where the pairs' candidates count, or a lane has the model to itself
        if (work == WORK_DERIVED || (work == WORK_GIVEN && f.lanes == 1))
            CHECK(steps <= rounds, "%d x %d, width %d: %d steps", S, nb, f.width, steps);
        if (work == WORK_DERIVED && f.width == WIDTH_TURNS && f.lanes == 1)
            CHECK(steps < rounds, "%d x %d: %d steps", S, nb, steps);
        // and else turns
        if (work == WORK_FEW || (work == WORK_GIVEN && f.lanes > 1))
            CHECK(f.width != WIDTH_ROUNDS, "%d x %d, width %d", S, nb, f.width);
    }
    // what is sought per model goes by these in code shared between the layouts
    CHECK(f.lanes >= 1 && f.turns * f.lanes >= nb && S * f.lanes <= 64, "%d x %d", S, nb);
}

static void check_step_c(int S)
{
    const CostLds l = cost_lds(S, 64);
    const int least = l.least;
    const StepCLds c = step_c_lds(S, l.tab);
    std::vector<int> owner(least + 64, 0);
    auto own = [&](int first, int words) {
        CHECK(first >= 0 && first + words <= least, "%d models: %d words from %d of %d", S, words, first, least);
        for (int x = first; x < first + words && x < (int)owner.size(); ++x) CHECK(++owner[x] == 1, "%d models: word %d", S, x);
    };
    own(l.key, S), own(l.fast, S), own(l.pin, S);
    own(l.tab, 64 * S);
    own(c.rows, 32 * S);
    own(c.even, 32), own(c.odd, 32);
    own(c.copy - 32, 64);
    // read four words at a time
    CHECK(c.rows % 4 == 0 && c.even % 4 == 0 && c.odd % 4 == 0 && least % 4 == 0, "%d models", S);
    // the row of nothing left to run is behind the others, and nothing else is in it by then
    CHECK(c.rows + 32 * S + 32 <= least && (c.odd < c.rows || c.odd >= c.rows + 32 * (S + 1)), "%d models", S);
    CHECK(least <= l.tab + 64 * S + 32 * (S + 1) + 64 + (S < 16 ? 32 : 0), "%d models: %d words", S, least);
}

static void check_launch(int S, int spread, int groups, int waves)
{
    const LdsPlan p = lds_plan(S, spread, groups, waves, 256);
    const CostLds l = cost_lds(S, p.window);
    const int flags = waves > 1 ? WAVE_FLAGS : 0, all = 4 * waves * (p.words + flags);
    CHECK(p.window >= 64 && p.window % 64 == 0, "%d models, %d groups", S, groups);
    CHECK(p.words >= l.least && (p.words + flags) % 4 == 0, "%d models, %d groups", S, groups);
    CHECK(p.words - l.tab - 67 * S - 2 >= 2 * 14 * S, "%d models, %d groups: %d words", S, groups, p.words);
    CHECK(all == p.bytes, "%d models, %d groups: %d of %d", S, groups, all, p.bytes);
    // A compute unit has room for the workgroups that it has at a time, or, if that is less, for
    // as many as with the least request (LDS is granted by 1280 bytes).
    auto resident = [](int bytes) { return 128 / ((bytes + 1279) / 1280); };
    const int mean = (groups + 255) / 256, most = 25 / waves;
    const int wanted = mean < 4 / waves ? 4 / waves : mean > most ? most : mean;
    const int by_least = resident(4 * waves * (cost_lds(S, 64).least + flags));
    const int room = wanted < by_least ? wanted : by_least;
    CHECK(resident(p.bytes) >= room, "%d models, %d groups of %d: %d for %d", S, groups, waves, resident(p.bytes), room);
    // and, where all can be resident and the window doesn't hold all that a pipeline's costs
    // can spread over, what is granted is in use, and no more could be
    if (p.window < spread && mean <= most && (S > 16 || p.bytes + 1280 <= 64 * 1024)) {
        const int granted = 128 / resident(p.bytes) * 1280;
        CHECK(granted - p.bytes < 16 * waves, "%d models, %d groups of %d: %d of %d", S, groups, waves, p.bytes, granted);
        CHECK(resident(granted + 1280) < room || resident(p.bytes) == by_least, "%d models, %d groups of %d: %d",
              S, groups, waves, p.bytes);
    }
    // what a kernel may have without an attribute set, or two wavefronts of many models with it
    CHECK(p.bytes <= (waves == 2 && S > 16 ? LDS_MOST : 64 * 1024), "%d models, %d groups of %d", S, groups, waves);
}

int main()
{
    for (int S = 1; S <= 64; ++S)
        for (int waves = 1; waves <= 2; ++waves)
            for (int groups : {1, 255, 256, 257, 512, 1024, 3001, 4099, 7168, 86400})
                for (int spread : {1, 100, 32767}) check_launch(S, spread, groups, waves);
    for (int S = 1; S <= 64; ++S) check_step_c(S);
    for (int S = 1; S <= 64; ++S)
        for (int nb = 1; nb <= 16; ++nb)
            for (FrontWork work : {WORK_DERIVED, WORK_GIVEN, WORK_FEW}) check_lanes(S, nb, work);
    if (failures) {
        std::printf("%d failures\n", failures);
        return 1;
    }
    std::printf("plan ok\n");
    return 0;
}
