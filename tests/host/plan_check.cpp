// Host-side check of how the one-wavefront solve lies in lanes.  Built and run by
// tests/test_host_plan.py (no GPU needed).  The properties are stated from what the kernels do
// with the layout, not from the formulas under test:
//   every (model, batch size) pair is taken once, by a lane of the wavefront;
//   where there are more pairs than lanes, no more of them one after the other than whole
//   models side by side would take, with or without gaps between them.
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

static void check_lanes(int S, int nb)
{
    const FrontLayout f = front_layout(S, nb);
    for (int spread = 0; spread < 2; ++spread) {
        std::vector<int> taken(S * nb, 0);
        int steps = 0;
        auto take = [&](int s, int j) {
            if (s < S && j < nb) ++taken[s * nb + j];
        };
        if (f.width == WIDTH_TURNS) {
            steps = f.turns;
            CHECK(f.width_log < 0 || f.lanes == 1 << f.width_log, "%d x %d", S, nb);
            CHECK(f.lanes > 1, "%d x %d", S, nb);
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
        CHECK(steps <= (with_gaps < without ? with_gaps : without), "%d x %d, width %d: %d steps", S, nb,
              f.width, steps);
    }
    // what is sought per model goes by these in code shared between the layouts
    CHECK(f.lanes >= 1 && f.turns * f.lanes >= nb && S * f.lanes <= 64, "%d x %d", S, nb);
}

int main()
{
    for (int S = 1; S <= 64; ++S)
        for (int nb = 1; nb <= 16; ++nb) check_lanes(S, nb);
    if (failures) {
        std::printf("%d failures\n", failures);
        return 1;
    }
    std::printf("plan ok\n");
    return 0;
}
