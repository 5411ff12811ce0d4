// How the one-wavefront solve lies in lanes: host arithmetic that its launches follow
// (cost_solver.h).
#pragma once

namespace themis {

// Ways the (model, batch size) pairs lie in a wavefront besides 4, 8 or 16 lanes per model,
// see Front (cost_front.h).
constexpr int WIDTH_TURNS = 0, WIDTH_PACKED = 1, WIDTH_ROUNDS = 2;

struct FrontLayout {
    int width;                   // 4, 8, 16 or WIDTH_..
    int width_log;               // of the lanes per model, below zero: without gaps
    int lanes, turns;            // lanes per model, and the batch sizes of each
    int round_log, per_round;    // the same of a round of whole models, and the models of one
};

// Lanes per model: a power of two, or where that takes more turns (or doesn't fit) as many as
// there are batch sizes or all models leave room for (9 x 14: seven and two turns, not four
// and four).
//
// Where there are more pairs than lanes: in turns if that takes no more of them than whole models
// take rounds, with two lanes per model or more.  Turns leave lanes idle where the models don't
// divide the wavefront: 12 x 16 in four turns 39.3 us, in three rounds 34.1 (7000 pipelines);
// 22 x 16, eight and six: 87.1 and 73.8; 300 x 33 x 16, sixteen and nine: 112 and 69.  A single
// lane per model has no other's candidates to go by: 300 x 63 x 3, three of either, 10.8 and
// 8.4.  With as many of either, and two lanes, turns take 0.84 to 0.99 of the time in the mean
// of a shape.
inline FrontLayout front_layout(int S, int n_batch)
{
    FrontLayout f{};
    while (1 << f.width_log < n_batch) ++f.width_log;
    if (f.width_log < 2 && S <= 16) f.width_log = 2;
    f.round_log = f.width_log;
    f.per_round = 64 >> f.round_log;
    auto rounds = [&](int models) { return (S + models - 1) / models; };
    if (rounds(64 / n_batch) < rounds(f.per_round)) f.per_round = 64 / n_batch, f.round_log = -1;
    while (S << f.width_log > 64) --f.width_log;
    f.lanes = 1 << f.width_log;
    const int fit = 64 / S < n_batch ? 64 / S : n_batch;
    auto turns = [&](int lanes) { return (n_batch + lanes - 1) / lanes; };
    if (turns(fit) < turns(f.lanes)) f.lanes = fit, f.width_log = -1;
    f.turns = turns(f.lanes);
    if (f.turns > 1)
        f.width = f.lanes > 1 && f.turns <= rounds(f.per_round) ? WIDTH_TURNS : WIDTH_ROUNDS;
    else
        f.width = f.width_log >= 2 ? 1 << f.width_log : WIDTH_PACKED;
    return f;
}

}  // namespace themis
