// How the one-wavefront solve lies in lanes and in LDS: whole-number arithmetic that its launches
// and its kernels follow (cost_solver.h).
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

// What is sought of a (model, batch size) pair: of many candidates with the replicas derived, of
// those with the replicas given, or of one (one core count), or that of the fallback besides.
enum FrontWork { WORK_DERIVED, WORK_GIVEN, WORK_FEW };

// Lanes per model: a power of two, or where that takes more turns (or doesn't fit) as many as
// there are batch sizes or all models leave room for (9 x 14: seven and two turns, not four
// and four).
//
// Where there are more pairs than lanes: in turns, but where they leave lanes idle that whole models
// in rounds put to use, as the models don't divide the wavefront, and what the pairs still have
// to do then counts.  Turns against rounds in the time of 150 shapes of 11 to 64 models, at 300
// and 7000 pipelines: derived with as few turns as rounds 0.85 to 1.05 (mean 0.97), with more 1.02
// to 1.50 (12 x 16 1.09, 33 x 16 1.47), and as many of either but a single lane per model, which
// has no other's candidates to go by, 0.97 to 1.11; given 0.77 to 1.02, but with more turns and a
// single lane 0.93 to 1.20; one candidate 0.81 to 1.00; fallback 0.65 to 1.00.
inline FrontLayout front_layout(int S, int n_batch, FrontWork work)
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
    const int most = rounds(f.per_round);
    const bool fewer = work == WORK_DERIVED ? f.turns < most + (f.lanes > 1)
                       : work == WORK_GIVEN ? f.turns <= most || f.lanes > 1
                                            : true;
    if (f.turns > 1)
        f.width = fewer ? WIDTH_TURNS : WIDTH_ROUNDS;
    else
        f.width = f.width_log >= 2 ? 1 << f.width_log : WIDTH_PACKED;
    return f;
}

// LDS words of one wavefront, of which there are `words` (at least `least`).  From `tab` on, steps
// B and C take a table of up to 64 words per model and S + 1 rows: of eight 32-bit cells behind as
// many guard cells, of sixteen without, or of 64 16-bit cells (see StepCLds); wider windows a
// table of one model and 16-bit rows with a guard cell (and one of padding) in front of each;
// step G lists as long as there are words.
struct CostLds {
    int best, key, fast, pin, tab, rows, least, words;
};
// Step C: rows of 32 words, the last one that of nothing left to run; a model's latencies at
// even and at odd costs, 32 words each; a copy of the row at hand behind 32 guard words.  Of
// pipelines of many models a compute unit has room for few wavefronts, so the latencies go
// where nothing is meanwhile: those at even costs in the last row, which is filled when the
// rows are complete, those at odd ones (from 16 models on) in the words of the best candidates,
// which steps A and G use.  (With words of their own for both, twice over, 7000 x 56 models with
// three batch sizes took 38.1 us and take 33.8, six wavefronts of a compute unit and seven;
// 20000 x 14 50.6 and 48.8, 20000 x 20 80.8 and 78.2.)
struct StepCLds {
    int rows, even, odd, copy, words;
};
constexpr StepCLds step_c_lds(int S, int tab)
{
    StepCLds c{};
    c.rows = tab + 64 * S;
    c.even = c.rows + 32 * S;
    const int behind = c.even + 32;
    c.odd = S >= 16 ? 0 : behind;
    c.copy = (S >= 16 ? behind : behind + 32) + 32;
    c.words = c.copy + 32;
    return c;
}
constexpr CostLds cost_lds(int S, int window, int words = 0)
{
    CostLds l{};
    l.best = 0;  // two words per model
    l.key = 2 * S;
    l.fast = l.key + S;
    l.pin = l.fast + S;
    l.tab = (l.pin + S + 3) & ~3;
    l.rows = l.tab + window;
    const int w = l.rows + (S + 1) * (window + 2) / 2;
    const int b = l.tab + 64 * S + 8 + 16 * (S + 1), c = step_c_lds(S, l.tab).words;
    l.least = ((w > b ? w > c ? w : c : b > c ? b : c) + 3) & ~3;
    l.words = words;
    return l;
}

// A launch's window (cells of the largest one with rows in LDS) and LDS.
// bytes; LDS is granted in whole units, and a kernel that may have more than LDS_UNASKED needs an
// attribute set, which takes the host 0.14 us
constexpr int LDS_PER_CU = 160 * 1024, LDS_UNIT = 1280, LDS_UNASKED = 64 * 1024, LDS_MOST = LDS_PER_CU / 2;
constexpr int MAX_WINDOW = 8192;
// Wavefronts of a compute unit that share its LDS, and how many of them are resident then, as
// what 28 leave each other is five units.  Registers allow 32, but some twenty are in flight on
// average, and the room of the others lets step G list more candidates (measured while it
// could only list all of them: at 16384 x 8 with a twelfth of the objectives 32 / 28 / 24 / 20
// took 579 / 122 / 121 / 129 us, at 86400 x 6 51 / 51 / 55 / 60).
constexpr int SHARED_PER_CU = 28, RESIDENT_PER_CU = 25, SIMDS_PER_CU = 4;
struct LdsPlan {
    int window, words;  // words: of one wavefront, and WAVE_FLAGS behind them where there are two
    int bytes;          // of a workgroup
};
constexpr int WAVE_FLAGS = 4;
// groups: workgroups of the launch, of `waves` wavefronts; spread: of a pipeline's costs
inline LdsPlan lds_plan(int S, int spread, int groups, int waves, int cus)
{
    const int flags = waves > 1 ? WAVE_FLAGS : 0;
    auto bytes_for = [&](int window) { return 4 * waves * (cost_lds(S, window).least + flags); };
    // what leaves room for as many workgroups
    auto filled = [](int bytes) {
        const int units = (bytes + LDS_UNIT - 1) / LDS_UNIT, all = LDS_PER_CU / LDS_UNIT;
        return all / (all / units) * LDS_UNIT;
    };
    // Where all workgroups can be resident, what those of a compute unit leave each other in
    // whole units, all of it: of a quotient of bytes the last unit is granted too, and the
    // compute unit has one workgroup fewer, that waits until another ends (3001 x 7 models,
    // twelve and room for eleven: 12.75 us, with room 11.84).  With a quarter more of them to be on
    // the safe side the lists of step G run out of words: 5000 x 7 models, 256 candidates each,
    // 126 us, 92 without.
    const int per_cu = (groups + cus - 1) / cus, few = 4 / waves, most = SHARED_PER_CU / waves;
    const bool all = per_cu <= RESIDENT_PER_CU / waves;
    int bytes = all ? LDS_PER_CU / LDS_UNIT / (per_cu < few ? few : per_cu) * LDS_UNIT
                    : LDS_PER_CU / (per_cu > most ? most : per_cu);
    // (60 x 64 models whose rows by cost are in HBM with less than is unasked take 163 us instead
    // of 109, up to 16 models nothing does)
    if (S <= 16 && bytes > LDS_UNASKED) bytes = LDS_UNASKED / LDS_UNIT * LDS_UNIT;
    // (the least there is to have, and what no further workgroup could have: stability test of
    // 4096 x 16 models 56.6 us without that, 43.1 with it)
    const int least = filled(bytes_for(64));
    const bool tight = bytes < bytes_for(64);
    if (tight) bytes = least;
    LdsPlan p{};
    p.window = 64;
    while (p.window + 64 <= MAX_WINDOW && p.window < spread && bytes_for(p.window + 64) <= bytes) p.window += 64;
    if (!all && !tight) bytes = p.window > 64 ? bytes_for(p.window) : least;
    // no more than the costs of a pipeline can spread over need
    if (p.window >= spread && filled(bytes_for(p.window)) < bytes) bytes = filled(bytes_for(p.window));
    p.words = (bytes / 4 / waves & ~3) - flags;
    p.bytes = 4 * waves * (p.words + flags);
    return p;
}

// Whether an instance's two solves of the stability test get a wavefront each.
//
// That halves its chain where there is one (a single model is done with step A), which shows far
// beyond the twelve pairs per compute unit that can be in flight: of seven mixes of rates and
// objectives, with half of the rates predicted to stay or none, pairs are the sooner done in most
// up to 9000 instances of 2 to 33 models, at 15000 with few models no longer.  What they cost is
// the launch of twice the wavefronts, where next to all instances are done with step A.
// Microseconds in one wavefront and two, instances that need steps B and C / that don't: 4099 x 5
// models 35.7, 20.7 / 7.3, 7.0; 7000 x 2 14.5, 13.3 / 7.9, 8.3; 6000 x 4 24.3, 21.9 / 7.3, 8.0;
// 7000 x 8 47.0, 32.5 / 11.6, 10.5; 7000 x 33 271, 239 / 116, 112; 9000 x 3 21.7, 19.5 / 9.3, 9.9;
// 15000 x 3 26.3, 26.7 / 12.7, 14.6; 15000 x 8 58.4, 46.9 / 16.5, 17.0.
// The second wavefront's work is in vain where the first finds no solution, and it stops when it is
// told.  If that is so for every instance of the batch: 2000 x 5 6.9, 6.9; 4099 x 5 6.8, 9.7;
// 7000 x 5 6.9, 13.0; 4099 x 24 10.3, 23.8 (for half of them 15.4, 12.9; 18.7, 16.9; 113, 76).
inline bool stability_in_pairs(int S, int instances, int cus)
{
    return S > 1 && instances <= 28 * cus;
}

}  // namespace themis
