// Which sweep a context takes, by the acceptance that its ladder will have.
// The sweeps that correct fields where an update is accepted (pairs.hip) or
// stop at the first accepted step (ahead.hip) cost more the more is accepted;
// the list-streaming sweep costs the same at any temperature.  Host only.
#pragma once
#include <math.h>

#include <algorithm>
#include <vector>

#include "ahead.hpp"

namespace rlpt {

// Share of two-mode updates accepted at temperature T in equilibrium.  It is the
// same within about 0.02 for dense samples of 32 to 256 modes, other linewidths
// and splits, and sparse ones of 32 terms per mode (0.05 more below T = 1 at 8
// terms per mode); with the spherical constraint about that of 0.72 T.
inline double update_acceptance(double T, int rho) {
    static const double at[][2] = {{0.25, 0.004}, {0.5, 0.014}, {0.75, 0.037}, {1.0, 0.095},  {1.33, 0.205}, {1.78, 0.348},
                                   {2.37, 0.485}, {3.16, 0.603}, {4.22, 0.695}, {5.62, 0.771}, {7.5, 0.827},  {10.0, 0.87},
                                   {17.8, 0.926}, {31.6, 0.958}, {100.0, 0.987}};
    constexpr int n = sizeof(at) / sizeof(at[0]);
    if (rho == 2) T *= 0.72;
    if (T <= at[0][0]) return at[0][1];
    for (int i = 1; i < n; ++i)
        if (T <= at[i][0]) {
            const double f = log(T / at[i - 1][0]) / log(at[i][0] / at[i - 1][0]);
            return at[i - 1][1] + f * (at[i][1] - at[i - 1][1]);
        }
    return at[n - 1][1];
}

// Whether `copies` copies of dense samples of N >= 88 modes in one ladder of
// baths are swept faster in pair space than from their lists: up to an
// acceptance that was measured over N and the number of copies (us per sweep at
// two ladders, T = 0.25-1.5 and 1-3, both sweeps on an MI355X; where the lines
// cross, by linear interpolation).  With at most a copy per compute unit the
// chain of the hottest bath is the sweep's time, with more the mean of all.  The
// lists' side is uneven (its tiles change with the number of copies), hence a
// table.  Lists against pairs, cold and warm ladder: N = 96, 8 copies 103 against
// 65 and 121, 640 copies 248 against 122 and 248, 2048 copies 281 against 244 and
// 511; N = 128, 640 copies 289 against 197 and 415; N = 256, 8 copies 954 against
// 430 and 994, 640 copies 2618 against 869 and 2133 (3892 at T = 2-6).
// In equilibrium, that is: the first sweeps from a random state accept more, on
// any ladder, and take longer (N = 128, 640 copies, T = 0.25-1.5: 594, 433, 374, 337
// against 328 from the lists, level after the fourth sweep and ahead in all after some
// ten; N = 256 the first only, 3246 against 2626).  The sweep does not change in a
// run: replayed graphs and resumed runs have the same bits.
inline bool pair_space_pays(int N, int64_t copies, bool shared_pairs, int cus, double mean, double hottest) {
    struct Row {
        int N;
        double few[2];   // hottest bath's acceptance at 8 and 80 copies
        double many[4];  // mean acceptance at 320, 640, 1024 and 2048 copies
    };
    static const Row rows[] = {{0, {0.45, 0.35}, {0.49, 0.33, 0.15, 0.13}},   {104, {0.50, 0.42}, {0.65, 0.15, 0.17, 0.16}},
                               {120, {0.57, 0.45}, {0.60, 0.20, 0.29, 0.21}}, {137, {0.42, 0.34}, {0.46, 0.20, 0.23, 0.15}},
                               {152, {0.48, 0.39}, {0.22, 0.25, 0.30, 0.21}}, {176, {0.50, 0.44}, {0.28, 0.30, 0.31, 0.32}},
                               {208, {0.54, 0.47}, {0.33, 0.38, 0.41, 0.46}}, {240, {0.56, 0.49}, {0.38, 0.42, 0.46, 0.52}}};
    const Row* r = rows;
    for (const Row& q : rows)
        if (N >= q.N) r = &q;
    // one sequence of pairs for a sample's copies lets the lists be read from the caches
    const double scale = shared_pairs ? 0.85 : 1.0;
    if (copies <= cus) {
        const double f = std::min(std::max(log2((double)copies / 8.0) / log2(10.0), 0.0), 1.0);
        return hottest <= scale * (r->few[0] + f * (r->few[1] - r->few[0]));
    }
    static const double at[4] = {320, 640, 1024, 2048};
    double line = r->many[3];
    for (int i = 0; i < 4; ++i)
        if ((double)copies <= at[i]) {
            line = r->many[i];
            if (i > 0) {
                const double f = log2((double)copies / at[i - 1]) / log2(at[i] / at[i - 1]);
                line = r->many[i - 1] + f * (r->many[i] - r->many[i - 1]);
            }
            break;
        }
    return mean <= scale * line;
}

struct Ladder {
    double mean = 0, hottest = 0;  // acceptance
};

inline Ladder ladder_acceptance(const std::vector<double>& temps, int rho) {
    Ladder l;
    for (double T : temps) l.mean += update_acceptance(T, rho) / (double)temps.size();
    if (!temps.empty()) l.hottest = update_acceptance(temps.back(), rho);
    return l;
}

// Whether the sweep of several steps at a time (ahead.hip) pays on a ladder,
// against one step at a time.  A round decides W steps unless one is accepted,
// so a step costs p / (1 - (1 - p)^W) rounds at acceptance p (beside a part that
// does not follow it, most of it a sweep's draws).  A round's time over a step's
// of the other sweep was measured where nearly everything is accepted (T =
// 50-100, 0.98; up to a copy per compute unit): packed lists of up to 128 entries 0.7-0.8 at N = 8,
// 0.9-1.0 at 16, 1.4 from 128 on (1.06 in FP64 with 256 threads, N = 1024); of
// up to 256, 384 and 512 entries 0.7, 0.8 and 0.9; chunked lists 1.25 at N = 32,
// 1.45 at 36, 1.6 at 40, 1.8-1.9 from 48 on.  The hottest copies bound the sweep
// while every workgroup is resident at once; beyond that the sum over the copies
// does, or those that share a place.  In FP64 with 512 threads the other sweep is
// half as fast past a copy per compute unit, too.  On the measured grid (268 sizes, numbers of copies
// and types, three ladders) the choice is the faster sweep within 5 %, but for 14
// points in 804 (6 to 35 %).  Us per sweep, one step at a time -> several, at T =
// 0.25-1.5, 1-3 and 50-100: N = 1024 of mean degree 40, FP32, 256 copies 403 -> 177, 340,
// 557; 768 copies 404 -> 323, 656, 1662; FP64 545 -> 307, 391, 546 and 549 ->
// 810, 990, 1628; N = 48 FP32, 8 copies 30 -> 21, 32, 53; N = 24 23 -> 9, 12, 18.
inline bool ahead_pays(int precision, const AheadLaunch& L, size_t lds_bytes, int64_t copies, int cus,
                       bool others_crowd, const std::vector<double>& temps, int rho) {
    double round;
    if (L.chunks > 0) round = std::min(1.95, 1.3 + 0.04 * std::max(0, L.max_N - 32));
    else if (L.slots > kShortSlots) round = L.slots > 12 ? 0.95 : L.slots > 8 ? 0.85 : 0.8;
    else round = std::min(L.block == 256 ? 1.1 : 1.45, 0.45 + 0.028 * L.max_N);
    const double W = L.block / 128;
    const double fixed = 0.06 + 2.0 / L.max_N;
    const int n = (int)temps.size();
    std::vector<double> cost(n);  // of a copy at each bath, the hottest first, over the other sweep's
    double mean = 0.0;
    for (int i = 0; i < n; ++i) {
        const double p = update_acceptance(temps[n - 1 - i], rho);
        cost[i] = round * (fixed + (1.0 - fixed) * p / (1.0 - pow(1.0 - p, W)));
        mean += cost[i] / n;
    }
    // resident workgroups of a compute unit: by registers, and by LDS
    const int by_regs = L.block == 1024 || (L.block == 512 && precision == RLPT_FP64) ? 1 : 2;
    const int64_t room = (int64_t)cus * std::min(by_regs, (int)(kMaxLds / lds_bytes));
    double t = std::max(cost[0], mean * (double)copies / (double)room);
    for (int64_t k = 1; k * room < copies; ++k)  // of the k room + 1 hottest copies, k + 1 go one after another
        t = std::max(t, (double)(k + 1) * cost[k * room * n / copies]);
    return t < (!others_crowd ? 1.0 : L.chunks > 0 ? 1.65 : 1.7);
}

}  // namespace rlpt
