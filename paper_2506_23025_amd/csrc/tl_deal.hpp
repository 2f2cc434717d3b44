// Dealing out the workgroups of one launch to the GEMMs it carries (host side), shared by the
// weight-streaming kernels of both packed formats.
//
// A workgroup serves one job and walks a run of consecutive 16-row tiles of its matrix, in items
// of up to t_max tiles.  Its time, in units of an average tile, is
//     passes x (time of the run + start-up),
// where an item costs its latency and its barrier once (item_first for its first tile, tile_extra
// for each further one) and the start-up is what a workgroup does before its first tile (fetching
// the activation rows, building the operands).  Bisection on a common finishing time gives the
// fewest workgroups each job needs; spare workgroups go to the job with the costliest run.
#pragma once

namespace tl {

struct DealJob {
    int tiles;          // 16-row tiles of the job's matrix
    int passes;         // passes over K of a workgroup of this job
    double start_up;    // start-up of a pass, in tiles
};

struct DealModel {
    int t_max;          // tiles per item
    bool item_cost;     // count items (false: a run costs its tiles)
    double item_first;  // cost of the first tile of an item, in average tiles
    double tile_extra;  // cost of each further tile of an item
};

inline double deal_run_time(const DealModel& m, int run)
{
    if (!m.item_cost) return double(run);
    // a run of 4 goes as 2 + 2 when items hold 3
    const int items = run <= m.t_max ? 1 : (m.t_max == 3 ? (run == 4 ? 2 : (run + 2) / 3) : (m.t_max == 2 ? (run + 1) / 2 : (run + m.t_max - 1) / m.t_max));
    return m.item_first * double(items) + m.tile_extra * double(run - items);
}

inline double deal_run_cost(const DealModel& m, const DealJob& j, int w)
{
    return double(j.passes) * (deal_run_time(m, (j.tiles + w - 1) / w) + j.start_up);
}

// longest run that takes no more than `per`; 0 if one tile takes longer
inline int deal_longest_run(const DealModel& m, double per)
{
    // from the estimate with whole items, a few steps up or down
    const double per_tile = m.item_cost ? (m.item_first + m.tile_extra * double(m.t_max - 1)) / double(m.t_max) : 1.0;
    int run = int(per / per_tile);
    if (run < 1) run = 1;
    while (run > 1 && deal_run_time(m, run) > per) --run;
    while (deal_run_time(m, run + 1) <= per) ++run;
    return deal_run_time(m, run) > per ? 0 : run;
}

// Of every job the fewest workgroups that finish it by tau, and their sum.  The longest run depends on a job's passes and start-up alone, in which the jobs
// of a call are mostly alike: 24 blocks of six matrices 26 -> 2.2 us of the host, 16 matrices 8.2 -> 2.0.
inline int deal_groups_of_all(const DealModel& m, const DealJob* jobs, int count, double tau, int* wg)
{
    int need = 0, longest = 0;
    for (int j = 0; j < count; ++j) {
        const DealJob& a = jobs[j];
        if (j == 0 || a.passes != jobs[j - 1].passes || a.start_up != jobs[j - 1].start_up) longest = deal_longest_run(m, tau / double(a.passes) - a.start_up);
        const int run = longest < a.tiles ? longest : a.tiles;
        wg[j] = run < 1 ? a.tiles : (a.tiles + run - 1) / run;
        need += wg[j];
    }
    return need;
}

inline int deal_groups_for(const DealModel& m, const DealJob& j, double tau)
{
    int w;
    deal_groups_of_all(m, &j, 1, tau, &w);
    return w;
}

// wg[j] >= 1 workgroups for job j, G in all when the jobs hold at least G tiles (fewer jobs than G)
inline void deal_workgroups(const DealModel& m, const DealJob* jobs, int count, int G, int* wg)
{
    double lo = 0.0, hi = 0.0;
    for (int j = 0; j < count; ++j) { const double c = deal_run_cost(m, jobs[j], 1); if (c > hi) hi = c; }
    for (int it = 0; it < 24; ++it) {
        const double mid = 0.5 * (lo + hi);
        if (deal_groups_of_all(m, jobs, count, mid, wg) <= G) hi = mid; else lo = mid;
    }
    int used = deal_groups_of_all(m, jobs, count, hi, wg);
    // Spare groups, one by one to the job with the costliest run (the first of equals).  A job keeps getting them until its run is
    // a tile shorter, so all of those are handed over at once: hundreds of spare groups cost the host more than the kernel
    // takes otherwise (12 jobs of 1024 tiles on 2048 groups: 52 us one at a time, 4.3 like this).
    auto cost_of = [&](int j) { return wg[j] < jobs[j].tiles ? deal_run_cost(m, jobs[j], wg[j]) : -1.0; };
    constexpr int kKept = 64;                              // costs kept between turns; a longer list is worked out anew each turn
    double kept[kKept];
    if (count <= kKept) for (int j = 0; j < count; ++j) kept[j] = cost_of(j);
    while (used < G) {
        int best = -1;
        double most = -1.0;
        for (int j = 0; j < count; ++j) {
            const double c = count <= kKept ? kept[j] : cost_of(j);
            if (c > most) { most = c; best = j; }
        }
        if (best < 0) break;
        const int tiles = jobs[best].tiles, run = (tiles + wg[best] - 1) / wg[best];
        int next = run > 1 ? (tiles + run - 2) / (run - 1) : tiles;       // fewest groups with a shorter run
        if (next > wg[best] + (G - used)) next = wg[best] + (G - used);
        used += next - wg[best];
        wg[best] = next;
        if (count <= kKept) kept[best] = cost_of(best);
    }
    while (used > G) {                                     // cannot happen unless there are more jobs than groups
        int best = -1;
        for (int j = 0; j < count; ++j)
            if (wg[j] > 1 &&
                (best < 0 || deal_run_cost(m, jobs[j], wg[j]) < deal_run_cost(m, jobs[best], wg[best]))) best = j;
        if (best < 0) break;
        --wg[best]; --used;
    }
}

}  // namespace tl
