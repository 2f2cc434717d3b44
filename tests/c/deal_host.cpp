// Host-side check of the allocator that deals a launch's workgroups out to its GEMMs
// (csrc/tl_deal.hpp): every job gets at least one workgroup and no more than it has tiles, the
// counts add up to the workgroups available whenever the jobs hold that many tiles, equal jobs get
// equal shares, a costlier job never gets fewer workgroups than a cheaper one of the same size,
// and no single move of a workgroup from one job to another shortens the longest run.
#include "tl_deal.hpp"

#include <chrono>
#include <cstdio>
#include <cstdlib>
#include <vector>

using namespace tl;

static int fail(const char* what, int a, int b)
{
    std::printf("FAILED: %s (%d, %d)\n", what, a, b);
    return 1;
}

static double makespan(const DealModel& m, const std::vector<DealJob>& jobs, const std::vector<int>& wg)
{
    double t = 0.0;
    for (size_t j = 0; j < jobs.size(); ++j) {
        const double c = deal_run_cost(m, jobs[j], wg[j]);
        if (c > t) t = c;
    }
    return t;
}

// The spare groups one at a time, each to the job with the costliest run, the first of equals.
static void deal_one_by_one(const DealModel& m, const DealJob* jobs, int count, int G, int* wg)
{
    double lo = 0.0, hi = 0.0;
    for (int j = 0; j < count; ++j) { const double c = deal_run_cost(m, jobs[j], 1); if (c > hi) hi = c; }
    for (int it = 0; it < 24; ++it) {
        const double mid = 0.5 * (lo + hi);
        int need = 0;
        for (int j = 0; j < count; ++j) need += deal_groups_for(m, jobs[j], mid);
        if (need <= G) hi = mid; else lo = mid;
    }
    int used = 0;
    for (int j = 0; j < count; ++j) { wg[j] = deal_groups_for(m, jobs[j], hi); used += wg[j]; }
    while (used < G) {
        int best = -1;
        for (int j = 0; j < count; ++j)
            if (wg[j] < jobs[j].tiles &&
                (best < 0 || deal_run_cost(m, jobs[j], wg[j]) > deal_run_cost(m, jobs[best], wg[best]))) best = j;
        if (best < 0) break;
        ++wg[best]; ++used;
    }
}

int main()
{
    const DealModel m{3, true, 2.1, 0.43};
    unsigned s = 12345u;
    auto rnd = [&](unsigned n) { s = s * 1664525u + 1013904223u; return (s >> 8) % n; };
    for (int trial = 0; trial < 400; ++trial) {
        const int count = 1 + int(rnd(32));
        std::vector<DealJob> jobs(count);
        long total = 0;
        for (auto& j : jobs) {
            j.tiles = 1 + int(rnd(trial % 3 == 0 ? 8 : 2000));
            j.passes = 1 + int(rnd(3));
            j.start_up = 0.15 * double(1 + rnd(16)) + (j.passes > 1 ? 1.5 : 0.0);
            total += j.tiles;
        }
        const int cap = 256;
        const int G = total < cap ? int(total) : cap;
        if (G < count) continue;                            // the launchers never ask for fewer groups than jobs
        std::vector<int> wg(count, -1);
        deal_workgroups(m, jobs.data(), count, G, wg.data());
        int used = 0;
        for (int j = 0; j < count; ++j) {
            if (wg[j] < 1) return fail("a job without a workgroup", trial, j);
            if (wg[j] > jobs[j].tiles) return fail("more workgroups than tiles", trial, j);
            used += wg[j];
        }
        if (used != G) return fail("counts do not add up", used, G);
        // no single move helps
        const double t0 = makespan(m, jobs, wg);
        for (int a = 0; a < count; ++a)
            for (int b = 0; b < count; ++b) {
                if (a == b || wg[a] <= 1 || wg[b] >= jobs[b].tiles) continue;
                std::vector<int> w2 = wg;
                --w2[a]; ++w2[b];
                if (makespan(m, jobs, w2) < t0 - 1e-9) return fail("a single move shortens the longest run", trial, a * 100 + b);
            }
    }
    // handing spare groups over in one go changes nothing, whatever the model, the jobs and the groups
    for (int trial = 0; trial < 600; ++trial) {
        const DealModel mm{1 + int(rnd(3)), trial % 5 != 0, 2.1, 0.43};
        const int count = 1 + int(rnd(trial % 7 == 0 ? 100 : 32));
        std::vector<DealJob> jobs(count);
        long total = 0;
        for (int i = 0; i < count; ++i) {
            DealJob& j = jobs[i];
            j.tiles = i > 0 && trial % 2 ? jobs[0].tiles : 1 + int(rnd(trial % 3 == 0 ? 40 : 2000));
            j.passes = 1 + int(rnd(trial % 4 ? 1 : 3));
            j.start_up = 0.15 * double(1 + (trial % 2 ? 15 : rnd(16)));
            total += j.tiles;
        }
        const int cap = 256 << rnd(4);
        const int G = total < cap ? int(total) : cap;
        if (G < count) continue;
        std::vector<int> wg(count), ref(count);
        deal_workgroups(mm, jobs.data(), count, G, wg.data());
        deal_one_by_one(mm, jobs.data(), count, G, ref.data());
        long used = 0;
        for (int w : ref) used += w;
        if (used <= G && wg != ref) return fail("not what one group at a time gives", trial, count);
    }
    // and takes less of the host's time than the launch (52 us one group at a time on the machine where this takes 4.3)
    {
        std::vector<DealJob> jobs(12, DealJob{1024, 1, 4.8});
        std::vector<int> wg(12);
        double least = 1e9;
        for (int r = 0; r < 50; ++r) {
            const auto t0 = std::chrono::steady_clock::now();
            deal_workgroups(DealModel{2, true, 2.1, 0.43}, jobs.data(), 12, 2048, wg.data());
            const double us = std::chrono::duration<double, std::micro>(std::chrono::steady_clock::now() - t0).count();
            if (us < least) least = us;
        }
        if (least > 25.0) return fail("dealing takes too long (us)", int(least), 25);
    }
    // blocks of rows of one matrix are worked out once: six matrices of four blocks take a third of the time of 24 matrices (all that time without that)
    {
        auto time_of = [&](const std::vector<DealJob>& jobs) {
            std::vector<int> wg(jobs.size());
            double least = 1e9;
            for (int r = 0; r < 200; ++r) {
                const auto t0 = std::chrono::steady_clock::now();
                deal_workgroups(m, jobs.data(), int(jobs.size()), 256, wg.data());
                const double us = std::chrono::duration<double, std::micro>(std::chrono::steady_clock::now() - t0).count();
                if (us < least) least = us;
            }
            return least;
        };
        std::vector<DealJob> blocks, apart;
        for (int tiles : {66, 21, 345, 37, 68, 120})
            for (int q = 0; q < 4; ++q) {
                blocks.push_back(DealJob{tiles, 1, 2.4});
                apart.push_back(DealJob{tiles + q, 1, 2.4 + 0.15 * q});
            }
        const double us = time_of(blocks), of = time_of(apart);
        if (us > 0.75 * of) return fail("blocks of rows of one matrix take too long (ns)", int(1e3 * us), int(1e3 * of));
    }
    // equal jobs, equal shares; and the sweep of the benchmark: five jobs of 256 tiles and five of 896,
    // 1, 2, 4, 8, 16 rows each
    {
        std::vector<DealJob> jobs(8, DealJob{500, 1, 0.15});
        std::vector<int> wg(8);
        deal_workgroups(m, jobs.data(), 8, 256, wg.data());
        for (int j = 0; j < 8; ++j)
            if (wg[j] != 32) return fail("equal jobs, unequal shares", j, wg[j]);
    }
    {
        std::vector<DealJob> jobs;
        for (int tiles : {256, 896})
            for (int rows : {1, 2, 4, 8, 16}) jobs.push_back(DealJob{tiles, 1, 0.15 * rows});
        std::vector<int> wg(jobs.size());
        deal_workgroups(m, jobs.data(), int(jobs.size()), 256, wg.data());
        for (int half = 0; half < 2; ++half)
            for (int i = 1; i < 5; ++i)
                if (wg[5 * half + i] < wg[5 * half + i - 1]) return fail("more rows, fewer workgroups", half, i);
        for (int i = 0; i < 5; ++i)
            if (wg[5 + i] <= wg[i]) return fail("more tiles, not more workgroups", i, wg[i]);
    }
    std::printf("ok\n");
    return 0;
}
