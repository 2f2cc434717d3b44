// Which jobs of a grouped call go through the tiled kernel, and how a shared launch hands its jobs out (host side; plain C++).
#pragma once

#include <cstdint>

namespace tl {

// A job's alternatives.  Times in us, of a call of its own.
struct KernelChoice {
    bool streams;          // the weight-streaming kernel can take it and shares its launches with other jobs
    double stream;         // time there
    double fixed;          // what of that its launches cost whatever they hold
    double launch;         // the same of one launch shared with others
    double launches;       // how many of those it would fill (blocks of rows over blocks per launch)
    double tiled;          // time in the tiled kernel, the caller's band included; as much as `stream` or more where it cannot win
};

// A job of a shared launch pays only for the part of the launch that it fills, while a launch of the tiled kernel serves one job.  So a job
// is tiled if that beats its streaming time less the launch it shares (16 layers of 512 x 1024 at M = 256, choosing as if alone 83 us, like this
// 65; the linears of a block at M = 48 with groups of 128 72 and 65); and what is left streams, unless it is so little that it would
// not pay for its launch.  tiled[j] implies that job j alone would be tiled too; with one job it is just that.
constexpr double kBetween = 1.0;                           // a launch of its own between others, us (ties went wrong by 2 us of 29 and 4 of 58 without)

inline void choose_grouped(const KernelChoice* c, int n, bool* tiled)
{
    double rest = 0.0, all = 0.0, launch = 0.0, launches = 0.0;
    bool any = false, can = true;
    for (int j = 0; j < n; ++j) {
        if (!c[j].streams) { tiled[j] = false; continue; }
        const double own = c[j].stream - c[j].fixed, shared = own + c[j].launch * c[j].launches;
        tiled[j] = n > 1 ? c[j].tiled + kBetween < shared && c[j].tiled < c[j].stream : c[j].tiled < c[j].stream;
        if (tiled[j]) continue;
        any = true;
        can = can && c[j].tiled < c[j].stream;
        rest += own;
        all += c[j].tiled;
        launches += c[j].launches;
        if (c[j].launch > launch) launch = c[j].launch;
    }
    if (!any || !can || all >= rest + launch * (launches > 1.0 ? launches : 1.0)) return;
    for (int j = 0; j < n; ++j) tiled[j] = c[j].streams;
}

// How the workgroups of a shared launch of the 2-bit streaming kernel find their jobs, when K is one pass: in a table of jobs (1 KB of arguments, two
// scalar look-ups in turn) or each in a record of its own (16 KB).  records: whether the launch can do without the table; several: more workgroups
// than CUs; w_bytes: its packed words; captured: it becomes part of a graph.
// The records cost the host 1.1 us, which is what a small call waits for.  The look-ups cost the device 0.2 to 0.5 us where a CU holds one workgroup,
// nothing where it holds several.  So the table takes launches below 8 MB (two layers of 2048 x 2048 called in a loop 5.4 -> 4.3 us, 4096 x 4096 5.6 ->
// 4.8; 18 x 4672 x 4096, 9.1 MB, 5.6 and by the table 5.9), but not under capture, since a replay pays nothing for arguments (the three 3.1, 4.6 and
// 5.1 us, by the table 3.3, 5.0 and 5.5), unless there are several workgroups to a CU.
constexpr int kTableJobs = 16;
inline bool jobs_by_table(int count, bool one_pass, bool records, bool several, int64_t w_bytes, bool captured)
{
    if (!one_pass || count < 2 || count > kTableJobs) return false;
    return !records || (w_bytes < (int64_t(8) << 20) && (several || !captured));
}

}  // namespace tl
