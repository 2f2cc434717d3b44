// Which jobs of a grouped call share launches, and how a shared launch hands its jobs out (host side; plain C++).
#pragma once

#include <cstdint>

namespace tl {

// A job's alternatives.  Times in us; 0 throughout where the streaming kernel is the one whatever the others take (few rows).
struct KernelChoice {
    bool streams;          // the weight-streaming kernel can take it and shares its launches with other jobs
    double stream;         // a call of its own there
    double tiled;          // a call of its own in the tiled kernel, the caller's band included; as much as `stream` or more where it cannot win
    double own;            // what it adds to the launches that it shares, beside its part of
    double launch;         // what one of those costs whatever it holds
    double launches;       // how many of them it would fill (blocks of rows over blocks per launch)
};

// Which jobs of a grouped call run as calls of their own though they could share launches.  A job that shares pays only for the part of the launch that
// it fills, which is what makes small ones cheap (16 layers of 512 x 1024 at M = 256, choosing as if alone 83 us, sharing 65; the linears of a block
// at M = 48 with groups of 128 72 and 65); but shared launches hold 512 rows and mostly one workgroup per CU, where a call of its own is one launch of as many
// as fit, or the tiled kernel's.  So a job leaves if its call is shorter than what it adds; and what is left shares, unless it is so little
// that it would not pay for its launch.  A job alone is a call of its own, tiled or not.
inline void choose_grouped(const KernelChoice* c, int n, bool* alone)
{
    if (n == 1) { alone[0] = c[0].streams && c[0].tiled < c[0].stream; return; }
    double rest = 0.0, all = 0.0, launch = 0.0, launches = 0.0, total = 0.0;
    bool any = false, can = true;
    for (int j = 0; j < n; ++j) total += c[j].launches;
    const double spared = total > 1.0 ? 1.0 - 1.0 / total : 0.0;       // the first launch is not
    for (int j = 0; j < n; ++j) {
        alone[j] = false;
        if (!c[j].streams) continue;
        const double call = c[j].tiled < c[j].stream ? c[j].tiled : c[j].stream;
        alone[j] = call < c[j].own + spared * c[j].launch * c[j].launches;
        if (alone[j]) continue;
        any = true;
        can = can && c[j].stream > 0.0;
        rest += c[j].own;
        all += call;
        launches += c[j].launches;
        if (c[j].launch > launch) launch = c[j].launch;
    }
    if (!any || !can || all >= rest + launch * (launches > 1.0 ? launches : 1.0)) return;
    for (int j = 0; j < n; ++j) alone[j] = c[j].streams;
}

// How the workgroups of a shared launch of the 2-bit streaming kernel find their jobs, when K is one pass: in a table of jobs (68 bytes of arguments each, two
// scalar look-ups in turn) or each in a record of its own (16 KB).  records: whether the launch can do without the table; several: more workgroups
// than CUs; w_bytes: its packed words; captured: it becomes part of a graph.
// The records cost the host 1.1 us, which is what a small call waits for.  The look-ups cost the device 0.2 to 0.5 us where a CU holds one workgroup,
// nothing where it holds several.  So the table takes launches below 8 MB (two layers of 2048 x 2048 called in a loop 5.4 -> 4.3 us, 4096 x 4096 5.6 ->
// 4.8; 18 x 4672 x 4096, 9.1 MB, 5.6 and by the table 5.9), but not under capture, since a replay pays nothing for arguments (the three 3.1, 4.6 and
// 5.1 us, by the table 3.3, 5.0 and 5.5), unless there are several workgroups to a CU.
// A launch that cannot do without it, of group scales and more than 256 workgroups, has as many jobs as a launch holds: the form for any K and N, with
// records for 256, leaves wavefronts out (block of 174 rows, 1024 wide with groups of 256, 17.7 -> 22.0 us).
constexpr int kTableJobs = 16, kTableMost = 32;
inline bool jobs_by_table(int count, bool one_pass, bool records, bool several, int64_t w_bytes, bool captured)
{
    if (!one_pass || count < 2 || count > (records ? kTableJobs : kTableMost)) return false;
    return !records || (w_bytes < (int64_t(8) << 20) && (several || !captured));
}

}  // namespace tl
