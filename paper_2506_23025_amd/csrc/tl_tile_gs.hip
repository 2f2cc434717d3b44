// 2-bit words with group scales: instances of the tiled matrix-core kernel and the choice among
// them.
#include "tl_tile.hpp"

namespace tl {

namespace {

// Last parameter: 16-k blocks per scale that is fetched.  The large tiles fetch one scale per 64 k (groups that are
// multiples of 64; a scale per 16 k would cost four transfers a step instead of one: 128 x 128, K = 4096, 256 tiles
// 39.7 against 36.0 us), the small ones one per 16 k (no difference: their one transfer has room for them).
typedef TileCfg<kTileGs, false, 8, 4, 2, 4, 1, 2, 3, 4> T256x256;
typedef TileCfg<kTileGs, false, 8, 4, 1, 4, 2, 4, 3, 4> T128x256;
typedef TileCfg<kTileGs, false, 8, 2, 1, 4, 2, 4, 4, 4> T128x128;
typedef TileCfg<kTileGs, false, 8, 2, 1, 4, 2, 4, 3, 1> T128x128any;
typedef TileCfg<kTileGs, false, 8, 2, 1, 2, 4, 4, 3, 1> T128x64any;
typedef TileCfg<kTileGs, false, 4, 2, 1, 2, 4, 4, 4, 1> T64x64any;
typedef TileCfg<kTileGs, false, 2, 2, 1, 2, 4, 4, 4, 1> T32x64any;

constexpr int kShapes = 7, kFirstAny = 3;     // from kFirstAny on any group that is a multiple of 16
constexpr TileCost kCost[kShapes] = {
    {256, 256, 64, 256, 6.8, 6.8, 0.955, 1.444, 1.444, 0.743, 2.24},
    {128, 256, 128, 256, 7.29, 7.29, 1.089, 1.505, 1.505, 0.838, 3.37},
    {128, 128, 128, 256, 5.31, 5.31, 0.632, 0.861, 0.861, 0.826, 2.76},
    {128, 128, 128, 256, 5.32, 5.32, 0.617, 0.842, 0.842, 0.865, 2.88},
    {128, 64, 128, 256, 4.43, 4.43, 0.379, 0.475, 0.475, 0.909, 1.9},
    {64, 64, 128, 512, 1.61, 3.79, 0.282, 0.343, 0.545, 0.432, 3.76},
    {32, 64, 128, 512, 1.13, 3.29, 0.227, 0.265, 0.398, 0.375, 3.68},
};

// K that is no multiple of 64
typedef TileCfg<kTileGs, true, 4, 2, 1, 4, 2, 4, 2, 1> R64x128;
typedef TileCfg<kTileGs, true, 2, 2, 1, 2, 4, 4, 2, 1> R32x64;      // two workgroups per CU
typedef TileCfg<kTileGs, true, 1, 2, 1, 2, 4, 4, 2, 1> R16x64;      // two workgroups per CU

constexpr int kRagged = 3;
constexpr TileCost kRaggedCost[kRagged] = {
    {64, 128, 128, 256, 4.6, 4.6, 0.734, 0.951, 0.951, 0.807, 1.38},
    {32, 64, 128, 512, 1.45, 2.96, 0.363, 0.42, 0.58, 0.429, 2.69},
    {16, 64, 128, 512, 0.96, 2.32, 0.349, 0.398, 0.531, 0.434, 3.1},
};

int pick(int64_t M, int64_t N, int64_t K, int64_t group, double* us)
{
    const bool ragged = K % 64 != 0;
    const TileCost* const cost = ragged ? kRaggedCost : kCost;
    const int count = ragged ? kRagged : kShapes;
    int best = count - 1;
    double t_best = 1e300;
    for (int i = ragged || group % 64 == 0 ? 0 : kFirstAny; i < count; ++i) {
        if (int64_t(cost[i].bm) * K > int64_t(1) << 30) continue;         // row offsets within a tile are 32-bit
        const double t = tile_time(cost[i], M, N, K);
        if (t < t_best) { t_best = t; best = i; }
    }
    if (us) *us = t_best;
    return best;
}

}  // namespace

// What the weight-streaming kernel takes (us) for more than 16 rows in one launch: m rows of a block, b blocks of 16, s slices of 512 weights, p passes of 8
// slices; w workgroups to a CU and xt tiles to a CU (as in launch_lean_rows).  A line each for groups of 256s, 128s, 64s and 32s.  Fitted, with
// the tiles' times, to 2500 calls over M = 1 .. 2048, N = 512 .. 16384, K = 512 .. 14336 and 1500 with K no multiple of 64, weights out of the caches:
// 14 % for nine in ten, and the one chosen is 0.3 % slower than the best on average, 10 % in one of a hundred.
struct StreamLine { double start, row, row_slice, per_tile[9], start_p, pass, pass_row, tile_slice, tile_pass; };
static const StreamLine& stream_line(int64_t group)
{
    static constexpr StreamLine lines[4] = {
        {3.19, 0.042, 0.006, {0, 0.14, 0.225, 0.368, 0.448, 0.711, 0.748, 0.757, 0.843}, 2.74, 0.933, 0.102, 0.062, 0.386},
        {3.23, 0.053, 0.004, {0, 0.147, 0.244, 0.399, 0.462, 0.759, 0.792, 0.841, 0.929}, 2.91, 0.873, 0.106, 0.052, 0.459},
        {3.2, 0.051, 0.004, {0, 0.164, 0.273, 0.452, 0.538, 0.88, 0.927, 1.014, 1.074}, 3.42, 0.536, 0.131, 0.102, 0.473},
        {3.42, 0.061, 0.0, {0, 0.24, 0.399, 0.69, 0.756, 1.35, 1.405, 1.505, 1.473}, 2.59, 1.093, 0.07, 0.1, 0.803},
    };
    return lines[group % 256 == 0 ? 0 : group % 128 == 0 ? 1 : group % 64 == 0 ? 2 : 3];
}
static double stream_gs_time(int64_t M, int64_t N, int64_t K, int64_t group)
{
    const StreamLine& c = stream_line(group);
    const int64_t s = (K + 511) / 512, tiles = (N + 15) / 16, b = (M + 15) / 16;
    const double m = double(M < 16 ? M : 16);
    int64_t share = 256 * (8 / (s < 8 ? s : 8)) / b;
    if (s > 8 && share < (tiles + 31) / 32) share = (tiles + 31) / 32;
    if (share < 1) share = 1;
    const int64_t groups = tiles < share ? tiles : share;
    const double w = double((groups * b + 255) / 256), xt = double((tiles + groups - 1) / groups) * w;
    const double p = double((s + 7) / 8);
    const double t = s <= 8 ? c.start + c.row * m + c.row_slice * m * double(s) * w + c.per_tile[s] * xt
                            : c.start_p + w * p * (c.pass + c.pass_row * m) + xt * (c.tile_slice * double(s) + c.tile_pass * p);
    return K % 64 != 0 ? 1.1 * t + 0.35 : t;
}

// What the plain kernel on the vector ALUs takes (us) for up to 4 rows: chunks of 1024 weights, of which a part costs as much as a whole one, in as many
// rounds as there are 200 workgroups of 16 columns; one or two columns leave wavefronts out.
static double plain_gs_time(int64_t M, int64_t N, int64_t K)
{
    const double chunks = double((K + 1023) / 1024), groups = double((N + 15) / 16);
    return 2.6 + chunks * (N <= 2 ? 1.2 + 0.3 * double(M) : 2.5) * (groups > 200.0 ? groups / 200.0 : 1.0);
}

// Tiled kernel or what would take the call without it: the weight-streaming kernel, which up to 16 rows was the fastest in all calls of the fit but a
// few of groups of 64s and 32s (by up to 7 and 15 %), or, for other groups and N, the plain kernel.  That one wins in calls of up to 4 rows alone (in none
// of 1050 calls of more; in 51 of 350 others, 1 x 1 x 5344 17.7 us tiled and 11.5, 2 x 64 x 960 5.8 and 5.2), where the tiled kernel takes 0.9 us
// less than the fit of larger calls says.  Over those 1400 calls of M = 1 .. 8192, N = 1 .. 16384, K = 16 .. 14336 the one chosen is 0.4 % slower than
// the best on average and 15 % in one of a hundred.
bool tile_gs_preferred(int64_t M, int64_t N, int64_t K, int64_t group)
{
    const bool streams = gemv_gs_supports(M, N, K, group);
    if ((M <= 16 && streams) || K < 8 || K > (int64_t(1) << 24) || M > (int64_t(1) << 24) || N > (int64_t(1) << 24)) return false;
    if (streams) {
        const KernelChoice c = tile_gs_choice(M, N, K, group);
        return c.tiled < c.stream;
    }
    if (M > 4) return true;
    double us;
    pick(M, N, K, group, &us);
    return us - 0.9 < plain_gs_time(M, N, K);
}

KernelChoice tile_gs_choice(int64_t M, int64_t N, int64_t K, int64_t group)
{
    KernelChoice c{gemv_gs_supports(M, N, K, group), 0.0, 0.0, 0.0, 0.0, 0.0};
    if (!c.streams || M <= 16) return c;
    c.stream = over_stream_launches(M, [&](int64_t m) { return stream_gs_time(m, N, K, group); });
    // In shared launches: fitted to 600 groups of 2 to 8 alike jobs of M = 17 .. 1500, N = 64 .. 8192, K = 64 .. 8192, 10 % on average.  The way chosen there
    // takes 1.1 % longer than the better one (1.6 % without the 1 us); counted as 1.15 to 1.3 times as long as in a launch of its own 9 %, up to 3.7 times.
    const StreamLine& line = stream_line(group);
    const int64_t s = (K + 511) / 512, p = (s + 7) / 8;
    constexpr double crowd[9] = {0, 1.42, 1.37, 1.19, 1.24, 1.07, 1.18, 1.06, 1.07};
    const double blocks = double((M + 15) / 16);
    c.launch = 4.42;
    c.launches = blocks / 32.0;
    const double x = blocks * double((N + 15) / 16) / 256.0;
    c.own = 1.0 + (s <= 8 ? crowd[s] * line.per_tile[s] * x : 1.08 * (line.tile_slice * double(s) + line.tile_pass * double(p)) * x + 2.44 * double(p) * c.launches);
    c.tiled = c.stream;
    // Below the fit, K < 512, both times are too long, the tiled kernel's by 36 % at K = 64 and 10 % at 448 (96 x 64 x 2912 3.7 us, streaming 4.7; 1572 x 128 x
    // 96 3.6 and 4.3).  Over 384 such calls the one chosen is 0.2 % slower than the best, 7 % in one of a hundred (without the factors 6.7 and 31 %).
    const double band = K % 64 != 0 || K >= 512 ? 1.0 : K <= 128 ? 0.76 : K <= 256 ? 0.82 : 0.92;
    if (band * (K % 64 != 0 ? tile_at_least(kRaggedCost, kRagged, K) : tile_at_least(kCost, kShapes, K)) >= c.stream) return c;
    pick(M, N, K, group, &c.tiled);
    c.tiled *= band;
    return c;
}

int tile_gs_shape(int64_t M, int64_t N, int64_t K, int64_t group) { return (K % 64 != 0 ? kRaggedShape : 0) + pick(M, N, K, group, nullptr); }

hipError_t tile_gs_init()
{
    hipError_t e = tile_prepare<T256x256>();
    if (e == hipSuccess) e = tile_prepare<T128x256>();
    if (e == hipSuccess) e = tile_prepare<T128x128>();
    if (e == hipSuccess) e = tile_prepare<T128x128any>();
    if (e == hipSuccess) e = tile_prepare<T128x64any>();
    if (e == hipSuccess) e = tile_prepare<T64x64any>();
    if (e == hipSuccess) e = tile_prepare<T32x64any>();
    if (e == hipSuccess) e = tile_prepare<R64x128>();
    if (e == hipSuccess) e = tile_prepare<R32x64>();
    if (e == hipSuccess) e = tile_prepare<R16x64>();
    return e;
}

hipError_t launch_tile_gs(const __half* x, const uint32_t* Wp, const __half* scales, int64_t group, __half* y,
                          int64_t M, int64_t N, int64_t K, hipStream_t s)
{
    TileParams p{};
    p.x = x; p.W = reinterpret_cast<const unsigned char*>(Wp); p.scales = scales; p.y = y; p.gamma = 1.f;
    p.M = int(M); p.N = int(N); p.K = int(K);
    p.row_bytes = int((K + 15) / 16 * 4);
    // a group longer than K is the one group there is
    p.group16 = int((group < K ? group : K + 15) / 16);
    const int shape = pick(M, N, K, group, nullptr);
    if (K % 64 != 0) {
        switch (shape) {
            case 0: return tile_launch<R64x128>(p, s);
            case 1: return tile_launch<R32x64>(p, s);
            default: return tile_launch<R16x64>(p, s);
        }
    }
    switch (shape) {
        case 0: return tile_launch<T256x256>(p, s);
        case 1: return tile_launch<T128x256>(p, s);
        case 2: return tile_launch<T128x128>(p, s);
        case 3: return tile_launch<T128x128any>(p, s);
        case 4: return tile_launch<T128x64any>(p, s);
        case 5: return tile_launch<T64x64any>(p, s);
        default: return tile_launch<T32x64any>(p, s);
    }
}

}  // namespace tl
