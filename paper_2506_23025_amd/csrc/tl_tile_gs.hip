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
    {256, 256, 64, 256, 6.3, 6.3, 1.205, 1.454, 1.454, 0.93, 0.5},
    {128, 256, 128, 256, 7.85, 7.85, 1.29, 1.525, 1.525, 0.91, 0.75},
    {128, 128, 128, 256, 5.6, 5.6, 0.73, 0.863, 0.863, 0.90, 1.2},
    {128, 128, 128, 256, 5.45, 5.45, 0.815, 0.932, 0.932, 0.91, 1.1},
    {128, 64, 128, 256, 4.45, 4.45, 0.415, 0.49, 0.49, 0.91, 0.95},
    {64, 64, 128, 512, 2.0, 3.8, 0.28, 0.321, 0.542, 0.42, 2.85},
    {32, 64, 128, 512, 1.4, 3.2, 0.236, 0.258, 0.407, 0.39, 2.9},
};

// K that is no multiple of 64
typedef TileCfg<kTileGs, true, 4, 2, 1, 4, 2, 4, 2, 1> R64x128;
typedef TileCfg<kTileGs, true, 2, 2, 1, 2, 4, 4, 2, 1> R32x64;      // two workgroups per CU
typedef TileCfg<kTileGs, true, 1, 2, 1, 2, 4, 4, 2, 1> R16x64;      // two workgroups per CU

constexpr int kRagged = 3;
constexpr TileCost kRaggedCost[kRagged] = {
    {64, 128, 128, 256, 4.2, 4.2, 0.83, 0.83, 0.83, 0.6, 2.0},
    {32, 64, 128, 512, 2.4, 2.4, 0.38, 0.38, 0.54, 0.6, 2.0},
    {16, 64, 128, 512, 2.1, 2.1, 0.36, 0.36, 0.53, 0.6, 2.0},
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

// What the weight-streaming kernel takes (us) for more than 16 rows, W being decoded once per b blocks of 16: t tiles of 16 output rows, s slices
// of 512 weights, p passes of 8 slices; groups that are odd multiples of 128 need every product twice.  Fitted to 2550 calls over M = 17 ..
// 2048, N = 512 .. 16384, K = 512 .. 14336: 14 % for nine in ten, 20 % with
// several passes.
static double stream_gs_time(int64_t M, int64_t N, int64_t K, int64_t group)
{
    const bool whole = group % 256 == 0;
    const int s = int((K + 511) / 512);
    const double p = double((s + 7) / 8), b = double((M + 15) / 16), launches = double(((M + 15) / 16 + 31) / 32);
    const double x = b * double((N + 15) / 16) / 256.0;
    if (s <= 8) {
        constexpr double per_whole[9] = {0, 0.132, 0.241, 0.379, 0.443, 0.644, 0.681, 0.712, 0.789};
        constexpr double per_odd[9] = {0, 0.182, 0.341, 0.615, 0.665, 1.21, 1.29, 1.35, 1.43};
        return whole ? 4.5 * launches + 0.136 * b + per_whole[s] * x : 4.95 * launches + 0.055 * b + per_odd[s] * x;
    }
    return 1.9 + 3.2 * launches * p + 0.1 * b + x * (whole ? 0.0475 * double(s) + 0.71 * p : 0.145 * double(s) + 0.77 * p);
}

// Tiled kernel or what would take the call without it: the weight-streaming kernel, which never loses up to 16 rows (over the calls of the
// fit the one chosen is 0.2 % slower than the best on average and 6 % in one of a hundred), or, for other groups, the plain kernel on the
// vector ALUs, 3 + K / 4096 (6.5 + 1.25 per row, up to 16) for every 512 workgroups of 16 x 16 outputs (us; 4096 -> 4096: M = 1
// 11.3, M = 4 14.6, M = 16 29.8, M = 37 45.8).
bool tile_gs_preferred(int64_t M, int64_t N, int64_t K, int64_t group)
{
    const bool streams = gemv_gs_supports(M, N, K, group);
    if ((M <= 16 && streams) || K < 8 || K > (int64_t(1) << 24) || M > (int64_t(1) << 24) || N > (int64_t(1) << 24)) return false;
    if (streams) {
        const KernelChoice c = tile_gs_choice(M, N, K, group);
        return c.tiled < c.stream;
    }
    double us;
    pick(M, N, K, group, &us);
    const double groups = double((M + 15) / 16) * double((N + 15) / 16) / 512.0;
    return us < 3.0 + double(K) / 4096.0 * (6.5 + 1.25 * double(M < 16 ? M : 16)) * (groups > 1.0 ? groups : 1.0);
}

KernelChoice tile_gs_choice(int64_t M, int64_t N, int64_t K, int64_t group)
{
    KernelChoice c{gemv_gs_supports(M, N, K, group), 0.0, 0.0, 0.0, 0.0, 0.0};
    if (!c.streams || M <= 16) return c;
    c.stream = stream_gs_time(M, N, K, group);
    c.launch = 4.5;
    c.launches = double((M + 15) / 16) / 32.0;
    c.fixed = c.launch * (c.launches > 1.0 ? double(int64_t(c.launches + 0.999)) : 1.0);
    c.tiled = c.stream;
    if (tile_at_least(kCost, kShapes, K) >= c.stream) return c;
    pick(M, N, K, group, &c.tiled);
    if (K > 4096) c.tiled *= 1.1;                          // the streaming kernel's time is less certain there: 20 % for nine in ten
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
