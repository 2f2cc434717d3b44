// Both 1.6-bit byte codes: instances of the tiled matrix-core kernel and the choice among them.
#include "tl_tile.hpp"

namespace tl {

namespace {

// Steps of 160 k (two sets of waves take 3 and 2 of its five 32-k blocks) or 320 k (four sets: 3, 3, 2, 2).
typedef TileCfg<kTile1p6, false, 8, 4, 1, 4, 2, 5, 3> T128x256;
typedef TileCfg<kTile1p6, false, 8, 2, 1, 4, 2, 5, 3> T128x128;
typedef TileCfg<kTile1p6, false, 4, 2, 1, 4, 2, 5, 3> T64x128;
typedef TileCfg<kTile1p6, false, 4, 2, 1, 2, 4, 10, 3> T64x64;
typedef TileCfg<kTile1p6, false, 2, 2, 1, 2, 4, 10, 3> T32x64;

constexpr int kShapes = 5;
constexpr TileCost kCost[kShapes] = {
    {128, 256, 160, 256, 9.4, 9.4, 1.64, 1.98, 1.98, 0.90, 0.5},
    {128, 128, 160, 256, 6.0, 6.0, 0.904, 1.09, 1.09, 0.88, 1.05},
    {64, 128, 160, 256, 4.0, 4.0, 0.715, 0.818, 0.818, 0.90, 1.25},
    {64, 64, 320, 256, 3.8, 3.8, 0.748, 0.88, 0.88, 0.93, 1.4},
    {32, 64, 320, 256, 2.85, 2.85, 0.631, 0.728, 0.728, 0.93, 1.45},
};

// K that is no multiple of 8
typedef TileCfg<kTile1p6, true, 4, 2, 1, 4, 2, 5, 2> R64x128;
typedef TileCfg<kTile1p6, true, 2, 2, 1, 4, 2, 5, 2> R32x128;
typedef TileCfg<kTile1p6, true, 1, 2, 1, 2, 4, 10, 2> R16x64;

constexpr int kRagged = 3;
constexpr TileCost kRaggedCost[kRagged] = {
    {64, 128, 160, 256, 4.76, 4.76, 0.847, 0.979, 0.979, 0.93, 0.92},
    {32, 128, 160, 256, 3.53, 3.53, 0.668, 0.729, 0.729, 0.93, 1.07},
    {16, 64, 320, 256, 2.88, 2.88, 0.662, 0.679, 0.679, 1.0, 1.37},
};

int pick(int64_t M, int64_t N, int64_t K, double* us)
{
    const bool ragged = K % 8 != 0;
    const TileCost* const cost = ragged ? kRaggedCost : kCost;
    const int count = ragged ? kRagged : kShapes;
    int best = count - 1;
    double t_best = 1e300;
    for (int i = 0; i < count; ++i) {
        if (int64_t(cost[i].bm) * K > int64_t(1) << 30) continue;         // row offsets within a tile are 32-bit
        const double t = tile_time(cost[i], M, N, K);
        if (t < t_best) { t_best = t; best = i; }
    }
    if (us) *us = t_best;
    return best;
}

}  // namespace

// What the weight-streaming kernel (gemv3) takes (us) for more than 16 rows, W being decoded once per b blocks of 16: t tiles of 16 output
// rows, s half slices of 64 packed bytes.  While K is one pass, workgroups of s waves share the CUs and walk runs of tiles, and the fullest
// CU sets the pace; beyond that workgroups of up to 4 tiles go in rounds of 256, each staging its rows of x.  Fitted to calls over
// M = 17 .. 2048, N = 512 .. 16384: 1100 of K = 512 .. 4800, with up to 7 half slices 1700 more and beyond one pass 1400 with weights out
// of the caches: 8 % for nine in ten calls, 10 % with several passes.  (The lines of 3 and 5 half slices had been fitted to launches of more
// workgroups than the CUs held: 13 and 15 % above what the calls take now.  Without the rows, which cost a full block 1.6 us per pass of 15
// waves, calls of 47 and 24 rows lost 13 and 11 %: 9536 -> 10688 and 8320 -> 14080 29.8 and 22.7 us tiled, 34.0 and 25.2 streaming.)
static double stream3_time(int64_t M, int64_t N, int64_t K)
{
    const int64_t tiles = (N + 15) / 16, b = (M + 15) / 16;
    const int64_t s = (((K + 4) / 5 + 15) / 16 + 3) / 4;
    if (s <= 15) {
        constexpr double start[16] = {0, 3.98, 3.94, 3.98, 3.89, 3.98, 4.14, 4.39, 3.89, 4.13, 4.22, 4.2, 4.17, 4.58, 4.73, 4.66};
        constexpr double per_tile[16] = {0, 0.114, 0.16, 0.2, 0.258, 0.339, 0.393, 0.445, 0.509, 0.611, 0.642, 0.687, 0.727, 0.83, 0.88, 0.948};
        const int64_t share = 256 * gemv3_per_cu(int(s)) / b, groups = tiles < share ? tiles : (share < 1 ? 1 : share);
        return start[s] + per_tile[s] * double((tiles + groups - 1) / groups) * double((b * groups + 255) / 256);
    }
    int64_t groups = tiles < 256 ? tiles : 256, per_group = (tiles + groups - 1) / groups;
    if (per_group > 4) { per_group = 4; groups = (tiles + 3) / 4; }
    const double rounds = double((b * groups + 255) / 256), passes = double((s + 14) / 15), T = double(per_group);
    return 1.66 + rounds * (1.53 + 0.35 * passes + double(s) / 15.0 * (T * (0.67 + 0.07 * T) + 1.57 / 16.0 * double(M) / double(b)));
}

// Tiled or weight-streaming kernel, which never loses up to 16 rows: where K % 8 == 0, over 3200 calls of K up to 4800 the one chosen is 0.15 %
// slower than the best on average and 6 % in one of a hundred, over 1800 with longer K 0.1 and 4 %.
bool tile3_preferred(int64_t M, int64_t N, int64_t K)
{
    if (M <= 16 || K < 8 || K > (int64_t(1) << 24) || M > (int64_t(1) << 24) || N > (int64_t(1) << 24)) return false;
    const KernelChoice c = tile3_choice(M, N, K);
    return c.tiled < c.stream;
}

KernelChoice tile3_choice(int64_t M, int64_t N, int64_t K)
{
    KernelChoice c{gemv3_groups(M, N, K), 0.0, 0.0, 0.0, 0.0, 0.0};
    if (M <= 16 || K < 8 || K > (int64_t(1) << 24) || M > (int64_t(1) << 24) || N > (int64_t(1) << 24)) return c;
    c.stream = over_stream_launches(M, [&](int64_t m) { return stream3_time(m, N, K); });
    if (c.streams) {
        // In shared launches: fitted to 480 groups of 2 to 8 alike jobs of M = 17 .. 1500, N = 64 .. 8192, K = 64 .. 4800, 7 % on average.  The way chosen there takes
        // 0.7 % longer than the better one; counted as in a launch of its own 13 %, up to 2.8 times.
        constexpr double per_tile[16] = {0, 0.304, 0.242, 0.24, 0.263, 0.336, 0.395, 0.444, 0.543, 0.647, 0.74, 0.76, 0.8, 0.929, 0.974, 1.161};
        const double blocks = double((M + 15) / 16);
        c.launch = 4.63;
        c.launches = blocks / 32.0;
        c.own = blocks * double((N + 15) / 16) / 256.0 * per_tile[(((K + 4) / 5 + 15) / 16 + 3) / 4];
    }
    c.tiled = c.stream;
    if (K % 8 != 0) {
        if (K < 64) {                                      // below the fit: tiles, as far as anything was measured a third either way
            c.streams = false;
            c.tiled = 0.0;
            return c;
        }
        // Rows of x that start anywhere cost the streaming kernel 5 %, 10 with several passes, and 0.3 us.  Fitted with the three tiles' times to 1250
        // calls over M = 17 .. 2048, N = 512 .. 16384, K = 64 .. 14336; on 1250 others the one chosen is 0.18 % slower than the best and 7 % in
        // one of a hundred.
        c.tiled = c.stream = c.stream * (c.streams ? 1.05 : 1.1) + 0.3 * double((M + kStreamRows - 1) / kStreamRows);
        if (tile_at_least(kRaggedCost, kRagged, K) < c.stream) pick(M, N, K, &c.tiled);
        return c;
    }
    // One step of K and less: the tiles' times, fitted from K = 512 on, are 5 to 10 % too long.  Over 1143 such calls the one chosen is 0.4 %
    // slower than the best (without the factor 1.4 %, with 0.84 for K up to 960 2.6 % here and 5.6 % up to there).
    const double band = K <= 320 ? 0.92 : 1.0;
    if (band * tile_at_least(kCost, kShapes, K) >= c.stream) return c;
    pick(M, N, K, &c.tiled);
    c.tiled *= band;
    return c;
}

int tile3_shape(int64_t M, int64_t N, int64_t K) { return (K % 8 != 0 ? kRaggedShape : 0) + pick(M, N, K, nullptr); }

hipError_t tile3_init()
{
    hipError_t e = tile_prepare<T128x256>();
    if (e == hipSuccess) e = tile_prepare<T128x128>();
    if (e == hipSuccess) e = tile_prepare<T64x128>();
    if (e == hipSuccess) e = tile_prepare<T64x64>();
    if (e == hipSuccess) e = tile_prepare<T32x64>();
    if (e == hipSuccess) e = tile_prepare<R64x128>();
    if (e == hipSuccess) e = tile_prepare<R32x128>();
    if (e == hipSuccess) e = tile_prepare<R16x64>();
    return e;
}

hipError_t launch_tile3(const __half* x, const uint8_t* Wp, int64_t stride, float gamma, __half* y,
                        int64_t M, int64_t N, int64_t K, bool fx, hipStream_t s)
{
    TileParams p{};
    p.x = x; p.W = Wp; p.y = y; p.gamma = gamma;
    p.M = int(M); p.N = int(N); p.K = int(K);
    p.row_bytes = int(stride);
    p.group16 = 1;
    p.fx = fx;
    const int shape = pick(M, N, K, nullptr);
    if (K % 8 != 0) {
        switch (shape) {
            case 0: return tile_launch<R64x128>(p, s);
            case 1: return tile_launch<R32x128>(p, s);
            default: return tile_launch<R16x64>(p, s);
        }
    }
    switch (shape) {
        case 0: return tile_launch<T128x256>(p, s);
        case 1: return tile_launch<T128x128>(p, s);
        case 2: return tile_launch<T64x128>(p, s);
        case 3: return tile_launch<T64x64>(p, s);
        default: return tile_launch<T32x64>(p, s);
    }
}

}  // namespace tl
