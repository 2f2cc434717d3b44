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
    {64, 128, 160, 256, 5.4, 5.4, 0.96, 0.96, 0.96, 0.6, 2.0},
    {32, 128, 160, 256, 3.7, 3.7, 0.70, 0.70, 0.70, 0.6, 2.0},
    {16, 64, 320, 256, 3.1, 3.1, 0.63, 0.63, 0.63, 0.6, 2.0},
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

// Tiled kernel or what would take the call without it.  Where K % 8 == 0 that is the weight-streaming kernel (gemv3): it
// never loses up to 16 rows.  The weight-streaming
// kernel decodes W once per 16 rows; its time (us, W in MB of packed bytes, b blocks of 16 rows): 5 + b (0.12 + 0.28 W)
// while K is one pass (4096 -> 14336: b = 4 19.0, b = 32 114.6; 4096 -> 4096: b = 32 38.2); beyond, rounds of 256
// 16-row tiles of W that take 10.4 us at K = 11008 (11008 -> 4096: b = 1 11.4, b = 2 21.6, b = 32 334).  The tiled kernel on the same: 4096 -> 14336 b = 32 57,
// 11008 -> 4096 b = 32 62, 4096 -> 4096 b = 32 26.
// Other K: the plain kernel on the vector ALUs, 3 + K / 4096 (7 + 7.5 per row, up to 4) for every 1024 workgroups of 4 x 4
// outputs (4090 -> 4099: M = 1 17.8, M = 4 39, M = 16 159, M = 37 324; 1001 -> 1024: M = 1 6.8, M = 16 13).
bool tile3_preferred(int64_t M, int64_t N, int64_t K)
{
    if ((M <= 16 && K % 8 == 0) || K < 8 || K > (int64_t(1) << 24) || M > (int64_t(1) << 24) || N > (int64_t(1) << 24)) return false;
    double us;
    pick(M, N, K, &us);
    if (K % 8 != 0) {
        const double groups = double((M + 3) / 4) * double((N + 3) / 4) / 1024.0;
        return us < 3.0 + double(K) / 4096.0 * (7.0 + 7.5 * double(M < 4 ? M : 4)) * (groups > 1.0 ? groups : 1.0);
    }
    const double w_mb = double(N) * double((K + 4) / 5) / 1.0e6;
    const double blocks = double((M + 15) / 16);
    const double rounds = double(((M + 15) / 16 * ((N + 15) / 16) + 255) / 256);
    const double t_stream = gemv3_groups(M < 4096 ? M : 4096, N, K) ? 5.0 + blocks * (0.12 + 0.28 * w_mb)
                                                                    : 1.0 + rounds * 10.4 * double(K) / 11008.0;
    return 1.08 * us < t_stream;                          // a band: near the crossover the models are within that of each other
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
