// 2-bit words, one gamma: instances of the tiled matrix-core kernel and the choice among them.
#include "tl_tile.hpp"

namespace tl {

namespace {

// waves x fragments -> tile; the larger the tile, the fewer bytes cross LDS and L2 per matrix instruction.
typedef TileCfg<kTile2Bit, false, 8, 4, 2, 4, 1, 2, 4> T256x256;    // steps of 64
typedef TileCfg<kTile2Bit, false, 8, 4, 1, 4, 2, 4, 4> T128x256;    // steps of 128 from here on: sets of waves share K
typedef TileCfg<kTile2Bit, false, 8, 2, 1, 4, 2, 4, 4> T128x128;
typedef TileCfg<kTile2Bit, false, 8, 2, 1, 2, 4, 4, 4> T128x64;
typedef TileCfg<kTile2Bit, false, 4, 2, 1, 2, 4, 4, 4> T64x64;      // two workgroups per CU
typedef TileCfg<kTile2Bit, false, 2, 2, 1, 2, 4, 4, 4> T32x64;      // two workgroups per CU

constexpr int kShapes = 6;
constexpr TileCost kCost[kShapes] = {
    {256, 256, 64, 256, 6.2, 6.2, 1.07, 1.32, 1.32, 0.87, 0.5},
    {128, 256, 128, 256, 7.3, 7.3, 1.17, 1.43, 1.43, 0.84, 0.5},
    {128, 128, 128, 256, 4.9, 4.9, 0.656, 0.786, 0.786, 0.88, 0.9},
    {128, 64, 128, 256, 4.3, 4.3, 0.336, 0.43, 0.43, 0.92, 1.15},
    {64, 64, 128, 512, 2.25, 3.35, 0.229, 0.273, 0.475, 0.43, 2.1},
    {32, 64, 128, 512, 1.35, 2.65, 0.191, 0.213, 0.318, 0.43, 2.4},
};

// Row offsets within a tile are 32-bit: tiles of 256 rows up to K = 2^22, of 128 up to 2^23.
inline bool fits(const TileCost& c, int64_t K) { return int64_t(c.bm) * K <= int64_t(1) << 30; }

int pick(int64_t M, int64_t N, int64_t K, double* us)
{
    int best = kShapes - 2;
    double t_best = 1e300;
    for (int i = 0; i < kShapes; ++i) {
        if (!fits(kCost[i], K)) continue;
        const double t = tile_time(kCost[i], M, N, K);
        if (t < t_best) { t_best = t; best = i; }
    }
    if (us) *us = t_best;
    return best;
}

// K that is no multiple of 64
typedef TileCfg<kTile2Bit, true, 8, 2, 1, 4, 2, 4, 2> R128x128;     // steps of 128
typedef TileCfg<kTile2Bit, true, 4, 2, 1, 4, 2, 4, 2> R64x128;
typedef TileCfg<kTile2Bit, true, 2, 2, 1, 2, 4, 4, 2> R32x64;       // two workgroups per CU
typedef TileCfg<kTile2Bit, true, 1, 2, 1, 1, 8, 8, 2> R16x32;       // steps of 256, two workgroups per CU

constexpr int kRagged = 4;
constexpr TileCost kRaggedCost[kRagged] = {
    {128, 128, 128, 256, 4.19, 5.56, 1.064, 1.297, 1.249, 0.82, 2.75},
    {64, 128, 128, 256, 3.05, 3.47, 0.573, 0.685, 0.643, 0.87, 1.51},
    {32, 64, 128, 512, 0.94, 2.01, 0.319, 0.356, 0.464, 0.43, 2.14},
    {16, 32, 256, 512, 0.50, 1.55, 0.323, 0.363, 0.478, 0.50, 2.34},
};

int pick_ragged(int64_t M, int64_t N, int64_t K, double* us)
{
    int best = kRagged - 1;
    double t_best = 1e300;
    for (int i = 0; i < kRagged; ++i) {
        if (!fits(kRaggedCost[i], K)) continue;
        const double t = tile_time(kRaggedCost[i], M, N, K);
        if (t < t_best) { t_best = t; best = i; }
    }
    if (us) *us = t_best;
    return best;
}

}  // namespace

// Where the streaming kernel cannot run (K below 64, more than 4096 rows): in none of 249 calls of K = 8 .. 63, M = 1 .. 20000 and of longer K, M = 4097 .. 20000, over
// N = 1 .. 16384, was the plain kernel on the vector ALUs ahead (at K = 8 .. 63 it takes 1.25 to 1.5 times as long up to 4 rows, 2 to 16 times
// beyond): what it pays for is whole chunks of 1024 weights.
bool tile_ragged_preferred(int64_t M, int64_t N, int64_t K)
{
    return K >= 8 && K <= (int64_t(1) << 24) && M <= (int64_t(1) << 24) && N <= (int64_t(1) << 24);
}

// What the weight-streaming kernel takes (us) for K that is no multiple of 64: m rows of a block, b blocks of 16, s slices of 512 weights; w workgroups
// to a CU and xt tiles to a CU.
static double stream_any_time(int64_t M, int64_t N, int64_t K)
{
    const int64_t s = (K + 511) / 512, tiles = (N + 15) / 16, b = (M + 15) / 16;
    const double m = double(M < 16 ? M : 16);
    if (s > 8 && s <= 32 && tiles * b <= 512) return 2.77 + 0.019 * m + double(s) * (0.009 + 0.018 * m + 0.124 * (tiles * b <= 256 ? 1.0 : 2.0));
    int64_t share = 256 * (8 / (s < 8 ? s : 8)) / b;
    if (s > 8 && share < (tiles + 31) / 32) share = (tiles + 31) / 32;
    if (share < 1) share = 1;
    const int64_t groups = tiles < share ? tiles : share;
    const double w = double((groups * b + 255) / 256), xt = double((tiles + groups - 1) / groups) * w;
    constexpr double per_tile[9] = {0, 0.139, 0.207, 0.341, 0.368, 0.604, 0.67, 0.724, 0.752};
    if (s <= 8) return 2.73 + 0.052 * m + 0.013 * m * double(s) * w + per_tile[s] * xt;
    const double p = double((s + 7) / 8);
    return 4.33 + w * p * (0.911 + 0.178 * m) + xt * (0.049 * double(s) + 0.344 * p);
}

// What a job of more than 16 rows adds to shared launches of that form, which have one workgroup per CU: fitted to 320 groups of 2 to 8 alike jobs of
// M = 17 .. 1500, N = 64 .. 8192, K = 64 .. 8192, 10 % on average.  The way chosen there takes 1.0 % longer than the better one; counted as in a
// launch of its own 9 %, up to 2.8 times.
double stream_any_share(int64_t M, int64_t N, int64_t K)
{
    constexpr double per_tile[9] = {0, 0.58, 0.51, 0.55, 0.585, 0.72, 0.9, 0.865, 0.97};
    const int64_t s = (K + 511) / 512, p = (s + 7) / 8;
    const double blocks = double((M + 15) / 16), x = blocks * double((N + 15) / 16) / 256.0;
    return s <= 8 ? per_tile[s] * x : 0.133 * double(s) * x + 3.08 * double(p) * blocks / 32.0;
}

// Tiled or weight-streaming kernel for K that is no multiple of 64.  Fitted, with the tiles' times, to 1300 calls of M = 17 .. 2048 and 600 of fewer rows, N = 512
// .. 16384, K = 64 .. 14336, weights out of the caches; on as many others the one chosen is 0.8 % slower than the best (13 % in one of a
// hundred) and 0.2 % (6 %).  Up to 4 rows the streaming kernel was the fastest in all.
KernelChoice tile_ragged_choice(int64_t M, int64_t N, int64_t K)
{
    KernelChoice c{gemv_any_supports(M, N, K), 0.0, 0.0, 0.0, 0.0, 0.0};
    if (!c.streams || M <= 4) return c;
    c.stream = stream_any_time(M, N, K);
    c.launch = 4.2;
    c.launches = double((M + 15) / 16) / 32.0;
    c.own = M <= 16 ? c.stream - 3.0 : stream_any_share(M, N, K);
    c.tiled = c.stream;
    if (tile_at_least(kRaggedCost, kRagged, K) < c.stream) pick_ragged(M, N, K, &c.tiled);
    return c;
}

hipError_t launch_tile_ragged(const __half* x, const uint32_t* Wp, float gamma, __half* y,
                              int64_t M, int64_t N, int64_t K, hipStream_t s)
{
    TileParams p{};
    p.x = x; p.W = reinterpret_cast<const unsigned char*>(Wp); p.y = y; p.gamma = gamma;
    p.M = int(M); p.N = int(N); p.K = int(K);
    p.row_bytes = int((K + 15) / 16 * 4);
    p.group16 = 1;
    switch (pick_ragged(M, N, K, nullptr)) {
        case 0: return tile_launch<R128x128>(p, s);
        case 1: return tile_launch<R64x128>(p, s);
        case 2: return tile_launch<R32x64>(p, s);
        default: return tile_launch<R16x32>(p, s);
    }
}

bool mfma_supports(int64_t M, int64_t N, int64_t K)
{
    return M >= 1 && N >= 1 && K >= 64 && (K % 64) == 0 && K <= (int64_t(1) << 24) &&
           M <= (int64_t(1) << 24) && N <= (int64_t(1) << 24);
}

double mfma_at_least(int64_t K) { return tile_at_least(kCost, kShapes, K); }

double mfma_time(int64_t M, int64_t N, int64_t K)
{
    double us;
    pick(M, N, K, &us);
    return us;
}

int mfma_shape(int64_t M, int64_t N, int64_t K) { return pick(M, N, K, nullptr); }
int tile_ragged_shape(int64_t M, int64_t N, int64_t K) { return kRaggedShape + pick_ragged(M, N, K, nullptr); }

hipError_t mfma_init()
{
    hipError_t e = tile_prepare<T256x256>();
    if (e == hipSuccess) e = tile_prepare<T128x256>();
    if (e == hipSuccess) e = tile_prepare<T128x128>();
    if (e == hipSuccess) e = tile_prepare<T128x64>();
    if (e == hipSuccess) e = tile_prepare<T64x64>();
    if (e == hipSuccess) e = tile_prepare<T32x64>();
    if (e == hipSuccess) e = tile_prepare<R128x128>();
    if (e == hipSuccess) e = tile_prepare<R64x128>();
    if (e == hipSuccess) e = tile_prepare<R32x64>();
    if (e == hipSuccess) e = tile_prepare<R16x32>();
    return e;
}

hipError_t launch_mfma(const __half* x, const uint32_t* Wp, float gamma, __half* y,
                       int64_t M, int64_t N, int64_t K, hipStream_t s)
{
    TileParams p{};
    p.x = x; p.W = reinterpret_cast<const unsigned char*>(Wp); p.y = y; p.gamma = gamma;
    p.M = int(M); p.N = int(N); p.K = int(K);
    p.row_bytes = int(K / 4);
    p.group16 = 1;
    switch (pick(M, N, K, nullptr)) {
        case 0: return tile_launch<T256x256>(p, s);
        case 1: return tile_launch<T128x256>(p, s);
        case 2: return tile_launch<T128x128>(p, s);
        case 3: return tile_launch<T128x64>(p, s);
        case 4: return tile_launch<T64x64>(p, s);
        default: return tile_launch<T32x64>(p, s);
    }
}

}  // namespace tl
