// C-ABI entry points that touch the device: argument checks, kernel choice, launch.
#include "tl_internal.hpp"

#include <cmath>

namespace tl {

float half_bits_to_float(uint16_t h)
{
    const int sign = (h >> 15) & 1;
    const int e = (h >> 10) & 0x1F;
    const int f = h & 0x3FF;
    float v;
    if (e == 0) v = std::ldexp(static_cast<float>(f), -24);
    else if (e == 31) v = f ? NAN : INFINITY;
    else v = std::ldexp(static_cast<float>(1024 + f), e - 25);
    return sign ? -v : v;
}

namespace {

inline bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

inline bool dims_ok(int64_t M, int64_t N, int64_t K)
{
    const int64_t lim = int64_t(1) << 31;
    return M >= 1 && N >= 1 && K >= 1 && M < lim && N < lim && K < lim &&
           M * N < (int64_t(1) << 40) && N * K < (int64_t(1) << 42) && M * K < (int64_t(1) << 40);
}

inline tl_status from_hip(hipError_t e) { return e == hipSuccess ? TL_OK : TL_ERR_HIP; }

// What the small-M kernel takes (us) for more than 16 rows: t tiles of 16 output rows, b blocks of 16 or 32 activation rows, s slices of
// 512 weights, p passes of 8 slices.  In one pass a block costs its activations and a share of every tile, which depends on s
// alone (a workgroup has s waves, and as many more workgroups fit as 8 / s allows), not on the bytes of W.  Fitted with the
// tiled kernel's times (see TileCost): 10 % for nine in ten calls, 15 % with several passes.  The one line that is older is that of up to
// 16 blocks of 32 rows with 8 slices: it is 0.8 of the time for most N, and right where t b is a multiple of 256.
inline double small_m_time(int64_t M, int64_t N, int64_t K)
{
    const int s = int((K + 511) / 512);
    const double t = double((N + 15) / 16);
    const double p = double((s + 7) / 8);
    if (tl::gemv_two_blocks(M, N, K)) {
        const int64_t blocks = (M + 31) / 32;
        const double b = double(blocks);
        if (s > 8) {
            // launches of at most 4096 tiles
            const int64_t tiles = (N + 15) / 16, cap = tiles >= 4096 ? 1 : 4096 / tiles;
            return 5.16 * p * double((blocks + cap - 1) / cap) + 0.51 * b + b * t / 256.0 * (0.09 * double(s) + 0.49 * p);
        }
        if (s == 8 && blocks <= 16) return 4.0 + b * (0.31 + 0.2 * double(N) * double(K) / 4.0e6);
        constexpr double per_tile[9] = {0, 0, 0.334, 0.63, 0.53, 0.82, 0.87, 0.95, 1.02};
        return 5.8 * double((blocks + 31) / 32) + 0.148 * b + per_tile[s] * b * t / 256.0;
    }
    const int64_t blocks = (M + 15) / 16;
    const double b = double(blocks), launches = double((blocks + 31) / 32);
    if (s <= 8) {
        constexpr double per_tile[9] = {0, 0.114, 0.185, 0.30, 0.32, 0.56, 0.57, 0.62, 0.62};
        return 4.5 * launches + 0.173 * b + per_tile[s] * b * t / 256.0;
    }
    if (b * t >= 512.0) return 1.2 + 2.44 * launches * p + 0.133 * b + b * t / 256.0 * (0.059 * double(s) + 0.39 * p);
    if (N % 16 == 0) return 3.0 + 1.3 * p + 0.115 * double(s) * b * t / 256.0;
    return 1.7 + 3.2 * p + 0.06 * b + 0.166 * double(s) * b * t / 256.0;
}

// The same for a call that is one launch of the lean kernel (gemv_rows_form): b blocks of 16 rows, w workgroups and xt tiles to a CU (as in launch_lean_rows).
// Fitted to 860 calls over M = 17 .. 2048, N = 512 .. 16384, K = 512 .. 2048 with every alternative timed, weights out of the caches; of those the one
// chosen is 0.6 % slower than the best on average (before that launch was there 1.8 % slower than the best of the others).
inline double rows_form_time(int64_t M, int64_t N, int64_t K)
{
    const int64_t s = (K + 511) / 512, tiles = N / 16, b = (M + 15) / 16;
    int64_t share = 256 * (8 / s) / b;
    if (share < 1) share = 1;
    const int64_t groups = tiles < share ? tiles : share;
    const double w = double((groups * b + 255) / 256), xt = double((tiles + groups - 1) / groups) * w;
    constexpr double per_tile[5] = {0, 0.141, 0.21, 0.343, 0.385};
    return 3.86 + 0.048 * double(s) * w + per_tile[s] * xt;
}

// Small-M kernel or tiled matrix-core kernel, when both can run the shape.  A band rather than the bare comparison decides, since machines
// differ by several percent (the same library: 18.3 and 19.6 us for the same launch): beyond 16 rows the small-M kernel keeps a shape
// unless the models put the tiled kernel ahead by more than 7 %.  Over 1740 calls of K beyond 2048 the one chosen is 1.3 % slower than the best on
// average and 20 % in one of a hundred; with the constants before these fits 4.6 to 6.5 % and a factor of 2 (14701 x 2304 at M = 1295 141 us for 93).
inline KernelChoice choice_2bit(int64_t M, int64_t N, int64_t K)
{
    if (K % 64 != 0) return tile_ragged_choice(M, N, K);
    KernelChoice c{gemv_supports(M, N, K), 0.0, 0.0, 0.0, 0.0, 0.0};
    if (!c.streams || M <= 16 || !mfma_supports(M, N, K)) return c;
    const double apart = small_m_time(M, N, K);
    const bool two_blocks = gemv_two_blocks(M, N, K);
    const double passes = double((K + 4095) / 4096);
    if (passes == 1.0) c.launch = two_blocks ? 5.0 : 4.5;
    else if (!two_blocks && double((M + 15) / 16) * double((N + 15) / 16) >= 512.0) c.launch = 4.5;
    c.launches = double((M + (two_blocks ? 31 : 15)) / (two_blocks ? 32 : 16)) / 32.0;
    // Less 1 us, by which a call of its own between others is longer than alone (ties went wrong by 2 us of 29 and 4 of 58 without; over 160 groups of 2 to 8
    // alike jobs of M = 17 .. 1500 and K up to 8192 the way chosen takes 0.5 % longer than the better one, without 1.6 %).
    c.own = apart - c.launch * (c.launches > 1.0 ? double(int64_t(c.launches + 0.999)) : 1.0) - 1.0;
    c.stream = gemv_rows_form(M, N, K) ? rows_form_time(M, N, K) : apart;
    c.tiled = c.stream;
    // The one launch's time is the better known.  Below its fit, K < 512, both times are too long, the tiled kernel's the more (24 x 128 x 128 2.7 us
    // against 3.9, the one launch 3.4 against 4.05): over 253 such calls the one chosen is 0.2 % slower than the best, 6 % in one of a
    // hundred (with 1.03 2.2 and 23 %, with 0.9 0.4 and 11 %).
    const double band = !gemv_rows_form(M, N, K) ? 1.07 : K < 512 ? 0.95 : 1.03;
    if (band * mfma_at_least(K) <= c.stream) c.tiled = band * mfma_time(M, N, K);
    return c;
}

// The same for a job of a call in which some K is no multiple of 64 (any_k), and which shares those jobs' launches.
inline KernelChoice choice_2bit_among(int64_t M, int64_t N, int64_t K, bool any_k)
{
    KernelChoice c = choice_2bit(M, N, K);
    if (any_k && K % 64 == 0 && c.stream > 0.0 && gemv_any_supports(M, N, K) && !gemv_two_blocks(M, N, K)) {
        const double share = stream_any_share(M, N, K);
        if (share > c.own) c.own = share;
    }
    return c;
}

// Which kernel takes a call of its own.
enum class Runs { plain, streams, tiled };

inline Runs runs_2bit(int64_t M, int64_t N, int64_t K)
{
    const KernelChoice c = choice_2bit(M, N, K);
    if (c.streams && !(c.tiled < c.stream)) return Runs::streams;
    if (K % 64 != 0) return c.streams || tile_ragged_preferred(M, N, K) ? Runs::tiled : Runs::plain;
    return mfma_supports(M, N, K) ? Runs::tiled : Runs::plain;
}

inline Runs runs_1p6(int64_t M, int64_t N, int64_t K)
{
    if (tile3_preferred(M, N, K)) return Runs::tiled;
    return gemv3_supports(M < kStreamRows ? M : kStreamRows, N, K) ? Runs::streams : Runs::plain;
}

inline Runs runs_gs(int64_t M, int64_t N, int64_t K, int64_t group)
{
    if (tile_gs_preferred(M, N, K, group)) return Runs::tiled;
    return gemv_gs_supports(M, N, K, group) ? Runs::streams : Runs::plain;
}

// Enqueues the jobs of a grouped call, 64 at a time: `fuse` adds one to the shared launches, `flush` sends those, `single` calls one by itself.
template <class Job, class Choice, class Fuse, class Flush, class Single>
tl_status run_grouped(const Job* jobs, int64_t count, Choice&& choice, Fuse&& fuse, Flush&& flush, Single&& single)
{
    for (int64_t first = 0; first < count; first += 64) {
        const int n = int(count - first < 64 ? count - first : 64);
        KernelChoice c[64];
        bool alone[64];
        for (int j = 0; j < n; ++j) c[j] = choice(jobs[first + j]);
        choose_grouped(c, n, alone);
        for (int j = 0; j < n; ++j) {
            if (c[j].streams && !alone[j]) {
                fuse(jobs[first + j]);
            } else {
                const tl_status st = single(jobs[first + j]);
                if (st != TL_OK) return st;
            }
        }
        const tl_status st = flush();
        if (st != TL_OK) return st;
    }
    return TL_OK;
}

}  // namespace
}  // namespace tl

extern "C" {

tl_status tl_unpack_dev(tl_format fmt, const void* packed, int64_t N, int64_t K, int8_t* W_out,
                        void* stream)
{
    if (!packed || !W_out) return TL_ERR_NULL;
    if (!tl::dims_ok(1, N, K)) return TL_ERR_SHAPE;
    hipStream_t s = static_cast<hipStream_t>(stream);
    if (fmt == TL_FMT_2BIT)
        return tl::from_hip(tl::launch_unpack2(static_cast<const uint32_t*>(packed), N, K, W_out, s));
    if (fmt == TL_FMT_1P6BIT || fmt == TL_FMT_1P6BIT_FX)
        return tl::from_hip(tl::launch_unpack3(static_cast<const uint8_t*>(packed), N, K,
                                               static_cast<int64_t>(tl_row_stride_bytes(fmt, K)),
                                               W_out, fmt == TL_FMT_1P6BIT_FX, s));
    return TL_ERR_UNSUPPORTED;
}

tl_path tl_ternary_gemm_which(int64_t M, int64_t N, int64_t K)
{
    if (!tl::dims_ok(M, N, K)) return TL_PATH_AUTO;
    if (K % 64 != 0) return TL_PATH_GENERIC;
    switch (tl::runs_2bit(M, N, K)) {
        case tl::Runs::streams: return TL_PATH_GEMV;
        case tl::Runs::tiled: return TL_PATH_MFMA;
        default: return TL_PATH_GENERIC;
    }
}

tl_status tl_ternary_gemm_path(const void* x, const void* Wpacked, uint16_t gamma_fp16_bits, void* y,
                               int64_t M, int64_t N, int64_t K, void* stream, tl_path path)
{
    if (!x || !Wpacked || !y) return TL_ERR_NULL;
    if (!tl::dims_ok(M, N, K)) return TL_ERR_SHAPE;
    if (!tl::aligned16(x) || !tl::aligned16(Wpacked) || !tl::aligned16(y)) return TL_ERR_ALIGN;
    const float gamma = tl::half_bits_to_float(gamma_fp16_bits);
    hipStream_t s = static_cast<hipStream_t>(stream);
    const __half* xh = static_cast<const __half*>(x);
    const uint32_t* wp = static_cast<const uint32_t*>(Wpacked);
    __half* yh = static_cast<__half*>(y);

    if (path == TL_PATH_AUTO) {
        path = tl_ternary_gemm_which(M, N, K);
        // shapes of the any-shape path: the streaming or the tiled kernel's form for such K
        if (path == TL_PATH_GENERIC && K % 64 != 0) {
            const tl::Runs r = tl::runs_2bit(M, N, K);
            if (r == tl::Runs::streams) return tl::from_hip(tl::launch_gemv(xh, wp, gamma, yh, M, N, K, s));
            if (r == tl::Runs::tiled) return tl::from_hip(tl::launch_tile_ragged(xh, wp, gamma, yh, M, N, K, s));
        }
    }
    switch (path) {
        case TL_PATH_GENERIC:
            return tl::from_hip(tl::launch_gemm_generic(xh, wp, gamma, yh, M, N, K, s));
        case TL_PATH_GEMV:
            if (!tl::gemv_supports(M, N, K)) return TL_ERR_UNSUPPORTED;
            return tl::from_hip(tl::launch_gemv(xh, wp, gamma, yh, M, N, K, s));
        case TL_PATH_MFMA:
            if (!tl::mfma_supports(M, N, K)) return TL_ERR_UNSUPPORTED;
            return tl::from_hip(tl::launch_mfma(xh, wp, gamma, yh, M, N, K, s));
        default:
            return TL_ERR_UNSUPPORTED;
    }
}

tl_status tl_ternary_gemm(const void* x, const void* Wpacked, uint16_t gamma_fp16_bits, void* y,
                          int64_t M, int64_t N, int64_t K, void* stream)
{
    return tl_ternary_gemm_path(x, Wpacked, gamma_fp16_bits, y, M, N, K, stream, TL_PATH_AUTO);
}

tl_status tl_ternary_gemm_grouped(const tl_gemm_job* jobs, int64_t count, void* stream)
{
    if (count == 0) return TL_OK;
    if (!jobs) return TL_ERR_NULL;
    if (count < 0 || count > 4096) return TL_ERR_SHAPE;
    for (int64_t i = 0; i < count; ++i) {
        const tl_gemm_job& j = jobs[i];
        if (!j.x || !j.Wpacked || !j.y) return TL_ERR_NULL;
        if (!tl::dims_ok(j.M, j.N, j.K)) return TL_ERR_SHAPE;
        if (!tl::aligned16(j.x) || !tl::aligned16(j.Wpacked) || !tl::aligned16(j.y)) return TL_ERR_ALIGN;
    }
    hipStream_t s = static_cast<hipStream_t>(stream);
    // Jobs the small-M kernel takes share launches; the others, and those with so many rows that a call of their own is faster, go one by one.
    tl::GemmDesc fused[64];
    int nf = 0;
    bool any_k = false;
    for (int64_t i = 0; i < count; ++i) any_k = any_k || jobs[i].K % 64 != 0;
    return tl::run_grouped(
        jobs, count, [any_k](const tl_gemm_job& j) { return tl::choice_2bit_among(j.M, j.N, j.K, any_k); },
        [&](const tl_gemm_job& j) {
            fused[nf++] = tl::GemmDesc{static_cast<const __half*>(j.x), static_cast<const uint32_t*>(j.Wpacked),
                                       static_cast<__half*>(j.y), tl::half_bits_to_float(j.gamma_fp16_bits), j.M, j.N, j.K};
        },
        [&] {
            const hipError_t e = nf ? tl::launch_gemv_jobs(fused, nf, s) : hipSuccess;
            nf = 0;
            return tl::from_hip(e);
        },
        [&](const tl_gemm_job& j) { return tl_ternary_gemm(j.x, j.Wpacked, j.gamma_fp16_bits, j.y, j.M, j.N, j.K, stream); });
}

namespace {

tl_status gemm_1p6(const void* x, const void* Wpacked, uint16_t gamma_fp16_bits, void* y,
                   int64_t M, int64_t N, int64_t K, void* stream, bool fx)
{
    if (!x || !Wpacked || !y) return TL_ERR_NULL;
    if (!tl::dims_ok(M, N, K)) return TL_ERR_SHAPE;
    if (!tl::aligned16(x) || !tl::aligned16(Wpacked) || !tl::aligned16(y)) return TL_ERR_ALIGN;
    const float gamma = tl::half_bits_to_float(gamma_fp16_bits);
    const int64_t stride = static_cast<int64_t>(tl_row_stride_bytes(TL_FMT_1P6BIT, K));
    hipStream_t s = static_cast<hipStream_t>(stream);
    const tl::Runs r = tl::runs_1p6(M, N, K);
    if (r == tl::Runs::tiled)
        return tl::from_hip(tl::launch_tile3(static_cast<const __half*>(x), static_cast<const uint8_t*>(Wpacked), stride,
                                             gamma, static_cast<__half*>(y), M, N, K, fx, s));
    if (r == tl::Runs::streams) {
        // more rows than one launch takes: one launch per kStreamRows rows
        const __half* xh = static_cast<const __half*>(x);
        __half* yh = static_cast<__half*>(y);
        for (int64_t m0 = 0; m0 < M; m0 += tl::kStreamRows) {
            const int64_t rows = M - m0 < tl::kStreamRows ? M - m0 : tl::kStreamRows;
            const hipError_t e = tl::launch_gemv3(xh + m0 * K, static_cast<const uint8_t*>(Wpacked), stride, gamma,
                                                  yh + m0 * N, rows, N, K, fx, s);
            if (e != hipSuccess) return tl::from_hip(e);
        }
        return TL_OK;
    }
    return tl::from_hip(tl::launch_gemm3_generic(static_cast<const __half*>(x),
                                                 static_cast<const uint8_t*>(Wpacked), stride, gamma,
                                                 static_cast<__half*>(y), M, N, K, fx, s));
}

}  // namespace

tl_status tl_ternary_gemm_1p6(const void* x, const void* Wpacked, uint16_t gamma_fp16_bits, void* y,
                              int64_t M, int64_t N, int64_t K, void* stream)
{
    return gemm_1p6(x, Wpacked, gamma_fp16_bits, y, M, N, K, stream, false);
}

tl_status tl_ternary_gemm_1p6_fx(const void* x, const void* Wpacked, uint16_t gamma_fp16_bits, void* y,
                                 int64_t M, int64_t N, int64_t K, void* stream)
{
    return gemm_1p6(x, Wpacked, gamma_fp16_bits, y, M, N, K, stream, true);
}

tl_status tl_ternary_gemm_gs(const void* x, const void* Wpacked, const void* scales, int64_t group,
                             void* y, int64_t M, int64_t N, int64_t K, void* stream)
{
    if (!x || !Wpacked || !scales || !y) return TL_ERR_NULL;
    if (!tl::dims_ok(M, N, K)) return TL_ERR_SHAPE;
    if (group < 16 || group % 16 != 0) return TL_ERR_SHAPE;
    if (!tl::aligned16(x) || !tl::aligned16(Wpacked) || !tl::aligned16(scales) || !tl::aligned16(y)) return TL_ERR_ALIGN;
    hipStream_t s = static_cast<hipStream_t>(stream);
    const __half* xh = static_cast<const __half*>(x);
    const uint32_t* wp = static_cast<const uint32_t*>(Wpacked);
    const __half* sh = static_cast<const __half*>(scales);
    __half* yh = static_cast<__half*>(y);
    const tl::Runs r = tl::runs_gs(M, N, K, group);
    if (r == tl::Runs::tiled) return tl::from_hip(tl::launch_tile_gs(xh, wp, sh, group, yh, M, N, K, s));
    if (r == tl::Runs::streams) {
        const hipError_t e = tl::launch_gemv_gs(xh, wp, sh, group, yh, M, N, K, s);
        if (e != hipErrorInvalidValue) return tl::from_hip(e);
        (void)hipGetLastError();                 // nothing was launched: the plain kernel takes it
    }
    return tl::from_hip(tl::launch_gemm_generic_gs(xh, wp, sh, group, yh, M, N, K, s));
}

tl_status tl_ternary_gemm_1p6_grouped(const tl_gemm_job* jobs, int64_t count, tl_format format, void* stream)
{
    if (count == 0) return TL_OK;
    if (!jobs) return TL_ERR_NULL;
    if (count < 0 || count > 4096) return TL_ERR_SHAPE;
    if (format != TL_FMT_1P6BIT && format != TL_FMT_1P6BIT_FX) return TL_ERR_VALUE;
    for (int64_t i = 0; i < count; ++i) {
        const tl_gemm_job& j = jobs[i];
        if (!j.x || !j.Wpacked || !j.y) return TL_ERR_NULL;
        if (!tl::dims_ok(j.M, j.N, j.K)) return TL_ERR_SHAPE;
        if (!tl::aligned16(j.x) || !tl::aligned16(j.Wpacked) || !tl::aligned16(j.y)) return TL_ERR_ALIGN;
    }
    const bool fx = format == TL_FMT_1P6BIT_FX;
    hipStream_t s = static_cast<hipStream_t>(stream);
    // Jobs whose K fits one pass of the stream form share launches; the others, and those with so many rows that a call of
    // their own is faster, go one by one.  So does one that shares with nobody and would fill several launches: a call of its own is one, however many
    // rows (1080 x 62 x 274 13.0 us in three, 4.7 tiled).  Of fewer rows the shared launch's records are the faster way in (376 x 192 x 2112
    // replayed 4.7 us and 5.5 as a call of its own).
    tl::Gemm3Desc fused[64];
    const tl_gemm_job* last = nullptr;
    int nf = 0;
    return tl::run_grouped(
        jobs, count,
        [](const tl_gemm_job& j) { return tl::tile3_choice(j.M, j.N, j.K); },
        [&](const tl_gemm_job& j) {
            last = &j;
            fused[nf++] = tl::Gemm3Desc{static_cast<const __half*>(j.x), static_cast<const uint8_t*>(j.Wpacked),
                                        static_cast<__half*>(j.y), tl::half_bits_to_float(j.gamma_fp16_bits),
                                        j.M, j.N, j.K, static_cast<int64_t>(tl_row_stride_bytes(TL_FMT_1P6BIT, j.K))};
        },
        [&] {
            const int n = nf;
            nf = 0;
            if (n == 1 && last->M > tl::kMaxBlocks3 * 16) return gemm_1p6(last->x, last->Wpacked, last->gamma_fp16_bits, last->y, last->M, last->N, last->K, stream, fx);
            return tl::from_hip(n ? tl::launch_gemv3_jobs(fused, n, fx, s) : hipSuccess);
        },
        [&](const tl_gemm_job& j) { return gemm_1p6(j.x, j.Wpacked, j.gamma_fp16_bits, j.y, j.M, j.N, j.K, stream, fx); });
}

tl_status tl_ternary_gemm_gs_grouped(const tl_gemm_gs_job* jobs, int64_t count, void* stream)
{
    if (count == 0) return TL_OK;
    if (!jobs) return TL_ERR_NULL;
    if (count < 0 || count > 4096) return TL_ERR_SHAPE;
    for (int64_t i = 0; i < count; ++i) {
        const tl_gemm_gs_job& j = jobs[i];
        if (!j.x || !j.Wpacked || !j.scales || !j.y) return TL_ERR_NULL;
        if (!tl::dims_ok(j.M, j.N, j.K)) return TL_ERR_SHAPE;
        if (j.group < 16 || j.group % 16 != 0) return TL_ERR_SHAPE;
        if (!tl::aligned16(j.x) || !tl::aligned16(j.Wpacked) || !tl::aligned16(j.scales) || !tl::aligned16(j.y)) return TL_ERR_ALIGN;
    }
    hipStream_t s = static_cast<hipStream_t>(stream);
    // Jobs the weight-streaming kernel takes share launches; the others, and those with so many rows that a call of
    // their own is faster, go one by one.
    tl::GemmGsDesc fused[64];
    int nf = 0;
    return tl::run_grouped(
        jobs, count, [](const tl_gemm_gs_job& j) { return tl::tile_gs_choice(j.M, j.N, j.K, j.group); },
        [&](const tl_gemm_gs_job& j) {
            fused[nf++] = tl::GemmGsDesc{static_cast<const __half*>(j.x), static_cast<const uint32_t*>(j.Wpacked),
                                         static_cast<const __half*>(j.scales), static_cast<__half*>(j.y), j.M, j.N, j.K, j.group};
        },
        [&] {
            const hipError_t e = nf ? tl::launch_gemv_gs_jobs(fused, nf, s) : hipSuccess;
            nf = 0;
            return tl::from_hip(e);
        },
        [&](const tl_gemm_gs_job& j) { return tl_ternary_gemm_gs(j.x, j.Wpacked, j.scales, j.group, j.y, j.M, j.N, j.K, stream); });
}

// For the tests, which assert what they run; not part of the interface.  form: 0 2-bit words, 1 a 1.6-bit code, 2 group scales, 3 2-bit words on
// TL_PATH_MFMA.  The kernel that a call of its own runs in: 0 plain, 1 streaming, 2 tiled.
__attribute__((visibility("default"))) int tl_internal_runs(int form, int64_t M, int64_t N, int64_t K, int64_t group)
{
    switch (form) {
        case 0: return int(tl::runs_2bit(M, N, K));
        case 1: return int(tl::runs_1p6(M, N, K));
        case 2: return int(tl::runs_gs(M, N, K, group));
        case 3: return tl::mfma_supports(M, N, K) ? 2 : -1;
        default: return -1;
    }
}

// Likewise: the tiled kernel's instance for such a call, or -1 where another kernel takes it.
__attribute__((visibility("default"))) int tl_internal_tile_instance(int form, int64_t M, int64_t N, int64_t K, int64_t group)
{
    if (tl_internal_runs(form, M, N, K, group) != int(tl::Runs::tiled)) return -1;
    switch (form) {
        case 1: return tl::tile3_shape(M, N, K);
        case 2: return tl::tile_gs_shape(M, N, K, group);
        default: return K % 64 != 0 ? tl::tile_ragged_shape(M, N, K) : tl::mfma_shape(M, N, K);
    }
}

// Likewise: per job of a grouped call (M, N, K, group each) 0 where it shares the streaming kernel's launches, 1 and 2 where it runs as a call of its own
// though it could, tiled and streaming, and -1 where that kernel cannot take it.
__attribute__((visibility("default"))) void tl_internal_grouped_tiled(int form, const int64_t* jobs, int count, int* out)
{
    tl::KernelChoice c[64];
    bool alone[64];
    if (count > 64) count = 64;
    bool any_k = false;
    for (int j = 0; j < count; ++j) any_k = any_k || jobs[4 * j + 2] % 64 != 0;
    for (int j = 0; j < count; ++j) {
        const int64_t M = jobs[4 * j], N = jobs[4 * j + 1], K = jobs[4 * j + 2], group = jobs[4 * j + 3];
        c[j] = form == 0 ? tl::choice_2bit_among(M, N, K, any_k) : (form == 1 ? tl::tile3_choice(M, N, K) : tl::tile_gs_choice(M, N, K, group));
    }
    tl::choose_grouped(c, count, alone);
    for (int j = 0; j < count; ++j) out[j] = !c[j].streams ? -1 : !alone[j] ? 0 : c[j].tiled < c[j].stream ? 1 : 2;
}

// Likewise: jobs_by_table.
__attribute__((visibility("default"))) int tl_internal_jobs_by_table(int count, int one_pass, int records, int several, int64_t w_bytes, int captured)
{
    return tl::jobs_by_table(count, one_pass != 0, records != 0, several != 0, w_bytes, captured != 0) ? 1 : 0;
}

// Likewise: workgroups of `waves` waves that a launch of the 1.6-bit streaming kernel puts on a CU, and the LDS that one is given.
__attribute__((visibility("default"))) int tl_internal_stream3_per_cu(int waves, int* lds) { return tl::gemv3_per_cu(waves, lds); }

tl_status tl_init(void)
{
    hipError_t e = tl::gemv_init();
    if (e == hipSuccess) e = tl::gemv3_init();
    if (e == hipSuccess) e = tl::mfma_init();
    if (e == hipSuccess) e = tl::tile3_init();
    if (e == hipSuccess) e = tl::tile_gs_init();
    return tl::from_hip(e);
}

tl_status tl_probe_copy(void* dst, const void* src, size_t bytes, void* stream)
{
    if (!dst || !src) return TL_ERR_NULL;
    if (bytes % 16 != 0) return TL_ERR_SHAPE;
    if (!tl::aligned16(dst) || !tl::aligned16(src)) return TL_ERR_ALIGN;
    return tl::from_hip(tl::launch_probe_copy(dst, src, bytes, static_cast<hipStream_t>(stream)));
}

tl_status tl_probe_read(const void* src, size_t bytes, void* sink, void* stream)
{
    if (!src || !sink) return TL_ERR_NULL;
    if (bytes % 16 != 0) return TL_ERR_SHAPE;
    if (!tl::aligned16(src) || (reinterpret_cast<uintptr_t>(sink) & 3u)) return TL_ERR_ALIGN;
    return tl::from_hip(tl::launch_probe_read(src, bytes, sink, static_cast<hipStream_t>(stream)));
}

tl_status tl_probe_mfma(const void* x, int64_t x_elems, const void* Wpacked, int64_t w_words, int64_t iters,
                        void* sink, double* flops, void* stream)
{
    if (!x || !Wpacked || !sink) return TL_ERR_NULL;
    if (x_elems < 1 || w_words < 1 || iters < 1 || iters > (int64_t(1) << 24)) return TL_ERR_SHAPE;
    if ((reinterpret_cast<uintptr_t>(x) & 1u) || (reinterpret_cast<uintptr_t>(Wpacked) & 3u) ||
        (reinterpret_cast<uintptr_t>(sink) & 3u)) return TL_ERR_ALIGN;
    return tl::from_hip(tl::launch_probe_mfma(static_cast<const __half*>(x), x_elems, static_cast<const uint32_t*>(Wpacked),
                                              w_words, iters, static_cast<float*>(sink), flops, static_cast<hipStream_t>(stream)));
}

}  // extern "C"
