// Weight-streaming small-M kernel for the 2-bit format (decode batches, M <= 16 per pass).
//
// The result it computes is App. B "Inference" of the paper, Y = X (gamma What)^T, with the
// Sec. 3.1 decode d = ((b >> 2j) & 3) - 1 done in registers.  How it is organised is ours:
//
//  * One workgroup owns a set of 16-row tiles of W; wave w of the group owns the K-slice
//    [512 (w + NW p), 512 (w + NW p) + 512) in pass p.  A wave therefore keeps its part of
//    the activations in registers (64 VGPRs per pass, laid out as MFMA B operands) and only
//    the packed weights stream: every byte of W is read exactly once, in full 128-byte
//    lines (8 adjacent lanes x dwordx4), non-temporally.
//  * The contraction runs on v_mfma_f32_16x16x32_f16 with W as the 16-row operand and the
//    (at most 16) activation rows as the 16 columns, so the cost per weight does not grow
//    with M.  Coalesced loads give a lane 16 bytes of ONE row; the MFMA wants lane
//    (i, g) to hold row i.  The 2 KB tile slice is turned through wave-private LDS
//    (ds_write_b128 / ds_read_b128, XOR-swizzled, no barrier: a wave only reads what it
//    wrote itself).
//  * Decode costs 10 to 11 VALU operations per 16 weights.  `word & (3 << 2j | 3 << (2j+16))`
//    leaves two codes in the mantissa fields of an fp16 pair, i.e. the subnormal numbers
//    c * 4^j * 2^-24 (gfx950 MFMA does not flush fp16 subnormals).  The matrix core aligns
//    products by their exponent FIELDS, so a code low in the mantissa loses accuracy
//    (measured: ~2^-17 relative at j = 0, none at j >= 3).  Shifted copies of the word therefore
//    bring every code to j in {2, 3, 4}: the stream and lean kernels use the word as loaded and
//    two copies (<< 4, >> 6: 2 shifts + 8 ANDs per word), the general kernel three copies
//    (<< 4, >> 2, >> 8: 3 shifts + 8 ANDs).  Products of
//    different j carry different power-of-two factors, so they go to three accumulators
//    that are combined once per tile: sum_j 2^(24-2j) acc_j = sum_k x_k c_k.  With
//    c = w + 1 the result is sum_k x_k c_k - sum_k x_k; the second sum comes from one more
//    group of MFMAs per wave whose 16-row operand is a constant, and seeds the accumulator.
//  * Split-K partial tiles of the NW waves are added in a fixed order through LDS, scaled
//    by gamma, rounded to fp16 (RNE) and stored.  No atomics: results are deterministic.
//  * One launch can carry up to 32 independent jobs (a job = one matrix and at most 16, in
//    one variant 32, activation rows); a workgroup finds its job from its index.
//  * Four forms.  The stream form (gemv_stream_kernel: K up to 8 slices per pass) gives a wave
//    one slice for the whole kernel and a workgroup a run of consecutive tiles of one job, so
//    activations are staged once and only weights move afterwards.  The lean form
//    (gemv_lean_kernel) is the stream form cut down to the decode shapes (K the same number of
//    slices in every job or, in a second copy, several passes over K; one block of 16 rows, one
//    gamma, N a multiple of 16) and is what those launches run; its further copies take group
//    scales, any K and N, and many rows of short K.  The
//    long-K form (gemv_longk_kernel) takes lone calls with 4096 < K <= 16384 whose workgroups
//    get one or two tiles each: a wave walks its up to four slices with the next one's data
//    already in flight.  The general form (gemv_kernel) loops a wave over slices and a
//    workgroup over items of any job; it takes the calls with K > 4096 that are too small
//    for the stream form's passes to pay and that the long-K form does not cover (K > 16384,
//    N not a multiple of 16, more than 512 tiles).
#include "tl_internal.hpp"
#include "tl_deal.hpp"

#include <atomic>
#include <cstddef>
#include <type_traits>

namespace tl {

namespace {

constexpr int kTMax = 4;          // tiles per work item
constexpr int kSliceK = 512;      // K elements a wave owns per pass
constexpr int kWaveLds = 16384;   // bytes of LDS per wave: 16 activation rows x 1 KB
constexpr int kMaxJobs = 32;      // jobs per launch (the table is 2.7 KB of kernel arguments)

struct GemvJob {                  // 80 bytes, lives in the kernel argument segment
    const __half* x;              // first activation row of this 16-row block
    const uint32_t* W;
    __half* y;                    // first output row of this block
    float gamma;
    int Mrem;                     // 1..16 activation rows (stream form with two row blocks: 1..32)
    int N, K;
    int tiles;                    // ceil(N / 16)
    int items;                    // general form: work items of this job, ceil(tiles / T)
    int slices;                   // ceil(K / 512)
    int mr;                       // general form: staged rows, the power of two >= Mrem
    int run, plus;                // stream form: tiles per workgroup, and how many of the job's first workgroups take one more
    const __half* scales;         // per-group scales [K / group][N] (kernels with GS), else unused
    int hpg;                      // per-group scales: scale units of a slice per group
    int reserved;
};

struct GemvBatch {
    int count;
    int total_items;
    int red_off;                  // byte offset in LDS of the split-K reduction area
    int pad;
    int item0[kMaxJobs];          // first work item of job j; INT_MAX for unused entries
    GemvJob job[kMaxJobs];
};

// s_waitcnt immediate for "vmcnt <= n" only (gfx9 layout: vmcnt in bits 3:0 and 15:14,
// expcnt 6:4 and lgkmcnt 11:8 left at their maxima, i.e. not waited for).
constexpr int vmcnt_imm(int n)
{
    return (n & 0xF) | ((n >> 4) << 14) | (0x7 << 4) | (0xF << 8);
}

__device__ __forceinline__ f16x8 as_f16x8(u32x4 v)
{
    return __builtin_bit_cast(f16x8, v);
}

// What a workgroup needs to know about one work item; every member is wave-uniform.
struct ItemCtx {
    const unsigned char* Wb;
    const unsigned char* xb;
    __half* y;
    float gamma;
    int Mrem, MR;
    int N, K;
    uint32_t row_bytes;           // bytes per packed row
    int chunks;                   // 64-weight (16-byte) chunks per row
    int tiles, items, idx;        // tile t of the item is idx + t * items
    int slices;
};

// The job table of a launch, one job per lane (lanes 0 .. kMaxJobs - 1), read from the kernel argument
// segment with vector loads: every workgroup needs one entry chosen by its index, and a
// scalar look-up would be two dependent trips to memory before the first weight is requested.
struct JobTable {
    uint32_t d[20];               // the 20 dwords of GemvJob
    int item0;
};

__device__ __forceinline__ JobTable load_table(int lane)
{
    typedef const __attribute__((address_space(4))) unsigned char* kptr;
    kptr ka = (kptr)__builtin_amdgcn_kernarg_segment_ptr();     // GemvBatch is the only argument
    const int k = lane & (kMaxJobs - 1);
    JobTable r;
    r.item0 = 0x7fffffff;
#pragma unroll
    for (int i = 0; i < 20; ++i) r.d[i] = 0u;
    // only lanes 0 .. kMaxJobs - 1 load (the entries are read with v_readlane from those lanes): half
    // of the addresses for the CU's address path, which all eight waves go through at once
    if (lane < kMaxJobs) {
        r.item0 = *(const __attribute__((address_space(4))) int*)(ka + offsetof(GemvBatch, item0) + 4 * k);
        const __attribute__((address_space(4))) u32x4* jp =
            (const __attribute__((address_space(4))) u32x4*)(ka + offsetof(GemvBatch, job) + sizeof(GemvJob) * k);
#pragma unroll
        for (int i = 0; i < 5; ++i) {
            const u32x4 q = jp[i];
            r.d[4 * i] = q[0]; r.d[4 * i + 1] = q[1]; r.d[4 * i + 2] = q[2]; r.d[4 * i + 3] = q[3];
        }
    }
    return r;
}

// Work item g -> its job (the last one whose first item is <= g) and position in it.
__device__ __forceinline__ ItemCtx load_item(const JobTable& tb, int g)
{
    const unsigned long long m = __builtin_amdgcn_ballot_w64(g >= tb.item0) & ((1ull << kMaxJobs) - 1);
    const int ji = __builtin_popcountll(m) - 1;
    uint32_t f[20];
#pragma unroll
    for (int i = 0; i < 19; ++i) f[i] = __builtin_amdgcn_readlane(tb.d[i], ji);
    const int item0 = __builtin_amdgcn_readlane(tb.item0, ji);
    ItemCtx c;
    c.xb = reinterpret_cast<const unsigned char*>(uintptr_t(f[0]) | (uintptr_t(f[1]) << 32));
    c.Wb = reinterpret_cast<const unsigned char*>(uintptr_t(f[2]) | (uintptr_t(f[3]) << 32));
    c.y = reinterpret_cast<__half*>(uintptr_t(f[4]) | (uintptr_t(f[5]) << 32));
    c.gamma = __builtin_bit_cast(float, f[6]);
    c.Mrem = int(f[7]);
    c.N = int(f[8]); c.K = int(f[9]);
    c.row_bytes = f[9] >> 2;
    c.chunks = int(f[9] >> 6);
    c.tiles = int(f[10]); c.items = int(f[11]); c.idx = g - item0;
    c.slices = int(f[12]);
    c.MR = int(f[13]);
    return c;
}

static_assert(sizeof(GemvJob) == 80 && offsetof(GemvJob, gamma) == 24 && offsetof(GemvJob, mr) == 52 &&
              offsetof(GemvJob, run) == 56 && offsetof(GemvJob, scales) == 64 && offsetof(GemvJob, hpg) == 72,
              "load_item decodes GemvJob by dword position");

// T: tiles per work item; MULTI: the launch carries more than one job.
// A workgroup takes the items blockIdx.x, blockIdx.x + gridDim.x, ...
template <int T, bool MULTI>
__global__ void __launch_bounds__(512)
gemv_kernel(GemvBatch b)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char lds_raw[];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int NW = blockDim.x >> 6;
    unsigned char* const my_lds = lds_raw + wave * kWaveLds;

    // ---- coalesced load mapping: 8 lanes per 128-byte line, 8 rows per instruction ----
    const int lr = lane >> 3;                  // row within the half tile
    const int lc = lane & 7;                   // chunk within the slice
    // ---- MFMA mapping: lane (i, g) = (row / activation column, k group) -----------------
    const int mi = lane & 15;
    const int mg = lane >> 4;

    // LDS offsets (bytes, relative to my_lds); immediates add the row / tile / half part
    const uint32_t ww_off = uint32_t(lr) * 128u + (uint32_t(lc ^ lr) << 4);
    const uint32_t wr_off0 = uint32_t(mi) * 128u + (uint32_t((mg) ^ (mi & 7)) << 4);
    const uint32_t wr_off1 = uint32_t(mi) * 128u + (uint32_t((4 + mg) ^ (mi & 7)) << 4);

    u32x4 wreg[T][2];
    auto issue_w = [&](const ItemCtx& c, int t, int slice) {
        int tile = c.idx + t * c.items;
        if (tile >= c.tiles) tile = c.tiles - 1;           // loaded again, never used
        int chunk = slice * 8 + lc;
        if (chunk >= c.chunks) chunk = 0;                  // multiplied by zero activations
        const unsigned char* tb = c.Wb + size_t(tile) * 16u * c.row_bytes;
        uint32_t off0 = uint32_t(lr) * c.row_bytes + uint32_t(chunk) * 16u;
        uint32_t off1 = off0 + 8u * c.row_bytes;
        if ((c.N & 15) != 0 && tile == c.tiles - 1) {      // scalar branch: rows past N read row N-1
            const int last = c.N - 1 - tile * 16;
            off0 = uint32_t(lr < last ? lr : last) * c.row_bytes + uint32_t(chunk) * 16u;
            off1 = uint32_t(lr + 8 < last ? lr + 8 : last) * c.row_bytes + uint32_t(chunk) * 16u;
        }
        // the pointers were put together from table registers: say that they are global
        typedef const __attribute__((address_space(1))) u32x4* gptr;
        wreg[t][0] = __builtin_nontemporal_load((gptr)(tb + off0));
        wreg[t][1] = __builtin_nontemporal_load((gptr)(tb + off1));
    };

    // Activation rows go straight from global memory into the LDS staging area (LDS-DMA, no
    // registers): one instruction per staged row, lane l fetches the 16-byte piece
    // l ^ (r & 7) of the slice and the hardware drops it at slot l, which is the swizzled
    // layout the operand set-up reads.  Rows past Mrem repeat row Mrem-1; lanes past K
    // store zeros instead (their weights are whatever chunk 0 holds).
    auto issue_x = [&](const ItemCtx& c, int slice) {
        for (int r = 0; r < c.MR; ++r) {
            const int rr = r < c.Mrem ? r : c.Mrem - 1;
            const int kx = slice * kSliceK + ((lane ^ (r & 7)) << 3);
            if (kx < c.K) {
                __builtin_amdgcn_global_load_lds(
                    (const __attribute__((address_space(1))) void*)(c.xb + size_t(rr) * c.K * 2 + uint32_t(kx) * 2u),
                    (__attribute__((address_space(3))) void*)(my_lds + r * 1024),
                    16, 0, 0);
            } else {
                *reinterpret_cast<u32x4*>(my_lds + r * 1024 + (uint32_t(lane) << 4)) = u32x4{0u, 0u, 0u, 0u};
            }
        }
    };

    // One pass of a wave: 512 k of the T tiles of an item.  FIRST (a compile-time tag) marks
    // the very first pass of the workgroup, whose activations were requested before its
    // weights; that copy of the body runs straight from the kernel entry, so the compiler's
    // wait counts in it are exact and tile t is decoded as soon as its own two loads have
    // arrived.  Every other pass starts with all of its loads complete.
    auto do_pass = [&](auto first_tag, const ItemCtx& cur, const ItemCtx& nxt, bool pre, int slice,
                       f32x4 (&part)[T]) {
        constexpr bool FIRST = decltype(first_tag)::value;
        // The compiler does not track LDS-DMA, so wait by hand.  First pass: until only the
        // 2T weight loads issued after the activation rows are outstanding (loads of a wave
        // return in order).  Later passes: weights were requested first, so for all.
        if constexpr (FIRST) __builtin_amdgcn_s_waitcnt(vmcnt_imm(2 * T));
        else __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));
        const bool more = (slice + NW) < cur.slices;

        const int xrow = mi & (cur.MR - 1);                // staged activation row of this lane's column
        const uint32_t xr_off = uint32_t(xrow) * 1024u + uint32_t(mg) * 128u;
        const uint32_t sw = uint32_t(xrow & 7);
        // ---------------- activations of this slice -> MFMA B registers --------------------
        // staging layout: row r, 16-byte piece P at slot P ^ (r & 7)
        // breg[h][wd][e]: (x[k], x[k + 8]) with k = slice0 + 64 (4h + g) + 16 wd + e
        uint32_t breg[2][4][8];
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int wd = 0; wd < 4; ++wd) {
                const u32x4 lo = *reinterpret_cast<const u32x4*>(
                    my_lds + xr_off + h * 512 + ((uint32_t(2 * wd) ^ sw) << 4));
                const u32x4 hi = *reinterpret_cast<const u32x4*>(
                    my_lds + xr_off + h * 512 + ((uint32_t(2 * wd + 1) ^ sw) << 4));
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    breg[h][wd][2 * r] = __builtin_amdgcn_perm(hi[r], lo[r], 0x05040100u);
                    breg[h][wd][2 * r + 1] = __builtin_amdgcn_perm(hi[r], lo[r], 0x07060302u);
                }
            }
        // nsx[r] = -2^-20 sum_k x[m][k] over the slice, in the layout of an accumulator:
        // an MFMA whose 16-row operand is the constant -2^-20 in every position.
        f32x4 nsx = f32x4{0.f, 0.f, 0.f, 0.f};
        {
            const uint32_t c = 0x80108010u;               // fp16 pair of -2^-20 (subnormal 0x0010, sign set)
            const u32x4 a = u32x4{c, c, c, c};
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const u32x4 bb = u32x4{breg[h][0][e], breg[h][1][e], breg[h][2][e], breg[h][3][e]};
                    nsx = __builtin_amdgcn_mfma_f32_16x16x32_f16(as_f16x8(a), as_f16x8(bb), nsx, 0, 0, 0);
                }
        }
        // ---------------- per tile: turn through LDS, decode, MFMA ---------------------------
        // The staging rows are dead once breg is built, so region t (2 KB) reuses them; LDS
        // operations of one wave execute in order.
#pragma unroll
        for (int t = 0; t < T; ++t) {
            unsigned char* const reg_t = my_lds + t * 2048;
            *reinterpret_cast<u32x4*>(reg_t + ww_off) = wreg[t][0];
            *reinterpret_cast<u32x4*>(reg_t + 1024 + ww_off) = wreg[t][1];
            if (more) issue_w(cur, t, slice + NW);         // refill for the next pass
            else if (pre) issue_w(nxt, t, wave);           // or for the next item
            if (cur.idx + t * cur.items < cur.tiles) {     // scalar: tiles past the end are skipped
                // acc[0] starts from -2^-20 sum x: with the 2^20 below it carries the "-1" of c = w + 1
                f32x4 acc[3] = {nsx, f32x4{0.f, 0.f, 0.f, 0.f}, f32x4{0.f, 0.f, 0.f, 0.f}};
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const u32x4 wv = *reinterpret_cast<const u32x4*>(reg_t + (h ? wr_off1 : wr_off0));
                    // element e of each half-word is moved to mantissa bits 4..9 (position
                    // class 2, 3 or 4): e = 0..2 by << 4, e = 3..5 by >> 2, e = 6..7 by >> 8
                    const u32x4 sh[3] = {wv << 4, wv >> 2, wv >> 8};
#pragma unroll
                    for (int e = 0; e < 8; ++e) {
                        const int j = e % 3;                        // accumulator: class j + 2
                        const uint32_t mask = 0x00300030u << (2 * j);
                        const u32x4 a = sh[e / 3] & mask;
                        const u32x4 bb = u32x4{breg[h][0][e], breg[h][1][e], breg[h][2][e], breg[h][3][e]};
                        acc[j] = __builtin_amdgcn_mfma_f32_16x16x32_f16(as_f16x8(a), as_f16x8(bb), acc[j], 0, 0, 0);
                    }
                }
                // fp16 bits c << (2j + 4) are the subnormal c 4^(j+2) 2^-24: undo with 2^(20 - 2j)
                part[t] += acc[0] * 1048576.f + acc[1] * 262144.f + acc[2] * 65536.f;
            }
        }
        // The staging rows share LDS with the tile regions, so the next activations can only
        // be fetched once the last tile has been read; the next pass waits for them.
        if (more) issue_x(cur, slice + NW);
        else if (pre) issue_x(nxt, wave);
    };

    // Split-K reduction across the waves and output.  Layout [t][wave][lane] of f32x4 in LDS.
    // A workgroup with a single item reuses the staging space (red_off = 0); otherwise the
    // area lies behind it, because the next item's activations are already arriving there.
    // The first barrier also keeps this item's partial sums from overtaking a wave that
    // still reads the previous ones.
    // The barriers wait for LDS traffic only (s_waitcnt lgkmcnt(0); s_barrier): the next item's
    // weights and activations stay in flight across them, which __syncthreads would drain.
    auto lds_barrier = [&]() {
        __builtin_amdgcn_s_waitcnt(0xF | (0x3 << 14) | (0x7 << 4));
        __builtin_amdgcn_s_barrier();
    };
    auto epilogue = [&](const ItemCtx& cur, const f32x4 (&part)[T]) {
        lds_barrier();
        f32x4* red = reinterpret_cast<f32x4*>(lds_raw + b.red_off);
#pragma unroll
        for (int t = 0; t < T; ++t) red[(t * NW + wave) * 64 + lane] = part[t];
        lds_barrier();
        const float gamma = cur.gamma;
        for (int o = threadIdx.x; o < T * 64; o += blockDim.x) {
            const int t = o >> 6;
            const int l = o & 63;
            const int tile = cur.idx + t * cur.items;
            if (tile >= cur.tiles) continue;
            f32x4 v[8];
#pragma unroll
            for (int w = 0; w < 8; ++w)                     // all reads in flight, then a fixed-order sum
                v[w] = (w < NW) ? red[(t * NW + w) * 64 + l] : f32x4{0.f, 0.f, 0.f, 0.f};
            const f32x4 s = ((v[0] + v[1]) + (v[2] + v[3])) + ((v[4] + v[5]) + (v[6] + v[7]));
            const int n = tile * 16 + 4 * (l >> 4);
            if ((l & 15) < cur.Mrem) {
                typedef __attribute__((address_space(1))) __half* gh_ptr;
                gh_ptr dst = (gh_ptr)(cur.y + size_t(l & 15) * cur.N + n);
                if (n + 3 < cur.N && (cur.N & 3) == 0) {    // four consecutive n: one 8-byte store
                    const f16x2 lo = {(_Float16)(gamma * s[0]), (_Float16)(gamma * s[1])};
                    const f16x2 hi = {(_Float16)(gamma * s[2]), (_Float16)(gamma * s[3])};
                    *(__attribute__((address_space(1))) u32x2*)dst =
                        u32x2{__builtin_bit_cast(uint32_t, lo), __builtin_bit_cast(uint32_t, hi)};
                } else {
#pragma unroll
                    for (int r = 0; r < 4; ++r)
                        if (n + r < cur.N) *(__attribute__((address_space(1))) _Float16*)(dst + r) = (_Float16)(gamma * s[r]);
                }
            }
        }
    };

    int g = blockIdx.x;
    // A launch of one job reads it with scalar loads at fixed offsets (one trip to memory,
    // nothing depends on a look-up); several jobs go through the table in registers.
    JobTable table;
    if constexpr (MULTI) table = load_table(lane);
    auto get_item = [&](int gi) -> ItemCtx {
        if constexpr (MULTI) {
            return load_item(table, gi);
        } else {
            const GemvJob& J = b.job[0];
            ItemCtx c;
            c.xb = reinterpret_cast<const unsigned char*>(J.x);
            c.Wb = reinterpret_cast<const unsigned char*>(J.W);
            c.y = J.y;
            c.gamma = J.gamma;
            c.Mrem = J.Mrem; c.MR = J.mr;
            c.N = J.N; c.K = J.K;
            c.row_bytes = uint32_t(J.K) >> 2;
            c.chunks = J.K >> 6;
            c.tiles = J.tiles; c.items = J.items; c.idx = gi;
            c.slices = J.slices;
            return c;
        }
    };
    ItemCtx cur = get_item(g);
    // Activations go first: they are short L2 hits, and the loads of one wave return in
    // order, so the weight stream queued behind them overlaps the operand set-up.
    if (wave < cur.slices) {
        issue_x(cur, wave);
#pragma unroll
        for (int t = 0; t < T; ++t) issue_w(cur, t, wave);
    }
    // The next item of this workgroup: its first weights and activations are requested
    // during the last pass over the current one, so HBM stays busy through the epilogue.
    int gn = g + int(gridDim.x);
    bool has_next = gn < b.total_items;
    ItemCtx nxt = get_item(has_next ? gn : g);
    bool pre = has_next && wave < nxt.slices;

    f32x4 part[T];
#pragma unroll
    for (int t = 0; t < T; ++t) part[t] = f32x4{0.f, 0.f, 0.f, 0.f};
    int slice = wave;
    if (slice < cur.slices) {
        do_pass(std::true_type{}, cur, nxt, pre, slice, part);
        slice += NW;
    }
    for (;;) {
        for (; slice < cur.slices; slice += NW)             // wave-uniform trip count
            do_pass(std::false_type{}, cur, nxt, pre, slice, part);
        if (wave >= cur.slices && pre) {                    // a wave with no slice of this item
            issue_x(nxt, wave);
#pragma unroll
            for (int t = 0; t < T; ++t) issue_w(nxt, t, wave);
        }
        epilogue(cur, part);
        if (!has_next) break;
        cur = nxt;
        g = gn;
        gn = g + int(gridDim.x);
        has_next = gn < b.total_items;
        nxt = get_item(has_next ? gn : g);
        pre = has_next && wave < nxt.slices;
#pragma unroll
        for (int t = 0; t < T; ++t) part[t] = f32x4{0.f, 0.f, 0.f, 0.f};
        slice = wave;
    }
}

// LDS per wave of the stream form: 16 KB of activation staging, or two tile regions and two
// sets of T partial-sum tiles, whichever is more.
constexpr int stream_wave_lds(int T)
{
    return 4096 + 2 * T * 1024 > kWaveLds ? 4096 + 2 * T * 1024 : kWaveLds;
}

// ------------------------------------------------------------------------------------------
// Stream form of the kernel, for launches in which every job has K <= 512 * (waves per group):
// wave w owns K slice w for good, so its activations are fetched and turned into MFMA operands
// once, and all that moves afterwards is the weight stream.  A workgroup serves one job (its
// index picks the job; GemvBatch::item0[j] is the first workgroup of job j) and walks a run of
// consecutive tiles of it, T at a time (GemvJob::run, plus: tiles per workgroup, and how many of the
// job's first workgroups take one more).  While item i is decoded the loads of item i + 1 are in flight,
// each tile waits only for its own two loads, and there is one LDS-only barrier per item.
// The loop body holds nothing but weight loads and the output stores, which is what keeps the
// compiler's wait counts exact; the last item is a second copy of the body without refills.
// PASSES: some job of the launch has K longer than the waves' slices together.
// NB: blocks of 16 activation rows a job may have (1 or 2).  With two, every decoded weight
// operand feeds two MFMAs, one per block: the decode, which is what limits the kernel, is paid
// once for 32 rows.  With PASSES the kept sums take 1 KB per tile and row block.
template <int T, bool MULTI, bool PASSES, int NB>
__global__ void __launch_bounds__(512)
gemv_stream_kernel(GemvBatch b)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char lds_raw[];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int NW = blockDim.x >> 6;
    // LDS of a wave: activation rows (16 KB) while the operands are built; afterwards two tile
    // regions at 0 and 2 KB, and from 4 KB two sets of T NB partial-sum tiles (1 KB each).
    constexpr int kStride = stream_wave_lds(T * NB);
    unsigned char* const my_lds = lds_raw + wave * kStride;

    const int lr = lane >> 3, lc = lane & 7;   // load mapping: row of the half tile, chunk of the slice
    const int mi = lane & 15, mg = lane >> 4;  // MFMA mapping: row / activation column, k group
    const uint32_t ww_off = uint32_t(lr) * 128u + (uint32_t(lc ^ lr) << 4);
    const uint32_t wr_off0 = uint32_t(mi) * 128u + (uint32_t((mg) ^ (mi & 7)) << 4);
    const uint32_t wr_off1 = uint32_t(mi) * 128u + (uint32_t((4 + mg) ^ (mi & 7)) << 4);

    // ---- this workgroup's job and run of items ----------------------------------------------
    ItemCtx J;
    int ipg, plus;
    if constexpr (MULTI) {
        const JobTable table = load_table(lane);
        J = load_item(table, int(blockIdx.x));             // idx: position among the job's workgroups
        const unsigned long long m = __builtin_amdgcn_ballot_w64(int(blockIdx.x) >= table.item0) & ((1ull << kMaxJobs) - 1);
        const int ji = __builtin_popcountll(m) - 1;
        ipg = int(__builtin_amdgcn_readlane(table.d[14], ji));
        plus = int(__builtin_amdgcn_readlane(table.d[15], ji));
    } else {
        const GemvJob& G = b.job[0];
        J.xb = reinterpret_cast<const unsigned char*>(G.x);
        J.Wb = reinterpret_cast<const unsigned char*>(G.W);
        J.y = G.y;
        J.gamma = G.gamma;
        J.Mrem = G.Mrem; J.MR = G.mr;
        J.N = G.N; J.K = G.K;
        J.row_bytes = uint32_t(G.K) >> 2;
        J.chunks = G.K >> 6;
        J.tiles = G.tiles; J.items = G.items; J.idx = int(blockIdx.x);
        J.slices = G.slices;
        ipg = G.run; plus = G.plus;
    }
    const int local = J.idx;
    const int tile0 = local * ipg + (local < plus ? local : plus);      // first tile of the run
    const int tile_end = tile0 + ipg + (local < plus ? 1 : 0);
    const int n_items = (tile_end - tile0 + T - 1) / T;
    // K longer than the waves' slices together (NW x 512) is walked in passes: pass c gives wave
    // w the slice c NW + w, streams the whole run of tiles, and leaves the sums of the run in
    // LDS (1 KB per tile behind the waves' areas) for the next pass to add to.
    const int n_pass = PASSES ? (J.slices + NW - 1) / NW : 1;
    unsigned char* const ysum = lds_raw + NW * kStride;
    int slice = wave;
    bool active = slice < J.slices;
    uint32_t col_off = 0;
    const bool ragged_n = (J.N & 15) != 0;
    typedef const __attribute__((address_space(1))) u32x4* gptr;

    u32x4 wreg[T][2];
    auto chunk_offset = [&](int sl) {
        int chunk = sl * 8 + lc;                           // 16-byte chunk of this lane within the row
        if (chunk >= J.chunks) chunk = 0;                  // past K: multiplied by zero activations
        return uint32_t(chunk) * 16u;
    };
    // Several passes, one row block of at most 4 rows: the next pass's activation rows are fetched
    // into registers while the last item of this pass is worked on (plain loads, so the compiler's
    // wait counts stay exact), and that item refills with the next pass's first weights.
    constexpr bool kAheadOk = PASSES && NB == 1;
    u32x4 xpre[kAheadOk ? 4 : 1];
    auto issue_w = [&](int first, int t) {
        int tile = first + t;
        if (tile >= tile_end) tile = tile_end - 1;         // past the run: its last tile again, never stored
        const unsigned char* tb = J.Wb + size_t(tile) * 16u * J.row_bytes;
        // rows past N read row N-1 (no branch: the loop body stays one scheduling region)
        const int last = (ragged_n && tile == J.tiles - 1) ? J.N - 1 - tile * 16 : 15;
        const uint32_t off0 = uint32_t(lr < last ? lr : last) * J.row_bytes + col_off;
        const uint32_t off1 = uint32_t(lr + 8 < last ? lr + 8 : last) * J.row_bytes + col_off;
        wreg[t][0] = __builtin_nontemporal_load((gptr)(tb + off0));
        wreg[t][1] = __builtin_nontemporal_load((gptr)(tb + off1));
    };

    uint32_t breg[NB][2][4][8];                // this wave's activations as MFMA B operands, per row block
    f32x4 nsx[NB];                             // -2^-20 sum_k x[m][k] over the slice, as an accumulator
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) nsx[nb] = f32x4{0.f, 0.f, 0.f, 0.f};
    // Start of a pass: fetch this wave's activation slice and the first item's weights together,
    // then turn the activations into operand registers.
    // ahead_here: the end of the pass before has requested this pass's activation rows (into xpre)
    // and its first item's weights already.
    auto begin_pass = [&](int pass, bool ahead_here) {
    slice = pass * NW + wave;
    active = slice < J.slices;
    if (!ahead_here) col_off = chunk_offset(slice);
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) nsx[nb] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) {
        // rows of this block: block 0 takes the first 16 (or fewer), block 1 what is left
        const int rows = nb == 0 ? (J.Mrem < 16 ? J.Mrem : 16) : J.Mrem - 16;
        int mr = 1;
        while (mr < rows) mr *= 2;
        if (active && rows > 0) {
            // activation rows by LDS-DMA, swizzled: lane l fetches piece l ^ (r & 7) of row r.
            // Kept as short rolled loops: this is on the way to the first weight load, and at
            // the start of a kernel every instruction line is a miss in the instruction cache.
            // Staged rows past `rows` are never written: an MFMA column depends on its own column
            // of B alone, and the outputs of those columns are not stored.
            typedef const __attribute__((address_space(1))) unsigned char* gbytes;
            const size_t row_stride = size_t(J.K) * 2;
            gbytes src = (gbytes)(J.xb + size_t(16 * nb) * row_stride + size_t(slice) * (kSliceK * 2));
            if (kAheadOk && ahead_here) {
                if constexpr (kAheadOk) {
#pragma unroll
                    for (int r = 0; r < 4; ++r)
                        if (r < rows) *reinterpret_cast<u32x4*>(my_lds + r * 1024 + (uint32_t(lane) << 4)) = xpre[r];
                }
            } else if ((slice + 1) * kSliceK <= J.K) {     // the whole slice lies inside K
                const uint32_t lane16 = uint32_t(lane) << 4;
#pragma unroll 1
                for (int r = 0; r < rows; ++r) {
                    __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(src + (lane16 ^ (uint32_t(r & 7) << 4))),
                                                     (__attribute__((address_space(3))) void*)(my_lds + r * 1024), 16, 0, 0);
                    src += row_stride;
                }
            } else {
#pragma unroll 1
                for (int r = 0; r < rows; ++r) {
                    const int kk = (lane ^ (r & 7)) << 3;  // first of this lane's 8 activations within the slice
                    if (slice * kSliceK + kk < J.K) {
                        __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(src + uint32_t(kk) * 2u),
                                                         (__attribute__((address_space(3))) void*)(my_lds + r * 1024), 16, 0, 0);
                    } else {
                        *reinterpret_cast<u32x4*>(my_lds + r * 1024 + (uint32_t(lane) << 4)) = u32x4{0u, 0u, 0u, 0u};
                    }
                    src += row_stride;
                }
            }
            if (kAheadOk && ahead_here) {
                // nothing to request; the registers' own loads are waited for by the compiler
            } else if (nb == 0) {
#pragma unroll
                for (int t = 0; t < T; ++t) issue_w(tile0, t);
                // the compiler does not track LDS-DMA: wait until only the 2T weight loads are outstanding
                __builtin_amdgcn_s_waitcnt(vmcnt_imm(2 * T));
            } else {
                __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));  // requested after the weights: wait for all
            }
            const int xrow = mi & (mr - 1);
            const uint32_t xr_off = uint32_t(xrow) * 1024u + uint32_t(mg) * 128u;
            const uint32_t sw = uint32_t(xrow & 7);
            // breg[nb][h][wd][e]: (x[k], x[k + 8]) with k = slice0 + 64 (4h + g) + 16 wd + e.
            // Columns that stand for no activation row get zeros (byte selector 0x0c), not the
            // unwritten staging rows: nothing is stored from them, and multiplying zeros costs
            // the matrix pipes less power than multiplying copies of real rows.
            const bool live = mi < rows;
            const uint32_t sel_lo = live ? 0x05040100u : 0x0c0c0c0cu;
            const uint32_t sel_hi = live ? 0x07060302u : 0x0c0c0c0cu;
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int wd = 0; wd < 4; ++wd) {
                    const u32x4 lo = *reinterpret_cast<const u32x4*>(
                        my_lds + xr_off + h * 512 + ((uint32_t(2 * wd) ^ sw) << 4));
                    const u32x4 hi = *reinterpret_cast<const u32x4*>(
                        my_lds + xr_off + h * 512 + ((uint32_t(2 * wd + 1) ^ sw) << 4));
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        breg[nb][h][wd][2 * r] = __builtin_amdgcn_perm(hi[r], lo[r], sel_lo);
                        breg[nb][h][wd][2 * r + 1] = __builtin_amdgcn_perm(hi[r], lo[r], sel_hi);
                    }
                }
            const uint32_t c = 0x80108010u;               // fp16 pair of -2^-20
            const u32x4 a = u32x4{c, c, c, c};
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const u32x4 bb = u32x4{breg[nb][h][0][e], breg[nb][h][1][e], breg[nb][h][2][e], breg[nb][h][3][e]};
                    nsx[nb] = __builtin_amdgcn_mfma_f32_16x16x32_f16(as_f16x8(a), as_f16x8(bb), nsx[nb], 0, 0, 0);
                }
            if (NB > 1 && nb == 0) __builtin_amdgcn_s_waitcnt(0xF | (0x3 << 14) | (0x7 << 4));   // staging read before it is refilled
        } else {
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int wd = 0; wd < 4; ++wd)
#pragma unroll
                    for (int e = 0; e < 8; ++e) breg[nb][h][wd][e] = 0u;
        }
    }
    };

    // One item (tiles first .. first + T - 1): tile t goes through LDS region t & 1 into MFMA
    // order, is decoded and multiplied; REFILL: its registers are loaded again at once for the
    // next item.  Tiles past the run are computed from whatever was loaded and never stored.
    auto item = [&](auto refill_tag, int first, int refill_first, int parity, bool first_pass_rt, bool last_pass_rt) {
        constexpr bool REFILL = decltype(refill_tag)::value;
        const bool first_pass = PASSES ? first_pass_rt : true;
        const bool last_pass = PASSES ? last_pass_rt : true;
        f32x4 part[NB][T];
#pragma unroll
        for (int nb = 0; nb < NB; ++nb)
#pragma unroll
            for (int t = 0; t < T; ++t) part[nb][t] = f32x4{0.f, 0.f, 0.f, 0.f};
        if (active) {
#pragma unroll
            for (int t = 0; t < T; ++t) {
                unsigned char* const reg_t = my_lds + (t & 1) * 2048;
                *reinterpret_cast<u32x4*>(reg_t + ww_off) = wreg[t][0];
                *reinterpret_cast<u32x4*>(reg_t + 1024 + ww_off) = wreg[t][1];
                if constexpr (REFILL) issue_w(refill_first, t);
                if (REFILL || first + t < tile_end) {      // the last item may be short
                    f32x4 acc[NB][3];
#pragma unroll
                    for (int nb = 0; nb < NB; ++nb) {
                        acc[nb][0] = nsx[nb];
                        acc[nb][1] = f32x4{0.f, 0.f, 0.f, 0.f};
                        acc[nb][2] = f32x4{0.f, 0.f, 0.f, 0.f};
                    }
#pragma unroll
                    for (int h = 0; h < 2; ++h) {
                        const u32x4 wv = *reinterpret_cast<const u32x4*>(reg_t + (h ? wr_off1 : wr_off0));
                        // element e of each half-word sits at bits 2e, 2e+1; the mantissa bits
                        // 4..9 (classes 0..2 -> accumulators) hold e = 2,3,4 as loaded, e = 0,1
                        // after << 4 and e = 5,6,7 after >> 6
                        const u32x4 sh[3] = {wv << 4, wv, wv >> 6};
#pragma unroll
                        for (int e = 0; e < 8; ++e) {
                            const int src = e < 2 ? 0 : (e < 5 ? 1 : 2);
                            const int j = e < 2 ? e : (e < 5 ? e - 2 : e - 5);
                            const uint32_t mask = 0x00300030u << (2 * j);
                            const u32x4 a = sh[src] & mask;
#pragma unroll
                            for (int nb = 0; nb < NB; ++nb) {
                                const u32x4 bb = u32x4{breg[nb][h][0][e], breg[nb][h][1][e], breg[nb][h][2][e], breg[nb][h][3][e]};
                                acc[nb][j] = __builtin_amdgcn_mfma_f32_16x16x32_f16(as_f16x8(a), as_f16x8(bb), acc[nb][j], 0, 0, 0);
                            }
                        }
                    }
#pragma unroll
                    for (int nb = 0; nb < NB; ++nb)
                        part[nb][t] = acc[nb][0] * 1048576.f + acc[nb][1] * 262144.f + acc[nb][2] * 65536.f;
                }
            }
        }
        // split-K: partial sums into this wave's set `parity`, one barrier, fixed-order sum.
        // The other set is still being read by waves that lag one item behind, never more:
        // they must pass this item's barrier before anybody writes that set again.
        unsigned char* const red = my_lds + 4096 + parity * (T * NB * 1024);
#pragma unroll
        for (int nb = 0; nb < NB; ++nb)
#pragma unroll
            for (int t = 0; t < T; ++t) reinterpret_cast<f32x4*>(red + (nb * T + t) * 1024)[lane] = part[nb][t];
        __builtin_amdgcn_s_waitcnt(0xF | (0x3 << 14) | (0x7 << 4));     // lgkmcnt(0): LDS only, loads stay in flight
        __builtin_amdgcn_s_barrier();
        if (const int o = threadIdx.x; o < T * NB * 64) {  // T NB <= waves: one output quad per thread
            const int q = o >> 6;                           // nb * T + t
            const int nb = q / T;
            const int t = q - nb * T;
            const int l = o & 63;
            const int row = 16 * nb + (l & 15);
            const int tile = first + t;
            f32x4 v[8];
#pragma unroll
            for (int w = 0; w < 8; ++w)
                v[w] = (w < NW) ? reinterpret_cast<const f32x4*>(lds_raw + w * kStride + 4096 + parity * (T * NB * 1024) + q * 1024)[l]
                                : f32x4{0.f, 0.f, 0.f, 0.f};
            f32x4 s = ((v[0] + v[1]) + (v[2] + v[3])) + ((v[4] + v[5]) + (v[6] + v[7]));
            // sums of the earlier passes over K: kept by the thread that owns this output quad
            f32x4* const keep = reinterpret_cast<f32x4*>(ysum + ((tile - tile0) * NB + nb) * 1024) + l;
            if (!first_pass && tile < tile_end) s += *keep;
            if (!last_pass && tile < tile_end) *keep = s;
            const int n = tile * 16 + 4 * (l >> 4);
            if (last_pass && tile < tile_end && row < J.Mrem) {
                typedef __attribute__((address_space(1))) __half* gh_ptr;
                gh_ptr dst = (gh_ptr)(J.y + size_t(row) * J.N + n);
                const float gamma = J.gamma;
                if (n + 3 < J.N && (J.N & 3) == 0) {       // four consecutive n: one 8-byte store
                    const f16x2 lo = {(_Float16)(gamma * s[0]), (_Float16)(gamma * s[1])};
                    const f16x2 hi = {(_Float16)(gamma * s[2]), (_Float16)(gamma * s[3])};
                    *(__attribute__((address_space(1))) u32x2*)dst =
                        u32x2{__builtin_bit_cast(uint32_t, lo), __builtin_bit_cast(uint32_t, hi)};
                } else {
#pragma unroll
                    for (int r = 0; r < 4; ++r)
                        if (n + r < J.N) *(__attribute__((address_space(1))) _Float16*)(dst + r) = (_Float16)(gamma * s[r]);
                }
            }
        }
    };

    bool ahead_here = false;
    for (int pass = 0; pass < n_pass; ++pass) {
        const bool first_pass = pass == 0, last_pass = pass + 1 == n_pass;
        begin_pass(PASSES ? pass : 0, ahead_here);
        ahead_here = false;
        int i = 0;
        for (; i + 1 < n_items; ++i) item(std::true_type{}, tile0 + i * T, tile0 + (i + 1) * T, i & 1, first_pass, last_pass);
        bool cross = false;
        if constexpr (kAheadOk) {
            const int next_slice = (pass + 1) * NW + wave;
            cross = !last_pass && active && next_slice < J.slices && J.Mrem <= 4;
            if (cross) {
                typedef const __attribute__((address_space(1))) unsigned char* gbytes;
                gbytes src = (gbytes)(J.xb + size_t(next_slice) * (kSliceK * 2));
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int piece = lane ^ (r & 7);      // the staging order of begin_pass
                    xpre[r] = u32x4{0u, 0u, 0u, 0u};
                    if (r < J.Mrem && next_slice * kSliceK + piece * 8 < J.K)
                        xpre[r] = *(gptr)(src + size_t(r) * (size_t(J.K) * 2) + uint32_t(piece) * 16u);
                }
                col_off = chunk_offset(next_slice);
                item(std::true_type{}, tile0 + i * T, tile0, i & 1, first_pass, last_pass);
                ahead_here = true;
            }
        }
        if (!cross) item(std::false_type{}, tile0 + i * T, 0, i & 1, first_pass, last_pass);
        if (PASSES && !last_pass) {
            // the next pass stages activations over the partial-sum sets: everybody must be done reading
            __builtin_amdgcn_s_waitcnt(0xF | (0x3 << 14) | (0x7 << 4));
            __builtin_amdgcn_s_barrier();
        }
    }
}

// ------------------------------------------------------------------------------------------
// Lean stream kernel: the stream form for launches in which every job has as many 512-weight
// slices as the workgroup has waves, or (PASSES) more, one block of at most 16 activation
// rows, one gamma or (GS) group scales, and N a multiple of 16 -- the decode shapes.  What differs from
// gemv_stream_kernel is the way in and the loop, not the arithmetic:
//  * Every workgroup has a 64-byte record of its own in the kernel arguments (pointers of its job,
//    first tile and length of its run), read with one scalar load at an address that depends on
//    the workgroup index alone: no table search stands between the kernel entry and the first
//    requests, and one- and many-job launches run the same code.
//  * A lane's two weight addresses within a tile are computed once; a tile's loads are that
//    offset on a scalar base which steps from tile to tile, so the loop spends no vector
//    instructions on addresses.
//  * Every wave is active in every tile (no predicated tile bodies); the last item comes in one
//    copy per tile count.
// The vector ALU is what limits the steady state of these kernels (64 ANDs + 16 shifts + 16 MFMA
// issues + 8 combine operations per wave and tile are 104 of the ~120 issue slots a tile may
// take if the loop is to keep up with HBM), so every instruction that is not decode counts.
constexpr int kLeanMaxGroups = 256;

// Group scales in the lean kernel, by what the groups are multiples of: 256, 128, 64 or 32 weights.  Weights per scale that is fetched:
__host__ __device__ constexpr int lean_scale_unit(int gs) { return gs == 256 ? 256 : gs == 32 ? 32 : 64; }

// bytes of 16 packed rows
__host__ __device__ constexpr size_t packed_tile_bytes(int K) { return size_t((unsigned(K) + 15u) >> 4) * 64u; }

struct WgRec {                    // 64 bytes; rec[blockIdx.x] is read with scalar loads
    const unsigned char* W;       // packed row 0 of the first tile of the run
    const unsigned char* x;       // activations of the job, fp16 [Mrem][K]
    __half* y;                    // outputs of the job, fp16 [Mrem][N]
    float gamma;
    int K, N;
    int Mrem;                     // 1..16
    int tile0, ntiles;            // the run: tiles tile0 .. tile0 + ntiles - 1 of the job (ntiles >= 1)
    const unsigned char* sc;      // group scales [groups][N] fp16, and 1 / (scale units of 256 weights per group): unit u lies in
    uint32_t group_inv;           // group (2 u group_inv) >> 32; see group_inverse
    int pad;
};
static_assert(sizeof(WgRec) == 64, "one record per 64-byte line");

struct LeanBatch {
    WgRec rec[kLeanMaxGroups];
    __device__ const WgRec& mine() const { return rec[blockIdx.x]; }
};

// A launch of one job: 64 bytes of arguments instead of 16 KB.  The records cost nothing on the device but 1 us of
// the host per launch (written, copied, copied again into the argument segment), which is a fifth of a small decode call:
// 2048 -> 2048 at M = 1 called in a loop 5.3 us with them, 3.4 us without (that, and no bisection for a
// single job in launch_stream).  Workgroup g works its own record out: `per` tiles, the first `plus` workgroups one more.
struct LeanOne {
    const unsigned char* W;       // packed row 0 of the matrix
    const unsigned char* x;
    __half* y;
    float gamma;
    int K, N;
    int Mrem;
    int per, plus;
    uint32_t group_inv;           // see WgRec
    const unsigned char* sc;
    __device__ WgRec mine() const { return at(int(blockIdx.x)); }
    __device__ WgRec at(int g) const
    {
        WgRec r;
        r.tile0 = g * per + (g < plus ? g : plus);
        r.ntiles = per + (g < plus ? 1 : 0);
        r.W = W + size_t(r.tile0) * (size_t(4) * size_t(K));          // 16 rows of K / 4 bytes
        r.x = x; r.y = y; r.gamma = gamma;
        r.K = K; r.N = N; r.Mrem = Mrem;
        r.sc = sc; r.group_inv = group_inv;
        return r;
    }
};

// The same for any number of rows (`Mrem` of them), blockIdx.y being the block of 16, and for any K and N.
struct LeanAny : LeanOne {
    __device__ WgRec mine() const
    {
        WgRec r = LeanOne::mine();
        const int m0 = int(blockIdx.y) * 16;
        r.W = W + size_t(r.tile0) * packed_tile_bytes(K);
        r.x = x + size_t(m0) * (size_t(2) * size_t(K));
        r.y = y + size_t(m0) * size_t(N);
        r.Mrem = Mrem - m0 < 16 ? Mrem - m0 : 16;
        return r;
    }
};
static_assert(sizeof(LeanOne) == 64, "the arguments of a lone call");
static_assert(kMaxJobs <= kTableMost, "a table holds the jobs of a launch");

// Up to R jobs: 68 bytes of arguments each, and a workgroup finds its job by two scalar look-ups in turn (see jobs_by_table).
template <int R>
struct LeanJobs {
    static constexpr int kJobs = R;
    int first[R];                 // first workgroup of job j; INT_MAX for unused entries
    LeanOne job[R];
    __device__ WgRec mine() const
    {
        int j = 0;
#pragma unroll
        for (int i = 1; i < 8; ++i) j += int(blockIdx.x) >= first[i] ? 1 : 0;
        if (j == 7) {
#pragma unroll
            for (int i = 8; i < 16; ++i) j += int(blockIdx.x) >= first[i] ? 1 : 0;
        }
        if constexpr (R > 16) {
            if (j == 15) {
#pragma unroll
                for (int i = 16; i < R; ++i) j += int(blockIdx.x) >= first[i] ? 1 : 0;
            }
        }
        const LeanOne& J = job[j];
        WgRec r = J.at(int(blockIdx.x) - first[j]);
        r.W = J.W + size_t(r.tile0) * packed_tile_bytes(J.K);
        return r;
    }
};

template <class Args>
constexpr bool kIsTable = false;
template <int R>
constexpr bool kIsTable<LeanJobs<R>> = true;

// Activations whose rows start at any even address (K no multiple of 64), to the places the operand set-up reads: through registers, a row to a
// request.  Lane l takes piece l of the slice, eighth l % 8 of chunk l / 8; a row's last chunk is its last 64 weights (16 packed bytes).  What
// lies past K or, in the last chunk, before the chunk's own weights becomes zero; the piece across K is fetched from the row's last 16
// bytes and shifted down.  Rows past the last one repeat it.
typedef const __attribute__((address_space(1))) unsigned char* global_bytes;
typedef u32x4 __attribute__((aligned(2))) u32x4_any;
typedef u32x2 __attribute__((aligned(2))) u32x2_any;
__device__ __forceinline__ int first_weight(int chunk, int K)
{
    const int last = ((K + 15) & ~15) - 64;
    return chunk * 64 < last ? chunk * 64 : last;
}
template <int COUNT>
__device__ __forceinline__ void fetch_rows(global_bytes x, int rows, int K, int slice, int lane, u32x4 (&v)[COUNT])
{
    const int k = first_weight(slice * 8 + (lane >> 3), K) + (lane & 7) * 8;
    const uint32_t at = uint32_t(k < K - 8 ? k : K - 8) * 2u;
    uint32_t row = 0;
#pragma unroll
    for (int r = 0; r < COUNT; ++r) {
        v[r] = *(const __attribute__((address_space(1))) u32x4_any*)(x + row + at);
        row += r + 1 < rows ? uint32_t(K) * 2u : 0u;
    }
}
// the 16 bytes of a piece that ends n / 16 elements past K
__device__ __forceinline__ u32x4 shifted_down(u32x4 w, int n)
{
    uint64_t lo = uint64_t(w[0]) | (uint64_t(w[1]) << 32), hi = uint64_t(w[2]) | (uint64_t(w[3]) << 32);
    if (n >= 64) { lo = hi; hi = 0; }
    const int m = n & 63;
    if (m) { lo = (lo >> m) | (hi << (64 - m)); hi >>= m; }
    if (n >= 128) lo = 0;
    return u32x4{uint32_t(lo), uint32_t(lo >> 32), uint32_t(hi), uint32_t(hi >> 32)};
}
// At the start of a kernel every line of code is a miss in the instruction cache: many rows are put right in LDS, by little code, since
// all of them in registers took 16 rows 0.4 to 0.6 us longer; up to four rows in registers, which the LDS's latency made 0.1 to 0.25 us longer.
template <int COUNT>
__device__ __forceinline__ void put_rows(unsigned char* area, int rows, int K, int slice, int lane, u32x4 (&v)[COUNT])
{
    const bool tail = (slice + 1) * kSliceK > K;
    const int chunk = slice * 8 + (lane >> 3);
    const int k = first_weight(chunk, K) + (lane & 7) * 8;
    const int past = k + 8 - K;                            // elements past K
    const bool zero = past >= 8 || k < chunk * 64;
    if (COUNT <= 4 && tail) {
        const int n = zero ? 128 : 16 * (past > 0 ? past : 0);
#pragma unroll
        for (int r = 0; r < COUNT; ++r) v[r] = shifted_down(v[r], n);
    }
#pragma unroll
    for (int r = 0; r < COUNT; ++r) *reinterpret_cast<u32x4*>(area + r * 1024 + (uint32_t(lane ^ (r & 7)) << 4)) = v[r];
    if (COUNT <= 4 || !tail) return;
#pragma unroll 1
    for (int r = 0; r < rows; ++r)
        if (zero) *reinterpret_cast<u32x4*>(area + r * 1024 + (uint32_t(lane ^ (r & 7)) << 4)) = u32x4{0u, 0u, 0u, 0u};
    const unsigned long long cut = __builtin_amdgcn_ballot_w64(past > 0 && !zero);
    if (cut) {                                             // one piece of the slice, lane l's: lane r does row r's
        const int l = __builtin_ctzll(cut), n = 16 * (first_weight(slice * 8 + (l >> 3), K) + (l & 7) * 8 + 8 - K);
        if (lane < rows) {
            u32x4* const p = reinterpret_cast<u32x4*>(area + lane * 1024 + (uint32_t(l ^ (lane & 7)) << 4));
            *p = shifted_down(*p, n);
        }
    }
}
// the lane's place in its row of packed words: the row's last chunk, and what lies past it, are its last 16 bytes
__device__ __forceinline__ uint32_t chunk_place(uint32_t chunk, uint32_t row_bytes)
{
    return chunk * 16u < row_bytes - 16u ? chunk * 16u : row_bytes - 16u;
}
// four consecutive columns of y from `col` on, as many as there are
__device__ __forceinline__ void store_quad_any(__attribute__((address_space(1))) __half* row, int col, int N, f32x4 s, float gamma)
{
    if (col + 4 <= N) {
        const f16x2 lo = {(_Float16)(gamma * s[0]), (_Float16)(gamma * s[1])};
        const f16x2 hi = {(_Float16)(gamma * s[2]), (_Float16)(gamma * s[3])};
        *(__attribute__((address_space(1))) u32x2_any*)(row + col) = u32x2{__builtin_bit_cast(uint32_t, lo), __builtin_bit_cast(uint32_t, hi)};
    } else {
#pragma unroll
        for (int r = 0; r < 3; ++r)
            if (col + r < N) *(__attribute__((address_space(1))) _Float16*)(row + col + r) = (_Float16)(gamma * s[r]);
    }
}

// PASSES: jobs may have K beyond the waves' slices (the down projection among the linears of a block).  Such a job's run is
// streamed once per NW slices; between passes the sums of the run wait in LDS (1 KB per tile behind the waves' areas)
// with the thread that owns the output quad.  The last item of a pass asks for the next pass's first weights; the
// activations follow once every wave has left the sums of that item, which share LDS with them.  Waves past the last
// slice take no part in the last pass but for the exchange (multiplying zeros instead, 7936 x 5248 at M = 18, two slices in the last of
// two passes, took 12.5 us and the general form 11.1; now 11.3; 65 rows of 11648 x 4480 25.3, 23.6 and 22.3).
// GS = 256: group scales, groups of whole units of 256 weights (half a slice).  The halves of a tile are summed one after the
// other in the same accumulators, each scaled by its group's scales of the lane's four output rows, which are
// requested with the tile's weights (block at M = 1 / 4 / 16 14.5 / 14.3 / 17.1 us).
// GS = 128, 64, 32: groups of multiples of as many.  In the order above a product's 32 weights come from four chunks of 64, so a unit's sum
// would never stand alone in an accumulator; here a lane takes a word of every chunk (32: half a word), and 64 (32) weights are two products (one).
// What bounds them is the scaling of every unit's sum on the vector ALU, 4 operations for 16 x 16 outputs beside the 11 (32: 13) of the decode per
// product pair (product): block at M = 4 15.2 / 17.3 / 24.7 us with groups of 128 / 64 / 32, decode sweep 21.0 / 24.3 / 36.5.  Groups of 128 took
// 25.8 and 36.5 in the general form, every product issued twice with other lanes masked off; the others went to the tiled kernel one by one, 68
// and 131 us.
// GS, several jobs: an N that is a multiple of 4 as well; through ANY such a launch, its x in registers, took up to 13 % longer (block of 8 rows, 1088 wide,
// one N no multiple of 16, 6.5 -> 6.0 us).  Lone calls go without, which would cost them 0.05 to 0.2 us.
// ANY: any K from 64 on and any N (GS: N a multiple of 4), jobs with fewer slices than waves among them.  Packed rows then start at multiples of 4
// bytes, rows of x and y at any even address.  A row's last 16-byte chunk of weights is its last 16 bytes, wherever they start: no
// request leaves the row, and what overlaps the chunk before meets zeros.  The activations come through registers.  Calls with K no multiple of 64
// ran in the tiled kernel's form for those: up to 4 rows of 512 .. 16384 x 64 .. 14336 weights this one is 1.8 times as fast on average
// (666 calls, none slower), 4099 x 4090 at M = 1 / 16 / 37 8.0 / 8.3 / 10.7 -> 4.3 / 5.7 / 6.8 us.
template <int T, bool PASSES, int GS, bool ANY, class Args>
__global__ void __launch_bounds__(512)
gemv_lean_kernel(Args b)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char lds_raw[];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int NW = blockDim.x >> 6;
    constexpr int kStride = stream_wave_lds(T);
    constexpr bool FINE = GS != 0 && GS < 256;
    // LDS of a wave after the operands are built: two tile regions, from `kSums` on two sets of T partial-sum tiles.  FINE: rows of a tile
    // 144 bytes apart, the tile's scales behind them.
    constexpr int kScales = 16 * 144, kRegion = FINE ? kScales + 512 : 2048, kSums = 2 * kRegion;
    static_assert(kSums + 2 * T * 1024 <= kStride, "LDS of a wave");
    unsigned char* const my_lds = lds_raw + wave * kStride;
    typedef const __attribute__((address_space(1))) unsigned char* gbytes;

    const auto& R = b.mine();
    const int K = R.K, N = R.N, rows = R.Mrem, ntiles = R.ntiles;
    const unsigned char* const Wrun = R.W;
    const uint32_t row_bytes = ANY ? ((uint32_t(K) + 15u) >> 4) * 4u : uint32_t(K) >> 2;
    const uint32_t tile_bytes = 16u * row_bytes;

    const int lr = lane >> 3, lc = lane & 7;   // load mapping: row of the half tile, chunk of the slice
    const int mi = lane & 15, mg = lane >> 4;  // MFMA mapping: row / activation column, k group

    const int slices = (K + kSliceK - 1) / kSliceK;
    const int n_pass = PASSES ? (slices + NW - 1) / NW : 1;
    // ---- activations of a slice: LDS-DMA, swizzled (lane l fetches piece l ^ (r & 7) of row r)
    auto stage_x = [&](int slice) {
        int l = lane;
        if constexpr (PASSES) asm volatile("" : "+v"(l));  // see exchange
        const size_t row_stride = size_t(K) * 2;
        gbytes src = (gbytes)(R.x + size_t(slice) * (kSliceK * 2));
        if ((slice + 1) * kSliceK <= K) {                   // the whole slice lies inside K
            const uint32_t lane16 = uint32_t(l) << 4;
#pragma unroll 1
            for (int r = 0; r < rows; ++r) {
                __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(src + (lane16 ^ (uint32_t(r & 7) << 4))),
                                                 (__attribute__((address_space(3))) void*)(my_lds + r * 1024), 16, 0, 0);
                src += row_stride;
            }
        } else {
#pragma unroll 1
            for (int r = 0; r < rows; ++r) {
                const int kk = (l ^ (r & 7)) << 3;         // first of this lane's 8 activations within the slice
                if (slice * kSliceK + kk < K) {
                    __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(src + uint32_t(kk) * 2u),
                                                     (__attribute__((address_space(3))) void*)(my_lds + r * 1024), 16, 0, 0);
                } else {
                    *reinterpret_cast<u32x4*>(my_lds + r * 1024 + (uint32_t(l) << 4)) = u32x4{0u, 0u, 0u, 0u};
                }
                src += row_stride;
            }
        }
    };
    auto stage_any = [&](int slice, auto&& between) {      // `between`: what is asked for between the activations and their way to LDS
        auto with = [&](auto count) {
            u32x4 v[decltype(count)::value];
            int k = K;
            if constexpr (PASSES) asm volatile("" : "+s"(k));  // the rows' addresses worked out here, not kept over the passes
            fetch_rows((gbytes)R.x, rows, k, slice, lane, v);
            __builtin_amdgcn_sched_barrier(0);
            between();
            put_rows(my_lds, rows, k, slice, lane, v);
        };
        if (rows <= 1) with(std::integral_constant<int, 1>{});
        else if (rows <= 4) with(std::integral_constant<int, 4>{});
        else if (rows <= 8) with(std::integral_constant<int, 8>{});
        else with(std::integral_constant<int, 16>{});
    };
    // A job with fewer slices than waves, which the table of records does not hold: looking for it there cost the decode sweep 18.2 -> 20.0 us.
    constexpr bool kIdle = ANY || kIsTable<Args>;
    const bool idle = kIdle && wave >= slices;             // this wave has no slice at all
    if constexpr (!ANY) {
        if (!idle) stage_x(wave);
    }
    constexpr int H = GS == 256 ? 2 : 1;
    // GS: the job's scales from the run's first row as a raw buffer, the lane's rows in it, and the units' groups
    constexpr int kUnit = lean_scale_unit(GS);             // weights per scale that is fetched
    const uint32_t last_unit = uint32_t(K - 1) / uint32_t(kUnit);
    auto group_of = [&](uint32_t u) {                      // a product: two divisions would stand before the first request
        return uint32_t((uint64_t(2u * (u < last_unit ? u : last_unit)) * R.group_inv) >> 32);   // past K: the last one (its activations are zeros)
    };
    // FINE: one request fetches the scales of a tile and slice: lane l those of unit l / 8 and two rows (kUnit 32: l / 4 and four rows)
    constexpr int kUnitLanes = kUnit == 32 ? 4 : 8;
    typedef typename std::conditional<kUnit == 32, u32x2, uint32_t>::type fine_t;
    const __amdgpu_buffer_rsrc_t sres = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<unsigned char*>(R.sc) + size_t(R.tile0) * 32u, 0,
        GS ? (group_of(last_unit) + 1u) * uint32_t(N) * 2u - uint32_t(R.tile0) * 32u : 0u, 0x00020000);
    const uint32_t sc_lane = uint32_t(mg) * 8u;
    uint32_t sc_unit[H] = {};
    uint32_t sc_fine = 0;
    auto scales_of = [&](int slice) {
        if constexpr (FINE) {
            // past K: outside the buffer, which reads as zero
            const uint32_t unit = uint32_t(slice) * (kSliceK / kUnit) + uint32_t(lane / kUnitLanes);
            sc_fine = unit <= last_unit ? group_of(unit) * uint32_t(N) * 2u + uint32_t(lane % kUnitLanes) * uint32_t(sizeof(fine_t)) : 0x80000000u;
        } else if constexpr (GS != 0) {
#pragma unroll
            for (int h = 0; h < H; ++h) sc_unit[h] = group_of(uint32_t(2 * slice + h)) * uint32_t(N) * 2u;
        }
    };
    scales_of(wave);
    // ---- weights: the lane's two 16-byte pieces of a tile, relative to the tile's first row
    auto offset_of = [&](int slice) {
        uint32_t chunk = uint32_t(slice) * 8u + uint32_t(lc);
        if constexpr (ANY) return uint32_t(lr) * row_bytes + chunk_place(chunk, row_bytes);
        if (chunk >= (uint32_t(K) >> 6)) chunk = 0;        // past K: multiplied by zero activations
        return uint32_t(lr) * row_bytes + chunk * 16u;
    };
    uint32_t voff0 = offset_of(wave);
    uint32_t voff1 = voff0 + 8u * row_bytes;
    // the run as a raw buffer (no stride, byte offsets, size = the run): base in scalar registers
    // (with an N that need not be a multiple of 16, of the rows that exist; the others read zeros)
    constexpr bool kPartTile = ANY || (GS != 0 && !std::is_base_of<LeanOne, Args>::value);
    const int run_rows = kPartTile && N - R.tile0 * 16 < ntiles * 16 ? N - R.tile0 * 16 : ntiles * 16;
    const __amdgpu_buffer_rsrc_t wres = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<unsigned char*>(Wrun), 0, kPartTile ? uint32_t(run_rows) * row_bytes : uint32_t(ntiles) * tile_bytes, 0x00020000);
    u32x4 wreg[T][2];
    u32x2 sreg[T][H];
    fine_t freg[T];
    auto issue_w = [&](int idx, int t) {                   // idx: tile of the run; past the run: its last tile again
        const int c = idx < ntiles ? idx : ntiles - 1;
        // Buffer loads: descriptor and tile offset are scalar, the lane offset is a register that
        // never changes, so a request costs the vector ALU nothing.  That matters beyond the
        // instruction count: a wave whose data has arrived must get its next request out while
        // the other wave of its SIMD keeps the vector ALU busy.
        const uint32_t so = uint32_t(c) * tile_bytes;
        wreg[t][0] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(wres, voff0, so, 2));   // 2: nt
        wreg[t][1] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(wres, voff1, so, 2));
        if constexpr (FINE && kUnit == 32) {
            freg[t] = __builtin_bit_cast(u32x2, __builtin_amdgcn_raw_buffer_load_b64(sres, sc_fine, uint32_t(c) * 32u, 0));
        } else if constexpr (FINE) {
            freg[t] = __builtin_amdgcn_raw_buffer_load_b32(sres, sc_fine, uint32_t(c) * 32u, 0);
        } else if constexpr (GS != 0) {
#pragma unroll
            for (int h = 0; h < H; ++h)
                sreg[t][h] = __builtin_bit_cast(u32x2, __builtin_amdgcn_raw_buffer_load_b64(sres, sc_lane, __builtin_amdgcn_readfirstlane(sc_unit[h] + uint32_t(c) * 32u), 0));
        }
    };
    // in tile order, and kept so: the loop's wait counts are the worse of this order and its own
    auto first_tiles = [&]() {
#pragma unroll
        for (int t = 0; t < T; ++t) {
            issue_w(t, t);
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    if constexpr (ANY) {
        if (!idle) stage_any(wave, first_tiles);
    } else {
        if (!idle) {
            first_tiles();
            // the compiler does not track LDS-DMA: wait until only the weight (and scale) loads are outstanding
            __builtin_amdgcn_s_waitcnt(vmcnt_imm((FINE ? 3 : GS ? 4 : 2) * T));
        }
    }

    // ---- activations -> MFMA B operands (see gemv_stream_kernel) and the -sum(x) seed ----------
    u32x4 breg[16];
    constexpr int kSeeds = GS == 64 ? 8 : GS == 128 ? 4 : H;
    f32x4 nsx[kSeeds];
    auto build = [&] {
        int l = lane;
        if constexpr (PASSES) asm volatile("" : "+v"(l));  // see exchange
        const int mi = l & 15, mg = l >> 4;
#pragma unroll
        for (int h = 0; h < kSeeds; ++h) nsx[h] = f32x4{0.f, 0.f, 0.f, 0.f};
        int mr = 1;
        while (mr < rows) mr *= 2;
        const int xrow = mi & (mr - 1);
        const uint32_t xr_off = uint32_t(xrow) * 1024u + (FINE ? 0u : uint32_t(mg) * 128u);
        const uint32_t sw = uint32_t(xrow & 7);
        const bool live = mi < rows;
        const uint32_t sel_lo = live ? 0x05040100u : 0x0c0c0c0cu;
        const uint32_t sel_hi = live ? 0x07060302u : 0x0c0c0c0cu;
        const uint32_t c = 0x80108010u;                   // fp16 pair of -2^-20
        const u32x4 a = u32x4{c, c, c, c};
        if constexpr (GS == 32) {
            // breg[v]: unit v's eight activations of this lane, in order
            const uint32_t keep = live ? ~0u : 0u;
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const u32x4 q = *reinterpret_cast<const u32x4*>(my_lds + xr_off + (v >> 1) * 128 + ((uint32_t(4 * (v & 1) + mg) ^ sw) << 4));
#pragma unroll
                for (int r = 0; r < 4; ++r) breg[v][r] = q[r] & keep;
            }
            return;
        } else if constexpr (FINE) {
            // breg[2 c], [2 c + 1]: of chunk c the lane's 16 activations x[16 g + j], as pairs (j, j + 8) of even and of odd j
            const uint32_t at = (uint32_t(2 * mg) ^ sw) << 4;
#pragma unroll
            for (int ch = 0; ch < 8; ++ch) {
                const u32x4 lo = *reinterpret_cast<const u32x4*>(my_lds + xr_off + ch * 128 + at);
                const u32x4 hi = *reinterpret_cast<const u32x4*>(my_lds + xr_off + ch * 128 + (at ^ 16u));
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    breg[2 * ch][r] = __builtin_amdgcn_perm(hi[r], lo[r], sel_lo);
                    breg[2 * ch + 1][r] = __builtin_amdgcn_perm(hi[r], lo[r], sel_hi);
                }
                const int u = ch * kSeeds / 8;
                nsx[u] = __builtin_amdgcn_mfma_f32_16x16x32_f16(as_f16x8(a), as_f16x8(breg[2 * ch]), nsx[u], 0, 0, 0);
                nsx[u] = __builtin_amdgcn_mfma_f32_16x16x32_f16(as_f16x8(a), as_f16x8(breg[2 * ch + 1]), nsx[u], 0, 0, 0);
            }
            return;
        } else {
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int wd = 0; wd < 4; ++wd) {
                const u32x4 lo = *reinterpret_cast<const u32x4*>(my_lds + xr_off + h * 512 + ((uint32_t(2 * wd) ^ sw) << 4));
                const u32x4 hi = *reinterpret_cast<const u32x4*>(my_lds + xr_off + h * 512 + ((uint32_t(2 * wd + 1) ^ sw) << 4));
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    breg[h * 8 + 2 * r][wd] = __builtin_amdgcn_perm(hi[r], lo[r], sel_lo);
                    breg[h * 8 + 2 * r + 1][wd] = __builtin_amdgcn_perm(hi[r], lo[r], sel_hi);
                }
            }
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int e = 0; e < 8; ++e)
                nsx[GS ? h : 0] = __builtin_amdgcn_mfma_f32_16x16x32_f16(as_f16x8(a), as_f16x8(breg[h * 8 + e]), nsx[GS ? h : 0], 0, 0, 0);
        }
    };
    if constexpr (!PASSES) {
        if (!idle) build();
    }

    const uint32_t ww_off = FINE ? uint32_t(lr) * 144u + (uint32_t(lc) << 4) : uint32_t(lr) * 128u + (uint32_t(lc ^ lr) << 4);
    constexpr uint32_t kUpperRows = FINE ? 8 * 144 : 1024;
    // FINE: the lane's word of the first chunk (kUnit 32: of its first half), its scales' places: [4 rows][unit], 8 bytes each
    const uint32_t wr_fine = uint32_t(mi) * 144u + uint32_t(kUnit == 32 ? mg >> 1 : mg) * 4u;
    constexpr uint32_t kQuad = 8 * kSliceK / kUnit;
    const uint32_t sw_off = kScales + (kUnit == 32 ? uint32_t(lane & 3) * kQuad + uint32_t(lane >> 2) * 8u
                                                  : uint32_t((lane & 7) >> 1) * kQuad + uint32_t(lane >> 3) * 8u + uint32_t(lane & 1) * 4u);
    const uint32_t sr_off = kScales + uint32_t(mg) * kQuad;
    const uint32_t half_sel = mg & 1 ? 0x07060302u : 0x05040100u;
    const uint32_t wr_off0 = uint32_t(mi) * 128u + (uint32_t((mg) ^ (mi & 7)) << 4);
    const uint32_t wr_off1 = uint32_t(mi) * 128u + (uint32_t((4 + mg) ^ (mi & 7)) << 4);
    // times the 2^16 (2^18, 2^20) left in the partial sums
    const float gamma = GS == 32 ? 1048576.f : FINE ? 262144.f : GS ? 65536.f : R.gamma * 65536.f;
    typedef __attribute__((address_space(1))) __half* gh_ptr;

    // FINE: the tile in LDS region `reg`.  A unit's sum is complete in its accumulators and then scaled.
    auto fine_tile = [&](const unsigned char* reg) {
        f32x4 sum = {0.f, 0.f, 0.f, 0.f};
        if constexpr (FINE) {
            const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
            auto scaled = [&](int u, f32x4 v) {            // u: unit of kUnit weights
                const f16x4 s = reinterpret_cast<const f16x4*>(reg + sr_off)[u];
                const f32x4 f = {float(s[0]), float(s[1]), float(s[2]), float(s[3])};
                sum = __builtin_elementwise_fma(f, v, sum);
            };
            if constexpr (kUnit == 32) {
                // Lane (i, g) of unit v takes the eight codes 8 g ..: the half word is spread so that code 2q stands at bit 4q of the lower half and 2q + 1
                // at bit 4q of the upper one; each pair is brought to bit 4 and loses its offset there, (c - 1) 2^-20, exact.
                const f16x2 one = __builtin_bit_cast(f16x2, 0x00100010u);
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    const uint32_t w = *reinterpret_cast<const uint32_t*>(reg + wr_fine + (v >> 1) * 16 + (v & 1) * 8);
                    const uint32_t p = __builtin_amdgcn_perm(w >> 2, w, half_sel);
                    u32x4 a = {(p << 4) & 0x00300030u, p & 0x00300030u, (p >> 4) & 0x00300030u, (p >> 8) & 0x00300030u};
#pragma unroll
                    for (int r = 0; r < 4; ++r) a[r] = __builtin_bit_cast(uint32_t, __builtin_bit_cast(f16x2, uint32_t(a[r])) - one);
                    scaled(v, __builtin_amdgcn_mfma_f32_16x16x32_f16(as_f16x8(a), as_f16x8(breg[v]), zero, 0, 0, 0));
                }
            } else {
                // Lane (i, g) takes word g of a chunk, codes j and j + 8 as a pair: even j at bit 4, odd ones at bit 6, an accumulator for each
                f32x4 even, odd;
#pragma unroll
                for (int ch = 0; ch < 8; ++ch) {
                    const uint32_t w = *reinterpret_cast<const uint32_t*>(reg + wr_fine + ch * 16);
                    const u32x4 sh = {w << 4, w, w >> 4, w >> 8};
                    const bool first = GS == 64 || (ch & 1) == 0;
                    even = __builtin_amdgcn_mfma_f32_16x16x32_f16(as_f16x8(sh & 0x00300030u), as_f16x8(breg[2 * ch]), first ? nsx[ch * kSeeds / 8] : even, 0, 0, 0);
                    odd = __builtin_amdgcn_mfma_f32_16x16x32_f16(as_f16x8(sh & 0x00C000C0u), as_f16x8(breg[2 * ch + 1]), first ? zero : odd, 0, 0, 0);
                    if (GS == 64 || (ch & 1)) scaled(GS == 64 ? ch : ch - 1, __builtin_elementwise_fma(even, f32x4{4.f, 4.f, 4.f, 4.f}, odd));
                }
            }
        }
        return sum;
    };

    // split-K: each wave's partial sums of nt tiles are in its set `parity`; one LDS-only barrier, fixed-order sum.  A thread owns an output
    // quad of tile threadIdx.x / 64 of the item.
    const int ot = int(threadIdx.x) >> 6;
    const uint32_t ycol = uint32_t(R.tile0) * 16u + 4u * uint32_t(mg);       // + 16 (first + ot)
    gh_ptr const yrow = (gh_ptr)(R.y + size_t(mi) * size_t(N));
    unsigned char* const ysum = lds_raw + NW * kStride;
    auto sum_of = [&](int t, int l, int parity) {
        f32x4 v[8];
#pragma unroll
        for (int w = 0; w < 8; ++w)
            v[w] = (w < NW) ? reinterpret_cast<const f32x4*>(lds_raw + w * kStride + kSums + parity * (T * 1024) + t * 1024)[l]
                            : f32x4{0.f, 0.f, 0.f, 0.f};
        return ((v[0] + v[1]) + (v[2] + v[3])) + ((v[4] + v[5]) + (v[6] + v[7]));
    };
    auto put = [&](gh_ptr row, uint32_t col, f32x4 s) {
        if constexpr (ANY) {
            store_quad_any(row, int(col), N, s, gamma);
        } else {
            if (kPartTile && col >= uint32_t(N)) return;   // N is a multiple of 4
            const f16x2 lo = {(_Float16)(gamma * s[0]), (_Float16)(gamma * s[1])};
            const f16x2 hi = {(_Float16)(gamma * s[2]), (_Float16)(gamma * s[3])};
            *(__attribute__((address_space(1))) u32x2*)(row + col) = u32x2{__builtin_bit_cast(uint32_t, lo), __builtin_bit_cast(uint32_t, hi)};
        }
    };
    auto exchange = [&](int nt, int first, int parity, bool first_pass, bool last_pass) {
        __builtin_amdgcn_s_waitcnt(0xF | (0x3 << 14) | (0x7 << 4));
        __builtin_amdgcn_s_barrier();
        if constexpr (!PASSES) {
            if (ot < nt) {
                const f32x4 s = sum_of(ot, lane, parity);
                if (mi < rows) put(yrow, ycol + 16u * uint32_t(first + ot), s);
            }
        } else if (wave < nt) {
            // The thread's places are worked out here.  Kept over the loop they took registers that others were spilled for, and a
            // reload waits for every weight on its way (block with groups of 256 at M = 1 / 4 / 16 16.5 / 16.8 / 19.0 -> 15.0 / 15.5 / 18.0 us).
            int l = lane;
            asm volatile("" : "+v"(l));
            f32x4 s = sum_of(wave, l, parity);
            f32x4* const keep = reinterpret_cast<f32x4*>(ysum + (first + wave) * 1024) + l;
            if (!first_pass) s += *keep;
            if (!last_pass) *keep = s;
            if (last_pass && (l & 15) < rows)
                put((gh_ptr)(R.y + size_t(l & 15) * size_t(N)), uint32_t(R.tile0 + first + wave) * 16u + 4u * uint32_t(l >> 4), s);
        }
    };

    // One item of NT tiles starting at tile `first` of the run.  REFILL: each tile's registers are
    // loaded again at once with the tile T further on.
    // REFILL 2 (PASSES): with the first tiles of the next pass, to whose slice the offsets have been moved.
    auto item = [&](auto nt_tag, auto refill_tag, int first, int parity, bool first_pass, bool last_pass) {
        constexpr int NT = decltype(nt_tag)::value;
        constexpr int REFILL = decltype(refill_tag)::value;
        f32x4 part[NT];
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            unsigned char* const reg_t = my_lds + (t & 1) * kRegion;
            // Writing a tile to LDS and asking for the tile that takes its registers is a handful
            // of LDS, scalar and memory instructions; they run at raised priority so that they do
            // not queue behind the other wave's decode (measured: decode sweep 17.55 -> 17.2 us).
            if constexpr (REFILL != 0) __builtin_amdgcn_s_setprio(3);
            *reinterpret_cast<u32x4*>(reg_t + ww_off) = wreg[t][0];
            *reinterpret_cast<u32x4*>(reg_t + kUpperRows + ww_off) = wreg[t][1];
            if constexpr (FINE) *reinterpret_cast<fine_t*>(reg_t + sw_off) = freg[t];
            u32x2 sc_cur[H];
            if constexpr (GS == 256) {
#pragma unroll
                for (int h = 0; h < H; ++h) {
                    // This tile's scales are taken over here, before the refill replaces them: left to itself the compiler
                    // copies those of all tiles at the head of the loop and waits for every request of the item there
                    // (block at M = 4 17.0 -> 16.6 us).
                    sc_cur[h] = sreg[t][h];
                    asm volatile("" : "+v"(sc_cur[h]));
                }
            }
            if constexpr (REFILL != 0) {
                issue_w(REFILL == 2 ? t : first + T + t, t);
                __builtin_amdgcn_s_setprio(0);
                // the requests leave here, as soon as the registers are free: left to itself the
                // scheduler sinks all of an item's loads to its end, which costs two tiles of lead
                __builtin_amdgcn_sched_barrier(0);
            }
            if constexpr (FINE) {
                part[t] = fine_tile(reg_t);
            } else {
            f32x4 acc[3];
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const u32x4 wv = *reinterpret_cast<const u32x4*>(reg_t + (h ? wr_off1 : wr_off0));
                // element e of each half-word sits at bits 2e, 2e+1; the mantissa bits 4..9 (classes
                // 0..2 -> accumulators) hold e = 2,3,4 as loaded, e = 0,1 after << 4 and e = 5,6,7 after >> 6
                const u32x4 sh[3] = {wv << 4, wv, wv >> 6};
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const int src = e < 2 ? 0 : (e < 5 ? 1 : 2);
                    const int j = e < 2 ? e : (e < 5 ? e - 2 : e - 5);
                    const uint32_t mask = 0x00300030u << (2 * j);
                    const u32x4 a = sh[src] & mask;
                    // first product of an accumulator: class 0 starts from the -sum(x) seed, the others from zero
                    const f32x4 c0 = ((GS || h == 0) && (e == 0 || e == 1 || e == 4)) ? (j == 0 ? nsx[GS ? h : 0] : f32x4{0.f, 0.f, 0.f, 0.f}) : acc[j];
                    acc[j] = __builtin_amdgcn_mfma_f32_16x16x32_f16(as_f16x8(a), as_f16x8(breg[h * 8 + e]), c0, 0, 0, 0);
                }
                if constexpr (GS != 0) {
                    // register r of the accumulator is output row 4 (lane / 16) + r of the tile
                    const f16x4 sh4 = __builtin_bit_cast(f16x4, sc_cur[h]);
                    const f32x4 sc = {float(sh4[0]), float(sh4[1]), float(sh4[2]), float(sh4[3])};
                    const f32x4 sum = __builtin_elementwise_fma(__builtin_elementwise_fma(acc[0], f32x4{4.f, 4.f, 4.f, 4.f}, acc[1]),
                                                                f32x4{4.f, 4.f, 4.f, 4.f}, acc[2]);
                    part[t] = h == 0 ? sc * sum : __builtin_elementwise_fma(sc, sum, part[t]);
                }
            }
            // the three classes carry 2^-20, 2^-18 and 2^-16: two fused multiply-adds leave the sum at
            // 2^-16, and that power of two goes into the scale of the epilogue (exact, same roundings)
            if constexpr (GS == 0)
                part[t] = __builtin_elementwise_fma(__builtin_elementwise_fma(acc[0], f32x4{4.f, 4.f, 4.f, 4.f}, acc[1]),
                                                    f32x4{4.f, 4.f, 4.f, 4.f}, acc[2]);
            }
        }
        if constexpr (REFILL == 2) {
#pragma unroll
            for (int t = NT; t < T; ++t) issue_w(t, t);
        }
#pragma unroll
        for (int t = 0; t < NT; ++t) reinterpret_cast<f32x4*>(my_lds + kSums + parity * (T * 1024) + t * 1024)[lane] = part[t];
        exchange(NT, first, parity, first_pass, last_pass);
    };
    const int n_items = (ntiles + T - 1) / T;
    typedef std::integral_constant<int, 0> None;
    typedef std::integral_constant<int, 1> Refill;
    typedef std::integral_constant<int, 2> NextPass;
    typedef std::integral_constant<int, 1> N1;
    typedef std::integral_constant<int, (T >= 2 ? 2 : 1)> N2;
    typedef std::integral_constant<int, T> NT;
    auto last_item = [&](auto refill, int i, bool first_pass, bool last_pass) {
        const int rem = ntiles - i * T;                    // 1 .. T tiles are left
        if (T == 1 || rem == 1) item(N1{}, refill, i * T, i & 1, first_pass, last_pass);
        else if (T == 2 || rem == 2) item(N2{}, refill, i * T, i & 1, first_pass, last_pass);
        else item(NT{}, refill, i * T, i & 1, first_pass, last_pass);
    };
    // The items of a wave without a slice, which it can only be in the last pass: it takes part in the exchange alone.
    auto idle_items = [&](bool first_pass) {
        for (int i = 0; i < n_items; ++i) {
            const int left = ntiles - i * T;
#pragma unroll
            for (int t = 0; t < T; ++t) reinterpret_cast<f32x4*>(my_lds + kSums + (i & 1) * (T * 1024) + t * 1024)[lane] = f32x4{0.f, 0.f, 0.f, 0.f};
            exchange(left < T ? left : T, i * T, i & 1, first_pass, true);
        }
    };
    if constexpr (kIdle) {
        if (idle) { idle_items(true); return; }
    }
    if constexpr (!PASSES) {
        int i = 0;
        for (; i + 1 < n_items; ++i) item(NT{}, Refill{}, i * T, i & 1, true, true);
        last_item(None{}, i, true, true);
    } else {
        // The operands are built in one place, at the start of a pass: built before the loop and at the end of a pass, they were copied into the same
        // registers in each, 136 instructions (4096 x 11008 with groups of 256 at M = 1 8.5 -> 7.8 us, block of four linears at M = 4 14.4 -> 13.9, with
        // groups of 256 15.2 -> 14.3).
        for (int pass = 0; pass < n_pass; ++pass) {
            const bool first_pass = pass == 0, last_pass = pass + 1 == n_pass;
            build();
            int i = 0;
            for (; i + 1 < n_items; ++i) item(NT{}, Refill{}, i * T, i & 1, first_pass, last_pass);
            if (last_pass) {
                last_item(None{}, i, first_pass, true);
            } else {
                const int slice = (pass + 1) * NW + wave;
                // no slice: outside the buffers, which read as zero without a request to memory
                voff0 = slice < slices ? offset_of(slice) : 0x80000000u;
                voff1 = voff0 + 8u * row_bytes;
                scales_of(slice);
                last_item(NextPass{}, i, first_pass, false);
                // the activations land where other waves may still be reading this item's sums
                __builtin_amdgcn_s_waitcnt(0xF | (0x3 << 14) | (0x7 << 4));
                __builtin_amdgcn_s_barrier();
                if (slice >= slices) { idle_items(false); return; }
                if constexpr (ANY) {
                    stage_any(slice, [] {});
                } else {
                    stage_x(slice);
                    __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));  // requested after the weights: wait for all
                }
            }
        }
    }
}

// ------------------------------------------------------------------------------------------
// Long-K form of the lean kernel: 4096 < K <= 16384 and at most T tiles per workgroup, i.e. the
// lone down projection of a block at decode batch sizes (11008 -> 4096, 14336 -> 4096), where a
// workgroup's whole share is one or two tiles and the time is a chain of memory round trips unless
// they overlap.  Wave w owns the K slices w, w + 8, w + 16, w + 24 ("passes").  All of a pass's
// data -- the activation slice by LDS-DMA, the T tile slices of weights into one of two register
// sets -- is requested while the pass before it is decoded, so the chain is one round trip plus
// the decodes:
//     x(0), W(0), W(1) | build(0) | x(1) | decode(0) | wait all | build(1) | W(2), x(2) | decode(1) | ...
// The accumulators of the T tiles stay in registers over all passes (three position classes each),
// the -sum(x) seeds of the passes add up in one accumulator, and the waves exchange partial sums
// once, at the end.  The LDS-DMA requests are inline assembly: for a transfer it knows of, the
// compiler drains the memory pipeline before every later LDS access, which would undo the overlap;
// every wait for them is an explicit s_waitcnt (and since the compiler's own count of outstanding
// loads starts afresh at each of those, the weight loads issued after it are waited for exactly).
constexpr int kLongMaxPasses = 4;
constexpr int kLongWaveLds = kWaveLds + 2048;     // 16 KB of activation staging + one tile slice

// ROWS: 0, or any K and N (see gemv_lean_kernel) and up to ROWS rows, whose next slice waits in registers while a pass is decoded.
template <int T, int ROWS, class Args>
__global__ void __launch_bounds__(512)
gemv_longk_kernel(Args b)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char lds_raw[];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int NW = blockDim.x >> 6;
    unsigned char* const my_lds = lds_raw + wave * kLongWaveLds;
    unsigned char* const tile_buf = my_lds + kWaveLds;
    typedef const __attribute__((address_space(1))) unsigned char* gbytes;

    const auto& R = b.mine();
    const int K = R.K, N = R.N, rows = R.Mrem, ntiles = R.ntiles;
    const int slices = (K + kSliceK - 1) / kSliceK;
    const int P = __builtin_amdgcn_readfirstlane((slices - wave + NW - 1) / NW);   // passes of this wave, >= 1
    const uint32_t row_bytes = ROWS ? ((uint32_t(K) + 15u) >> 4) * 4u : uint32_t(K) >> 2;
    const uint32_t tile_bytes = 16u * row_bytes;

    const int lr = lane >> 3, lc = lane & 7;   // load mapping: row of the half tile, chunk of the slice
    const int mi = lane & 15, mg = lane >> 4;  // MFMA mapping: row / activation column, k group

    // ---- activations of slice wave + NW * p -> staging, swizzled (lane l fetches piece l ^ (r & 7) of row r)
    const uint32_t stage_addr = uint32_t(uintptr_t((const __attribute__((address_space(3))) unsigned char*)my_lds));
    auto dma16 = [&](gbytes src, uint32_t lds_base) {       // lane l: 16 bytes from src (per lane) to lds_base + 16 l
        const uint32_t base = __builtin_amdgcn_readfirstlane(lds_base);
        // s_nop: the wait state that a transfer needs behind a scalar write of M0
        asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off" : : "v"(src), "s"(base) : "memory");
    };
    u32x4 xv[ROWS ? ROWS : 1];
    auto stage_x = [&](int p) {
        if constexpr (ROWS != 0) {
            fetch_rows((gbytes)R.x, rows, K, wave + NW * p, lane, xv);
            __builtin_amdgcn_sched_barrier(0);
            return;
        }
        const int sl = wave + NW * p;
        const size_t row_stride = size_t(K) * 2;
        gbytes src = (gbytes)(R.x + size_t(sl) * (kSliceK * 2));
        if ((sl + 1) * kSliceK <= K) {                      // the whole slice lies inside K
            const uint32_t lane16 = uint32_t(lane) << 4;
#pragma unroll 1
            for (int r = 0; r < rows; ++r) {
                dma16(src + (lane16 ^ (uint32_t(r & 7) << 4)), stage_addr + uint32_t(r) * 1024u);
                src += row_stride;
            }
        } else {
#pragma unroll 1
            for (int r = 0; r < rows; ++r) {
                const int kk = (lane ^ (r & 7)) << 3;      // first of this lane's 8 activations within the slice
                if (sl * kSliceK + kk < K) {
                    dma16(src + uint32_t(kk) * 2u, stage_addr + uint32_t(r) * 1024u);
                } else {
                    *reinterpret_cast<u32x4*>(my_lds + r * 1024 + (uint32_t(lane) << 4)) = u32x4{0u, 0u, 0u, 0u};
                }
                src += row_stride;
            }
        }
    };

    // ---- weights: the T tile slices of a pass into register set `set`
    const __amdgpu_buffer_rsrc_t wres = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<unsigned char*>(R.W), 0, ROWS ? uint32_t(N - R.tile0 * 16 < ntiles * 16 ? N - R.tile0 * 16 : ntiles * 16) * row_bytes : uint32_t(ntiles) * tile_bytes, 0x00020000);
    u32x4 wreg[2][T][2];
    auto issue_w = [&](auto set_tag, int p) {
        constexpr int SET = decltype(set_tag)::value;
        uint32_t chunk = uint32_t(wave + NW * p) * 8u + uint32_t(lc);
        if (!ROWS && chunk >= (uint32_t(K) >> 6)) chunk = 0;        // past K: multiplied by zero activations
        const uint32_t voff0 = uint32_t(lr) * row_bytes + (ROWS ? chunk_place(chunk, row_bytes) : chunk * 16u);
        const uint32_t voff1 = voff0 + 8u * row_bytes;
#pragma unroll
        for (int t = 0; t < T; ++t) {
            const uint32_t so = uint32_t(t < ntiles ? t : ntiles - 1) * tile_bytes;   // past the run: its last tile again
            wreg[SET][t][0] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(wres, voff0, so, 2));   // 2: nt
            wreg[SET][t][1] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(wres, voff1, so, 2));
        }
    };

    // ---- staged activations -> MFMA B operands (as in gemv_lean_kernel); the pass's -sum(x) goes into nsx
    uint32_t breg[2][4][8];
    f32x4 nsx = f32x4{0.f, 0.f, 0.f, 0.f};
    int mr = 1;
    while (mr < rows) mr *= 2;
    const int xrow = mi & (mr - 1);
    const uint32_t xr_off = uint32_t(xrow) * 1024u + uint32_t(mg) * 128u;
    const uint32_t sw = uint32_t(xrow & 7);
    const bool live = mi < rows;
    const uint32_t sel_lo = live ? 0x05040100u : 0x0c0c0c0cu;
    const uint32_t sel_hi = live ? 0x07060302u : 0x0c0c0c0cu;
    auto build = [&](int p) {
        if constexpr (ROWS != 0) put_rows(my_lds, rows, K, wave + NW * p, lane, xv);
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int wd = 0; wd < 4; ++wd) {
                const u32x4 lo = *reinterpret_cast<const u32x4*>(my_lds + xr_off + h * 512 + ((uint32_t(2 * wd) ^ sw) << 4));
                const u32x4 hi = *reinterpret_cast<const u32x4*>(my_lds + xr_off + h * 512 + ((uint32_t(2 * wd + 1) ^ sw) << 4));
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    breg[h][wd][2 * r] = __builtin_amdgcn_perm(hi[r], lo[r], sel_lo);
                    breg[h][wd][2 * r + 1] = __builtin_amdgcn_perm(hi[r], lo[r], sel_hi);
                }
            }
        const uint32_t c = 0x80108010u;                   // fp16 pair of -2^-20
        const u32x4 a = u32x4{c, c, c, c};
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const u32x4 bb = u32x4{breg[h][0][e], breg[h][1][e], breg[h][2][e], breg[h][3][e]};
                nsx = __builtin_amdgcn_mfma_f32_16x16x32_f16(as_f16x8(a), as_f16x8(bb), nsx, 0, 0, 0);
            }
        // the staging area may be written again: every read above has returned
        __builtin_amdgcn_s_waitcnt(0xF | (0x3 << 14) | (0x7 << 4));      // lgkmcnt(0)
    };

    // ---- one pass of the T tiles from register set `set` into the tiles' accumulators
    const uint32_t ww_off = uint32_t(lr) * 128u + (uint32_t(lc ^ lr) << 4);
    const uint32_t wr_off0 = uint32_t(mi) * 128u + (uint32_t((mg) ^ (mi & 7)) << 4);
    const uint32_t wr_off1 = uint32_t(mi) * 128u + (uint32_t((4 + mg) ^ (mi & 7)) << 4);
    f32x4 acc[T][3];
#pragma unroll
    for (int t = 0; t < T; ++t)
#pragma unroll
        for (int j = 0; j < 3; ++j) acc[t][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    auto decode = [&](auto set_tag) {
        constexpr int SET = decltype(set_tag)::value;
#pragma unroll
        for (int t = 0; t < T; ++t) {
            *reinterpret_cast<u32x4*>(tile_buf + ww_off) = wreg[SET][t][0];
            *reinterpret_cast<u32x4*>(tile_buf + 1024 + ww_off) = wreg[SET][t][1];
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const u32x4 wv = *reinterpret_cast<const u32x4*>(tile_buf + (h ? wr_off1 : wr_off0));
                // element e of each half-word sits at bits 2e, 2e+1; the mantissa bits 4..9 (classes
                // 0..2 -> accumulators) hold e = 2,3,4 as loaded, e = 0,1 after << 4 and e = 5,6,7 after >> 6
                const u32x4 sh[3] = {wv << 4, wv, wv >> 6};
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const int src = e < 2 ? 0 : (e < 5 ? 1 : 2);
                    const int j = e < 2 ? e : (e < 5 ? e - 2 : e - 5);
                    const uint32_t mask = 0x00300030u << (2 * j);
                    const u32x4 a = sh[src] & mask;
                    const u32x4 bb = u32x4{breg[h][0][e], breg[h][1][e], breg[h][2][e], breg[h][3][e]};
                    acc[t][j] = __builtin_amdgcn_mfma_f32_16x16x32_f16(as_f16x8(a), as_f16x8(bb), acc[t][j], 0, 0, 0);
                }
            }
        }
    };
    using Set0 = std::integral_constant<int, 0>;
    using Set1 = std::integral_constant<int, 1>;

    // ---- prologue: x(0), W(0), W(1) requested at once
    stage_x(0);
    issue_w(Set0{}, 0);
    if (P > 1) {
        issue_w(Set1{}, 1);
        __builtin_amdgcn_s_waitcnt(vmcnt_imm(4 * T));      // x(0) is in
        build(0);
        __builtin_amdgcn_s_waitcnt(vmcnt_imm(2 * T));      // W(0) is in
        stage_x(1);
    } else {
        __builtin_amdgcn_s_waitcnt(vmcnt_imm(2 * T));
        build(0);
        __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));
    }
    for (int p = 0; p < P; p += 2) {
        decode(Set0{});                                    // pass p
        if (p + 1 < P) {
            __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));      // x(p + 1) and W(p + 1) are in
            build(p + 1);
            if (p + 2 < P) {
                issue_w(Set0{}, p + 2);
                stage_x(p + 2);
            }
            decode(Set1{});                                // pass p + 1
            if (p + 2 < P) {
                __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));
                build(p + 2);
                if (p + 3 < P) {
                    issue_w(Set1{}, p + 3);
                    stage_x(p + 3);
                }
            }
        }
    }

    // ---- split-K: partial sums (at 2^-16, see gemv_lean_kernel) into the staging area, one barrier, fixed-order sum
    const float gamma = R.gamma * 65536.f;
    typedef __attribute__((address_space(1))) __half* gh_ptr;
#pragma unroll
    for (int t = 0; t < T; ++t) {
        const f32x4 four = f32x4{4.f, 4.f, 4.f, 4.f};
        const f32x4 part = __builtin_elementwise_fma(__builtin_elementwise_fma(acc[t][0] + nsx, four, acc[t][1]), four, acc[t][2]);
        reinterpret_cast<f32x4*>(my_lds + t * 1024)[lane] = part;
    }
    __builtin_amdgcn_s_waitcnt(0xF | (0x3 << 14) | (0x7 << 4));
    __builtin_amdgcn_s_barrier();
    const int ot = int(threadIdx.x) >> 6;
    if (ot < T && ot < ntiles) {
        f32x4 v[8];
#pragma unroll
        for (int w = 0; w < 8; ++w)
            v[w] = (w < NW) ? reinterpret_cast<const f32x4*>(lds_raw + w * kLongWaveLds + ot * 1024)[lane]
                            : f32x4{0.f, 0.f, 0.f, 0.f};
        const f32x4 s = ((v[0] + v[1]) + (v[2] + v[3])) + ((v[4] + v[5]) + (v[6] + v[7]));
        if (mi < rows) {
            gh_ptr const yrow = (gh_ptr)(R.y + size_t(mi) * size_t(N));
            const uint32_t ycol = uint32_t(R.tile0 + ot) * 16u + 4u * uint32_t(mg);
            if constexpr (ROWS != 0) {
                store_quad_any(yrow, int(ycol), N, s, gamma);
                return;
            }
            const f16x2 lo = {(_Float16)(gamma * s[0]), (_Float16)(gamma * s[1])};
            const f16x2 hi = {(_Float16)(gamma * s[2]), (_Float16)(gamma * s[3])};
            *(__attribute__((address_space(1))) u32x2*)(yrow + ycol) =
                u32x2{__builtin_bit_cast(uint32_t, lo), __builtin_bit_cast(uint32_t, hi)};
        }
    }
}

using KernelFn = void (*)(GemvBatch);

template <bool MULTI>
KernelFn pick_kernel_t(int T)
{
    switch (T) {
        case 1: return gemv_kernel<1, MULTI>;
        case 2: return gemv_kernel<2, MULTI>;
        case 3: return gemv_kernel<3, MULTI>;
        default: return gemv_kernel<4, MULTI>;
    }
}

KernelFn pick_kernel(int T, bool multi)
{
    return multi ? pick_kernel_t<true>(T) : pick_kernel_t<false>(T);
}

template <bool MULTI, bool PASSES>
KernelFn pick_stream_t(int T)
{
    switch (T) {
        case 1: return gemv_stream_kernel<1, MULTI, PASSES, 1>;
        case 2: return gemv_stream_kernel<2, MULTI, PASSES, 1>;
        case 3: return gemv_stream_kernel<3, MULTI, PASSES, 1>;
        default: return gemv_stream_kernel<4, MULTI, PASSES, 1>;
    }
}

KernelFn pick_stream(int T, bool multi, bool passes, int nb)
{
    if (nb == 2) {                                         // two row blocks: T <= 2
        if (passes) return T == 1 ? gemv_stream_kernel<1, true, true, 2> : gemv_stream_kernel<2, true, true, 2>;
        if (T == 1) return multi ? gemv_stream_kernel<1, true, false, 2> : gemv_stream_kernel<1, false, false, 2>;
        return multi ? gemv_stream_kernel<2, true, false, 2> : gemv_stream_kernel<2, false, false, 2>;
    }
    if (passes) return multi ? pick_stream_t<true, true>(T) : pick_stream_t<false, true>(T);
    return multi ? pick_stream_t<true, false>(T) : pick_stream_t<false, false>(T);
}

int pow2_at_least(int v)
{
    int r = 1;
    while (r < v) r *= 2;
    return r;
}

constexpr int kMaxLds = 8 * kWaveLds;    // most dynamic LDS any launch asks for (8 waves, one item)

// Launch policy.  One 16-row job alone: 8-wave groups, one per CU, one item each while that
// covers the matrix.  Several jobs: 4-wave groups (two passes over K = 4096), two per CU, so
// that one group's wait for HBM overlaps the other's arithmetic, each looping over its items.
struct GemvPolicy {
    int nw_single = 8, nw_grouped = 4;
    int grid_cap = 512;                 // resident workgroups of the grouped form (2 per CU)
    int t_grouped = 0;                  // 0: pick from the tile count
    int stream = 3;                     // bit 0: stream form for one job, bit 1: for several
    int stream_groups = 256;            // workgroups of the stream form (one per CU)
    int two_blocks = 1;                 // jobs of more than 16 rows go in blocks of 32 (two row blocks per wave)
    double start_up_per_row = 0.15;     // stream form: start-up of a pass in tiles per activation row
    double pass_start = 1.5;            // stream form: wait of every pass but the first for its activations, in tiles
    int item_cost = 1;                  // stream form: allocation counts items, not only tiles
    double item_first = 2.1;            // cost of the first tile of an item, in average tiles
    double tile_extra = 0.43;           // cost of each further tile of an item
    int t_stream = 0;                   // stream form: cap on tiles per item (0: none)
    int long_k_min_run = 3;             // K > 4096 streams if the call averages this many tile passes per workgroup
    int lean = 1;                       // launches the lean kernel can take go to it
    int longk = 1;                      // lone calls with 4096 < K <= 16384 and at most two tiles per workgroup: long-K form
};
const GemvPolicy g_policy{};   // fixed in the library; development builds patch this line to try other values

constexpr int kStreamWaves = 8;         // waves of a stream-form workgroup when K >= 4096
constexpr int kStreamMaxPasses = 8;     // passes over K the stream form takes: K <= 32768
constexpr int kStreamMaxRun = 32;       // tiles of a run whose sums fit the 32 KB of LDS left over

template <class Args>
using LeanFn = void (*)(Args);

template <class Args, bool PASSES, int GS, bool ANY>
LeanFn<Args> pick_lean(int T)
{
    switch (T) {
        case 1: return gemv_lean_kernel<1, PASSES, GS, ANY, Args>;
        case 2: return gemv_lean_kernel<2, PASSES, GS, ANY, Args>;
        default: return gemv_lean_kernel<3, PASSES, GS, ANY, Args>;
    }
}

constexpr int lean_lds(bool passes) { return 8 * stream_wave_lds(3) + (passes ? kStreamMaxRun * 1024 : 0); }

// kept: tiles of the longest run of a job of several passes
template <bool PASSES, int GS, bool ANY, class Args>
hipError_t launch_lean_args(const Args& args, dim3 grid, int NW, int T, int kept, hipStream_t s)
{
    const LeanFn<Args> fn = pick_lean<Args, PASSES, GS, ANY>(T);
    static std::atomic<bool> lds_raised[kMaxDevices][4];
    const int dev = device_slot();
    if (dev < 0 || !lds_raised[dev][T]) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(fn),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, lean_lds(PASSES));
        if (e != hipSuccess) return e;
        if (dev >= 0) lds_raised[dev][T] = true;
    }
    hipLaunchKernelGGL(fn, grid, dim3(NW * 64), size_t(NW) * stream_wave_lds(T) + size_t(kept) * 1024, s, args);
    return hipGetLastError();
}

template <bool ANY, class Args>
hipError_t launch_lean_args(const Args& args, dim3 grid, int NW, int T, int kept, int gs, hipStream_t s)
{
    auto with = [&](auto tag) {
        constexpr int GS = decltype(tag)::value;
        if constexpr (!(std::is_same<Args, LeanAny>::value && GS == 0 && !ANY))   // which is one pass over K
            if (kept) return launch_lean_args<true, GS, ANY>(args, grid, NW, T, kept, s);
        return launch_lean_args<false, GS, ANY>(args, grid, NW, T, 0, s);
    };
    switch (gs) {
        case 0: return with(std::integral_constant<int, 0>{});
        case 32: return with(std::integral_constant<int, 32>{});
        case 64: return with(std::integral_constant<int, 64>{});
        case 128: return with(std::integral_constant<int, 128>{});
        default: return with(std::integral_constant<int, 256>{});
    }
}

// What the groups of a scale are multiples of, of the kinds the lean kernel knows; 0: of none
int lean_scale_kind(int64_t group) { return group % 256 == 0 ? 256 : group % 128 == 0 ? 128 : group % 64 == 0 ? 64 : group % 32 == 0 ? 32 : 0; }

// ceil(2^31 / units per group): u * inverse / 2^31 rounded down is u / hpg for every u and hpg up to 2^15 (the error of the
// inverse, below 2^-31, times u stays below the 1 / hpg that is missing to the next whole number), and K holds at most
// kStreamWaves kStreamMaxPasses slices.  (J.hpg is at most the units of K, see launch_gemv_gs_jobs.)
uint32_t group_inverse(const GemvJob& J)
{
    if (J.scales == nullptr) return 0;
    const uint32_t hpg = uint32_t(J.hpg);
    return uint32_t(((uint64_t(1) << 31) + hpg - 1) / hpg);
}
static_assert(kSliceK / 32 * kStreamWaves * kStreamMaxPasses <= 1 << 15, "group_inverse");

LeanOne one_job(const uint32_t* W, const __half* x, __half* y, float gamma, int K, int N, int rows, int tiles, int grid,
                const __half* scales = nullptr, uint32_t group_inv = 0)
{
    return LeanOne{reinterpret_cast<const unsigned char*>(W), reinterpret_cast<const unsigned char*>(x), y, gamma, K, N, rows,
                   tiles / grid, tiles % grid, group_inv, reinterpret_cast<const unsigned char*>(scales)};
}

// Launch of the lean kernel: wg[j] workgroups for job j, each with a run of consecutive tiles
// (the first tiles % wg[j] of them one tile longer), written out as one record per workgroup.
hipError_t launch_lean(const GemvBatch& b, const int* wg, int NW, int T, int kept, int gs, bool any, bool table, hipStream_t s)
{
    if (b.count == 1 && gs == 0 && !any) {
        const GemvJob& J = b.job[0];
        const LeanOne args = one_job(J.W, J.x, J.y, J.gamma, J.K, J.N, J.Mrem, J.tiles, wg[0]);
        return kept ? launch_lean_args<true, 0, false>(args, dim3(wg[0]), NW, T, kept, s) : launch_lean_args<false, 0, false>(args, dim3(wg[0]), NW, T, 0, s);
    }
    if (table) {
        auto fill = [&](auto gs_tag, auto jobs_tag) {
            constexpr int GS = decltype(gs_tag)::value;
            LeanJobs<decltype(jobs_tag)::value> lj;
            int grid = 0;
            for (int j = 0; j < lj.kJobs; ++j) {
                lj.first[j] = j < b.count ? grid : 0x7fffffff;
                if (j >= b.count) continue;
                const GemvJob& J = b.job[j];
                lj.job[j] = one_job(J.W, J.x, J.y, J.gamma, J.K, J.N, J.Mrem, J.tiles, wg[j], J.scales, group_inverse(J));
                grid += wg[j];
            }
            return any ? launch_lean_args<false, GS, true>(lj, dim3(grid), NW, T, 0, s) : launch_lean_args<false, GS, false>(lj, dim3(grid), NW, T, 0, s);
        };
        // the larger table takes small launches 0.1 us longer
        auto with = [&](auto gs_tag) {
            if constexpr (decltype(gs_tag)::value != 0)
                if (b.count > kTableJobs) return fill(gs_tag, std::integral_constant<int, kTableMost>{});
            return fill(gs_tag, std::integral_constant<int, kTableJobs>{});
        };
        switch (gs) {
            case 0: return with(std::integral_constant<int, 0>{});
            case 32: return with(std::integral_constant<int, 32>{});
            case 64: return with(std::integral_constant<int, 64>{});
            case 128: return with(std::integral_constant<int, 128>{});
            default: return with(std::integral_constant<int, 256>{});
        }
    }
    LeanBatch lb;
    int grid = 0;
    for (int j = 0; j < b.count; ++j) {
        const GemvJob& J = b.job[j];
        const int per = J.tiles / wg[j], plus = J.tiles % wg[j];
        const size_t tile_bytes = packed_tile_bytes(J.K);
        const uint32_t inv = group_inverse(J);
        for (int g = 0; g < wg[j]; ++g) {
            WgRec& r = lb.rec[grid++];
            r.tile0 = g * per + (g < plus ? g : plus);
            r.ntiles = per + (g < plus ? 1 : 0);
            r.W = reinterpret_cast<const unsigned char*>(J.W) + size_t(r.tile0) * tile_bytes;
            r.x = reinterpret_cast<const unsigned char*>(J.x);
            r.y = J.y;
            r.gamma = J.gamma;
            r.K = J.K; r.N = J.N; r.Mrem = J.Mrem;
            r.sc = reinterpret_cast<const unsigned char*>(J.scales);
            r.group_inv = inv; r.pad = 0;
        }
    }
    return any ? launch_lean_args<true>(lb, dim3(grid), NW, T, kept, gs, s) : launch_lean_args<false>(lb, dim3(grid), NW, T, kept, gs, s);
}

// Tiles per item of a launch whose longest run is `run` (see launch_stream), at most one output quad per thread
int tiles_per_item(int run, int NW)
{
    const int T = run <= 3 ? run : (run == 4 ? 2 : 3);
    return T < NW ? T : NW;
}

// rows: 0, or the rows of a call of any K and N
template <class Args>
LeanFn<Args> pick_longk(int T, int rows)
{
    if constexpr (std::is_same<Args, LeanAny>::value) {
        if (rows <= 1) return T == 1 ? gemv_longk_kernel<1, 1, Args> : gemv_longk_kernel<2, 1, Args>;
        if (rows <= 4) return T == 1 ? gemv_longk_kernel<1, 4, Args> : gemv_longk_kernel<2, 4, Args>;
        return T == 1 ? gemv_longk_kernel<1, 16, Args> : gemv_longk_kernel<2, 16, Args>;
    } else {
        return T == 1 ? gemv_longk_kernel<1, 0, Args> : gemv_longk_kernel<2, 0, Args>;
    }
}

template <class Args>
hipError_t launch_longk_args(const Args& args, dim3 grid, int T, int rows, hipStream_t s)
{
    const LeanFn<Args> fn = pick_longk<Args>(T, rows);
    static std::atomic<bool> lds_raised[kMaxDevices][3][3];
    const int dev = device_slot(), kind = rows <= 1 ? 0 : (rows <= 4 ? 1 : 2);
    if (dev < 0 || !lds_raised[dev][T][kind]) {
        const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(fn),
                                                 hipFuncAttributeMaxDynamicSharedMemorySize, kStreamWaves * kLongWaveLds);
        if (e != hipSuccess) return e;
        if (dev >= 0) lds_raised[dev][T][kind] = true;
    }
    hipLaunchKernelGGL(fn, grid, dim3(kStreamWaves * 64), size_t(kStreamWaves) * kLongWaveLds, s, args);
    return hipGetLastError();
}

// One product: a set of workgroups for every block of 16 rows (blockIdx.y), as many in all as the CUs hold with 8 waves each.
// any: of any K and N; else K is a multiple of 64 and N of 16, and there are scales or K is one pass.
hipError_t launch_lean_rows(const __half* x, const uint32_t* W, float gamma, const __half* scales, uint32_t group_inv, __half* y,
                            int64_t M, int64_t N, int64_t K, int gs, bool any, hipStream_t s)
{
    const int slices = int((K + kSliceK - 1) / kSliceK), NW = slices < kStreamWaves ? slices : kStreamWaves;
    const int tiles = int((N + 15) / 16), blocks = int((M + 15) / 16);
    if (scales == nullptr && slices > kStreamWaves && slices <= kStreamWaves * kLongMaxPasses && int64_t(tiles) * blocks <= 2 * kLeanMaxGroups) {
        // one or two tiles to a workgroup: the long-K form
        const int T = tiles * blocks <= kLeanMaxGroups ? 1 : 2, groups = (tiles + T - 1) / T;
        const LeanAny args{one_job(W, x, y, gamma, int(K), int(N), int(M), tiles, groups)};
        return launch_longk_args(args, dim3(groups, blocks), T, int(M), s);
    }
    int64_t share = int64_t(kLeanMaxGroups) * (kStreamWaves / NW) / blocks;
    const int64_t longest = slices > NW ? kStreamMaxRun : (int64_t(1) << 31) / int64_t(packed_tile_bytes(int(K)));   // a run's kept sums, its bytes
    if (share < (tiles + longest - 1) / longest) share = (tiles + longest - 1) / longest;
    const int groups = share < 1 ? 1 : (tiles < share ? tiles : int(share));
    const int run = (tiles + groups - 1) / groups, T = tiles_per_item(run, NW);
    const LeanAny args{one_job(W, x, y, gamma, int(K), int(N), int(M), tiles, groups, scales, group_inv)};
    const int kept = slices > NW ? run : 0;
    if (!any && gs == 256 && blocks == 1) {                // spares 0.1 us of working out which block
        const LeanOne& one = args;
        return kept ? launch_lean_args<true, 256, false>(one, dim3(groups), NW, T, kept, s) : launch_lean_args<false, 256, false>(one, dim3(groups), NW, T, 0, s);
    }
    return any ? launch_lean_args<true>(args, dim3(groups, blocks), NW, T, kept, gs, s) : launch_lean_args<false>(args, dim3(groups, blocks), NW, T, kept, gs, s);
}

// Calls in which every GEMM has 4096 < K <= 16384 and N a multiple of 16, and which hold at most two
// tiles per workgroup in all (the lone down projection of a block: 11008 -> 4096, 14336 -> 4096):
// the long-K form of the lean kernel, one record per workgroup with its one or two tiles.  Returns
// false, and launches nothing, for any other call.
bool launch_longk(const GemmDesc* jobs, int count, hipStream_t s, hipError_t* err)
{
    int64_t tiles_total = 0;
    for (int i = 0; i < count; ++i) {
        const GemmDesc& d = jobs[i];
        const int64_t slices = (d.K + kSliceK - 1) / kSliceK;
        if (slices <= kStreamWaves || slices > int64_t(kStreamWaves) * kLongMaxPasses || (d.N & 15) != 0) return false;
        tiles_total += ((d.M + 15) / 16) * (d.N / 16);
        if (tiles_total > 2 * kLeanMaxGroups) return false;
    }
    const int T = tiles_total <= kLeanMaxGroups ? 1 : 2;
    int64_t groups = 0;
    for (int i = 0; i < count; ++i) groups += ((jobs[i].M + 15) / 16) * ((jobs[i].N / 16 + T - 1) / T);
    if (groups > kLeanMaxGroups) return false;
    if (count == 1 && jobs[0].M <= 16) {
        const GemmDesc& d = jobs[0];
        *err = launch_longk_args(one_job(d.W, d.x, d.y, d.gamma, int(d.K), int(d.N), int(d.M), int(d.N / 16), int(groups)), dim3(unsigned(groups)), T, 0, s);
        return true;
    }
    LeanBatch lb;
    int grid = 0;
    for (int i = 0; i < count; ++i) {
        const GemmDesc& d = jobs[i];
        const int tiles = int(d.N / 16);
        const size_t tile_bytes = size_t(16) * (size_t(d.K) / 4);
        for (int64_t m0 = 0; m0 < d.M; m0 += 16) {
            for (int t0 = 0; t0 < tiles; t0 += T) {
                WgRec& r = lb.rec[grid++];
                r.tile0 = t0;
                r.ntiles = tiles - t0 < T ? tiles - t0 : T;
                r.W = reinterpret_cast<const unsigned char*>(d.W) + size_t(t0) * tile_bytes;
                r.x = reinterpret_cast<const unsigned char*>(d.x + m0 * d.K);
                r.y = d.y + m0 * d.N;
                r.gamma = d.gamma;
                r.K = int(d.K); r.N = int(d.N);
                r.Mrem = int(d.M - m0 < 16 ? d.M - m0 : 16);
                r.sc = nullptr; r.group_inv = 0; r.pad = 0;
            }
        }
    }
    *err = launch_longk_args(lb, dim3(grid), T, 0, s);
    return true;
}

// Whether what is enqueued now becomes part of a graph.  (The null stream cannot be captured, and asking about it while another stream is fails.)
bool being_captured(hipStream_t s)
{
    if (s == nullptr) return false;
    hipStreamCaptureStatus status = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(s, &status) == hipSuccess) return status != hipStreamCaptureStatusNone;
    (void)hipGetLastError();
    return false;
}

// Stream form: one job per workgroup, a run of consecutive tiles each.  Workgroups are dealt
// out to the jobs so that all finish together (see run_cost below); spare ones go to the job
// with the costliest runs, one by one.  Returns hipErrorInvalidValue without launching if a multi-pass job's
// runs would not fit the LDS (the caller then uses the general kernel).
// any: jobs of any K and N among them, for the lean kernel's form for those alone.
// gs: 0, or the kind of scales (see lean_scale_kind); below 256 the lean kernel takes them in one of its forms.
hipError_t launch_stream(GemvBatch& b, int max_slices, int nb, hipStream_t s, int gs = 0, bool any = false)
{
    const GemvPolicy pol = g_policy;
    const int NW = max_slices < kStreamWaves ? max_slices : kStreamWaves;
    auto passes = [&](int j) { return (b.job[j].slices + NW - 1) / NW; };
    int64_t total_tiles = 0, w_bytes = 0;
    bool multi_pass = false, short_jobs = false;           // short: fewer slices than waves
    for (int j = 0; j < b.count; ++j) {
        total_tiles += b.job[j].tiles;
        w_bytes += int64_t(b.job[j].tiles) * int64_t(packed_tile_bytes(b.job[j].K));
        short_jobs |= b.job[j].slices < NW;
        multi_pass |= passes(j) > 1;
    }
    // One workgroup of 8 waves per CU; with shorter K (fewer waves per workgroup) as many more
    // workgroups, so that a CU still runs 8 waves (K = 1024: 1024 workgroups of 2 waves).
    const int64_t g_all = int64_t(pol.stream_groups) * (kStreamWaves / NW);
    // With scales the table of jobs also takes what no records hold, more than 256 workgroups or jobs with fewer slices than waves; without, the latter
    // are left to the general form.
    const bool beyond = (total_tiles < g_all ? total_tiles : g_all) > kLeanMaxGroups;
    const bool records = gs == 0 || !(short_jobs || beyond);
    bool table = nb == 1 && !(gs == 0 && short_jobs) && jobs_by_table(b.count, !multi_pass, records, beyond, w_bytes, false);
    if (table && records && !beyond) table = !being_captured(s);
    // What has scales and neither the plain records nor the table take goes to the form for any K and N, for which the workgroups are dealt out once: dealing
    // them out twice cost the host as much again (blocks of 33 to 64 rows 8 us of 23 in a loop).
    if (gs != 0 && !table && !records) any = true;
    const int64_t g_max = any && !table ? kLeanMaxGroups : g_all;
    const int G = total_tiles < g_max ? int(total_tiles) : int(g_max);
    // Time of a workgroup in tile units: passes x (run time + start-up), see tl_deal.hpp.  The
    // start-up of a pass is fetching the activation slice (1 KB per row and wave through the same
    // address path as the weights) and building the operands: measured about 0.15 tiles per
    // activation row; a job of several passes pays part of that round trip in every pass but the
    // first (pass_start tiles).  A run is worked off in items of up to t_max tiles, and an item
    // costs its latency and barrier once: measured (block launch, runs of 15 ... 19 tiles) 1.0 us
    // for the first tile of an item and 0.2 us for each further one, i.e. 2.1 and 0.43 in units
    // of an average tile.
    const DealModel model{nb == 2 ? 2 : 3, pol.item_cost != 0, pol.item_first, pol.tile_extra};
    DealJob dj[kMaxJobs];
    for (int j = 0; j < b.count; ++j) {
        const int rows = b.job[j].Mrem < 16 * nb ? b.job[j].Mrem : 16 * nb;
        dj[j] = DealJob{b.job[j].tiles, passes(j),
                        pol.start_up_per_row * double(rows) + (passes(j) > 1 ? pol.pass_start : 0.0)};
    }
    int wg[kMaxJobs];
    if (b.count == 1) wg[0] = G;                           // all of them (G is at most the job's tiles)
    else deal_workgroups(model, dj, b.count, G, wg);
    int run = 1;                                           // longest run of tiles of a workgroup
    for (int j = 0; j < b.count; ++j) {
        const int r = (b.job[j].tiles + wg[j] - 1) / wg[j];
        if (passes(j) > 1 && r > kStreamMaxRun / nb) return hipErrorInvalidValue;   // 1 KB of kept sums per tile and row block
        if (r > run) run = r;
    }
    // Tiles per item.  Measured: items of 3 tiles stream 3-4 % faster than items of 4 (6 KB
    // against 8 KB requested per wave at a time; with more in flight the memory system slows
    // down), a run of 4 goes best as 2 + 2 (the second pair loads while the first is decoded),
    // and shorter runs are one item.
    int T = tiles_per_item(run, NW);
    if (pol.t_stream > 0 && T > pol.t_stream) T = pol.t_stream;
    if (nb == 2) {                       // two row blocks per job: at most 2 tiles per item (registers)
        if (T > 2) T = 2;
        if (2 * T > NW) T = NW / 2;
        if (T < 1) return hipErrorInvalidValue;
    }
    if (T < 1) T = 1;
    // The lean kernel takes the launch when every job has at least one slice per wave (more: several passes), N is a
    // multiple of 16 throughout and the workgroups fit its record table; with scales else its form for any K and N.  (The linears of a block, K = 4096 three times
    // and 11008, against the general form: M = 1 14.05 -> 13.2, M = 4 14.2 -> 13.9, M = 16 17.6 -> 16.2-16.7 us.)
    bool lean = nb == 1 && T <= 3 && (gs != 0 || (pol.lean && (!short_jobs || table)));
    int total_groups = 0, kept = 0;
    for (int j = 0; j < b.count; ++j) {
        lean = lean && (gs != 0 || (b.job[j].N & 15) == 0);
        total_groups += wg[j];
        const int r = (b.job[j].tiles + wg[j] - 1) / wg[j];
        if (passes(j) > 1 && r > kept) kept = r;
    }
    if (any) return launch_lean(b, wg, NW, T, kept, gs, true, table, s);
    if (lean && (total_groups <= kLeanMaxGroups || table || b.count == 1)) return launch_lean(b, wg, NW, T, kept, gs, false, table, s);
    if (gs != 0) return hipErrorInvalidValue;              // not reached: nothing else reads scales
    for (int j = 0; j < kMaxJobs; ++j) b.item0[j] = 0x7fffffff;
    int grid = 0;
    for (int j = 0; j < b.count; ++j) {
        b.item0[j] = grid;
        b.job[j].items = 0;
        b.job[j].run = b.job[j].tiles / wg[j];
        b.job[j].plus = b.job[j].tiles % wg[j];
        grid += wg[j];
    }
    const size_t lds = size_t(NW) * stream_wave_lds(T * nb) + (multi_pass ? size_t(kStreamMaxRun) * 1024 : 0);
    b.total_items = 0;                                 // the stream form has no item queue
    b.red_off = 0;
    b.pad = 0;
    const bool multi = b.count > 1;
    KernelFn fn = pick_stream(T, multi, multi_pass, nb);
    static std::atomic<bool> lds_raised[kMaxDevices][4][2][kTMax + 1];
    const int variant = nb == 2 ? (multi_pass ? 3 : 2) : (multi_pass ? 1 : 0);
    const int dev = device_slot();
    if (dev < 0 || !lds_raised[dev][variant][multi][T]) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(fn),
                                           hipFuncAttributeMaxDynamicSharedMemorySize,
                                           8 * stream_wave_lds(T) + kStreamMaxRun * 1024);
        if (e != hipSuccess) return e;
        if (dev >= 0) lds_raised[dev][variant][multi][T] = true;
    }
    hipLaunchKernelGGL(fn, dim3(grid), dim3(NW * 64), lds, s, b);
    return hipGetLastError();
}

// Launch one batch (<= kMaxJobs jobs, tiles / slices / M filled in): sets items and grid.
hipError_t launch_batch(GemvBatch& b, bool grouped, bool stream_form, int nb, hipStream_t s)
{
    const GemvPolicy pol = g_policy;
    int64_t total_tiles = 0;
    int max_slices = 1;
    for (int j = 0; j < b.count; ++j) {
        total_tiles += b.job[j].tiles;
        if (b.job[j].slices > max_slices) max_slices = b.job[j].slices;
    }
    if (stream_form && max_slices <= kStreamWaves * kStreamMaxPasses && (pol.stream & (b.count > 1 ? 2 : 1))) {
        const hipError_t e = launch_stream(b, max_slices, nb, s);
        if (e != hipErrorInvalidValue) return e;           // else: runs too long for its LDS, general kernel
    }
    if (nb != 1) {
        // jobs of two row blocks exist for the stream form only: each goes on as two jobs of 16 rows
        GemvBatch h;
        h.count = 0;
        for (int j = 0; j < b.count; ++j) {
            for (int part = 0; part < 2; ++part) {
                const int rows = b.job[j].Mrem - 16 * part;
                if (rows <= 0) break;
                GemvJob q = b.job[j];
                q.x = b.job[j].x + size_t(16 * part) * size_t(q.K);
                q.y = b.job[j].y + size_t(16 * part) * size_t(q.N);
                q.Mrem = rows < 16 ? rows : 16;
                q.mr = pow2_at_least(q.Mrem);
                h.job[h.count++] = q;
                if (h.count == kMaxJobs) {
                    const hipError_t e = launch_batch(h, true, false, 1, s);
                    if (e != hipSuccess) return e;
                    h.count = 0;
                }
            }
        }
        return h.count ? launch_batch(h, true, false, 1, s) : hipSuccess;
    }
    int NW = grouped ? pol.nw_grouped : pol.nw_single;
    if (NW > max_slices) NW = max_slices;
    int resident = grouped ? pol.grid_cap : (NW <= 4 ? 512 : 256);
    int T = (grouped && pol.t_grouped) ? pol.t_grouped : int((total_tiles + resident - 1) / resident);
    if (T > kTMax) T = kTMax;
    if (T < 1) T = 1;
    int total_items = 0;
    for (int j = 0; j < kMaxJobs; ++j) b.item0[j] = 0x7fffffff;
    for (int j = 0; j < b.count; ++j) {
        b.job[j].items = (b.job[j].tiles + T - 1) / T;
        b.item0[j] = total_items;
        total_items += b.job[j].items;
    }
    b.total_items = total_items;
    // Workgroups that loop keep the reduction area behind the staging area; with 8 waves
    // that is more LDS than a CU has, so a looping launch uses 4-wave groups, two per CU.
    if (total_items > resident && NW > 4) { NW = 4; resident = 512; }
    const int grid = total_items < resident ? total_items : resident;
    const bool looping = total_items > grid;
    b.red_off = looping ? NW * kWaveLds : 0;
    const int lds = NW * kWaveLds + (looping ? T * NW * 1024 : 0);
    b.pad = 0;

    const bool multi = b.count > 1;
    KernelFn fn = pick_kernel(T, multi);
    // More than the default 64 KB of dynamic LDS needs the attribute; it is set once per
    // kernel instance and device (idempotent, so threads that meet only repeat it).
    static std::atomic<bool> lds_raised[kMaxDevices][2][kTMax + 1];
    const int dev = device_slot();
    if (dev < 0 || !lds_raised[dev][multi][T]) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(fn),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, kMaxLds);
        if (e != hipSuccess) return e;
        if (dev >= 0) lds_raised[dev][multi][T] = true;
    }
    hipLaunchKernelGGL(fn, dim3(grid), dim3(NW * 64), size_t(lds), s, b);
    return hipGetLastError();
}

}  // namespace

// Raises the dynamic-LDS limit of every kernel instance of this file on the current device (the
// launchers do it on first use otherwise).
hipError_t gemv_init()
{
    const int stream_lds = 8 * kWaveLds + kStreamMaxRun * 1024;
    auto raise = [](KernelFn fn, int bytes) {
        return hipFuncSetAttribute(reinterpret_cast<const void*>(fn), hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
    };
    for (int T = 1; T <= 2; ++T) {
        auto raise_long = [](const void* fn) { return hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, kStreamWaves * kLongWaveLds); };
        hipError_t e = raise_long(reinterpret_cast<const void*>(pick_longk<LeanBatch>(T, 0)));
        if (e == hipSuccess) e = raise_long(reinterpret_cast<const void*>(pick_longk<LeanOne>(T, 0)));
        for (int rows : {1, 4, 16})
            if (e == hipSuccess) e = raise_long(reinterpret_cast<const void*>(pick_longk<LeanAny>(T, rows)));
        if (e != hipSuccess) return e;
    }
    for (int T = 1; T <= 3; ++T) {
        hipError_t e = hipSuccess;
        auto raise_lean = [&](auto gs_tag) {
            constexpr int GS = decltype(gs_tag)::value;
            auto raise_one = [&](const void* fn, bool passes) {
                if (e == hipSuccess) e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, lean_lds(passes));
            };
            raise_one(reinterpret_cast<const void*>(pick_lean<LeanBatch, false, GS, false>(T)), false);
            raise_one(reinterpret_cast<const void*>(pick_lean<LeanBatch, true, GS, false>(T)), true);
            typedef typename std::conditional<GS == 0, LeanOne, LeanAny>::type Alone;
            if constexpr (GS == 0) raise_one(reinterpret_cast<const void*>(pick_lean<LeanAny, false, 0, false>(T)), false);
            if constexpr (GS == 256) {
                raise_one(reinterpret_cast<const void*>(pick_lean<LeanOne, false, 256, false>(T)), false);
                raise_one(reinterpret_cast<const void*>(pick_lean<LeanOne, true, 256, false>(T)), true);
            }
            raise_one(reinterpret_cast<const void*>(pick_lean<Alone, false, GS, false>(T)), false);
            raise_one(reinterpret_cast<const void*>(pick_lean<Alone, true, GS, false>(T)), true);
            raise_one(reinterpret_cast<const void*>(pick_lean<LeanJobs<kTableJobs>, false, GS, false>(T)), false);
            raise_one(reinterpret_cast<const void*>(pick_lean<LeanJobs<kTableJobs>, false, GS, true>(T)), false);
            if constexpr (GS != 0) {
                raise_one(reinterpret_cast<const void*>(pick_lean<LeanJobs<kTableMost>, false, GS, false>(T)), false);
                raise_one(reinterpret_cast<const void*>(pick_lean<LeanJobs<kTableMost>, false, GS, true>(T)), false);
            }
            raise_one(reinterpret_cast<const void*>(pick_lean<LeanBatch, false, GS, true>(T)), false);
            raise_one(reinterpret_cast<const void*>(pick_lean<LeanBatch, true, GS, true>(T)), true);
            raise_one(reinterpret_cast<const void*>(pick_lean<LeanAny, false, GS, true>(T)), false);
            raise_one(reinterpret_cast<const void*>(pick_lean<LeanAny, true, GS, true>(T)), true);
        };
        raise_lean(std::integral_constant<int, 0>{});
        raise_lean(std::integral_constant<int, 32>{});
        raise_lean(std::integral_constant<int, 64>{});
        raise_lean(std::integral_constant<int, 128>{});
        raise_lean(std::integral_constant<int, 256>{});
        if (e != hipSuccess) return e;
    }
    for (int T = 1; T <= kTMax; ++T)
        for (int multi = 0; multi < 2; ++multi) {
            hipError_t e = raise(pick_kernel(T, multi != 0), kMaxLds);
            for (int passes = 0; passes < 2 && e == hipSuccess; ++passes) {
                e = raise(pick_stream(T, multi != 0, passes != 0, 1), stream_lds);
                if (e == hipSuccess && T <= 2) e = raise(pick_stream(T, multi != 0, passes != 0, 2), stream_lds);
            }
            if (e != hipSuccess) return e;
        }
    return hipSuccess;
}

bool gemv_supports(int64_t M, int64_t N, int64_t K)
{
    return M >= 1 && N >= 1 && K >= 64 && (K % 64) == 0 && K <= (int64_t(1) << 24) &&
           N <= (int64_t(1) << 24) && M <= (int64_t(1) << 20);
}

// K that is no multiple of 64: several such jobs, or some among others, share launches of the lean kernel's form for any K.
bool gemv_any_supports(int64_t M, int64_t N, int64_t K)
{
    return M >= 1 && M <= 4096 && N >= 1 && N <= (int64_t(1) << 24) && K >= 64 && K <= int64_t(kStreamWaves) * kStreamMaxPasses * kSliceK;
}

namespace {

// Jobs (each passing gemv_any_supports; all with groups of one kind, or none) in blocks of 16 rows, kMaxJobs of them to a launch
struct AnyJob {
    const __half* x;
    const uint32_t* W;
    const __half* scales;
    __half* y;
    float gamma;
    int64_t M, N, K, group;
};

// Scale units of a group; a group longer than K is the one group there is (the quotient itself need not fit 32 bits)
int units_per_group(int64_t K, int64_t group, int kind)
{
    const int64_t unit = lean_scale_unit(kind), all = (K + unit - 1) / unit;
    return int(group / unit < all ? group / unit : all);
}

hipError_t launch_rows(const GemvJob& j, int64_t M, int gs, bool any, hipStream_t s)
{
    return launch_lean_rows(j.x, j.W, j.gamma, j.scales, group_inverse(j), j.y, M, j.N, j.K, gs, any || j.N % 16 != 0, s);
}

// Blocks of 16 rows in one launch, or, where their runs are too long for what a launch keeps of their sums, half of them in each of two: one launch per
// block took 26 jobs of 33 rows and K up to 11008 418 us (the general kernel 216), halves take 174.
hipError_t launch_blocks(const GemvJob* blocks, int count, int gs, bool any, hipStream_t s)
{
    if (count == 1) return launch_rows(blocks[0], blocks[0].Mrem, gs, any, s);
    GemvBatch b;
    b.count = count;
    int max_slices = 1;
    for (int q = 0; q < count; ++q) {
        b.job[q] = blocks[q];
        if (blocks[q].slices > max_slices) max_slices = blocks[q].slices;
    }
    const hipError_t e = launch_stream(b, max_slices, 1, s, gs, any);
    if (e != hipErrorInvalidValue) return e;
    const hipError_t first = launch_blocks(blocks, count / 2, gs, any, s);
    return first == hipSuccess ? launch_blocks(blocks + count / 2, count - count / 2, gs, any, s) : first;
}

hipError_t launch_any_jobs(const AnyJob* jobs, int count, hipStream_t s, int gs = 0)
{
    GemvJob blocks[kMaxJobs];
    int held = 0;
    auto flush = [&]() -> hipError_t {
        const hipError_t e = held ? launch_blocks(blocks, held, gs, true, s) : hipSuccess;
        held = 0;
        return e;
    };
    for (int i = 0; i < count; ++i) {
        const AnyJob& d = jobs[i];
        GemvJob j{};
        j.x = d.x; j.W = d.W; j.y = d.y; j.gamma = d.gamma;
        j.N = int(d.N); j.K = int(d.K);
        j.tiles = int((d.N + 15) / 16);
        j.slices = int((d.K + kSliceK - 1) / kSliceK);
        j.scales = d.scales; j.hpg = gs ? units_per_group(d.K, d.group, gs) : 0;
        if (count == 1) return launch_rows(j, d.M, gs, true, s);
        for (int64_t m0 = 0; m0 < d.M; m0 += 16) {
            GemvJob q = j;
            q.x = d.x + m0 * d.K;
            q.y = d.y + m0 * d.N;
            q.Mrem = int(d.M - m0 < 16 ? d.M - m0 : 16);
            blocks[held++] = q;
            if (held == kMaxJobs) {
                const hipError_t e = flush();
                if (e != hipSuccess) return e;
            }
        }
    }
    return flush();
}

}  // namespace

hipError_t launch_gemv_jobs(const GemmDesc* jobs, int count, hipStream_t s)
{
    bool any_k = false;
    for (int i = 0; i < count; ++i) any_k = any_k || jobs[i].K % 64 != 0;
    if (any_k) {
        // A job of such a K, and with it those that would share a launch of blocks of 16 rows anyway: a launch of its own costs it more than the form for any K
        // costs its neighbours (270 calls of 1 to 50 aligned jobs, M = 1 .. 64, K = 512 .. 11008, with one or two of such K 0.72 of the time of the aligned
        // jobs' own launches and the tiled kernel's for the others, the slowest 1.03).  But not those of K up to 2048 if all do not fit one launch, since launches of their own hold more
        // workgroups than that form's records: 38 jobs of 64 rows, K = 512, with one of K = 1296 182 us apart, 214 together.
        constexpr int kAtOnce = 64;
        AnyJob mixed[kAtOnce];
        GemmDesc rest[kAtOnce];
        for (int first = 0; first < count; first += kAtOnce) {
            const int last = count - first < kAtOnce ? count : first + kAtOnce;
            auto with_them = [](const GemmDesc& d) { return d.K % 64 != 0 || (gemv_any_supports(d.M, d.N, d.K) && !gemv_two_blocks(d.M, d.N, d.K)); };
            int64_t blocks = 0;
            for (int i = first; i < last; ++i)
                if (with_them(jobs[i])) blocks += (jobs[i].M + 15) / 16;
            int m = 0, r = 0;
            for (int i = first; i < last; ++i) {
                const GemmDesc& d = jobs[i];
                if (d.K % 64 != 0 || ((d.K > 2048 || blocks <= kMaxJobs) && with_them(d)))
                    mixed[m++] = AnyJob{d.x, d.W, nullptr, d.y, d.gamma, d.M, d.N, d.K, 0};
                else
                    rest[r++] = d;
            }
            hipError_t e = m ? launch_any_jobs(mixed, m, s) : hipSuccess;
            if (e == hipSuccess && r) e = launch_gemv_jobs(rest, r, s);
            if (e != hipSuccess) return e;
        }
        return hipSuccess;
    }
    if (count == 1 && gemv_rows_form(jobs[0].M, jobs[0].N, jobs[0].K)) {
        const GemmDesc& d = jobs[0];
        return launch_lean_rows(d.x, d.W, d.gamma, nullptr, 0, d.y, d.M, d.N, d.K, 0, false, s);
    }
    if (g_policy.longk) {
        hipError_t e = hipSuccess;
        if (launch_longk(jobs, count, s, &e)) return e;
    }
    // A user job with M > 16 becomes ceil(M / 16) kernel jobs (blocks of 16 activation rows).
    int64_t blocks_total = 0;
    for (int i = 0; i < count; ++i) blocks_total += (jobs[i].M + 15) / 16;
    const bool grouped = blocks_total > 1;

    // Two batches fill side by side: jobs for the stream form and jobs for the general kernel.
    // K <= 4096 always streams.  Longer K streams in several passes, each of which starts with
    // a round trip to memory for the activations; that pays once the call holds enough work to
    // give every workgroup a run of a few tiles (e.g. the linears of a whole block), otherwise
    // the general kernel takes those jobs.
    int64_t call_tiles = 0;                                   // tiles of the whole call
    for (int i = 0; i < count; ++i) call_tiles += ((jobs[i].M + 15) / 16) * ((jobs[i].N + 15) / 16);
    // (measured: one job of 512 tiles is better off in the general kernel, 11008 -> 8192 at M = 1
    // 9.7 against 10.9 us; two jobs of 256 tiles stream better, 11008 -> 4096 at M = 32 16.1 against 20.3 us)
    const bool long_k_streams = call_tiles >= int64_t(g_policy.stream_groups) * g_policy.long_k_min_run ||
                                (blocks_total >= 2 && call_tiles >= int64_t(g_policy.stream_groups) * 2);
    // bs: stream form; bs2: stream form with jobs of up to 32 rows (two blocks of 16 per wave);
    // bg: general kernel
    GemvBatch bs, bs2, bg;
    bs.count = 0;
    bs2.count = 0;
    bg.count = 0;
    auto flush = [&](GemvBatch& b) -> hipError_t {
        if (b.count == 0) return hipSuccess;
        hipError_t e = launch_batch(b, grouped, &b != &bg, &b == &bs2 ? 2 : 1, s);
        b.count = 0;
        return e;
    };
    const bool stream_on = (g_policy.stream & 3) == 3;
    for (int i = 0; i < count; ++i) {
        const GemmDesc& d = jobs[i];
        const int slices = int((d.K + kSliceK - 1) / kSliceK);
        // more than 16 rows and one pass over K: blocks of 32 rows, decoded once for both halves
        const bool two_blocks = stream_on && g_policy.two_blocks && gemv_two_blocks(d.M, d.N, d.K);
        const int64_t mstep = two_blocks ? 32 : 16;
        for (int64_t m0 = 0; m0 < d.M; m0 += mstep) {
            GemvJob j;
            j.x = d.x + m0 * d.K;
            j.W = d.W;
            j.y = d.y + m0 * d.N;
            j.gamma = d.gamma;
            j.Mrem = int(d.M - m0 < mstep ? d.M - m0 : mstep);
            j.N = int(d.N); j.K = int(d.K);
            j.tiles = int((d.N + 15) / 16);
            j.items = 0;
            j.slices = slices;
            j.mr = pow2_at_least(j.Mrem < 16 ? j.Mrem : 16);
            j.run = j.plus = 0;
            j.scales = nullptr; j.hpg = 0; j.reserved = 0;
            const bool streams = j.slices <= kStreamWaves ||
                                 (long_k_streams && j.slices <= kStreamWaves * kStreamMaxPasses);
            GemvBatch& b = two_blocks ? bs2 : (streams ? bs : bg);
            if (two_blocks && j.slices > kStreamWaves) {
                // several passes: the kept sums allow runs of kStreamMaxRun / 2 tiles, so a launch holds
                // at most that many tiles per workgroup
                int64_t held = j.tiles;
                for (int q = 0; q < b.count; ++q) held += b.job[q].tiles;
                if (b.count > 0 && held > int64_t(g_policy.stream_groups) * (kStreamMaxRun / 2)) {
                    hipError_t e = flush(b);
                    if (e != hipSuccess) return e;
                }
            }
            b.job[b.count++] = j;
            if (b.count == kMaxJobs) {
                hipError_t e = flush(b);
                if (e != hipSuccess) return e;
            }
        }
    }
    hipError_t e = flush(bs);
    if (e != hipSuccess) return e;
    e = flush(bs2);
    if (e != hipSuccess) return e;
    return flush(bg);
}

bool gemv_gs_supports(int64_t M, int64_t N, int64_t K, int64_t group)
{
    const int64_t slices = (K + kSliceK - 1) / kSliceK;
    // (the kernel addresses the scales with 32-bit byte offsets)
    if (((K - 1) / group + 1) * N * 2 >= (int64_t(1) << 31)) return false;
    if (N < 4 || N % 4 != 0 || lean_scale_kind(group) == 0) return false;
    // Other K: a row's last chunk of packed words starts anywhere in units of 16 weights and meets zeros up to its own, which are a unit of 64 or part
    // of one; units of 32 would lie across its halves.
    if (K % 64 != 0) return group % 64 == 0 && gemv_any_supports(M, N, K);
    return gemv_supports(M, N, K) && slices <= kStreamWaves * kStreamMaxPasses &&
           (slices <= kStreamWaves || (N + 15) / 16 <= int64_t(256) * kStreamMaxRun);
}

hipError_t launch_gemv_gs_jobs(const GemmGsDesc* jobs, int count, hipStream_t s)
{
    for (int i = 0; i < count; ++i)
        if (!gemv_gs_supports(jobs[i].M, jobs[i].N, jobs[i].K, jobs[i].group)) return hipErrorInvalidValue;
    if (count == 1) {
        const GemmGsDesc& d = jobs[0];
        const int kind = lean_scale_kind(d.group);
        GemvJob j{};
        j.scales = d.scales;
        j.hpg = units_per_group(d.K, d.group, kind);
        for (int64_t m0 = 0; m0 < d.M; m0 += kStreamRows) {
            const hipError_t e = launch_lean_rows(d.x + m0 * d.K, d.W, 1.f, d.scales, group_inverse(j), d.y + m0 * d.N, d.M - m0 < kStreamRows ? d.M - m0 : kStreamRows,
                                                  d.N, d.K, kind, d.K % 64 != 0 || d.N % 16 != 0, s);
            if (e != hipSuccess) return e;
        }
        return hipSuccess;
    }
    // Each kind of groups has instances of its own and shares launches, kMaxJobs blocks of 16 activation rows per launch; so do, kind
    // by kind, jobs of other K.
    for (int kind = 32; kind <= 256; kind *= 2) {
        GemvJob blocks[kMaxJobs];
        int held = 0;
        auto flush = [&]() -> hipError_t {
            const hipError_t e = held ? launch_blocks(blocks, held, kind, false, s) : hipSuccess;
            held = 0;
            return e;
        };
        constexpr int kAtOnce = 64;
        AnyJob other[kAtOnce];
        int others = 0;
        for (int i = 0; i < count; ++i) {
            const GemmGsDesc& d = jobs[i];
            if (lean_scale_kind(d.group) != kind) continue;
            if (d.K % 64 != 0) {
                other[others++] = AnyJob{d.x, d.W, d.scales, d.y, 1.f, d.M, d.N, d.K, d.group};
                if (others == kAtOnce) {
                    const hipError_t e = launch_any_jobs(other, others, s, kind);
                    if (e != hipSuccess) return e;
                    others = 0;
                }
                continue;
            }
            const int slices = int((d.K + kSliceK - 1) / kSliceK);
            const int hpg = units_per_group(d.K, d.group, kind);
            for (int64_t m0 = 0; m0 < d.M; m0 += 16) {
                GemvJob j;
                j.x = d.x + m0 * d.K;
                j.W = d.W;
                j.y = d.y + m0 * d.N;
                j.gamma = 1.f;
                j.Mrem = int(d.M - m0 < 16 ? d.M - m0 : 16);
                j.N = int(d.N); j.K = int(d.K);
                j.tiles = int((d.N + 15) / 16);
                j.items = 0;
                j.slices = slices;
                j.mr = pow2_at_least(j.Mrem);
                j.run = j.plus = 0;
                j.scales = d.scales; j.hpg = hpg; j.reserved = 0;
                blocks[held++] = j;
                if (held == kMaxJobs) {
                    const hipError_t e = flush();
                    if (e != hipSuccess) return e;
                }
            }
        }
        hipError_t e = flush();
        if (e == hipSuccess && others) e = launch_any_jobs(other, others, s, kind);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

hipError_t launch_gemv_gs(const __half* x, const uint32_t* Wp, const __half* scales, int64_t group,
                          __half* y, int64_t M, int64_t N, int64_t K, hipStream_t s)
{
    const GemmGsDesc d{x, Wp, scales, y, M, N, K, group};
    return launch_gemv_gs_jobs(&d, 1, s);
}

hipError_t launch_gemv(const __half* x, const uint32_t* Wp, float gamma, __half* y,
                       int64_t M, int64_t N, int64_t K, hipStream_t s)
{
    GemmDesc d{x, Wp, y, gamma, M, N, K};
    return launch_gemv_jobs(&d, 1, s);
}

}  // namespace tl
