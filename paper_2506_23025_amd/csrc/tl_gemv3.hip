// Weight-streaming small-M kernel for the 1.6-bit formats (5 trits per byte: plain base 3, byte = sum_i (w_i + 1) 3^i, the block code
// of Sec. 3.2 without its fixed-point scaling, or that code itself).
//
// Same organisation as the 2-bit kernel (tl_gemv.hip): a workgroup owns 16-row tiles, a wave owns a part of K and keeps its activations
// in registers as MFMA B operands, packed rows stream once, split-K partial tiles are summed through LDS in a fixed order.
// What differs is the geometry and the decode:
//
//  * A wave's part is a half slice of 64 packed bytes = 320 weights per row; a lane's 16 bytes of a tile (row lane % 16, 16-byte chunk
//    lane / 16) hold 80 weights and lie in its registers as the matrix instruction wants them: no turn through LDS.  Half lines per
//    request cost the memory a little (a bare load loop 20.0 instead of 16.7 us for 100 MB); the decode takes longer than that.
//  * Up to 15 waves in a workgroup, one workgroup per CU (more with shorter K, see gemv3_per_cu): four waves per SIMD cover the chain byte -> address -> look-up -> operand
//    (two LDS round trips and two waves per SIMD, in slices of 128 bytes, took 28 us for the decode sweep where this takes 22.4).
//  * Decode is a table look-up: a 256-entry table of 8-byte entries in LDS maps a byte to its five digits c = w + 1 as fp16 (subnormal)
//    pairs: word 0 = c0 << 6 | c2 << 14 | c3 << 22, word 1 = c1 << 6 | c4 << 22 (every digit is used at bit 6 of its half: the matrix
//    instruction aligns products by exponent field, and subnormals with only their lowest bits set lose low-order product bits).  The
//    two words of two neighbouring bytes, with c2 masked out of the first word of each, are one A operand of
//    v_mfma_f32_16x16x32_f16 as they stand: (c0, c3), (c1, c4) per byte, against the activation pairs (x[5b], x[5b+3]) and
//    (x[5b+1], x[5b+4]); a byte permute brings the c2 of two bytes together, at bit 6, for an operand of eight bytes.  Per 5 weights:
//    1 address operation (a shift with a byte select), 1 LDS read, 1 AND, 1/2 permute, and 10 products per 320 x 16 weights.
//  * What bounds it: issue and look-ups.  Decode sweep 22.4 us; without the look-ups 19.5, without them and the products 16.3, without
//    the weight loads 21.9, with look-ups free of bank conflicts 21.6.  Leaving c2 in the first words and cancelling it by a product of
//    its own saves the ANDs, adds rounding and gives 22.1: not done.
//  * The paper expects the 1.6-bit form to cost more arithmetic per weight than the 2-bit form (Sec. 3.3 results, "Limitations").
//  * K is any number from 8 on.  Rows of packed bytes start at multiples of 16 bytes whatever K is; rows of x at any even address where K is no
//    multiple of 8, and then their pieces come through registers (ANY_K), which costs 0.3 us and 5 % (10 % with several passes).  Such calls ran
//    in the tiled kernel's form for odd K: up to 16 rows of 512 .. 16384 x 64 .. 14336 weights this one is 1.6 to 2.1 times as fast on average
//    (1 x 2577 x 12738 29.0 -> 7.2 us, 7 x 4864 x 3806 12.1 -> 5.7), slower by up to 3 % (0.15 us) in 13 of 1000 calls, K below 290 at 9 rows and more.
//  * Two forms.  gemv3_stream_kernel (K in one pass of at most 15 half slices, K <= 4800): a wave keeps its half slice, a workgroup walks
//    a run of tiles in items with the next item's weights in flight; gemv3_grouped_kernel is the same body fed from one record per
//    workgroup, so that one launch carries several GEMMs.  gemv3_kernel (longer K): waves loop over half slices, one item of up to 4
//    tiles per workgroup.
#include "tl_internal.hpp"
#include "tl_deal.hpp"

#include <atomic>
#include <type_traits>

namespace tl {

namespace {

constexpr int kT3Max = 4;            // tiles per workgroup
constexpr int kHalf3 = 320;          // weights per half slice (64 packed bytes), a wave's share of a pass
constexpr int kXRowHalf = 656;       // bytes per staged activation row (640 + 16: 16 rows in different banks)
constexpr int kWaveLds = 16 * kXRowHalf;
constexpr int kLutBytes = 2048;      // 256 entries of 8 bytes
constexpr int kWaves3 = 15;
constexpr int kLds3 = kWaves3 * kWaveLds + kLutBytes;           // 159488 bytes

struct Gemv3Params {
    const __half* x;
    const uint8_t* W;
    __half* y;
    float gamma;
    int M, N, K;
    int stride;      // bytes per packed row (multiple of 16)
    int tiles;       // ceil(N / 16)
    int groups;      // gridDim.x
    int fx;          // bytes hold the fixed-point code of Sec. 3.2 instead of plain base 3
};

constexpr int vmcnt_imm3(int n)
{
    return (n & 0xF) | ((n >> 4) << 14) | (0x7 << 4) | (0xF << 8);
}

__device__ __forceinline__ f16x8 as_h8(u32x4 v) { return __builtin_bit_cast(f16x8, v); }

// Barrier that waits for this wave's LDS traffic only; the weight loads and activation
// transfers already requested stay in flight across it (__syncthreads would drain them).
__device__ __forceinline__ void lds_barrier3()
{
    __builtin_amdgcn_s_waitcnt(0xF | (0x3 << 14) | (0x7 << 4));      // lgkmcnt(0)
    __builtin_amdgcn_s_barrier();
}

// 16 bytes per lane to LDS at `lds` + 16 lane.  Written out by hand (see tl_tile.hpp): the compiler would wait for a transfer it knows of
// before later LDS accesses.
__device__ __forceinline__ void dma16(uint32_t voff, const void* sbase, uint32_t lds)
{
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1" : : "v"(voff), "s"(sbase), "s"(__builtin_amdgcn_readfirstlane(lds)) : "memory");
}

// 8 * (byte B of w): the offset of that byte's table entry, in one instruction (the shift
// reads its operand through a byte select).
template <int B>
__device__ __forceinline__ uint32_t byte_times_8(uint32_t w)
{
    uint32_t r;
    const uint32_t three = 3u;
    if constexpr (B == 0) asm("v_lshlrev_b32_sdwa %0, %1, %2 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:DWORD src1_sel:BYTE_0" : "=v"(r) : "v"(three), "v"(w));
    if constexpr (B == 1) asm("v_lshlrev_b32_sdwa %0, %1, %2 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:DWORD src1_sel:BYTE_1" : "=v"(r) : "v"(three), "v"(w));
    if constexpr (B == 2) asm("v_lshlrev_b32_sdwa %0, %1, %2 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:DWORD src1_sel:BYTE_2" : "=v"(r) : "v"(three), "v"(w));
    if constexpr (B == 3) asm("v_lshlrev_b32_sdwa %0, %1, %2 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:DWORD src1_sel:BYTE_3" : "=v"(r) : "v"(three), "v"(w));
    return r;
}

// byte -> digits table.  Plain form: base-3 digits, least significant first (bytes 243..255
// never occur; they decode like byte - 243).  Fixed-point form (Sec. 3.2): the block value is
// floor(243 b / 256), the inverse of b = ceil(256 V / 243), and its base-3 digits go most
// significant first; all 256 bytes decode, and to the digits App. F, Alg. 1 gives.
__device__ __forceinline__ void fill_table(u32x2* lut, bool fx)
{
    for (unsigned b = threadIdx.x; b < 256; b += blockDim.x) {
        unsigned c[5];
        if (fx) {
            unsigned v = (b * 243u) >> 8;
#pragma unroll
            for (int i = 4; i >= 0; --i) { c[i] = v % 3u; v /= 3u; }
        } else {
            unsigned v = b >= 243 ? b - 243 : b;
#pragma unroll
            for (int i = 0; i < 5; ++i) { c[i] = v % 3u; v /= 3u; }
        }
        lut[b] = u32x2{(c[0] << 6) | (c[2] << 14) | (c[3] << 22), (c[1] << 6) | (c[4] << 22)};
    }
}

// The activations of a half slice (a lane's 16 bytes, 80 weights) as MFMA B operands: with k = 20 d the first weight of dword d,
// b[2d] = (k, k+3), (k+1, k+4), (k+5, k+8), (k+6, k+9) for its bytes 0 and 1, b[2d + 1] the same ten further on for bytes 2
// and 3, b[8 + e] = (k+2, k+7), (k+12, k+17) of dwords 2e and 2e + 1.
__device__ __forceinline__ void build_operands_half(const unsigned char* row, u32x4 (&b)[10])
{
#pragma unroll
    for (int e = 0; e < 2; ++e) {                          // 40 weights, two dwords, at a time: registers
        __builtin_amdgcn_sched_barrier(0);
        u32x4 xv[5];
#pragma unroll
        for (int i = 0; i < 5; ++i) xv[i] = *reinterpret_cast<const u32x4*>(row + 80 * e + 16 * i);
        auto pair = [&](int lo, int hi) {
            return __builtin_amdgcn_perm(xv[hi >> 3][(hi >> 1) & 3], xv[lo >> 3][(lo >> 1) & 3],
                                         (((hi & 1) ? 0x0706u : 0x0504u) << 16) | ((lo & 1) ? 0x0302u : 0x0100u));
        };
#pragma unroll
        for (int k = 0; k < 40; k += 20) {
            const int d = 2 * e + k / 20;
            b[2 * d] = u32x4{pair(k, k + 3), pair(k + 1, k + 4), pair(k + 5, k + 8), pair(k + 6, k + 9)};
            b[2 * d + 1] = u32x4{pair(k + 10, k + 13), pair(k + 11, k + 14), pair(k + 15, k + 18), pair(k + 16, k + 19)};
        }
        b[8 + e] = u32x4{pair(2, 7), pair(12, 17), pair(22, 27), pair(32, 37)};
    }
    __builtin_amdgcn_sched_barrier(0);
}

// Activation rows of half slice `hs` to LDS at `area`: rows of 40 pieces of 16 bytes, 41 apart (16 rows in different banks), by
// LDS-DMA; pieces past K are zeros.  Rows from `rows` on stay unwritten (an MFMA column depends on its own column of B alone).
__device__ __forceinline__ void stage_half(const unsigned char* x, int hs, int rows, int K, unsigned char* area, int lane)
{
    const int total = rows * 41;
    const unsigned char* const src = x + size_t(hs) * (kHalf3 * 2);
    const uint32_t base = uint32_t(uintptr_t((const __attribute__((address_space(3))) unsigned char*)area));
#pragma unroll 1
    for (int i = 0; i < total; i += 64) {
        const uint32_t piece = uint32_t(i + lane);
        const uint32_t row = (piece * 1599u) >> 16;        // piece / 41, pieces up to 767
        const uint32_t col = piece - row * 41u;
        if (int(piece) < total && col < 40u) {
            if (hs * kHalf3 + int(col) * 8 < K)
                dma16(row * (uint32_t(K) * 2u) + col * 16u, src, base + uint32_t(i) * 16u);
            else
                *reinterpret_cast<u32x4*>(area + piece * 16u) = u32x4{0u, 0u, 0u, 0u};
        }
    }
}

// The same for a K that is no multiple of 8, whose rows start at any even address: the pieces come through registers, round i of a wave being
// the pieces 64 i .. 64 i + 63 of rows of 40.  A piece that reaches past K is fetched from the row's last 16 bytes and shifted down, one past K
// altogether is zero; pieces past the last row repeat that row.  Rounds I0 .. I0 + R - 1.
typedef u32x4 __attribute__((aligned(2))) u32x4_any;
template <int I0, int R>
__device__ __forceinline__ void fetch_pieces(const unsigned char* x, int hs, int rows, int K, int lane, u32x4 (&v)[R])
{
    asm volatile("" : "+v"(lane));                         // places worked out here, not kept in registers over the passes
#pragma unroll
    for (int i = 0; i < R; ++i) {
        const uint32_t piece = uint32_t((I0 + i) * 64 + lane);
        uint32_t row = (piece * 1639u) >> 16;              // piece / 40, pieces up to 639
        uint32_t k = uint32_t(hs) * kHalf3 + (piece - row * 40u) * 8u;
        if (row >= uint32_t(rows)) row = uint32_t(rows) - 1u;
        if (k > uint32_t(K) - 8u) k = uint32_t(K) - 8u;
        v[i] = *(const __attribute__((address_space(1))) u32x4_any*)((const __attribute__((address_space(1))) unsigned char*)x + (row * uint32_t(K) + k) * 2u);
    }
}
template <int I0, int R>
__device__ __forceinline__ void put_pieces(int hs, int K, unsigned char* area, int lane, const u32x4 (&v)[R])
{
    const bool tail = (hs + 1) * kHalf3 > K;
    asm volatile("" : "+v"(lane));
#pragma unroll
    for (int i = 0; i < R; ++i) {
        const uint32_t piece = uint32_t((I0 + i) * 64 + lane);
        const uint32_t row = (piece * 1639u) >> 16, col = piece - row * 40u;
        u32x4 w = v[i];
        if (tail) {
            const int past = hs * kHalf3 + int(col) * 8 + 8 - K;              // elements past K, 16 bits each
            const int n = 16 * (past > 0 ? past : 0);
            const uint64_t lo = uint64_t(w[0]) | (uint64_t(w[1]) << 32), hi = uint64_t(w[2]) | (uint64_t(w[3]) << 32);
            uint64_t a = lo, b = hi;
            if (n >= 128) { a = 0; b = 0; }
            else if (n >= 64) { a = hi >> (n - 64); b = 0; }
            else if (n > 0) { a = (lo >> n) | (hi << (64 - n)); b = hi >> n; }
            w = u32x4{uint32_t(a), uint32_t(a >> 32), uint32_t(b), uint32_t(b >> 32)};
        }
        *reinterpret_cast<u32x4*>(area + row * kXRowHalf + col * 16u) = w;
    }
}
// The activations of half slice `hs` so, with `between` (the weights' requests, the table) between asking for them and their way to LDS
template <class Between>
__device__ __forceinline__ void stage_pieces(const unsigned char* x, int hs, int rows, int K, unsigned char* area, int lane, Between&& between)
{
    auto rounds = [&](auto count) {
        u32x4 v[decltype(count)::value];
        fetch_pieces<0>(x, hs, rows, K, lane, v);
        __builtin_amdgcn_sched_barrier(0);
        between();
        put_pieces<0>(hs, K, area, lane, v);
    };
    if (rows <= 1) rounds(std::integral_constant<int, 1>{});
    else if (rows <= 4) rounds(std::integral_constant<int, 3>{});
    else if (rows <= 8) rounds(std::integral_constant<int, 5>{});
    else rounds(std::integral_constant<int, 10>{});
}

// the staged rows -> operands, and c0 - 2^-18 sum_k x over the half slice in accumulator layout (constant 16-row operand)
__device__ __forceinline__ f32x4 operands_and_seed(const unsigned char* area, int rows, int mi, int mg, u32x4 (&bop)[10])
{
    int MR = 1;
    while (MR < rows) MR *= 2;
    build_operands_half(area + (mi & (MR - 1)) * kXRowHalf + mg * 160, bop);
    const u32x4 c = {0x80408040u, 0x80408040u, 0x80408040u, 0x80408040u};        // -2^-18
    f32x4 nsx = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int q = 0; q < 10; ++q)
        nsx = __builtin_amdgcn_mfma_f32_16x16x32_f16(as_h8(c), as_h8(bop[q]), nsx, 0, 0, 0);
    return nsx;
}

// table addresses of a lane's 16 bytes
__device__ __forceinline__ void addresses(u32x4 w, uint32_t (&at)[4][4])
{
#pragma unroll
    for (int d = 0; d < 4; ++d) {
        at[d][0] = byte_times_8<0>(w[d]);
        at[d][1] = byte_times_8<1>(w[d]);
        at[d][2] = byte_times_8<2>(w[d]);
        at[d][3] = byte_times_8<3>(w[d]);
    }
}

// c0 + 2^-18 sum_k x_k (w_k + 1) of a tile's half slice.  All look-ups are issued before the first is used, so that their latency
// runs under the arithmetic of the ones before.  The table starts the LDS: a byte offset into it is an LDS address.
__device__ __forceinline__ f32x4 tile_sum_half(const uint32_t (&at)[4][4], const u32x4 (&bop)[10], f32x4 c0)
{
    auto lut_at = [](uint32_t off) { return *(const __attribute__((address_space(3))) u32x2*)(uintptr_t(off)); };
    u32x4 e[4][2];                                         // bytes 0 and 1 (2 and 3) of dword d: their table words side by side
    f32x4 acc[2] = {c0, f32x4{0.f, 0.f, 0.f, 0.f}};
    u32x4 mid[2];
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const u32x2 lo = lut_at(at[q][2 * j]), hi = lut_at(at[q][2 * j + 1]);
            e[q][j] = u32x4{lo[0], lo[1], hi[0], hi[1]};
        }
#pragma unroll
    for (int d = 0; d < 4; ++d) {
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            // The second byte of a table word is c2 alone, six bits up; without it the words are an operand as they stand.  The empty
            // statement makes them new values once c2 is out, so that they are masked where they stand (the compiler would keep the words
            // for c2 and copy the others).  The mask itself stays visible to it: gfx950 asks for two wait states between a vector
            // instruction and the matrix instruction that reads its result, and the compiler sees to them for its own only.
            const uint32_t m = __builtin_amdgcn_perm(e[d][j][2], e[d][j][0], 0x0c050c01u);
            uint32_t w0 = e[d][j][0], w1 = e[d][j][2];
            asm("" : "+v"(w0), "+v"(w1) : "v"(m));
            w0 &= 0x00c000c0u;
            w1 &= 0x00c000c0u;
            const u32x4 a = {w0, e[d][j][1], w1, e[d][j][3]};
            acc[j] = __builtin_amdgcn_mfma_f32_16x16x32_f16(as_h8(a), as_h8(bop[2 * d + j]), acc[j], 0, 0, 0);
            mid[d >> 1][2 * (d & 1) + j] = m;
        }
        if (d & 1) acc[d >> 1] = __builtin_amdgcn_mfma_f32_16x16x32_f16(as_h8(mid[d >> 1]), as_h8(bop[8 + (d >> 1)]), acc[d >> 1], 0, 0, 0);
    }
    return acc[0] + acc[1];
}

// Sum of the first `parts` waves' values at `from` (one f32x4, kWaveLds apart), in a fixed order
__device__ __forceinline__ f32x4 sum_parts(const unsigned char* from, int parts)
{
    f32x4 s = f32x4{0.f, 0.f, 0.f, 0.f};
    auto some = [&](auto count) {
        constexpr int C = decltype(count)::value;
        f32x4 v[C];
#pragma unroll
        for (int q = 0; q < C; ++q) v[q] = *reinterpret_cast<const f32x4*>(from + q * kWaveLds);
#pragma unroll
        for (int step = 1; step < C; step *= 2)
#pragma unroll
            for (int q = 0; q < C; q += 2 * step) v[q] += v[q + step];
        s += v[0];
        from += C * kWaveLds;
    };
    if (parts & 8) some(std::integral_constant<int, 8>{});
    if (parts & 4) some(std::integral_constant<int, 4>{});
    if (parts & 2) some(std::integral_constant<int, 2>{});
    if (parts & 1) some(std::integral_constant<int, 1>{});
    return s;
}

// four consecutive columns of a row of y, `left` of which exist; `aligned`: as one 8-byte store
typedef __attribute__((address_space(1))) __half* gh_ptr;
__device__ __forceinline__ void store_quad(gh_ptr dst, f32x4 s, float gamma, int left, bool aligned)
{
    if (left >= 4 && aligned) {
        const f16x2 lo = {(_Float16)(gamma * s[0]), (_Float16)(gamma * s[1])};
        const f16x2 hi = {(_Float16)(gamma * s[2]), (_Float16)(gamma * s[3])};
        *(__attribute__((address_space(1))) u32x2*)dst = u32x2{__builtin_bit_cast(uint32_t, lo), __builtin_bit_cast(uint32_t, hi)};
    } else {
#pragma unroll
        for (int r = 0; r < 4; ++r)
            if (r < left) *(__attribute__((address_space(1))) _Float16*)(dst + r) = (_Float16)(gamma * s[r]);
    }
}

// ------------------------------------------------------------------------------------------
// Stream form, for K of at most kWaves3 half slices: wave w owns half slice w (64 packed bytes, 320 weights) for the whole
// kernel, so activations are staged and turned into operands once; a workgroup walks a run of
// consecutive tiles, T at a time ("item"), with the next item's weights requested as soon as
// a tile's registers are free, two alternating sets of partial sums and one LDS-only barrier
// per item -- the organisation of the 2-bit stream kernel (tl_gemv.hip) with this file's
// decode.  Params::groups workgroups; workgroup g takes tiles [g per + min(g, extra), ...).
// What a workgroup of the stream form works on: one block of at most 16 activation rows of one
// GEMM and a run of consecutive tiles of its matrix.  x and y point at the block's first row.
struct Run3 {
    const unsigned char* W;   // the matrix (first row)
    const unsigned char* x;
    __half* y;
    float gamma;
    int K, N;
    int stride;               // bytes per packed row
    int Mrem;                 // activation rows, 1..16
    int tile0, tile_end;      // the run
    int fx;                   // which byte code the table is filled for
    int pad;
};
static_assert(sizeof(Run3) == 64, "one record per 64-byte line");

// Records (workgroups) of a grouped launch: 16 KB of kernel arguments, or 32 KB where two workgroups fit on a CU (K of up to 7 half
// slices) and the launch holds 2048 tiles or more, which is 4 and more for each of the 512.  Kernel alone / call by call, 512 against 256,
// means over calls of K = 512 .. 2240: 0.86 .. 0.95 / 1.03 .. 1.07 times as long with 1024 to 2047 tiles (the larger arguments cost the host
// 0.5 us), 0.82 .. 0.97 / 1.0 with 2048 to 2559, 0.75 .. 0.82 / 0.78 .. 0.84 with 4096 to 6143; ten layers of K = 1024 13.8 -> 10.3 us.
constexpr int kRec3Few = 256, kRec3Many = 512;

template <int R>
struct Rec3Batch {
    Run3 rec[R];
};

template <int T, bool ANY_K>
__device__ __forceinline__ void gemv3_stream_body(const Run3& p)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char lds_raw[];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int NW = blockDim.x >> 6;
    u32x2* const lut = reinterpret_cast<u32x2*>(lds_raw);
    unsigned char* const my_lds = lds_raw + kLutBytes + wave * kWaveLds;

    const int rows = p.Mrem, K = p.K, N = p.N;
    const uint32_t stride = uint32_t(p.stride);
    const int chunks = p.stride >> 4;
    const int tile0 = p.tile0, ntiles = p.tile_end - p.tile0;
    const int mi = lane & 15, mg = lane >> 4;              // row of the tile / activation column, chunk of the slice
    const bool active = wave * 4 < chunks;

    const bool pieces = ANY_K && (K & 7) != 0;             // rows of x start anywhere
    if (active && !pieces) stage_half(p.x, wave, rows, K, my_lds, lane);
    // ---- weights: a lane's 16 bytes of a tile lie where the matrix instruction wants them (row mi, k group mg).  The run is a raw buffer
    // of the rows that exist: rows past N read zeros, and a request costs the vector ALU nothing.  Not marked non-temporal, here and in
    // gemv3_kernel: two requests share a 128-byte line, and so marked calls of K = 1600 .. 14336 took 2 to 5 % longer (up to 14 %), shorter
    // K and grouped calls 0 to 1 %
    uint32_t voff;
    {
        const int chunk = wave * 4 + mg;
        voff = uint32_t(mi) * stride + uint32_t(chunk < chunks ? chunk : 0) * 16u;      // past the row: meets zero activations
    }
    const uint32_t tile_bytes = 16u * stride;
    const int run_rows = N - tile0 * 16 < ntiles * 16 ? N - tile0 * 16 : ntiles * 16;
    const __amdgpu_buffer_rsrc_t wres = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<unsigned char*>(p.W) + size_t(tile0) * tile_bytes, 0, uint32_t(run_rows) * stride, 0x00020000);
    u32x4 wreg[T];
    auto issue_w = [&](int idx, int t) {                   // idx: tile of the run; past the run: its last tile again
        const int c = idx < ntiles ? idx : ntiles - 1;
        wreg[t] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(wres, voff, uint32_t(c) * tile_bytes, 0));
    };
    auto between = [&]() {
        if (active) {
#pragma unroll
            for (int t = 0; t < T; ++t) {
                issue_w(t, t);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        fill_table(lut, p.fx != 0);
    };
    if (ANY_K && active && pieces) stage_pieces(p.x, wave, rows, K, my_lds, lane, between);
    else between();
    u32x4 bop[10];
    f32x4 nsx = f32x4{0.f, 0.f, 0.f, 0.f};
    if (active) {
        __builtin_amdgcn_s_waitcnt(vmcnt_imm3(T));         // the activations are in; the weights stay in flight
        nsx = operands_and_seed(my_lds, rows, mi, mg, bop);
    }
    lds_barrier3();                                        // the table is complete

    const float gamma = p.gamma * 262144.f;                // times the 2^18 left in the partial sums
    gh_ptr const ylane = (gh_ptr)(p.y + size_t(mi) * N + size_t(tile0) * 16 + 4 * mg);
    const int nleft = N - tile0 * 16 - 4 * mg;             // columns from the lane's first one on
    const bool aligned = (N & 3) == 0;
    const int parts = (chunks + 3) >> 2;                   // waves with a slice of K
    int turn = wave;                                       // waves take turns at adding up an item: tile `turn` of it
    auto finish = [&](int first, int parity) {
        lds_barrier3();
        if (turn < T && first + turn < ntiles) {
            const f32x4 s = sum_parts(lds_raw + kLutBytes + parity * (T * 1024) + turn * 1024 + lane * 16, parts);
            const int n = (first + turn) * 16;
            if (mi < rows) store_quad(ylane + n, s, gamma, nleft - n, aligned);
        }
        turn -= T;
        if (turn < 0) turn += NW;
    };
    const int n_items = (ntiles + T - 1) / T;
    if (!active) {
        for (int i = 0; i < n_items; ++i) finish(i * T, i & 1);
        return;
    }
    auto item = [&](auto refill_tag, int first, int parity) {
        constexpr bool REFILL = decltype(refill_tag)::value;
        unsigned char* const red = my_lds + parity * (T * 1024);
#pragma unroll
        for (int t = 0; t < T; ++t) {
            if (!REFILL && first + t >= ntiles) break;
            uint32_t at[4][4];
            addresses(wreg[t], at);
            if constexpr (REFILL) {
                __builtin_amdgcn_sched_barrier(0);
                issue_w(first + T + t, t);
                __builtin_amdgcn_sched_barrier(0);
            }
            reinterpret_cast<f32x4*>(red + t * 1024)[lane] = tile_sum_half(at, bop, nsx);
        }
        finish(first, parity);
    };
    int i = 0;
    for (; i + 1 < n_items; ++i) item(std::true_type{}, i * T, i & 1);
    item(std::false_type{}, i * T, i & 1);
}

// ------------------------------------------------------------------------------------------
// Longer K: wave w owns the half slices w, w + NW, ...; a workgroup's T tiles are its whole work.  Their sums stay in registers over all
// passes, and a pass's activations and weights are requested while the pass before it is worked on: the activations as soon as the operands
// are built, each tile's weights as soon as their registers are free.  Against the form with slices of 128 bytes, seven waves and no
// overlap of the passes: 11008 -> 4096 at M = 1 / 16 6.8 / 11.4 -> 5.8 / 9.2 us, 14336 -> 14336 17.6 / 23.5 -> 14.5 / 18.3.
template <int T, bool ANY_K>
__global__ void __launch_bounds__(1024)
gemv3_kernel(Gemv3Params p)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char lds_raw[];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int NW = blockDim.x >> 6;
    unsigned char* const my_lds = lds_raw + kLutBytes + wave * kWaveLds;
    const int m0 = blockIdx.y * 16;
    const int rows = (p.M - m0 < 16) ? (p.M - m0) : 16;
    const int K = p.K, N = p.N, tiles = p.tiles, groups = p.groups, grp = blockIdx.x;
    const uint32_t stride = uint32_t(p.stride);
    const int chunks = p.stride >> 4, slices = (chunks + 3) >> 2;
    const int mi = lane & 15, mg = lane >> 4;
    const unsigned char* const xb = reinterpret_cast<const unsigned char*>(p.x + size_t(m0) * K);

    u32x4 wreg[T];
    auto issue_w = [&](int slice, int t) {                 // past the last tile: that tile again
        int tile = grp + t * groups;
        if (tile >= tiles) tile = tiles - 1;
        const int left = N - tile * 16;
        const int chunk = slice * 4 + mg;
        const __amdgpu_buffer_rsrc_t res = __builtin_amdgcn_make_buffer_rsrc(
            const_cast<unsigned char*>(p.W) + size_t(tile) * (16u * size_t(stride)), 0, uint32_t(left < 16 ? left : 16) * stride, 0x00020000);
        wreg[t] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(
            res, uint32_t(mi) * stride + uint32_t(chunk < chunks ? chunk : 0) * 16u, 0, 0));
    };
    int slice = wave;                                      // slices >= NW: every wave has one
    auto between = [&]() {
#pragma unroll
        for (int t = 0; t < T; ++t) {
            issue_w(slice, t);
            __builtin_amdgcn_sched_barrier(0);
        }
        fill_table(reinterpret_cast<u32x2*>(lds_raw), p.fx != 0);
    };
    if constexpr (ANY_K) {
        stage_pieces(xb, slice, rows, K, my_lds, lane, between);
    } else {
        stage_half(xb, slice, rows, K, my_lds, lane);
        between();
    }
    f32x4 part[T];
#pragma unroll
    for (int t = 0; t < T; ++t) part[t] = f32x4{0.f, 0.f, 0.f, 0.f};
    bool first = true;
    auto pass = [&](auto more_tag) {
        constexpr bool MORE = decltype(more_tag)::value;
        if constexpr (!ANY_K) asm volatile("s_waitcnt vmcnt(%0)" : : "n"(T) : "memory");       // the activations, asked for before the weights
        u32x4 bop[10];
        const f32x4 nsx = operands_and_seed(my_lds, rows, mi, mg, bop);
        if (first) lds_barrier3();                         // the table is complete
        else asm volatile("s_waitcnt lgkmcnt(0)" : : : "memory");
        first = false;
        // ANY_K: the next pass's first rounds of pieces (4, 3 or no rows), as many as there are registers for
        constexpr int AHEAD = T <= 2 ? 3 : (T == 3 ? 2 : 0);
        u32x4 ahead[AHEAD > 0 ? AHEAD : 1];
        if constexpr (MORE && ANY_K) {
            if constexpr (AHEAD > 0) fetch_pieces<0>(xb, slice + NW, rows, K, lane, ahead);
            __builtin_amdgcn_sched_barrier(0);
        } else if constexpr (MORE) {
            // the weights as well, before anything is asked for behind the compiler's back
            __builtin_amdgcn_s_waitcnt(vmcnt_imm3(0));
            stage_half(xb, slice + NW, rows, K, my_lds, lane);
            __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
        for (int t = 0; t < T; ++t) {
            uint32_t at[4][4];
            addresses(wreg[t], at);
            __builtin_amdgcn_sched_barrier(0);
            if constexpr (MORE) issue_w(slice + NW, t);
            __builtin_amdgcn_sched_barrier(0);
            part[t] += tile_sum_half(at, bop, nsx);
            __builtin_amdgcn_sched_barrier(0);
        }
        if constexpr (MORE && ANY_K) {
            if constexpr (AHEAD > 0) put_pieces<0>(slice + NW, K, my_lds, lane, ahead);
            auto others = [&](auto count) {
                u32x4 v[decltype(count)::value - AHEAD];
                fetch_pieces<AHEAD>(xb, slice + NW, rows, K, lane, v);
                put_pieces<AHEAD>(slice + NW, K, my_lds, lane, v);
            };
            if (rows > 8) others(std::integral_constant<int, 10>{});
            else if (rows * 40 > AHEAD * 64) others(std::integral_constant<int, 5>{});
        }
        slice += NW;
    };
    while (slice + NW < slices) pass(std::true_type{});
    pass(std::false_type{});
    // ---- sums of the waves
    unsigned char* const red = my_lds;
#pragma unroll
    for (int t = 0; t < T; ++t) reinterpret_cast<f32x4*>(red + t * 1024)[lane] = part[t];
    lds_barrier3();
    if (wave < T) {
        const int tile = grp + wave * groups;
        if (tile >= tiles) return;
        const f32x4 s = sum_parts(lds_raw + kLutBytes + wave * 1024 + lane * 16, NW);
        const int n = tile * 16 + 4 * mg;
        if (mi < rows) store_quad((gh_ptr)(p.y + size_t(m0 + mi) * N + n), s, p.gamma * 262144.f, N - n, (N & 3) == 0);
    }
}

// One GEMM: blockIdx.y is the block of 16 activation rows, the tiles are split evenly over gridDim.x.
template <int T, bool ANY_K>
__global__ void __launch_bounds__(1024)
gemv3_stream_kernel(Gemv3Params p)
{
    const int m0 = blockIdx.y * 16;
    const int per = p.tiles / p.groups, extra = p.tiles % p.groups;
    const int g = blockIdx.x;
    Run3 r;
    r.W = p.W;
    r.x = reinterpret_cast<const unsigned char*>(p.x + size_t(m0) * p.K);
    r.y = p.y + size_t(m0) * p.N;
    r.gamma = p.gamma;
    r.K = p.K; r.N = p.N; r.stride = p.stride;
    r.Mrem = (p.M - m0 < 16) ? (p.M - m0) : 16;
    r.tile0 = g * per + (g < extra ? g : extra);
    r.tile_end = r.tile0 + per + (g < extra ? 1 : 0);
    r.fx = p.fx;
    gemv3_stream_body<T, ANY_K>(r);
}

// Several GEMMs: the host has dealt out the workgroups and written one record for each.
template <int T, bool ANY_K, int R>
__global__ void __launch_bounds__(1024)
gemv3_grouped_kernel(Rec3Batch<R> b)
{
    gemv3_stream_body<T, ANY_K>(b.rec[blockIdx.x]);
}

using Kernel3Fn = void (*)(Gemv3Params);

// any_k: for a K that is no multiple of 8 (in a grouped launch, that of some job)
template <bool ANY_K>
Kernel3Fn pick3(int T)
{
    switch (T) {
        case 1: return gemv3_kernel<1, ANY_K>;
        case 2: return gemv3_kernel<2, ANY_K>;
        case 3: return gemv3_kernel<3, ANY_K>;
        default: return gemv3_kernel<4, ANY_K>;
    }
}
Kernel3Fn pick3(int T, bool any_k) { return any_k ? pick3<true>(T) : pick3<false>(T); }

template <bool ANY_K>
Kernel3Fn pick3_stream(int T)
{
    switch (T) {
        case 1: return gemv3_stream_kernel<1, ANY_K>;
        case 2: return gemv3_stream_kernel<2, ANY_K>;
        default: return gemv3_stream_kernel<3, ANY_K>;
    }
}
Kernel3Fn pick3_stream(int T, bool any_k) { return any_k ? pick3_stream<true>(T) : pick3_stream<false>(T); }

template <int R>
using Grouped3Fn = void (*)(Rec3Batch<R>);

template <int R>
Grouped3Fn<R> pick3_grouped(int T, bool any_k)
{
    switch (T) {
        case 1: return any_k ? gemv3_grouped_kernel<1, true, R> : gemv3_grouped_kernel<1, false, R>;
        case 2: return any_k ? gemv3_grouped_kernel<2, true, R> : gemv3_grouped_kernel<2, false, R>;
        default: return any_k ? gemv3_grouped_kernel<3, true, R> : gemv3_grouped_kernel<3, false, R>;
    }
}

}  // namespace

hipError_t gemv3_init()
{
    for (int any_k = 0; any_k < 2; ++any_k)
        for (int T = 1; T <= kT3Max; ++T) {
            auto raise = [](const void* fn) { return hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, kLds3); };
            hipError_t e = raise(reinterpret_cast<const void*>(pick3(T, any_k != 0)));
            if (e == hipSuccess && T <= 3) e = raise(reinterpret_cast<const void*>(pick3_stream(T, any_k != 0)));
            if (e == hipSuccess && T <= 3) e = raise(reinterpret_cast<const void*>(pick3_grouped<kRec3Few>(T, any_k != 0)));
            if (e == hipSuccess && T <= 3) e = raise(reinterpret_cast<const void*>(pick3_grouped<kRec3Many>(T, any_k != 0)));
            if (e != hipSuccess) return e;
        }
    return hipSuccess;
}

bool gemv3_supports(int64_t M, int64_t N, int64_t K)
{
    return M >= 1 && N >= 1 && K >= 8 && K <= (int64_t(1) << 24) &&
           N <= (int64_t(1) << 24) && (M + 15) / 16 <= 65535;
}

// What a CU holds of the stream form: LDS is handed out in units of 1280 bytes of 160 KB, and one workgroup of 15 waves fills it.  With one
// wave 12 workgroups would fit and with two 7, but from 8 waves on another one only adds a start (N from 20000 on: one wave 8 workgroups
// 1.018 times as fast as 12, two waves 4 1.12 times as fast as 7).  Asked for more than fit (3 and 5 waves: 5 and 3 instead of 4 and 2),
// the last ones ran as a second round: 1.18 to 1.28 times as long.
int gemv3_per_cu(int waves, int* lds)
{
    const int bytes = (waves * kWaveLds + kLutBytes + 1279) / 1280 * 1280;
    const int by_lds = 160 * 1024 / bytes, by_waves = waves <= 2 ? 8 / waves : kWaves3 / waves;
    if (lds) *lds = bytes;
    return by_lds < by_waves ? by_lds : by_waves;
}

bool gemv3_groups(int64_t M, int64_t N, int64_t K)
{
    // K in one pass of the stream form
    return gemv3_supports(M, N, K) && (K + 4) / 5 <= int64_t(kWaves3) * 64;
}

// Several GEMMs in one launch of the stream form: every block of 16 activation rows of every GEMM
// is a job, the workgroups are dealt out to the jobs (tl_deal.hpp; the constants of the cost model are
// those measured for the 2-bit kernel: no others were tried for this one), and each workgroup gets a
// record with its run.
hipError_t launch_gemv3_jobs(const Gemm3Desc* jobs, int count, bool fx, hipStream_t s)
{
    for (int i = 0; i < count; ++i)
        if (!gemv3_groups(jobs[i].M, jobs[i].N, jobs[i].K)) return hipErrorInvalidValue;
    struct Block { int job; int64_t m0; int rows; };
    Block blk[kMaxBlocks3];
    int nb = 0;
    static std::atomic<bool> lds_raised[kMaxDevices][2][2][4];
    auto flush = [&]() -> hipError_t {
        if (nb == 0) return hipSuccess;
        DealJob dj[kMaxBlocks3];
        int NW = 1;
        int64_t total_tiles = 0;
        bool any_k = false;
        for (int q = 0; q < nb; ++q) {
            const Gemm3Desc& d = jobs[blk[q].job];
            const int tiles = int((d.N + 15) / 16);
            const int slices = int((d.stride + 63) / 64);
            dj[q] = DealJob{tiles, 1, 0.15 * double(blk[q].rows)};
            total_tiles += tiles;
            any_k = any_k || d.K % 8 != 0;
            if (slices > NW) NW = slices;
        }
        const int most = gemv3_per_cu(NW) >= 2 && total_tiles >= 8 * kRec3Few ? kRec3Many : kRec3Few;
        const int G = total_tiles < most ? int(total_tiles) : most;
        const DealModel model{3, true, 2.1, 0.43};
        int wg[kMaxBlocks3];
        deal_workgroups(model, dj, nb, G, wg);
        int run = 1, grid = 0;
        for (int q = 0; q < nb; ++q) {
            const int r = (dj[q].tiles + wg[q] - 1) / wg[q];
            if (r > run) run = r;
            grid += wg[q];
        }
        if (grid > most) return hipErrorInvalidValue;       // more jobs than workgroups: cannot happen with kMaxBlocks3 <= kRec3Few
        int T = run <= 3 ? run : (run == 4 ? 2 : 3);
        if (T > NW) T = NW;                                // the epilogue gives every thread at most one output quad
        auto send = [&](auto many) -> hipError_t {
            constexpr int R = decltype(many)::value;
            Rec3Batch<R> rb;
            int g = 0;
            for (int q = 0; q < nb; ++q) {
                const Gemm3Desc& d = jobs[blk[q].job];
                const int per = dj[q].tiles / wg[q], plus = dj[q].tiles % wg[q];
                for (int w = 0; w < wg[q]; ++w) {
                    Run3& r = rb.rec[g++];
                    r.W = d.W;
                    r.x = reinterpret_cast<const unsigned char*>(d.x + blk[q].m0 * d.K);
                    r.y = d.y + blk[q].m0 * d.N;
                    r.gamma = d.gamma;
                    r.K = int(d.K); r.N = int(d.N); r.stride = int(d.stride);
                    r.Mrem = blk[q].rows;
                    r.tile0 = w * per + (w < plus ? w : plus);
                    r.tile_end = r.tile0 + per + (w < plus ? 1 : 0);
                    r.fx = fx ? 1 : 0;
                }
            }
            const Grouped3Fn<R> fn = pick3_grouped<R>(T, any_k);
            const int dev = device_slot();
            std::atomic<bool>& raised = lds_raised[dev < 0 ? 0 : dev][any_k][R == kRec3Many][T];
            if (dev < 0 || !raised) {
                const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(fn),
                                                         hipFuncAttributeMaxDynamicSharedMemorySize, kLds3);
                if (e != hipSuccess) return e;
                if (dev >= 0) raised = true;
            }
            hipLaunchKernelGGL(fn, dim3(grid), dim3(NW * 64), size_t(NW) * kWaveLds + kLutBytes, s, rb);
            return hipGetLastError();
        };
        const hipError_t e = most == kRec3Many ? send(std::integral_constant<int, kRec3Many>{}) : send(std::integral_constant<int, kRec3Few>{});
        nb = 0;
        return e;
    };
    for (int i = 0; i < count; ++i) {
        for (int64_t m0 = 0; m0 < jobs[i].M; m0 += 16) {
            blk[nb++] = Block{i, m0, int(jobs[i].M - m0 < 16 ? jobs[i].M - m0 : 16)};
            if (nb == kMaxBlocks3) {
                const hipError_t e = flush();
                if (e != hipSuccess) return e;
            }
        }
    }
    return flush();
}

hipError_t launch_gemv3(const __half* x, const uint8_t* Wp, int64_t stride, float gamma, __half* y,
                        int64_t M, int64_t N, int64_t K, bool fx, hipStream_t s)
{
    Gemv3Params p;
    p.fx = fx ? 1 : 0;
    p.x = x; p.W = Wp; p.y = y; p.gamma = gamma;
    p.M = int(M); p.N = int(N); p.K = int(K);
    p.stride = int(stride);
    p.tiles = int((N + 15) / 16);
    const int slices = int((stride + 63) / 64);
    int groups = p.tiles < 256 ? p.tiles : 256;
    static std::atomic<bool> lds_raised[kMaxDevices][2][2][kT3Max + 1];
    const bool any_k = K % 8 != 0;
    const int dev = device_slot();
    auto raise = [&](Kernel3Fn fn, int form, int T) -> hipError_t {
        if (dev >= 0 && lds_raised[dev][any_k][form][T]) return hipSuccess;
        const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(fn),
                                                 hipFuncAttributeMaxDynamicSharedMemorySize, kLds3);
        if (e == hipSuccess && dev >= 0) lds_raised[dev][any_k][form][T] = true;
        return e;
    };
    dim3 grid(groups, unsigned((M + 15) / 16));
    if (slices <= kWaves3) {
        // every block of 16 activation rows is a set of workgroups of its own (blockIdx.y); they
        // share the CUs, as many workgroups in all as 256 CUs hold, so that the launch is one round
        // with longer runs
        const int mblocks = int((M + 15) / 16);
        const int NW = slices;
        int share = 256 * gemv3_per_cu(NW) / mblocks;
        if (share < 1) share = 1;
        const int64_t runs = (int64_t(p.tiles) * 16 * stride + (int64_t(1) << 31) - 1) >> 31;     // a run is addressed with 32 bits
        if (share < runs) share = int(runs);
        groups = p.tiles < share ? p.tiles : share;
        grid.x = unsigned(groups);
        // K in one pass: the stream form.  Tiles per item as for the 2-bit stream kernel: runs
        // of up to 3 tiles are one item, a run of 4 goes as 2 + 2, longer runs in items of 3.
        const int run = (p.tiles + groups - 1) / groups;
        int T = run <= 3 ? run : (run == 4 ? 2 : 3);
        if (T > NW) T = NW;                                // the epilogue gives every thread at most one output quad
        p.groups = groups;
        Kernel3Fn fn = pick3_stream(T, any_k);
        const hipError_t e = raise(fn, 1, T);
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(fn, grid, dim3(NW * 64), size_t(NW) * kWaveLds + kLutBytes, s, p);
        return hipGetLastError();
    }
    int T = (p.tiles + groups - 1) / groups;
    if (T > kT3Max) { T = kT3Max; groups = (p.tiles + T - 1) / T; }
    p.groups = groups;
    grid.x = unsigned(groups);
    Kernel3Fn fn = pick3(T, any_k);
    const hipError_t e = raise(fn, 0, T);
    if (e != hipSuccess) return e;
    const int passes = (slices + kWaves3 - 1) / kWaves3, NW = (slices + passes - 1) / passes;       // as even as they get
    hipLaunchKernelGGL(fn, grid, dim3(NW * 64), size_t(NW) * kWaveLds + kLutBytes, s, p);
    return hipGetLastError();
}

}  // namespace tl
