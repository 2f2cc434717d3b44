// The tiled matrix-core kernel for many activation rows: Y = X (gamma What)^T of App. B with the
// packed forms of Sec. 3 decoded to fp16 in registers right before the matrix instruction that
// consumes them.  One kernel for every packed form (2-bit words, 2-bit words with group scales,
// both 1.6-bit byte codes) and every K; what differs is how a step's weights get into LDS.
//
// A workgroup of 8 waves owns a BM x BN tile of Y.  K is walked in steps of KS = 32 NP; the waves form
// WK sets that share the NP 32-k blocks of a step out among them, and WM x WN waves per set, each with
// FM x FN fragments of v_mfma_f32_16x16x32_f16.
//
//  * What bounds it: at full size the matrix pipes are busy 0.59 of the time; without the X fragment reads the kernel is
//    20 % faster, without the decode 6 %, on zero operands, i.e. at the highest clock, 13 %.  Bare loops of the matrix
//    instruction on this data gave 1.85 (32x32x16, W as the row operand), 2.0 (32x32x16, X as the row operand) and 2.3
//    PFLOP/s (16x16x32), so the 16x16x32 form is used.  Small tiles are bound by latency: the start and end of a launch (5 to 6 us
//    of a 20 us call) and the barrier of each step; no unit is busy for more than 0.38 of the time.
//  * X goes to LDS as it lies in memory, by LDS-DMA (global_load_lds_dwordx4: no registers, no
//    vector instructions), ST steps ahead.  16-byte pieces of a row are swizzled by row on the way
//    in so that the fragment reads are free of bank conflicts.
//  * W stays packed in LDS: a 2-bit word holds 16 codes of one column, 1/8 of the bytes of fp16.  A lane
//    (column i, k quarter g) needs half a word as pairs of neighbours: one byte permute, one shift, and per pair one mask and one packed
//    fma (decode8_codes, decode8_values): 10 vector operations per 8 weights and lane between the matrix instructions of a fragment, and a
//    decoded operand feeds FM of them.
//  * 1.6-bit forms are transcoded to 2-bit words once per workgroup and step: a thread looks up the
//    8 bytes of a column's 40 weights in a 256-entry table of 10-bit entries and writes 80 bits of
//    codes to LDS two steps before they are used.  A step is then 160 k or a multiple.
//  * Group scales (one per 16 k, or per set and step, and column) travel with the step by LDS-DMA
//    and multiply the decoded operand: s (c - 1) is exact in fp16.
//  * One barrier per step, and it stands before the last block's matrix instructions, whose
//    operands are in registers by then; the transfers of the step ST further on are spread between the matrix
//    instructions (all of them right behind the barrier: 385k instead of 361k clocks for two tiles of
//    256 x 256 x 4096).
//  * The W fragments are the 16-row operand, so a lane ends up with four consecutive columns of a row of Y;
//    they are turned through LDS and stored in 16-byte pieces.
//
// Measured, 4096 -> 14336, M = 2048 (256 x 256 tiles): 172 to 184 us (1.31 to 1.40 PFLOP/s) on four machines where the
// kernel before (128 x 256 tiles of 32x32x16, X through registers) took 207 to 216.
#pragma once
#include "tl_grid.hpp"
#include "tl_internal.hpp"

#include <atomic>
#include <type_traits>

namespace tl {

enum TileFmt { kTile2Bit = 0, kTileGs = 1, kTile1p6 = 2 };

struct TileParams {
    const __half* x;
    const unsigned char* W;      // packed rows
    const __half* scales;        // kTileGs: [ceil(K / group)][N]
    __half* y;
    float gamma;
    int M, N, K;
    int row_bytes;               // bytes per packed row
    int group16;                 // kTileGs: 16-k blocks per group
    int fx;                      // kTile1p6: fixed-point byte code
    int tiles_m, tiles_n;
};

// RAGGED: K (at least 8) is not a multiple of 64 (2-bit) or 8 (1.6-bit): rows of X and W start anywhere, X goes
// through registers (masked past K) and 2-bit words are fetched one by one.
// UNIT: 16-k blocks per scale that is fetched (kTileGs): a set's part of a step, 2 NB of them, or 1, which takes any group.
template <int FMT_, bool RAGGED_, int FM_, int FN_, int WM_, int WN_, int WK_, int NP_, int ST_, int UNIT_ = 1>
struct TileCfg {
    static constexpr int FMT = FMT_, FM = FM_, FN = FN_, WM = WM_, WN = WN_, WK = WK_, NP = NP_;
    static constexpr bool RAGGED = RAGGED_;
    static constexpr int ST = RAGGED ? 2 : ST_;
    static constexpr int NB = (NP + WK - 1) / WK;                 // blocks of a set (sets past NP % WK have one less)
    static constexpr int BM = 16 * FM * WM, BN = 16 * FN * WN;
    static constexpr int KS = 32 * NP;
    static constexpr int P = KS / 8;                              // 16-byte pieces per X row and step
    static constexpr int XD = (BM * P + 511) / 512;               // pieces per thread and step
    static constexpr int XST = XD * 8192;                         // bytes of an X stage (surplus pieces land in its padding)
    static constexpr bool CODES = FMT == kTile1p6;                // W goes through the transcoder
    static constexpr int CH = KS / 80;                            // 1.6-bit: 16-byte chunks per column and step
    static constexpr int WST = CODES ? BN * CH * 16 : BN * KS / 4;   // bytes of a W stage (raw bytes or words)
    static constexpr int WSLOTS = CODES ? 2 : ST;
    static constexpr int WL = WST / 16 / 8;                       // lanes per wave in the W transfer (16 bytes each)
    static constexpr int WD = RAGGED ? (CODES ? BN * CH * 2 / 512 : WST / 4 / 512) : 1;   // fetches per thread and step (RAGGED)
    static constexpr int DEP = 4;                                 // RAGGED: steps of X and W on their way in registers
    static constexpr int CST = CODES ? BN * KS / 4 : 0;           // a slot of transcoded words, [word][column]
    static constexpr bool PARTIAL = CODES || KS > 64;   // the last step may reach past K
    static constexpr int UNIT = UNIT_;
    static constexpr int NU = FMT == kTileGs ? 2 * NP / UNIT : 0; // scale rows per step
    static constexpr int SD = (NU * BN + 511) / 512;              // scale transfers per wave and step
    static constexpr int SST = SD * 2048;
    static constexpr int OFF_W = ST * XST;
    static constexpr int OFF_S = OFF_W + WSLOTS * WST;
    static constexpr int OFF_C = OFF_S + ST * SST;
    static constexpr int OFF_T = OFF_C + 2 * CST;
    static constexpr int RING = OFF_T + (CODES ? 1024 : 0);
    // sums of the sets: all of them side by side (four sets and more), else half of the waves hand theirs over
    static constexpr int SROW = BN * 4 + 16;                      // bytes per row of a set's sums (padded: 16 rows in different banks)
    static constexpr bool SHARE = WK >= 4;
    static constexpr int RED = SHARE ? WK * BM * SROW : (WK > 1 ? 4 * FM * FN * 1024 : 0);
    static constexpr int OUT = 8 * 16 * (FN * 32 + 16);           // 16 rows of every wave's tile as fp16
    static constexpr int LDS = RING > RED ? (RING > OUT ? RING : OUT) : (RED > OUT ? RED : OUT);
    // waves per SIMD: two workgroups per CU where LDS and registers hold them
    static constexpr int OCC = LDS <= 80 * 1024 && FM * FN <= (RAGGED ? (CODES ? 0 : 4) : 8) ? 4 : 2;
    static_assert(WM * WN * WK == 8, "8 waves");
    static_assert(LDS <= 160 * 1024, "tile does not fit");
    static_assert(FN == 2 || FN == 4, "rolling decode: a fragment is decoded while the others are multiplied");
    static_assert(BN % 64 == 0 || FMT == kTile2Bit, "a wave fetches scales and bytes of one row of units or chunks");
    static_assert((CODES ? KS % 80 == 0 : KS % 64 == 0) && WL <= 64 && WD >= 1, "step");
    static_assert(UNIT == 1 || (UNIT == 2 * NB && NP % WK == 0), "scale unit: 16 k, or a set's part of a step");
};

namespace tile {

// rows of X and Y start at any even byte where K or N is odd; the memory takes such addresses in one piece
typedef u32x4 __attribute__((aligned(2))) u32x4_any;
typedef u32x2 __attribute__((aligned(2))) u32x2_any;

template <int N>
__device__ __forceinline__ void wait_vm()
{
    asm volatile("s_waitcnt vmcnt(%0)" : : "n"(N) : "memory");
}

// LDS writes and reads of this wave done, then the workgroup's barrier; global transfers stay in flight
__device__ __forceinline__ void lds_barrier()
{
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" : : : "memory");
}

// The transfers are written out by hand (LDS base in M0, lane l lands at base + 16 l, of 2 bytes at base + 4 l): a transfer
// the compiler knows of makes it drain the memory pipeline before every later LDS access.  Every
// wait for them is an explicit wait_vm.  gfx950 asks for one wait state between a scalar write of M0 and the transfer that
// reads it; the compiler adds it for its own transfers and looks into no string, so it stands here (dma16_lanes has
// the exec write in between).  Five more states would be due after a vector instruction that writes the base's scalar
// registers; none does, and a test reads the built code for both.
__device__ __forceinline__ void dma16(uint32_t voff, const void* sbase, uint32_t lds)
{
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1" : : "v"(voff), "s"(sbase), "s"(__builtin_amdgcn_readfirstlane(lds)) : "memory");
}
// the same for the lanes of `mask` only (all lanes are active around it)
__device__ __forceinline__ void dma16_lanes(uint32_t voff, const void* sbase, uint32_t lds, unsigned long long mask)
{
    asm volatile("s_mov_b32 m0, %2\n\ts_mov_b64 exec, %3\n\tglobal_load_lds_dwordx4 %0, %1\n\ts_mov_b64 exec, -1"
                 : : "v"(voff), "s"(sbase), "s"(__builtin_amdgcn_readfirstlane(lds)), "s"(mask) : "memory");
}
__device__ __forceinline__ void dma2(uint32_t voff, const void* sbase, uint32_t lds)   // zero-extended to a dword
{
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_ushort %0, %1" : : "v"(voff), "s"(sbase), "s"(__builtin_amdgcn_readfirstlane(lds)) : "memory");
}

__device__ __forceinline__ uint32_t pkfma(uint32_t a, uint32_t b, uint32_t c)
{
    const f16x2 r = __builtin_elementwise_fma(__builtin_bit_cast(f16x2, a), __builtin_bit_cast(f16x2, b),
                                              __builtin_bit_cast(f16x2, c));
    return __builtin_bit_cast(uint32_t, r);
}

// Half of a packed word (8 codes, in order) -> fp16 pairs of neighbours, in two parts.  The half word is doubled, so that code 2q stands
// at bit 4q of the lower half and code 2q + 1 at bit 4q + 2 of the upper half; one packed fma with a factor of its own for each half
// takes the positions away.  sel: the byte selector of this lane's half.
//  * kScaled: (c - 1) 2^-9, from the subnormals c 2^(p - 24), times 2^(15 - p): no merge, the same sum for all; the factor 2^9 is exact and
//    goes into gamma.
//  * kUnit: (c - 1) itself, from 1024 + c 2^p (bits merged into k1024): group scales, the smallest of which kScaled would cost bits.
//  * kMoved: as kUnit, with the odd codes moved down by 2 beforehand, one operation more, the same factor for both halves: tiles of 16 rows
//    (one product per decoded operand), whose calls it keeps 1.5 % (2-bit) and 1.2 % (1.6-bit) faster than kScaled, 2.4 and 0.2 % than
//    kUnit (means over 167 and 161 calls with odd K, M = 2 .. 300).
// 10 operations where the odd codes moved down took 11; in two halves of a fragment's products instead of one: 128 x 128 tiles
// 31.1 -> 30.3 us at 1024 x 4096 x 4096, with both 256 x 256 tiles 171.3 -> 169.5 us at 2048 x 14336 x 4096.
enum Decode { kScaled, kUnit, kMoved };

template <Decode D>
__device__ __forceinline__ uint32_t decode_selector(bool upper)
{
    if constexpr (D == kMoved) return upper ? 0x07060302u : 0x05040100u;
    return upper ? 0x03020302u : 0x01000100u;
}
template <Decode D>
__device__ __forceinline__ u32x4 decode8_codes(uint32_t w, uint32_t sel, uint32_t k1024)
{
    const uint32_t u = __builtin_amdgcn_perm(D == kMoved ? w >> 2 : w, w, sel);
    const uint32_t v = u >> 8;
    constexpr uint32_t c0 = D == kMoved ? 0x00030003u : 0x000C0003u, c1 = D == kMoved ? 0x00300030u : 0x00C00030u;
    if constexpr (D == kScaled) return u32x4{u & c0, u & c1, v & c0, v & c1};
    return u32x4{(u & c0) | k1024, (u & c1) | k1024, (v & c0) | k1024, (v & c1) | k1024};
}
template <Decode D>
__device__ __forceinline__ u32x4 decode8_values(u32x4 o)
{
    // 2^-p or 2^(15 - p), and -(2^(10 - p) + 1) or -2^-9, for the positions 0 and 4, odd codes 2 further up unless moved
    constexpr uint32_t m0 = D == kMoved ? 0x3C003C00u : D == kUnit ? 0x34003C00u : 0x70007800u, m1 = D == kMoved ? 0x2C002C00u : D == kUnit ? 0x24002C00u : 0x60006800u;
    constexpr uint32_t a0 = D == kMoved ? 0xE401E401u : D == kUnit ? 0xDC04E401u : 0x98009800u, a1 = D == kMoved ? 0xD410D410u : D == kUnit ? 0xCC40D410u : 0x98009800u;
    return u32x4{pkfma(o[0], m0, a0), pkfma(o[1], m1, a1), pkfma(o[2], m0, a0), pkfma(o[3], m1, a1)};
}

// Piece q of row r of an X stage lies at 16-byte slot r P + slot.  A fragment read takes 4 neighbouring pieces of
// 16 rows; the slots put one piece of 16 consecutive rows into different bank quads.
template <int P>
__device__ __forceinline__ int slot_of(int row, int q)
{
    if constexpr (P == 8) return q ^ ((row >> 1) & 7);
    else if constexpr (P == 20) { const int s = q + ((row >> 2) & 3); return s >= 20 ? s - 20 : s; }
    else if constexpr (P == 40) { const int s = q + ((row >> 1) & 7); return s >= 40 ? s - 40 : s; }
    else return q ^ (row & 15);                           // P = 16, 32
}
template <int P>
__device__ __forceinline__ int piece_of(int row, int slot)
{
    if constexpr (P == 8) return slot ^ ((row >> 1) & 7);
    else if constexpr (P == 20) { const int s = slot - ((row >> 2) & 3); return s < 0 ? s + 20 : s; }
    else if constexpr (P == 40) { const int s = slot - ((row >> 1) & 7); return s < 0 ? s + 40 : s; }
    else return slot ^ (row & 15);
}

}  // namespace tile

template <class C>
__global__ void __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(C::OCC, C::OCC)))
tile_kernel(TileParams p)
{
    using namespace tile;
    extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
    constexpr int FM = C::FM, FN = C::FN, NB = C::NB, WK = C::WK, NP = C::NP, KS = C::KS, P = C::P, BN = C::BN, BM = C::BM, ST = C::ST;
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int set = wave / (C::WM * C::WN);
    const int wm = (wave / C::WN) % C::WM, wn = wave % C::WN;
    const uint32_t lds0 = uint32_t(uintptr_t((const __attribute__((address_space(3))) unsigned char*)lds));

    // Tile order: workgroup ids go round the 8 XCDs, each with an L2 of its own.  An XCD takes a
    // contiguous piece of an order that walks the grid in bands of 4 row blocks, column by column, so the
    // workgroups resident on it share row blocks of X four columns at a time and columns of W.
    int tm, tn;
    {
        const int total = p.tiles_m * p.tiles_n;
        const int xcd = int(blockIdx.x) & 7, q = int(blockIdx.x) >> 3;
        const int rem = total & 7;
        const int lin = xcd * (total >> 3) + (xcd < rem ? xcd : rem) + q;
        const int per_band = 4 * p.tiles_n;
        const int band = lin / per_band, r = lin - band * per_band;
        const int height = p.tiles_m - 4 * band < 4 ? p.tiles_m - 4 * band : 4;
        tn = r / height;
        tm = 4 * band + (r - tn * height);
    }
    const int m_base = tm * BM, n_base = tn * BN;
    const int K = p.K;
    const int nblk = (K + 31) >> 5;                       // 32-k blocks
    const int steps = (nblk + NP - 1) / NP;
    // the set's blocks of a step: NB of them, or one less, from block0 on
    constexpr int kFullSets = NP % WK == 0 ? WK : NP % WK;
    const bool short_set = kFullSets < WK && set >= kFullSets;
    const int block0 = set * NB - (kFullSets < WK && set > kFullSets ? set - kFullSets : 0);

    // ---- X transfers ------------------------------------------------------------------------------
    const unsigned char* const xtile = reinterpret_cast<const unsigned char*>(p.x + size_t(m_base) * K);
    uint32_t xoff[C::XD];                                 // row start within the tile, bytes
    const int mlast = p.M - 1 - m_base;
#pragma unroll
    for (int d = 0; d < C::XD; ++d) {
        const int lin = (d * 8 + wave) * 64 + lane;
        const int row = lin / P;
        xoff[d] = uint32_t(row < mlast ? row : mlast) * uint32_t(K) * 2u;   // rows past M repeat the last one, never stored
        if constexpr (!C::RAGGED) xoff[d] += uint32_t(piece_of<P>(row, lin - row * P)) * 16u;
    }
    // the piece of transfer d (LDS-DMA form: worked out again where it is needed, not kept in a register)
    auto piece = [&](int d) {
        int l = lane;
        if constexpr (!C::RAGGED) asm volatile("" : "+v"(l));
        const int lin = (d * 8 + wave) * 64 + l;
        const int row = lin / P;
        return uint32_t(piece_of<P>(row, lin - row * P));
    };
    // DMA form, step s into stage st = s mod ST.  Pieces past K read the row's first piece: their weights are zero, and
    // a NaN there stays within its own row.
    auto issue_x = [&](int s, int st, int d, auto inside) {
        const uint32_t dst = lds0 + uint32_t(st) * C::XST + uint32_t(wave) * 1024u + uint32_t(d) * 8192u;
        if (!C::PARTIAL || decltype(inside)::value || (s + 1) * KS <= K) {
            dma16(xoff[d], xtile + size_t(s) * (KS * 2), dst);
        } else {
            const uint32_t q = piece(d), k = uint32_t(s) * KS + q * 8u;
            dma16(k < uint32_t(K) ? xoff[d] + uint32_t(s) * (KS * 2) : xoff[d] - q * 16u, xtile, dst);
        }
    };
    // ---- W transfers --------------------------------------------------------------------------------
    const unsigned char* const wtile = p.W + size_t(n_base) * size_t(p.row_bytes);
    const int nlast = p.N - 1 - n_base;
    constexpr int PW = C::CODES ? C::CH : KS / 64;           // 16-byte pieces per column and step
    uint32_t woff, wpc;
    {
        const int lin = wave * C::WL + lane;
        const int col = lin / PW;
        wpc = uint32_t(lin - col * PW);
        woff = uint32_t(col < nlast ? col : nlast) * uint32_t(p.row_bytes);
    }
    auto issue_w = [&](int s, int st, auto inside) {
        const uint32_t base = lds0 + C::OFF_W + uint32_t(C::CODES ? s & 1 : st) * C::WST;
        const uint32_t dst = base + uint32_t(wave) * (C::WL * 16);
        constexpr unsigned long long lanes = C::WL == 64 ? ~0ull : (1ull << (C::WL & 63)) - 1;
        const unsigned char* src = wtile + size_t(s) * (PW * 16);
        uint32_t o = woff + wpc * 16u;
        if constexpr (C::PARTIAL && !decltype(inside)::value) {
            if ((uint32_t(s) * PW + wpc) * 16u >= uint32_t(p.row_bytes)) o = woff;   // past the row: fetched, never used
        }
        if constexpr (C::WL == 64) dma16(o, src, dst);
        else dma16_lanes(o, src, dst, lanes);
    };

    // ---- scale transfers: transfer d of a wave fetches 64 columns of one scale row of the step.  The steps are asked for
    // in order, so the row's group is carried along instead of divided out.
    constexpr int SD1 = C::SD > 0 ? C::SD : 1;
    int sgroup[SD1], sleft[SD1], sblk[SD1];               // group, 16-k blocks into it, 16-k block
    const int group16 = C::FMT == kTileGs ? p.group16 : 1;
    const int sgroups = (KS / 16) / group16, sblocks = (KS / 16) - sgroups * group16;
    const int slast = ((K - 1) >> 4) / group16;
#pragma unroll
    for (int d = 0; d < C::SD; ++d) {
        int unit = (d * 8 + wave) * 64 / BN;              // BN is a multiple of 64: one scale row per transfer
        if (unit >= C::NU) unit = C::NU - 1;              // surplus waves fetch into padding
        sblk[d] = unit * C::UNIT;
        sgroup[d] = sblk[d] / group16;
        sleft[d] = sblk[d] - sgroup[d] * group16;
    }
    // the row of transfer d for the next step that has not been asked for
    auto scale_row = [&](int d) {
        const __half* const r = p.scales + size_t(sblk[d] * 16 < K ? sgroup[d] : slast) * size_t(p.N) + n_base;
        sblk[d] += KS / 16;
        sgroup[d] += sgroups;
        sleft[d] += sblocks;
        if (sleft[d] >= group16) { sleft[d] -= group16; ++sgroup[d]; }
        return r;
    };
    auto scale_col = [&](int d) {
        const int col = (d * 8 + wave) * 64 % BN + lane;
        return uint32_t(col < nlast ? col : nlast);
    };
    auto issue_s = [&](int st, int d) {
        dma2(scale_col(d) * 2u, scale_row(d), lds0 + C::OFF_S + uint32_t(st) * C::SST + uint32_t(d * 8 + wave) * 256u);
    };
    // Transfer d of a step's D: the weights, the scales, then X (the order matters for the 1.6-bit forms: their
    // bytes are waited for one step before X).
    constexpr int D = 1 + C::SD + C::XD;
    auto issue = [&](int s, int st, auto dt, auto inside) {
        constexpr int d = decltype(dt)::value;
        if constexpr (d == 0) issue_w(s, st, inside);
        else if constexpr (d <= C::SD) issue_s(st, d - 1);
        else issue_x(s, st, d - 1 - C::SD, inside);
    };

    // ---- 1.6-bit bytes -> 2-bit words: 8 bytes (40 weights) per thread -----------------------------------
    const int nbytes = (K + 4) / 5;
    uint32_t* const table = reinterpret_cast<uint32_t*>(lds + C::OFF_T);
    // round r of a step's: threads take a column's 8 bytes each (BN is a multiple of 64: chunk and half are a wave's)
    constexpr int ROUNDS = C::CODES ? (BN * C::CH * 2 + 511) / 512 : 0;
    auto transcode_one = [&](int s, int r, u32x2 raw, auto inside) {
        const int w0 = r * 512 + wave * 64;
        const int part = w0 / BN, col = w0 - part * BN + lane;
        const int ch = part >> 1, half = part & 1;
        uint32_t e[8];
#pragma unroll
        for (int b = 0; b < 8; ++b) e[b] = table[(raw[b >> 2] >> (8 * (b & 3))) & 255u];
        if (!decltype(inside)::value && (s + 1) * (C::CH * 16) >= nbytes) {
            // Bytes past the row count as weight 0, and so do the last byte's digits past K, whatever they are: X holds the
            // row's first activations there and not zeros.
            const int b0 = (s * C::CH + ch) * 16 + half * 8;
            const uint32_t keep = (1u << (2 * (K - (nbytes - 1) * 5))) - 1u;
#pragma unroll
            for (int b = 0; b < 8; ++b) {
                const uint32_t m = b0 + b < nbytes - 1 ? ~0u : (b0 + b == nbytes - 1 ? keep : 0u);
                e[b] = (e[b] & m) | (0x155u & ~m);
            }
        }
        const uint32_t d0 = e[0] | (e[1] << 10) | (e[2] << 20) | (e[3] << 30);
        const uint32_t d1 = (e[3] >> 2) | (e[4] << 8) | (e[5] << 18) | (e[6] << 28);
        const uint32_t d2 = (e[6] >> 4) | (e[7] << 6);       // 16 bits
        uint32_t* const c = reinterpret_cast<uint32_t*>(lds + C::OFF_C + (s & 1) * C::CST) + (ch * 5) * BN + col;
        uint16_t* const mid = reinterpret_cast<uint16_t*>(c + 2 * BN);
        if (half == 0) {
            c[0] = d0;
            c[BN] = d1;
            mid[0] = uint16_t(d2);
        } else {                              // 80 bits from bit 80 on
            mid[1] = uint16_t(d0);
            c[3 * BN] = (d0 >> 16) | (d1 << 16);
            c[4 * BN] = (d1 >> 16) | (d2 << 16);
        }
    };
    auto transcode = [&](int s, auto inside) {
#pragma unroll
        for (int r = 0; r < ROUNDS; ++r) {
            __builtin_amdgcn_sched_barrier(0);            // one round's look-ups in registers at a time
            const int w0 = r * 512 + wave * 64;
            if (BN * C::CH * 2 - r * 512 >= 512 || w0 < BN * C::CH * 2) {
                const int part = w0 / BN, col = w0 - part * BN + lane;
                transcode_one(s, r, *reinterpret_cast<const u32x2*>(lds + C::OFF_W + (s & 1) * C::WST + (col * C::CH + (part >> 1)) * 16 + (part & 1) * 8), inside);
            }
        }
    };

    // ---- RAGGED: X, W and the scales of a step through registers, DEP steps ahead.  Rows start anywhere, so a thread fetches
    // its 16 bytes of X from wherever they lie; a piece that reaches past K is fetched from the row's last 16
    // bytes and shifted down, which leaves zeros past K (so whatever W holds there does not matter), and one that lies
    // past K altogether is zero.  All fetches are unconditional: their steps and offsets are held inside the rows.
    typedef const __attribute__((address_space(1))) unsigned char* gbytes;
    constexpr int DEP = C::DEP;
    u32x4 rx[C::RAGGED ? DEP : 1][C::XD];
    uint32_t rw[C::RAGGED ? DEP : 1][C::WD * (C::CODES ? 2 : 1)];
    uint16_t rs[C::RAGGED ? DEP : 1][SD1];
    auto fetch = [&](int t, auto slot) {
        if constexpr (C::RAGGED) {
            constexpr int j = decltype(slot)::value;
#pragma unroll
            for (int d = 0; d < C::XD; ++d) {
                uint32_t k = uint32_t(t) * KS + piece(d) * 8u;
                k = k < uint32_t(K) - 8u ? k : uint32_t(K) - 8u;
                rx[j][d] = *(const __attribute__((address_space(1))) u32x4_any*)((gbytes)xtile + xoff[d] + k * 2u);
            }
#pragma unroll
            for (int d = 0; d < C::WD; ++d) {
                if constexpr (C::CODES) {
                    const int w0 = d * 512 + wave * 64;
                    const int part = w0 / BN, col = w0 - part * BN + lane;
                    uint32_t o = (uint32_t(t) * C::CH + uint32_t(part >> 1)) * 16u + uint32_t(part & 1) * 8u;
                    o = o < uint32_t(p.row_bytes) - 8u ? o : uint32_t(p.row_bytes) - 8u;
                    const u32x2 v = *(const __attribute__((address_space(1))) u32x2*)((gbytes)wtile + uint32_t(col < nlast ? col : nlast) * uint32_t(p.row_bytes) + o);
                    rw[j][2 * d] = v[0];
                    rw[j][2 * d + 1] = v[1];
                } else {
                    const int lin = d * 512 + tid;        // word: column lin / (KS / 16)
                    const int col = lin / (KS / 16);
                    uint32_t o = (uint32_t(t) * (KS / 16) + uint32_t(lin - col * (KS / 16))) * 4u;
                    o = o < uint32_t(p.row_bytes) - 4u ? o : uint32_t(p.row_bytes) - 4u;
                    rw[j][d] = *(const __attribute__((address_space(1))) uint32_t*)((gbytes)wtile + uint32_t(col < nlast ? col : nlast) * uint32_t(p.row_bytes) + o);
                }
            }
#pragma unroll
            for (int d = 0; d < C::SD; ++d)
                rs[j][d] = *((const __attribute__((address_space(1))) uint16_t*)scale_row(d) + scale_col(d));
        }
    };
    // step t from its registers into stage t & 1
    auto put = [&](int t, auto slot) {
        if constexpr (C::RAGGED) {
            constexpr int j = decltype(slot)::value;
            const bool tail = (t + 1) * KS > K;
#pragma unroll
            for (int d = 0; d < C::XD; ++d) {
                u32x4 v = rx[j][d];
                if (tail) {
                    const int past = t * KS + int(piece(d)) * 8 + 8 - K;      // elements past K, 16 bits each
                    const uint64_t lo = uint64_t(v[0]) | (uint64_t(v[1]) << 32), hi = uint64_t(v[2]) | (uint64_t(v[3]) << 32);
                    const int n = 16 * (past > 0 ? past : 0);
                    uint64_t a = lo, b = hi;
                    if (n >= 128) { a = 0; b = 0; }
                    else if (n >= 64) { a = hi >> (n - 64); b = 0; }
                    else if (n > 0) { a = (lo >> n) | (hi << (64 - n)); b = hi >> n; }
                    v = u32x4{uint32_t(a), uint32_t(a >> 32), uint32_t(b), uint32_t(b >> 32)};
                }
                *reinterpret_cast<u32x4*>(lds + (t & 1) * C::XST + (d * 8 + wave) * 1024 + lane * 16) = v;
            }
#pragma unroll
            for (int d = 0; d < C::WD; ++d) {
                if constexpr (C::CODES) transcode_one(t, d, u32x2{rw[j][2 * d], rw[j][2 * d + 1]}, std::true_type{});
                else *reinterpret_cast<uint32_t*>(lds + C::OFF_W + (t & 1) * C::WST + (d * 512 + tid) * 4) = rw[j][d];
            }
#pragma unroll
            for (int d = 0; d < C::SD; ++d)
                *reinterpret_cast<uint32_t*>(lds + C::OFF_S + (t & 1) * C::SST + (d * 512 + tid) * 4) = rs[j][d];
        }
    };

    // ---- fragments ---------------------------------------------------------------------------------------
    const int fi = lane & 15, fg = lane >> 4;             // row of X / column of W, k quarter of a block
    constexpr Decode kDecode = FM == 1 ? kMoved : C::FMT == kTileGs ? kUnit : kScaled;
    const uint32_t sel = decode_selector<kDecode>(fg & 1);
    // in a vector register the compiler cannot see through: mask and merge are then one v_and_or_b32 (not kScaled)
    uint32_t k1024;
    asm volatile("v_mov_b32 %0, 0x64006400" : "=v"(k1024));
    const int xrow = wm * 16 * FM + fi;                   // + 16 a: the swizzle depends on row % 16 alone
    uint32_t xa[NB];                                      // fragment addresses within a stage, block ks
#pragma unroll
    for (int ks = 0; ks < NB; ++ks) {
        const int blk = block0 + ks < NP ? block0 + ks : 0;
        xa[ks] = uint32_t(xrow * P + slot_of<P>(xrow, blk * 4 + fg)) * 16u;
    }
    const int wcol = wn * 16 * FN + fi;                   // + 16 b
    f16x8 xf[2][FM];
    u32x4 wf[FN];
    // The lane's packed word per fragment: of all blocks of a step, or (1.6-bit forms, three blocks: registers) of one block
    constexpr int NCW = C::CODES ? 1 : NB;
    uint32_t cw[FN][NCW];
    uint32_t sc[FN][C::FMT == kTileGs && C::UNIT == 1 ? NB : 1];
    constexpr int NS = C::FMT == kTileGs && C::UNIT == 1 ? NB : 1;
    auto read_x = [&](auto par, int st, auto kst, auto from, auto to) {
        constexpr int PAR = decltype(par)::value, ks = decltype(kst)::value;
        const unsigned char* const b = lds + st * C::XST + xa[ks];
#pragma unroll
        for (int a = decltype(from)::value; a < decltype(to)::value; ++a)
            xf[PAR][a] = *reinterpret_cast<const f16x8*>(b + a * (16 * P * 16));
    };
    auto read_w = [&](int s, int st, auto kst, auto inside) {
        const int word0 = block0 * 2 + (fg >> 1);      // + 2 ks
#pragma unroll
        for (int b = 0; b < FN; ++b) {
            const int col = wcol + 16 * b;
            if constexpr (C::CODES) {
                const uint32_t* const c = reinterpret_cast<const uint32_t*>(lds + C::OFF_C + (s & 1) * C::CST) + col;
                cw[b][0] = c[(word0 + 2 * decltype(kst)::value) * BN];
            } else {
                const uint32_t* const c = reinterpret_cast<const uint32_t*>(lds + C::OFF_W + st * C::WST) + col * (KS / 16);
#pragma unroll
                for (int ks = 0; ks < NCW; ++ks) cw[b][ks] = c[word0 + 2 * ks];
            }
            if constexpr (C::PARTIAL && !C::CODES && !decltype(inside)::value) {
                if ((s + 1) * NP > nblk) {                // blocks past K: weights 0
#pragma unroll
                    for (int ks = 0; ks < NCW; ++ks)
                        if (s * NP + block0 + ks >= nblk) cw[b][ks] = 0x55555555u;
                }
            }
            if constexpr (C::FMT == kTileGs) {
                const uint32_t* const q = reinterpret_cast<const uint32_t*>(lds + C::OFF_S + st * C::SST) + col;
#pragma unroll
                for (int u = 0; u < NS; ++u) sc[b][u] = C::UNIT == 1 ? q[(word0 + 2 * u) * BN] : q[set * BN];
            }
        }
    };
    // one fragment (16 columns x 32 k): 6 (7 if moved) and 4 vector operations
    const float gamma = kDecode == kScaled ? p.gamma * 512.f : p.gamma;
    auto decode_codes = [&](int b, uint32_t word) { wf[b] = decode8_codes<kDecode>(word, sel, k1024); };
    auto decode_values = [&](int b, uint32_t scale) {
        u32x4 o = decode8_values<kDecode>(wf[b]);
        if constexpr (C::FMT == kTileGs) {
            const _Float16 s1 = __builtin_bit_cast(f16x2, scale)[0];
            const f16x2 s2 = {s1, s1};
#pragma unroll
            for (int q = 0; q < 4; ++q) o[q] = __builtin_bit_cast(uint32_t, __builtin_bit_cast(f16x2, uint32_t(o[q])) * s2);
        }
        wf[b] = o;
    };

    f32x4 acc[FM][FN];
#pragma unroll
    for (int a = 0; a < FM; ++a)
#pragma unroll
        for (int b = 0; b < FN; ++b) acc[a][b] = f32x4{0.f, 0.f, 0.f, 0.f};

    typedef std::integral_constant<int, 0> I0;
    typedef std::integral_constant<int, 1> I1;
    typedef std::integral_constant<int, 2> I2;
    typedef std::integral_constant<int, 3> I3;
    typedef std::false_type Any;
    // The D transfers of a step are spread over its 2 FN NB slots (two per fragment's matrix instructions): all at
    // once, they would hold up the waves at the CU's one address path (16 clocks per transfer) with
    // nothing left in the matrix pipes.  Slots count from the barrier on: the first 2 FN belong to the last block
    // of step s - ST, the others to the next step's blocks.
    auto run = [&](auto nb) {
    constexpr int NB = decltype(nb)::value;
    constexpr int SLOTS = 2 * FN * NB;
    typedef std::integral_constant<int, 0> IFirst;
    typedef std::integral_constant<int, 2 * FN> IEarly;
    typedef std::integral_constant<int, SLOTS> ISlots;
    auto issue_slots = [&](int s, int st, auto from, auto to, auto inside) {
        auto one = [&](auto dt) {
            constexpr int d = decltype(dt)::value;
            if constexpr (d < D) {
                constexpr int slot = d * SLOTS / D;
                if constexpr (slot >= decltype(from)::value && slot < decltype(to)::value) issue(s, st, dt, inside);
            }
        };
        one(std::integral_constant<int, 0>{}); one(std::integral_constant<int, 1>{}); one(std::integral_constant<int, 2>{});
        one(std::integral_constant<int, 3>{}); one(std::integral_constant<int, 4>{}); one(std::integral_constant<int, 5>{});
        one(std::integral_constant<int, 6>{}); one(std::integral_constant<int, 7>{}); one(std::integral_constant<int, 8>{});
    };
    static_assert(D <= 9, "transfers per step");

    // ---- prologue: the first steps are requested, step 0 (and for the 1.6-bit forms the words of step 1) complete
    if constexpr (C::CODES) {
        for (int b = tid; b < 256; b += 512) {
            unsigned c[5];
            if (p.fx) {
                unsigned v = (unsigned(b) * 243u) >> 8;
                for (int i = 4; i >= 0; --i) { c[i] = v % 3u; v /= 3u; }
            } else {
                unsigned v = b >= 243 ? b - 243 : b;
                for (int i = 0; i < 5; ++i) { c[i] = v % 3u; v /= 3u; }
            }
            table[b] = c[0] | (c[1] << 2) | (c[2] << 4) | (c[3] << 6) | (c[4] << 8);
        }
    }
    if constexpr (C::RAGGED) {
        static_assert(DEP == 4, "slots");
        fetch(0, I0{}); fetch(1, I1{}); fetch(2, I2{}); fetch(3, I3{});
        if constexpr (C::CODES) lds_barrier();            // the table
        put(0, I0{}); fetch(4, I0{});
        put(1, I1{}); fetch(5, I1{});
        lds_barrier();
    } else if constexpr (C::CODES) {
        issue_w(0, 0, Any{});
        if (steps > 1) issue_w(1, 1, Any{});
#pragma unroll
        for (int d = 0; d < C::XD; ++d) {
            issue_x(0, 0, d, Any{});
            if (steps > 1) issue_x(1, 1, d, Any{});
        }
        wait_vm<0>();
        lds_barrier();
        transcode(0, Any{});
        if (steps > 1) transcode(1, Any{});
        lds_barrier();
        if (steps > 2) issue_slots(2, 2, IFirst{}, IEarly{}, Any{});
    } else {
#pragma unroll
        for (int b = 0; b + 1 < ST; ++b)
            if (b < steps) issue_slots(b, b, IFirst{}, ISlots{}, Any{});
        if (steps > ST - 1) {
            wait_vm<(ST - 2) * D>();
            issue_slots(ST - 1, ST - 1, IFirst{}, IEarly{}, Any{});
        } else {
            wait_vm<0>();
        }
        lds_barrier();
    }
    typedef std::integral_constant<int, FM> IFM;
    read_x(I0{}, 0, I0{}, I0{}, IFM{});
    read_w(0, 0, I0{}, Any{});
#pragma unroll
    for (int b = 0; b + 1 < FN; ++b) { decode_codes(b, cw[b][0]); decode_values(b, sc[b][0]); }

    // The barrier of step s: behind it all reads of stage s are done and step s + 1 is in LDS.
    auto turn = [&](int s, auto mode) {
        if constexpr (C::RAGGED) {
            lds_barrier();
        } else if constexpr (C::CODES) {
            // X of step s + 2 may still be on its way, its bytes may not
            if (decltype(mode)::value < 2 || s + 2 < steps) wait_vm<C::XD>(); else wait_vm<0>();
            lds_barrier();
        } else {
            // steps s + 2 .. s + ST - 1 may still be on their way, as far as there are any
            if constexpr (decltype(mode)::value < 2) {
                wait_vm<(ST - 2) * D>();
            } else {
                const int r = steps - 2 - s;
                if (ST > 2 && r >= ST - 2) wait_vm<(ST - 2) * D>();
                else if (ST > 3 && r >= ST - 3) wait_vm<(ST > 3 ? ST - 3 : 0) * D>();
                else if (r >= 1) wait_vm<D>();
                else wait_vm<0>();
            }
            lds_barrier();
        }
    };

    // One step.  A block walks its FN weight fragments; while fragment b is multiplied with the FM fragments of X,
    // the fragment before it is replaced by the next block's (fragment FN - 1 by its own block's), the next block's X is
    // requested, and the transfers' slots come by.
    // mode 0: the step requested next exists and lies inside K (no condition in the loop); 1: it exists; 2: there may
    // be none (the last step reads ahead into whatever the ring holds and drops it).
    // st: s mod ST.  An odd number of blocks swaps the two sets of X fragments from step to step: PAR0 is the set of
    // the step's first block; with SWAP = false they are copied, and every step starts from set 0.
    // The reads of X are kept in front of a half's products; only in the large tiles without the transcoder's registers the compiler may
    // move them (256 x 256 172.5 -> 170.9 us; 128 x 256 of the 1.6-bit form 56.1 -> 63.9).
    constexpr bool kLoose = FM * FN == 32 && !C::CODES;
    // The half of a fragment's products whose end decodes the codes (the values come at the end of the second): the first, unless the halves
    // are so short that the words just asked for would be waited for.  All in the second half against both, 64 x 64 / 32 x 64 tiles: group
    // scales 2.1 / 3.1 % faster (in the first half they had lost 2.1 / 1.5 % to a decode all in the second), 1.6-bit 0.8 / 2.6, 2-bit words
    // 0.5 / 1.0 (means over calls of M = 17 .. 2048, N = 512 .. 16384, K = 512 .. 14336).
    constexpr int kCodes = FM <= 4 ? 1 : 0;
    int st = 0, st_before = ST - 1;
    auto step = [&](int s, auto par0, auto swap, auto mode, auto slot) {
        constexpr int MODE = decltype(mode)::value;
        typedef std::integral_constant<bool, MODE == 0> In;
        const int st_next = st + 1 == ST ? 0 : st + 1;
        auto block = [&](auto kst) {
            constexpr int ks = decltype(kst)::value;
            constexpr int PAR = (decltype(par0)::value + ks) & 1;
            constexpr bool END = ks + 1 == NB;
            typedef std::integral_constant<int, PAR ^ 1> NextPar;
            typedef std::integral_constant<int, (END ? 0 : ks + 1)> Next;
            constexpr int nx = Next::value;
            __builtin_amdgcn_sched_barrier(0);
            const uint32_t own = cw[FN - 1][NCW == 1 ? 0 : ks], own_sc = sc[FN - 1][NS == 1 ? 0 : ks];
            if constexpr (END) turn(s, mode);
            if constexpr (END || NCW == 1) read_w(END ? s + 1 : s, END ? st_next : st, Next{}, In{});
            auto half = [&](auto bt, auto ht) {           // half of fragment b's matrix instructions
                constexpr int b = decltype(bt)::value, h = decltype(ht)::value;
                constexpr int from = h * FM / 2, to = (h + 1) * FM / 2;
                constexpr int i = 2 * b + h;              // a share of the next block's X
                read_x(NextPar{}, END ? st_next : st, Next{}, std::integral_constant<int, i * FM / (2 * FN)>{}, std::integral_constant<int, (i + 1) * FM / (2 * FN)>{});
                if constexpr (!kLoose) __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int a = from; a < to; ++a)
                    acc[a][b] = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, wf[b]), xf[PAR][a], acc[a][b], 0, 0, 0);
                if constexpr (h == kCodes) {
                    if constexpr (b == 0) decode_codes(FN - 1, own);
                    else decode_codes(b - 1, cw[b - 1][NCW == 1 ? 0 : nx]);
                }
                if constexpr (h == 1) {
                    if constexpr (b == 0) decode_values(FN - 1, own_sc);
                    else decode_values(b - 1, sc[b - 1][NS == 1 ? 0 : nx]);
                }
                __builtin_amdgcn_sched_barrier(0);
                if constexpr (!C::RAGGED) {
                    constexpr int slot = (END ? 0 : 2 * FN * (ks + 1)) + 2 * b + h;
                    const int t = END ? s + ST : s + ST - 1;
                    if constexpr (MODE < 2 || !END || C::CODES)
                        if (MODE < 2 || t < steps) issue_slots(t, END ? st : st_before, std::integral_constant<int, slot>{}, std::integral_constant<int, slot + 1>{}, In{});
                }
            };
            auto fragment = [&](auto bt) { half(bt, std::integral_constant<int, 0>{}); half(bt, std::integral_constant<int, 1>{}); };
            fragment(std::integral_constant<int, 0>{});
            fragment(std::integral_constant<int, 1>{});
            if constexpr (FN > 2) {
                fragment(std::integral_constant<int, (FN > 2 ? 2 : 0)>{});
                fragment(std::integral_constant<int, (FN > 2 ? 3 : 0)>{});
            }
            if constexpr (END) {
                if constexpr (C::RAGGED) {                // slot: (s + 2) mod DEP
                    put(s + 2, slot);
                    fetch(s + 2 + DEP, slot);
                } else if constexpr (C::CODES) { if (MODE == 0 || s + 2 < steps) transcode(s + 2, In{}); }
                if constexpr (PAR == 0 && !decltype(swap)::value) {
#pragma unroll
                    for (int a = 0; a < FM; ++a) xf[0][a] = xf[1][a];
                }
            }
        };
        block(std::integral_constant<int, 0>{});
        if constexpr (NB > 1) block(std::integral_constant<int, (NB > 1 ? 1 : 0)>{});
        if constexpr (NB > 2) block(std::integral_constant<int, (NB > 2 ? 2 : 0)>{});
        static_assert(NB <= 3, "blocks per set and step");
        st_before = st;
        st = st_next;
    };
    constexpr bool kSwap = (NB & 1) && !C::CODES;
    typedef std::integral_constant<int, kSwap ? 1 : 0> IOdd;
    typedef std::integral_constant<bool, kSwap> Swap;
    int s = 0;
    if constexpr (C::RAGGED) {
        for (;;) {
            step(s, I0{}, Swap{}, I2{}, I2{});
            if (++s >= steps) break;
            step(s, IOdd{}, Swap{}, I2{}, I3{});
            if (++s >= steps) break;
            step(s, I0{}, Swap{}, I2{}, I0{});
            if (++s >= steps) break;
            step(s, IOdd{}, Swap{}, I2{}, I1{});
            if (++s >= steps) break;
        }
    } else {
        constexpr int ahead = C::CODES ? 3 : ST;
        const int inside_steps = K / KS;
        if constexpr (kSwap) {
            for (; s + 1 + ahead < inside_steps; s += 2) {
                step(s, I0{}, Swap{}, I0{}, I0{});
                step(s + 1, I1{}, Swap{}, I0{}, I0{});
            }
        } else {
            for (; s + ahead < inside_steps; ++s) step(s, I0{}, std::false_type{}, I0{}, I0{});
        }
        if constexpr (!C::CODES)
            for (; s + ahead < steps; ++s) step(s, I0{}, std::false_type{}, I1{}, I0{});
        for (; s < steps; ++s) step(s, I0{}, std::false_type{}, I2{}, I0{});
    }
    };
    if constexpr (kFullSets < WK) {
        if (short_set) run(std::integral_constant<int, NB - 1>{});
        else run(std::integral_constant<int, NB>{});
    } else {
        run(std::integral_constant<int, NB>{});
    }

    // ---- group scales: columns with an infinite scale.  s (c - 1) makes a zero weight under it NaN, and terms of both signs too, where
    // s times the group's sum is an infinity (the streaming kernel, which takes few rows, scales sums).  A thread that was
    // about to store a value that is not finite (`odd`, the sum of 0 times every value, is NaN then) looks through the
    // scales of its columns and, where one is not finite, works its outputs out again from the groups of such scales.
    // (512 x 4096 x 4096, groups of 128: 23.8 us, with five such columns 181, with a row of NaN in X, where nothing is worked
    // out again, 29; looking at the outputs costs nothing that shows.)
    constexpr bool kRedo = C::FMT == kTileGs && !C::RAGGED;
    float odd = 0.f;
    auto look = [&](float value) {
        if constexpr (kRedo) odd = fmaf(value, 0.f, odd);
    };
    auto look2 = [&](uint32_t pair) {
        const f16x2 v = __builtin_bit_cast(f16x2, pair);
        look(v[0]);
        look(v[1]);
    };
    // columns n0 .. n0 + cols - 1, rows m0, m0 + step, ... (count of them)
    auto redo = [&](int n0, int cols, int m0, int step, int count) {
        if constexpr (kRedo) {
            if (odd == odd) return;
#pragma unroll 1
            for (int n = n0; n < n0 + cols && n < p.N; ++n) {
                const uint16_t* const sc = reinterpret_cast<const uint16_t*>(p.scales) + n;
                bool finite = true;
#pragma unroll 16
                for (int g = 0; g <= slast; ++g) finite &= (sc[size_t(g) * size_t(p.N)] & 0x7c00u) != 0x7c00u;
                if (finite) continue;
                const uint32_t* const w = reinterpret_cast<const uint32_t*>(p.W + size_t(n) * size_t(p.row_bytes));
#pragma unroll 1
                for (int i = 0; i < count; ++i) {
                    const int m = m0 + i * step;
                    if (m >= p.M) break;
                    float y = 0.f;
#pragma unroll 1
                    for (int g = 0; g <= slast; ++g) {
                        const float scale = __half2float(p.scales[size_t(g) * size_t(p.N) + n]);
                        if (__builtin_isfinite(scale)) continue;             // finite, and lost in what the others give
                        const int end = (g + 1) * group16 < (K >> 4) ? (g + 1) * group16 : K >> 4;
                        float sum = 0.f;
#pragma unroll 4
                        for (int b = g * group16; b < end; ++b) {
                            const uint32_t word = w[b];
                            const f16x8* const x = reinterpret_cast<const f16x8*>(p.x + size_t(m) * size_t(K) + b * 16);
                            const f16x8 lo = x[0], hi = x[1];
#pragma unroll
                            for (int j = 0; j < 8; ++j) {
                                sum = fmaf(float(int((word >> (2 * j)) & 3u) - 1), float(lo[j]), sum);
                                sum = fmaf(float(int((word >> (2 * j + 16)) & 3u) - 1), float(hi[j]), sum);
                            }
                        }
                        y = fmaf(scale, sum, y);
                    }
                    p.y[size_t(m) * size_t(p.N) + n] = __float2half_rn(y);
                }
            }
        }
    };

    // ---- sums of the sets, all at once: every set leaves its tile in LDS, then all 512 threads add the sets' quads of
    // columns in a fixed order, round and store.  (Halving the sets in turn leaves the last adds and the output to one
    // set's waves: four sets 19.5 against 18.8 us at 512 x 4096 x 4096, eight 11.4 against 10.8 us at 37 x 4099 x 4090; two
    // sets the same either way, 30.0 us at 1024 x 4096 x 4096.)
    if constexpr (C::SHARE) {
        lds_barrier();
        {
            unsigned char* const t = lds + set * (BM * C::SROW) + (wm * 16 * FM + fi) * C::SROW + (wn * 16 * FN + 4 * fg) * 4;
#pragma unroll
            for (int a = 0; a < FM; ++a)
#pragma unroll
                for (int b = 0; b < FN; ++b) *reinterpret_cast<f32x4*>(t + a * (16 * C::SROW) + b * 64) = acc[a][b];
        }
        lds_barrier();
        for (int q = tid; q < BM * BN / 4; q += 512) {
            const int row = q / (BN / 4), c4 = q - row * (BN / 4);
            const unsigned char* const t = lds + row * C::SROW + c4 * 16;
            f32x4 v[WK];
#pragma unroll
            for (int h = 0; h < WK; ++h) v[h] = *reinterpret_cast<const f32x4*>(t + h * (BM * C::SROW));
#pragma unroll
            for (int step = 1; step < WK; step *= 2)
#pragma unroll
                for (int h = 0; h < WK; h += 2 * step) v[h] += v[h + step];
            const int m = m_base + row, n = n_base + c4 * 4;
            if (m >= p.M || n >= p.N) continue;
            __half* const dst = p.y + size_t(m) * p.N + n;
            const f32x4 s = v[0] * gamma;
            look(s[0]); look(s[1]); look(s[2]); look(s[3]);
            if (n + 4 <= p.N) {
                const f16x2 lo = {(_Float16)s[0], (_Float16)s[1]}, hi = {(_Float16)s[2], (_Float16)s[3]};
                *reinterpret_cast<u32x2_any*>(dst) = u32x2{__builtin_bit_cast(uint32_t, lo), __builtin_bit_cast(uint32_t, hi)};
            } else {
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (n + e < p.N) reinterpret_cast<_Float16*>(dst)[e] = (_Float16)s[e];
            }
        }
        redo(n_base + tid % (BN / 4) * 4, 4, m_base + tid / (BN / 4), 2048 / BN, (BM * BN / 4 + 511) / 512);
        return;
    }
    // ---- sums of the sets, halving: set h adds set h + half (fixed order) ------------------------------------
    if constexpr (WK > 1) {
        const int wr = wave % (C::WM * C::WN);
#pragma unroll
        for (int half = WK / 2; half >= 1; half >>= 1) {
            lds_barrier();
            if (set >= half && set < 2 * half) {
                f32x4* const red = reinterpret_cast<f32x4*>(lds) + ((set - half) * (C::WM * C::WN) + wr) * (FM * FN * 64) + lane;
#pragma unroll
                for (int a = 0; a < FM; ++a)
#pragma unroll
                    for (int b = 0; b < FN; ++b) red[(a * FN + b) * 64] = acc[a][b];
            }
            lds_barrier();
            if (set < half) {
                const f32x4* const red = reinterpret_cast<const f32x4*>(lds) + (set * (C::WM * C::WN) + wr) * (FM * FN * 64) + lane;
#pragma unroll
                for (int a = 0; a < FM; ++a)
#pragma unroll
                    for (int b = 0; b < FN; ++b) acc[a][b] += red[(a * FN + b) * 64];
            }
        }
        lds_barrier();
        if (set != 0) return;
    } else {
        lds_barrier();
    }

    // ---- output: y[m][n] = fp16(gamma acc).  A lane holds row m = lane % 16 of a fragment and the columns
    // 4 (lane / 16) + r: each strip of 16 rows is turned through the wave's own piece of LDS.
    constexpr int OROW = FN * 32 + 16;
    unsigned char* const ob = lds + wave * (16 * OROW);
    const int n0 = n_base + wn * 16 * FN;
#pragma unroll
    for (int a = 0; a < FM; ++a) {
        const int m0 = m_base + wm * 16 * FM + 16 * a;
#pragma unroll
        for (int b = 0; b < FN; ++b) {
            const f16x2 lo = {(_Float16)(gamma * acc[a][b][0]), (_Float16)(gamma * acc[a][b][1])};
            const f16x2 hi = {(_Float16)(gamma * acc[a][b][2]), (_Float16)(gamma * acc[a][b][3])};
            *reinterpret_cast<u32x2*>(ob + fi * OROW + b * 32 + fg * 8) =
                u32x2{__builtin_bit_cast(uint32_t, lo), __builtin_bit_cast(uint32_t, hi)};
        }
        // a wave reads what it wrote itself: LDS operations of one wave execute in order
        asm volatile("" : : : "memory");
        if ((p.N & 7) == 0) {
#pragma unroll
            for (int i = 0; i < FN / 2; ++i) {            // 16 rows x 2 FN pieces of 8 columns
                const int q = i * 64 + lane;
                const int row = q / (2 * FN), pc = q - row * (2 * FN);
                const u32x4 v = *reinterpret_cast<const u32x4*>(ob + row * OROW + pc * 16);
                look2(v[0]); look2(v[1]); look2(v[2]); look2(v[3]);
                const int m = m0 + row, n = n0 + pc * 8;
                if (m < p.M && n < p.N) *reinterpret_cast<u32x4*>(p.y + size_t(m) * p.N + n) = v;
            }
        } else {
            // The same pieces at any even address, the last columns one by one.  (All of them one by one: 1714 x 3045 x 512 22.0 us, like this 17.4;
            // in one loop with the aligned form that one loses 1 %.)
#pragma unroll
            for (int i = 0; i < FN / 2; ++i) {
                const int q = i * 64 + lane;
                const int row = q / (2 * FN), pc = q - row * (2 * FN);
                const u32x4 v = *reinterpret_cast<const u32x4*>(ob + row * OROW + pc * 16);
                look2(v[0]); look2(v[1]); look2(v[2]); look2(v[3]);
                const int m = m0 + row, n = n0 + pc * 8;
                if (m >= p.M) continue;
                __half* const dst = p.y + size_t(m) * p.N + n;
                if (n + 8 <= p.N) {
                    *reinterpret_cast<u32x4_any*>(dst) = v;
                } else {
#pragma unroll 1
                    for (int e = 0; n + e < p.N; ++e)
                        reinterpret_cast<uint16_t*>(dst)[e] = *reinterpret_cast<const uint16_t*>(ob + row * OROW + pc * 16 + 2 * e);
                }
            }
        }
        asm volatile("" : : : "memory");
    }
    // a lane's columns are the same in every strip and round
    const int rows0 = m_base + wm * 16 * FM;
    redo(n0 + lane % (2 * FN) * 8, 8, rows0 + lane / (2 * FN), 32 / FN, FM * FN / 2);
}

// ---- host side ----------------------------------------------------------------------------------------------

// The dynamic-LDS limit of an instance on the current device, raised once per device.
template <class C>
hipError_t tile_prepare()
{
    static std::atomic<bool> raised[kMaxDevices];
    const int dev = device_slot();
    if (dev >= 0 && raised[dev].load(std::memory_order_relaxed)) return hipSuccess;
    const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&tile_kernel<C>),
                                             hipFuncAttributeMaxDynamicSharedMemorySize, C::LDS);
    if (e == hipSuccess && dev >= 0) raised[dev].store(true, std::memory_order_relaxed);
    return e;
}

template <class C>
hipError_t tile_launch(TileParams p, hipStream_t s)
{
    const hipError_t e = tile_prepare<C>();
    if (e != hipSuccess) return e;
    p.tiles_n = (p.N + C::BN - 1) / C::BN;
    // one launch, but for outputs of 137 GB and more
    const int64_t rows = tile_row_blocks(p.tiles_n) * C::BM;
    for (int64_t m = 0, M = p.M; m < M; m += rows) {
        p.M = int(M - m < rows ? M - m : rows);
        p.tiles_m = (p.M + C::BM - 1) / C::BM;
        hipLaunchKernelGGL((tile_kernel<C>), dim3(unsigned(p.tiles_m) * unsigned(p.tiles_n)), dim3(kTileThreads), C::LDS, s, p);
        const hipError_t launched = hipGetLastError();
        if (launched != hipSuccess) return launched;
        p.x += int64_t(p.M) * p.K;
        p.y += int64_t(p.M) * p.N;
    }
    return hipSuccess;
}

// What a tile shape costs (us): launch + rounds x (start + steps x time per step), in rounds of `slots` workgroups.  Up to 256 workgroups
// start_few and per step step_few while few CUs are at work, up to step_256 when each has a workgroup (the chip slows down under
// load), beyond that `start` and `step` (CUs may have two); a last round that is not full costs `last` of a full one and more.  Fitted to 24700 calls drawn
// over M = 17 .. 2048, N = 512 .. 16384, K = 512 .. 14336, every instance timed on each: nine in ten lie within 8 %.  The forms for odd K keep an older fit without the load and with the same launch and
// last round for all shapes, nine in ten within 20 %: what they choose among differs by more.
struct TileCost {
    int bm, bn, ks, slots;
    double start_few, start, step_few, step_256, step, last, launch;
};

inline double tile_time(const TileCost& c, int64_t M, int64_t N, int64_t K)
{
    const double tiles = double((M + c.bm - 1) / c.bm) * double((N + c.bn - 1) / c.bn);
    const double steps = double((K + c.ks - 1) / c.ks);
    const double full = double(int64_t(tiles / c.slots));
    const double rest = tiles - full * c.slots;
    double rounds = full;
    if (rest > 0.0) rounds += full == 0.0 ? 1.0 : c.last + (1.0 - c.last) * rest / c.slots;
    if (tiles <= 256.0) return c.launch + c.start_few + steps * (c.step_few + (c.step_256 - c.step_few) * tiles / 256.0);
    return c.launch + rounds * (c.start + steps * c.step);
}

// No shape of `count` takes less on a K, whatever M and N are: spares a caller whose other kernel is faster the whole choice.
inline double tile_at_least(const TileCost* c, int count, int64_t K)
{
    double least = 1e300;
    for (int i = 0; i < count; ++i) {
        const double t = c[i].launch + (c[i].start_few < c[i].start ? c[i].start_few : c[i].start) + double(K) * (c[i].step_few / c[i].ks);
        if (t < least) least = t;
    }
    return least;
}

}  // namespace tl
