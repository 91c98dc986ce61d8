// 4-bit GEMM on the matrix cores: y[M][N] = x[M][K] dequant(W)^T for M >= 2,
// from a few concurrent sequences (one pass over the weights for up to 64
// rows of x) to whole prompts.  Batching sequences is this library's
// extension of the paper's batch-1 decoding; the tiling follows the
// operator-level GEMM tiling the paper's compiler applies (Sec. 2.3).
//
// Numerics.  Codes are dequantized exactly (q - 8), multiplied by the group
// scale and rounded once to fp16 (relative error at most 2^-11 per weight;
// |q - 8| s must stay below the fp16 range, i.e. scales below 8188), and
// v_mfma_f32_16x16x32_f16 accumulates in fp32.
//
// Up to four rows of x (R = 4) a 16-row tile holds each row four times, once
// for each lane group's words and zero elsewhere, so that after the four words
// a tile's sums are those of single groups, in the lane that holds the group's
// scale.  The codes go to the matrix cores as (q - 8) 2^-20, exact subnormals
// (11 operations per word), and the scale is applied in fp32.  (Raw codes,
// with the sums started from -8 times those of x, take 7 operations, but their
// rounding error grows with |x| where q = 8: activations of 1e3 to 6e4 at zero
// weights put results outside the documented bound.  Exact codes cost 4% on
// 28672 x 4096, 14.5 -> 15.15 us, and under 0.5% on the steps.)  Before, M = 2
// ran on the vector kernel (fp32 scales as well); 3B-class step at M = 2 345 ->
// 279 us, 8B-class 787 -> 624, at M = 4 369 -> 288 and 822 -> 642 (against the
// step's earlier kernel).  From M = 5 on two such tiles were 15-24% slower than
// one of 16.
//
// Loads.  Codes, scales and x all go straight into LDS (buffer loads with
// the LDS destination, 16 bytes per lane), so the bytes in flight are bounded
// by the 160 KiB of LDS and not by registers.  A lane's position in LDS is
// fixed (16 bytes after the previous lane's), so the XOR placement that keeps
// the matrix-core reads free of bank conflicts is made by permuting which
// piece of a row each lane fetches.  The buffer range check stands in for
// every edge: pieces outside x, past K or past a wave's share of K are loaded
// from kOutOffset, and zeros arrive in LDS.  The loads are written in assembly
// because the compiler puts a wait for every load in flight before any LDS
// read that follows its own form of them; they have no register result, and
// each wait for them is written out and counts the loads issued since.
//
// Blocks.  A block is NW x KW waves.  Each wave owns 16 TN rows of W against
// 16 TM rows of x; the NW waves of a column group share x through LDS, the KW
// groups split K and are summed through LDS at the end in a fixed order.  The
// dequantization of a weight is shared by 16 TM rows of x: a wave spends
// about 64 VALU cycles per 16 TM matrix cycles on a 16 x 32 piece of W, so
// tall tiles (TM = 8) are matrix-bound and short ones VALU-bound.
//   * CK = 256 (M <= 64, one pass over W): a wave's codes come in whole
//     128-byte lines, one line per row, and a tile's line is refilled as soon
//     as it has been read.
//   * CK = XK = 64 (taller): codes come in 64-deep slots, four of them, three
//     always in flight; W is read again by every block of x rows, from L2.
// K order inside a 16 x 32 multiply: lane 16 c + li takes word t of its own
// group for row li, and x's 8-element pieces are read in the same order.
//
// Measured on one MI355X (cold weights; before = passes of 16 rows below
// M = 65, a tile kernel that wrote dequantized weights to LDS above):
//   16384 x 3072, M = 2048     188-193 us = 1070-1100 TFLOP/s (before 262-269)
//   3B-class layers, M = 512   2.8 ms for 112 linears (before 8.0 ms)
//   3B-class step, M = 48      470 us (before 1270)
//   8B-class step, M = 8       707 us = 6.0 TB/s (before 866-879)
#include <algorithm>
#include <array>
#include <cmath>
#include <cstdlib>
#include <type_traits>

#include "wq_device.h"
#include "wq_internal.h"

namespace wq {
namespace {

using namespace dev;

typedef _Float16 half8 __attribute__((ext_vector_type(8)));
typedef float float4v __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef __attribute__((address_space(3))) uint8_t lds_u8;

constexpr int kStageK = 256;                        // k of one weight stage: a 128-byte line of codes per row
constexpr int kStageGroups = kStageK / kGroup;      // 8
constexpr uint32_t kOutOffset = kPrefillOutOffset;  // past every buffer: reads zeros

template <typename T>
using lds_ptr = __attribute__((address_space(3))) T*;

// LDS byte address -> pointer.
template <typename T>
__device__ __forceinline__ lds_ptr<T> at(uint32_t addr) {
    return reinterpret_cast<lds_ptr<T>>((lds_u8*)(size_t)addr);
}

// ------------------------------------------------ direct-to-LDS loads

__device__ __forceinline__ u32x4 make_desc(const void* p, uint32_t bytes) {
    const uint64_t a = reinterpret_cast<uint64_t>(p);
    u32x4 r;
    r.x = __builtin_amdgcn_readfirstlane((uint32_t)a);
    r.y = __builtin_amdgcn_readfirstlane((uint32_t)(a >> 32) & 0xFFFFu);
    r.z = __builtin_amdgcn_readfirstlane(bytes);
    r.w = kRawBufferFlags;
    return r;
}

template <int CPOL = kCpolDefault>
__device__ __forceinline__ void dma16(u32x4 desc, uint32_t voff, uint32_t soff, uint32_t lds) {
    if constexpr (CPOL == kCpolNonTemporal)
        asm volatile("s_mov_b32 m0, %3\n\ts_nop 0\n\tbuffer_load_dwordx4 %0, %1, %2 offen nt lds" ::"v"(voff), "s"(desc), "s"(soff), "s"(lds) : "memory");
    else
        asm volatile("s_mov_b32 m0, %3\n\ts_nop 0\n\tbuffer_load_dwordx4 %0, %1, %2 offen lds" ::"v"(voff), "s"(desc), "s"(soff), "s"(lds) : "memory");
}

template <int VM>
__device__ __forceinline__ void wait_dma() {
    static_assert(VM >= 0 && VM < 64, "vmcnt");
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(VM) : "memory");
}

// Before a barrier, or before a wave's own loads overwrite LDS that it has read.
template <int NW>
__device__ __forceinline__ void block_sync() {
    if constexpr (NW > 1) asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
    else asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
}

__device__ __forceinline__ void block_barrier() {
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

// Eight codes of one word times the scale, (q - 8) s rounded once to fp16, in
// natural order.  Any scale: a byte's two codes become the exact 1024 + q and
// 1024 + 16 q, then q - 8, then the product.
__device__ __forceinline__ half8 dequant8(uint32_t w, half2v sc) {
    const half2v kmul = {(_Float16)1.0f, (_Float16)0.0625f};
    const half2v kadd = {(_Float16)-1032.0f, (_Float16)-72.0f};
    const uint32_t magic = 0x64646464u, mask = 0xFFF0FF0Fu;
    u32x4 r;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const uint32_t t = __builtin_amdgcn_perm(magic, w, 0x04000400u | (uint32_t)(j * 0x00010001)) & mask;
        r[j] = __builtin_bit_cast(uint32_t, (as_h2(t) * kmul + kadd) * sc);
    }
    return __builtin_bit_cast(half8, r);
}

// The same for scales below 2^-4: a code in bits 4..7 of a half is the
// subnormal q 2^-20, and fma(q 2^-20, s 2^20, -8 s) rounds the exact
// (q - 8) s once, so the result has the same bits; s 2^20 stays finite and
// both factors are exact.  11 operations instead of 16.
constexpr uint32_t kSmallScale = 0x2C00;  // 2^-4
__device__ __forceinline__ half8 dequant8_small(uint32_t w, half2v s20, half2v m8s) {
    const uint32_t od = w & 0xF0F0F0F0u, ev = (w << 4) & 0xF0F0F0F0u;
    u32x4 r;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const uint32_t t = __builtin_amdgcn_perm(od, ev, 0x0C000C00u | (uint32_t)((4 + j) << 16 | j));
        r[j] = __builtin_bit_cast(uint32_t, __builtin_elementwise_fma(as_h2(t), s20, m8s));
    }
    return __builtin_bit_cast(half8, r);
}

// The codes without a scale: (q - 8) 2^-20, exact subnormals.
__device__ __forceinline__ half8 codes8(uint32_t w) {
    const half2v m8 = {(_Float16)-0x1p-17f, (_Float16)-0x1p-17f};
    const uint32_t od = w & 0xF0F0F0F0u, ev = (w << 4) & 0xF0F0F0F0u;
    u32x4 r;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const uint32_t t = __builtin_amdgcn_perm(od, ev, 0x0C000C00u | (uint32_t)((4 + j) << 16 | j));
        r[j] = __builtin_bit_cast(uint32_t, as_h2(t) + m8);
    }
    return __builtin_bit_cast(half8, r);
}

// Rows of 16-byte chunks in LDS: chunk ch of a row lies at position ch ^
// place(row), so that a matrix-core read is free of bank conflicts (64 banks
// of 4 bytes).  A 16-byte-per-lane read is served 16 lanes at a time, lanes
// 0-3, 12-15 and 20-27 together, then 4-11, 16-19 and 28-31, and so on; with
// lane 16 c + li reading row li, each such set is all 16 rows, rows 0-3 and
// 12-15 at one chunk and rows 4-11 at the next lane group's chunk, which
// differs in one of the low bits only.  So the top bit of place() tells the
// two sets of rows apart, the bits below it the rows of a set.  Rows of 256
// bytes or more start on the same bank and take 16 positions; of 128 bytes,
// on two, and take 8 for each pair.  (With row & 7 in its place every read
// of a 128-byte row took 8 extra cycles, of a 256-byte row 4; 12 to 25% of
// the LDS cycles.)
template <int ROW_BYTES>
__device__ __forceinline__ int place(int row) {
    static_assert(ROW_BYTES == 128 || ROW_BYTES >= 256, "chunk rows");
    const int mid = ((row >> 2) ^ (row >> 3)) & 1;  // rows 4-11
    const int high = (row >> 3) & 1;
    return ROW_BYTES == 128 ? mid << 2 | high << 1 | (row >> 1 & 1) : mid << 3 | high << 2 | (row & 3);
}

template <int TM, int TN, int NW, int KW, int XK, int CK, int W, int R>
struct Cfg {
    static constexpr int kWaves = NW * KW;
    static constexpr int kThreads = kWaves * kWave;
    static constexpr int kRowsM = R * TM;                // rows of x (a tile holds 16, or 4 in 4 places)
    static constexpr int kRowsN = 16 * TN * NW;
    static constexpr int QS = kStageK / XK;              // x stages per weight stage
    static constexpr int XBytes = 16 * TM * XK * 2;      // one x buffer
    static constexpr int XLoads = XBytes / 1024;         // x loads of a stage
    static constexpr int NX = (XLoads + NW - 1) / NW;    // per wave (the surplus repeats other loads)
    static constexpr int CSlots = kStageK / CK;
    static constexpr int CSlotBytes = 16 * TN * CK / 2;  // codes of one slot of a wave
    static constexpr int NC = CSlotBytes / 1024;         // loads per slot
    static constexpr int SRow = 16 * W;                  // bytes of scales per row and window
    static constexpr int SBytes = (16 * TN * SRow + 1023) / 1024 * 1024;  // one window of a wave
    static constexpr int NS = SBytes / 1024;             // scale loads per window
    static constexpr int WaveBytes = CSlots * CSlotBytes + 2 * SBytes;
    static constexpr int RunBytes = KW * 2 * XBytes + kWaves * WaveBytes;
    static constexpr int RedBytes = KW > 1 ? kWaves * TM * TN * 1024 : 0;  // partial tiles, afterwards
    static constexpr int LdsBytes = RunBytes > RedBytes ? RunBytes : RedBytes;
    static_assert(R == 16 || (R == 4 && XK == 128 && CK == kStageK), "x rows per tile");
    static_assert(XBytes % 1024 == 0, "x loads are whole");
    static_assert(W == 2 || W == 4, "the next window is complete before the last stage of a window");
    static_assert(CSlotBytes % 1024 == 0 && SBytes % 1024 == 0, "slot loads are whole");
    static_assert((CK == kStageK && XK == 128) || (CK == 64 && XK == 64), "code slots");
};

struct GemmArgs {
    const void* packed;
    const uint16_t* scales;
    const uint16_t* x;
    uint16_t* y;
    int64_t n;
    int32_t ng;
    int32_t m;
};

// One block: rows [row0, row0 + kRowsN) of W, rows [m0, m0 + kRowsM) of x.
//
// `turn` (one pass over W) is the scale window at which the block starts its
// walk along K, round to the one before.  A block's rows are read one line at
// the same column at a time; where K is a multiple of 8192 (code rows 4 KiB
// apart) those lines share a few memory channels, and blocks that all start
// at column 0 share the same few.  Measured at M = 8: 131072 x 8192 126 ->
// 108 us; at K = 3072 and 14336, where rows spread by themselves, turning
// gained nothing (0 to -2%).
template <int TM, int TN, int NW, int KW, int XK, int CK, int W, int R>
__device__ __forceinline__ void gemm_block(const GemmArgs& a, int64_t row0, int64_t m0, int turn, lds_u8* lds) {
    using C = Cfg<TM, TN, NW, KW, XK, CK, W, R>;
    constexpr int QS = C::QS, NX = C::NX, NC = C::NC, NS = C::NS;
    constexpr int WPL = XK / 32;  // words per lane of an x stage
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int wn = wave % NW, wk = wave / NW;
    const int li = lane & 15, c = lane >> 4;
    const int ng = a.ng;
    const int nst = (ng + kStageGroups - 1) / kStageGroups;
    const int sb = wk * nst / KW, se = (wk + 1) * nst / KW;
    const int iters = (nst + KW - 1) / KW;  // of the longest range: the barriers are shared
    const int mrows = (int)min((int64_t)C::kRowsM, a.m - m0);
    // Only whole windows can turn, and only rows whose scales start on a dword.
    const int range = se - sb;
    const bool turns = CK == kStageK && range > 0 && range % W == 0 && ng % 256 == 0 &&
                       !(reinterpret_cast<uintptr_t>(a.scales) & 2);
    const int start = sb + (turns ? turn * W % range : 0);
    const int wrap = turns ? range : 0;  // what a stage past the end goes back by
    const uint32_t xrow_bytes = (uint32_t)ng * 64u;
    const u32x4 dw = make_desc(a.packed, (uint32_t)(a.n * ng * 16));
    // Scales are read in whole dwords: the descriptor starts at the dword
    // that holds the first scale and ends with the one that holds the last.
    const uint32_t spar = (uint32_t)(reinterpret_cast<uintptr_t>(a.scales) >> 1) & 1u;
    const u32x4 ds = make_desc(a.scales - spar, (uint32_t)(((a.n * ng + spar) * 2 + 3) & ~(int64_t)3));
    const u32x4 dx = make_desc(a.x + m0 * (int64_t)ng * kGroup, (uint32_t)mrows * xrow_bytes);

    const uint32_t lds0 = (uint32_t)(size_t)lds;
    const uint32_t xlds = lds0 + wk * 2 * C::XBytes;                                 // two buffers
    const uint32_t clds = lds0 + KW * 2 * C::XBytes + wave * C::WaveBytes;           // code slots
    const uint32_t slds = clds + C::CSlots * C::CSlotBytes;                          // two scale slots
    const int64_t wrow = row0 + wn * 16 * TN;                                        // this wave's first row

    // ---- loads.  Lane offsets within a load; wave-uniform parts are scalar.
    // Past the wave's range the buffer is empty: zeros arrive.
    auto in_range = [&](u32x4 d, bool ok) {
        d.z = ok ? d.z : 0u;
        return d;
    };
    // x: one load covers XR rows of an x stage, 16-byte chunks XOR-placed by row.
    constexpr int XCH = XK / 8;       // chunks per row
    constexpr int XR = 64 / XCH;      // rows per load
    auto issue_x = [&](int st, bool ok, int q, int buf) {
        const int k0 = st * kStageK + q * XK;
#pragma unroll
        for (int i = 0; i < NX; ++i) {
            const int ld = (wn * NX + i) % C::XLoads;       // load index in the stage
            const int r = lane / XCH, ph = lane % XCH;      // row within the load, LDS chunk
            const int src = ph ^ place<XK * 2>(ld * XR + r);
            // R = 4: row r of the load is x row r, kept for one lane group only.
            const bool kept = R == 16 || src / 4 == ld % 4;
            const uint32_t voff =
                kept && k0 + 8 * src < ng * kGroup ? (uint32_t)r * xrow_bytes + (uint32_t)src * 16u : kOutOffset;
            const uint32_t soff = (uint32_t)(R == 16 ? ld * XR : ld / 4 * 4) * xrow_bytes + (uint32_t)k0 * 2u;
            dma16(in_range(dx, ok), voff, __builtin_amdgcn_readfirstlane(soff), xlds + buf * C::XBytes + ld * 1024);
        }
    };
    // Codes of slot q (CK deep) of stage st, load i: 1024 / (CK / 2) rows.
    constexpr int CCH = CK / 32;      // 16-byte chunks (groups) per row and slot
    constexpr int CR = 64 / CCH;      // rows per load
    auto issue_codes = [&](int st, bool ok, int q, int i) {
        const int r = lane / CCH, ph = lane % CCH;
        const int src = CK == kStageK ? ph ^ place<128>(i * CR + r) : ph;
        const uint32_t voff = ((uint32_t)r * (uint32_t)ng + (uint32_t)src) * 16u;
        const uint32_t soff = (uint32_t)((wrow + i * CR) * ng + st * kStageGroups + q * CCH) * 16u;
        dma16<CK == kStageK ? kCpolNonTemporal : kCpolDefault>(in_range(dw, ok), voff, __builtin_amdgcn_readfirstlane(soff), clds + q * C::CSlotBytes + i * 1024);
    };
    // Scale window `w` of the walk (W stages from `st`): 16-byte pieces of each row,
    // from the dword holding the row's first scale of the window.  Where that
    // scale is the dword's upper half (`odd`), the row's scales sit one place
    // later: its last one is the first of the next window, which has long
    // been loaded when it is read.
    constexpr int SP = W;             // 16-byte pieces per row
    constexpr int SR = 64 / SP;       // rows per load
    // Piece pc of a row lies at position pc ^ splace(row): 16 rows of 16 W
    // bytes cover the banks once per piece.
    auto splace = [](int row) { return W == 4 ? (row >> 2) & 3 : (row >> 3) & 1; };
    auto issue_scales = [&](int w, int st) {
        const int g0 = st * kStageGroups;
        const int r = lane / SP, pc = lane % SP ^ splace(r);
        const int left = w * W < range ? se - st : min(se - st, 0);  // stages of the range from the window on
        const bool ok = left >= pc && (16 * TN % SR == 0 || r < 16 * TN);
#pragma unroll
        for (int i = 0; i < NS; ++i) {
            const uint32_t e = spar + (uint32_t)((wrow + i * SR + r) * ng + g0 + pc * 8);
            dma16(ds, ok ? (e & ~1u) * 2u : kOutOffset, 0u, slds + (w & 1) * C::SBytes + i * 1024);
        }
    };
    const uint32_t odd = (spar + (uint32_t)((wrow + li) * ng)) & 1u;  // 16 ng is even: the same for every tile
    const bool shifted = ((spar | (uint32_t)ng) & 1u) != 0;           // some row is odd

    float4v acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) acc[i][j] = float4v{0.0f, 0.0f, 0.0f, 0.0f};

    // Operand A, of x buffer `buf`: word t, or all of them.
    half8 fa[TM][WPL];
    auto load_word = [&](int buf, int t) {
        const int ch = WPL * c + t;
        const uint32_t off = xlds + buf * C::XBytes + (uint32_t)li * (XK * 2) + (uint32_t)((ch ^ place<XK * 2>(li)) * 16);
#pragma unroll
        for (int i = 0; i < TM; ++i) fa[i][t] = *at<const half8>(off + i * 16 * XK * 2);
    };
    auto load_a = [&](int buf) {
#pragma unroll
        for (int t = 0; t < WPL; ++t) load_word(buf, t);
    };
    // The lane's scale of group g (0..7) of a stage, `it` stages into the range,
    // of row li; the other tiles' lie 16 rows on.
    auto scale_addr = [&](int g, int it) {
        const uint32_t pos = (uint32_t)g + odd;
        const uint32_t piece = (uint32_t)it + pos / 8;
        return slds + ((piece / W) & 1u) * C::SBytes + (uint32_t)li * C::SRow + (piece % W ^ (uint32_t)splace(li)) * 16 +
               (pos % 8) * 2u;
    };
    auto read_scale = [&](uint32_t addr, int tt) {
        return (uint32_t)*at<const uint16_t>(addr + tt * 16 * C::SRow);
    };
    // Some of the stage's groups lie past the row or past the range: their
    // scales count as zero.
    auto cut = [&](int it, int st) { return it >= range || (st + 1) * kStageGroups > ng; };
    auto keep_group = [&](int g, int it, int st) {
        return it < range && st * kStageGroups + g < ng ? 0xFFFFu : 0u;
    };
    // The stage after `st`, and the one W on.
    auto after = [&](int st, int by) { return st + by >= se ? st + by - wrap : st + by; };
    // What a lane's scales are used as: themselves, and times 2^20 and -8 for
    // the short dequantization (two at once, in the halves).
    struct Scales {
        half2v s, s20, m8;
    };
    auto scales_of = [&](uint32_t pair) {
        const half2v k1024 = {(_Float16)1024.0f, (_Float16)1024.0f};
        const half2v km8 = {(_Float16)-8.0f, (_Float16)-8.0f};
        const half2v s = as_h2(pair);
        return Scales{s, s * k1024 * k1024, s * km8};
    };
    // Multiplies of tile tt with the x in `fa`; the scale is half h of its
    // pair.
    auto multiply = [&](auto small, const uint32_t* wd, const Scales& sc, int h, int tt) {
        auto both = [&](half2v v) { return half2v{v[h], v[h]}; };
        constexpr bool fast = decltype(small)::value;
        if constexpr (R == 4) {
            float4v d[TM];
#pragma unroll
            for (int i = 0; i < TM; ++i) d[i] = float4v{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
            for (int t = 0; t < WPL; ++t) {
                const half8 fb = codes8(wd[t]);
#pragma unroll
                for (int i = 0; i < TM; ++i)
                    d[i] = __builtin_amdgcn_mfma_f32_16x16x32_f16(fa[i][t], fb, d[i], 0, 0, 0);
            }
            const float s = (float)sc.s[h] * 0x1p20f;
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int v = 0; v < 4; ++v) acc[i][tt][v] = __builtin_fmaf(d[i][v], s, acc[i][tt][v]);
            return;
        }
#pragma unroll
        for (int t = 0; t < WPL; ++t) {
            half8 fb;
            if constexpr (fast) fb = dequant8_small(wd[t], both(sc.s20), both(sc.m8));
            else fb = dequant8(wd[t], both(sc.s));
#pragma unroll
            for (int i = 0; i < TM; ++i)
                acc[i][tt] = __builtin_amdgcn_mfma_f32_16x16x32_f16(fa[i][t], fb, acc[i][tt], 0, 0, 0);
        }
    };
    // Whether every lane's scales allow the short dequantization.
    auto all_small = [&](uint32_t mx) { return __builtin_amdgcn_ballot_w64(max(mx & 0xFFFFu, mx >> 16) >= kSmallScale) == 0; };
    using Small = std::integral_constant<bool, true>;
    using Any = std::integral_constant<bool, false>;

    issue_x(start, range > 0, 0, 0);
    issue_scales(0, start);
#pragma unroll
    for (int q = 0; q < C::CSlots; ++q)
#pragma unroll
        for (int i = 0; i < NC; ++i) issue_codes(start, range > 0, q, i);

    if constexpr (CK == kStageK) {
        // One slot of whole lines.  A tile's codes (both 128-deep halves) go
        // to registers one tile ahead of their multiplies, and the tile's two
        // loads for the next stage are issued as soon as they have been read.
        struct Tile {
            uint32_t w[2][4];
        };
        uint32_t pair[TN];  // scales of both halves
        auto read_scales = [&](int it, int st) {
            const uint32_t a0 = scale_addr(c, it);
            const uint32_t a1 = shifted ? scale_addr(4 + c, it) : a0 + 8;
#pragma unroll
            for (int tt = 0; tt < TN; ++tt) pair[tt] = read_scale(a0, tt) | read_scale(a1, tt) << 16;
            if (cut(it, st)) {
                const uint32_t keep = keep_group(c, it, st) | keep_group(4 + c, it, st) << 16;
#pragma unroll
                for (int tt = 0; tt < TN; ++tt) pair[tt] &= keep;
            }
            typedef uint16_t u16x2 __attribute__((ext_vector_type(2)));
            u16x2 mx = {0, 0};
#pragma unroll
            for (int tt = 0; tt < TN; ++tt)
                mx = __builtin_elementwise_max(mx, __builtin_bit_cast(u16x2, pair[tt] & 0x7FFF7FFFu));
            return __builtin_bit_cast(uint32_t, mx);
        };
        auto read_tile = [&](Tile& T, int tt) {
            const uint32_t row = 16 * tt + li;
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const int g = 4 * h + c;
                const uint32_t ca = clds + row * 128 + (uint32_t)((g ^ place<128>(li)) * 16);
                const u32x4 v = *at<const u32x4>(ca);
                T.w[h][0] = v.x; T.w[h][1] = v.y; T.w[h][2] = v.z; T.w[h][3] = v.w;
            }
            asm volatile("" ::: "memory");
        };
        // The reads of T have completed (the last one issued has).
        auto tile_read_done = [&](Tile& T) { asm volatile("" : "+v"(T.w[0][3]), "+v"(T.w[1][3])::"memory"); };
        auto refill = [&](int st, bool ok, int tt) {
            issue_codes(st, ok, 0, 2 * tt);
            issue_codes(st, ok, 0, 2 * tt + 1);
        };
        // Two x stages: the second half of every tile waits in registers.
        // The first half of the tiles is refilled in the first x stage,
        // the others in the second.
        constexpr int TH = (TN + 1) / 2;
        for (int it = 0, st = start; it < iters; ++it, st = after(st, 1)) {
            const int next = after(st, 1);
            const bool more = it + 1 < range;
            Tile T[TN];
            if (it == 0) wait_dma<2 * TN>();
            else wait_dma<2 * (TN - TH)>();
            block_sync<NW>();
            if (it % W == 0) issue_scales(it / W + 1, after(st, W));
            issue_x(st, it < range, 1, 1);
            load_a(0);
            const uint32_t mx = read_scales(it, st);
            const bool small = R == 16 && all_small(mx);  // R = 4 has one form
            auto first = [&](auto sm) {
                // Newer than tile 0's codes: at most every other tile's and x.
                if (it == 0) wait_dma<2 * (TN - 1) + NX>();
                read_tile(T[0], 0);
#pragma unroll
                for (int tt = 0; tt < TN; ++tt) {
                    if (tt + 1 < TN) {
                        if (it == 0 || tt + 1 >= TH) {
                            // Old codes after tile tt + 1, x, refills so far.
                            constexpr int base = NX;
                            const int n = 2 * (TN - 2 - tt) + base + 2 * (tt < TH ? tt : TH);
                            if (n >= base + 6) wait_dma<base + 6>();
                            else if (n >= base + 4) wait_dma<base + 4>();
                            else if (n >= base + 2) wait_dma<base + 2>();
                            else wait_dma<base>();
                        }
                        read_tile(T[tt + 1], tt + 1);
                    }
                    tile_read_done(T[tt]);
                    if (tt < TH) refill(next, more, tt);
                    multiply(sm, T[tt].w[0], scales_of(pair[tt]), 0, tt);
                }
            };
            auto second = [&](auto sm) {
#pragma unroll
                for (int tt = 0; tt < TN; ++tt) {
                    if (tt >= TH) refill(next, more, tt);
                    multiply(sm, T[tt].w[1], scales_of(pair[tt]), 1, tt);
                }
            };
            if (small) first(Small{});
            else first(Any{});
            wait_dma<2 * TH>();  // x stage 1
            block_sync<NW>();
            issue_x(next, more, 0, 0);
            load_a(1);
            if (small) second(Small{});
            else second(Any{});
        }
    } else {
        // One slot per x stage, each refilled for the next weight stage once
        // used: QS - 1 slots are always in flight.
        for (int it = 0, st = start; it < iters; ++it, st = after(st, 1)) {
            const int next = after(st, 1);
            const bool more = it + 1 < range;
#pragma unroll
            for (int q = 0; q < QS; ++q) {
                // The x stage's loads, issued before the previous x stage's
                // refills (NC) and, into a new weight stage, its scales.
                if (it == 0 && q == 0) wait_dma<0>();
                else wait_dma<NC>();
                block_sync<NW>();
                const int buf = q & 1;
                if (q == QS - 1) {
                    issue_x(next, more, 0, buf ^ 1);
                } else {
                    if (q == 0 && it % W == 0) issue_scales(it / W + 1, after(st, W));
                    issue_x(st, it < range, q + 1, buf ^ 1);
                }
                // Words of the lane: WPL from word w0 of the stage's row.
                const int w0 = q * (XK / 8) + WPL * c;
                const uint32_t sa = scale_addr(w0 / 4, it);
                const uint32_t keep = cut(it, st) ? keep_group(w0 / 4, it, st) : 0xFFFFu;
                uint32_t wd[TN][WPL];
                half2v sc[TN];
#pragma unroll
                for (int tt = 0; tt < TN; ++tt) {
                    const uint32_t ca = clds + q * C::CSlotBytes + (uint32_t)(16 * tt + li) * (CK / 2) + (uint32_t)(WPL * c) * 4;
                    const u32x2 v = *at<const u32x2>(ca);
                    wd[tt][0] = v.x; wd[tt][1] = v.y;
                    const uint32_t sv = read_scale(sa, tt) & keep;
                    sc[tt] = as_h2(sv | (sv << 16));
                }
                load_word(buf, 0);
#pragma unroll
                for (int t = 0; t < WPL; ++t) {
                    if (t + 1 < WPL) load_word(buf, t + 1);
#pragma unroll
                    for (int tt = 0; tt < TN; ++tt) {
                        const half8 fb = dequant8(wd[tt][t], sc[tt]);
#pragma unroll
                        for (int i = 0; i < TM; ++i)
                            acc[i][tt] = __builtin_amdgcn_mfma_f32_16x16x32_f16(fa[i][t], fb, acc[i][tt], 0, 0, 0);
                    }
                }
                asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
#pragma unroll
                for (int i = 0; i < NC; ++i) issue_codes(next, more, q, i);
            }
        }
    }
    wait_dma<0>();

    // ---- results: D[4 c + v][li] of tile (i, j) is x row 16 i + 4 c + v, W row 16 j + li.
    // R = 4: it is x row 4 i + v over the groups of lane group c.
    if constexpr (R == 4) {
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j)
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    float t = acc[i][j][v];
                    t += __shfl_xor(t, 16);
                    t += __shfl_xor(t, 32);
                    acc[i][j][v] = t;
                }
    }
    auto out_row = [&](int i, int v) { return R == 16 ? 16 * i + 4 * c + v : 4 * i + v; };
    auto mine = [&](int v) { return R == 16 || v == c; };
    typedef __attribute__((address_space(3))) float lds_f32;
    if constexpr (KW > 1) {
        block_barrier();
        lds_f32* red = (lds_f32*)lds;
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j)
#pragma unroll
                for (int v = 0; v < 4; ++v) red[((wave * TM + i) * TN + j) * 256 + v * 64 + lane] = acc[i][j][v];
        block_barrier();
        // Tile (i, j) of column group wn is summed, in order, by the wave of
        // K part (i TN + j) % KW.
#pragma unroll
        for (int i = 0; i < TM; ++i) {
#pragma unroll
            for (int j = 0; j < TN; ++j) {
                if ((i * TN + j) % KW != wk) continue;
                const int64_t col = wrow + 16 * j + li;
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    float t = 0.0f;
#pragma unroll
                    for (int w = 0; w < KW; ++w) t += red[(((w * NW + wn) * TM + i) * TN + j) * 256 + v * 64 + lane];
                    const int mr = out_row(i, v);
                    if (mine(v) && mr < mrows && col < a.n) gbl(a.y)[(m0 + mr) * a.n + col] = __half_as_ushort(__float2half_rn(t));
                }
            }
        }
    } else {
#pragma unroll
        for (int i = 0; i < TM; ++i) {
#pragma unroll
            for (int j = 0; j < TN; ++j) {
                const int64_t col = wrow + 16 * j + li;
                if (col >= a.n) continue;
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const int mr = out_row(i, v);
                    if (mine(v) && mr < mrows) gbl(a.y)[(m0 + mr) * a.n + col] = __half_as_ushort(__float2half_rn(acc[i][j][v]));
                }
            }
        }
    }
}

// Block b of a linear's blocks_n x blocks_m tiles.  Four x tiles by all
// weight tiles form a patch, walked with the x tile fastest, so that the
// blocks running at one time share both operands in L2.
__device__ __forceinline__ void tile_of(int b, int blocks_n, int blocks_m, int& bn, int& bm) {
    constexpr int kPatch = 4;
    const int g = b / (kPatch * blocks_n);
    const int gm = min(kPatch, blocks_m - g * kPatch);
    const int r = b - g * kPatch * blocks_n;
    bm = g * kPatch + r % gm;
    bn = r / gm;
}

// Workgroups are dealt to the 8 XCDs in turn; give each XCD (and its L2) a
// contiguous run of tiles.  Only the order changes.  Measured at M = 2048:
// 128256 x 3072 1.59 -> 1.48 ms, 16384 x 3072 217 -> 214 us; at M <= 64,
// where every weight is read once, there is nothing to share.
__device__ __forceinline__ int xcd_run(int b, int blocks) {
    constexpr int kXcds = 8;
    const int x = b % kXcds;
    return x * (blocks / kXcds) + min(x, blocks % kXcds) + b / kXcds;
}

// One linear.
template <typename C, int TM, int TN, int NW, int KW, int XK, int CK, int W, int R>
__device__ __forceinline__ void run_tile(const GemmArgs& a, int b, int blocks_m, lds_u8* lds) {
    const int blocks_n = (int)((a.n + C::kRowsN - 1) / C::kRowsN);
    int bn = b, bm = 0;
    if (blocks_m > 1) tile_of(b, blocks_n, blocks_m, bn, bm);
    gemm_block<TM, TN, NW, KW, XK, CK, W, R>(a, (int64_t)bn * C::kRowsN, (int64_t)bm * C::kRowsM, blocks_m > 1 ? 0 : bn,
                                          lds);
}

template <int TM, int TN, int NW, int KW, int XK, int CK, int W, int R, int OCC>
__global__ __launch_bounds__(NW* KW* kWave, OCC) void gemm_kernel(const GemmArgs a, int blocks_m) {
    using C = Cfg<TM, TN, NW, KW, XK, CK, W, R>;
    __shared__ __align__(16) uint8_t s_lds[C::LdsBytes];
    const int b = blocks_m > 1 ? xcd_run(blockIdx.x, gridDim.x) : (int)blockIdx.x;
    run_tile<C, TM, TN, NW, KW, XK, CK, W, R>(a, b, blocks_m, (lds_u8*)s_lds);
}

// Index of a block's rows of W among the sizes that plans hold.
constexpr int plan_size(int rows_n) {
    int size = 0;
    while ((16 << size) < rows_n) ++size;
    return size;
}

// Independent linears of one launch, found by binary search over their first
// blocks: from a plan in device memory (M <= 64) ...
template <int TM, int TN, int NW, int KW, int XK, int CK, int W, int R, int OCC>
__global__ __launch_bounds__(NW* KW* kWave, OCC) void gemm_plan_kernel(const GemmPlanEntry* __restrict__ entries, int count, int m) {
    using C = Cfg<TM, TN, NW, KW, XK, CK, W, R>;
    constexpr int size = plan_size(C::kRowsN);
    __shared__ __align__(16) uint8_t s_lds[C::LdsBytes];
    const int64_t b = blockIdx.x;
    const int blocks_m = (m + C::kRowsM - 1) / C::kRowsM;
    int lo = 0, hi = count - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) / 2;
        if ((int64_t)entries[mid].first[size] * blocks_m <= b) lo = mid;
        else hi = mid - 1;
    }
    const GemmPlanEntry& e = entries[lo];
    const GemmArgs a{e.packed, e.scales, e.x, e.y, e.n, e.ng, m};
    run_tile<C, TM, TN, NW, KW, XK, CK, W, R>(a, (int)(b - (int64_t)e.first[size] * blocks_m), blocks_m, (lds_u8*)s_lds);
}

// ... or from the launch's own arguments (prompts: no plan to keep).
struct GemmEntry {
    const void* packed;
    const uint16_t* scales;
    const uint16_t* x;
    uint16_t* y;
    int64_t n;
    int32_t ng;
    int32_t first_block;
};
constexpr int kListEntries = 64;
struct GemmList {
    int32_t count;
    int32_t m;
    GemmEntry e[kListEntries];
};
static_assert(sizeof(GemmList) <= 3600, "launch arguments stay below 4 KiB");

template <int TM, int TN, int NW, int KW, int XK, int CK, int W, int R, int OCC>
__global__ __launch_bounds__(NW* KW* kWave, OCC) void gemm_list_kernel(const GemmList l) {
    using C = Cfg<TM, TN, NW, KW, XK, CK, W, R>;
    __shared__ __align__(16) uint8_t s_lds[C::LdsBytes];
    const int b = blockIdx.x;
    int lo = 0, hi = l.count - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) / 2;
        if (l.e[mid].first_block <= b) lo = mid;
        else hi = mid - 1;
    }
    const GemmArgs a{l.e[lo].packed, l.e[lo].scales, l.e[lo].x, l.e[lo].y, l.e[lo].n, l.e[lo].ng, l.m};
    // First blocks are multiples of 8: every linear is dealt to all XCDs.
    const int blocks_m = (l.m + C::kRowsM - 1) / C::kRowsM;
    const int blocks = (int)((a.n + C::kRowsN - 1) / C::kRowsN) * blocks_m;
    const int r = b - l.e[lo].first_block;
    if (r >= blocks) return;
    run_tile<C, TM, TN, NW, KW, XK, CK, W, R>(a, xcd_run(r, blocks), blocks_m, (lds_u8*)s_lds);
}

// ------------------------------------------------------------- dispatch

// The compiled block shapes: TM, TN, NW, KW, XK, CK, W, R and blocks per CU
// that the registers are compiled for.  16 rows of W with K over eight waves
// are for few rows of deep K: 4096 x 14336 at M = 8 17.2 -> 12.1 us, 3072 x
// 8192 10.8 -> 8.1.
#define WQ_GEMM_CONFIGS(X)        \
    X(1, 2, 4, 1, 128, 256, 4, 16, 4) \
    X(1, 2, 4, 2, 128, 256, 2, 16, 2) \
    X(1, 2, 2, 4, 128, 256, 2, 16, 2) \
    X(1, 2, 1, 8, 128, 256, 2, 16, 1) \
    X(1, 1, 1, 4, 128, 256, 2, 16, 2) \
    X(2, 2, 8, 1, 128, 256, 4, 16, 2) \
    X(2, 4, 2, 2, 128, 256, 2, 16, 2) \
    X(2, 2, 2, 2, 128, 256, 2, 16, 2) \
    X(2, 4, 1, 4, 128, 256, 2, 16, 1) \
    X(2, 2, 1, 4, 64, 64, 2, 16, 2)   \
    X(2, 1, 1, 4, 128, 256, 2, 16, 1) \
    X(3, 4, 4, 1, 128, 256, 2, 16, 2) \
    X(3, 2, 2, 2, 128, 256, 2, 16, 2) \
    X(3, 2, 1, 4, 128, 256, 2, 16, 1) \
    X(3, 1, 1, 4, 128, 256, 2, 16, 1) \
    X(4, 2, 8, 1, 128, 256, 2, 16, 2) \
    X(4, 2, 4, 1, 64, 64, 2, 16, 4)   \
    X(4, 4, 2, 2, 128, 256, 2, 16, 1) \
    X(4, 2, 2, 2, 64, 64, 2, 16, 2)   \
    X(4, 2, 1, 4, 64, 64, 2, 16, 1)   \
    X(6, 4, 4, 1, 64, 64, 2, 16, 2)   \
    X(8, 4, 4, 1, 64, 64, 2, 16, 2)   \
    X(8, 4, 8, 1, 64, 64, 2, 16, 1)   \
    X(8, 2, 2, 2, 64, 64, 2, 16, 1)   \
    X(1, 2, 4, 1, 128, 256, 4, 4, 4) \
    X(1, 2, 4, 2, 128, 256, 2, 4, 2) \
    X(1, 2, 2, 4, 128, 256, 2, 4, 2) \
    X(1, 2, 1, 8, 128, 256, 2, 4, 1) \
    X(1, 1, 1, 4, 128, 256, 2, 4, 2) \
    X(1, 1, 1, 8, 128, 256, 2, 4, 1) \
    X(1, 1, 1, 8, 128, 256, 2, 16, 1)

struct Config {
    int tm, tn, nw, kw, xk, ck, r;
    int occ;  // blocks per CU
    int rows_m, rows_n;
    hipError_t (*one)(const GemmArgs&, int64_t, int, hipStream_t);
    hipError_t (*plan)(const GemmPlanEntry*, int, int64_t, int, hipStream_t);
    hipError_t (*list)(const GemmList&, int64_t, hipStream_t);
};

template <int TM, int TN, int NW, int KW, int XK, int CK, int W, int R, int OCC>
hipError_t launch_one(const GemmArgs& a, int64_t blocks, int blocks_m, hipStream_t stream) {
    hipLaunchKernelGGL((gemm_kernel<TM, TN, NW, KW, XK, CK, W, R, OCC>), dim3((unsigned)blocks), dim3(NW * KW * kWave), 0, stream, a, blocks_m);
    return hipGetLastError();
}
template <int TM, int TN, int NW, int KW, int XK, int CK, int W, int R, int OCC>
hipError_t launch_plan(const GemmPlanEntry* entries, int count, int64_t blocks, int m, hipStream_t stream) {
    if constexpr (TM <= 4) {
        using C = Cfg<TM, TN, NW, KW, XK, CK, W, R>;
        static_assert(plan_size(C::kRowsN) < kGemmPlanSizes && C::kRowsN == 16 << plan_size(C::kRowsN), "plans hold these sizes");
        hipLaunchKernelGGL((gemm_plan_kernel<TM, TN, NW, KW, XK, CK, W, R, OCC>), dim3((unsigned)blocks), dim3(NW * KW * kWave), 0, stream, entries, count, m);
        return hipGetLastError();
    } else {
        return hipErrorInvalidValue;  // plans are made for M <= 64 only
    }
}
template <int TM, int TN, int NW, int KW, int XK, int CK, int W, int R, int OCC>
hipError_t launch_list(const GemmList& l, int64_t blocks, hipStream_t stream) {
    if constexpr (TM >= 2 && R == 16) {
        hipLaunchKernelGGL((gemm_list_kernel<TM, TN, NW, KW, XK, CK, W, R, OCC>), dim3((unsigned)blocks), dim3(NW * KW * kWave), 0, stream, l);
        return hipGetLastError();
    } else {
        return hipErrorInvalidValue;  // lists are made for M > 64 only
    }
}

template <int TM, int TN, int NW, int KW, int XK, int CK, int W, int R, int OCC>
constexpr Config config_of() {
    using C = Cfg<TM, TN, NW, KW, XK, CK, W, R>;
    static_assert(C::LdsBytes <= 160 * 1024, "a block fits one CU");
    const int by_lds = 160 * 1024 / C::LdsBytes;
    return Config{TM, TN, NW, KW, XK, CK, R, by_lds < OCC ? by_lds : OCC, C::kRowsM, C::kRowsN,
                  launch_one<TM, TN, NW, KW, XK, CK, W, R, OCC>, launch_plan<TM, TN, NW, KW, XK, CK, W, R, OCC>,
                  launch_list<TM, TN, NW, KW, XK, CK, W, R, OCC>};
}

#define WQ_GEMM_ROW(...) config_of<__VA_ARGS__>(),
const Config kConfigs[] = {WQ_GEMM_CONFIGS(WQ_GEMM_ROW)};
#undef WQ_GEMM_ROW
constexpr int kConfigCount = sizeof(kConfigs) / sizeof(kConfigs[0]);

// Estimated microseconds of a block of `c` over k when `resident` of them
// share a CU: a start and an end, and per x stage its bytes' way into LDS and
// the waves' matrix and vector cycles, which add up within a wave and overlap
// (all but a quarter of the smaller) between the waves of a SIMD.  The
// constants are fitted to 80 shapes (N 1000..28672, K 1600..14336, M 8..2048),
// every block shape timed on each, cold weights: the shape picked is within
// 8% of the fastest on all but three of them, where it is within 13%.
double block_us(const Config& c, int64_t k, int resident) {
    const double waves = c.nw * c.kw;
    const double per_simd = std::max(1.0, resident * waves / 4.0);
    const double pieces = c.tn * c.xk / 32.0;  // 16 x 32 pieces of W per wave and x stage
    const double valu = (c.ck == kStageK ? 12 : 16) * 4.0 * 1.73, mfma = 16.0 * c.tm * 1.62;
    const double cycles =
        pieces * (per_simd <= 1.0 ? valu + mfma : std::max(valu, mfma) + 0.26 * std::min(valu, mfma));
    const double bytes = c.kw * 16 * c.tm * c.xk * 2.0 + waves * 16 * c.tn * c.xk * 0.5625;
    const double stages = std::ceil((double)k / (c.xk * c.kw));
    return 2.9 + stages * (0.06 + resident * bytes / 168e3 + per_simd * cycles / 2300.0);
}

// Estimated microseconds of a launch of `lin` (count linears) at m rows:
// whole rounds of resident blocks and a last one with fewer per CU, or, for
// several linears (longest K first), an even spread of their blocks and the
// end of a short one, at least the longest alone.
struct Shape {
    int64_t n, k;
};
double launch_us(const Config& c, const Shape* lin, int count, int64_t m) {
    constexpr int kCus = 256;
    const int64_t bm = (m + c.rows_m - 1) / c.rows_m;
    const int64_t slots = (int64_t)kCus * c.occ;
    int64_t blocks = 0;
    double work = 0.0, longest = 0.0, shortest = 1e30, bytes = 0.0;
    for (int i = 0; i < count; ++i) blocks += (lin[i].n + c.rows_n - 1) / c.rows_n * bm;
    const int resident = (int)std::min<int64_t>(c.occ, (blocks + kCus - 1) / kCus);
    for (int i = 0; i < count; ++i) {
        const double t = block_us(c, lin[i].k, resident);
        work += t * (double)((lin[i].n + c.rows_n - 1) / c.rows_n * bm);
        longest = std::max(longest, count > 1 ? block_us(c, lin[i].k, 1) : t);
        shortest = std::min(shortest, t);
        bytes += (double)lin[i].n * lin[i].k * 0.5625;
    }
    double t;
    if (count > 1) {
        t = std::max(longest, work / ((double)kCus * resident) + 0.5 * shortest);
    } else {
        const int64_t full = blocks / slots, rest = blocks % slots;
        t = full * longest;
        if (rest) {
            const int r = (int)std::min<int64_t>(c.occ, (rest + kCus - 1) / kCus);
            t += full < 3 ? block_us(c, lin[0].k, r) : longest * std::max(0.5, (double)rest / slots);
        }
    }
    return std::max(t, bytes / 4.2e6 + 2.0);
}

bool config_allowed(const Config& c, int64_t m) {
    // R = 4 up to four rows: the times of 16 rows (single linears within 3%, 3B
    // step at M = 4 289-293 against 291 us) with scales in fp32.  One pass over W up to 64 rows, with the lowest tile that holds them;
    // from there on tiles of at least 32 rows (48 rows, and 64 x 256 in whole
    // lines, were never the fastest).
    if (m <= 4) return c.r == 4;
    if (m <= 64) return c.r == 16 && c.rows_m >= m && c.rows_m < m + 16;
    return c.r == 16 && c.tm >= 2 && c.tm != 3 && !(c.tm == 4 && c.rows_n == 256);
}

int pick_config(const Shape* lin, int count, int64_t m) {
    if (const char* e = std::getenv("WQ_GEMM_CONFIG")) {
        const int i = std::atoi(e);
        if (i >= 0 && i < kConfigCount && (m > 64 ? kConfigs[i].tm >= 2 && kConfigs[i].r == 16 : kConfigs[i].tm <= 4)) return i;
    }
    int best = -1;
    double best_us = 0.0;
    for (int i = 0; i < kConfigCount; ++i) {
        if (!config_allowed(kConfigs[i], m)) continue;
        const double us = launch_us(kConfigs[i], lin, count, m);
        if (best < 0 || us < best_us) {
            best = i;
            best_us = us;
        }
    }
    return best;
}

int64_t blocks_of(const Config& c, int64_t n, int64_t m) {
    return (n + c.rows_n - 1) / c.rows_n * ((m + c.rows_m - 1) / c.rows_m);
}

}  // namespace

int gemm_plan_config(const wq_linear* lin, int count, int64_t m) {
    // The estimate depends on the shapes only; a long list repeats its layers.
    std::array<Shape, 64> s;
    const int n = std::min(count, (int)s.size());
    for (int i = 0; i < n; ++i) {
        const wq_linear& l = lin[(int64_t)i * count / n];
        s[i] = Shape{l.N, l.K};
    }
    return pick_config(s.data(), n, m);
}

int gemm_plan_size(int config) {
    return plan_size(kConfigs[config].rows_n);
}

hipError_t launch_gemm_plan(int config, const GemmPlanEntry* entries, int count, int64_t blocks_n, int m,
                            hipStream_t stream) {
    const Config& c = kConfigs[config];
    return c.plan(entries, count, blocks_n * ((m + c.rows_m - 1) / c.rows_m), m, stream);
}

hipError_t launch_gemm(const uint32_t* packed, const uint16_t* scales, const uint16_t* x, uint16_t* y, int64_t n,
                       int64_t k, int64_t m, hipStream_t stream) {
    const Shape s{n, k};
    const Config& c = kConfigs[pick_config(&s, 1, m)];
    const GemmArgs a{packed, scales, x, y, n, (int32_t)(k / kGroup), (int32_t)m};
    return c.one(a, blocks_of(c, n, m), (int)((m + c.rows_m - 1) / c.rows_m), stream);
}

hipError_t launch_gemm_list(const wq_linear* lin, int count, int64_t m, hipStream_t stream) {
    // Linears of one launch are independent, so their blocks may come in any
    // order: the longest K first, and the launch ends on short blocks.
    for (int i0 = 0; i0 < count;) {
        std::array<Shape, kListEntries> s;
        const int n = std::min(count - i0, kListEntries);
        for (int i = 0; i < n; ++i) s[i] = Shape{lin[i0 + i].N, lin[i0 + i].K};
        const Config& c = kConfigs[pick_config(s.data(), n, m)];
        GemmList l{};
        l.m = (int32_t)m;
        int64_t blocks = 0;
        int taken = 0;
        for (; taken < n; ++taken) {
            const wq_linear& w = lin[i0 + taken];
            const int64_t more = (blocks_of(c, w.N, m) + 7) / 8 * 8;
            if (taken > 0 && blocks + more > INT32_MAX) break;
            l.e[taken] = GemmEntry{w.packed_w, w.scales, w.x, w.y, w.N, (int32_t)(w.K / kGroup), (int32_t)blocks};
            blocks += more;
        }
        l.count = taken;
        std::sort(l.e, l.e + taken, [](const GemmEntry& a, const GemmEntry& b) {
            return a.ng != b.ng ? a.ng > b.ng : a.first_block < b.first_block;
        });
        int64_t first = 0;
        for (int i = 0; i < taken; ++i) {
            l.e[i].first_block = (int32_t)first;
            first += (blocks_of(c, l.e[i].n, m) + 7) / 8 * 8;
        }
        const hipError_t e = c.list(l, blocks, stream);
        if (e != hipSuccess) return e;
        i0 += taken;
    }
    return hipSuccess;
}

}  // namespace wq
