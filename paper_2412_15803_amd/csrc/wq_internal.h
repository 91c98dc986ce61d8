// Internal launch interface between the C-ABI layer (wq_api.hip) and the
// kernels (wq_kernels.hip).  Arguments are already validated by the caller.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>

#include "wq.h"
#include "wq_limits.h"

namespace wq {

// Records `message` as the calling thread's last error message (the one
// wq_last_error_message returns) and returns `st`.
wq_status record_error(wq_status st, const char* message);

// WQ_OK for hipSuccess; otherwise WQ_ERR_HIP with the runtime's message,
// recorded as the thread's last error message for entry point `fn`.
wq_status hip_error(const char* fn, hipError_t e);

// Quantize + pack.
hipError_t launch_pack(const float* w, uint32_t* packed, uint16_t* scales,
                       int64_t n, int64_t k, hipStream_t stream);

// y[M][N] = x[M][K] * dequant(W)^T, picking the kernel for (M, K).
hipError_t launch_gemv(const uint32_t* packed, const uint16_t* scales,
                       const uint16_t* x, uint16_t* y,
                       int64_t n, int64_t k, int64_t m, hipStream_t stream);

// Smallest batch that uses the matrix cores.  At M = 2, vector kernel against
// GEMM: 3B-class step 345 against 279 us, 8B-class step 787 against 624,
// 128256 x 3072 67.9 against 39.2 (a linear alone in its launch:
// vector_takes_pair).
constexpr int kMatrixCoreMinM = 2;

// Largest batch of the planned decode steps (and of the vector kernel);
// larger ones (prompts) keep no plan.
constexpr int kMaxSmallBatchM = 64;

// Whether a small batch of m rows (2 <= m <= kMaxSmallBatchM) runs on the
// matrix cores: from kMatrixCoreMinM rows on.  Tuning overrides, read at
// every call (for comparing the two paths): WQ_SMALL_BATCH_VECTOR=1 sends
// every small batch to the vector kernel, WQ_MATRIX_MIN_M=n moves the
// threshold to n.
bool use_matrix_cores(int64_t m);

// y[M][N] on the matrix cores, any M (wq_gemm.hip), for the shapes gemm_fits
// (wq_limits.h) accepts.
hipError_t launch_gemm(const uint32_t* packed, const uint16_t* scales, const uint16_t* x, uint16_t* y,
                       int64_t n, int64_t k, int64_t m, hipStream_t stream);

// Independent linears at M > kMaxSmallBatchM, as few launches as their
// arguments allow; every one fits gemm_fits.
hipError_t launch_gemm_list(const wq_linear* lin, int count, int64_t m, hipStream_t stream);

// One linear of a grouped launch as the kernel sees it (built on the host,
// uploaded once per distinct descriptor list).
struct DecodeEntry {
    const void* packed;      // [n][ng] 16-byte groups
    const uint16_t* scales;  // [n][ng]
    const uint16_t* x;       // [ng * 32]
    uint16_t* y;             // [n]
    int64_t n;
    int64_t first_step;      // first step of this linear in its class's numbering
    int64_t steps;           // steps of this linear: ceil(n / rows per step)
    int32_t ng;              // groups of 32 per row
    int32_t lpr;             // lanes per row (16, 32 or 64)
    int32_t gpl;             // groups per lane (lpr * gpl >= ng)
    int32_t pad;             // rows per wave (small-batch vector launches)
};
static_assert(sizeof(DecodeEntry) == 72, "DecodeEntry layout");

// Linears of one launch with the same step shape.  The class's steps are
// split into `blocks` equal contiguous ranges, one per workgroup, for the
// workgroups [blocks_begin, blocks_begin + blocks) of the grid.
struct DecodeClass {
    int32_t lpr, gpl;     // the class's step shape
    int32_t first;        // offset of its linears in the class list
    int32_t count;        // number of linears
    int64_t steps;        // steps over all its linears
    int32_t blocks_begin;
    int32_t blocks;
};
static_assert(sizeof(DecodeClass) == 32, "DecodeClass layout");

// One workgroup's share of its class in a grouped launch: steps [begin,
// end) of the class's numbering, and the position (in the class's list) of
// the linear that holds step `begin`.
struct DecodeBlock {
    int32_t pos;
    int32_t begin, end;
    int32_t pad;
};
static_assert(sizeof(DecodeBlock) == 16, "DecodeBlock layout");

// Device-side view of one grouped launch: the entries, the class
// descriptors, per class the indices of its linears in order, and per
// workgroup its share.
struct DecodePlan {
    const DecodeEntry* entries;
    const DecodeClass* classes;
    const int32_t* class_lin;
    const DecodeBlock* blocks;
    int32_t nclasses;
};

// Small-batch decode step: independent linears in one launch of the
// matrix-core kernel.  The block shape is picked for the whole list and the
// number of rows m; its blocks span 16 << size rows of W, size =
// gemm_plan_size(config).  Entry i owns the blocks from first[size] * blocks_m
// on, ceil(n / rows) x blocks_m of them.  The plan holds `first` for every
// size, so that it does not depend on m and one resident copy serves all
// batches of a list.
constexpr int kGemmPlanSizes = 5;
struct GemmPlanEntry {
    const void* packed;      // [n][ng] 16-byte groups
    const uint16_t* scales;  // [n][ng]
    const uint16_t* x;       // [m][ng * 32]
    uint16_t* y;             // [m][n]
    int64_t n;
    int32_t ng;
    int32_t first[kGemmPlanSizes];
};
static_assert(sizeof(GemmPlanEntry) == 64, "GemmPlanEntry layout");
int gemm_plan_config(const wq_linear* lin, int count, int64_t m);
int gemm_plan_size(int config);
hipError_t launch_gemm_plan(int config, const GemmPlanEntry* entries, int count, int64_t blocks_n, int m,
                            hipStream_t stream);

// Small-batch decode step below kMatrixCoreMinM rows (or any small batch when
// forced): independent linears in
// one launch of the vector kernel.  Entry i owns waves [first_step,
// first_step + steps) of the grid, `pad` rows each (a multiple of 8, at most
// 256); batch rows [m0, m0 + m), m <= 8.
hipError_t launch_grouped_mb(const DecodeEntry* entries, int count, int64_t waves, int64_t m0, int m,
                             hipStream_t stream);
// Waves to split such a launch into for m batch rows (m <= 8) on `device`:
// a few times what the device holds at once.
hipError_t mb_target_waves(int m, int device, int64_t& waves);
// Rows per wave for a linear of ng groups per row when each wave is to
// stream about `work` (row, padded group) pairs.
int mb_rows_for_work(int64_t work, int64_t ng);

// The vector small-batch kernel walks a row's groups in 32-group tiles, two
// row sets per wave, when those pad the row less than 64-group tiles do.
__host__ __device__ constexpr bool mb_two_sets(int64_t ng) { return (ng + 31) / 32 * 32 < (ng + 63) / 64 * 64; }
__host__ __device__ constexpr int64_t mb_padded_groups(int64_t ng) {
    return mb_two_sets(ng) ? (ng + 31) / 32 * 32 : (ng + 63) / 64 * 64;
}

constexpr int kMbRows = 256;  // rows of a wave of the vector kernel at most
constexpr int kMbU = 4;       // rows of a step (per row set)
// Waves a single small-batch linear aims for: one per SIMD (2 to 12% faster
// than the 2048-wave split at M = 2 on the 8B-class shapes, 512 and 2048
// slower).
#ifndef WQ_MB_SINGLE_WAVES
#define WQ_MB_SINGLE_WAVES (256 * 4)
#endif
constexpr int64_t kMbSingleWaves = WQ_MB_SINGLE_WAVES;

// The vector kernel's launch of one linear.  x is loaded once per K tile and
// wave, so the rows a wave owns set how many weight bytes each x load serves
// (with 4 rows and 4 batch rows, x is 3.5x the weight bytes).  So: as many
// rows per wave, in whole steps of the row's tiling (4 rows with 64-group
// tiles, 8 with two row sets), as leave about kMbSingleWaves waves once each
// row run's K tiles are split over up to 4 waves (two tiles each at least).
struct MbSingle {
    int64_t rows_per_wave, blocks;  // blocks of four waves
    int split;
};
constexpr MbSingle mb_single(int64_t n, int64_t ng) {
    const int64_t r = mb_two_sets(ng) ? 2 * kMbU : kMbU;
    const int64_t steps = (n + r - 1) / r;
    const int64_t ntiles = mb_two_sets(ng) ? (ng + 31) / 32 : (ng + 63) / 64;
    int64_t max_split = 1;
    while (max_split < 4 && ntiles >= 2 * max_split) max_split *= 2;
    const int64_t spw = std::max<int64_t>(1, std::min<int64_t>(steps * max_split / kMbSingleWaves, kMbRows / r));
    const int64_t rows_per_wave = spw * r;
    const int64_t runs = (n + rows_per_wave - 1) / rows_per_wave;
    int split = 1;
    while (split < max_split && runs * split < kMbSingleWaves) split *= 2;
    return MbSingle{rows_per_wave, (runs * split + 3) / 4, split};
}

// Two rows of x against one linear alone in its launch: whether the vector
// kernel is the faster one.  The GEMM takes about one block of 16 to 128 rows
// per CU and round, so its time steps up where N passes a power of two and
// grows with K where N leaves CUs idle; the vector kernel's follows the bytes
// where its blocks fill whole rounds of the CUs and a row's 64-group tiles
// divide evenly over the waves that share it, and otherwise steps up by as
// much as two.  Measured at M = 2 (GEMM / vector, us, cold weights):
//   few rows              512 x 4096 5.0 / 4.2, 256 x 3328 4.8 / 4.0, 2048 x 3584 5.2 / 4.7, 2304 x 8192 8.0 / 7.3; 512 x 3072 4.9 / 5.0, 3072 x 6144 6.6 / 7.0
//   whole rounds          10240 x 8192 16.9 / 13.6, 12288 x 16384 28.7 / 25.1, 20480 x 4096 15.7 / 13.6, 11264 x 14336 25.1 / 23.1
//   a round nearly empty  14592 x 8192 17.3 / 23.7 (261 blocks), 25600 x 4096 16.2 / 21.5 (267), 28928 x 3584 14.8 / 22.9 (259)
//   uneven tiles          16384 x 6144 14.5 / 17.3, 11264 x 10240 19.5 / 22.9
//   below a power of two  16384 x 4096 10.4 / 11.5, 28672 x 4096 17.4 / 18.2, 14336 x 13312 24.9 / 28.9; 13312 x 16384 29.3 / 26.5
//   many rows             46080 x 14336 68.6 / 82.1, 44032 x 16384 80.1 / 95.4, 128256 x 3072 39.7 / 67.9
// Over 3500 random shapes (N 64..131072, K 1536..16384) the choice is 0.6%
// slower than the faster kernel on average (always the GEMM 12%, always the
// vector kernel 14%) and 12% at the 99th percentile.
constexpr bool vector_takes_pair(int64_t n, int64_t k) {
    if (n <= 2048) return k > 3072;
    if (n <= 3072 && k > 6144) return true;
    const int64_t ng = k / 32, tiles = (ng + 63) / 64;
    const bool even = !mb_two_sets(ng) && (tiles == 2 || tiles % 4 == 0 || (tiles > 4 && tiles % 4 == 3));
    if (!even || n > 40960 || mb_single(n, ng).blocks % 256 != 0) return false;
    if (tiles % 4 == 0) return true;
    int64_t half = 8192;  // the power of two below n
    while (half * 2 < n) half *= 2;
    if (tiles == 2) return n > 8192 && n <= half + half / 2;
    return n <= 6144 || (n > 8192 && n <= half + half / 4);
}

// Largest groups-per-lane of the grouped kernel (K <= 16384).
constexpr int kDecodeMaxGpl = 8;
constexpr int kMaxClasses = 16;

// Launch the grouped batch-1 GEMV over a plan in device memory with
// `blocks` workgroups (the sum of the classes' workgroups), each one CU's
// worth of waves.
hipError_t launch_grouped_m1(const DecodePlan& plan, int max_gpl, int blocks, hipStream_t stream);

// Workgroups of the grouped kernel (for max_gpl) that the device holds at
// once: one per CU.
hipError_t grouped_capacity(int max_gpl, int device, int& blocks);

}  // namespace wq
