// Internal launch interface between the C-ABI layer (wq_api.hip) and the
// kernels (wq_kernels.hip).  Arguments are already validated by the caller.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

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
__host__ __device__ inline bool mb_two_sets(int64_t ng) { return (ng + 31) / 32 * 32 < (ng + 63) / 64 * 64; }
__host__ __device__ inline int64_t mb_padded_groups(int64_t ng) {
    return mb_two_sets(ng) ? (ng + 31) / 32 * 32 : (ng + 63) / 64 * 64;
}

// Two rows of x against one linear alone in its launch: whether the vector
// kernel is the faster one.  The GEMM takes about one block of 16 to 128 rows
// per CU and round, so its time steps up where N passes a power of two and
// grows with K where N leaves CUs idle; the vector kernel's follows the bytes,
// best where a row's 64-group tiles divide evenly over the four waves of a
// block.  Measured at M = 2 (GEMM / vector, us, cold weights):
//   few rows            512 x 4096 4.9 / 4.0, 2048 x 3584 5.2 / 4.7; 2560 x 4096 5.3 / 5.4, 1024 x 3072 4.9 / 5.0
//   code rows 4 KiB apart   4096 x 8192 8.4 / 7.8, 28672 x 8192 28.6 / 27.2; 65536 x 8192 54.0 / 57.6
//   even tiles, deep    4096 x 14336 12.2 / 11.4, 6144 x 13824 15.3 / 14.5; 8192 x 14336 16.4 / 17.5, 4096 x 10240 9.4 / 10.5
//   N past a power of 2 20480 x 4096 15.0 / 12.8, 10240 x 14336 24.3 / 20.8; 14336 x 4096 9.8 / 10.1, 40960 x 6144 31.2 / 34.5
//   N up to 32768       32768 x 4096 21.2 / 17.2, 28672 x 4096 16.2 / 15.7, 30720 x 14336 65.9 / 55.1; 28672 x 14336 46.4 / 48.3,
//                       16384 x 4096 10.3 / 11.0
// Over 357 measured shapes (N 128..128256, K 2048..16384) the choice is within 1%
// of the faster kernel on average (always the GEMM 7.4%, always the vector
// kernel 7.0%).
inline bool vector_takes_pair(int64_t n, int64_t k) {
    const int64_t ng = k / 32, tiles = (ng + 63) / 64;
    if (n <= 2048) return k >= 3584;
    const bool even = !mb_two_sets(ng) && (tiles == 2 || tiles % 4 == 0 || (tiles > 4 && tiles % 4 == 3));
    if (!even || n >= 65536) return false;
    if (k % 8192 == 0 || (tiles >= 7 && n <= 6144)) return true;
    int64_t half = 8192;  // the power of two below n
    while (half * 2 < n) half *= 2;
    return n > 8192 && (n <= half + half / 4 || (n > (tiles == 2 ? 16384 : 28672) && n <= 32768));
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
