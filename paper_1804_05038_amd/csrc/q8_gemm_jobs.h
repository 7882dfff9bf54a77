// q8_gemm_jobs.h -- what the panel products' kernels take: one or several products of a launch.
#ifndef Q8_GEMM_JOBS_H
#define Q8_GEMM_JOBS_H

#include "q8_internal.h"

struct GemmArgs {
    const int8_t *W;       // [rows x ld] int8
    const int8_t *Wt;      // the same matrix tile-packed (q8_pack_tiles), or NULL: every matrix-core operand of 16 rows x 64 k
                           // bytes is then one contiguous KiB instead of 16 pieces of rows that lie ld bytes apart, which the
                           // memory system delivers about 2.5 times as fast (measured: 192 KB per block, 2.1 against 5.3 us)
    const int8_t *xq;      // [n x ld] int8 codes of the n vectors
    const float *xscale;   // [n]
    const float *bias;     // [rows] or NULL
    float *Y;              // [n x ldy]
    int32_t *tap_acc;      // [n x rows] or NULL
    float *part_max;       // STATS: [n x ntiles] maximum of each 16-row tile
    double *part_sum;      // STATS: [n x ntiles] sum of exp(y - maximum)
    int rows, ld, n, ldy, ntiles;
    int tiled;             // Y as [ntiles][n][16]: every 16 x 16 result tile is one contiguous KiB
    float w_scale;
    const float *row_scale; // NULL, or one weight scale per row in place of w_scale
};
#define GEMM_MAX_JOBS 3
struct GemmJobs {          // products of one launch (blockIdx.z), all over the same number of vectors
    GemmArgs j[GEMM_MAX_JOBS];
};

// q8_gemm_once.hip; rows: of one block of gemm_once_kernel's three forms (64: 64 rows x 64 vectors, k of at most 2048 bytes;
// 128: 128 rows x cols vectors (32 or 64), k of at most 1024; x 64 with trade: see there)
q8_status q8i_gemm_once(q8_ctx *ctx, const GemmJobs &jobs, int max_rows, int n, int njobs, int rows, int cols, bool trade);
q8_status q8i_gemm_resident_1024(q8_ctx *ctx, const GemmJobs &jobs, int max_rows, int n, int njobs);
// row_blocks: of all products; each has as many shares of the vectors as give every compute unit a block
q8_status q8i_gemm_stream(q8_ctx *ctx, const GemmJobs &jobs, int max_rows, int n, int njobs, int row_blocks);
// q8_gemm_quant.hip; tiles of 16 rows per block (q8_part_rows)
q8_status q8i_gemm_part(q8_ctx *ctx, const GemmJobs &jobs, int max_rows, int max_ld, int n, int njobs, int tiles);

#endif
