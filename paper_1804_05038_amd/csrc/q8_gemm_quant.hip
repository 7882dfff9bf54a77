// q8_gemm_quant.hip -- a panel product of few vectors in one launch: every block quantizes the vectors it multiplies.
#include "q8_gemm_jobs.h"
#include "q8_route.h"

// Block of eight waves: 16 RT rows x 16 vectors.  A wave takes the floats of two vectors, makes their codes by itself (maximum
// over its lanes) and leaves them in LDS; then each wave multiplies the block's rows by its eighth of the k range (at most SW
// steps of 64 bytes), from weights that were requested with the floats; the eight parts' exact sums meet in LDS.  Codes and
// sums as quantize_rows_kernel and the other panel products make them, value for value.
// The quantization is done again by every block of the same vectors (128 KB of floats for 16 vectors of 2048, 1.4 us of what a
// compute unit takes in), which is less than the launch of its own (4.5 us and the gap behind it) as long as few blocks'
// worth of rows share a compute unit: q8_quant_rows has the rule and both sides (1024 rows of 2048 bytes times 30 vectors, w(h_i) of
// a sentence: 8.3 -> 4.3 us per call; 3072 x 512 times 64: 7.3 -> 3.5).
struct GemmQuantArgs {
    const int8_t *W, *Wt;                // [rows x ld], the same tile-packed or NULL
    const float *X, *bias, *row_scale;   // [n x ldx], [rows] or NULL, [rows] or NULL (then w_scale)
    float *Y;                            // [n x ldy]
    int rows, ld, K, n, ldx, ldy;
    float w_scale;
};

template <int RT, int SW>
__global__ __launch_bounds__(512) void gemm_quant_kernel(GemmQuantArgs a)
{
    constexpr int FC = 2 * SW, PITCH = 1024 * FC / 4 + 16, SP = 20;
    extern __shared__ __align__(16) int8_t s_q[];                      // [16][PITCH] codes, [8 parts][RT][16 vectors][SP] sums
    __shared__ float s_scale[16];
    int *s_p = (int *)(s_q + 16 * PITCH);
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), i = lane & 15, g = lane >> 4;
    const int r0 = (int)blockIdx.x * 16 * RT, c0 = (int)blockIdx.y * 16, rows = a.rows, ld = a.ld, K = a.K;

    // ---- requests: floats, weights, what the results need (outside the panel or the matrix: zero) ----
    const __amdgpu_buffer_rsrc_t rx = q8_rsrc(a.X, ((size_t)(a.n - 1) * a.ldx + K) * sizeof(float));
    float4 v[2][FC];
#pragma unroll
    for (int q = 0; q < 2; ++q)
#pragma unroll
        for (int c = 0; c < FC; ++c) {
            const int col = c0 + 2 * wave + q, k = 4 * (lane + 64 * c);
            v[q][c] = __builtin_bit_cast(float4, __builtin_amdgcn_raw_buffer_load_b128(rx, (int)(col < a.n && k < K ? ((unsigned)col * (unsigned)a.ldx + k) * 4u : Q8_OOB), 0, 0));
        }
    const bool tiled = a.Wt != nullptr;
    const int S = (ld + 63) >> 6, k0 = S * wave >> 3, k1 = S * (wave + 1) >> 3;
    const __amdgpu_buffer_rsrc_t rw = tiled ? q8_rsrc(a.Wt, (size_t)((rows + 15) >> 4) * 16 * ld) : q8_rsrc(a.W, (size_t)rows * ld);
    v4i av[RT][SW];
#pragma unroll
    for (int t = 0; t < RT; ++t) {
        const int row0 = r0 + 16 * t;
        const unsigned base = tiled ? ((unsigned)(row0 >> 4) * (unsigned)(ld >> 6) << 10) + 16u * lane : (unsigned)(row0 + i) * (unsigned)ld + 16u * g;
        const bool ok = (tiled ? row0 : row0 + i) < rows;
#pragma unroll
        for (int s = 0; s < SW; ++s) {
            const int ks = k0 + s;
            const bool in = ok && ks < k1 && 64 * ks + (tiled ? 0 : 16 * g) < ld;
            av[t][s] = __builtin_bit_cast(v4i, __builtin_amdgcn_raw_buffer_load_b128(rw, (int)(in ? base + (tiled ? 1024u : 64u) * ks : Q8_OOB), 0, 0));
        }
    }
    // this thread finishes row `row` of vectors col, col + 32 / RT, ..
    const int row = tid % (16 * RT), col0 = tid / (16 * RT), at = min(r0 + row, rows - 1);
    const float bias = a.bias ? a.bias[at] : 0.0f, rs = a.row_scale ? a.row_scale[at] : a.w_scale;
    __builtin_amdgcn_sched_barrier(0);

    // ---- codes ----
    float scale[2], inv[2];
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        float m = 0.0f;
#pragma unroll
        for (int c = 0; c < FC; ++c) m = fmaxf(m, fmaxf(fmaxf(fabsf(v[q][c].x), fabsf(v[q][c].y)), fmaxf(fabsf(v[q][c].z), fabsf(v[q][c].w))));
        q8_scale_of(wave_max_f(m), scale[q], inv[q]);
        if (lane == 0) s_scale[2 * wave + q] = scale[q];
    }
#pragma unroll
    for (int q = 0; q < 2; ++q)
#pragma unroll
        for (int c = 0; c < FC; ++c)
            *(int *)(s_q + (2 * wave + q) * PITCH + 4 * (lane + 64 * c)) = q8_pack4(v[q][c].x, v[q][c].y, v[q][c].z, v[q][c].w, inv[q]);
    __syncthreads();

    // ---- products (steps past the part have zero weights) ----
    v4i acc[RT];
#pragma unroll
    for (int t = 0; t < RT; ++t) acc[t] = (v4i){0, 0, 0, 0};
#pragma unroll
    for (int s = 0; s < SW; ++s) {
        const v4i x = *(const v4i *)(s_q + i * PITCH + 64 * min(k0 + s, 4 * FC - 1) + 16 * g);
#pragma unroll
        for (int t = 0; t < RT; ++t) acc[t] = __builtin_amdgcn_mfma_i32_16x16x64_i8(av[t][s], x, acc[t], 0, 0, 0);
    }
#pragma unroll
    for (int t = 0; t < RT; ++t) *(v4i *)(s_p + ((wave * RT + t) * 16 + i) * SP + 4 * g) = acc[t];
    __syncthreads();
#pragma unroll
    for (int j = 0; j < (RT + 1) / 2; ++j) {
        const int col = col0 + j * 32 / RT;
        if (col >= 16 || c0 + col >= a.n || r0 + row >= rows) continue;
        int sum = 0;
#pragma unroll
        for (int w = 0; w < 8; ++w) sum += s_p[((w * RT + (row >> 4)) * 16 + col) * SP + (row & 15)];
        float y = (float)sum * (rs * s_scale[col]);
        if (a.bias) y = y + bias;
        a.Y[(size_t)(c0 + col) * a.ldy + r0 + row] = y;
    }
}

// The same from codes that are there already, up to three products in a launch: a wave loads its part of 16 vectors' codes as the
// matrix cores take them, so nothing waits for anything but its own operands until the parts' sums meet.
template <int RT, int SW>
__global__ __launch_bounds__(512) void gemm_part_kernel(GemmJobs jobs)
{
    constexpr int SP = 20;
    __shared__ __align__(16) int s_p[8 * RT * 16 * SP];                // [8 parts][RT][16 vectors][SP]
    const GemmArgs &a = jobs.j[blockIdx.z];
    const int r0 = (int)blockIdx.x * 16 * RT, c0 = (int)blockIdx.y * 16, rows = a.rows, ld = a.ld;
    if (r0 >= rows) return;                                            // the grid is sized for the largest job
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), i = lane & 15, g = lane >> 4;
    const bool tiled = a.Wt != nullptr;
    const int S = (ld + 63) >> 6, k0 = S * wave >> 3, k1 = S * (wave + 1) >> 3;
    const __amdgpu_buffer_rsrc_t rq = q8_rsrc(a.xq, (size_t)a.n * ld), rw = tiled ? q8_rsrc(a.Wt, (size_t)a.ntiles * 16 * ld) : q8_rsrc(a.W, (size_t)rows * ld);
    v4i xv[SW], av[RT][SW], acc[RT];
#pragma unroll
    for (int s = 0; s < SW; ++s) {
        const int k = 64 * (k0 + s) + 16 * g;
        xv[s] = __builtin_bit_cast(v4i, __builtin_amdgcn_raw_buffer_load_b128(rq, (int)(c0 + i < a.n && k0 + s < k1 && k < ld ? (unsigned)(c0 + i) * (unsigned)ld + k : Q8_OOB), 0, 0));
    }
#pragma unroll
    for (int t = 0; t < RT; ++t) {
        const int row0 = r0 + 16 * t;
        const unsigned base = tiled ? ((unsigned)(row0 >> 4) * (unsigned)(ld >> 6) << 10) + 16u * lane : (unsigned)(row0 + i) * (unsigned)ld + 16u * g;
        const bool ok = (tiled ? row0 : row0 + i) < rows;
#pragma unroll
        for (int s = 0; s < SW; ++s) {
            const int ks = k0 + s;
            const bool in = ok && ks < k1 && 64 * ks + (tiled ? 0 : 16 * g) < ld;
            av[t][s] = __builtin_bit_cast(v4i, __builtin_amdgcn_raw_buffer_load_b128(rw, (int)(in ? base + (tiled ? 1024u : 64u) * ks : Q8_OOB), 0, 0));
        }
        acc[t] = (v4i){0, 0, 0, 0};
    }
    // this thread finishes row `row` of vectors col0, col0 + 32 / RT, ..
    const int row = tid % (16 * RT), col0 = tid / (16 * RT), at = min(r0 + row, rows - 1);
    const float bias = a.bias ? a.bias[at] : 0.0f, rs = a.row_scale ? a.row_scale[at] : a.w_scale;
    float xs[(RT + 1) / 2];
#pragma unroll
    for (int j = 0; j < (RT + 1) / 2; ++j) xs[j] = a.xscale[min(c0 + col0 + j * 32 / RT, a.n - 1)];
#pragma unroll
    for (int s = 0; s < SW; ++s)
#pragma unroll
        for (int t = 0; t < RT; ++t) acc[t] = __builtin_amdgcn_mfma_i32_16x16x64_i8(av[t][s], xv[s], acc[t], 0, 0, 0);
#pragma unroll
    for (int t = 0; t < RT; ++t) *(v4i *)(s_p + ((wave * RT + t) * 16 + i) * SP + 4 * g) = acc[t];
    __syncthreads();
#pragma unroll
    for (int j = 0; j < (RT + 1) / 2; ++j) {
        const int col = col0 + j * 32 / RT;
        if (col >= 16 || c0 + col >= a.n || r0 + row >= rows) continue;
        int sum = 0;
#pragma unroll
        for (int w = 0; w < 8; ++w) sum += s_p[((w * RT + (row >> 4)) * 16 + col) * SP + (row & 15)];
        float y = (float)sum * (rs * xs[j]);
        if (a.bias) y = y + bias;
        a.Y[(size_t)(c0 + col) * a.ldy + r0 + row] = y;
    }
}

template <int RT> static q8_status launch_part(q8_ctx *ctx, const GemmJobs &jobs, int max_rows, int max_ld, int n, int njobs)
{
    const dim3 grid((max_rows + 16 * RT - 1) / (16 * RT), (n + 15) / 16, njobs);
    if (max_ld <= 1024) Q8_LAUNCH(ctx, Q8_KERNEL_MFMA, (gemm_part_kernel<RT, 2>), grid, dim3(512), 0, jobs);
    else Q8_LAUNCH(ctx, Q8_KERNEL_MFMA, (gemm_part_kernel<RT, 4>), grid, dim3(512), 0, jobs);
    return q8i_launch_check(ctx, "gemm");
}

q8_status q8i_gemm_part(q8_ctx *ctx, const GemmJobs &jobs, int max_rows, int max_ld, int n, int njobs, int tiles)
{
    return tiles == 1 ? launch_part<1>(ctx, jobs, max_rows, max_ld, n, njobs) : tiles == 2 ? launch_part<2>(ctx, jobs, max_rows, max_ld, n, njobs)
                                                                                          : launch_part<4>(ctx, jobs, max_rows, max_ld, n, njobs);
}

template <int RT, int SW> static q8_status launch_quant(q8_ctx *ctx, const GemmQuantArgs &a)
{
    constexpr size_t smem = (size_t)16 * (512 * SW + 16) + (size_t)8 * RT * 16 * 20 * sizeof(int);
    static Q8OncePerDevice asked;
    const q8_status st = q8i_lds(ctx, asked, (const void *)gemm_quant_kernel<RT, SW>, smem, "panel product kernel");
    if (st) return st;
    Q8_LAUNCH(ctx, Q8_KERNEL_MFMA, (gemm_quant_kernel<RT, SW>), dim3((a.rows + 16 * RT - 1) / (16 * RT), (a.n + 15) / 16), dim3(512), smem, a);
    return q8i_launch_check(ctx, "gemm");
}

template <int RT> static q8_status launch_quant_rt(q8_ctx *ctx, const GemmQuantArgs &a)
{
    if (a.ld <= 512) return launch_quant<RT, 1>(ctx, a);
    if (a.ld <= 1024) return launch_quant<RT, 2>(ctx, a);
    return launch_quant<RT, 4>(ctx, a);
}

// Y = dequantize(W . q(X)) + bias in one launch; *launched = 0 where two are faster, or the shape is not for this kernel.
q8_status q8i_gemm_quant(q8_ctx *ctx, const q8_mat *W, const float *row_scale, const float *X, int n, int ldx, const float *bias, float *Y, int ldy,
                         int *launched)
{
    *launched = 0;
    const int rt = q8_quant_rows(W->rows, W->ld, n);
    if (!rt || W->cols % 4 || (size_t)((W->rows + 15) / 16 * 16) * W->ld >= (1u << 31) || (size_t)n * ldx * sizeof(float) >= (1u << 31)) return Q8_OK;
    const GemmQuantArgs a = {W->data, W->ld % 64 == 0 ? W->tiles : nullptr, X, bias, row_scale, Y, W->rows, W->ld, W->cols, n, ldx, ldy, W->scale};
    *launched = 1;
    return rt == 1 ? launch_quant_rt<1>(ctx, a) : rt == 2 ? launch_quant_rt<2>(ctx, a) : launch_quant_rt<4>(ctx, a);
}
