// q8_gemm_once.hip -- panel products (see q8_gemm.hip) whose blocks request everything that they need before their first
// wait: rows of 513 to 2048 bytes, plain output.  In a file of its own: with these kernels in q8_gemm.hip's code object the
// others there, unchanged, took longer (a decoder step of 64 sentences 0.4 us of 107).
#include "q8_gemm_resident.h"
#include "q8_index.h"
#include <type_traits>

// ============================================================== whole tiles on their way at once ==
// Block of eight waves: 32 RP rows x 32 CG vectors, the k range (at most 512 KP bytes) cut into KP parts; wave (rp, kp)
// multiplies 32 rows by its part of all vectors.  Everything a block needs is requested before its first wait, up to
// 256 KB, and the products of 32 vectors begin when these are in LDS, while the rest is still arriving.  The parts' exact
// sums meet in LDS; a wave finishes its share of the vector tiles.  Weights packed or row by row, 16 x 16 results: 64
// contiguous bytes of a row, or a whole KiB of a packed tile, per request.
// What bounds it is what a compute unit takes in: requests are accepted at some 90 GB/s.  1024 x 2048 x 1024 with 64 x 64
// (us after the first block starts): all requested 3.0, first 32 vectors in LDS 3.6, last products 5.5, sums exchanged 6.0,
// stores done 6.7; the kernel with stages of 256 bytes, two of them on their way, took in 44 GB/s (a stage per 0.74 us)
// and ended at 9.2, of which 1.7 were biases requested behind the last products.  Kernel trace: 11.0 -> 8.4 us.
//
// TRADE: row-major weights whose rows are whole 128 bytes.  The 64 bytes that 16 rows have in a step then lie in the same half
// of their lines, and a compute unit takes such requests in at a lower rate than ones that fall on both halves, as those of
// other rows do; so odd rows request the two steps of a line the other way round, and what has arrived trades places before
// the products (64 selects for a wave's 64 operand registers).  3072 rows x 1000 and 8192 x 320 vectors: 640 bytes 13.7 and
// 13.9 -> 11.8 and 11.4, 1024 bytes 16.1 and 15.3 -> 12.6 and 12.1 (kernel trace).  A form of its own, so that the others keep
// their registers, in 128 registers, so that two blocks share a compute unit (with 130: 15.1 in place of 12.6).
template <int RP, int KP, int CG, bool TRADE>
__global__ __launch_bounds__(512, TRADE ? 4 : 2) void gemm_once_kernel(GemmJobs jobs)
{
    static_assert(RP * KP == 8 && (KP == 2 || KP == 4) && 2 * CG % KP == 0, "eight waves, even shares of the vector tiles");
    constexpr int ROWS = 32 * RP, COLS = 32 * CG, KB = 512 * KP, PITCH = KB + 16, PPC = KB / 16, PT = PPC / 16, CT = 2 * CG, KEEP = CT / KP;
    extern __shared__ __align__(16) int8_t s_g[];                      // [COLS x PITCH] codes, then the parts' sums
    const GemmArgs &a = jobs.j[blockIdx.z];
    if ((int)blockIdx.x * ROWS >= a.rows) return;                      // the grid is sized for the largest job
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int i = lane & 15, g = lane >> 4, rp = wave % RP, kp = wave / RP;
    const int r0 = (int)blockIdx.x * ROWS + 32 * rp, c0 = (int)blockIdx.y * COLS, ld = a.ld, n = a.n, rows = a.rows;

    // ---- requests (outside the matrix or the panel: zero) ----
    const __amdgpu_buffer_rsrc_t rx = q8_rsrc(a.xq, (size_t)n * ld);
    v4i xv[CG][PT];
    auto vectors = [&](int c) {
#pragma unroll
        for (int u = 0; u < PT; ++u) {
            const int e = u * 512 + tid, col = c0 + 32 * c + e / PPC, k = 16 * (e & (PPC - 1));
            xv[c][u] = __builtin_bit_cast(v4i, __builtin_amdgcn_raw_buffer_load_b128(rx, (int)(col < n && k < ld ? (unsigned)col * (unsigned)ld + k : Q8_OOB), 0, 0));
        }
    };
    vectors(0);
    const bool tiled = a.Wt != nullptr;
    const int flip = TRADE && !tiled ? i & 1 : 0;
    const __amdgpu_buffer_rsrc_t rw = tiled ? q8_rsrc(a.Wt, (size_t)a.ntiles * 16 * ld) : q8_rsrc(a.W, (size_t)rows * ld);
    v4i av[2][8];
#pragma unroll
    for (int u = 0; u < 2; ++u) {
        const int row0 = r0 + 16 * u;
        const unsigned base = tiled ? ((unsigned)(row0 >> 4) * (unsigned)(ld >> 6) << 10) + 16u * lane : (unsigned)(row0 + i) * (unsigned)ld + 16u * g;
        const unsigned step = tiled ? 1024u : 64u;
        const bool ok = (tiled ? row0 : row0 + i) < rows;
#pragma unroll
        for (int s = 0; s < 8; ++s) {
            const int ks = kp * 8 + (s ^ flip);
            av[u][s] = __builtin_bit_cast(v4i, __builtin_amdgcn_raw_buffer_load_b128(rw, (int)(ok && 64 * ks + (tiled ? 0 : 16 * g) < ld ? base + step * ks : Q8_OOB), 0, 0));
        }
    }
#pragma unroll
    for (int c = 1; c < CG; ++c) vectors(c);
    const __amdgpu_buffer_rsrc_t rs = q8_rsrc(a.xscale, (size_t)n * sizeof(float));
    const __amdgpu_buffer_rsrc_t rb = q8_rsrc(a.bias, a.bias ? (size_t)rows * sizeof(float) : 0);
    float bias[2][4], xs[KEEP];
#pragma unroll
    for (int j = 0; j < KEEP; ++j) xs[j] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rs, (c0 + 16 * (kp * KEEP + j) + i) * 4, 0, 0));
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
        for (int r = 0; r < 4; ++r) bias[u][r] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rb, (r0 + 16 * u + 4 * g + r) * 4, 0, 0));
    __builtin_amdgcn_sched_barrier(0);

    // ---- products, 32 vectors at a time ----
    v4i acc[2][CT];
#pragma unroll
    for (int c = 0; c < CG; ++c) {
#pragma unroll
        for (int u = 0; u < PT; ++u) {
            const int e = u * 512 + tid;
            *(v4i *)(s_g + (32 * c + e / PPC) * PITCH + 16 * (e & (PPC - 1))) = xv[c][u];
        }
        __syncthreads();
        if (TRADE && c == 0) {
#pragma unroll
            for (int u = 0; u < 2; ++u)
#pragma unroll
                for (int s = 0; s < 8; s += 2) {
                    const v4i even = flip ? av[u][s + 1] : av[u][s], odd = flip ? av[u][s] : av[u][s + 1];
                    av[u][s] = even;
                    av[u][s + 1] = odd;
                }
        }
        const int8_t *bp = s_g + (32 * c + i) * PITCH + kp * 512 + 16 * g;
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            acc[0][2 * c + t] = acc[1][2 * c + t] = (v4i){0, 0, 0, 0};
#pragma unroll
            for (int s = 0; s < 8; ++s) {
                const v4i x = *(const v4i *)(bp + 16 * t * PITCH + 64 * s);
                acc[0][2 * c + t] = __builtin_amdgcn_mfma_i32_16x16x64_i8(av[0][s], x, acc[0][2 * c + t], 0, 0, 0);
                acc[1][2 * c + t] = __builtin_amdgcn_mfma_i32_16x16x64_i8(av[1][s], x, acc[1][2 * c + t], 0, 0, 0);
            }
        }
    }

    // ---- the other parts' sums of this wave's vector tiles, then dequantization: lane (i, g) has rows 4 g + r of vector i ----
    const bool vec_ok = ((a.ldy & 3) == 0) && (((uintptr_t)a.Y & 15) == 0);
    const __amdgpu_buffer_rsrc_t rr = q8_rsrc(a.row_scale, a.row_scale ? (size_t)rows * sizeof(float) : 0);
    auto finish = [&](auto part) {
        constexpr int PART = decltype(part)::value;
        __syncthreads();                                               // (every wave has read its codes)
#pragma unroll
        for (int to = 0; to < KP; ++to) {
            if (to == PART) continue;
            v4i *out = (v4i *)s_g + (size_t)((rp * KP + to) * (KP - 1) + (PART < to ? PART : PART - 1)) * 2 * KEEP * 64 + lane;
#pragma unroll
            for (int j = 0; j < KEEP; ++j) { out[(2 * j) * 64] = acc[0][to * KEEP + j]; out[(2 * j + 1) * 64] = acc[1][to * KEEP + j]; }
        }
        __syncthreads();
#pragma unroll
        for (int j = 0; j < KEEP; ++j) {
            const int col = c0 + 16 * (PART * KEEP + j) + i;
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                v4i sum = acc[u][PART * KEEP + j];
#pragma unroll
                for (int from = 0; from < KP - 1; ++from)
                    sum += ((const v4i *)s_g)[(size_t)((rp * KP + PART) * (KP - 1) + from) * 2 * KEEP * 64 + (2 * j + u) * 64 + lane];
                if (col >= n) continue;
                const int row4 = r0 + 16 * u + 4 * g;
                float *y = a.Y + (size_t)col * a.ldy, v[4];
                const float c = a.w_scale * xs[j];
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    v[r] = (float)sum[r] * (a.row_scale ? __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rr, (row4 + r) * 4, 0, 0)) * xs[j] : c);
                    if (a.bias) v[r] = v[r] + bias[u][r];
                }
                if (vec_ok && row4 + 3 < rows) *(float4 *)(y + row4) = make_float4(v[0], v[1], v[2], v[3]);
                else {
#pragma unroll
                    for (int r = 0; r < 4; ++r)
                        if (row4 + r < rows) y[row4 + r] = v[r];
                }
            }
        }
    };
    if constexpr (KP == 2) {
        if (kp == 0) finish(std::integral_constant<int, 0>{});
        else finish(std::integral_constant<int, 1>{});
    } else {
        if (kp == 0) finish(std::integral_constant<int, 0>{});
        else if (kp == 1) finish(std::integral_constant<int, 1>{});
        else if (kp == 2) finish(std::integral_constant<int, 2>{});
        else finish(std::integral_constant<int, 3>{});
    }
}

// The same with the weights kept for several groups of 32 vectors: block (row block, share of the groups).  Groups are
// requested two ahead, two of them take turns in LDS.  With 64 rows of 2048 bytes a group takes 1.6 us: 64 KB in, and 256 KB
// through LDS (codes written, read by two row pairs, four parts' sums out and in), which is what bounds it.  (Four row
// tiles per wave instead of two would halve the reads and do not fit the registers.)
__global__ __launch_bounds__(512, 2) void gemm_stream_kernel(GemmJobs jobs, int shares)
{
    constexpr int RP = 2, KP = 4, ROWS = 32 * RP, KB = 512 * KP, PPC = KB / 16, PT = PPC / 16, OWN = 4 / KP;
    extern __shared__ __align__(16) int8_t s_g[];                      // [2][32 x KB] codes, [8 waves][4 tiles] sums
    const GemmArgs &a = jobs.j[blockIdx.z];
    if ((int)blockIdx.x * ROWS >= a.rows) return;                      // the grid is sized for the largest job
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int i = lane & 15, g = lane >> 4, rp = wave % RP, kp = wave / RP;
    const int r0 = (int)blockIdx.x * ROWS + 32 * rp, ld = a.ld, n = a.n, rows = a.rows;
    const int groups = (n + 31) >> 5, first = groups * (int)blockIdx.y / shares, end = groups * ((int)blockIdx.y + 1) / shares;
    v4i *s_e = (v4i *)(s_g + 2 * 32 * KB);

    const __amdgpu_buffer_rsrc_t rx = q8_rsrc(a.xq, (size_t)n * ld);
    auto vectors = [&](v4i (&xv)[PT], int grp) {
#pragma unroll
        for (int u = 0; u < PT; ++u) {
            const int e = u * 512 + tid, col = 32 * grp + e / PPC, k = 16 * (e & (PPC - 1));
            xv[u] = __builtin_bit_cast(v4i, __builtin_amdgcn_raw_buffer_load_b128(rx, (int)(grp < end && col < n && k < ld ? (unsigned)col * (unsigned)ld + k : Q8_OOB), 0, 0));
        }
    };
    v4i x0[PT], x1[PT];
    vectors(x0, first);
    const bool tiled = a.Wt != nullptr;
    const __amdgpu_buffer_rsrc_t rw = tiled ? q8_rsrc(a.Wt, (size_t)a.ntiles * 16 * ld) : q8_rsrc(a.W, (size_t)rows * ld);
    v4i av[2][8];
#pragma unroll
    for (int u = 0; u < 2; ++u) {
        const int row0 = r0 + 16 * u;
        const unsigned base = tiled ? ((unsigned)(row0 >> 4) * (unsigned)(ld >> 6) << 10) + 16u * lane : (unsigned)(row0 + i) * (unsigned)ld + 16u * g;
        const unsigned step = tiled ? 1024u : 64u;
        const bool ok = (tiled ? row0 : row0 + i) < rows;
#pragma unroll
        for (int s = 0; s < 8; ++s) {
            const int ks = kp * 8 + s;
            av[u][s] = __builtin_bit_cast(v4i, __builtin_amdgcn_raw_buffer_load_b128(rw, (int)(ok && 64 * ks + (tiled ? 0 : 16 * g) < ld ? base + step * ks : Q8_OOB), 0, 0));
        }
    }
    vectors(x1, first + 1);
    const __amdgpu_buffer_rsrc_t rs = q8_rsrc(a.xscale, (size_t)n * sizeof(float));
    const __amdgpu_buffer_rsrc_t rb = q8_rsrc(a.bias, a.bias ? (size_t)rows * sizeof(float) : 0), rr = q8_rsrc(a.row_scale, a.row_scale ? (size_t)rows * sizeof(float) : 0);
    // this wave finishes OWN of the group's four tiles of 16 rows x 16 vectors: tile q = 2 (vector half) + row tile, q / OWN = kp
    const int own = kp * OWN;
    float bias[OWN][4], rsv[OWN][4];
#pragma unroll
    for (int j = 0; j < OWN; ++j)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int at = (r0 + 16 * ((own + j) % 2) + 4 * g + r) * 4;
            bias[j][r] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rb, at, 0, 0));
            rsv[j][r] = a.row_scale ? __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rr, at, 0, 0)) : a.w_scale;
        }
    const bool vec_ok = ((a.ldy & 3) == 0) && (((uintptr_t)a.Y & 15) == 0);
    auto group = [&](v4i (&xv)[PT], int grp) {
        int8_t *buf = s_g + (grp & 1) * 32 * KB;
#pragma unroll
        for (int u = 0; u < PT; ++u) {                                 // (16 lanes read one piece of 16 vectors: on different banks)
            const int e = u * 512 + tid, col = e / PPC, pc = e & (PPC - 1);
            *(v4i *)(buf + col * KB + 16 * (pc ^ (col & 15))) = xv[u];
        }
        float xs[OWN];
#pragma unroll
        for (int j = 0; j < OWN; ++j) xs[j] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rs, (32 * grp + 16 * ((own + j) / 2) + i) * 4, 0, 0));
        vectors(xv, grp + 2);
        __syncthreads();
        v4i acc[2][2];
#pragma unroll
        for (int t = 0; t < 2; ++t) {
#pragma unroll
            for (int u = 0; u < 2; ++u) acc[u][t] = (v4i){0, 0, 0, 0};
#pragma unroll
            for (int s = 0; s < 8; ++s) {
                const v4i x = *(const v4i *)(buf + (16 * t + i) * KB + 16 * ((kp * 32 + 4 * s + g) ^ i));
#pragma unroll
                for (int u = 0; u < 2; ++u) acc[u][t] = __builtin_amdgcn_mfma_i32_16x16x64_i8(av[u][s], x, acc[u][t], 0, 0, 0);
            }
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) s_e[(wave * 4 + q) * 64 + lane] = acc[q % 2][q / 2];
        __syncthreads();
#pragma unroll
        for (int j = 0; j < OWN; ++j) {
            v4i sum = s_e[(rp * 4 + own + j) * 64 + lane];
#pragma unroll
            for (int from = 1; from < KP; ++from) sum += s_e[((from * RP + rp) * 4 + own + j) * 64 + lane];
            const int col = 32 * grp + 16 * ((own + j) / 2) + i;
            if (col >= n) continue;
            const int row4 = r0 + 16 * ((own + j) % 2) + 4 * g;
            float *y = a.Y + (size_t)col * a.ldy, v[4];
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                v[r] = (float)sum[r] * (rsv[j][r] * xs[j]);
                if (a.bias) v[r] = v[r] + bias[j][r];
            }
            if (vec_ok && row4 + 3 < rows) *(float4 *)(y + row4) = make_float4(v[0], v[1], v[2], v[3]);
            else {
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    if (row4 + r < rows) y[row4 + r] = v[r];
            }
        }
    };
    for (int grp = first; grp < end; grp += 2) {
        group(x0, grp);
        if (grp + 1 < end) group(x1, grp + 1);
    }
}

template <int RP, int KP, int CG, bool TRADE>
static q8_status launch_once(q8_ctx *ctx, const GemmJobs &jobs, int max_rows, int n, int njobs)
{
    constexpr size_t smem = (size_t)32 * CG * (512 * KP + 16);
    static Q8OncePerDevice asked;
    const q8_status st = q8i_lds(ctx, asked, (const void *)gemm_once_kernel<RP, KP, CG, TRADE>, smem, "panel product kernel");
    if (st) return st;
    const dim3 grid((max_rows + 32 * RP - 1) / (32 * RP), (n + 32 * CG - 1) / (32 * CG), njobs);
    Q8_LAUNCH(ctx, Q8_KERNEL_MFMA, (gemm_once_kernel<RP, KP, CG, TRADE>), grid, dim3(512), smem, jobs);
    return q8i_launch_check(ctx, "gemm");
}

q8_status q8i_gemm_once(q8_ctx *ctx, const GemmJobs &jobs, int max_rows, int n, int njobs, int rows, int cols, bool trade)
{
    if (rows == 64) return launch_once<2, 4, 2, false>(ctx, jobs, max_rows, n, njobs);
    if (cols == 32) return launch_once<4, 2, 1, false>(ctx, jobs, max_rows, n, njobs);
    return trade ? launch_once<4, 2, 2, true>(ctx, jobs, max_rows, n, njobs) : launch_once<4, 2, 2, false>(ctx, jobs, max_rows, n, njobs);
}

q8_status q8i_gemm_stream(q8_ctx *ctx, const GemmJobs &jobs, int max_rows, int n, int njobs, int row_blocks)
{
    const int groups = (n + 31) / 32, most = 256 / row_blocks, shares = most < 1 ? 1 : most < groups ? most : groups;
    constexpr size_t smem = (size_t)2 * 32 * 2048 + (size_t)8 * 4 * 1024;
    static Q8OncePerDevice asked;
    const q8_status st = q8i_lds(ctx, asked, (const void *)gemm_stream_kernel, smem, "streaming panel product kernel");
    if (st) return st;
    Q8_LAUNCH(ctx, Q8_KERNEL_MFMA, gemm_stream_kernel, dim3((max_rows + 63) / 64, shares, njobs), dim3(512), smem, jobs, shares);
    return q8i_launch_check(ctx, "gemm");
}

q8_status q8i_gemm_resident_1024(q8_ctx *ctx, const GemmJobs &jobs, int max_rows, int n, int njobs)
{
    constexpr size_t smem = (size_t)64 * (1024 + 16);
    static Q8OncePerDevice asked;
    const q8_status st = q8i_lds(ctx, asked, (const void *)gemm_resident_kernel<16>, smem, "resident product kernel");
    if (st) return st;
    Q8_LAUNCH(ctx, Q8_KERNEL_MFMA, gemm_resident_kernel<16>, dim3((max_rows + 63) / 64, (n + 63) / 64, njobs), dim3(256), smem, jobs);
    return q8i_launch_check(ctx, "gemm");
}
