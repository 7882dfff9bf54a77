// q8_fp32.hip -- the 32-bit engine that the paper measures its 8-bit engine against
// (Section 4, Tables 3 and 6: "32-bit" columns): the same model with fp32 weights and no
// quantization anywhere.  Only the products differ; gates, attention, softmax, top-k and the
// search are the kernels of the 8-bit path.  A product is y = (float)(sum in double) + bias.
#include "q8_internal.h"

struct F32Job {
    const float *W;        // [rows x ld] fp32
    const float *X;        // [n x ldx]
    const float *bias;     // [rows] or NULL
    float *Y;              // [n x ldy]
    int rows, cols, ld, ldx, ldy;
    int flat;              // X is contiguous, in whole 16-byte pieces
};
#define F32_MAX_JOBS 3
struct F32Jobs {
    F32Job j[F32_MAX_JOBS];
    int nblk[F32_MAX_JOBS + 1];      // job t owns blocks [nblk[t], nblk[t + 1])
};
// ---- the streaming product's pieces ----
// A product is bound by its weights' way from memory (4 bytes per two operations at one vector), so every
// wave keeps two rounds of 16-byte loads in flight: RW rows x UN chunks of 256 columns are multiplied
// while the next RW x UN arrive.  Vectors sit in LDS as floats.  A product of two floats is exact in
// double (24 + 24 bits), so fma rounds where a separate multiply and add would: same sums, half the
// instructions.
template <int RW, int UN>
struct F32Regs {
    float4 w[RW][UN];
};

// One row through a descriptor of its own (a lane past the row, and a row that is not there, read as zero
// without traffic; every load is unconditional, so the compiler's wait counts stay exact).
__device__ __forceinline__ __amdgpu_buffer_rsrc_t f32_row(const float *W, int row, int rows, int ld)
{
    const int r = __builtin_amdgcn_readfirstlane(row);
    return q8_rsrc(W + (size_t)(r < rows ? r : 0) * ld, r < rows ? (size_t)ld * sizeof(float) : 0);
}

template <int RW, int UN>
__device__ __forceinline__ void f32_load(F32Regs<RW, UN> &R, const __amdgpu_buffer_rsrc_t (&row)[RW], int cols, int c0, int lane)
{
#pragma unroll
    for (int u = 0; u < RW; ++u)
#pragma unroll
        for (int t = 0; t < UN; ++t) {
            const int k = ((c0 + t) * 64 + lane) * 4;
            const unsigned off = k < cols ? (unsigned)k * 4u : Q8_OOB;
            R.w[u][t] = __builtin_bit_cast(float4, __builtin_amdgcn_raw_buffer_load_b128(row[u], (int)off, 0, 0));
        }
}

// LDS pitch of a vector: where a row's last chunk of 256 columns is incomplete, four zeros at least follow the vector.
// The lanes past cols read those: their weights are zeros, and zero times an infinite entry of x would not be zero.
// GAP is false in kernels whose vectors are all whole chunks: nothing is masked and nothing lies between them (in one
// kernel for both, a decoder step and output layer of such vectors took 75.5 us instead of 72.8).
__host__ __device__ constexpr int f32_pitch(int cols) { return cols % 256 == 0 ? cols : ((cols + 3) & ~3) + 4; }
template <bool GAP>
__device__ __forceinline__ int f32_pitch_of(int cols) { return GAP ? f32_pitch(cols) : cols; }

// x: N vectors in LDS, pitch floats apart (f32_pitch, zeros past cols).
template <int N, int RW, int UN, bool GAP>
__device__ __forceinline__ void f32_fma(const F32Regs<RW, UN> &R, const float *x, int pitch, int cols, int c0, int lane, double (&acc)[RW][N])
{
#pragma unroll
    for (int t = 0; t < UN; ++t) {
        if ((c0 + t) * 256 >= cols) break;                      // uniform
        const int k = ((c0 + t) * 64 + lane) * 4, kx = GAP ? min(k, pitch - 4) : k;
        double w[RW][4];
#pragma unroll
        for (int u = 0; u < RW; ++u) {
            float4 v = R.w[u][t];
            if (GAP && (cols & 3)) {                                     // what lies past cols in the row counts for nothing
                v.x = k < cols ? v.x : 0.0f; v.y = k + 1 < cols ? v.y : 0.0f;
                v.z = k + 2 < cols ? v.z : 0.0f; v.w = k + 3 < cols ? v.w : 0.0f;
            }
            w[u][0] = (double)v.x; w[u][1] = (double)v.y; w[u][2] = (double)v.z; w[u][3] = (double)v.w;
        }
#pragma unroll
        for (int j = 0; j < N; ++j) {
            const float4 xv = *(const float4 *)(x + (size_t)j * pitch + kx);
            const double x0 = (double)xv.x, x1 = (double)xv.y, x2 = (double)xv.z, x3 = (double)xv.w;
#pragma unroll
            for (int u = 0; u < RW; ++u) {
                acc[u][j] = fma(w[u][0], x0, acc[u][j]);
                acc[u][j] = fma(w[u][1], x1, acc[u][j]);
                acc[u][j] = fma(w[u][2], x2, acc[u][j]);
                acc[u][j] = fma(w[u][3], x3, acc[u][j]);
            }
        }
    }
}

// The rest of a product whose first UN chunks are on their way in R.
template <int N, int RW, int UN, bool GAP>
__device__ __forceinline__ void f32_product(F32Regs<RW, UN> &R, const __amdgpu_buffer_rsrc_t (&row)[RW], const float *x, int pitch,
                                            int cols, int lane, double (&acc)[RW][N])
{
    const int nchunk = (cols + 255) >> 8;
    if (nchunk <= UN) {
        f32_fma<N, RW, UN, GAP>(R, x, pitch, cols, 0, lane, acc);
        return;
    }
    for (int c0 = 0; c0 < nchunk; c0 += 2 * UN) {
        F32Regs<RW, UN> S;
        f32_load<RW, UN>(S, row, cols, c0 + UN, lane);
        f32_fma<N, RW, UN, GAP>(R, x, pitch, cols, c0, lane, acc);
        f32_load<RW, UN>(R, row, cols, c0 + 2 * UN, lane);
        f32_fma<N, RW, UN, GAP>(S, x, pitch, cols, c0 + UN, lane, acc);
    }
}

// N vectors into LDS at the pitch of f32_fma, by a block of 256 threads.  Loads come back in the order they were
// issued, so the vectors are requested before the weights and stored to LDS behind the weights' requests: staging
// them in one go after the requests made the block wait for the weights first (GRU r 11.7 us, readout 11.8 us).
// flat (contiguous vectors of whole 16-byte pieces): they lie as they will in LDS, but for the zeros between them, and XB
// pieces per thread are requested at once; longer vectors and all other layouts follow in f32_x_store.
template <int XB>
struct F32X {
    float4 v[XB];
};
template <int XB>
__device__ __forceinline__ void f32_x_load(F32X<XB> &R, const float *X, int total, int flat)
{
    const __amdgpu_buffer_rsrc_t rx = q8_rsrc(X, flat ? (size_t)total * sizeof(float) : 0);
#pragma unroll
    for (int i = 0; i < XB; ++i)
        R.v[i] = __builtin_bit_cast(float4, __builtin_amdgcn_raw_buffer_load_b128(rx, (i * 256 + (int)threadIdx.x) * 16, 0, 0));
    __builtin_amdgcn_sched_barrier(0);
}
template <int N, int XB, bool GAP>
__device__ __forceinline__ void f32_x_store(const F32X<XB> &R, float *s, const float *X, int cols, int ldx, int flat)
{
    __builtin_amdgcn_sched_barrier(0);
    const int pitch = f32_pitch_of<GAP>(cols);
    if (flat) {
        const int total = N * cols;
        auto store = [&](auto at) {                            // element k of the run goes to at(k)
#pragma unroll
            for (int i = 0; i < XB; ++i) {
                const int k = (i * 256 + (int)threadIdx.x) * 4;
                if (k < total) *(float4 *)(s + at(k)) = R.v[i];
            }
            for (int k = (XB * 256 + (int)threadIdx.x) * 4; k < total; k += 1024) *(float4 *)(s + at(k)) = *(const float4 *)(X + k);
        };
        if (!GAP || pitch == cols) {
            store([](int k) { return k; });
        } else {
            // four further on per vector before it; the quotient by a reciprocal: k < 2^16, so (k + 1/2) / cols lies further
            // from an integer than the roundings move it
            const float inv = __builtin_amdgcn_rcpf((float)cols);
            store([&](int k) { return k + 4 * (int)(((float)k + 0.5f) * inv); });
            if ((int)threadIdx.x < N) *(float4 *)(s + (size_t)threadIdx.x * pitch + cols) = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
        }
        return;
    }
    for (int j = 0; j < N; ++j)
        for (int k = threadIdx.x; k < pitch; k += 256) s[(size_t)j * pitch + k] = k < cols ? X[(size_t)j * ldx + k] : 0.0f;
}

// Plain products: the block stages the vectors once and its waves walk over groups of RW rows.
// STATS (one product, RW = 4): the block's four waves hold the 16 rows of a tile, and the tile's
// (max, sum of exp) per vector go to part_max / part_sum, which the selection kernel starts from.
// Measured (5 vectors, kernel trace): 50000 x 512 with the statistics 22.6 us (102 MB, 4.5 TB/s), the two products of
// s' (4096 x 1024) 6.3 us.  The five product launches of a decoder step and output layer took 130 us of 176 before (a
// row pair per wave without a second round in flight; a multiply, an add and a conversion of x per entry; 10
// reductions of 18 instructions per row pair), the statistics a launch of 4.8 us; now 73 us for all of it.
struct F32Stats {
    float *part_max;
    double *part_sum;
    int ntiles;
};
template <int N, int RW, int UN, bool STATS, bool GAP>
__global__ __launch_bounds__(256) void gemv_f32_kernel(F32Jobs jobs, F32Stats st)
{
    extern __shared__ __align__(16) float s_x[];
    __shared__ float s_y[STATS ? 16 * N : 1];
    int t = 0;
    while (t + 1 < F32_MAX_JOBS && (int)blockIdx.x >= jobs.nblk[t + 1]) ++t;
    const F32Job &J = jobs.j[t];
    const int blk = blockIdx.x - jobs.nblk[t], nblk = jobs.nblk[t + 1] - jobs.nblk[t];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int cols = J.cols, rows = J.rows, pitch = f32_pitch_of<GAP>(cols);
    __amdgpu_buffer_rsrc_t row[RW];
    F32Regs<RW, UN> R;
    auto request = [&](int r0) {
#pragma unroll
        for (int u = 0; u < RW; ++u) row[u] = f32_row(J.W, r0 + u, rows, J.ld);
        f32_load<RW, UN>(R, row, cols, 0, lane);
    };
    const __amdgpu_buffer_rsrc_t rb = q8_rsrc(J.bias, J.bias ? (size_t)rows * sizeof(float) : 0);
    int r0 = (blk * 4 + wave) * RW;
    F32X<N> X;
    f32_x_load<N>(X, J.X, N * cols, J.flat);
    request(r0);
    f32_x_store<N, N, GAP>(X, s_x, J.X, cols, J.ldx, J.flat);
    __syncthreads();
    // (the trip count is the block's, so that STATS can meet inside: a wave past the last row works on zeros)
    for (int b0 = blk * 4 * RW; b0 < rows; b0 += nblk * 4 * RW) {
        double acc[RW][N];
#pragma unroll
        for (int u = 0; u < RW; ++u)
#pragma unroll
            for (int j = 0; j < N; ++j) acc[u][j] = 0.0;
        // the bias of the sum this lane will store: asked for ahead of everything that it would have to wait behind
        const int idx = wave_sums_index<RW * N>(lane), u = idx / N, j = idx - u * N, rw = r0 + u;
        const bool mine = (lane & 15) < (RW * N + 3) / 4 && idx < RW * N;
        const float bias = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rb, (int)(mine && rw < rows ? (unsigned)rw * 4u : Q8_OOB), 0, 0));
        f32_product<N, RW, UN, GAP>(R, row, s_x, pitch, cols, lane, acc);
        r0 += nblk * 4 * RW;
        request(r0);                                           // the next group's first round, behind the reduction
        double v[RW * N];
#pragma unroll
        for (int e = 0; e < RW * N; ++e) v[e] = acc[e / N][e % N];
        float y = (float)wave_sums_d<RW * N>(v, lane);
        if (J.bias) y = y + bias;
        if (mine && rw < rows) J.Y[(size_t)j * J.ldy + rw] = y;
        if constexpr (STATS) {
            if (mine) s_y[j * 16 + wave * RW + u] = rw < rows ? y : -INFINITY;
            __syncthreads();
            if (tid < 16 * N) {
                // 16 lanes per vector: the tile's maximum, then the sum of e^(logit - maximum)
                const float l = s_y[tid];
                float m = l;
                m = fmaxf(m, __int_as_float(dpp_mov_i<DPP_XOR1>(__float_as_int(m))));
                m = fmaxf(m, __int_as_float(dpp_mov_i<DPP_XOR2>(__float_as_int(m))));
                m = fmaxf(m, __int_as_float(dpp_mov_i<DPP_HALF_MIRROR>(__float_as_int(m))));
                m = fmaxf(m, __int_as_float(dpp_mov_i<DPP_MIRROR>(__float_as_int(m))));
                double e = l > -INFINITY ? (double)exp_le0(l - m) : 0.0;
                e += dpp_mov_d<DPP_XOR1>(e);
                e += dpp_mov_d<DPP_XOR2>(e);
                e += dpp_mov_d<DPP_HALF_MIRROR>(e);
                e += dpp_mov_d<DPP_MIRROR>(e);
                if ((tid & 15) == 0) {
                    const size_t o = (size_t)(tid >> 4) * st.ntiles + b0 / 16;
                    st.part_max[o] = m;
                    st.part_sum[o] = e;
                }
            }
            __syncthreads();
        }
    }
}

// A whole GRU cell (Eq. 1): a wave owns one hidden unit, its three rows of Wx and, unless the recurrent
// pre-activations are given (gh_pre, [n x 3H], bias included), of Wh; the gates follow in the lanes.  Was a
// launch of products, 2 x n x 3H floats written and read back, and a launch of gates: 20.8 + 4.5 us -> 7.3 us
// (512 / 1024 columns, 1024 units, 5 vectors), 7.8 us for 2048 columns with gh_pre.
struct F32GruArgs {
    const float *Wx, *Wh, *bx, *bh, *x, *h_prev, *gh_pre;
    float *h_out;
    int I, H, ldx_w, ldh_w, flat;
};
template <int N, bool GH_PRE, bool GAP>
__global__ __launch_bounds__(256) void gru_f32_kernel(F32GruArgs a)
{
    extern __shared__ __align__(16) float s_x[];
    __shared__ float s_pre[4][6 * N];
    constexpr int UN = GH_PRE ? 4 : 2;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, H = a.H, I = a.I;
    const int unit = __builtin_amdgcn_readfirstlane(blockIdx.x * 4 + wave);
    const int px = f32_pitch_of<GAP>(I), ph = f32_pitch_of<GAP>(H);
    __amdgpu_buffer_rsrc_t rx[3], rh[3];
    F32Regs<3, UN> X, Hh;
#pragma unroll
    for (int g = 0; g < 3; ++g) {
        rx[g] = f32_row(a.Wx, unit < H ? g * H + unit : 3 * H, 3 * H, a.ldx_w);
        if (!GH_PRE) rh[g] = f32_row(a.Wh, unit < H ? g * H + unit : 3 * H, 3 * H, a.ldh_w);
    }
    constexpr int XB = GH_PRE ? 2 * N : N;
    F32X<XB> xv;
    F32X<N> hv;
    f32_x_load<XB>(xv, a.x, N * I, a.flat);
    if (!GH_PRE) f32_x_load<N>(hv, a.h_prev, N * H, a.flat);
    f32_load<3, UN>(X, rx, I, 0, lane);
    if (!GH_PRE) f32_load<3, UN>(Hh, rh, H, 0, lane);
    f32_x_store<N, XB, GAP>(xv, s_x, a.x, I, I, a.flat);
    if (!GH_PRE) f32_x_store<N, N, GAP>(hv, s_x + (size_t)N * px, a.h_prev, H, H, a.flat);
    __syncthreads();
    double acc[3][N];
    auto finish = [&](int base, const float *bias) {
        double v[3 * N];
#pragma unroll
        for (int e = 0; e < 3 * N; ++e) v[e] = acc[e / N][e % N];
        float y = (float)wave_sums_d<3 * N>(v, lane);
        const int idx = wave_sums_index<3 * N>(lane), g = idx / N;
        if ((lane & 15) < (3 * N + 3) / 4 && idx < 3 * N && unit < H) {
            if (bias) y = y + bias[g * H + unit];
            s_pre[wave][base + idx] = y;
        }
    };
#pragma unroll
    for (int e = 0; e < 3 * N; ++e) acc[e / N][e % N] = 0.0;
    f32_product<N, 3, UN, GAP>(X, rx, s_x, px, I, lane, acc);
    finish(0, a.bx);
    if (!GH_PRE) {
#pragma unroll
        for (int e = 0; e < 3 * N; ++e) acc[e / N][e % N] = 0.0;
        f32_product<N, 3, UN, GAP>(Hh, rh, s_x + (size_t)N * px, ph, H, lane, acc);
        finish(3 * N, a.bh);
    }
    __builtin_amdgcn_wave_barrier();                           // a wave reads back its own sums
    if (lane < N && unit < H) {
        float gx[3], gh[3];
#pragma unroll
        for (int g = 0; g < 3; ++g) {
            gx[g] = s_pre[wave][g * N + lane];
            gh[g] = GH_PRE ? a.gh_pre[(size_t)lane * 3 * H + g * H + unit] : s_pre[wave][3 * N + g * N + lane];
        }
        a.h_out[(size_t)lane * H + unit] = gru_gates(gx, gh, a.h_prev[(size_t)lane * H + unit]);
    }
}

// t = tanh(((W_s s + W_y y) + W_c c) + b_t) (first layer of g, Eq. 2): a wave owns one unit and the three
// rows that meet in it.  Was a launch of three products and a launch that added them up: 20.8 + 4.8 us -> 7.3 us.
struct F32ReadoutArgs {
    const float *W[3], *x[3], *b_t;
    float *t_out;
    int cols[3], ld[3], R, flat;
};
template <int N, bool GAP>
__global__ __launch_bounds__(256) void readout_f32_kernel(F32ReadoutArgs a)
{
    extern __shared__ __align__(16) float s_x[];
    __shared__ float s_pre[4][3 * N];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int unit = __builtin_amdgcn_readfirstlane(blockIdx.x * 4 + wave);
    __amdgpu_buffer_rsrc_t row[3][1];
    F32Regs<1, 4> R[3];
    F32X<N> x0, x1;
    F32X<2 * N> x2;
    f32_x_load<N>(x0, a.x[0], N * a.cols[0], a.flat);
    f32_x_load<N>(x1, a.x[1], N * a.cols[1], a.flat);
    f32_x_load<2 * N>(x2, a.x[2], N * a.cols[2], a.flat);
#pragma unroll
    for (int m = 0; m < 3; ++m) {
        row[m][0] = f32_row(a.W[m], unit, a.R, a.ld[m]);
        f32_load<1, 4>(R[m], row[m], a.cols[m], 0, lane);
    }
    const int p0 = f32_pitch_of<GAP>(a.cols[0]), p1 = f32_pitch_of<GAP>(a.cols[1]);
    f32_x_store<N, N, GAP>(x0, s_x, a.x[0], a.cols[0], a.cols[0], a.flat);
    f32_x_store<N, N, GAP>(x1, s_x + (size_t)N * p0, a.x[1], a.cols[1], a.cols[1], a.flat);
    f32_x_store<N, 2 * N, GAP>(x2, s_x + (size_t)N * (p0 + p1), a.x[2], a.cols[2], a.cols[2], a.flat);
    __syncthreads();
    double v[3 * N];
    float *s = s_x;
#pragma unroll
    for (int m = 0; m < 3; ++m) {
        const int pitch = f32_pitch_of<GAP>(a.cols[m]);
        double acc[1][N];
#pragma unroll
        for (int j = 0; j < N; ++j) acc[0][j] = 0.0;
        f32_product<N, 1, 4, GAP>(R[m], row[m], s, pitch, a.cols[m], lane, acc);
#pragma unroll
        for (int j = 0; j < N; ++j) v[m * N + j] = acc[0][j];
        s += (size_t)N * pitch;
    }
    const float y = (float)wave_sums_d<3 * N>(v, lane);
    const int idx = wave_sums_index<3 * N>(lane);
    if ((lane & 15) < (3 * N + 3) / 4 && idx < 3 * N) s_pre[wave][idx] = y;
    __builtin_amdgcn_wave_barrier();
    if (lane < N && unit < a.R) {
        float p = s_pre[wave][lane] + s_pre[wave][N + lane];
        p = p + s_pre[wave][2 * N + lane];
        if (a.b_t) p = p + a.b_t[unit];
        a.t_out[(size_t)lane * a.R + unit] = tanh_rn(p);
    }
}

// =================================================================== host launchers ==

// whether the vectors of a launch are one run of whole 16-byte pieces
static bool f32_flat(const float *X, int n, int cols, int ldx) { return ((uintptr_t)X & 15) == 0 && cols % 4 == 0 && (n == 1 || ldx == cols); }

// Dynamic LDS above 64 KB has to be asked for once per kernel and device; asking again costs a call.
static bool f32_lds(const void *kernel, size_t smem)
{
    if (smem <= 65536) return true;
    if (hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem) == hipSuccess) return true;
    (void)hipGetLastError();
    return false;
}
#define F32_MAX_LDS (150 * 1024)

#define F32_FOR_N(n, M) \
    switch (n) {        \
    case 1: M(1); break; case 2: M(2); break; case 3: M(3); break; case 4: M(4); break; \
    case 5: M(5); break; case 6: M(6); break; case 7: M(7); break; default: M(8); break; \
    }

q8_status q8i_gemv_f32(q8_ctx *ctx, const q8i_f32_job *d, int njobs, int n, float *part_max, double *part_sum)
{
    F32Jobs jobs;
    F32Stats st = {part_max, part_sum, q8i_out_tiles(d[0].W->rows)};
    int blocks = 0, max_pitch = 0;
    bool gap = false;
    long long rows = 0;
    for (int t = 0; t < njobs; ++t) rows += d[t].W->rows;
    // Rows per wave: what fills the chip's 1024 SIMDs first (a wave's loads in flight are the same 8 either way),
    // then what halves the reads of x from LDS.  The statistics need the 16 rows of a tile in one block.
    const int rw = part_max || rows >= 8192 ? 4 : rows >= 2048 ? 2 : 1;
    for (int t = 0; t < F32_MAX_JOBS; ++t) {
        const q8i_f32_job &q = d[t < njobs ? t : 0];
        jobs.j[t] = {q.W->data, q.X, q.bias, q.Y, q.W->rows, q.W->cols, q.W->ld, q.ldx, q.ldy, f32_flat(q.X, n, q.W->cols, q.ldx)};
        jobs.nblk[t] = blocks;
        if (t < njobs) {
            int b = (q.W->rows + 4 * rw - 1) / (4 * rw);
            // (more blocks than are resident together only stage the vectors more often)
            if (b > 1024) b = 1024;
            blocks += b;
            if (f32_pitch(q.W->cols) > max_pitch) max_pitch = f32_pitch(q.W->cols);
            gap = gap || q.W->cols % 256;
        }
    }
    jobs.nblk[F32_MAX_JOBS] = blocks;
    for (int t = njobs; t < F32_MAX_JOBS; ++t) jobs.nblk[t] = blocks;
    const size_t smem = (size_t)n * max_pitch * sizeof(float);
#define F32_GEMV_G(K, G)                                                                                                    \
    (part_max ? gemv_f32_kernel<K, 4, 2, true, G> : rw == 4 ? gemv_f32_kernel<K, 4, 2, false, G>                            \
     : rw == 2 ? gemv_f32_kernel<K, 2, 4, false, G> : gemv_f32_kernel<K, 1, 8, false, G>)
#define F32_GEMV(K)                                                                                                        \
    do {                                                                                                                   \
        void (*kern)(F32Jobs, F32Stats) = gap ? F32_GEMV_G(K, true) : F32_GEMV_G(K, false);                                \
        if (!f32_lds((const void *)kern, smem)) return q8_fail(ctx, Q8_ERR_DEVICE, "32-bit product: %zu bytes of LDS refused", smem); \
        Q8_LAUNCH(ctx, Q8_KERNEL_GEMV, kern, dim3(blocks), dim3(256), smem, jobs, st);                                     \
    } while (0)
    F32_FOR_N(n, F32_GEMV)
    return q8i_launch_check(ctx, "gemv_f32");
}

// A kernel that reads a vector in all its blocks must not write its result over it; where a caller asked for that,
// products and the element-wise part are separate launches.
static bool f32_apart(const float *out, size_t out_n, const float *in, size_t in_n) { return out + out_n <= in || in + in_n <= out; }

bool q8i_gru_f32_ok(const q8_gru_weights_f32 *g, bool gh_pre, const float *x, const float *h_prev, const float *h_out, int n)
{
    const size_t I = g->Wx.cols, H = g->Wh.cols;
    if (((size_t)n * (((I + 3) & ~3) + (gh_pre ? 0 : ((H + 3) & ~3)))) * 4 > F32_MAX_LDS) return false;
    // (with gh_pre the previous state is read by the thread that writes the new one)
    return f32_apart(h_out, n * H, x, n * I) && (gh_pre || f32_apart(h_out, n * H, h_prev, n * H));
}

q8_status q8i_gru_f32(q8_ctx *ctx, const q8_gru_weights_f32 *g, const float *x, const float *h_prev, const float *gh_pre,
                      float *h_out, int n)
{
    const int I = g->Wx.cols, H = g->Wh.cols;
    const bool flat = f32_flat(x, n, I, I) && (gh_pre || f32_flat(h_prev, n, H, H));
    const F32GruArgs a = {g->Wx.data, g->Wh.data, g->bx, g->bh, x, h_prev, gh_pre, h_out, I, H, g->Wx.ld, g->Wh.ld, flat};
    const size_t smem = (size_t)n * (f32_pitch(I) + (gh_pre ? 0 : f32_pitch(H))) * sizeof(float);
    const dim3 grid((H + 3) / 4);
    const bool gap = I % 256 || (!gh_pre && H % 256);
#define F32_GRU(K)                                                                                                          \
    do {                                                                                                                    \
        void (*kern)(F32GruArgs) = gap ? (gh_pre ? gru_f32_kernel<K, true, true> : gru_f32_kernel<K, false, true>)          \
                                       : (gh_pre ? gru_f32_kernel<K, true, false> : gru_f32_kernel<K, false, false>);       \
        if (!f32_lds((const void *)kern, smem)) return q8_fail(ctx, Q8_ERR_DEVICE, "32-bit GRU kernel: %zu bytes of LDS refused", smem); \
        Q8_LAUNCH(ctx, Q8_KERNEL_GRU, kern, grid, dim3(256), smem, a);                                                      \
    } while (0)
    F32_FOR_N(n, F32_GRU)
    return q8i_launch_check(ctx, "gru_f32");
}

bool q8i_readout_f32_ok(const q8_readout_weights_f32 *ro, const float *s, const float *y, const float *c, const float *t_out, int n)
{
    const size_t H = ro->W_s.cols, E = ro->W_y.cols, C = ro->W_c.cols, R = ro->W_s.rows;
    if ((size_t)n * (((H + 3) & ~3) + ((E + 3) & ~3) + ((C + 3) & ~3)) * 4 > F32_MAX_LDS) return false;
    return f32_apart(t_out, n * R, s, n * H) && f32_apart(t_out, n * R, y, n * E) && f32_apart(t_out, n * R, c, n * C);
}

q8_status q8i_readout_f32(q8_ctx *ctx, const q8_readout_weights_f32 *ro, const float *s, const float *y, const float *c, float *t_out, int n)
{
    const q8_matf *W[3] = {&ro->W_s, &ro->W_y, &ro->W_c};
    const float *x[3] = {s, y, c};
    F32ReadoutArgs a;
    size_t smem = 0;
    bool gap = false;
    a.flat = 1;
    for (int m = 0; m < 3; ++m) {
        a.W[m] = W[m]->data; a.x[m] = x[m]; a.cols[m] = W[m]->cols; a.ld[m] = W[m]->ld;
        a.flat &= f32_flat(x[m], n, W[m]->cols, W[m]->cols);
        gap = gap || W[m]->cols % 256;
        smem += (size_t)n * f32_pitch(W[m]->cols) * sizeof(float);
    }
    a.b_t = ro->b_t; a.t_out = t_out; a.R = ro->W_s.rows;
    const dim3 grid((a.R + 3) / 4);
#define F32_READOUT(K)                                                                                                      \
    do {                                                                                                                    \
        void (*kern)(F32ReadoutArgs) = gap ? readout_f32_kernel<K, true> : readout_f32_kernel<K, false>;                    \
        if (!f32_lds((const void *)kern, smem)) return q8_fail(ctx, Q8_ERR_DEVICE, "32-bit readout kernel: %zu bytes of LDS refused", smem); \
        Q8_LAUNCH(ctx, Q8_KERNEL_READOUT, kern, grid, dim3(256), smem, a);                                                  \
    } while (0)
    F32_FOR_N(n, F32_READOUT)
    return q8i_launch_check(ctx, "readout_f32");
}
