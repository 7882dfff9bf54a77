// q8_gemm.hip -- the 8-bit product of Section 3 for panels of more than 8 vectors (source
// positions of one sentence, or the hypotheses of many sentences decoded together, which
// Section 6 names as the next step): a blocked int8 GEMM on the gfx950 matrix cores.
// The arithmetic is that of the streaming kernels: per-vector activation codes, exact
// int32 sums, one fp32 scale product, separate bias addition.
#include "q8_internal.h"
#include "q8_index.h"
#include "q8_gemm_resident.h"
#include "q8_route.h"

// Block tiles (row tiles per wave, vector tiles): matrices of more than 8192 rows (the
// vocabulary) and the rest.
#ifndef GB_BIG_RT
#define GB_BIG_RT 2
#define GB_BIG_NT 8
#endif
#ifndef GB_SMALL_RT
#define GB_SMALL_RT 1
#define GB_SMALL_NT 4
#endif
typedef int v16i __attribute__((ext_vector_type(16)));

#define GB_K 128           // k bytes per stage
#define GB_PITCH 144       // LDS bytes per staged vector: 16 lanes x 16 bytes fall on 64 distinct banks

// Block tile: 64 RT rows x 16 NT vectors, four waves, wave w owns row tiles w RT .. w RT + RT - 1.
// The vectors' codes go through LDS (every wave multiplies the same ones), double-buffered,
// one barrier per stage; each wave reads its own weight rows straight from memory, one stage
// ahead.  v_mfma_i32_16x16x64_i8 operands: A = 16 weight rows x 64 k (lane: row lane % 16,
// k bytes 16 (lane / 16) .. + 15), B = the same split for 16 vectors; result: lane holds rows
// 4 (lane / 16) + r, r = 0..3, of vector lane % 16.
template <int RT, int NT, bool STATS>
__global__ __launch_bounds__(256) void gemm_block_kernel(GemmJobs jobs)
{
    const int bx = blockIdx.x, by = blockIdx.y, bz = blockIdx.z;
    const GemmArgs &a = jobs.j[bz];
    constexpr int BN = 16 * NT;
    if (bx * 64 * RT >= a.rows) return;                  // the grid is sized for the largest job
    constexpr int PIECES = BN * (GB_K / 16) / 256;      // 16-byte pieces of a stage per thread
    __shared__ __align__(16) int8_t s_b[2][BN * GB_PITCH];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int i = lane & 15, g = lane >> 4;
    const int r0 = (bx * 4 + wave) * 16 * RT;
    const int c0 = by * BN;
    const int ld = a.ld, n = a.n, rows = a.rows;

    // Every load below is unconditional and in bounds (rows, vectors and k offsets are clamped);
    // what lies outside the matrix is replaced by zeros when a stage is consumed.  That keeps the
    // number of loads per step fixed, so that waiting for one stage leaves the later ones in flight.
    const int8_t *wp[RT];
    bool row_ok[RT];
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) {
        const int row = r0 + 16 * rt + i;
        row_ok[rt] = row < rows;
        wp[rt] = a.W + (size_t)(row_ok[rt] ? row : rows - 1) * ld;
        if (a.Wt) {            // this lane's 16 bytes of the row tile's first k step (tiles past the matrix: the last one, dropped below)
            const int tile = min((r0 + 16 * rt) >> 4, a.ntiles - 1);
            wp[rt] = a.Wt + (size_t)tile * (ld >> 6) * 1024 + lane * 16;
        }
    }
    const bool tiled = a.Wt != nullptr;
    const int kc_last = (ld >> 6) - 1;
    const int8_t *bp_g[PIECES];
    bool col_ok[PIECES];
#pragma unroll
    for (int u = 0; u < PIECES; ++u) {
        const int col = c0 + ((u * 256 + tid) >> 3);
        col_ok[u] = col < n;
        bp_g[u] = a.xq + (size_t)(col_ok[u] ? col : n - 1) * ld;
    }
    const int kb = (tid & 7) * 16;            // k offset of this thread's pieces within a stage
    const int klast = ld - 16;

    // Software pipeline over stages of GB_K k bytes, loads two stages ahead: while stage s is
    // multiplied out of LDS, stage s + 1 sits in one register set (or is still arriving) and
    // stage s + 2 is in flight into the other.
    struct Stage {
        v4i b[PIECES];       // this thread's pieces of the vectors' codes
        v4i a[RT][2];        // this lane's weight operands
    };
    Stage R0, R1;
    v4i acur[RT][2];
    const v4i zero4 = (v4i){0, 0, 0, 0};
    auto load_stage = [&](Stage &R, int k0) {
        const int kB = min(k0 + kb, klast);
#pragma unroll
        for (int u = 0; u < PIECES; ++u) R.b[u] = *(const v4i *)(bp_g[u] + kB);
#pragma unroll
        for (int kc = 0; kc < 2; ++kc) {
            const int kA = tiled ? min((k0 >> 6) + kc, kc_last) * 1024 : min(k0 + 64 * kc + 16 * g, klast);
#pragma unroll
            for (int rt = 0; rt < RT; ++rt) R.a[rt][kc] = *(const v4i *)(wp[rt] + kA);
        }
    };
    auto store_stage = [&](const Stage &R, int buf, int k0) {
        const bool kB_ok = k0 + kb < ld;
#pragma unroll
        for (int u = 0; u < PIECES; ++u) {
            const int p = u * 256 + tid;
            *(v4i *)(s_b[buf] + (p >> 3) * GB_PITCH + (p & 7) * 16) = (col_ok[u] && kB_ok) ? R.b[u] : zero4;
        }
#pragma unroll
        for (int kc = 0; kc < 2; ++kc) {
            const bool kA_ok = k0 + 64 * kc + 16 * g < ld;
#pragma unroll
            for (int rt = 0; rt < RT; ++rt) acur[rt][kc] = (row_ok[rt] && kA_ok) ? R.a[rt][kc] : zero4;
        }
    };

    v4i acc[RT][NT];
#pragma unroll
    for (int rt = 0; rt < RT; ++rt)
#pragma unroll
        for (int t = 0; t < NT; ++t) acc[rt][t] = zero4;

    const int nst = (ld + GB_K - 1) / GB_K;
    load_stage(R0, 0);
    load_stage(R1, GB_K);                      // past the last stage: a clamped, unused reload
    store_stage(R0, 0, 0);
    load_stage(R0, 2 * GB_K);
    __syncthreads();
    // step s: multiply stage s (LDS buffer s & 1), move stage s + 1 from Rn to the other buffer,
    // which was last read before the previous barrier, and reuse Rn for stage s + 3
    auto step = [&](Stage &Rn, int s) {
        const int8_t *bp = s_b[s & 1] + i * GB_PITCH + 16 * g;
        v4i av[RT][2];
#pragma unroll
        for (int rt = 0; rt < RT; ++rt)
#pragma unroll
            for (int kc = 0; kc < 2; ++kc) av[rt][kc] = acur[rt][kc];
        store_stage(Rn, (s + 1) & 1, (s + 1) * GB_K);
        load_stage(Rn, (s + 3) * GB_K);
#pragma unroll
        for (int kc = 0; kc < 2; ++kc)
#pragma unroll
            for (int t = 0; t < NT; ++t) {
                const v4i bv = *(const v4i *)(bp + t * 16 * GB_PITCH + 64 * kc);
#pragma unroll
                for (int rt = 0; rt < RT; ++rt)
                    acc[rt][t] = __builtin_amdgcn_mfma_i32_16x16x64_i8(av[rt][kc], bv, acc[rt][t], 0, 0, 0);
            }
        __syncthreads();
    };
    int s = 0;
    for (; s + 1 < nst; s += 2) {                // always both halves: the load counts per path stay fixed
        step(R1, s);
        step(R0, s + 1);
    }
    if (s < nst) step(R1, s);

    // Epilogue, written so that the loads and the cross-lane steps of all NT tiles of a row tile
    // are issued together instead of one tile after the other.
    const bool vec_ok = ((a.ldy & 3) == 0) && (((uintptr_t)a.Y & 15) == 0);
    const bool bias_vec = (((uintptr_t)a.bias) & 15) == 0;
    float cs[NT], xs[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t) {
        const int col = c0 + 16 * t + i;
        xs[t] = col < n ? a.xscale[col] : 0.0f;
        cs[t] = a.w_scale * xs[t];
    }
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) {
        const int row0 = r0 + 16 * rt + 4 * g;
        if (r0 + 16 * rt >= rows) continue;              // wave-uniform
        float4 b = make_float4(0.f, 0.f, 0.f, 0.f);
        if (a.bias) {
            if (bias_vec && row0 + 3 < rows) {
                b = *(const float4 *)(a.bias + row0);
            } else {
                if (row0 < rows) b.x = a.bias[row0];
                if (row0 + 1 < rows) b.y = a.bias[row0 + 1];
                if (row0 + 2 < rows) b.z = a.bias[row0 + 2];
                if (row0 + 3 < rows) b.w = a.bias[row0 + 3];
            }
        }
        float rsv[4] = {0.f, 0.f, 0.f, 0.f};
        if (a.row_scale) {
#pragma unroll
            for (int r = 0; r < 4; ++r) rsv[r] = a.row_scale[min(row0 + r, rows - 1)];
        }
        float y[NT][4], m[NT];
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            const int col = c0 + 16 * t + i;
            const bool col_ok = col < n;
            m[t] = -INFINITY;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                y[t][r] = -INFINITY;
                if (col_ok && row0 + r < rows) {
                    y[t][r] = (float)acc[rt][t][r] * (a.row_scale ? rsv[r] * xs[t] : cs[t]);
                    if (a.bias) y[t][r] = y[t][r] + (r == 0 ? b.x : r == 1 ? b.y : r == 2 ? b.z : b.w);
                    if (a.tap_acc) a.tap_acc[(size_t)col * rows + row0 + r] = acc[rt][t][r];
                }
                m[t] = fmaxf(m[t], y[t][r]);
            }
            if (a.tiled) {
                // rows past the matrix carry -inf; whoever reads the tile skips them
                if (col_ok)
                    *(float4 *)(a.Y + ((size_t)((r0 + 16 * rt) >> 4) * n + col) * 16 + 4 * g) =
                        make_float4(y[t][0], y[t][1], y[t][2], y[t][3]);
            } else if (col_ok) {
                if (vec_ok && row0 + 3 < rows) {
                    *(float4 *)(a.Y + (size_t)col * a.ldy + row0) = make_float4(y[t][0], y[t][1], y[t][2], y[t][3]);
                } else {
#pragma unroll
                    for (int r = 0; r < 4; ++r)
                        if (row0 + r < rows) a.Y[(size_t)col * a.ldy + row0 + r] = y[t][r];
                }
            }
        }
        if (STATS) {
            // (max, sum of exp) of the tile's 16 rows per vector: lanes i, i+16, i+32, i+48
#pragma unroll
            for (int t = 0; t < NT; ++t)
                m[t] = fmaxf(m[t], __int_as_float(__builtin_amdgcn_ds_swizzle(__float_as_int(m[t]), SWZ_XOR16)));
#pragma unroll
            for (int t = 0; t < NT; ++t) m[t] = fmaxf(m[t], __shfl_xor(m[t], 32, 64));
            double sd[NT];
#pragma unroll
            for (int t = 0; t < NT; ++t) {
                sd[t] = 0.0;
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    if (y[t][r] > -INFINITY) sd[t] += (double)exp_le0(y[t][r] - m[t]);
            }
#pragma unroll
            for (int t = 0; t < NT; ++t) sd[t] += __shfl_xor(sd[t], 16, 64);
#pragma unroll
            for (int t = 0; t < NT; ++t) sd[t] += __shfl_xor(sd[t], 32, 64);
            const int tile = (r0 + 16 * rt) >> 4;
#pragma unroll
            for (int t = 0; t < NT; ++t) {
                const int col = c0 + 16 * t + i;
                if (col < n && g == 0) {
                    a.part_max[(size_t)col * a.ntiles + tile] = m[t];
                    a.part_sum[(size_t)col * a.ntiles + tile] = sd[t];
                }
            }
        }
    }
}

// ===================================================================== large panels ==
// Plain products over many vectors: block tile 32 RW rows x 32 CW CT vectors, four waves (RW x CW), a wave 32 rows x 32 CT
// vectors of v_mfma_i32_32x32x32_i8 results.  The tile is as large as still gives most compute units a block, so that a
// unit, which takes in some 77 GB/s, asks for few bytes (that is not all of it: 1024 x 2048 x 1024 with 64 x 64 tiles asks
// for 256 KB per unit, 3.4 us, and multiplies for 1.8 of its 10.7 us; what the rest goes into is not known).  k runs in
// stages of 256 bytes, and stages s + 1 and s + 2 are on
// their way while s is multiplied: a vector piece's register is requested again once it is in LDS, a weight register
// once its instruction has used it.  One barrier per stage (two LDS buffers).  Weights come tile-packed or row by row;
// everything outside the matrix or the panel reads as zero through bounds-checked descriptors.
// Measured (kernel trace), 1000 vectors: products of 512 + 1024 bytes and 3072 rows each 19.7 (K-resident) -> 17.4 us,
// the readout's three 17.4 (staged) -> 11.9, rows of 2048 bytes times 3072 17.4 -> 17; 1024 x 2048 x 1024 12.8 -> 10.7.
template <int RW, int CW, int CT>
__global__ __launch_bounds__(256, 2) void gemm_tile_kernel(GemmJobs jobs)
{
    static_assert(RW * CW == 4, "four waves");
    constexpr int ROWS = 32 * RW, COLS = 32 * CW * CT, KB = 256, PITCH = KB + 16, PB = COLS * (KB / 16) / 256;
    extern __shared__ __align__(16) int8_t s_t[];        // [2][COLS x PITCH]
    const GemmArgs &a = jobs.j[blockIdx.z];
    if ((int)blockIdx.x * ROWS >= a.rows) return;        // the grid is sized for the largest job
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int i = lane & 31, h = lane >> 5;
    const int wr = wave / CW, wc = wave - wr * CW;
    const int r0 = (int)blockIdx.x * ROWS + 32 * wr, c0 = (int)blockIdx.y * COLS;
    const int ld = a.ld, n = a.n, rows = a.rows, nst = (ld + KB - 1) / KB;
    const bool tiled = a.Wt != nullptr;
    const __amdgpu_buffer_rsrc_t rx = q8_rsrc(a.xq, (size_t)n * ld);
    const __amdgpu_buffer_rsrc_t rw = tiled ? q8_rsrc(a.Wt, (size_t)a.ntiles * 16 * ld) : q8_rsrc(a.W, (size_t)rows * ld);
    // weights: lane (row i, k half h) of k step m of stage s holds bytes 256 s + 32 m + 16 h .. of row r0 + i
    const int row = r0 + i;
    const unsigned wbase = tiled ? (unsigned)(row >> 4) * (unsigned)(ld >> 6) * 1024u + (unsigned)h * 256u + (unsigned)(i & 15) * 16u
                                 : (unsigned)row * (unsigned)ld + 16u * h;
    auto load_a = [&](int st, int m) {
        const int k = KB * st + 32 * m;
        const unsigned off = row < rows && k + 16 * h < ld ? wbase + (tiled ? (unsigned)(k >> 6) * 1024u + (unsigned)((k >> 5) & 1) * 512u : (unsigned)k) : Q8_OOB;
        return __builtin_bit_cast(v4i, __builtin_amdgcn_raw_buffer_load_b128(rw, (int)off, 0, 0));
    };
    // vectors: thread's piece u of a stage is piece (tid % 16) of vector u * 16 + tid / 16
    const int bcol = tid >> 4, bpc = (tid & 15) * 16;
    auto load_b = [&](v4i (&b)[PB], int st) {
        const int k = KB * st + bpc;
#pragma unroll
        for (int u = 0; u < PB; ++u) {
            const int col = c0 + u * 16 + bcol;
            b[u] = __builtin_bit_cast(v4i, __builtin_amdgcn_raw_buffer_load_b128(rx, (int)(col < n && k < ld ? (unsigned)col * (unsigned)ld + (unsigned)k : Q8_OOB), 0, 0));
        }
    };
    v4i A0[8], A1[8], B0[PB], B1[PB];
    load_b(B0, 0);
#pragma unroll
    for (int m = 0; m < 8; ++m) A0[m] = load_a(0, m);
    load_b(B1, 1);
#pragma unroll
    for (int m = 0; m < 8; ++m) A1[m] = load_a(1, m);
    v16i acc[CT];
#pragma unroll
    for (int t = 0; t < CT; ++t) acc[t] = (v16i){};
    auto step = [&](v4i (&A)[8], v4i (&B)[PB], int st) {
        int8_t *buf = s_t + (st & 1) * COLS * PITCH;
#pragma unroll
        for (int u = 0; u < PB; ++u) *(v4i *)(buf + (u * 16 + bcol) * PITCH + bpc) = B[u];
        load_b(B, st + 2);
        __syncthreads();
        const int8_t *bp = buf + (32 * CT * wc + i) * PITCH + 16 * h;
#pragma unroll
        for (int m = 0; m < 8; ++m) {
#pragma unroll
            for (int t = 0; t < CT; ++t)
                acc[t] = __builtin_amdgcn_mfma_i32_32x32x32_i8(A[m], *(const v4i *)(bp + 32 * t * PITCH + 32 * m), acc[t], 0, 0, 0);
            A[m] = load_a(st + 2, m);
        }
    };
    for (int st = 0; st < nst; st += 2) {
        step(A0, B0, st);
        if (st + 1 < nst) step(A1, B1, st + 1);
    }
    // result r of the lane: row r0 + 8 (r / 4) + 4 h + r % 4 of vector c0 + 32 (CT wc + t) + i
    const __amdgpu_buffer_rsrc_t rs = q8_rsrc(a.xscale, (size_t)n * sizeof(float));
    const __amdgpu_buffer_rsrc_t rb = q8_rsrc(a.bias, a.bias ? (size_t)rows * sizeof(float) : 0);
    const __amdgpu_buffer_rsrc_t rr = q8_rsrc(a.row_scale, a.row_scale ? (size_t)rows * sizeof(float) : 0);
    const bool vec_ok = ((a.ldy & 3) == 0) && (((uintptr_t)a.Y & 15) == 0);
    float bias[16], xs[CT], rsv[16];
#pragma unroll
    for (int t = 0; t < CT; ++t) xs[t] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rs, (c0 + 32 * (CT * wc + t) + i) * 4, 0, 0));
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        const int off = (r0 + 8 * (r >> 2) + 4 * h + (r & 3)) * 4;
        bias[r] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rb, off, 0, 0));
        rsv[r] = a.row_scale ? __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rr, off, 0, 0)) : a.w_scale;
    }
#pragma unroll
    for (int t = 0; t < CT; ++t) {
        const int col = c0 + 32 * (CT * wc + t) + i;
        if (col >= n) continue;
        float *y = a.Y + (size_t)col * a.ldy;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int row4 = r0 + 8 * q + 4 * h;
            float v[4];
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                v[r] = (float)acc[t][4 * q + r] * (rsv[4 * q + r] * xs[t]);
                if (a.bias) v[r] = v[r] + bias[4 * q + r];
            }
            if (vec_ok && row4 + 3 < rows) *(float4 *)(y + row4) = make_float4(v[0], v[1], v[2], v[3]);
            else {
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    if (row4 + r < rows) y[row4 + r] = v[r];
            }
        }
    }
}

// ===================================================== three products, k split over waves ==
// The readout's three partial products (Eq. 2's first layer: W_s q(s), W_y q(y), W_c q(H_t), 512 rows
// each, rows of 1024 / 512 / 2048 bytes) for a panel of slots in one K-resident launch.  The block
// kernel above needs ten staged steps for the longest rows and fills 120 blocks (10 us); here block
// (rg, cg) owns rows 32 rg .. 32 rg + 31 of all three matrices and slots 32 cg .. 32 cg + 31, whose codes
// for all three products sit in LDS (3632 bytes per slot), and the 3584 k bytes are cut into seven
// chunks of 512: wave (ut, chunk) multiplies one tile of 16 rows over one chunk against the two slot
// tiles, every load requested up front.  The exact int32 partial sums of a product's chunks meet in LDS
// and are dequantized once, as the block kernel does it.  Rows of other lengths take the block kernel.
#define KS3_ROWS 32
#define KS3_SLOTS 32
#define KS3_WAVES 14
struct Ksplit3Args {
    const int8_t *W[3], *Wt[3];    // [R x ld], and tile-packed or NULL
    const int8_t *xq[3];           // codes [n x ld]
    const float *xs[3];            // [n]
    float *Y[3];                   // [n x ldy]
    float w_scale[3];
    int R, n, ldy;
};

__global__ __launch_bounds__(64 * KS3_WAVES) void gemm_ksplit3_kernel(Ksplit3Args a)
{
    extern __shared__ __align__(16) int8_t s_k3[];
    constexpr int NT = 64 * KS3_WAVES;
    constexpr int LD0 = 1024, LD1 = 512, LD2 = 2048;
    constexpr int P0 = LD0 + 16, P1 = LD1 + 16, P2 = LD2 + 16;           // LDS pitches
    int8_t *s_x0 = s_k3, *s_x1 = s_x0 + KS3_SLOTS * P0, *s_x2 = s_x1 + KS3_SLOTS * P1;
    int *s_e = (int *)(s_x2 + KS3_SLOTS * P2);                           // [14 waves][2 slot tiles][16 slots][16 rows]
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int i = lane & 15, g = lane >> 4;
    const int rg = blockIdx.x, cg = blockIdx.y, n = a.n, c0 = cg * KS3_SLOTS, r0 = rg * KS3_ROWS;

    // ---- all loads up front (outside the arrays: zero) ----
    constexpr int U0 = (KS3_SLOTS * LD0 / 16 + NT - 1) / NT, U1 = (KS3_SLOTS * LD1 / 16 + NT - 1) / NT, U2 = (KS3_SLOTS * LD2 / 16 + NT - 1) / NT;
    const __amdgpu_buffer_rsrc_t rq0 = q8_rsrc(a.xq[0], (size_t)n * LD0), rq1 = q8_rsrc(a.xq[1], (size_t)n * LD1), rq2 = q8_rsrc(a.xq[2], (size_t)n * LD2);
    v4i b0[U0], b1[U1], b2[U2];
#pragma unroll
    for (int u = 0; u < U0; ++u) {
        const int p = u * NT + tid, slot = p / (LD0 / 16), piece = p - slot * (LD0 / 16);
        const unsigned off = (p < KS3_SLOTS * LD0 / 16 && c0 + slot < n) ? (unsigned)(c0 + slot) * LD0 + 16u * piece : Q8_OOB;
        b0[u] = __builtin_bit_cast(v4i, __builtin_amdgcn_raw_buffer_load_b128(rq0, (int)off, 0, 0));
    }
#pragma unroll
    for (int u = 0; u < U1; ++u) {
        const int p = u * NT + tid, slot = p / (LD1 / 16), piece = p - slot * (LD1 / 16);
        const unsigned off = (p < KS3_SLOTS * LD1 / 16 && c0 + slot < n) ? (unsigned)(c0 + slot) * LD1 + 16u * piece : Q8_OOB;
        b1[u] = __builtin_bit_cast(v4i, __builtin_amdgcn_raw_buffer_load_b128(rq1, (int)off, 0, 0));
    }
#pragma unroll
    for (int u = 0; u < U2; ++u) {
        const int p = u * NT + tid, slot = p / (LD2 / 16), piece = p - slot * (LD2 / 16);
        const unsigned off = (p < KS3_SLOTS * LD2 / 16 && c0 + slot < n) ? (unsigned)(c0 + slot) * LD2 + 16u * piece : Q8_OOB;
        b2[u] = __builtin_bit_cast(v4i, __builtin_amdgcn_raw_buffer_load_b128(rq2, (int)off, 0, 0));
    }
    // this wave: row tile ut, chunk ch -> product j, first k byte kbase
    const int ut = wave / 7, ch = wave % 7;
    const int j = ch < 2 ? 0 : ch == 2 ? 1 : 2;
    const int kbase = 512 * (ch < 2 ? ch : ch == 2 ? 0 : ch - 3);
    const int ldw = j == 0 ? LD0 : j == 1 ? LD1 : LD2;
    const int8_t *wt = a.Wt[j];
    const __amdgpu_buffer_rsrc_t rw = q8_rsrc(wt ? wt : a.W[j], (size_t)a.R * ldw);
    const int row0 = r0 + 16 * ut;                                       // R % 32 == 0: a whole tile inside the matrix
    v4i av[8];
#pragma unroll
    for (int s = 0; s < 8; ++s) {
        unsigned off = (unsigned)(row0 + i) * (unsigned)ldw + (unsigned)(kbase + 64 * s + 16 * g);
        if (wt) off = (((unsigned)(row0 >> 4) * (unsigned)(ldw >> 6) + (unsigned)((kbase >> 6) + s)) << 10) + 16u * lane;
        av[s] = __builtin_bit_cast(v4i, __builtin_amdgcn_raw_buffer_load_b128(rw, (int)off, 0, 0));
    }
    // dequantization factors of the (slot, row) pairs tid and tid + NT of 32 x 32
    const __amdgpu_buffer_rsrc_t rs0 = q8_rsrc(a.xs[0], (size_t)n * 4), rs1 = q8_rsrc(a.xs[1], (size_t)n * 4), rs2 = q8_rsrc(a.xs[2], (size_t)n * 4);
    float xs[2][3];
#pragma unroll
    for (int e = 0; e < 2; ++e) {
        const int pr = e * NT + tid, col = c0 + (pr >> 5);
        const int off = (int)((pr < KS3_SLOTS * KS3_ROWS && col < n) ? (unsigned)col * 4u : Q8_OOB);
        xs[e][0] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rs0, off, 0, 0));
        xs[e][1] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rs1, off, 0, 0));
        xs[e][2] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rs2, off, 0, 0));
    }
    __builtin_amdgcn_sched_barrier(0);

    // ---- codes into LDS ----
#pragma unroll
    for (int u = 0; u < U0; ++u) {
        const int p = u * NT + tid, slot = p / (LD0 / 16), piece = p - slot * (LD0 / 16);
        if (p < KS3_SLOTS * LD0 / 16) *(v4i *)(s_x0 + slot * P0 + 16 * piece) = b0[u];
    }
#pragma unroll
    for (int u = 0; u < U1; ++u) {
        const int p = u * NT + tid, slot = p / (LD1 / 16), piece = p - slot * (LD1 / 16);
        if (p < KS3_SLOTS * LD1 / 16) *(v4i *)(s_x1 + slot * P1 + 16 * piece) = b1[u];
    }
#pragma unroll
    for (int u = 0; u < U2; ++u) {
        const int p = u * NT + tid, slot = p / (LD2 / 16), piece = p - slot * (LD2 / 16);
        if (p < KS3_SLOTS * LD2 / 16) *(v4i *)(s_x2 + slot * P2 + 16 * piece) = b2[u];
    }
    __syncthreads();

    // ---- products ----
    v4i acc[2] = {(v4i){0, 0, 0, 0}, (v4i){0, 0, 0, 0}};
    {
        const int pitch = j == 0 ? P0 : j == 1 ? P1 : P2;
        const int8_t *bp = (j == 0 ? s_x0 : j == 1 ? s_x1 : s_x2) + i * pitch + kbase + 16 * g;
#pragma unroll
        for (int s = 0; s < 8; ++s)
#pragma unroll
            for (int t = 0; t < 2; ++t) {
                const v4i bv = *(const v4i *)(bp + t * 16 * pitch + 64 * s);
                acc[t] = __builtin_amdgcn_mfma_i32_16x16x64_i8(av[s], bv, acc[t], 0, 0, 0);
            }
    }
    // lane (i, g) holds rows 4 g + r, r = 0..3, of slot i of each tile
#pragma unroll
    for (int t = 0; t < 2; ++t) *(v4i *)(s_e + (((wave * 2 + t) * 16 + i) * 16 + 4 * g)) = acc[t];
    __syncthreads();

    // ---- chunks summed, dequantized, stored: consecutive threads, consecutive rows of a slot ----
#pragma unroll
    for (int e = 0; e < 2; ++e) {
        const int pr = e * NT + tid;
        if (pr >= KS3_SLOTS * KS3_ROWS) break;
        const int c = pr >> 5, r = pr & 31, col = c0 + c;
        const int at = ((c >> 4) * 16 + (c & 15)) * 16 + (r & 15), w0 = (r >> 4) * 7;        // wave (ut, chunk) = 7 ut + chunk
        const int e0 = s_e[(w0 + 0) * 512 + at] + s_e[(w0 + 1) * 512 + at];
        const int e1 = s_e[(w0 + 2) * 512 + at];
        const int e2 = ((s_e[(w0 + 3) * 512 + at] + s_e[(w0 + 4) * 512 + at]) + s_e[(w0 + 5) * 512 + at]) + s_e[(w0 + 6) * 512 + at];
        if (col < n) {
            const size_t o = (size_t)col * a.ldy + r0 + r;
            a.Y[0][o] = (float)e0 * (a.w_scale[0] * xs[e][0]);
            a.Y[1][o] = (float)e1 * (a.w_scale[1] * xs[e][1]);
            a.Y[2][o] = (float)e2 * (a.w_scale[2] * xs[e][2]);
        }
    }
}

// Whether the three products W[u] . xq[u] (no bias, no taps, plain output at pitch ldy) take the kernel above.
bool q8i_gemm_ksplit3_ok(const q8i_gemm_job *d, int n)
{
    const int R = d[0].W->rows;
    if (R % KS3_ROWS || n < 1 || (R / KS3_ROWS) * ((n + KS3_SLOTS - 1) / KS3_SLOTS) > 256) return false;
    static const int want[3] = {1024, 512, 2048};
    for (int u = 0; u < 3; ++u) {
        if (d[u].W->rows != R || d[u].W->ld != want[u] || d[u].bias || d[u].tap_acc || d[u].part_max || d[u].tiled || d[u].row_scale ||
            d[u].ldy != d[0].ldy || (size_t)n * want[u] >= (1u << 31))
            return false;
    }
    return true;
}

q8_status q8i_gemm_ksplit3(q8_ctx *ctx, const q8i_gemm_job *d, int n)
{
    Ksplit3Args a;
    for (int u = 0; u < 3; ++u) {
        a.W[u] = d[u].W->data; a.Wt[u] = d[u].W->tiles; a.xq[u] = d[u].xq; a.xs[u] = d[u].xscale; a.Y[u] = d[u].Y;
        a.w_scale[u] = d[u].W->scale;
    }
    a.R = d[0].W->rows; a.n = n; a.ldy = d[0].ldy;
    const size_t smem = (size_t)KS3_SLOTS * (1024 + 16 + 512 + 16 + 2048 + 16) + (size_t)KS3_WAVES * 2 * 1024;
    static Q8OncePerDevice asked;
    const q8_status st = q8i_lds(ctx, asked, (const void *)gemm_ksplit3_kernel, smem, "three-product kernel");
    if (st) return st;
    Q8_LAUNCH(ctx, Q8_KERNEL_MFMA, gemm_ksplit3_kernel, dim3(a.R / KS3_ROWS, (n + KS3_SLOTS - 1) / KS3_SLOTS), dim3(64 * KS3_WAVES), smem, a);
    return q8i_launch_check(ctx, "three products");
}

// ================================================================ vocabulary panel ==
// The vocabulary product for a panel of hypothesis slots (many sentences side by side).  Unlike
// the block kernel above, a block keeps its share of the vectors' codes in LDS for its whole
// life (up to 160 KB per workgroup on gfx950) and streams tile-packed 16-row weight tiles past
// them, one tile ahead in registers: no barrier after the prologue, every weight byte read once
// per column group.  Per (row tile, column tile): KC matrix-core steps, then dequantize, bias,
// and the tile's (max, sum of exp) per slot with the cross-lane steps on v_permlane16/32_swap.
// The logits themselves are not kept (64 MB per step at 320 slots): the selection computes
// those of the few tiles that can hold one of the k best again.
struct PanelArgs {
    const int8_t *tiles;   // tile-packed weights (q8_pack_tiles)
    const int8_t *xq;      // [n x ld] codes
    const float *xscale, *bias;
    float *part_max;       // [n x ntiles]
    double *part_sum;
    int rows, ld, n, ntiles, cols_per_group, bias_rows;
    float w_scale;
};

#define VP_WAVES Q8_PANEL_WAVES
#define VP_STAGE Q8_PANEL_STAGE

// max of eight values (the plain form costs a canonicalization of every operand)
__device__ __forceinline__ float vp_max8(const float *v)
{
    float a, b, m;
    asm("v_max3_f32 %0, %1, %2, %3" : "=v"(a) : "v"(v[0]), "v"(v[1]), "v"(v[2]));
    asm("v_max3_f32 %0, %1, %2, %3" : "=v"(b) : "v"(v[3]), "v"(v[4]), "v"(v[5]));
    asm("v_max3_f32 %0, %1, %2, %3" : "=v"(m) : "v"(v[6]), "v"(v[7]), "v"(a));
    asm("v_max_f32 %0, %1, %2" : "=v"(a) : "v"(m), "v"(b));
    return a;
}

// Results are 32 rows x 32 slots, one v_mfma_i32_32x32x32_i8 accumulator: a lane then holds 16 rows of ONE slot, eight of
// each of the two 16-row tiles that the selection wants statistics of, so that a tile's maximum and its sum take
// seven steps in the lane and one across the wave's halves (the 16 x 16 form that this replaced spent 126 instructions
// per 16 x 16 results, 8 of them products; vector instructions bound it).  A unit is 64 rows x 32 slots: two
// accumulators keep the matrix core busy and share every operand read from LDS.  A wave takes a run of consecutive
// units, slots first, so that all waves end together whatever the number of rows; while it multiplies the last
// slots of its rows, every weight register it has used is refilled from its next rows, so the weights need no second
// set of registers and no wait of their own.
// Waves are not held in step: one wave's products run beside the other's statistics (a barrier per unit, with whole
// 64-byte lines of statistics leaving the block together, cost 8 of 43 us at 1000 slots).  A unit's statistics go
// through LDS all the same, so that a slot's four tiles leave as 16 and 32 contiguous bytes: every lane storing its own
// 4 and 8 bytes, into rows 12 and 25 KB apart, took 10 of 45 us.
// 50000 x 512 (kernel trace): 25 us at 320 slots, 55 us at 1000 with 16 x 16 results -> 18.5 / 41.2 us -> 17.8 / 38.0 with
// everything that goes to LDS requested at once, rows past the matrix masked by their biases instead of sixteen selects
// (the block that has them ended 3 us after the others) and longer runs for the waves that are served first; 40001 rows at
// 600 slots 43 -> 31.6 us; 50294 rows of 640 bytes at 320 slots 31 -> 21.3 us.  At 1000 slots, us after the first block
// starts: codes and weights there 5.6 (256 KB per compute unit), waves done 31 to 38; a unit of 2000 clocks per SIMD is 1024 of
// products and some 390 vector instructions, which take 1.4 times as long beside products; the clock is at 1.8 GHz there.
// (Products of one half beside the statistics of the other in one wave: the same, 39.8 against 40.4.)  Measured and not kept: units of 32 rows with every lane storing its own
// (the same, but 38 us at 600 slots), twelve waves per block (the same; sixteen spill), the weights requested after
// everything else (the same).
template <int KS>      // 32-byte k steps per row: ld = 32 KS
__global__ __launch_bounds__(64 * VP_WAVES, 2) void vocab_panel_kernel(PanelArgs a)
{
    // [cols_per_group x pitch] codes, the waves' statistics, the slots' dequantization factors, the block's biases
    extern __shared__ __align__(16) int8_t s_x[];
    constexpr int ld = 32 * KS, pitch = ld + 16, NTHR = 64 * VP_WAVES;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int i = lane & 31, h = lane >> 5;
    const int n = a.n, c_base = blockIdx.y * a.cols_per_group;
    const int cols = min(a.cols_per_group, n - c_base);       // > 0 by construction of the grid
    const int nct = (cols + 31) >> 5, nrp = (a.rows + 63) >> 6;
    double *s_sum = (double *)(s_x + (size_t)a.cols_per_group * pitch + wave * VP_STAGE);      // [32 slots][4 tiles]
    float *s_max = (float *)(s_sum + 128);
    float *s_c = (float *)(s_x + (size_t)a.cols_per_group * pitch + VP_WAVES * VP_STAGE), *s_b = s_c + a.cols_per_group;
    // Blocks whose numbers agree modulo 8 share an XCD: they take neighbouring runs, the same ones in every column
    // group, so that an XCD's L2 is asked for one eighth of the matrix and gives it to all groups.
    const int gx = gridDim.x, rank = gx % 8 == 0 ? ((int)blockIdx.x & 7) * (gx >> 3) + ((int)blockIdx.x >> 3) : (int)blockIdx.x;
    int u0, u1, rp0;                                          // the wave's units, the block's first rows
    {
        int first, end, skip;
        q8_panel_run(nrp, nct, gx, VP_WAVES, rank, 0, &first, &skip, &rp0);
        q8_panel_run(nrp, nct, gx, VP_WAVES, rank, VP_WAVES - 1, &skip, &end, &u1);
        q8_panel_wave_run(first, end, wave, &u0, &u1);
    }
    int rp = u0 / nct, ct = u0 - rp * nct;

    // weights: lane (row i, k half h) of k step s holds bytes 32 s + 16 h .. of row 64 rp + 32 t + i; in the packed order
    // that is 64-byte block s / 2 of the row's tile, piece 2 (s % 2) + h.  The whole offset is the vector offset and lies
    // inside the packed weights (rows past the matrix come as -inf below); a scalar offset is not sure to be checked.
    const __amdgpu_buffer_rsrc_t rw = q8_rsrc(a.tiles, (size_t)a.ntiles * (KS / 2) * 1024);
    const __amdgpu_buffer_rsrc_t rpm = q8_rsrc(a.part_max, (size_t)n * a.ntiles * 4), rps = q8_rsrc(a.part_sum, (size_t)n * a.ntiles * 8);
    v4i A[2][KS];
    auto weights = [&](unsigned at, int s) {
        return __builtin_bit_cast(v4i, __builtin_amdgcn_raw_buffer_load_b128(rw, (int)(at + q8_panel_step(s)), 0, 0));
    };
    // Everything the block keeps in LDS is requested before the first wait, through descriptors and not in branches, what is
    // needed first first: factors, biases, codes (16-byte pieces; slots past the panel are zero), then the weights.  (Biases
    // zero without any: adding zero changes no logit but the sign of a zero, which no comparison and no exponential sees.
    // Rows past the matrix have -inf, which makes their logits that.)
    {
        constexpr int PB = 4, PX = (256 * (ld / 16) + NTHR - 1) / NTHR < 18 ? (256 * (ld / 16) + NTHR - 1) / NTHR : 18;
        const __amdgpu_buffer_rsrc_t rc = q8_rsrc(a.xscale + c_base, (size_t)cols * 4);
        const __amdgpu_buffer_rsrc_t rb = q8_rsrc(a.bias, a.bias ? (size_t)a.rows * 4 : 0);
        const __amdgpu_buffer_rsrc_t rx = q8_rsrc(a.xq + (size_t)c_base * ld, (size_t)cols * ld);
        const int total = nct * 32 * (ld / 16);
        const float xs = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rc, tid * 4, 0, 0));
        float bv[PB];
        v4i xv[PX];
#pragma unroll
        for (int u = 0; u < PB; ++u) bv[u] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rb, (64 * rp0 + u * NTHR + tid) * 4, 0, 0));
#pragma unroll
        for (int u = 0; u < PX; ++u) {
            const int p = u * NTHR + tid;                        // piece p: slot p / (ld / 16), bytes 16 (p % (ld / 16)) ..
            xv[u] = __builtin_bit_cast(v4i, __builtin_amdgcn_raw_buffer_load_b128(rx, (int)(p < total ? (unsigned)p * 16u : Q8_OOB), 0, 0));
        }
        __builtin_amdgcn_sched_barrier(0);
        const unsigned at0 = q8_panel_weight(2 * rp, lane, KS, a.ntiles), at1 = q8_panel_weight(2 * rp + 1, lane, KS, a.ntiles);
#pragma unroll
        for (int s = 0; s < KS; ++s) A[0][s] = weights(at0, s);
        __builtin_amdgcn_sched_barrier(0);
        if (tid < a.cols_per_group) s_c[tid] = a.w_scale * xs;
#pragma unroll
        for (int u = 0; u < PB; ++u)
            if (u * NTHR + tid < a.bias_rows) s_b[u * NTHR + tid] = 64 * rp0 + u * NTHR + tid < a.rows ? bv[u] : -INFINITY;
#pragma unroll
        for (int u = 0; u < PX; ++u) {
            const int p = u * NTHR + tid, col = p / (ld / 16), ch = p - col * (ld / 16);
            if (p < total) *(v4i *)(s_x + col * pitch + ch * 16) = xv[u];
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int s = 0; s < KS; ++s) A[1][s] = weights(at1, s);
        // (the last pieces and biases of widths and heights that need more than the registers above)
        for (int p = PX * NTHR + tid; p < total; p += NTHR) {
            const int col = p / (ld / 16), ch = p - col * (ld / 16);
            *(v4i *)(s_x + col * pitch + ch * 16) = __builtin_bit_cast(v4i, __builtin_amdgcn_raw_buffer_load_b128(rx, p * 16, 0, 0));
        }
        for (int r = PB * NTHR + tid; r < a.bias_rows; r += NTHR) s_b[r] = 64 * rp0 + r < a.rows ? __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rb, (64 * rp0 + r) * 4, 0, 0)) : -INFINITY;
    }
    __syncthreads();

    const int8_t *bp = s_x + i * pitch + 16 * h;
    v2u st_max = {0u, 0u};
    v4u st_sum = {0u, 0u, 0u, 0u};
    int st_o4 = 0, st_o8 = 0;
    // (loads still out here would be waited for at the loop's head in every round, as if no store came after them)
    __builtin_amdgcn_s_waitcnt(0x0f70);                       // vmcnt(0)
    for (int u = u0; u < u1; ++u) {
        const int8_t *bt = bp + ct * 32 * pitch;
        v16i acc[2] = {{}, {}};
        if (ct == nct - 1 && u + 1 < u1) {                    // uniform: the next unit starts other rows
            const unsigned at0 = q8_panel_weight(2 * rp + 2, lane, KS, a.ntiles), at1 = q8_panel_weight(2 * rp + 3, lane, KS, a.ntiles);
#pragma unroll
            for (int s = 0; s < KS; ++s) {
                const v4i x = *(const v4i *)(bt + 32 * s);
                acc[0] = __builtin_amdgcn_mfma_i32_32x32x32_i8(A[0][s], x, acc[0], 0, 0, 0);
                acc[1] = __builtin_amdgcn_mfma_i32_32x32x32_i8(A[1][s], x, acc[1], 0, 0, 0);
                A[0][s] = weights(at0, s);
                A[1][s] = weights(at1, s);
            }
        } else {
#pragma unroll
            for (int s = 0; s < KS; ++s) {
                const v4i x = *(const v4i *)(bt + 32 * s);
                acc[0] = __builtin_amdgcn_mfma_i32_32x32x32_i8(A[0][s], x, acc[0], 0, 0, 0);
                acc[1] = __builtin_amdgcn_mfma_i32_32x32x32_i8(A[1][s], x, acc[1], 0, 0, 0);
            }
        }
        // result r of the lane: row 64 rp + 32 t + 8 (r / 4) + 4 h + r % 4 of slot 32 ct + i
        const float c = s_c[32 * ct + i];
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            const float *bias = s_b + 64 * (rp - rp0) + 32 * t + 4 * h;
            float y[16];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const float4 b = *(const float4 *)(bias + 8 * q);
                y[4 * q] = (float)acc[t][4 * q] * c + b.x;
                y[4 * q + 1] = (float)acc[t][4 * q + 1] * c + b.y;
                y[4 * q + 2] = (float)acc[t][4 * q + 2] * c + b.z;
                y[4 * q + 3] = (float)acc[t][4 * q + 3] * c + b.w;
            }
            float m[2] = {vp_max8(y), vp_max8(y + 8)};
            // the halves trade: lanes of half v hold tile v's maximum, then everybody gets both
            auto sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(m[0]), __float_as_uint(m[1]), false, false);
            const float mine = fmaxf(__uint_as_float(sw[0]), __uint_as_float(sw[1]));
            sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(mine), __float_as_uint(mine), false, false);
            m[0] = __uint_as_float(sw[0]); m[1] = __uint_as_float(sw[1]);
            double sd[2];
#pragma unroll
            for (int v = 0; v < 2; ++v) {
                sd[v] = (double)exp_le0(y[8 * v] - m[v]);
#pragma unroll
                for (int r = 1; r < 8; ++r) sd[v] += (double)exp_le0(y[8 * v + r] - m[v]);
            }
            const auto lo = __builtin_amdgcn_permlane32_swap((unsigned)__double2loint(sd[0]), (unsigned)__double2loint(sd[1]), false, false);
            const auto hi = __builtin_amdgcn_permlane32_swap((unsigned)__double2hiint(sd[0]), (unsigned)__double2hiint(sd[1]), false, false);
            s_max[i * 4 + 2 * t + h] = mine;
            s_sum[i * 4 + 2 * t + h] = __hiloint2double((int)hi[0], (int)lo[0]) + __hiloint2double((int)hi[1], (int)lo[1]);
        }
        // Lane L carries tiles 2 (L % 2), + 1 of slot L / 2 out.  Through descriptors, not in a branch, and nothing the
        // next unit needs is requested after them: stores count with the loads, and a wait for the weights must not
        // become one for these.
        __builtin_amdgcn_wave_barrier();                      // (the wave's own LDS: in order)
        const int tile = 4 * rp + 2 * (lane & 1), colr = 32 * ct + (lane >> 1);
        const unsigned o = colr < cols && tile < a.ntiles ? (unsigned)(c_base + colr) * (unsigned)a.ntiles + (unsigned)tile : Q8_OOB >> 2;
        const bool both = tile + 1 < a.ntiles;
        // The registers of a store are kept from reuse until the next unit's: taking one back waits for the store.
        asm volatile("" ::"v"(st_max), "v"(st_sum), "v"(st_o4), "v"(st_o8));
        st_max = *(const v2u *)(s_max + 2 * lane);
        st_sum = *(const v4u *)(s_sum + 2 * lane);
        const bool whole = 4 * rp + 4 <= a.ntiles;            // uniform
        st_o4 = (int)(whole ? o * 4u : Q8_OOB);
        st_o8 = (int)(whole && o < Q8_OOB >> 3 ? o * 8u : Q8_OOB);
        __builtin_amdgcn_raw_buffer_store_b64(st_max, rpm, st_o4, 0, 0);
        __builtin_amdgcn_raw_buffer_store_b128(st_sum, rps, st_o8, 0, 0);
        if (!whole && o < Q8_OOB >> 2) {                      // the last rows: some of the four tiles are missing
            __builtin_amdgcn_raw_buffer_store_b32(st_max.x, rpm, (int)(o * 4u), 0, 0);
            __builtin_amdgcn_raw_buffer_store_b64(__builtin_shufflevector(st_sum, st_sum, 0, 1), rps, (int)(o * 8u), 0, 0);
            if (both) {
                __builtin_amdgcn_raw_buffer_store_b32(st_max.y, rpm, (int)(o * 4u) + 4, 0, 0);
                __builtin_amdgcn_raw_buffer_store_b64(__builtin_shufflevector(st_sum, st_sum, 2, 3), rps, (int)(o * 8u) + 8, 0, 0);
            }
        }
        if (++ct == nct) { ct = 0; ++rp; }
    }
}

// Whether the panel kernel takes this product: tile-packed weights with rows of 512 or 640 bytes.
bool q8i_vocab_panel_ok(const q8_mat *W) { return W->tiles != nullptr && (W->ld == 512 || W->ld == 640); }

q8_status q8i_vocab_panel(q8_ctx *ctx, const q8_mat *W, const float *bias, const int8_t *xq, const float *xscale, int n,
                          float *part_max, double *part_sum)
{
    PanelArgs a;
    a.tiles = W->tiles; a.xq = xq; a.xscale = xscale; a.bias = bias;
    a.part_max = part_max; a.part_sum = part_sum;
    a.rows = W->rows; a.ld = W->ld; a.n = n; a.ntiles = (W->rows + 15) / 16; a.w_scale = W->scale;
    int gx, gy;
    const size_t smem = q8_panel_plan(W->rows, W->ld, n, &a.cols_per_group, &gx, &gy, &a.bias_rows);
    typedef void (*kern_t)(PanelArgs);
    const kern_t kern = W->ld == 512 ? vocab_panel_kernel<16> : vocab_panel_kernel<20>;
    static Q8OncePerDevice asked[2];
    const q8_status st = q8i_lds(ctx, asked[W->ld == 512 ? 0 : 1], (const void *)kern, Q8_PANEL_LDS, "vocabulary panel kernel");
    if (st) return st;
    Q8_LAUNCH(ctx, Q8_KERNEL_MFMA, kern, dim3(gx, gy), dim3(64 * VP_WAVES), smem, a);
    return q8i_launch_check(ctx, "vocabulary panel");
}

// Block (j, job): max-abs quantization of vector j's K floats into ld code bytes (pad bytes
// zero), Section 3's "8-bit approximation" of an activation.
struct QuantJob {
    const float *X;
    int K, ldx, ld;
    int8_t *xq;            // [n x ld]
    float *xscale;         // [n]
    int8_t *tap_xq;        // [n x K] or NULL
    float *tap_scale;      // [n] or NULL
};
struct QuantJobs {
    QuantJob j[GEMM_MAX_JOBS];
};

__global__ __launch_bounds__(256) void quantize_rows_kernel(QuantJobs jobs)
{
    __shared__ float s_scale[1];
    __shared__ float s_red[4];
    const QuantJob &J = jobs.j[blockIdx.y];
    const int j = blockIdx.x;
    // Vectors of at most 2048 floats in whole 16-byte pieces stay in registers between their maximum and their codes (read
    // again after the barrier, they are a second round trip: 5.4 -> 4.6 us for 1024 vectors of 2048).
    if (J.K <= 2048 && J.K % 4 == 0 && J.ld <= 2048) {
        const int tid = threadIdx.x;
        const __amdgpu_buffer_rsrc_t rx = q8_rsrc(J.X + (size_t)j * J.ldx, (size_t)J.K * sizeof(float));
        float4 v[2];
        float m = 0.0f;
#pragma unroll
        for (int t = 0; t < 2; ++t) v[t] = __builtin_bit_cast(float4, __builtin_amdgcn_raw_buffer_load_b128(rx, (t * 256 + tid) * 16, 0, 0));
#pragma unroll
        for (int t = 0; t < 2; ++t) m = fmaxf(m, fmaxf(fmaxf(fabsf(v[t].x), fabsf(v[t].y)), fmaxf(fabsf(v[t].z), fabsf(v[t].w))));
        m = wave_max_f(m);
        if ((tid & 63) == 0) s_red[tid >> 6] = m;
        __syncthreads();
        float scale, inv;
        q8_scale_of(fmaxf(fmaxf(s_red[0], s_red[1]), fmaxf(s_red[2], s_red[3])), scale, inv);
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            const int k = (t * 256 + tid) * 4;                   // (zeros past K)
            if (k < J.ld) *(int *)(J.xq + (size_t)j * J.ld + k) = q8_pack4(v[t].x, v[t].y, v[t].z, v[t].w, inv);
        }
        if (tid == 0) {
            J.xscale[j] = scale;
            if (J.tap_scale) J.tap_scale[j] = scale;
        }
        if (J.tap_xq) {
            __syncthreads();
            for (int k = tid; k < J.K; k += 256) J.tap_xq[(size_t)j * J.K + k] = J.xq[(size_t)j * J.ld + k];
        }
        return;
    }
    block_quantize<1>(J.X + (size_t)j * J.ldx, 1, J.K, J.ldx, J.ld, J.xq + (size_t)j * J.ld, s_scale, s_red);
    if (threadIdx.x == 0) {
        J.xscale[j] = s_scale[0];
        if (J.tap_scale) J.tap_scale[j] = s_scale[0];
    }
    if (J.tap_xq) {
        __syncthreads();
        for (int k = threadIdx.x; k < J.K; k += blockDim.x) J.tap_xq[(size_t)j * J.K + k] = J.xq[(size_t)j * J.ld + k];
    }
}

q8_status q8i_quantize_jobs(q8_ctx *ctx, const q8i_quant_job *d, int njobs, int n)
{
    QuantJobs jobs;
    for (int t = 0; t < GEMM_MAX_JOBS; ++t) {
        const q8i_quant_job &q = d[t < njobs ? t : 0];
        jobs.j[t] = {q.X, q.K, q.ldx, q.ld, q.xq, q.xscale, q.taps ? q.taps->xq : nullptr, q.taps ? q.taps->xscale : nullptr};
    }
    hipLaunchKernelGGL(quantize_rows_kernel, dim3(n, njobs), dim3(256), 0, ctx->stream, jobs);
    return q8i_launch_check(ctx, "quantize rows");
}

// Y = dequantize(W . codes) + bias for n already-quantized vectors, up to three products in
// one launch.  part_max / part_sum non-NULL (first job only is looked at): also the per-tile
// softmax statistics of the vocabulary layer.
q8_status q8i_gemm_jobs(q8_ctx *ctx, const q8i_gemm_job *d, int njobs, int n)
{
    GemmJobs jobs;
    int max_rows = 0;
    for (int t = 0; t < GEMM_MAX_JOBS; ++t) {
        const q8i_gemm_job &q = d[t < njobs ? t : 0];
        GemmArgs &a = jobs.j[t];
        a.W = q.W->data; a.Wt = (q.W->tiles && q.W->ld % 64 == 0) ? q.W->tiles : nullptr; a.xq = q.xq; a.xscale = q.xscale; a.bias = q.bias; a.Y = q.Y; a.tap_acc = q.tap_acc;
        a.part_max = q.part_max; a.part_sum = q.part_sum;
        a.rows = q.W->rows; a.ld = q.W->ld; a.n = n; a.ldy = q.ldy; a.ntiles = (q.W->rows + 15) / 16;
        a.tiled = q.tiled;
        a.w_scale = q.W->scale;
        a.row_scale = q.row_scale;
        if (a.rows > max_rows) max_rows = a.rows;
    }
    const bool stats = d[0].part_max != nullptr;
    q8_panel_shape shape = {njobs, {jobs.j[0].rows, jobs.j[1].rows, jobs.j[2].rows}, n, jobs.j[0].ld, jobs.j[0].ld, !stats, 1, 1, 1, 1};
    for (int t = 0; t < njobs; ++t) {
        const GemmArgs &a = jobs.j[t];
        if (a.ld < shape.min_ld) shape.min_ld = a.ld;
        if (a.ld > shape.max_ld) shape.max_ld = a.ld;
        if (a.tap_acc || a.tiled || (size_t)a.ntiles * 16 * a.ld >= (1u << 31) || (size_t)n * a.ld >= (1u << 31)) shape.plain = 0;
        if (!a.Wt) shape.packed = 0;
        if (a.ld % 64) shape.steps = 0;
        if (a.ld % 128) shape.lines = 0;
        if (a.ldy % 4 || ((uintptr_t)a.Y & 15)) shape.whole = 0;
    }
    if (const int tiles = q8_part_rows(&shape)) return q8i_gemm_part(ctx, jobs, max_rows, shape.max_ld, n, njobs, tiles);
    switch (q8_panel_route(&shape)) {
    case Q8_ROUTE_ONCE_64X64: return q8i_gemm_once(ctx, jobs, max_rows, n, njobs, 64, 64, false);
    case Q8_ROUTE_ONCE_128X32: return q8i_gemm_once(ctx, jobs, max_rows, n, njobs, 128, 32, false);
    case Q8_ROUTE_ONCE_128X64: return q8i_gemm_once(ctx, jobs, max_rows, n, njobs, 128, 64, false);
    case Q8_ROUTE_ONCE_128X64_TRADE: return q8i_gemm_once(ctx, jobs, max_rows, n, njobs, 128, 64, true);
    case Q8_ROUTE_STREAM: return q8i_gemm_stream(ctx, jobs, max_rows, n, njobs, (int)q8_panel_blocks(&shape, 64, n));
    case Q8_ROUTE_TILES_128: {
        const size_t smem = (size_t)2 * 128 * (256 + 16);
        static Q8OncePerDevice asked;
        const q8_status st = q8i_lds(ctx, asked, (const void *)gemm_tile_kernel<4, 1, 4>, smem, "large panel kernel");
        if (st) return st;
        Q8_LAUNCH(ctx, Q8_KERNEL_MFMA, (gemm_tile_kernel<4, 1, 4>), dim3((max_rows + 127) / 128, (n + 127) / 128, njobs), dim3(256), smem, jobs);
        return q8i_launch_check(ctx, "gemm");
    }
    case Q8_ROUTE_TILES_64:
        Q8_LAUNCH(ctx, Q8_KERNEL_MFMA, (gemm_tile_kernel<2, 2, 1>), dim3((max_rows + 63) / 64, (n + 63) / 64, njobs), dim3(256), (size_t)2 * 64 * (256 + 16), jobs);
        return q8i_launch_check(ctx, "gemm");
    case Q8_ROUTE_RESIDENT_1024: return q8i_gemm_resident_1024(ctx, jobs, max_rows, n, njobs);
    case Q8_ROUTE_RESIDENT:
        Q8_LAUNCH(ctx, Q8_KERNEL_MFMA, gemm_resident_kernel<8>, dim3((max_rows + 63) / 64, (n + 63) / 64, njobs), dim3(256), (size_t)64 * (512 + 16), jobs);
        return q8i_launch_check(ctx, "gemm");
    default: break;                                      // staged
    }
    if (max_rows > 8192) {
        const dim3 grid((max_rows + 64 * GB_BIG_RT - 1) / (64 * GB_BIG_RT), (n + 16 * GB_BIG_NT - 1) / (16 * GB_BIG_NT), njobs);
        if (stats) Q8_LAUNCH(ctx, Q8_KERNEL_MFMA, (gemm_block_kernel<GB_BIG_RT, GB_BIG_NT, true>), grid, dim3(256), 0, jobs);
        else Q8_LAUNCH(ctx, Q8_KERNEL_MFMA, (gemm_block_kernel<GB_BIG_RT, GB_BIG_NT, false>), grid, dim3(256), 0, jobs);
    } else {
        const dim3 grid((max_rows + 64 * GB_SMALL_RT - 1) / (64 * GB_SMALL_RT), (n + 16 * GB_SMALL_NT - 1) / (16 * GB_SMALL_NT), njobs);
        if (stats) Q8_LAUNCH(ctx, Q8_KERNEL_MFMA, (gemm_block_kernel<GB_SMALL_RT, GB_SMALL_NT, true>), grid, dim3(256), 0, jobs);
        else Q8_LAUNCH(ctx, Q8_KERNEL_MFMA, (gemm_block_kernel<GB_SMALL_RT, GB_SMALL_NT, false>), grid, dim3(256), 0, jobs);
    }
    return q8i_launch_check(ctx, "gemm");
}

q8_status q8i_gemm_mfma(q8_ctx *ctx, const q8_mat *W, const float *X, int n, int ldx, const float *bias, float *Y,
                        int ldy, const q8_taps *taps, int8_t *xq, float *xscale, const float *row_scale)
{
    q8i_quant_job qj = {X, W->cols, ldx, W->ld, xq, xscale, taps};
    q8_status st = q8i_quantize_jobs(ctx, &qj, 1, n);
    if (st) return st;
    q8i_gemm_job gj = {W, xq, xscale, bias, Y, ldy, taps ? taps->acc : nullptr, nullptr, nullptr, 0, row_scale};
    return q8i_gemm_jobs(ctx, &gj, 1, n);
}
