// q8_gru_tile.hip -- a GRU transition (Eq. 3, 4) for panels of vectors: both products and the gates in one launch that waits for
// nobody, without the two [n x 3H] arrays of pre-activations in memory.
#include "q8_internal.h"
#include "q8_index.h"

// Block of nine waves: 32 hidden units, their three gates, x 32 CT vectors.  The k range of both products (rows of Wx, then of
// Wh) is cut into three parts, two of the longer one (q8_gru_parts); wave (gate, part) multiplies the gate's 32 rows by its part
// of all vectors, so that weights are read once per block, straight into registers, and the codes go through LDS in stages of
// 128 bytes per part, two buffers, the stage after next on its way while one is multiplied.  Then the nine tiles of sums meet in LDS
// and every thread finishes four units of a vector at a time: dequantization, biases, gates, as the product kernels and
// gru_gates_q_kernel do, value for value.
// What bounds it is the way of a stage's 84 KB (1.5 us; the registers hold no more on their way), then the gates' double precision
// (3.2 us): 1000 vectors, H = 1024, us, rows of 512 + 1024 / 2048 + 1024 bytes 17.2 / 23.3 (products and gates apart 14.2 + 7.9 / 18.0 + 7.9, and
// 8.4 of another launch for the recurrent product).  The codes of the new states take a launch of their own (quantize_rows_kernel): blocks
// that exchanged maxima would have to be resident together, which a compute unit's worth of block is not beside another
// stream's.
struct GruTileArgs {
    const int8_t *Wx, *Wh, *Wxt, *Wht;   // [3H x ldx], [3H x ldh], and the same tile-packed or NULL
    const float *bx, *bh;                // [3H] or NULL
    const int8_t *xq, *hq;               // codes [n x ldx], [n x ldh]
    const float *xs, *hs;                // [n]
    const float *h_prev;                 // [n x ldp]
    float *h_out;                        // [n x ldo]
    int H, n, ldx, ldh, ldp, ldo;
    int nx, k0[3], steps[3], stages;     // q8_gru_parts
    float wx_scale, wh_scale;
};
#define GT_WAVES 9
#define GT_PITCH (128 + 16)

template <int CT>
__global__ __launch_bounds__(64 * GT_WAVES) void gru_tile_kernel(GruTileArgs a)
{
    constexpr int COLS = 32 * CT, PIECES = 8 * COLS, NQ = (PIECES + 191) / 192, NT = 64 * GT_WAVES;
    extern __shared__ __align__(16) int8_t s_g[];                      // [2][3][COLS][GT_PITCH] codes, then [9][COLS][32] sums
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int gate = wave % 3, part = wave / 3, i = lane & 15, g = lane >> 4;
    const int H = a.H, n = a.n, u0 = (int)blockIdx.x * 32, c0 = (int)blockIdx.y * COLS;
    const bool x = part < a.nx;
    const int ld = x ? a.ldx : a.ldh, k0 = a.k0[part], steps = a.steps[part];
    const int8_t *Wt = x ? a.Wxt : a.Wht;
    const bool tiled = Wt != nullptr && H % 16 == 0;                   // (a tile of 16 rows then belongs to one gate)
    const __amdgpu_buffer_rsrc_t rw = q8_rsrc(tiled ? Wt : x ? a.Wx : a.Wh, (size_t)(tiled ? (3 * H + 15) / 16 * 16 : 3 * H) * ld);
    const __amdgpu_buffer_rsrc_t rq = q8_rsrc(x ? a.xq : a.hq, (size_t)n * ld);
    auto weights = [&](int st, v4i (&av)[2][2]) {                      // (past the part, the row or the units: zero)
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const unsigned row0 = (unsigned)(gate * H + u0 + 16 * u);
            const unsigned base = tiled ? ((row0 >> 4) * (unsigned)(ld >> 6) << 10) + 16u * lane : (row0 + i) * (unsigned)ld + 16u * g;
            const bool ok = u0 + 16 * u + (tiled ? 0 : i) < H;
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                const int ks = k0 + 2 * st + q;
                const bool in = ok && 2 * st + q < steps && 64 * ks + (tiled ? 0 : 16 * g) < ld;
                av[u][q] = __builtin_bit_cast(v4i, __builtin_amdgcn_raw_buffer_load_b128(rw, (int)(in ? base + (tiled ? 1024u : 64u) * ks : Q8_OOB), 0, 0));
            }
        }
    };
    const int e0 = gate * 64 + lane, kend = min(ld, 64 * (k0 + steps));
    auto codes = [&](int st, v4i (&xv)[NQ]) {
#pragma unroll
        for (int q = 0; q < NQ; ++q) {
            const int e = q * 192 + e0, col = c0 + (e >> 3), k = 64 * (k0 + 2 * st) + 16 * (e & 7);
            xv[q] = __builtin_bit_cast(v4i, __builtin_amdgcn_raw_buffer_load_b128(rq, (int)(e < PIECES && col < n && k < kend ? (unsigned)col * (unsigned)ld + k : Q8_OOB), 0, 0));
        }
    };
    auto leave = [&](int st, const v4i (&xv)[NQ]) {
#pragma unroll
        for (int q = 0; q < NQ; ++q) {
            const int e = q * 192 + e0;
            if (e < PIECES) *(v4i *)(s_g + (((st & 1) * 3 + part) * COLS + (e >> 3)) * GT_PITCH + 16 * (e & 7)) = xv[q];
        }
    };
    v4i acc[2][2 * CT], xv[NQ], a0[2][2], a1[2][2];
#pragma unroll
    for (int t = 0; t < 2 * CT; ++t) acc[0][t] = acc[1][t] = (v4i){0, 0, 0, 0};
    auto stage = [&](int st, const v4i (&now)[2][2], v4i (&next)[2][2]) {
        weights(st + 1, next);
        const int8_t *bp = s_g + (((st & 1) * 3 + part) * COLS + i) * GT_PITCH + 16 * g;
#pragma unroll
        for (int t = 0; t < 2 * CT; ++t)
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                const v4i b = *(const v4i *)(bp + 16 * t * GT_PITCH + 64 * q);
                acc[0][t] = __builtin_amdgcn_mfma_i32_16x16x64_i8(now[0][q], b, acc[0][t], 0, 0, 0);
                acc[1][t] = __builtin_amdgcn_mfma_i32_16x16x64_i8(now[1][q], b, acc[1][t], 0, 0, 0);
            }
        if (st + 1 < a.stages) leave(st + 1, xv);
        codes(st + 2, xv);
        __syncthreads();
    };
    codes(0, xv);
    weights(0, a0);
    leave(0, xv);
    codes(1, xv);
    __syncthreads();
    for (int st = 0; st < a.stages; st += 2) {
        stage(st, a0, a1);
        if (st + 1 < a.stages) stage(st + 1, a1, a0);
    }

    // ---- sums of (gate, part), chunks of four units at ((wave, column), chunk ^ column % 8) ----
    v4i *s_sum = (v4i *)s_g;
#pragma unroll
    for (int t = 0; t < 2 * CT; ++t)
#pragma unroll
        for (int u = 0; u < 2; ++u) s_sum[(wave * COLS + 16 * t + i) * 8 + ((4 * u + g) ^ (i & 7))] = acc[u][t];
    __syncthreads();
    for (int e = tid; e < PIECES; e += NT) {
        const int c = e >> 3, ch = e & 7, col = c0 + c, unit = u0 + 4 * ch;
        if (col >= n || unit >= H) continue;
        const float cx = a.wx_scale * a.xs[col], chh = a.wh_scale * a.hs[col];
        const float4 hp = *(const float4 *)(a.h_prev + (size_t)col * a.ldp + unit);
        float gx[3][4], gh[3][4];
#pragma unroll
        for (int gt = 0; gt < 3; ++gt) {
            const v4i p0 = s_sum[(gt * COLS + c) * 8 + (ch ^ (c & 7))], p1 = s_sum[((3 + gt) * COLS + c) * 8 + (ch ^ (c & 7))],
                      p2 = s_sum[((6 + gt) * COLS + c) * 8 + (ch ^ (c & 7))];
            const v4i sx = a.nx == 2 ? p0 + p1 : p0, sh = a.nx == 2 ? p2 : p1 + p2;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                gx[gt][r] = (float)sx[r] * cx;
                gh[gt][r] = (float)sh[r] * chh;
            }
            if (a.bx) {
                const float4 b = *(const float4 *)(a.bx + gt * H + unit);
                gx[gt][0] = gx[gt][0] + b.x; gx[gt][1] = gx[gt][1] + b.y; gx[gt][2] = gx[gt][2] + b.z; gx[gt][3] = gx[gt][3] + b.w;
            }
            if (a.bh) {
                const float4 b = *(const float4 *)(a.bh + gt * H + unit);
                gh[gt][0] = gh[gt][0] + b.x; gh[gt][1] = gh[gt][1] + b.y; gh[gt][2] = gh[gt][2] + b.z; gh[gt][3] = gh[gt][3] + b.w;
            }
        }
        float hn[4];
        const float h4[4] = {hp.x, hp.y, hp.z, hp.w};
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const float xa[3] = {gx[0][r], gx[1][r], gx[2][r]}, ha[3] = {gh[0][r], gh[1][r], gh[2][r]};
            hn[r] = gru_gates(xa, ha, h4[r]);
        }
        *(float4 *)(a.h_out + (size_t)col * a.ldo + unit) = make_float4(hn[0], hn[1], hn[2], hn[3]);
    }
}

template <int CT> static q8_status gru_tile_launch(q8_ctx *ctx, const GruTileArgs &a)
{
    constexpr size_t codes = (size_t)2 * 3 * 32 * CT * GT_PITCH, sums = (size_t)GT_WAVES * 32 * CT * 32 * sizeof(int), smem = codes > sums ? codes : sums;
    static Q8OncePerDevice asked;
    const q8_status st = q8i_lds(ctx, asked, (const void *)gru_tile_kernel<CT>, smem, "panel GRU kernel");
    if (st) return st;
    Q8_LAUNCH(ctx, Q8_KERNEL_GRU, gru_tile_kernel<CT>, dim3((a.H + 31) / 32, (a.n + 32 * CT - 1) / (32 * CT)), dim3(64 * GT_WAVES), smem, a);
    return q8i_launch_check(ctx, "panel GRU");
}

bool q8i_gru_tile_ok(const q8_gru_weights *g, const float *h_prev, int ldp, const float *h_out, int ldo, int n, bool codes)
{
    const int H = g->Wh.cols, packed = H % 16 == 0 && g->Wx.tiles && g->Wx.ld % 64 == 0 && g->Wh.tiles && g->Wh.ld % 64 == 0;
    auto aligned = [](const void *p) { return ((uintptr_t)p & 15) == 0; };       // (states and biases move four at a time)
    return H % 4 == 0 && ldp % 4 == 0 && ldo % 4 == 0 && g->Wx.rows == 3 * H && g->Wh.rows == 3 * H && aligned(g->bx) && aligned(g->bh) &&
           aligned(h_prev) && aligned(h_out) &&
           (size_t)(3 * H + 15) * g->Wx.ld < (1u << 31) && (size_t)(3 * H + 15) * g->Wh.ld < (1u << 31) && (size_t)n * g->Wx.ld < (1u << 31) &&
           (size_t)n * g->Wh.ld < (1u << 31) && n > 8 && q8_gru_tile_better(H, g->Wx.ld, g->Wh.ld, n, codes, packed);
}

q8_status q8i_gru_tile(q8_ctx *ctx, const q8_gru_weights *g, const int8_t *xq, const float *xs, const int8_t *hq, const float *hs,
                       const float *h_prev, int ldp, float *h_out, int ldo, int n)
{
    GruTileArgs a = {g->Wx.data, g->Wh.data, g->Wx.ld % 64 == 0 ? g->Wx.tiles : nullptr, g->Wh.ld % 64 == 0 ? g->Wh.tiles : nullptr, g->bx, g->bh,
                     xq, hq, xs, hs, h_prev, h_out, g->Wh.cols, n, g->Wx.ld, g->Wh.ld, ldp, ldo, 0, {0, 0, 0}, {0, 0, 0}, 0, g->Wx.scale, g->Wh.scale};
    a.stages = q8_gru_parts(a.ldx, a.ldh, &a.nx, a.k0, a.steps);
    switch (q8_gru_tile_columns(a.H, n)) {
    case 1: return gru_tile_launch<1>(ctx, a);
    case 2: return gru_tile_launch<2>(ctx, a);
    case 3: return gru_tile_launch<3>(ctx, a);
    default: return gru_tile_launch<4>(ctx, a);
    }
}
