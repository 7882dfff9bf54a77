/* Host build of the index arithmetic that the kernels share (plain C). */
#include "q8_index.h"
#include "q8_route.h"

void q8x_position_runs(const int *off, int n_sent, int blocks, int *pos, int *end)
{
    for (int b = 0; b < blocks; ++b) q8_position_run(off, n_sent, b, blocks, pos + b, end + b);
}

void q8x_panel_runs(int row_groups, int slot_tiles, int blocks, int waves, int *u0, int *u1, int *rp0)
{
    for (int b = 0; b < blocks; ++b)
        for (int w = 0; w < waves; ++w) q8_panel_run(row_groups, slot_tiles, blocks, waves, b, w, u0 + b * waves + w, u1 + b * waves + w, rp0 + b * waves + w);
}

void q8x_panel_wave_runs(int first, int end, int *u0, int *u1)
{
    for (int w = 0; w < Q8_PANEL_WAVES; ++w) q8_panel_wave_run(first, end, w, u0 + w, u1 + w);
}

/* [64 lanes][ks] byte offsets that a wave reads for a half */
void q8x_panel_weights(int half, int ks, int ntiles, unsigned *at)
{
    for (int lane = 0; lane < 64; ++lane)
        for (int s = 0; s < ks; ++s) at[lane * ks + s] = q8_panel_weight(half, lane, ks, ntiles) + q8_panel_step(s);
}

/* Plans every height in [1, rows] (step apart) times n slots: the largest LDS and the most rows of biases that a block's run
 * needs beyond what the plan gives it (<= 0: enough); 0 in *worst_lds if a plan's groups do not cover the slots */
void q8x_panel_plans(int rows, int step, int ld, int n, unsigned long long *worst_lds, int *worst_bias)
{
    *worst_lds = 1;
    *worst_bias = -1000000;
    for (int r = 1; r <= rows; r += step) {
        int cols, gx, gy, bias_rows;
        const unsigned long long lds = q8_panel_plan(r, ld, n, &cols, &gx, &gy, &bias_rows);
        if ((long long)cols * gy < n || cols * (gy - 1) >= n || cols % 32 || gx * gy > 256) { *worst_lds = 0; return; }
        if (lds > *worst_lds) *worst_lds = lds;
        const int groups = (r + 63) / 64;
        for (int g = 0; g < gy; g += gy > 1 ? gy - 1 : 1) {           /* the first group, and the last, which may be narrower */
            const int own = n - g * cols < cols ? n - g * cols : cols, tiles = (own + 31) / 32;
            for (int b = 0; b < gx; b += gx > 7 ? gx / 7 : 1) {
                int u0, u1, rp0, first;
                q8_panel_run(groups, tiles, gx, Q8_PANEL_WAVES, b, 0, &first, &u1, &rp0);
                q8_panel_run(groups, tiles, gx, Q8_PANEL_WAVES, b, Q8_PANEL_WAVES - 1, &u0, &u1, &rp0);
                const int need = u1 > first ? ((u1 - 1) / tiles - rp0 + 1) * 64 - bias_rows : -bias_rows;
                if (need > *worst_bias) *worst_bias = need;
            }
        }
    }
}

int q8x_enc_one_better(int H, int ldx, int packed, int l) { return q8_enc_one_better(H, ldx, packed, l); }

int q8x_enc_one_launch(int H, int S, int max_l) { return q8_enc_one_launch(H, S, max_l); }

/* The most LDS of those of [1, S] sentences of H units that are one launch, and 0 if some plan's groups don't cover a set, or its blocks the device */
unsigned q8x_enc_lds(int H, int S)
{
    unsigned worst = 0;
    for (int s = 1; s <= S; ++s) {
        int members, sets, groups, slots;
        const unsigned lds = q8_enc_plan(H, s, &members, &sets, &groups, &slots);
        for (int i = 0; i < sets; ++i)
            if (s * (i + 1) / sets - s * i / sets > groups * slots || s * (i + 1) / sets == s * i / sets) return 0;
        if (members * 32 < H || slots > 16 || 2 * sets * members > 256) return 0;
        if (lds > worst && q8_enc_one_launch(H, s, 1024)) worst = lds;
    }
    return worst;
}

/* one product of n vectors (codes of ld bytes, results at `pitch` floats per vector) */
int q8x_panel_route(int rows, int ld, int n, int packed, int pitch)
{
    const q8_panel_shape s = {1, {rows, 0, 0}, n, ld, ld, 1, packed, ld % 64 == 0, ld % 128 == 0, pitch % 4 == 0};
    return q8_panel_route(&s);
}

int q8x_enc_scale(int it, int slot) { return q8_enc_scale(it, slot); }
int q8x_enc_x_scale(int it, int slot) { return q8_enc_x_scale(it, slot); }

int q8x_quant_rows(int rows, int ld, int n) { return q8_quant_rows(rows, ld, n); }
int q8x_part_rows(int rows, int ld, int n, int njobs)
{
    q8_panel_shape s = {njobs, {rows, rows, rows}, n, ld, ld, 1, 0, 0, 0, 0};
    return q8_part_rows(&s);
}

/* Columns (tiles of 32 vectors) per block, whether the launch takes the shape, and the parts of the k range, of gru_tile_kernel */
int q8x_gru_tile(int H, int ldx, int ldh, int n, int codes, int packed, int *columns, int *nx, int *k0, int *steps, int *stages)
{
    *columns = q8_gru_tile_columns(H, n);
    *stages = q8_gru_parts(ldx, ldh, nx, k0, steps);
    return q8_gru_tile_better(H, ldx, ldh, n, codes, packed);
}

/* The most LDS of a batched encoder of one group per set that multiplies X itself (rows of 128 xs bytes), and of any plan */
unsigned q8x_enc_x_lds(int H, int xs)
{
    unsigned worst = 0;
    for (int s = 1; s <= 1024; ++s) {
        int members, sets, groups, slots;
        const unsigned lds = q8_enc_plan(H, s, &members, &sets, &groups, &slots);
        if (groups == 1 && lds + Q8_ENC_X_LDS(xs) > worst) worst = lds + Q8_ENC_X_LDS(xs);
        if (groups <= 8 && lds > Q8_ENC_LDS_MOST) return 0;
    }
    return worst;
}
