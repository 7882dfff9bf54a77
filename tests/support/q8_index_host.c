/* Host build of the index arithmetic that the kernels share (plain C). */
#include "q8_index.h"

void q8x_position_runs(const int *off, int n_sent, int blocks, int *pos, int *end)
{
    for (int b = 0; b < blocks; ++b) q8_position_run(off, n_sent, b, blocks, pos + b, end + b);
}

void q8x_panel_runs(int row_groups, int slot_tiles, int blocks, int waves, int *u0, int *u1, int *rp0)
{
    for (int b = 0; b < blocks; ++b)
        for (int w = 0; w < waves; ++w) q8_panel_run(row_groups, slot_tiles, blocks, waves, b, w, u0 + b * waves + w, u1 + b * waves + w, rp0 + b * waves + w);
}

/* [64 lanes][ks] byte offsets that a wave reads for a half */
void q8x_panel_weights(int half, int ks, int ntiles, unsigned *at)
{
    for (int lane = 0; lane < 64; ++lane)
        for (int s = 0; s < ks; ++s) at[lane * ks + s] = q8_panel_weight(half, lane, ks, ntiles) + q8_panel_step(s);
}
