/* Host build of the index arithmetic that the kernels share (plain C). */
#include "q8_index.h"

void q8x_position_runs(const int *off, int n_sent, int blocks, int *pos, int *end)
{
    for (int b = 0; b < blocks; ++b) q8_position_run(off, n_sent, b, blocks, pos + b, end + b);
}
