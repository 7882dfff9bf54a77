// q8_index.h -- which part of a launch's work a block or a lane takes, where that is more than a product of block and
// lane numbers: plain integer arithmetic, the same on the device and in a host build, so that the bounds of the
// accesses that follow from it can be checked on the host for whole ranges of sizes.
#pragma once

#if defined(__HIPCC__)
#define Q8_INDEX_FN __host__ __device__ __forceinline__
#else
#define Q8_INDEX_FN static inline
#endif

// The positions of n_sent sentences back to back, [off[0], off[n_sent]) (a group of sentences out of a larger batch
// does not begin at 0), dealt to `blocks` blocks in even runs: block b takes [*pos, *end).
Q8_INDEX_FN void q8_position_run(const int *off, int n_sent, int b, int blocks, int *pos, int *end)
{
    const int first = off[0];
    const long long total = (long long)off[n_sent] - first;
    *pos = first + (int)(total * b / blocks);
    *end = first + (int)(total * (b + 1) / blocks);
}
