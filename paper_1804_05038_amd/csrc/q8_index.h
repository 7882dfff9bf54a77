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

// ---- the vocabulary panel (vocab_panel_kernel): units of 64 rows x 32 slots, dealt to the waves of a column group's blocks
// in even runs, slots first ----

#define Q8_PANEL_WAVES 8
#define Q8_PANEL_STAGE 1536      // bytes of LDS per wave: a unit's statistics on their way out
#define Q8_PANEL_LDS (160 * 1024)

// Grid and LDS bytes of `rows` rows of ld bytes (512 or 640) times n slots.  Column groups of equal size, as many slots as fit
// the LDS beside the rest (codes at pitch ld + 16, one float per slot) and 256; one block per compute unit.  A block's LDS
// also holds the biases of its run's rows, which may begin and end inside 64 rows: *bias_rows of them.  For the 65536 rows
// and 1024 slots that callers may ask for at most, a size always fits.
Q8_INDEX_FN unsigned long long q8_panel_plan(int rows, int ld, int n, int *cols_per_group, int *gx, int *gy, int *bias_rows)
{
    const int groups = (rows + 63) / 64;
    unsigned long long lds = 0;
    for (int most = 256; most >= 32; most -= 32) {
        const int ngroups = (n + most - 1) / most;
        *cols_per_group = ((n + ngroups - 1) / ngroups + 31) & ~31;
        *gy = (n + *cols_per_group - 1) / *cols_per_group;
        *gx = 256 / *gy;
        if (*gx < 1) *gx = 1;
        if (*gx > groups) *gx = groups;
        *bias_rows = ((groups + *gx - 1) / *gx + 2) * 64;
        lds = (unsigned long long)*cols_per_group * (ld + 16 + 4) + Q8_PANEL_WAVES * Q8_PANEL_STAGE + (unsigned long long)*bias_rows * 4;
        if (lds <= Q8_PANEL_LDS) break;
    }
    return lds;
}

// Units [*u0, *u1) of wave w of the block of rank b, and the 64-row group *rp0 that the block's first wave begins in.
Q8_INDEX_FN void q8_panel_run(int row_groups, int slot_tiles, int blocks, int waves, int b, int w, int *u0, int *u1, int *rp0)
{
    const long long units = (long long)row_groups * slot_tiles, nw = (long long)blocks * waves, w0 = (long long)b * waves;
    *u0 = (int)(units * (w0 + w) / nw);
    *u1 = (int)(units * (w0 + w + 1) / nw);
    *rp0 = (int)(units * w0 / nw) / slot_tiles;
}

// A block's units [first, end) among its eight waves, in runs back to back: of two waves that share a SIMD the one with the
// lower number is served first (a unit of 50000 x 512 x 1000 takes it 2.2 us, the other 2.5), so waves 0 to 3 take 9 parts
// of 16 where waves 4 to 7 take 7: 39.8 us with even runs, 38.8 with 17 and 15 of 32, 38.0 with 9 and 7; 17.9 us at 320
// slots, where a wave has four units, either way.
#define Q8_PANEL_FIRST 9
Q8_INDEX_FN void q8_panel_wave_run(int first, int end, int w, int *u0, int *u1)
{
    const int n = end - first, a = w < 4 ? Q8_PANEL_FIRST * w : 4 * Q8_PANEL_FIRST + (16 - Q8_PANEL_FIRST) * (w - 4), b = a + (w < 4 ? Q8_PANEL_FIRST : 16 - Q8_PANEL_FIRST);
    *u0 = first + (int)((long long)n * a / 64);
    *u1 = first + (int)((long long)n * b / 64);
}

// Byte offset, in tile-packed weights of ntiles tiles of ks / 2 blocks of 1 KiB, of what a lane multiplies in k step 0 of
// the 32-row half `half` (two tiles): row lane % 32, k half lane / 32.  Step s lies q8_panel_step(s) bytes further on.
// Tiles past the matrix (the last half's second tile, halves past the last, waves without a unit) are the last tile once
// more: nothing is read outside the packed weights, whatever becomes of an offset in a bounds check.
Q8_INDEX_FN unsigned q8_panel_weight(int half, int lane, int ks, int ntiles)
{
    const int i = lane & 31, t = 2 * half + (i >> 4), tile = t < ntiles ? t : ntiles - 1;
    return ((unsigned)tile * (unsigned)(ks / 2) << 10) + (unsigned)(lane >> 5) * 256u + (unsigned)(i & 15) * 16u;
}
Q8_INDEX_FN unsigned q8_panel_step(int s) { return (unsigned)(s >> 1) * 1024u + (unsigned)(s & 1) * 512u; }

// ---- a GRU transition's products and gates in one launch (gru_tile_kernel) ----

// The 64-byte steps of both products' rows in three parts: the first *nx of Wx, the others of Wh, the longer rows in two.
// Returns the stages of two steps that the longest part takes.
Q8_INDEX_FN int q8_gru_parts(int ldx, int ldh, int *nx, int *k0, int *steps)
{
    const int sx = (ldx + 63) / 64, sh = (ldh + 63) / 64;
    *nx = sx >= sh ? 2 : 1;
    const int two = *nx == 2 ? sx : sh, first = (two + 1) / 2, at = *nx == 2 ? 0 : 1;      // the part that the longer rows begin in
    k0[at] = 0;
    steps[at] = first;
    k0[at + 1] = first;
    steps[at + 1] = two - first;
    k0[*nx == 2 ? 2 : 0] = 0;
    steps[*nx == 2 ? 2 : 0] = *nx == 2 ? sh : sx;
    int most = first;
    if (sx + sh - two > most) most = sx + sh - two;
    return (most + 1) / 2;
}

// Tiles of 32 vectors per block: the fewest that leave a compute unit one block, four at most.
Q8_INDEX_FN int q8_gru_tile_columns(int H, int n)
{
    const int units = (H + 31) / 32, across = 256 / units > 0 ? 256 / units : 1, ct = ((n + 31) / 32 + across - 1) / across;
    return ct > 4 ? 4 : ct;
}

// Whether it is faster than the products and the gates apart.  Transitions alone (q8_gru_step panels, us, apart / in one launch):
// 64 + 64 bytes per row times 12 / 1024 vectors 10.9 / 7.3 and 12.0 / 8.5, H = 512, 512 + 256 bytes 10.8 / 8.2 and 20.3 / 12.0, H = 1000,
// 624 + 1008 bytes times 128 / 352 / 1024 12.3 / 11.1, 20.2 / 14.5 and 28.6 / 25.2, H = 1000, 2000 + 1008 bytes times 12 / 1024 14.6 / 12.7 and
// 37.5 / 32.3; but H = 1024, 1024 + 1024 bytes, row-major, times 12 / 128 11.1 / 13.8 and 13.5 / 14.4 (256: 16.4 / 15.0), H = 512,
// 1024 + 512 bytes, row-major, times 12 10.8 / 11.2, and more than a block per compute unit, H = 2048 times 700, 43.6 / 47.0.
// Where the codes of the new states are wanted they cost a launch of 4.8 us, which the gates' kernel apart makes by the way: us per decoder
// step with codes, apart / in tiles, H = 1000, 310 / 320 / 330 / 340 / 400 / 500 / 1000 vectors 58.1 / 61.2, 57.0 / 60.5, 67.4 / 62.4, 65.8 / 60.8, 67.6 / 62.3, 73.3 / 66.8, 99.1 / 91.9,
// H = 1024, packed, 337 / 350 / 500 / 1000 69.7 / 64.1, 60.9 / 55.6, 68.0 / 59.1, 99.3 / 89.2, row-major, E = 1024, 320 / 330 / 340 59.0 / 62.0, 67.4 / 68.4, 66.3 / 65.0 (up to 336 of
// E = 512 gru_panel_kernel's are 57); H = 300, 1000 vectors 55.3 / 57.1.  The line's other side gains too with fewer or more units: H = 512, 600
// vectors 51.2 / 49.0, H = 2048, 150 71.3 / 61.5.
// Rows of about the same length of both matrices leave one of the three parts half of all steps, and the products apart are at
// their best with rows of at most 1024 bytes (or whole 128 bytes of 2048): H = 1024, 1024 + 1024 bytes, 129 / 160 / 192 / 224 vectors 13.4 / 13.7 / 14.2 / 14.8 apart,
// 14.4 / 14.3 / 14.4 / 14.3 in one launch, H = 1000, 1008 + 1008 bytes, 129 / 160 / 176 11.3 / 11.9 / 13.4 and 12.1 / 12.3 / 12.4, H = 2048, 2048 + 2048 bytes, 129 / 176 / 224
// 21.5 / 24.7 / 26.0 and 23.8 / 25.1 / 25.4 (but H = 1400, 1408 + 1408 bytes, 129 20.8 and 18.0, and packed, H = 1024, 1024 + 1024 bytes, 129 / 144 / 176 10.9 / 11.1 / 12.8 and 11.3 / 11.4 / 11.5).
Q8_INDEX_FN int q8_gru_tile_better(int H, int ldx, int ldh, int n, int codes, int packed)
{
    const int cols = 32 * q8_gru_tile_columns(H, n), less = ldx < ldh ? ldx : ldh, more = ldx < ldh ? ldh : ldx;
    if ((long long)((H + 31) / 32) * ((n + cols - 1) / cols) > 256) return 0;
    if (codes) return (long long)n * H >= 340000;
    if (ldx + ldh < 1024) return 1;
    if (8 * less < 7 * more || (more > 1024 && less < 2048)) return n > 128;
    if (packed) return n > (more >= 1024 ? 144 : 128);
    return n > (ldx % 128 == 0 && ldh % 128 == 0 ? 192 : 160);
}

// ---- the encoder of one sentence (enc_one_kernel) ----

// Whether it is faster than encoder_persistent_kernel for a sentence of l words: a few don't pay for fetching both matrices into the
// registers of 64 blocks, above all not row-major ones (16 rows per request in place of one KiB).  q8_encode, us, the other / this:
// H = 1024, packed, rows of X of 512 bytes, 4 / 5 words 14.6 / 14.9, 17.0 / 16.3; 640, 5 / 6 words 17.0 / 17.0, 19.0 / 18.5; 1024, 7 / 8 words 21.1 / 21.6,
// 23.1 / 23.1.  H = 1024, row-major, 512, 5 / 6 words 16.9 / 17.3, 18.9 / 18.8; 640, 5 / 6 16.9 / 17.8, 18.9 / 19.4 (7: 20.9 / 21.2, 8: 23.1 / 22.7); H = 1000, 640,
// 5 words 17.0 / 16.9.  H = 512, packed, 1024, 1 / 3 words 9.0 / 8.0, 12.1 / 11.6.  Row-major: H = 256, 512, 1 / 3 words 9.0 / 8.2, 11.7 / 11.6; 704, 1 / 2 / 4 / 5 words
// 8.9 / 8.6, 10.0 / 10.5, 13.3 / 13.5, 15.2 / 15.2; 1024, 1 / 3 / 5 / 7 / 8 words 9.2 / 9.7, 11.7 / 13.4, 15.1 / 16.4, 18.6 / 19.4, 20.8 / 20.7.
Q8_INDEX_FN int q8_enc_one_better(int H, int ldx, int packed, int l)
{
    const int rows = !packed && H > 1000;
    if (H > 512) return l >= (ldx > 640 || (rows && ldx == 640) ? 8 : rows && ldx >= 512 ? 6 : 5);
    if (packed || ldx < 640 || H % 8) return 1;                        // (H % 8: the other is a launch per position)
    return ldx <= 704 ? l == 1 || l >= 5 : l >= (ldx <= 768 ? 7 : 8);
}

// ---- the batched encoder (enc_group_kernel) ----

#define Q8_ENC_UNITS 32
#define Q8_ENC_SLOTS 16
#define Q8_ENC_PITCH (1024 + 16)
#define Q8_ENC_TILE (16 * 16 + 32)      // ints per exchanged tile of sums: the unit tiles of a slot fall on different banks

// S sentences of H units: members of a set, sets per direction (as many as there are slots for, and as leave a compute unit at
// most one block), groups of a set with the most sentences and slots per group.  Returns the bytes of LDS, which grow with
// the groups (47872 for eight).
Q8_INDEX_FN unsigned q8_enc_plan(int H, int S, int *members, int *sets, int *groups, int *slots)
{
    *members = (H + Q8_ENC_UNITS - 1) / Q8_ENC_UNITS;
    const int most = 4 * (32 / *members);
    *sets = S < most ? S : most;
    const int ns = (S + *sets - 1) / *sets;
    *groups = (ns + Q8_ENC_SLOTS - 1) / Q8_ENC_SLOTS;
    *slots = (ns + *groups - 1) / *groups;
    return Q8_ENC_SLOTS * Q8_ENC_PITCH + 12 * Q8_ENC_TILE * 4 + (unsigned)*groups * (Q8_ENC_SLOTS * Q8_ENC_UNITS * 4 + Q8_ENC_SLOTS * 8);
}

// What the form that multiplies X itself adds: two turns of the codes of 16 rows of X, 2 xs steps of 64 bytes at a pitch that puts
// them on different banks, and of the sums, and the block's rows of Wx (none with xs = 0: the products of X are given).
#define Q8_ENC_X_PITCH(xs) (128 * (xs) + 16)
#define Q8_ENC_X_LDS(xs) ((xs) ? 2 * (Q8_ENC_SLOTS * Q8_ENC_X_PITCH(xs) + 12 * Q8_ENC_TILE * 4) + 12 * (xs) * 1024 : 0)
#define Q8_ENC_LDS_MOST 47872

// Whether S sentences of H units and up to max_l words run in that launch (else in one per time step, or three).  q8_encode_batch
// in us per batch, sentences of equal length, E = 512, a launch per time step / this: H = 1024, 9 sentences (one group per set) of 1 / 2 / 3 / 4 words
// 11.7 / 17.7, 17.4 / 20.4, 22.7 / 22.7, 28.3 / 24.8, 65 (two) 15.3 / 20.7, 25.1 / 26.4, 34.8 / 32.5, 43.8 / 37.1, 400 (seven) 35.5 / 41.4, 64.1 / 65.3, 98.1 / 91.5,
// 127.4 / 109.7.  With fewer units one group pays from 2 words on (H = 512, 9 sentences 16.8 / 15.6; H = 64, 257 sentences 17.7 / 14.9), two or three from 3
// (H = 512, 129 sentences 24.0 / 25.4, 33.6 / 30.7): 3 words are the line that no shape loses by.  From four groups on, whose launches
// per time step are of half the blocks, H <= 512 needs 6 to 7 words (H = 512, 400 sentences of 3 / 4 / 6 / 8 words 55.8 / 62.6, 70.0 / 74.6, 105.1 / 101.8, 139.2 / 127.3,
// 1024 sentences 99.8 / 105.7, 131.7 / 134.6, 197.0 / 188.0, 263.9 / 243.9; H = 256, 1024 sentences 67.6 / 73.2, 86.7 / 89.3, 126.2 / 125.2, 167.5 / 162.0).  A group of a
// set takes 2.6 us of a time step and more than eight lose to the three launches (measured when it took 4: 600 / 800 / 1024
// sentences of 1024 units, 10 words, 1.05 / 1.04 / 1.15 times as long, 400, seven groups, 0.81).
Q8_INDEX_FN int q8_enc_one_launch(int H, int S, int max_l)
{
    int members, sets, groups, slots;
    q8_enc_plan(H, S, &members, &sets, &groups, &slots);
    return groups <= 8 && max_l >= (H <= 512 && groups >= 4 ? 7 : 3);
}

// Where iteration `it` of a block (one group of slots at one time step, counted from the launch's first) keeps the scale of its
// slot: two sets of 16 in turn, because an iteration's scales are read while other waves write the next one's.
Q8_INDEX_FN int q8_enc_scale(int it, int slot) { return 16 * (it & 1) + slot; }
// ... and of its row of X: left there two iterations before it is read, while the scales of two before that are.
Q8_INDEX_FN int q8_enc_x_scale(int it, int slot) { return 16 * (it & 3) + slot; }
