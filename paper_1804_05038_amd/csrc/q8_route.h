// q8_route.h -- which kernel a panel product (q8i_gemm_jobs) takes: plain integer arithmetic on its sizes, the same in a host
// build, so that the tests of the kernels can be checked against the rule that the library follows.
#pragma once

enum q8_panel_kernel {
    Q8_ROUTE_STAGED,           // gemm_block_kernel
    Q8_ROUTE_RESIDENT,         // gemm_resident_kernel: rows of at most 512, and of at most 1024 bytes
    Q8_ROUTE_RESIDENT_1024,
    Q8_ROUTE_TILES_64,         // gemm_tile_kernel, 64 x 64 and 128 x 128
    Q8_ROUTE_TILES_128,
    Q8_ROUTE_ONCE_64X64,       // gemm_once_kernel, rows x vectors of a block
    Q8_ROUTE_ONCE_128X32,
    Q8_ROUTE_ONCE_128X64,
    Q8_ROUTE_ONCE_128X64_TRADE,
    Q8_ROUTE_STREAM            // gemm_stream_kernel
};

struct q8_panel_shape {
    int njobs, rows[3];        // products of the launch
    int n;                     // vectors
    int min_ld, max_ld;        // bytes per row of the products
    int plain;                 // no taps, no statistics, results vector by vector, operands below 2 GiB
    int packed;                // all weights tile-packed
    int steps, lines;          // all rows whole 64-byte steps, whole 128 bytes
    int whole;                 // all results in whole 16-byte pieces
};
typedef struct q8_panel_shape q8_panel_shape;

#define Q8_TILE_FILL (128LL * 128 * 128)       // results that are worth a launch of 128 x 128 tiles: 128 full ones

// blocks of rw rows x cw vectors that the launch's results touch
static inline long long q8_panel_blocks(const q8_panel_shape *s, int rw, int cw)
{
    long long b = 0;
    for (int t = 0; t < s->njobs; ++t) b += (long long)((s->rows[t] + rw - 1) / rw) * ((s->n + cw - 1) / cw);
    return b;
}

// Plain products with longer rows (kernel trace, us, each form beside the one that would run without it):
// rows of 513-1024 bytes: whole tiles at once, 128 rows x 32 vectors while these give a compute unit at most one block, else
//   x 64 (3072 x 1024 times 9 / 200 / 400 / 1000 vectors 4.6 / 5.3 / 7.2 / 10.4 against 5.3 / 6.6 / 8.7 K-resident and 13.8
//   in 128 x 128 tiles, 4096 x 1024 x 1000 11.4 against 15.5, 3000 rows of 1008 bytes, row-major, x 1000 11.2 against 14.6;
//   two such products of a decoder step times 100 / 320 4.8 / 7.2 against 6.2 / 7.5 with k split over two waves; x 32
//   beside x 64 vectors at 200 / 350 / 1000: 5.3 / 7.2 / 11.2 against 6.8 / 7.0 / 10.4), up to some 800 blocks, 700 of matrices
//   of more than 16384 rows: beyond, 128 x 128 tiles read less (50000 x 640 x 100 18.0 against 22.2, 20000 x 1024 x 300 22.0
//   against 23.6; 20000 x 640 x 200, 628 blocks, 18.0 against 18.1; two products of 3072 x 512 and x 1024 times 1000, 768 blocks,
//   17.4 against 14.2; 8192 x 1024 x 512 11.9 against 14.8), for more than 64 vectors, whole k steps, results in whole
//   16-byte pieces and no third of a tile past the vectors (33660 x 768 x 130 23.2 against 25.4, 50000 x 1024 x 130 31.6 against 34.5);
//   row-major rows of whole 128 bytes, which a compute unit takes in more slowly: 64 x 64 K-resident blocks, of half the
//   bytes, in place of x 32 where they are one round (3072 rows of 640 / 768 / 1024 bytes times 9 5.3 / 5.1 / 5.6 against 6.2 / 6.2 / 7.1,
//   times 64 6.2 / 6.2 / 6.6 against 6.4 / 6.6 / 7.4; 20000 x 640 x 9, two rounds, 7.4 against 6.4), x 64 with the trade;
//   the same for up to 8 vectors, which the batched step of few slots has (the staged kernel elsewhere; step of 1 / 4 / 8 slots, H = 1024,
//   packed, 37.8 / 40.7 / 41.7 against 39.3 / 43.0 / 43.9 staged and 39.2 / 41.6 / 42.6 with k split over two waves);
// rows of 1025-2048 bytes: 64 rows x 64 vectors at once where these nearly fill one round (1024 x 2048 x 1024 8.4 against
//   11.0 in 64 x 64 tiles, 9.6 streamed; 3000 x 2000 x 300, row-major, 9.0 against 13.0 staged, 9.9 streamed), else the weights
//   kept for a stream of vectors (1024 x 2048 times 30 / 130 6.3 / 6.5 against 9.0 / 9.1, 6.7 / 7.0 at once; 3072 x 2048 times
//   400 / 700 10.9 / 14.8 against 13.6 / 17.3; 2000 x 1500 x 700, row-major, 11.9 against 14.4), unless the rows' last
//   parts are mostly padding or a launch has many rounds (3072 x 1280 x 1000 17.7 against 15.9 in 128 x 128 tiles,
//   3072 x 2048 x 1000 18.2 in a decoder step against 17.4; 33658 x 2048 x 64 30.7 against 23.3 in 64 x 64 tiles);
// longer rows, and what is left: 128 x 128 tiles where the results fill enough of them (Q8_TILE_FILL), 64 x 64 tiles for packed
//   rows (8200 x 2048 times 9 / 64 / 200 9.2 / 9.7 / 19.2 against 17.3 / 18.8 / 22.5 staged), the staged kernel for row-major
//   ones, of which it requests a whole 128 bytes at a time.
static inline int q8_panel_route(const q8_panel_shape *s)
{
    long long rows = 0, results;
    if (!s->plain || (s->n <= 8 && (s->min_ld <= 512 || s->max_ld > 1024))) return Q8_ROUTE_STAGED;
    if (s->max_ld <= 512) return Q8_ROUTE_RESIDENT;
    for (int t = 0; t < s->njobs; ++t) rows += s->rows[t];
    results = rows * s->n;
    if (s->min_ld > 1024 && s->max_ld <= 2048) {
        const long long b = q8_panel_blocks(s, 64, 64);
        if (b > 150 && b <= 256) return Q8_ROUTE_ONCE_64X64;
        if (q8_panel_blocks(s, 64, s->n) <= 256 && b * 2048 <= 640LL * s->max_ld) return Q8_ROUTE_STREAM;
    } else if (s->max_ld <= 1024) {
        if (q8_panel_blocks(s, 128, 32) <= 256) return !s->packed && s->lines && q8_panel_blocks(s, 64, 64) <= 256 ? Q8_ROUTE_RESIDENT_1024 : Q8_ROUTE_ONCE_128X32;
        if (q8_panel_blocks(s, 128, 64) <= (rows > 16384 ? 700 : 800) || s->n <= 64 || (s->n > 128 && s->n <= 192) || !s->steps || !s->whole || results < Q8_TILE_FILL)
            return !s->packed && s->lines ? Q8_ROUTE_ONCE_128X64_TRADE : Q8_ROUTE_ONCE_128X64;
    }
    if (results >= Q8_TILE_FILL && (s->max_ld <= 1024 || s->n > 64 || !s->packed)) return Q8_ROUTE_TILES_128;
    return s->packed ? Q8_ROUTE_TILES_64 : Q8_ROUTE_STAGED;
}

// Tiles of 16 rows per block of gemm_quant_kernel for n vectors of a product: the fewest that need one round of blocks, four at
// most; 0 where quantization and product in two launches are faster, which is where too many blocks of four tiles quantize
// the same vectors again: more than 256 of them with rows of more than 1024 bytes, 550 of more than 512, 850 of fewer.  us per
// call, two launches / one: 1024 rows of 2048 bytes, packed, times 9 / 30 / 128 / 256 / 400 vectors 8.0 / 4.1, 8.3 / 4.3, 8.7 / 4.9, 9.1 / 5.8, 9.7 / 10.2;
// 3072 x 2048, row-major, times 64 / 100 11.2 / 7.0, 11.6 / 12.5; 1024 x 1024, row-major, times 400 / 700 9.0 / 7.3, 9.8 / 10.0; 2000 x 620 times 256 / 400
// 8.0 / 6.2, 8.1 / 9.5; 1024 x 512 times 64 / 700 6.7 / 3.5, 7.6 / 6.6; 8192 x 512, row-major, times 64 / 100 / 200 7.7 / 5.3, 7.6 / 7.6, 9.6 / 12.0.
static inline int q8_quant_rows(int rows, int ld, int n)
{
    const long long tiles = (rows + 15) / 16, groups = (n + 15) / 16;
    if (n <= 8 || ld > 2048 || (tiles + 3) / 4 * groups > (ld > 1024 ? 256 : ld > 512 ? 550 : 850)) return 0;
    return tiles * groups <= 256 ? 1 : tiles * groups <= 512 ? 2 : 4;
}

// The same for products of codes that are there already (gemm_part_kernel), all of a launch: 0 where the kernel of q8_panel_route is
// as fast or faster, which is where more than 256 blocks of four tiles read the same operands again, and rows of at most 512
// bytes (K-resident).  Four decoder steps at beam 5, us, without / with it: rows of 624 / 1008 / 2000 bytes, 4 / 12 sentences 325 / 291, 354 / 331,
// and with up to 64 blocks per vector group, 30 / 64 sentences 400 / 411, 490 / 545; rows of 512 / 1024 / 2048 bytes, 4 sentences 292 / 285.
static inline int q8_part_rows(const q8_panel_shape *s)
{
    long long tiles = 0, blocks = 0;
    const int groups = (s->n + 15) / 16;
    if (!s->plain || s->n <= 8 || s->max_ld > 2048 || s->max_ld <= 512) return 0;
    for (int t = 0; t < s->njobs; ++t) { tiles += (s->rows[t] + 15) / 16; blocks += (s->rows[t] + 63) / 64; }
    if (blocks * groups > 256) return 0;
    return tiles * groups <= 256 ? 1 : tiles * groups <= 512 ? 2 : 4;
}
