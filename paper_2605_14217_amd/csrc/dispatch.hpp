// What the host knows about a batch before its schedule exists, and the rules that choose from it: launch sizes, the small-batch
// kernel and its shape.  Host code without state; preft_api.hip launches by it, tests ask it.
#pragma once
#include "common.hpp"
#include "small_kernel.hpp"

#include <cmath>

namespace preft {

// Kernel selection for tests and benchmarks, carried by the mode argument of the call itself
// (PREFT_TEST_* of the public header): the library keeps no state between calls.
struct Knobs {
    int variant, waves, rowblocks, colsplit, resident;
};

// Upper bound of the units of a tile-kernel launch of height `rows`, from host-visible sizes,
// rounded to the 8 XCDs.
inline unsigned tile_grid(const ApplyArgs &a, int64_t S, int rows)
{
    const int64_t per_gtile = rows >= GTILE_ROWS ? 1 : GTILE_ROWS / rows;
    int64_t units = gtile_capacity(a.T, S, a.N) * per_gtile;
    if (!a.gathered_only) units += chunk_capacity(a.T, S) * (CHUNK_ROWS / rows);
    return (unsigned)(((units + 7) / 8) * 8 * (a.col_split > 1 ? a.col_split : 1));
}

// How many of N adapters n segments are expected to name.
inline int64_t likely_adapters(int64_t n, int64_t N)
{
    if (n <= 0 || N <= 0) return 0;
    return (int64_t)((double)N * -expm1(-(double)n / (double)N) + 0.5);
}

// How many 16-row tiles a batch is likely to have.  Rows in excess of one per segment belong to prompts: a prompt ends in a
// partial tile; the other segments, where every position counts, are gathered by adapter, which ends in a partial tile each.
inline int64_t likely_gathered(const ApplyArgs &a, int64_t S)
{
    const int64_t extra = a.T > S ? a.T - S : 0, prompts = S < extra / 16 + 1 ? S : extra / 16 + 1;
    int64_t singles = a.all_tokens ? (a.T < S ? a.T : S) - (extra ? prompts : 0) : 0;
    if (singles < 0) singles = 0;
    const int64_t owners = likely_adapters(singles, a.N), gathered = singles / 16 + owners / 2;
    return gathered > owners ? gathered : owners;
}
inline int64_t likely_tiles(const ApplyArgs &a, int64_t S)
{
    const int64_t extra = a.T > S ? a.T - S : 0, prompts = S < extra / 16 + 1 ? S : extra / 16 + 1;
    return extra / 16 + (extra ? prompts / 2 + 1 : 0) + likely_gathered(a, S);
}

// Whether what a call reads and writes of its activations (once each, `es` bytes an element) is little enough, with the factors that pass by, for the memory-side cache (256 MB) to still hold it
// from the kernel before, and for the kernel after: then it is read without the non-temporal hint, which has it fetched from memory.  y has just been written when a call adds to it, so
// what decides is how much passes between that kernel and this one.  Hint / none, us, the same buffers again, two in turn, four in turn (from 64 MB on these have left the cache): single launches:
// fp32, rank 16, 4096 -> 4096, 38 MB 22.4 / 21.9, 22.0 / 21.0, 21.7 / 20.7, 56 MB 25.1 / 24.2, 24.3 / 23.1, 23.9 / 23.9, 75 MB 32.6 / 29.3, 31.8 / 27.8, 32.0 / 35.8, 112 MB 37.5 / 33.8, 36.6 / 34.3, 37.1 /
// 41.4, 187 MB 64.0 / 57.5, 64.8 / 71.5, 68.3 / 73.0; rank 20, 1000 -> 2072 (rows off lines), 70 MB 38.1 / 33.8, 38.9 / 33.2, 39.7 / 37.1; rank 31, 3760 -> 600, 70 MB 34.2 / 30.1, 36.4 / 29.7, 36.8 / 35.4.
// Expands of two launches: rank 32, 4096 -> 4096, 56 MB 27.5 / 26.5, 27.2 / 25.9, 26.6 / 25.3, 75 MB 35.5 / 35.6, 35.1 / 35.1, 35.2 / 38.9; rank 64, 8192 -> 8192, 56 MB 30.8 / 29.4, 30.2 / 29.3,
// 30.2 / 31.4, 75 MB 39.5 / 38.5, 39.0 / 38.1, 39.2 / 43.7.  Column-split kernel, four in turn, 71 MB, 4096 decode rows, rank 48, 488 -> 8192 41.2 / 46.3.  So fp32 goes
// without it up to where three such calls fill the cache, bf16, which gains less, up to where four do.
// Below the size of the L2s together (32 MB) the lines of y that were read plainly are written back at the end of the kernel: rank 64, 4096 -> 4096, 28 MB 19.1 / 19.8, 19.2 / 19.5, 18.5 / 19.2; fp32, rank 4,
// 1024 -> 1024, 23 MB 9.8 / 10.9, 11.0 / 11.6, 11.5 / 11.2, 33 MB 16.8 / 19.0, 18.1 / 18.9, 17.5 / 18.4.  In place in fp32 (the tile is read twice in either form) 47 MB 30.4 / 30.7, 75 MB 51.2 / 59.2: always the hint.
// Factors count: 4096 decode rows of 512 adapters, rank 44, 4936 -> 896 (48 MB of activations, 260 of factors) 54.1 / 57.7.
constexpr int64_t STAY_F32 = (int64_t)76 << 20, STAY_BF16 = (int64_t)64 << 20;
inline bool activations_stay(const ApplyArgs &a, int64_t S, int64_t width, int es, int64_t most)
{
    const int64_t activations = a.T * (a.d_in + width) * es, factors = likely_adapters(S, a.N) * a.rank * (a.d_in + width) * es;
    return activations >= ((int64_t)(es == 4 ? 36 : 32) << 20) && activations + factors <= most;
}

// The same for the two launches of an in-place call: the expand reads h again where the shrink has read it, and neither has the hint.  Hint in the shrink, and in the expand from 76 MB on /
// none, us, the same buffer again, two in turn, four in turn: rank 64, d = 4096, 14 MB 35.6 / 39.1, 37.4 / 39.3, 38.2 / 38.9; 23 MB 43.8 / 41.5, 43.9 / 41.6, 43.9 / 40.5; 47 MB 54.0 / 49.6, 53.3 / 48.4, 53.0 /
// 48.3; 61 MB 59.7 / 54.2, 59.4 / 53.4, 60.0 / 59.2; 98 MB 78.5 / 69.1, 76.6 / 67.8, 76.0 / 79.1; 126 MB 99 / 87, 99 / 103, 98 / 112; 187 MB 125 / 112, 123 / 138, 123 / 145; 8192, 19 MB 62.1 / 60.0, 62.7 /
// 60.4, 63.0 / 60.2, 56 MB 79.1 / 72.4, 78.6 / 71.7, 78.6 / 73.7, 122 MB 104 / 94, 105 / 105, 105 / 110; 14336, 66 MB 118 / 105, 118 / 104, 118 / 115; rank 48 alike; rank 96, 4096, 61 MB 73.3 / 69.6, 72.7 / 70.5,
// 73.7 / 71.8, 126 MB 117 / 108, 112 / 119, 112 / 123.  h that is still in the cache gains up to 200 MB, h that is not loses from 76 MB on: so up to 64.
inline bool h_stays(const ApplyArgs &a)
{
    const int64_t bytes = a.T * (int64_t)a.d_in * 2;
    return bytes >= ((int64_t)20 << 20) && bytes <= ((int64_t)64 << 20);
}

// In place at rank 20-32, rows of 9216 and more: whether every wavefront of the 32-row tiles keeps 8 of its units in registers between the sweeps.  That costs
// half the wavefronts of a compute unit (40 of its registers are spilled besides, 84 bytes a lane); a tile of such rows (576 KB at 9216) does not outlast its first sweep in an XCD's L2 in any
// case.  All streamed / 8 kept, us, two buffers in turn, prompts of 600 rows: rank 32, d = 9216 / 10240 / 14336 / 28672, 6000 rows 62.6 / 61.8, 72.3 / 70.2, 102 / 103, 242 / 230; 12 000 rows 134 /
// 122, 158 / 140, 224 / 201, 457 / 444; 18 000 rows 233 / 190, 271 / 216, 367 / 310, 714 / 646; 30 000 rows 344 / 321, 401 / 364, 564 / 519, 1144 / 1083; 72 000 rows 713 / 712, 808 / 782, 1128 /
// 1083, 2408 / 2321; rank 20, 72 000 rows 645 / 645 (9216), 756 / 754; 4 layers of 1600 rows, 10240 132 / 73.  8192 and narrower: rank 32, 12 000 rows 109 / 106, 60 000 505 / 515, 4096 54 / 56,
// 2048 30 / 33, rank 20, 8192 99.5 / 104.8.
// Short segments leave the tiles part-empty, and the streamed form has more of them on their way: rank 20, 8320, 2500 rows in 239 prompts 122 / 170; rank 32, 12288, 2200 in 143 158 / 183, 10256, 3100 in
// 66 113 / 118; 4 layers, rank 28, 14336, 2600 in 225 552 / 898, rank 20, 14336, 1600 in 25 144 / 152; 12 000 in 120 231 / 212.
// And where the tiles are about as many as the compute units, the wavefronts that are missing are not made up for by another round of tiles: 7700 rows, 9216 / 10240 / 12288, rank 20 1.14 / 1.08 / 1.06 of the time of the
// streamed form, 24 1.11 / 1.06 / 1.04, 28 1.09 / 1.04 / 1.02, 32 1.03 / 0.98 / 0.95 (5000 rows 0.97 / 0.98 / 0.97, 9300 0.91-1.01, 0.92-0.99, 0.91-0.98); 8320, 5000 to 12 000 rows 0.93-1.15.
inline bool keeps_units(const ApplyArgs &a, int64_t S)
{
    if (a.d_in < 9216 || a.T < 72 * S || (a.d_in < 12288 && a.T > 6144 && a.T <= 8704)) return false;
    return a.d_in >= 10240 || a.T <= 32768;
}

// Small batches take a kernel of their own (small_kernel.hpp).
// Rows of segments of more than one row, if no segment is empty: prompts.  A step of decode rows alone has none, and where only
// prompt positions count it has next to nothing to do: its launches are sized for that (a kernel strides over what exceeds its grid).
inline int64_t prompt_rows(const ApplyArgs &a, int64_t S) { return a.T > S ? a.T - S : 0; }

// Units of a 16-row launch that a small batch is likely to list: 8 for every chunk, prompts of 16 rows and more; every gathered tile
// that all-position rows can make, and a few of prompts' short ends.
inline unsigned likely_units(const ApplyArgs &a, int64_t S)
{
    const int64_t rows = a.gathered_only ? 0 : prompt_rows(a, S), chunks = rows ? rows / CHUNK_ROWS + (rows / 16 < S ? rows / 16 : S) + 2 : 0;
    const int64_t gathered = gtile_capacity(a.T, S, a.N), units = chunks * (CHUNK_ROWS / 16) + (a.all_tokens || gathered < 8 ? gathered : 8);
    const unsigned bound = tile_grid(a, S, 16), likely = (unsigned)((units + 7) / 8 * 8);
    return likely < bound ? likely : bound;
}

// The column-split kernel keeps byte offsets within a first factor in 31 bits: up to the first 128 columns of the last rank's row (rank 127: 8.5
// million columns, 64: 17, 16: 71 million).  Beyond, the row-split kernel takes chunks of whole 128-column units, and the
// per-row kernels the rest; both count in 64 bits.
inline bool column_split_fits(const ApplyArgs &a) { return (int64_t)(a.rank - 1) * a.d_in + 128 <= ((int64_t)1 << 30); }

// widths the row-split shape with `cw` column groups takes
inline bool wide_widths_ok(const ApplyArgs &a, int cw)
{
    const int m = 128 * cw;
    return (a.d_in % m) == 0 && (a.d_out % m) == 0;
}

// Whether the matrix-core kernels take a bf16 call: from rank 4 on (ranks 1..3: the small-batch kernel, whose shrink is theirs, or the vector-ALU kernel).
inline bool mfma_takes(const ApplyArgs &a, const Knobs &k)
{
    if (a.rank < 4) return false;
    if (a.rank > 16 && wide_widths_ok(a, 1) && k.variant != 3) return true;      // the row-split kernel, its gathered tiles apart
    // the column-split kernel; ranks above 16 that are no multiple of 4 up to the widths of the small-batch kernel
    const bool narrow = a.d_in <= (1 << 22) && a.d_out <= (1 << 22);
    return column_split_fits(a) && ((a.rank % 4) == 0 || a.rank < 16 || wide_widths_ok(a, 1) || narrow);
}

constexpr int32_t SMALL_T = 1024;
constexpr int32_t SMALL_WIDTH = 1 << 22;                      // offsets within a row or a factor, and the launch, fit 32 bits
constexpr int64_t DEEP_WGS = 200;                             // at most one workgroup per compute unit, with room for a poor estimate

// Up to rank 16 the small-batch kernel stays ahead of the two launches (and of the single ones) beyond SMALL_T rows as long as the call is no long stream: the
// elements of x, of y twice and of the factors of the likely adapters.  What then costs it is that the shares of a tile repeat its shrink.  Two launches (or one) / this kernel, us:
// rank 16, 2000 rows of prompts of 400 beside 32 adapters, 512 -> 2072 (9 million elements) 8.3 / 7.1, 4096 -> 4096 (27) 17.0 / 13.9, 14336 -> 4096 (51) 30.9 / 22.9, 8192 -> 8192 (58)
// 27.1 / 28.2, 4096 -> 2 x 14336 (127) 51.7 / 69.8; 5000 rows, 4096 -> 512 16.4 / 13.2, 4096 -> 4096 (64) 31.9 / 24.2, 1024 -> 4096 + 2 x 1024 (68) 33.6 / 27.5, 14336 -> 4096 (118)
// 57.2 / 65.4, 8192 -> 8192 (127) 53.2 / 67.0; 2200 rows of prompts of 55, 4096 -> 4096 24.5 / 15.1; 2000 decode rows of 64 adapters, 8192 -> 8192 (65) 32.6 / 24.2, of 500, 4096 -> 512 (46)
// 22.2 / 17.5, 4096 -> 4096 (89) 32.0 / 32.3, 1024 -> 4096 + 2 x 1024 (82) 35.0 / 40.9.  Ranks 8 and 11 alike.  Rank 3, 5000 rows, 4096 -> 4096 31.1 / 21.3, 8192 -> 8192 51.7 / 56.0; 4000
// decode rows of 64 adapters, 4096 -> 2 x 14336 (265) 136 / 119; rank 1, 2000 of 500, 4096 -> 512 7.7 / 9.0.
constexpr int32_t SMALL_STREAM_T = 6144;
inline bool no_long_stream(const ApplyArgs &a, int64_t S, int64_t width)
{
    // Above rank 16 the small-batch kernel's order, in one launch or (small_in_two, room for z) two, against the kernels of larger batches: those have a workgroup for
    // every 64 or 128 rows, which leaves most of the chip idle up to 4096 rows.  The sums of z differ between the two, so the choice cannot depend on the room: it is
    // made where neither the call with room nor the one without is slower.  This order / theirs over random calls of 1025 to 6144 rows, geometric mean with room, without (slower calls of
    // all): whole widths (multiples of 128), rank 20-32 0.63, 0.45 (0 of 114), 36-64 0.63, 0.40 (4 of 155), 68-128 0.22, 0.34 (0 of 165); others 0.63, 0.60 (1 of 101), 0.57,
    // 0.56 (0 of 61), 0.48, 0.67 (6 of 82), none by more than a fifth.
    // What is left to them, as the single launch with its repeated shrink or the second launch is often the slower: decode rows, whose tiles they gather too, 0.90, 0.89 (91 of 453 slower, up to
    // 1.6); above rank 32 segments of fewer than 20 rows on narrow inputs, above rank 64 and 2048 rows of fewer than 64, 0.51, 0.83 (21 of 115, up to 1.8), ragged outputs of up to 512
    // columns, 1.03, 0.95 (19 of 55, up to 1.5; up to rank 32 above 3072 rows, rank 24, 512 -> 88, 5258 rows 5.5 / 10.0, 8.3), and those wider than 4096 above 1536 rows, 0.42, 0.73 (21 of 122, up to 1.8), all ragged ones above 4096 rows 0.65, 0.90 (34 of 163).
    if (a.rank > 16) {
        if (a.rank % 4 || (a.all_tokens && a.T < 2 * S)) return false;
        const bool ragged = a.d_in % 128 || width % 128;      // (not each width: packed calls with one ragged output have the others wide)
        if (ragged && width <= 512 && a.T > (a.rank <= 32 ? 3072 : SMALL_T)) return false;
        if (a.rank <= 32) return a.T <= 4096 || (a.T <= SMALL_STREAM_T && (ragged || a.d_in >= 2048));
        if ((a.T < 20 * S && a.d_in <= 1024) || (a.rank > 64 && a.T > 2048 && a.T < 64 * S)) return false;
        if (ragged) return a.T <= (width <= 4096 ? 4096 : 1536);
        if (a.rank > 64 && width > 8192 && a.T > 3072) return false;           // rank 128, 8192 -> 14336, 3500 rows without room 438 / 475 (with room 96, 121 as 64-row tiles in two launches)
        return a.T <= 4096 || (a.T <= SMALL_STREAM_T && a.d_in >= 2048 && width <= 16384 && a.rank <= 64);
    }
    if (a.T > SMALL_STREAM_T) return false;
    const int64_t d = a.d_in, singles = a.all_tokens && a.T < 2 * S;
    // Narrow inputs and outputs: rank 16, 1104 -> 1024, 1080 prompt rows 5.4 / 5.7, 768 -> 1296, 3500 7.1 / 7.7, rank 12, 2304 -> 1024, 2000 in 106 prompts 10.4 / 11.6; up to 3200 rows rank 8, 2048 -> 2048, 1600
    // / 2000 / 2800 7.4 / 8.2, 8.0 / 9.1, 9.4 / 10.3, 1024 -> 2048 6.8 / 7.2, 7.0 / 7.5, 8.2 / 9.0, rank 16, 1024 -> 2144, 3200 9.4 / 11.6 (4000 rows,
    // 2048 -> 2048 17.1 / 14.0; ranks that are no multiple of 4, rank 5 and 9, 1600 to 2800 rows 7.2-10.0 / 6.4-10.0).
    if (a.rank >= 4 && d <= 2304 && (width <= 1296 || (width <= 2176 && a.T <= 3200 && !singles && a.rank % 4 == 0))) return false;
    // (rank 1, 1024 -> 1024, 1300 rows 4.8 / 5.9, rank 2, 512 -> 1024, 2300 in 241 prompts 7.1 / 10.5)
    if (a.rank <= 2 && d <= 1024 && width <= 1024) return false;
    if (a.rank >= 4 && !singles && d > 8192 && width > 4096) return false;   // rank 11, 14336 -> 5176, 1470 prompt rows 26.7 / 42.5, rank 16, 14336 -> 5832, 1490 31 / 38, 4224, 1720 28 / 36 (rank 5, 14336 -> 4448, 1300 26 / 18)
    if (width > 10240 && !(a.rank < 4 && singles)) return false;          // rank 8, 912 -> 14336 + 4096 + 1512, 1240 prompt rows 28.3 / 34.0
    // (8192 -> 6144, rank 12, 1600 rows (33) 21.7 / 24.2, 2800 (57) 28.2 / 31.5)
    // (and where the activations have left the caches its order over y costs more than the expand's: four sets of buffers in turn / two, geometric mean of the time before over random calls of rank 4-16 of 40 to 56
    // million 0.90 / 0.88, of 56 to 76 1.05 / 0.92: rank 16, 4096 -> 3072 + 184, 6000 rows (64) 36.6 / 43.3, rank 11, 112 -> 1024 + 8192, 3400 (62) 30.1 / 38.3)
    const int64_t elements = a.T * (d + 2 * width) + likely_adapters(S, a.N) * a.rank * (d + width);
    const int64_t most = a.rank < 4 && singles ? 120000000 : d >= 8192 && width > 4608 && a.T >= 8 * S ? 24000000 : 56000000;
    return elements <= most;
}

// `widest`: columns of the widest output, `width`: of all outputs
inline bool takes_small(const ApplyArgs &a, int64_t S, int32_t widest, int64_t width, bool direft, const Knobs &k)
{
    if (a.rank < 4 && (k.variant || k.colsplit)) return false;            // those name the vector-ALU kernel there
    if (a.d_in > SMALL_WIDTH || widest > SMALL_WIDTH) return false;
    if (k.resident == 2 && a.rank > 16 && a.rank % 4 == 0) return true;
    if ((k.variant != 0 && k.variant != 5) || k.waves || k.rowblocks || k.resident) return false;
    if (!direft && k.colsplit) return k.colsplit > 1;
    // Ranks 1 and 2, next to nothing to expand: the vector-ALU kernel / this, us: rank 1, 8192 -> 512, 41 rows 4.8 / 6.9, 14336 -> 1024, 19 rows 6.5 / 9.6, 7040 -> 512, 850 rows 5.5 / 6.8, 2048 -> 408, 14 rows 3.7
    // / 4.1 (d_in from 4 to 8 times the columns, 10 calls 0.93, 8 times and more, 8 calls 1.14; below 4 times 0.77 and less); rank 2, 9016 -> 1024, 8 rows 6.6 / 7.4, 4096 -> 88, 1100 rows 8.6 / 9.9.
    if (!direft && (a.rank == 1 ? 4 : 8) * width <= a.d_in && a.rank <= 2) return false;
    // (and many rows of narrow prompts: rank 1, 512 -> 1024, 585 rows 4.7 / 6.1, 240 -> 1024, 504 4.5 / 5.6; up to 300 rows 0.87-1.03 of the time)
    if (!direft && a.rank == 1 && a.d_in <= 1024 && width <= 1024 && a.T > 384 && !(a.all_tokens && a.T < 2 * S)) return false;
    // A very wide output beside narrow ones: every share of these repeats the shrink as well, and the wide one's take 64 units where 32 of 8192 columns do: 4096 -> 136 + 208 + 8448, 2900 rows, rank 4 33.3 /
    // 47.5, 16 37.4 / 52.6; decode rows, rank 2, 2048 -> 256 + 384 + 14336, 4096 73 / 85 (4096 -> 512 + 8192, rank 16 32.7 / 33.4).
    if (!direft && a.T > SMALL_T && widest > 8192 && width > widest && 4 * (width - widest) < widest) return false;
    if (!direft) return a.T <= SMALL_T || (k.variant == 0 && no_long_stream(a, S, width));
    if (a.T > SMALL_T) return false;
    // In place the resident shapes of mfma_tile_kernel stay ahead up to rank 16 where their tile fits (rank 16, d = 4096, 1000
    // rows 11.4 and 13.1 us; d = 1000 6.4 and 5.4; rank 7, 4096: 14.6 and 11.5, 8192: 18.4 and 19.5;
    // rank 32, 4096: 24.3 and 17.3; rank 64, 8192, 1000 rows: 155 and 81)
    if (likely_tiles(a, S) > 200) return false;               // whatever n_layers: a layer's result is that of its one-layer call, bit for bit
    // Above rank 64 (128-row tiles / this, one launch either way, d = 512 / 2048 / 4096 / 8192, 300 prompt rows, rank 68 22.8 / 10.5, 67 / 25, 124 / 43, 252 / 80, rank 128 23.7 / 14.7, 69 / 41, 131 / 75, 272 / 146;
    // 32 decode rows, rank 128, 16-row tiles of the column-split kernel, 17.0 / 14.5, 44 / 39, 81 / 75, 149 / 141)
    if (a.rank > 64) return a.rank % 4 == 0;
    if (a.rank > 16) return true;
    // A few decode rows of an adapter each: tiles of which this kernel loads a quarter.  Rank 16, 32 rows of 32 adapters, resident / this, us: d = 4096 9.2 /
    // 8.2, 8192 14.8 / 13.2, 8 layers of 4096 17.5 / 13.6; rank 7, 8192 17.5 / 15.3; d = 14336 (streamed) 27.6 / 22.4; but 256 rows of 200 adapters
    // 12.5 / 13.6, of 32 10.4 / 11.0, and 8 layers of 46 tiles, more than a tile for every compute unit, 22.0 / 25.0.
    // That is for adapters drawn alike.  Where a few of them have most of the rows their tiles are full, and this kernel reads h twice: 16-64 rows of 8-64 adapters,
    // the i-th as likely as 1 / i^1.1, d = 4096, rank 8 and 16 9.1-10.3 / 10.5-10.7, 7 11.4-11.8 / 11.2-11.5, 8192, rank 16 15.1-16.9 / 17.2-18.7, 14336 25.8-28.3 /
    // 25.4-29.6.  The host cannot tell the two apart.
    if (a.all_tokens && prompt_rows(a, S) == 0 && likely_tiles(a, S) <= 32 && a.T <= 3 * likely_tiles(a, S)) return true;
    // Ranks 1-3, rows resident in a wavefront's registers / this, us: rank 1, d = 1024, 250 and 920 prompt rows 3.6 / 3.7, 4.2 / 3.9, 4096 7.6 / 7.1, 512 decode rows 8.2 /
    // 7.2, rank 3 9.7 / 8.4, 11.2 / 9.3, 11.1 / 8.6; but rank 1, d = 512, 250 rows 3.2 / 3.4.
    // rank 3, prompts of 7 rows, d = 128, 105 rows 4.3 / 5.4, 96 4.6 / 5.7.
    if (a.rank < 4 && a.d_in <= (a.rank == 1 ? 512 : 256)) return false;
    // Many part-empty tiles fill the chip with the layers of a call, each of which takes the kernel of its one-layer call: 8 layers, rank 2, d = 896, 81 rows in 74 tiles 6.7 / 9.2; 4 layers, rank 2, 3456,
    // 300 rows in 57 prompts 14.4 / 17.0 (full ones too, but one layer of those gains: 4 layers, rank 1, 2048, 360 rows in 31 tiles 7.0 / 9.0).
    // Narrow rows, full tiles too: 8 layers, rank 3, d = 512, 557 rows 12.8 / 17.5.
    if (a.rank < 4 && likely_tiles(a, S) > 24 && (a.d_in <= 512 || a.T < 8 * likely_tiles(a, S))) return false;
    // and wide rows of fuller tiles than a few decode rows: rank 1, d = 4096, 150 prompt rows 6.4 / 7.2, 74 decode rows of 3 adapters 6.4 / 7.3, rank 2, 230 prompt rows 7.2 / 7.9, 396 7.4 /
    // 8.2 (482 9.5 / 8.2; 160 decode rows of 313 adapters 7.1 / 5.3)
    if (a.rank <= 2 && a.d_in > 2048 && a.T <= 448 && a.T > 5 * likely_tiles(a, S)) return false;
    return (a.rank % 4) ? a.d_in <= 4096 : a.d_in <= 2048;
}

// a call of one output, or in place
inline bool takes_small(const ApplyArgs &a, int64_t S, int32_t width, bool direft, const Knobs &k) { return takes_small(a, S, width, width, direft, k); }

// In place its form for tiles of up to four rows runs for steps of decode rows alone (others pay 0.1 of 4.5 us for a second copy of the code).
inline bool small_in_place_few(const ApplyArgs &a, int64_t S) { return a.all_tokens && prompt_rows(a, S) == 0; }

// Whether a call of the small-batch kernel's order at rank 17 and up (multiples of 4) runs its sweeps as two launches: then a tile's shrink is not repeated
// by every share of its columns, and the expand shares its factors among 32 or 64 rows.  `width`: of all outputs.
// But it is a second chain of launch arguments, schedule and memory.  One launch / two, us, 32 decode rows of 32 adapters, 300 and 880 prompt rows: 4096 -> 4096, rank 48 12.5 / 14.0, 12.6 / 12.0, 18.4 /
// 13.9, rank 64 15.7 / 15.2, 15.7 / 12.1, 26.9 / 14.7, rank 96 21.3 / 17.8, 22.9 / 13.3, 34 / 17; 512 -> 2072, rank 48 5.6 / 8.6, 6.0 / 8.9, 7.4 / 8.8, rank 64 6.7 / 8.6, 7.1 / 8.9, 10.2 / 8.9, rank 128 10.8 /
// 10.9, 10.4 / 9.7, 18.1 / 11.0; rank 32, 8192 -> 8192 12.0 / 17.0, 15.3 / 15.8, 21.0 / 20.9.  In place, d = 8192, rank 20 20.1 / 15.1, 23.5 / 18.2, 25.7 / 25.8, rank 32 19.6 / 18.4, 22.2 / 20.2, 24.9 / 28.1;
// d = 4096, rank 32 11.7 / 11.6, 13.9 / 14.4, rank 48 20.5 / 14.6, 22.3 / 14.2, 23.1 / 16.5; d = 512, rank 48 6.2 / 8.7, 6.7 / 8.7, rank 64 8.6 / 8.9, 9.1 / 8.7, rank 128 (16-row tiles of the
// column-split kernel, 128-row tiles) 16.6 / 10.0, 23 / 9.8.
inline bool small_in_two(const ApplyArgs &a, int64_t S, int64_t width, bool direft, const Knobs &k)
{
    if (a.rank <= 16 || a.rank % 4 || k.variant == 5 || k.colsplit) return false;
    if (k.resident == 2) return true;
    const bool singles = a.T < 2 * S;
    if (!a.all_tokens && prompt_rows(a, S) < 64) return false;            // hardly a row to do
    // Above SMALL_T rows a second launch costs 2 to 4 us, and what it saves are the shrinks that the shares of the outputs repeat.  Two launches / one over random prompts of 1025 to 6144 rows,
    // geometric mean by columns of all outputs, up to 512, 1024, 2048, 4096, more: rank 20-32 1.44, 1.23, 1.17, 1.05, 0.90; 36-48 1.18, 1.10, 0.99, 0.90, 0.71; 52-64 1.22, 1.09, 0.93, 0.74,
    // 0.60; 68-128 1.06, 0.87, 0.77, 0.65, 0.50; next to no shrink to repeat: rank 44, 256 -> 1032, 2748 rows 11.4 / 9.2.  Activations that no cache holds any more (above 64 MB) come better in the expand's
    // order: rank 32, 4096 -> 4096, 4000 / 4600 / 5750 rows, four sets of buffers in turn 32.9 / 38.1, 35.0 / 42.8, 38.9 / 46.7.
    if (a.T > SMALL_T) return a.rank <= 32 ? width > (a.T > 3840 ? 2048 : 4096) : a.rank <= 64 ? width > 1024 && a.d_in * width > 640000 : width > 512;
    const int64_t tiles = likely_tiles(a, S), panels = tiles * width;
    // (tiles enough to fill the chip hide the single launch's shrinks: 900 decode rows of 200 / 500 adapters, one / two, 4096 -> 512, rank 68 29.0 / 33.7, 49.7 / 59.4, rank 128 43.5 / 49.4, 102 / 108, 4096 ->
    // 4096, rank 68 53.6 / 67.0, 115 / 149, 96 72 / 86, 149 / 170, 128 107 / 111, 203 / 208; 150 of 200, rank 96, 8192 -> 2144 55 / 50; 512 of 64, 4096 -> 512 22.5 / 19.2; in place, rank 96, 2880, 426 of 200 42.9 / 54.6)
    if (a.rank > 64 && singles && tiles > 160) return false;
    // (in place, decode rows of many adapters: rank 48, d = 3184, 209 of 376 20.8 / 23.6, 2688, 535 of 197 (184 tiles) 22.3 / 31.4, 4096, 730 of 54 (72 tiles) 25.5 / 22.9)
    if (direft && a.rank > 32 && a.rank <= 48 && a.d_in <= 4096 && singles && tiles > 128) return false;
    // (above rank 64, one / two: d = 104, 180 rows 7.7 / 14.5, 128, 109 8.1 / 9.3, 256, 68 7.9 / 9.9, 384, 362 9.3 / 10.5)
    if (direft) return a.rank > 64 ? a.d_in >= 512 : (a.rank > 48 ? a.d_in >= 1024 : a.rank > 32 ? a.d_in >= 2048 : a.d_in >= 8192 && tiles <= 48);
    if (a.rank > 112) return a.d_in > 640 || panels >= 24000;    // 512 -> 1056, 29 decode rows 8.5 / 9.7, 512 -> 608, 242 prompt rows 8.7 / 9.6; 512 -> 8192, 3 rows 10.1 / 9.4
    if (a.rank > 64) return a.d_in >= 4096 || (!singles && panels >= 100000);
    // (decode rows: rank 56, 8192 -> 320 + 8192 + 1024, 725 of 32 adapters 35.9 / 46.1, 1416 -> 1952, 234 of 200 20.3 / 28.7; over all, one and two alike)
    // (tiles x columns from 80 000 to 120 000: d_in 1024 0.95-1.27, 2048 0.84-1.15, 4096 0.75-0.96 of one launch's time; up to 160 000 0.57-1.04, 0.60-1.01, 0.59-0.92)
    if (a.rank > 48) return !singles && panels >= (a.d_in > 2048 ? 80000 : 120000);
    // (hardly a shrink to repeat: 512 -> 4096, 840 prompt rows 11.3 / 12.7, 296 -> 3640, 620 7.9 / 10.4, but 304 -> 14336, 730 18.2 / 14.5)
    return a.rank > 32 && !singles && panels >= 150000 && (a.d_in > 512 || width > 8192);
}

// Out of place its form for tiles of up to four rows is in the kernel where most of the tiles are gathered rows: a second copy of the code costs the others 0.3 to 0.6 us (rank
// 32, 512 -> 2072, 880 prompt rows 6.1 / 5.5).
inline bool small_few(const ApplyArgs &a, int64_t S) { return 2 * likely_gathered(a, S) > likely_tiles(a, S); }

// What a workgroup of the small-batch kernel is (out of place): the units of 128 columns it expands, and whether it has
// the compute unit to itself (deep).
//
// As many shares as make at most about one workgroup per compute unit: the repeated shrink costs nothing while compute units are idle, and a
// share's factors come lane by lane through the texture path, which is what a wide share waits for from rank 17 on.  Down to
// 8 units at rank 4-16 (4 of a narrow output), 2 at rank 17-32, 1 above.  Measured (us, 8 units a share / the rule's): rank 64, 376 -> 1024, 2 rows 11.3 / 6.2;
// 1024 -> 1024, 377 decode rows of 2 adapters 12.8 / 7.7; rank 96, 1024 -> 1024, 67 rows 15.8 / 9.5; rank 32, 1024 -> 1504, 10 rows
// 6.5 / 5.2; rank 16, 512 -> 1024, 200 rows 4.8 / 4.3.  More workgroups than that wait for one another: rank 96, 512 -> 1024, 45
// tiles, 4 / 8 shares 10.3 / 17.2; rank 5, 4096 -> 11168 + 512, 18 tiles, 9 / 12 shares 10.6 / 14.5; 4096 -> 2 x 14336, one tile, 28 / 56
// shares 7.6 / 12.4.
// Where even that is too many (rank 4-16): two on a compute unit, of 128 registers each, hide each other's trips, which also
// suits batches where every tile has an adapter of its own (4096 -> 4096, 512 decode rows of 64 adapters: 8 units, shallow 11.8, 16
// units, deep 17.5; 1000 rows of 5 adapters 13.7 and 11.6; 4096 -> 2 x 14336: up to 640 shallow workgroups 33.6 / 36.5, up to 300
// 36.0 / 29.5).  From rank 17 on the LDS does not hold two on a compute unit: deep, and above rank 32 with 4 wavefronts where many
// adapters meet more than a workgroup per compute unit (rank 64, 4096 -> 4096, 512 decode rows: 8 wavefronts 30.9, 4 wavefronts 23.6; 1000
// rows of 5 adapters 29.0 / 30.8).
struct SmallShape { int units; bool deep; int waves; };

inline SmallShape small_shape(const ApplyArgs &a, int64_t S, int n_slices, const Knobs &k)
{
    int most = 0, d[3] = {a.d_out, n_slices > 1 ? a.more[0].d_out : 0, n_slices > 2 ? a.more[1].d_out : 0};
    for (int i = 0; i < n_slices; ++i) { d[i] = (d[i] + 127) / 128; if (d[i] > most) most = d[i]; }
    if (k.colsplit) return {(most + k.colsplit - 1) / k.colsplit, true, SMALL_WAVES};
    const int64_t tiles = likely_tiles(a, S) + 1;
    auto workgroups = [&](int units) {
        int64_t shares = 0;
        for (int i = 0; i < n_slices; ++i) shares += (d[i] + units - 1) / units;
        return tiles * shares;
    };
    // mostly short segments, and enough adapters for most tiles to have one of their own
    const bool many_adapters = a.T < 16 * S && 32 * (S < a.N ? S : (int64_t)a.N) > a.T;
    const int waves = a.rank > 32 && many_adapters && workgroups(SMALL_WAVES) > DEEP_WGS ? 4 : SMALL_WAVES;
    const int least = a.rank > 32 ? 1 : a.rank > 16 ? 2 : most <= 2 * SMALL_WAVES ? 4 : SMALL_WAVES;
    const int widest = (many_adapters && a.rank <= 16 ? 1 : 4) * SMALL_WAVES;
    // a tile's workgroups share one XCD: 32 compute units for the tiles that meet there
    const int64_t tiles_of_xcd = tiles <= 9 ? 1 : (tiles + 10) / 8, most_shares = DEEP_WGS / tiles < 32 / tiles_of_xcd ? DEEP_WGS / tiles : 32 / tiles_of_xcd;
    int64_t shares = (most + least - 1) / least;
    if (shares > most_shares) shares = most_shares;
    for (; shares > 0 && waves == SMALL_WAVES; --shares) {
        int units = (int)((most + shares - 1) / shares);
        if (units > SMALL_WAVES) units = units > 2 * SMALL_WAVES ? 4 * SMALL_WAVES : 2 * SMALL_WAVES;   // whole rounds of the wavefronts
        if (units > widest) break;
        if (workgroups(units) <= most_shares * tiles) return {units, true, waves};
    }
    if (a.rank > 16) {
        for (int units = SMALL_WAVES; units <= 16 * SMALL_WAVES; units *= 2)
            if (workgroups(units) <= 288) return {units, true, waves};
        return {16 * SMALL_WAVES, true, waves};
    }
    for (int units = SMALL_WAVES; units <= 8 * SMALL_WAVES; units *= 2)
        if (workgroups(units) <= (many_adapters ? 300 : 640)) return {units, false, SMALL_WAVES};
    return {8 * SMALL_WAVES, false, SMALL_WAVES};
}

// Whether an in-place call of rank 17-31, no multiple of 4, takes 32-row tiles of the column-split kernel instead of 64-row tiles of the
// row-split one, as the multiples of 4 always do: twice as many tiles, and their second read of h follows the first sooner.  But large batches
// of narrow rows find that read in the caches either way; prompts of a few dozen rows fill 32-row tiles no better and read an adapter's factors for
// twice as many of them; and ranks 21 and 31 have the texture path busy with their unaligned factors as soon as the tiles fill the chip twice (each rank
// was measured: 17-30 differ by a few percent, those two by 20 more).  Row-split / column-split, us: 1500 rows, d = 1024 / 4096 / 8192, rank 18 18.1 /
// 9.7, 62 / 26, 116 / 45, rank 31 18.3 / 11.2, 64 / 32, 121 / 56; 29 000 rows, 8192, rank 18 267 / 250, 23 276 / 265, 29 263 / 265; 12 000 rows of prompts of
// 40, d = 4096, rank 18 109 / 98, 23 110 / 111, 31 115 / 139, d = 1024, 19 32 / 35, 31 33 / 41; 52 000 rows of prompts of 35, d = 8192, rank 17 787 / 1016, 18 792 / 904,
// 29 818 / 1066; 39 000 of prompts of 130, 485 / 391, 491 / 364, 502 / 416; 35 000 rows, d = 512, rank 31 25 / 30, 2048 89 / 86.
// Rank 31 (21 the same to 3 %), prompts of 600 rows, d = 1024 / 4096 / 14336: 6000 rows 20.9 / 13.0, 68 / 36, 225 / 115; 13 200 rows 24.3 / 20.7, 73 / 66, 299 / 264;
// 16 800 rows 29.0 / 31.6, 94 / 101, 379 / 409; 21 000 rows, 4096 / 8192 104 / 116, 230 / 236; 30 000 rows 181 / 150, 354 / 325, 160 000 rows 576 / 623, 1352 / 1279.
// Prompts of 40 rows, d = 1024 / 4096 / 14336: 5000 rows 22.5 / 18.3, 69 / 58, 225 / 195; 8000 rows 26.2 / 29.6, 87 / 87, 295 / 297, and 8000 of prompts of 190 beside 156
// decode rows 23.0 / 19.4, 69 / 59, 252 / 227, which the host cannot tell apart; 10 500 rows of prompts of 40, 27 / 33, 90 / 113, 310 / 393; of 65, 45 000 rows, 4096 263 / 330.
// A layer takes the kernel of its one-layer call, whatever that costs where layers add up to another number of tiles (rank 31, d = 4096, 4 x 3600 rows 91 / 67, 2 x 12 000
// 110 / 126, 4 x 4000 of prompts of 40 120 / 147).
inline bool odd_streams_in_place(const ApplyArgs &a, int64_t S)
{
    if (!column_split_fits(a)) return false;
    if (a.rank == 21 || a.rank == 31) {
        if (a.T <= 14336) return a.T <= 8192 || a.T >= 48 * S;
        if (a.T < 28672 || a.T < 128 * S) return false;
    }
    if (a.T < 64 * S && (a.T > 16384 || (a.T > 8192 && a.d_in < 2048))) return false;
    return a.T <= 16384 || a.d_in >= 8192 || (a.d_in >= 4096 && a.T <= 49152);
}

// Ranks above 16 that are no multiple of 4: whether the column-split kernel takes the whole call, chunks and gathered tiles.
inline bool odd_streams(const ApplyArgs &a, int64_t S, bool direft, const Knobs &k)
{
    return !wide_widths_ok(a, 1) || k.variant == 3 || (direft && a.rank <= 32 && k.variant == 0 && odd_streams_in_place(a, S));
}

// The expand launch of a call whose z is in the workspace: up to rank 32 a workgroup per 32 rows x 512 columns, above per 64 rows and panel.
constexpr int EXPAND_MB = 2;

inline int64_t expand_panels(const ApplyArgs &a, int n_slices, int64_t cols)
{
    int64_t panels = (a.d_out + cols - 1) / cols;
    for (int i = 1; i < n_slices; ++i) panels += (a.more[i - 1].d_out + cols - 1) / cols;
    return panels;
}

// Above rank 32: units of 128 columns in a panel of panel_expand_kernel, which every output holds a whole number of (the widths are
// multiples of 128 there).  Rank 65-128: one unit of factors is 35 KB of LDS.
inline int panel_units(const ApplyArgs &a, int n_slices)
{
    bool two = a.rank <= 64 && (a.d_out % 256) == 0;
    for (int i = 1; i < n_slices; ++i) two = two && (a.more[i - 1].d_out % 256) == 0;
    return two ? 2 : 1;
}

// the kernel numbers its tiles in 32 bits
inline bool expand_ids_fit(const ApplyArgs &a, int64_t S, int n_slices)
{
    const int64_t tiles = a.rank > 32 ? tile_grid(a, S, 16 * PANEL_RW) * expand_panels(a, n_slices, 128 * panel_units(a, n_slices))
                                      : tile_grid(a, S, 16 * EXPAND_MB) * expand_panels(a, n_slices, EXPAND_WAVES * 128);
    return tiles < ((int64_t)1 << 31);
}

}  // namespace preft
