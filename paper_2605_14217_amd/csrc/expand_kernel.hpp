// The expand sweep of LoRA as a launch of its own (bf16, z from the workspace):  y += s B z  (Eq. 2).
//
// A ZOUT launch of mfma_tile_kernel or mfma_wide_kernel has left z in the workspace in the form the MFMAs
// below take it (scaled, split into bf16 head and remainder): 1 KB per 16-row block, output and rank block of
// 16 (z_piece); lane l of a wavefront holds the 16-byte piece l (ranks 4 (l / 16) .. + 3 of row l % 16).
//
// Bound: HBM (y once in, once out).  What decides how much of it a kernel gets is the order in which the chip
// walks the rows.  Measured with kernels that only move the bytes (read and write y, 89 600 rows of 28 672 bf16):
// workgroups that loop over tiles or columns sustain 4.5-5.3 TB/s whatever they prefetch; the same tiles as
// one workgroup each, ids in memory order, 6.0-6.6 (16 or 32 rows x 1 KB; a flat elementwise pass 5.95): the
// hardware hands out workgroups in order, so the bytes in flight stay one narrow window of y.  Hence a
// workgroup takes one tile of 16 MB rows x 512 columns and ends, tiles of a row block side by side, and every
// request of the tile is issued before anything is computed.  A wavefront takes 128 columns and needs no barrier.
//
// z is the first operand of the MFMAs and the factors are the second: lane (n, g) of MFMA k then ends up with column 8 n + k of the rows
// 4 g .. 4 g + 3, the eight MFMAs of a 128-column unit with the 8 consecutive columns of those rows -- what the lane loads of y
// in 256-byte row pieces.  So y passes through registers only.  (Factors first, as in the kernels with both sweeps, leaves a lane
// the columns of one row, 64 bytes beside its neighbour's, and y goes through LDS on its way in and out: 2/3 of the LDS traffic,
// and its buffers.)  The factors are contiguous in the [d_out, r] layout: fetched in whole lines, turned through LDS.  (Fetched in
// MFMA order every lane is an access of its own in the texture path: at rank 64, 89 740 rows of 2 x 28 672, 5290 us instead of 4270.)
// Two row blocks per wavefront halve the factor traffic; four leave too few wavefronts in flight.
// gate+up of the 8B layer, rank 16, 36 864 rows (4.2 GB of y), whole call: one launch 931 us, y turned through LDS 801, now 783 = 5.8 TB/s.
// Above rank 32: panel_expand_kernel below.
#pragma once
#include "common.hpp"
#include "mfma_kernel.hpp"

namespace preft {

constexpr int EXPAND_WAVES = 4;                               // 128-column units (one per wavefront) of a workgroup

// Factors in LDS, 128 columns at a time.  MFMA k takes the columns 8 n + k, n = 0 .. 15 (a lane then ends up with the 8 consecutive
// columns that it loaded, see below), so those lie side by side: column c in group c % 8, at place c / 8 of it.  A column takes
// 16 bytes modulo 32: then the 16 columns of an 8-byte operand read, and the four pieces in each, meet no bank twice (measured, one read
// of a wavefront: 16, 48, 80, 144 bytes 1.87, as linear addresses; 24, 40, 72, 136 2.96; 128 8.99).  A group is 8 bytes longer, which spreads
// the writes.  Ranks that are not multiples of 4 lie as in memory (a lane then shifts its
// four factors into place and may look one word past them).
__host__ __device__ constexpr int factor_column_bytes(int r) { return ((2 * r + 15) & ~31) + 16; }
template <int NB>
struct FactorLds {
    static constexpr int GROUP = 16 * factor_column_bytes(16 * NB) + 8, BYTES = 8 * GROUP + 16;
    int r4, column;                                           // quarters of 4 factors, and bytes, of a column
    float inv;
    __device__ __forceinline__ explicit FactorLds(int r) : r4(r >> 2), column(factor_column_bytes(r)), inv(4.0f / (float)r) {}
    // where quarter i of a contiguous [128][r] block goes.  (i + 0.5) / r4 is below 128 and at least 0.5 / 32 away from a
    // whole number (rank 128; 0.5 / 16 up to rank 64): the rounding of the product, below 1e-4, never reaches one.
    __device__ __forceinline__ int quarter(int i) const
    {
        const int c = (int)(((float)i + 0.5f) * inv);
        return (c & 7) * GROUP + (c >> 3) * column + (i - c * r4) * 8;
    }
    // what lane (n16, g) brings to MFMA k of rank block b: the factors 16 b + 4 g .. + 3 of column 8 n16 + k (of ranks that do not
    // exist others, or zeros: their z is zero)
    template <bool ODD>
    __device__ __forceinline__ u32x2_t operand(const char *fac, int k, int b, int n16, int g, int r) const
    {
        const int rank0 = 16 * b + 4 * g, n = r - rank0;      // n: how many of the lane's four ranks exist
        if constexpr (ODD) {
            const uint32_t m01 = n >= 2 ? 0xffffffffu : n == 1 ? 0xffffu : 0u, m23 = n >= 4 ? 0xffffffffu : n == 3 ? 0xffffu : 0u;
            const int at = (8 * n16 + k) * r + (n > 0 ? rank0 : 0);
            const uint32_t *w3 = reinterpret_cast<const uint32_t *>(fac) + (at >> 1);
            const uint32_t sh = (at & 1) * 16, d0 = w3[0], d1 = w3[1], d2 = w3[2];
            return u32x2_t{__builtin_amdgcn_alignbit(d1, d0, sh) & m01, __builtin_amdgcn_alignbit(d2, d1, sh) & m23};
        } else {
            return *reinterpret_cast<const u32x2_t *>(fac + k * GROUP + n16 * column + (n > 0 ? rank0 : 0) * 2);
        }
    }
};

// The tiles of an expand launch: column panels (those of the first output, then those of the others) of row blocks, ids in
// memory order.
struct ExpandTiles {
    int pan0, pan1, panels, chunk_tiles;
    uint32_t n_ids, per_xcd;
};

template <int R, int COLS = EXPAND_WAVES * 128>
__device__ __forceinline__ ExpandTiles expand_tiles(const ApplyArgs &p, int n_slices)
{
    ExpandTiles t;
    auto panels_of = [](int d) { return (d + COLS - 1) / COLS; };
    t.pan0 = panels_of(p.d_out);
    t.pan1 = n_slices > 1 ? panels_of(p.more[0].d_out) : 0;
    t.panels = t.pan0 + t.pan1 + (n_slices > 2 ? panels_of(p.more[1].d_out) : 0);
    const PREFT_CONST int32_t *header = as_const(p.header);
    t.chunk_tiles = header[HDR_CHUNKS] * (CHUNK_ROWS / R);
    t.n_ids = (uint32_t)(t.chunk_tiles + (p.chunks_only ? 0 : header[HDR_GTILES])) * (uint32_t)t.panels;     // below 2^31 (host-checked)
    t.per_xcd = (t.n_ids + 7) >> 3;
    return t;
}

// One of them: `n_rows` rows, from row0 of the chunk or gathered tile `entry`; its first block of z; output, and panel of it.
struct ExpandTile {
    int4 entry;
    int row0, n_rows, sl, panel, d_out;
    int64_t block0, ldy_b;
    bool gathered;
    void *y;
    const void *const *Bt_pool;
};

template <int R>
__device__ __forceinline__ bool expand_tile(const ApplyArgs &p, const ExpandTiles &ts, uint32_t slot, ExpandTile &t)
{
    constexpr int TPC = CHUNK_ROWS / R, MB = R / 16;
    const uint32_t id = p.xcd_runs ? (slot & 7) * ts.per_xcd + (slot >> 3) : slot;
    if (id >= ts.n_ids) return false;
    const int tile_id = (int)(id / (uint32_t)ts.panels);
    t.panel = (int)id - tile_id * ts.panels;
    t.gathered = tile_id >= ts.chunk_tiles;
    t.row0 = t.gathered ? 0 : tile_id % TPC * R;              // within the chunk
    t.entry = __builtin_bit_cast(int4, *reinterpret_cast<const PREFT_CONST i32x4_t *>(
        t.gathered ? as_const(p.gtiles) + (tile_id - ts.chunk_tiles) : as_const(p.chunks) + tile_id / TPC));
    t.n_rows = min(R, t.entry.z - t.row0);
    t.block0 = t.gathered ? (int64_t)ts.chunk_tiles * MB + (tile_id - ts.chunk_tiles) : (int64_t)tile_id * MB;
    if (t.n_rows <= 0 || t.block0 >= p.z_blocks) return false;    // (tables whose segments overlap can list more tiles than z has room for)
    t.sl = 0;
    t.y = p.y;
    t.ldy_b = p.ldy * 2;
    t.d_out = p.d_out;
    t.Bt_pool = p.Bt_pool;
    if (t.panel >= ts.pan0) {
        t.sl = t.panel >= ts.pan0 + ts.pan1 ? 2 : 1;
        t.panel -= t.sl == 2 ? ts.pan0 + ts.pan1 : ts.pan0;
        t.y = p.more[t.sl - 1].y; t.ldy_b = p.more[t.sl - 1].ldy * 2; t.d_out = p.more[t.sl - 1].d_out; t.Bt_pool = p.more[t.sl - 1].Bt_pool;
    }
    return true;
}

// Of an output whose rows do not start on 128-byte lines, the lines at the ends of a row's 256-byte pieces are asked for by two wavefronts or panels: with
// the non-temporal hint they are fetched twice.  So y comes without it there, with it elsewhere (YHINT: no such output; only such; some: a test per tile,
// fenced in, or the compiler makes one of the two loads, without the hint).  Hint / none, whole calls, us: rank 16, 4096 -> 9640, 1400 rows 25.1 / 21.1, 5000 62 /
// 47, 45 000 457 / 403; rank 8, 1024 -> 5336, 2400 rows 20.6 / 17.4; rank 7, 1000 -> 2 x 2728, 2150 rows 24.9 / 22.1; on lines, 4096 -> 4096, 37 000
// rows 152 / 170.  Some: 1024 -> 8192 + 616 (off) + 14336, 5000 rows, hint / none / by output 94 / 104 / 86, 43 000 rows 756 / 808 / 733.
__host__ __device__ __forceinline__ bool shares_lines(const void *y, int64_t ldy_b) { return ((reinterpret_cast<uintptr_t>(y) | (uintptr_t)ldy_b) & 127) != 0; }
enum class YHint { All, None, ByOutput };

template <int NB, int MB, bool ODD, YHint YHINT>
__global__ __launch_bounds__(EXPAND_WAVES * 64, 4) void mfma_expand_kernel(ApplyArgs p, int n_slices)
{
    constexpr int R = 16 * MB;
    static_assert(CHUNK_ROWS % R == 0 && NB <= 2, "tile height must divide the chunk height; rank blocks as in z_rank_blocks");
    __shared__ __attribute__((aligned(16))) char fac[EXPAND_WAVES][FactorLds<NB>::BYTES];

    if (!schedule_matches(p)) return;
    const int wave = threadIdx.x >> 6;
    const int r = p.rank;
    char *fw = fac[wave];

    const ExpandTiles tiles = expand_tiles<R>(p, n_slices);
    for (uint32_t slot = blockIdx.x; slot < tiles.per_xcd * 8; slot += gridDim.x) {
        ExpandTile t;
        if (!expand_tile<R>(p, tiles, slot, t)) continue;
        int lane = threadIdx.x & 63;
        asm volatile("" : "+v"(lane));                        // recomputed for every tile: what hangs on the lane would fill the registers
        const int n16 = lane & 15, g = lane >> 4;             // columns 8 n16 .. + 7 of the unit, rows 4 g .. + 3 of a block
        const FactorLds<NB> fl(r);
        const int4 entry = t.entry;
        const int row0 = t.row0, n_rows = t.n_rows, sl = t.sl, d_out = t.d_out;
        const bool gathered = t.gathered;
        const int64_t ldy_b = t.ldy_b, block0 = t.block0;
        const void *const *Bt_pool = t.Bt_pool;
        const int c0 = (t.panel * EXPAND_WAVES + __builtin_amdgcn_readfirstlane(wave)) * 128;   // this wavefront's first column
        if (c0 >= d_out) continue;

        // Every request of the tile at once, none of them conditional on the lane: row slots past the tile alias
        // its last row, columns past the width the last ones, factor pieces past the width its last
        // piece.  Only the stores are masked.
        const bool col_ok = c0 + n16 * 8 < d_out;             // d_out % 8 == 0: a lane's 8 columns exist or not
        const int rows_left = col_ok ? n_rows - 4 * g : 0;    // the rows mb * 16 + v below that are the lane's to store
        gptr_t yp[MB][4];
        {
            int32_t row[MB][4];
#pragma unroll
            for (int mb = 0; mb < MB; ++mb)
#pragma unroll
                for (int v = 0; v < 4; ++v) row[mb][v] = entry.y + row0 + min(mb * 16 + 4 * g + v, n_rows - 1);
            if (gathered) {
#pragma unroll
                for (int mb = 0; mb < MB; ++mb)
#pragma unroll
                    for (int v = 0; v < 4; ++v) row[mb][v] = p.shorts[row[mb][v]].y;
            }
            gptr_t yc = as_global(t.y) + (int64_t)c0 * 2;       // uniform
            const int y_col = (col_ok ? n16 * 8 : d_out - 8 - c0) * 2;
#pragma unroll
            for (int mb = 0; mb < MB; ++mb)
#pragma unroll
                for (int v = 0; v < 4; ++v) yp[mb][v] = yc + (row[mb][v] * ldy_b + y_col);
        }
        // factors of the unit's 128 columns: 16 r contiguous 16-byte pieces, of which this lane takes lane + 64 j
        // (lanes past them the last one)
        gcptr_t Wp = as_global(as_const(Bt_pool)[entry.x]) + (int64_t)c0 * r * 2;
        const int w_last = last_factor_piece(d_out - c0, 128, r);            // last piece that exists, from column c0 on
        u32x4_t W[4 * NB];
#pragma unroll
        for (int j = 0; j < 4 * NB; ++j) W[j] = ld16(Wp + (uint32_t)(min(min(lane + 64 * j, 16 * r - 1), w_last) * 16));
        bf16x8_t zop[MB][NB];
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) {
            const int m = mb * 16 < n_rows ? mb : 0;          // row blocks past the tile: any z will do
            gcptr_t zb = as_global(p.zws) + (z_piece(block0 + m, n_slices, sl, NB, 0) + lane) * 16;
#pragma unroll
            for (int b = 0; b < NB; ++b) zop[mb][b] = as_bf16x8(ld16(zb + b * 1024));
        }
        u32x4_t Y[MB][4];
        auto load_y = [&](auto load) {
#pragma unroll
            for (int mb = 0; mb < MB; ++mb)
#pragma unroll
                for (int v = 0; v < 4; ++v) Y[mb][v] = load(yp[mb][v]);
        };
        if constexpr (YHINT == YHint::None) {
            load_y([](gptr_t a) { return ld16(a); });
        } else if (YHINT == YHint::ByOutput && shares_lines(t.y, ldy_b)) {
            asm volatile("" ::: "memory");
            load_y([](gptr_t a) { return ld16(a); });
            asm volatile("" ::: "memory");
        } else {
            load_y([](gptr_t a) { return ld16_stream(a); });
        }

#pragma unroll
        for (int j = 0; j < 4 * NB; ++j) {
            const int piece = min(lane + 64 * j, 16 * r - 1);
            if constexpr (ODD) {
                *reinterpret_cast<u32x4_t *>(fw + piece * 16) = W[j];
            } else {                                          // two 8-byte halves, neither straddles a column
                *reinterpret_cast<u32x2_t *>(fw + fl.quarter(2 * piece)) = u32x2_t{W[j][0], W[j][1]};
                *reinterpret_cast<u32x2_t *>(fw + fl.quarter(2 * piece + 1)) = u32x2_t{W[j][2], W[j][3]};
            }
        }
        // z as the first operand, the factors as the second: lane (n16, g) of MFMA k ends up with column 8 n16 + k of the rows
        // 4 g .. 4 g + 3 -- the elements it has loaded, so y needs no turn through LDS on its way in or out
#pragma unroll
        for (int k2 = 0; k2 < 4; ++k2) {
            u32x2_t w[2][NB];
#pragma unroll
            for (int e = 0; e < 2; ++e)
#pragma unroll
                for (int b = 0; b < NB; ++b) w[e][b] = fl.template operand<ODD>(fw, 2 * k2 + e, b, n16, g, r);
#pragma unroll
            for (int mb = 0; mb < MB; ++mb) {
                f32x4_t d[2];
#pragma unroll
                for (int e = 0; e < 2; ++e) {
                    d[e] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                    for (int b = 0; b < NB; ++b)
                        d[e] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(zop[mb][b], as_bf16x8(u32x4_t{w[e][b][0], w[e][b][1], w[e][b][0], w[e][b][1]}),
                                                                       d[e], 0, 0, 0);
                }
#pragma unroll
                for (int v = 0; v < 4; ++v) Y[mb][v][k2] = pack_bf16(bf16_lo(Y[mb][v][k2]) + d[0][v], bf16_hi(Y[mb][v][k2]) + d[1][v]);
            }
        }
#pragma unroll
        for (int mb = 0; mb < MB; ++mb)
#pragma unroll
            for (int v = 0; v < 4; ++v)
                if (mb * 16 + v < rows_left) st16_stream(yp[mb][v], Y[mb][v]);
    }
}

// The same in tiles of 16 RW rows x 128 PU columns whose factors the RW wavefronts share through LDS (above rank 32; widths multiples of 128 PU
// and chunks only, unless ANY).  At rank 64 the factors of a wavefront's own columns would be as many bytes as its 32 rows of y; shared by
// 64 rows they are half as many.  64 x 256 where every output is a multiple of 256 wide, else 64 x 128.
// gate+up of a 70B layer, rank 64, 89 740 rows, whole call: one launch 4845 us, two with y turned through LDS 4470, without 4165-4250, and 4060-4120
// since the shrink launch takes tiles of 128 rows (5.7 TB/s); 8192 -> 8192 946 / 855 / 842; rank 63, 8192 -> 28 672 2586 (one launch) / 2282; 8B layer,
// 37 000 rows, rank 64 gate+up 925 / 882, rank 63, 4096 -> 14336 542 (a wavefront's own factors) / 479; 4096 -> 14208 (64 x 128) 539 / 509.
// Three workgroups per compute unit, at the 4165-4250 and 842 of the figures above.  Four (128 registers) spill: gate+up 5324; kept from spilling by a
// barrier to the compiler's scheduler they have a wider window of y in flight, 4420 and 895; two 4690, 970.
// Tiles of 128 rows 4400, 890.  Tiles in memory order; dealt to the XCDs as runs 977 for 923, 65 for 67 (with y turned).
constexpr int PANEL_RW = 4;

// ANY: any widths (multiples of 8), and gathered tiles too, of which the first wavefront has the rows (calls of the small-batch kernel's order).
// Rank 65-128: 64 x 128, 35 KB of LDS (two units a workgroup: 4096 -> 4096, rank 96, 24 000 rows 144 / 150 us).
template <int NB, int RW, int PU, bool ODD, bool ANY = false, bool HINT = true>
__global__ __launch_bounds__(RW * 64, 3) void panel_expand_kernel(ApplyArgs p, int n_slices)
{
    constexpr int R = 16 * RW, NT = RW * 64;
    constexpr int W_ITERS = NB * 16 * 16 * PU / NT;           // 16 r PU pieces, r <= 16 NB
    static_assert(CHUNK_ROWS % R == 0 && PU <= 2, "tile height must divide the chunk height; two units of factors");
    __shared__ __attribute__((aligned(16))) char fac[PU][FactorLds<NB>::BYTES];

    if (!schedule_matches(p)) return;
    const int rb = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int r = p.rank;

    const ExpandTiles tiles = expand_tiles<R, PU * 128>(p, n_slices);
    for (uint32_t slot = blockIdx.x; slot < tiles.per_xcd * 8; slot += gridDim.x) {
        ExpandTile t;
        if (!expand_tile<R>(p, tiles, slot, t)) continue;     // uniform over the workgroup
        const int c0 = t.panel * PU * 128;
        int tid = threadIdx.x;
        asm volatile("" : "+v"(tid));                         // recomputed for every tile: what hangs on the lane would fill the registers
        const int lane = tid & 63, n16 = lane & 15, g = lane >> 4;           // columns 8 n16 .. + 7 of a unit, rows 4 g .. + 3 of the block
        const FactorLds<NB> fl(r);

        // every request of the tile first: its factors, this row block's z, its units of y (rows past the tile alias its last one)
        gcptr_t Wp = as_global(as_const(t.Bt_pool)[t.entry.x]) + (int64_t)c0 * r * 2;
        // the panel's last piece: lanes past it take it again
        const int w_last = ANY ? last_factor_piece(t.d_out - c0, 128 * PU, r) : 16 * r * PU - 1;
        u32x4_t W[W_ITERS];
#pragma unroll
        for (int j = 0; j < W_ITERS; ++j) W[j] = ld16(Wp + (uint32_t)(min(tid + j * NT, w_last) * 16));
        const int rank_blocks = z_rank_blocks(r);             // more than NB / 2; what is missing of NB is padding, z = 0
        const int zrb = rb * 16 < t.n_rows ? rb : 0;          // row blocks past the tile: any z will do
        gcptr_t zb = as_global(p.zws) + (z_piece(t.block0 + zrb, n_slices, t.sl, rank_blocks, 0) + lane) * 16;
        bf16x8_t zop[NB];
#pragma unroll
        for (int b = 0; b < NB; ++b) {
            u32x4_t zv = ld16(zb + (b <= NB / 2 ? b : min(b, rank_blocks - 1)) * 1024);
            if (b > NB / 2) {
#pragma unroll
                for (int k = 0; k < 4; ++k) zv[k] = b < rank_blocks ? zv[k] : 0u;
            }
            zop[b] = as_bf16x8(zv);
        }
        gptr_t yu[4];
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            int64_t row = (int64_t)t.entry.y + t.row0 + min(rb * 16 + 4 * g + v, t.n_rows - 1);
            if constexpr (ANY) { if (t.gathered) row = p.shorts[row].y; }
            yu[v] = as_global(t.y) + row * t.ldy_b + (int64_t)c0 * 2 + (ANY ? 0 : n16 * 16);
        }
        // where the lane's 8 columns of unit u begin (ANY: past the width the last 8, which are not stored again)
        auto y_off = [&](int u) { return ANY ? min(u * 256 + n16 * 16, (t.d_out - c0) * 2 - 16) : u * 256; };
        const bool mine = rb * 16 < t.n_rows;                 // a short prompt's tile: its other wavefronts only bring factors
        const int rows_left = t.n_rows - rb * 16 - 4 * g;
        u32x4_t Y[PU][4];
        if (mine) {
#pragma unroll
            for (int u = 0; u < PU; ++u)
#pragma unroll
                for (int v = 0; v < 4; ++v) Y[u][v] = ld16_hint<HINT>(yu[v] + y_off(u));
        }

        // factors to LDS: as they lie in memory, or in two 8-byte halves per piece, neither of which straddles a column
#pragma unroll
        for (int j = 0; j < W_ITERS; ++j) {
            const int piece = min(tid + j * NT, w_last), u = piece >= 16 * r ? 1 : 0, in_unit = piece - u * 16 * r;
            if constexpr (ODD) {
                *reinterpret_cast<u32x4_t *>(fac[u] + in_unit * 16) = W[j];
            } else {
                *reinterpret_cast<u32x2_t *>(fac[u] + fl.quarter(2 * in_unit)) = u32x2_t{W[j][0], W[j][1]};
                *reinterpret_cast<u32x2_t *>(fac[u] + fl.quarter(2 * in_unit + 1)) = u32x2_t{W[j][2], W[j][3]};
            }
        }
        __syncthreads();

        if (mine) {
#pragma unroll
            for (int u = 0; u < PU; ++u) {
#pragma unroll
                for (int k2 = 0; k2 < 4; ++k2) {              // columns 8 n16 + 2 k2 and + 1, as in mfma_expand_kernel
                    f32x4_t d[2];
#pragma unroll
                    for (int e = 0; e < 2; ++e) {
                        d[e] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                        for (int b = 0; b < NB; ++b) {
                            const u32x2_t w = fl.template operand<ODD>(fac[u], 2 * k2 + e, b, n16, g, r);
                            d[e] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(zop[b], as_bf16x8(u32x4_t{w[0], w[1], w[0], w[1]}), d[e], 0, 0, 0);
                        }
                    }
#pragma unroll
                    for (int v = 0; v < 4; ++v) Y[u][v][k2] = pack_bf16(bf16_lo(Y[u][v][k2]) + d[0][v], bf16_hi(Y[u][v][k2]) + d[1][v]);
                        }
#pragma unroll
                for (int v = 0; v < 4; ++v)
                    if (v < rows_left && (!ANY || c0 + u * 128 + n16 * 8 < t.d_out)) st16_stream(yu[v] + y_off(u), Y[u][v]);
            }
        }
        __syncthreads();                                      // the next tile's factors overwrite this one's
    }
}

// The same for rank 1-3, after a ZOUT launch of valu_tile_kernel: too thin for the matrix cores, and z stays in fp32.  A lane
// keeps the order its loads come in -- 8 columns of the rows 4 i + q -- so that y needs no turn through LDS; its factors are the
// RANK 16-byte pieces of those 8 columns, the sums those of valu_tile_kernel: the bits of the single launch.
template <int RANK, int MB>
__global__ __launch_bounds__(EXPAND_WAVES * 64) void thin_expand_kernel(ApplyArgs p, int n_slices)
{
    constexpr int R = 16 * MB;
    if (!schedule_matches(p)) return;
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int q = lane >> 4, c16 = lane & 15;                 // unit load order
    const ExpandTiles tiles = expand_tiles<R>(p, n_slices);
    for (uint32_t slot = blockIdx.x; slot < tiles.per_xcd * 8; slot += gridDim.x) {
        ExpandTile t;
        if (!expand_tile<R>(p, tiles, slot, t)) continue;
        const int c0 = (t.panel * EXPAND_WAVES + __builtin_amdgcn_readfirstlane(wave)) * 128;   // this wavefront's first column
        if (c0 >= t.d_out) continue;
        // row slots past the tile alias its last row, columns past the width the last ones; only the stores are masked
        int32_t row[MB][4];
        const bool col_ok = c0 + c16 * 8 < t.d_out;
        const int col = col_ok ? c16 * 8 : t.d_out - 8 - c0;
#pragma unroll
        for (int mb = 0; mb < MB; ++mb)
#pragma unroll
            for (int i = 0; i < 4; ++i) row[mb][i] = t.entry.y + t.row0 + min(mb * 16 + 4 * i + q, t.n_rows - 1);
        if (t.gathered) {
#pragma unroll
            for (int mb = 0; mb < MB; ++mb)
#pragma unroll
                for (int i = 0; i < 4; ++i) row[mb][i] = p.shorts[row[mb][i]].y;
        }
        gptr_t yc = as_global(t.y) + ((int64_t)c0 + col) * 2;
        u32x4_t Y[MB][4], raw[RANK], zv[MB][4];
#pragma unroll
        for (int mb = 0; mb < MB; ++mb)
#pragma unroll
            for (int i = 0; i < 4; ++i) Y[mb][i] = ld16_stream(yc + row[mb][i] * t.ldy_b);
        gcptr_t wp = as_global(as_const(t.Bt_pool)[t.entry.x]) + ((int64_t)c0 + col) * RANK * 2;
#pragma unroll
        for (int j = 0; j < RANK; ++j) raw[j] = ld16(wp + j * 16);
#pragma unroll
        for (int mb = 0; mb < MB; ++mb)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int s = min(mb * 16 + 4 * i + q, t.n_rows - 1);
                zv[mb][i] = ld16(as_global(p.zws) + (z_piece(t.block0 + s / 16, n_slices, t.sl, 1, 0) + s % 16) * 16);
            }
        float w[8 * RANK];
#pragma unroll
        for (int j = 0; j < RANK; ++j)
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                w[j * 8 + 2 * k] = bf16_lo(raw[j][k]);
                w[j * 8 + 2 * k + 1] = bf16_hi(raw[j][k]);
            }
#pragma unroll
        for (int mb = 0; mb < MB; ++mb)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                float out[8];
                Elem<bf16_tag>::unpack(Y[mb][i], out);
#pragma unroll
                for (int c = 0; c < 8; ++c) {
                    float d = 0.f;
#pragma unroll
                    for (int k = 0; k < RANK; ++k) d = fmaf(w[c * RANK + k], __uint_as_float(zv[mb][i][k]), d);
                    out[c] += d;
                }
                if (col_ok && mb * 16 + 4 * i + q < t.n_rows) st16_stream(yc + row[mb][i] * t.ldy_b, Elem<bf16_tag>::pack(out));
            }
    }
}

}  // namespace preft
