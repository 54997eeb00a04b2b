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
// The factors of its columns are contiguous in the [d_out, r] layout: they are fetched in whole lines and turned
// through LDS, 32 columns at a time.  (Fetched in MFMA order, lanes of neighbouring columns, every lane is an
// access of its own in the texture path: at rank 64, 89 740 rows of 2 x 28 672, 5290 us instead of 4270.)  Two row blocks per wavefront halve the factor traffic; four
// leave too few wavefronts in flight.
// gate+up of the 8B layer, rank 16, 36 864 rows (4.2 GB of y): 718 us = 5.9 TB/s, in a call that took 931 in one launch and takes 790.
// Rank 33-64: panel_expand_kernel below, this one where its panels do not fit the widths or the rank is no multiple of 4.
#pragma once
#include "common.hpp"
#include "mfma_kernel.hpp"

namespace preft {

constexpr int EXPAND_WAVES = 4;                               // 128-column units (one per wavefront) of a workgroup

// LDS of a wavefront: one 16-row turn buffer, and the factors of 32 columns.  A column's factors are padded by
// 8 bytes so that the 16 columns of an MFMA operand read spread over all banks; ranks that are not multiples of 4
// lie as in memory (a lane then shifts its four factors into place and may look one word past them).
constexpr int expand_fac_bytes(int NB) { return 32 * (32 * NB + 8) + 16; }

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

template <int NB, int MB, bool ODD>
__global__ __launch_bounds__(EXPAND_WAVES * 64, 2) void mfma_expand_kernel(ApplyArgs p, int n_slices)
{
    constexpr int R = 16 * MB;
    static_assert(CHUNK_ROWS % R == 0, "tile height must divide the chunk height");
    __shared__ u32x4_t turn[EXPAND_WAVES][16 * MFMA_TRS];
    __shared__ __attribute__((aligned(16))) char fac[EXPAND_WAVES][expand_fac_bytes(NB)];

    if (!schedule_matches(p)) return;
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int rl = lane & 15, g = lane >> 4;                  // MFMA order
    const int q = lane >> 4, c16 = lane & 15;                 // unit load order
    const int r = p.rank;
    u32x4_t *tr = turn[wave];
    char *fw = fac[wave];

    const ExpandTiles tiles = expand_tiles<R>(p, n_slices);
    for (uint32_t slot = blockIdx.x; slot < tiles.per_xcd * 8; slot += gridDim.x) {
        ExpandTile t;
        if (!expand_tile<R>(p, tiles, slot, t)) continue;
        const int4 entry = t.entry;
        const int row0 = t.row0, n_rows = t.n_rows, sl = t.sl, d_out = t.d_out;
        const bool gathered = t.gathered;
        const int64_t ldy_b = t.ldy_b, block0 = t.block0;
        const void *const *Bt_pool = t.Bt_pool;
        const int c0 = (t.panel * EXPAND_WAVES + __builtin_amdgcn_readfirstlane(wave)) * 128;   // this wavefront's first column
        if (c0 >= d_out) continue;

        // Every request of the tile at once, none of them conditional on the lane: row slots past the tile alias
        // its last row, columns past the width the last ones, factor pieces past a column group's end its last
        // piece.  Only the stores are masked.
        int32_t row[MB][4];
        const bool col_ok = c0 + c16 * 8 < d_out;             // d_out % 8 == 0: a lane's 8 columns exist or not
#pragma unroll
        for (int mb = 0; mb < MB; ++mb)
#pragma unroll
            for (int i = 0; i < 4; ++i) row[mb][i] = entry.y + row0 + min(mb * 16 + 4 * i + q, n_rows - 1);
        if (gathered) {
#pragma unroll
            for (int mb = 0; mb < MB; ++mb)
#pragma unroll
                for (int i = 0; i < 4; ++i) row[mb][i] = p.shorts[row[mb][i]].y;
        }
        u32x4_t Y[MB][4];
        gptr_t yc = as_global(t.y) + (int64_t)c0 * 2;           // uniform
        const int y_col = (col_ok ? c16 * 8 : d_out - 8 - c0) * 2;
#pragma unroll
        for (int mb = 0; mb < MB; ++mb)
#pragma unroll
            for (int i = 0; i < 4; ++i) Y[mb][i] = ld16_stream(yc + (row[mb][i] * ldy_b + y_col));
        // factors of the 32 columns of step s: 4 r contiguous 16-byte pieces, of which this lane takes lane + 64 j
        // (lanes past them the last one)
        gcptr_t Wp = as_global(as_const(Bt_pool)[entry.x]) + (int64_t)c0 * r * 2;
        const int w_last = last_factor_piece(d_out - c0, 128, r);            // last piece that exists, from column c0 on
        constexpr int AHEAD = NB >= 4 ? 2 : 4;                // register budget
        u32x4_t W[4][NB];
        auto load_w = [&](int s) {
#pragma unroll
            for (int j = 0; j < NB; ++j) W[s][j] = ld16(Wp + (uint32_t)(min(s * 4 * r + min(lane + 64 * j, 4 * r - 1), w_last) * 16));
        };
#pragma unroll
        for (int s = 0; s < AHEAD; ++s) load_w(s);
        bf16x8_t zop[MB][NB];
        const int rank_blocks = NB < 4 ? NB : z_rank_blocks(r);              // 33..48: the fourth block is padding, z = 0
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) {
            const int m = mb * 16 < n_rows ? mb : 0;          // row blocks past the tile: any z will do
            gcptr_t zb = as_global(p.zws) + (z_piece(block0 + m, n_slices, sl, rank_blocks, 0) + lane) * 16;
#pragma unroll
            for (int b = 0; b < NB; ++b) {
                u32x4_t zv = ld16(zb + (NB < 4 || b < 3 ? b : rank_blocks - 1) * 1024);
                if (NB == 4 && b == 3) {
#pragma unroll
                    for (int k = 0; k < 4; ++k) zv[k] = rank_blocks > 3 ? zv[k] : 0u;
                }
                zop[mb][b] = as_bf16x8(zv);
            }
        }
        // where the pieces land in LDS: two 8-byte halves, neither straddles a column (multiples of 4)
        int w_dst[NB][2];
#pragma unroll
        for (int j = 0; j < NB; ++j)
#pragma unroll
            for (int hh = 0; hh < 2; ++hh) {
                const int byte = min(lane + 64 * j, 4 * r - 1) * 16 + hh * 8;
                w_dst[j][hh] = ODD ? byte : byte + byte / (2 * r) * 8;
            }

        // to MFMA order: lane (row rl, g) holds columns 8g .. 8g+7 of step s
        u32x4_t yop[MB][4];
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) {
#pragma unroll
            for (int i = 0; i < 4; ++i) tr[(4 * i + q) * MFMA_TRS + c16] = Y[mb][i];
#pragma unroll
            for (int s = 0; s < 4; ++s) yop[mb][s] = tr[rl * MFMA_TRS + 4 * s + g];
        }
#pragma unroll
        for (int s = 0; s < 4; ++s) {
#pragma unroll
            for (int j = 0; j < NB; ++j) {
                if constexpr (ODD) {
                    *reinterpret_cast<u32x4_t *>(fw + w_dst[j][0]) = W[s][j];
                } else {
                    *reinterpret_cast<u32x2_t *>(fw + w_dst[j][0]) = u32x2_t{W[s][j][0], W[s][j][1]};
                    *reinterpret_cast<u32x2_t *>(fw + w_dst[j][1]) = u32x2_t{W[s][j][2], W[s][j][3]};
                }
            }
            if (s + AHEAD < 4) load_w(s + AHEAD);
            // MFMA e takes columns 2m + e of the step: lane (row, g) owns outputs 8g + 2v + e
            u32x2_t w[2][NB];
#pragma unroll
            for (int e = 0; e < 2; ++e)
#pragma unroll
                for (int b = 0; b < NB; ++b) {
                    const int rank0 = 16 * b + 4 * g, n = r - rank0;      // n: how many of the lane's four ranks exist
                    if constexpr (ODD) {
                        const uint32_t m01 = n >= 2 ? 0xffffffffu : n == 1 ? 0xffffu : 0u;
                        const uint32_t m23 = n >= 4 ? 0xffffffffu : n == 3 ? 0xffffu : 0u;
                        const int at = (2 * rl + e) * r + (n > 0 ? rank0 : 0);
                        const uint32_t *w3 = reinterpret_cast<const uint32_t *>(fw) + (at >> 1);
                        const uint32_t sh = (at & 1) * 16, d0 = w3[0], d1 = w3[1], d2 = w3[2];
                        w[e][b] = u32x2_t{__builtin_amdgcn_alignbit(d1, d0, sh) & m01, __builtin_amdgcn_alignbit(d2, d1, sh) & m23};
                    } else {
                        w[e][b] = *reinterpret_cast<const u32x2_t *>(fw + (2 * rl + e) * (2 * r + 8) + (n > 0 ? rank0 : 0) * 2);
                    }
                }
#pragma unroll
            for (int mb = 0; mb < MB; ++mb) {
                f32x4_t d[2];
#pragma unroll
                for (int e = 0; e < 2; ++e) {
                    d[e] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                    for (int b = 0; b < NB; ++b)
                        d[e] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(u32x4_t{w[e][b][0], w[e][b][1], w[e][b][0], w[e][b][1]}),
                                                                       zop[mb][b], d[e], 0, 0, 0);
                }
                const u32x4_t yv = yop[mb][s];
                float out[8];
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    out[2 * v]     = bf16_lo(yv[v]) + d[0][v];
                    out[2 * v + 1] = bf16_hi(yv[v]) + d[1][v];
                }
                yop[mb][s] = Elem<bf16_tag>::pack(out);
            }
        }
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) {
#pragma unroll
            for (int s = 0; s < 4; ++s) tr[rl * MFMA_TRS + 4 * s + g] = yop[mb][s];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const u32x4_t o = tr[(4 * i + q) * MFMA_TRS + c16];
                if (col_ok && mb * 16 + 4 * i + q < n_rows) st16_stream(yc + (row[mb][i] * ldy_b + c16 * 16), o);
            }
        }
    }
}

// The same in tiles of 16 RW rows x 128 PU columns whose factors the RW wavefronts share through LDS (rank 33-64 in multiples of 4, widths
// multiples of 128 PU; chunks only).  At rank 64 a wavefront of mfma_expand_kernel holds the factors of its own columns on their way, 200 registers
// and two wavefronts per SIMD, and every 32 rows fetch the factors again: too little y in flight (8B layer's o, 38 400 rows: 147 us =
// 4.3 TB/s).  Shared by 64 rows they take half the traffic and 8 pieces a lane: 163 registers, 52 KB of LDS, three workgroups per compute
// unit, which also hide the barrier.  Whole calls, rank 64, mfma_expand_kernel / this one, us: 4096 -> 4096, 1400 rows 46 / 46, 38 000 rows 227 / 208;
// 4096 -> 2 x 14336, 1400 rows 81 / 78, 38 000 rows 1031 / 923; 8192 -> 8192, 45 000 rows 484 / 444; 1024 -> 1024 69 / 67; rank 52
// alike.  Tiles in memory order; dealt to the XCDs as runs 977 for the 923, 65 for the 67.
// Short prompts, 4096 -> 2 x 14336: 120 of 10-16 rows 161 / 153, 200 of 20-60 360 / 317, 60 of 33-34 148 / 131, 40 of 20 93 / 99.
constexpr int PANEL_RW = 4, PANEL_PU = 2;

template <int NB, int RW, int PU>
__global__ __launch_bounds__(RW * 64, 3) void panel_expand_kernel(ApplyArgs p, int n_slices)
{
    constexpr int R = 16 * RW, NT = RW * 64;
    constexpr int W_ITERS = NB * 16 * 16 * PU / NT;           // 16 r PU pieces, r <= 16 NB
    static_assert(CHUNK_ROWS % R == 0, "tile height must divide the chunk height");
    __shared__ u32x4_t turn[RW][16 * MFMA_TRS];
    __shared__ __attribute__((aligned(16))) char fac[PU * 128 * (32 * NB + 8)];      // column c at byte c (2 r + 8)

    if (!schedule_matches(p)) return;
    const int rb = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int rl = lane & 15, g = lane >> 4;                  // MFMA order
    const int q = lane >> 4, c16 = lane & 15;                 // unit load order
    const int r = p.rank, cs = 2 * r + 8;
    u32x4_t *tr = turn[rb];

    const ExpandTiles tiles = expand_tiles<R, PU * 128>(p, n_slices);
    for (uint32_t slot = blockIdx.x; slot < tiles.per_xcd * 8; slot += gridDim.x) {
        ExpandTile t;
        if (!expand_tile<R>(p, tiles, slot, t)) continue;     // uniform over the workgroup
        const int c0 = t.panel * PU * 128;

        // every request of the tile first: its factors, this row block's z, its units of y (rows past the tile alias its last one)
        gcptr_t Wp = as_global(as_const(t.Bt_pool)[t.entry.x]) + (int64_t)c0 * r * 2;
        const int w_last = 16 * r * PU - 1;                   // the panel's last piece: lanes past it take it again
        u32x4_t W[W_ITERS];
#pragma unroll
        for (int j = 0; j < W_ITERS; ++j) W[j] = ld16(Wp + (uint32_t)(min((int)threadIdx.x + j * NT, w_last) * 16));
        const int rank_blocks = z_rank_blocks(r);             // 33..48: the fourth block is padding, z = 0
        const int zrb = rb * 16 < t.n_rows ? rb : 0;          // row blocks past the tile: any z will do
        gcptr_t zb = as_global(p.zws) + (z_piece(t.block0 + zrb, n_slices, t.sl, rank_blocks, 0) + lane) * 16;
        bf16x8_t zop[NB];
#pragma unroll
        for (int b = 0; b < NB; ++b) {
            u32x4_t zv = ld16(zb + (b < NB - 1 ? b : rank_blocks - 1) * 1024);
            if (b == NB - 1) {
#pragma unroll
                for (int k = 0; k < 4; ++k) zv[k] = rank_blocks == NB ? zv[k] : 0u;
            }
            zop[b] = as_bf16x8(zv);
        }
        gptr_t yu[4];
#pragma unroll
        for (int i = 0; i < 4; ++i)
            yu[i] = as_global(t.y) + ((int64_t)t.entry.y + t.row0 + min(rb * 16 + 4 * i + q, t.n_rows - 1)) * t.ldy_b + (int64_t)c0 * 2 + c16 * 16;
        const bool mine = rb * 16 < t.n_rows;                 // a short prompt's tile: its other wavefronts only bring factors
        u32x4_t Y[PU][4];
        if (mine) {
#pragma unroll
            for (int u = 0; u < PU; ++u)
#pragma unroll
                for (int i = 0; i < 4; ++i) Y[u][i] = ld16_stream(yu[i] + u * 256);
        }

        // factors to LDS: two 8-byte halves per piece, neither straddles a column (r % 4 == 0)
#pragma unroll
        for (int j = 0; j < W_ITERS; ++j) {
            const int piece = min((int)threadIdx.x + j * NT, w_last);
#pragma unroll
            for (int hh = 0; hh < 2; ++hh) {
                const int byte = piece * 16 + hh * 8;
                *reinterpret_cast<u32x2_t *>(fac + byte + byte / (2 * r) * 8) = u32x2_t{W[j][2 * hh], W[j][2 * hh + 1]};
            }
        }
        __syncthreads();

#pragma unroll
        for (int u = 0; u < PU; ++u) {
            if (!mine) break;
            u32x4_t yop[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) tr[(4 * i + q) * MFMA_TRS + c16] = Y[u][i];
#pragma unroll
            for (int s = 0; s < 4; ++s) yop[s] = tr[rl * MFMA_TRS + 4 * s + g];
#pragma unroll
            for (int s = 0; s < 4; ++s) {
                f32x4_t d[2];
#pragma unroll
                for (int e = 0; e < 2; ++e) {                 // columns 2m + e of the step, as in mfma_expand_kernel
                    d[e] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                    for (int b = 0; b < NB; ++b) {
                        const int rank0 = 16 * b + 4 * g;
                        const u32x2_t w = *reinterpret_cast<const u32x2_t *>(fac + (u * 128 + s * 32 + 2 * rl + e) * cs + (rank0 < r ? rank0 : 0) * 2);
                        d[e] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(u32x4_t{w[0], w[1], w[0], w[1]}), zop[b], d[e], 0, 0, 0);
                    }
                }
                const u32x4_t yv = yop[s];
                float out[8];
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    out[2 * v]     = bf16_lo(yv[v]) + d[0][v];
                    out[2 * v + 1] = bf16_hi(yv[v]) + d[1][v];
                }
                tr[rl * MFMA_TRS + 4 * s + g] = Elem<bf16_tag>::pack(out);
            }
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const u32x4_t o = tr[(4 * i + q) * MFMA_TRS + c16];
                if (rb * 16 + 4 * i + q < t.n_rows) st16_stream(yu[i] + u * 256, o);
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
