// Small batches (bf16, matrix cores): a step of a few dozen to about a thousand rows has a handful of 16-row tiles, and
// what counts is the chain of dependent trips to memory from launch to last store, not bytes.
//
// A workgroup of 8 wavefronts takes one 16-row tile and, out of place, one share of the columns of one output: it
// runs the whole shrink sweep of that output (the tile's x and the factor come from L2 after the first workgroup) and
// expands its share.  Packed outputs are separate workgroups: sharing x between them would put their expand sweeps
// behind one another.  In place a tile belongs to one workgroup (another's writes must not meet its reads).
// The trips: launch arguments; schedule header; tile; adapter pointers; up to BATCH units of x and of the factor
// per wavefront, all requested at once; and, requested before the cross-wavefront sum of z, the first DEPTH units of
// y and its factors.  Operand layouts and the order of every sum as in mfma_tile_kernel.
// Against the shape before (four workgroups per tile, each shrinking every output, two units in flight, the expand
// requested after the sum; one launch per output above rank 16): q+k+v 4096 -> 4096 + 2 x 1024 as a replayed graph, rank 16: 32
// decode rows 14.5 -> 9.0 us, a 1000-row batch 27.6 -> 14.7; rank 64: 49 -> 21, 75 -> 45; 4096 -> 4096 rank 16: 8.1 -> 7.5, 15.9 -> 11.6.
#pragma once
#include "common.hpp"
#include "expand_kernel.hpp"                                 // FactorLds
#include "mfma_kernel.hpp"

namespace preft {

constexpr int SMALL_WAVES = 8;

// Whether a unit's factors of the expand go through LDS in whole lines and y does not, as in mfma_expand_kernel (DIRECT below).  Where they are few (up
// to rank 16) the address arithmetic and the trip through LDS cost a lone tile more than y's two: 32 decode rows, 4096 -> 4096, rank 16 5.8 us, 6.1 with it; rank 32, tiles of up to four
// rows, 7.4 / 7.6.  Without / with it, us: rank 32, 900 prompt rows 14.4 / 13.5, in place, 32 decode rows, d = 4096 13.4 / 11.4; rank 7 (which had its factors in LDS
// already), 600 prompt rows 8.4 / 8.0, 200 decode rows 7.6 / 7.3.  (Factors straight from memory in that column order, 16 lines an instruction: in place 7.9 / 12.2, rank 48 17.7 / 36.)
// LINES: rank 17-32 out of place, shares of 8 units and more, where every wavefront has a unit (rank 32, 4096 -> 512, 300 rows, shares of 2 units, without / with 7.9 / 8.6).
// Not at ranks 20 and 28, whose columns are an odd number of 8-byte quarters: with / without it, us, in place, rank 28, d = 2048 / 4096 / 8192, 300 decode rows 10.5 / 9.4, 16.7 / 15.0, 28.9 / 25.8, rank 20, 32
// rows 8.3 / 8.0, 12.4 / 11.7, 19.9 / 18.5; 900 prompt rows, 4096 -> 4096, rank 28 15.2 / 13.1, rank 20 13.8 / 13.0.
template <int NB, bool DIREFT, bool ODD, bool LINES, int RK> constexpr bool small_direct(int NG)
{
    return ODD ? NB == 1 : NB == 2 && RK != 20 && RK != 28 && (DIREFT || (LINES && NG == 4));
}
// A wavefront's own LDS, in 16-byte vectors: a unit of activations and one of the factor in turn, later a unit's factors of the expand.
template <int NB, bool DIREFT, bool ODD, bool LINES, int RK>
constexpr int small_area()
{
    constexpr int turns = 2 * 16 * MFMA_TRS, factors = small_direct<NB, DIREFT, ODD, LINES, RK>(4) ? (FactorLds<NB>::BYTES + 15) / 16 : 0;
    return turns > factors ? turns : factors;
}

// DEEP: few workgroups, each alone on its compute unit: up to 256 registers for requests in flight.  Otherwise (rank <= 16: the LDS
// of more rank blocks does not fit twice) 128, two workgroups per compute unit, which hide one another's trips.
// One tile and share; `unit` and `share` are uniform over the workgroup.
//
// NG: groups of four rows that the tile fills at most, 1 or 4.  Of a gathered tile of one to four decode rows the other three quarters of
// every load of x and y would bring the same rows again, and the texture path is what a workgroup waits for: 256 KB of x and A
// for a 4096-wide shrink.  (32 decode rows of 32 adapters, rank 16, replayed: q+k+v 8.0 -> 6.5 us, 4096 -> 4096 7.1 -> 5.7, 4096 -> 2 x 14336
// 13.7 -> 10.9, 14336 -> 4096 14.5 -> 11.0, with the launch arguments asked for together.)  Rows that are not loaded leave what was in the turn buffer: their z and y are their own and are not stored.
struct SmallOutput {                                          // the output of a workgroup, and which share of its columns
    void *y;
    int64_t ldy;
    int d_out, share;
    const void *const *A_pool, *const *Bt_pool;
    int slice, slices, rank0;                                 // the shrink alone: which output of how many, and its first rank
};

// RK: 0, or the largest rank of the form: 1, 2, 3 and 4 are that rank, 8 the ranks 5 to 8, 20, 24 and 28 that rank.  An instruction brings four ranks of a unit of A:
// those that no such rank has are left out.  Ranks 1-3 are too thin for the matrix cores' expand, and z stays
// in fp32: the sums of valu_tile_kernel, a lane's 8 columns of its rows, whose factors are RK 16-byte pieces.
// Before / now, replayed, us: 32 decode rows of 32 adapters, a layer's six launches, rank 1 64.5 / 28.1, 3 118 / 33.5 (valu_tile_kernel: 16 rows of a tile on four wavefronts),
// 8 44.1 / 40.8; rank 4, 4096 -> 4096 5.7 / 4.8; 1000 prompt rows, rank 3, 4096 -> 2 x 14336 75 / 27; in place, d = 4096, rank 1 5.8 / 4.8, 3 7.3 / 5.4, 8 7.9 / 7.4.
//
// ZOUT: the shrink alone, of the NB rank blocks from o.rank0 on.  z goes to the workspace in the form the expand's MFMAs take it (z_piece), and an expand
// launch follows.
template <int NB, bool DIREFT, bool ODD, bool DEEP, int WAVES, int NG, int RK, bool ZOUT, bool LINES>
__device__ __forceinline__ void small_tile_rows(const ApplyArgs &p, const SmallOutput &o, const i32x4_t entry, bool gathered, int row0, int n_rows, int unit,
                                                u32x4_t (&area)[WAVES][small_area<NB, DIREFT, ODD, LINES, RK>()], float (&red)[WAVES * NB * 4 * 64])
{
    constexpr bool ANY = ODD && NB > 1;                       // ranks above 16 that are no multiple of 4
    constexpr bool DIRECT = !ZOUT && small_direct<NB, DIREFT, ODD, LINES, RK>(NG), THIN = RK >= 1 && RK <= 3;
    constexpr int RANKS = RK ? RK : 16 * NB;
    auto groups = [](int b) constexpr { return RANKS - 16 * b > 8 ? 4 : (RANKS - 16 * b + 3) / 4; };     // of four ranks in block b of a unit of A that are loaded: 1, 2 or 4
    // units of the shrink and of the expand sweep in flight (registers)
    constexpr int BATCH = ZOUT ? 2 : DEEP ? (NB == 1 ? 4 : NB <= 4 ? 2 : 1) : 2;
    // units of the expand that are asked for before the shrink's last ones are used (registers).  With that, waits for one unit at a time (sweep below) and
    // the bias ahead of the sums, 32 decode rows of 32 adapters, rank 16, replayed: 14336 -> 4096 10.9 -> 10.4 us, 4096 -> 2 x 14336 10.9 -> 10.6, in place, d = 4096,
    // 8.1 -> 7.9, 8 layers of it 12.8 -> 12.2, a layer's six launches 47.9 -> 45.7; 481 prompt rows, rank 8, q+k+v 9.2 -> 8.8.
    constexpr int EARLY = !ZOUT && NG == 1 && DEEP && NB <= 2 ? (DIREFT && NB == 1 ? 2 : 1) : 0;
    constexpr int DEPTH = DEEP ? (NB == 1 ? (DIRECT || NG == 1 ? 2 : 4) : NB == 2 ? (NG == 1 ? 1 : 2) : 1) : 1;
    constexpr bool W_LATE = NB > 4;                           // factors of the expand step by step (registers)
    static_assert(DEEP || NB == 1, "two workgroups of more rank blocks do not fit a compute unit");
    constexpr int PIECES = (RANKS + 3) / 4;                   // DIRECT: 16-byte pieces of a unit's factor block per lane
    const int per_share = p.col_split;                        // units of a share
    void *const y = o.y;
    const int64_t ldy = o.ldy;
    const int d_out = o.d_out, share = o.share;
    static_assert(!ZOUT || (!ODD && NB > 1 && NB <= WAVES), "multiples of 4 above 16; a wavefront writes a rank block");
    const int r = ZOUT ? min(p.rank - o.rank0, 16 * NB) : p.rank;        // ranks of this workgroup
    gcptr_t A = as_global(as_const(o.A_pool)[entry[0]]);
    if constexpr (ZOUT) A += (int64_t)o.rank0 * p.d_in * 2;
    gcptr_t Bt = ZOUT ? nullptr : as_global(as_const(o.Bt_pool)[entry[0]]);

    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    int lane = threadIdx.x & 63;
    asm volatile("" : "+v"(lane));                            // recomputed for every tile: what hangs on the lane would fill the registers
    const int rl = lane & 15, g = lane >> 4;                  // MFMA order
    const int q = lane >> 4, c16 = lane & 15;                 // unit load order
    u32x4_t *tr = area[wave], *tra = area[wave] + 16 * MFMA_TRS;

    // Row slot of the lane in load i (DIRECT: those that an accumulator of z times factors has for it).  Slots past the tile alias its last
    // row: same loads, same values; their stores are left out
    auto slot = [&](int i) { return DIRECT && NG > 1 ? 4 * q + i : 4 * i + q; };
    int32_t row[NG];
#pragma unroll
    for (int i = 0; i < NG; ++i) row[i] = entry[1] + row0 + min(slot(i), n_rows - 1);
    if (gathered) {
#pragma unroll
        for (int i = 0; i < NG; ++i) row[i] = p.shorts[row[i]].y;
    }
    gcptr_t xu[NG];
    gptr_t yu[NG];
#pragma unroll
    for (int i = 0; i < NG; ++i) {
        xu[i] = as_global(p.x) + row[i] * p.ldx * 2;
        yu[i] = as_global(y) + row[i] * ldy * 2;
    }

    // ---------------------------------------------------------------- requests of the expand
    const int c_units = (d_out + 127) >> 7;
    const int ubase = DIREFT ? 0 : share * per_share, uend = DIREFT ? c_units : min(ubase + per_share, c_units);
    const int y_last = d_out * 2 - 16;
    u32x4_t Y[DEPTH][NG];
    u32x2_t W[DIRECT || THIN ? 1 : DEPTH][W_LATE || DIRECT || THIN ? 1 : 4][2][NB];
    u32x4_t Wb[DIRECT || THIN ? DEPTH : 1][THIN ? RK : PIECES];
    auto load_w = [&](u32x2_t (&w)[2][NB], int u, int s) {
#pragma unroll
        for (int e = 0; e < 2; ++e) {
            // MFMA e of step s: columns 32 s + 8 (m / 4) + 4 e + m % 4 (past the width: the last one; not stored)
            const int col = min(u * 128 + 32 * s + 8 * (rl >> 2) + 4 * e + (rl & 3), d_out - 1);
#pragma unroll
            for (int b = 0; b < NB; ++b) {
                const int rank0 = 16 * b + 4 * g;
                if constexpr (ANY) w[e][b] = ld8_any(Bt + ((int64_t)col * r + quad_start(rank0, r)) * 2);
                else w[e][b] = ld8(Bt + ((int64_t)col * r + (rank0 < r ? rank0 : 0)) * 2);
            }
        }
    };
    auto load_yw = [&](int k, int u) {
        const int off = min(u * 256 + c16 * 16, y_last);
#pragma unroll
        for (int i = 0; i < NG; ++i) Y[k][i] = ld16(yu[i] + off);
        if constexpr (THIN) {                                 // the lane's 8 columns (past the width: the last 8)
            gcptr_t wp = Bt + (int64_t)(off >> 4) * (16 * RK);
#pragma unroll
            for (int j = 0; j < RK; ++j) Wb[k][j] = ld16(wp + j * 16);
        } else if constexpr (DIRECT) {                        // the unit's [128 columns][r] block, contiguous
            const int last = last_factor_piece(d_out - u * 128, 128, r);
#pragma unroll
            for (int j = 0; j < PIECES; ++j) Wb[k][j] = ld16(Bt + (int64_t)u * 256 * r + min(min(lane + 64 * j, 16 * r - 1), last) * 16);
        } else if constexpr (!W_LATE) {
#pragma unroll
            for (int s = 0; s < 4; ++s) load_w(W[k][s], u, s);
        }
    };
    // A request that hangs on a branch has every later wait wait for all that is on its way: the first ones ask for units that need not exist (the
    // last one again).
    auto request_early = [&] {
#pragma unroll
        for (int k = 0; k < EARLY; ++k) load_yw(k, min(ubase + wave + k * WAVES, c_units - 1));
    };
    // (only where every wavefront has a unit: rank 20, 512 -> 2072, 32 decode rows 4.2 us, 4.9 where all eight asked for those of two)
    constexpr bool ALWAYS_EARLY = NB == 1;
    const bool early = EARLY > 0 && uend - ubase >= WAVES;
    auto request_some = [&] {
#pragma unroll
        for (int k = 0; k < EARLY; ++k)
            if (ubase + wave + k * WAVES < uend) load_yw(k, ubase + wave + k * WAVES);
    };
    auto request_expand = [&] {
#pragma unroll
        for (int k = EARLY; k < DEPTH; ++k)
            if (ubase + wave + k * WAVES < uend) load_yw(k, ubase + wave + k * WAVES);
    };

    // ---------------------------------------------------------------- shrink
    f32x4_t acc[NB];
#pragma unroll
    for (int b = 0; b < NB; ++b) acc[b] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    {
        const int x_last = p.d_in * 2 - 16;                   // a row's last 16-byte piece; d_in % 8 == 0
        const int k_units = (p.d_in + 127) >> 7;
        auto load_a = [&](u32x4_t (&a)[4], int b, int off) {
#pragma unroll
            for (int i = 0; i < groups(b); ++i)                      // ranks past r alias the last one: their z is zeroed
                a[i] = ld16(A + (uint32_t)(min(16 * b + 4 * i + q, r - 1) * (x_last + 16) + off));
        };
        constexpr int HALVES = BATCH > 1 ? 2 : 1, H = BATCH / HALVES;
        auto request = [&](auto &x, auto &a, int u0, auto always) {
            constexpr int UNITS = sizeof(x) / sizeof(x[0]);
#pragma unroll
            for (int k = 0; k < UNITS; ++k)
                if (decltype(always)::value || u0 + k * WAVES < k_units) {
                    const int off = min((u0 + k * WAVES) * 256 + c16 * 16, x_last);
#pragma unroll
                    for (int i = 0; i < NG; ++i) x[k][i] = ld16(xu[i] + off);
#pragma unroll
                    for (int b = 0; b < NB; ++b) load_a(a[k][b], b, off);
                }
        };
        auto use = [&](auto &x, auto &a, int u0) {
            constexpr int UNITS = sizeof(x) / sizeof(x[0]);
#pragma unroll
            for (int k = 0; k < UNITS; ++k)
                if (u0 + k * WAVES < k_units) {
                    if ((u0 + k * WAVES) * 256 + c16 * 16 > x_last) {    // past the width: zero times zero
#pragma unroll
                        for (int i = 0; i < NG; ++i) x[k][i] = u32x4_t{0u, 0u, 0u, 0u};
#pragma unroll
                        for (int i = 0; i < 4; ++i)
#pragma unroll
                            for (int b = 0; b < NB; ++b) a[k][b][i] = u32x4_t{0u, 0u, 0u, 0u};
                    }
                    u32x4_t xo[4], ao[4];
#pragma unroll
                    for (int i = 0; i < NG; ++i) tr[slot(i) * MFMA_TRS + c16] = x[k][i];
#pragma unroll
                    for (int s = 0; s < 4; ++s) xo[s] = tr[rl * MFMA_TRS + 4 * s + g];
#pragma unroll
                    for (int b = 0; b < NB; ++b) {
#pragma unroll
                        for (int i = 0; i < groups(b); ++i) tra[(4 * i + q) * MFMA_TRS + c16] = a[k][b][i];
#pragma unroll
                        for (int s = 0; s < 4; ++s) ao[s] = tra[(rl & (4 * groups(b) - 1)) * MFMA_TRS + 4 * s + g];
#pragma unroll
                        for (int s = 0; s < 4; ++s)
                            acc[b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(ao[s]), as_bf16x8(xo[s]), acc[b], 0, 0, 0);
                    }
                }
        };
        // Tiles of few rows: `B` units on their way, each in registers of its own.  No request hangs on a branch (past the last unit: that one again, not
        // used), so a wait is for its own unit and the others go on arriving.
        auto sweep = [&](auto b_tag) {
            constexpr int B = decltype(b_tag)::value;
            if (wave >= k_units) { request_some(); return; }
            u32x4_t xr[B][1][NG], ar[B][1][NB][4];
            auto ask = [&](int k, int u) { request(xr[k], ar[k], min(u, k_units - 1), std::true_type{}); };
#pragma unroll
            for (int k = 0; k < B; ++k) ask(k, wave + k * WAVES);
            int u = wave;
            if constexpr (B == BATCH) {                       // (fewer only where they are all)
                for (; u + B * WAVES < k_units; u += B * WAVES) {
#pragma unroll
                    for (int k = 0; k < B; ++k) {
                        use(xr[k], ar[k], u + k * WAVES);
                        ask(k, u + (B + k) * WAVES);
                    }
                }
            }
            if (B == 1 && k_units <= WAVES) {                 // a unit each at most: the shrink's trip is the only one before the sums
                use(xr[0], ar[0], u);
                request_some();
            } else if (ALWAYS_EARLY || early) {
                request_early();
#pragma unroll
                for (int k = 0; k < B; ++k) use(xr[k], ar[k], u + k * WAVES);
            } else {
                request_some();
#pragma unroll
                for (int k = 0; k < B; ++k) use(xr[k], ar[k], u + k * WAVES);
            }
        };
        if constexpr ((NG == 1 || ZOUT) && BATCH > 1) {
            const int mine = k_units - wave;                  // units of this wavefront: of the first, every WAVES-th
            if (mine <= WAVES) sweep(std::integral_constant<int, 1>{});
            else if (BATCH > 2 && mine <= 2 * WAVES) sweep(std::integral_constant<int, 2>{});
            else sweep(std::integral_constant<int, BATCH>{});
        } else if constexpr (HALVES == 2) {
            // two halves of a batch take turns: one is on its way while the other is used
            u32x4_t xr[2][H][NG], ar[2][H][NB][4];
            request(xr[0], ar[0], wave, std::false_type{});
            request(xr[1], ar[1], wave + H * WAVES, std::false_type{});
            int u = wave;
            for (; u + 2 * H * WAVES < k_units; u += 2 * H * WAVES) {
                use(xr[0], ar[0], u);
                request(xr[0], ar[0], u + 2 * H * WAVES, std::false_type{});
                use(xr[1], ar[1], u + H * WAVES);
                request(xr[1], ar[1], u + 3 * H * WAVES, std::false_type{});
            }
            use(xr[0], ar[0], u);
            use(xr[1], ar[1], u + H * WAVES);
        } else {
            u32x4_t xr[1][H][NG], ar[1][H][NB][4];
            for (int u = wave; u < k_units; u += H * WAVES) {
                request(xr[0], ar[0], u, std::false_type{});
                use(xr[0], ar[0], u);
            }
        }
    }

    if constexpr (!ZOUT) request_expand();                    // before z is summed

    const FactorLds<DIRECT ? NB : 1> fl(r);
    char *const fw = reinterpret_cast<char *>(area[wave]);
    auto park = [&](int k) {                                  // a unit's factors to LDS
        if constexpr (DIRECT && !THIN) {
#pragma unroll
            for (int j = 0; j < PIECES; ++j) {
                const int piece = min(lane + 64 * j, 16 * r - 1);
                if constexpr (ODD) {
                    *reinterpret_cast<u32x4_t *>(fw + piece * 16) = Wb[k][j];
                } else {                                      // two 8-byte halves, neither straddles a column
                    *reinterpret_cast<u32x2_t *>(fw + fl.quarter(2 * piece)) = u32x2_t{Wb[k][j][0], Wb[k][j][1]};
                    *reinterpret_cast<u32x2_t *>(fw + fl.quarter(2 * piece + 1)) = u32x2_t{Wb[k][j][2], Wb[k][j][3]};
                }
            }
        }
    };
    // (at rank 17-32 before the sums, whose wait it fills; with half the factors it is quicker not to wait for them here)
    constexpr bool PARK_FIRST = NB == 2;
    if constexpr (PARK_FIRST) park(0);

    // the bias of ranks `lane` and, above rank 64, 64 + `lane`: its two trips beside the wait for the sums, not after it
    float bias[NB > 4 ? 2 : 1] = {};
    if constexpr (DIREFT) {
        gcptr_t bias_p = bias_of(p, entry[0]);
        if (bias_p) {
#pragma unroll
            for (int j = 0; j < (NB > 4 ? 2 : 1); ++j) bias[j] = Elem<bf16_tag>::load1(bias_p, (ZOUT ? o.rank0 : 0) + min(64 * j + lane, r - 1));
        }
    }

    // ---------------------------------------------------------------- sum over the wavefronts, z -> expand operand
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
        for (int v = 0; v < 4; ++v) red[((wave * NB + b) * 4 + v) * 64 + lane] = acc[b][v];
    __syncthreads();                                          // also: every read of the tile precedes every write (in place: a unit belongs to one wavefront)
    // DIRECT, up to four rows: those stand in rows 0, 4, 8, 12 of the operand, so that a lane's accumulators begin with its own row
    const int zlane = DIRECT && NG == 1 ? (rl >> 2) + 16 * g : lane;
    float zt[NG][THIN ? RK : 1];
    bf16x8_t zop[NB];
    u32x4_t zlow[ANY ? NB / 2 : 1];                           // what two parts of bf16 leave of z (whole_z), two rank blocks in one operand
#pragma unroll
    for (int b = 0; b < NB; ++b) {
        if constexpr (ZOUT) { if (b != wave) continue; }      // (uniform)
        const int rank0 = 16 * b + 4 * g;
        float zv[4], rem[4];
#pragma unroll
        for (int v = 0; v < (THIN ? RK : 4); ++v) {
            float s = 0.f;
#pragma unroll
            for (int w = 0; w < WAVES; ++w) s += red[((w * NB + b) * 4 + v) * 64 + zlane];
            float add = 0.f;
            if constexpr (DIREFT) add = __shfl(bias[b / 4], rank0 % 64 + v, 64);
            zv[v] = rank0 + v < r ? (s + add) * p.scale : 0.f;
            rem[v] = zv[v] - __uint_as_float((pack_bf16(zv[v], 0.f) & 0xffffu) << 16);
        }
        if constexpr (THIN) {                                 // lanes 0 to 15 hold the rows' z, the lane's rows are slot(i)
#pragma unroll
            for (int i = 0; i < NG; ++i)
#pragma unroll
                for (int v = 0; v < RK; ++v) zt[i][v] = __shfl(zv[v], slot(i), 64);
        } else if constexpr (ANY) {
            const WholeZ w = whole_z(zv);
            zop[b] = as_bf16x8(u32x4_t{w.head[0], w.head[1], w.mid[0], w.mid[1]});
            zlow[b / 2][2 * (b % 2)] = w.low[0];
            zlow[b / 2][2 * (b % 2) + 1] = w.low[1];
        } else {
            zop[b] = as_bf16x8(u32x4_t{pack_bf16(zv[0], zv[1]), pack_bf16(zv[2], zv[3]), pack_bf16(rem[0], rem[1]), pack_bf16(rem[2], rem[3])});
        }
    }

    if constexpr (ZOUT) {
        u32x4_t *zw = reinterpret_cast<u32x4_t *>(p.zws) + lane;
#pragma unroll
        for (int b = 0; b < NB; ++b)
            if (b == wave && 16 * b < r) zw[z_piece(unit, o.slices, o.slice, z_rank_blocks(p.rank), o.rank0 / 16 + b)] = as_u32x4(zop[b]);
        return;
    } else {

    // ---------------------------------------------------------------- expand
    // y plus the products of step s, in MFMA order (ANY only: `nan`, whether a result is NaN; finite_tag as in whole_z_products)
    auto products = [&](const u32x4_t y, const u32x2_t (&wv)[2][NB], int s, bool &nan, auto finite_tag) -> u32x4_t {
        float out[8];
#pragma unroll
        for (int e = 0; e < 2; ++e) {
            f32x4_t d = {0.f, 0.f, 0.f, 0.f};
            if constexpr (ANY) {
                d = whole_z_products<NB, decltype(finite_tag)::value>([&](int b) { return quad_from(wv[e][b], 16 * b + 4 * g, r); },
                                                                      [&](int b) { return zop[b]; }, [&](int i) { return zlow[i]; });
                nan = nan || __builtin_isunordered(d[0], d[1]) || __builtin_isunordered(d[2], d[3]);
            } else {
#pragma unroll
                for (int b = 0; b < NB; ++b) {
                    const u32x2_t w = wv[e][b];
                    d = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(u32x4_t{w[0], w[1], w[0], w[1]}), zop[b], d, 0, 0, 0);
                }
            }
            const uint32_t y01 = y[2 * e], y23 = y[2 * e + 1];
            out[4 * e + 0] = bf16_lo(y01) + d[0];
            out[4 * e + 1] = bf16_hi(y01) + d[1];
            out[4 * e + 2] = bf16_lo(y23) + d[2];
            out[4 * e + 3] = bf16_hi(y23) + d[3];
        }
        return Elem<bf16_tag>::pack(out);
    };
    // z as the first operand, the factors as the second: lane (n16, g) of MFMA k ends up with column 8 n16 + k of the rows
    // that it has loaded
    auto finish_direct = [&](int k, int u) {
        if (!PARK_FIRST || u != ubase + wave) park(k);
#pragma unroll
        for (int k2 = 0; k2 < 4; ++k2) {
            f32x4_t d[2];
#pragma unroll
            for (int e = 0; e < 2; ++e) {
                d[e] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int b = 0; b < NB; ++b) {
                    const u32x2_t w = fl.template operand<ODD>(fw, 2 * k2 + e, b, c16, g, r);
                    d[e] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(zop[b], as_bf16x8(u32x4_t{w[0], w[1], w[0], w[1]}), d[e], 0, 0, 0);
                }
            }
#pragma unroll
            for (int i = 0; i < NG; ++i) Y[k][i][k2] = pack_bf16(bf16_lo(Y[k][i][k2]) + d[0][i], bf16_hi(Y[k][i][k2]) + d[1][i]);
        }
        const int off = u * 256 + c16 * 16;
#pragma unroll
        for (int i = 0; i < NG; ++i)
            if (off <= y_last && slot(i) < n_rows) st16_stream(yu[i] + off, Y[k][i]);
    };
    auto finish_thin = [&](int k, int u) {
        float w[8 * RK + 1];
#pragma unroll
        for (int j = 0; j < RK; ++j)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                w[j * 8 + 2 * e] = bf16_lo(Wb[k][j][e]);
                w[j * 8 + 2 * e + 1] = bf16_hi(Wb[k][j][e]);
            }
        const int off = u * 256 + c16 * 16;
#pragma unroll
        for (int i = 0; i < NG; ++i) {
            float out[8];
            Elem<bf16_tag>::unpack(Y[k][i], out);
#pragma unroll
            for (int c = 0; c < 8; ++c) {
                float d = 0.f;
#pragma unroll
                for (int v = 0; v < RK; ++v) d = fmaf(w[c * RK + v], zt[i][v], d);
                out[c] += d;
            }
            if (off <= y_last && slot(i) < n_rows) st16_stream(yu[i] + off, Elem<bf16_tag>::pack(out));
        }
    };
    auto finish = [&](int k, int u) {
        u32x4_t yo[4];
#pragma unroll
        for (int i = 0; i < NG; ++i) tr[slot(i) * MFMA_TRS + c16] = Y[k][i];
#pragma unroll
        for (int s = 0; s < 4; ++s) yo[s] = tr[rl * MFMA_TRS + 4 * s + g];
        bool nan = false;
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            if constexpr (W_LATE) load_w(W[0][0], u, s);
            tr[rl * MFMA_TRS + 4 * s + g] = products(yo[s], W[k][W_LATE ? 0 : s], s, nan, std::false_type{});
        }
        const int off = u * 256 + c16 * 16;
        if constexpr (ANY) {
            if (__any(nan && rl < n_rows)) {                  // (rows that do not exist may hold anything)
#pragma unroll
                for (int i = 0; i < NG; ++i) tr[slot(i) * MFMA_TRS + c16] = ld16(yu[i] + min(off, y_last));
#pragma unroll 1
                for (int s = 0; s < 4; ++s) {
                    u32x2_t w[2][NB];
                    load_w(w, u, s);
                    u32x4_t &place = tr[rl * MFMA_TRS + 4 * s + g];
                    place = products(place, w, s, nan, std::true_type{});
                }
            }
        }
#pragma unroll
        for (int i = 0; i < NG; ++i) {
            const u32x4_t v = tr[slot(i) * MFMA_TRS + c16];
            if (off <= y_last && slot(i) < n_rows) st16_stream(yu[i] + off, v);
        }
    };
    for (int u = ubase + wave; u < uend; u += WAVES * DEPTH) {
#pragma unroll
        for (int k = 0; k < DEPTH; ++k)
            if (u + k * WAVES < uend) {
                if constexpr (THIN) finish_thin(k, u + k * WAVES);
                else if constexpr (DIRECT) finish_direct(k, u + k * WAVES);
                else finish(k, u + k * WAVES);
                if (u + (k + DEPTH) * WAVES < uend) load_yw(k, u + (k + DEPTH) * WAVES);
            }
    }
    }
}

// FEW: with the form for tiles of up to four rows (in place only for steps of decode rows: its second copy of the code costs the others 0.1 us of 4.5).
template <int NB, bool DIREFT, bool ODD, bool DEEP, int WAVES, bool FEW, int RK, bool ZOUT, bool LINES>
__device__ __forceinline__ void small_tile_one(const ApplyArgs &p, const SmallOutput &o, int unit, int n_chunk_units,
                                               u32x4_t (&area)[WAVES][small_area<NB, DIREFT, ODD, LINES, RK>()], float (&red)[WAVES * NB * 4 * 64])
{
    // the tile: 16 rows of a chunk, or a gathered tile (rows listed one by one)
    const bool gathered = unit >= n_chunk_units;
    const int row0 = gathered ? 0 : unit % (CHUNK_ROWS / 16) * 16;
    const i32x4_t entry = *reinterpret_cast<const PREFT_CONST i32x4_t *>(
        gathered ? as_const(p.gtiles) + (unit - n_chunk_units) : as_const(p.chunks) + unit / (CHUNK_ROWS / 16));
    const int n_rows = min(16, entry[2] - row0);
    if (n_rows <= 0) return;                                  // uniform over the workgroup
    if (!FEW || n_rows > 4) small_tile_rows<NB, DIREFT, ODD, DEEP, WAVES, 4, RK, ZOUT, LINES>(p, o, entry, gathered, row0, n_rows, unit, area, red);
    else if constexpr (FEW) small_tile_rows<NB, DIREFT, ODD, DEEP, WAVES, 1, RK, ZOUT, LINES>(p, o, entry, gathered, row0, n_rows, unit, area, red);
}

// A launch out of place: blockIdx.x = 8 share + XCD, blockIdx.y = the slot of a tile on that XCD (in place: blockIdx.x = 8 slot + XCD).  The shares of a
// tile -- those of the first output, then those of the others -- sit on one XCD, and the slots that have a tile come first.  A
// launch has as many slots as the batch is likely to need; what exceeds it is strided over.
struct SmallLaunch { int shares0, shares1; };

template <int NB, bool DIREFT, bool ODD, bool DEEP, int WAVES, bool FEW, int RK, bool LINES>
__device__ __forceinline__ void small_tile_body(const ApplyArgs &p, const SmallLaunch &l)
{
    __shared__ u32x4_t area[WAVES][small_area<NB, DIREFT, ODD, LINES, RK>()];
    __shared__ float red[WAVES * NB * 4 * 64];

    // What the launch arguments say is asked for together with the header: each line of them that is touched later is a trip of its own (in
    // place, rank 16, d = 512, 220 rows 4.4 us without, 4.3 with).
    SmallOutput o = {p.y, p.ldy, p.d_out, 0, p.A_pool, p.Bt_pool, 0, 1, 0};
    if constexpr (!DIREFT) {
        o.share = blockIdx.x >> 3;
        if (o.share >= l.shares0) {
            const int sl = o.share >= l.shares0 + l.shares1 ? 2 : 1;
            o.share -= sl == 2 ? l.shares0 + l.shares1 : l.shares0;
            o.y = p.more[sl - 1].y; o.ldy = p.more[sl - 1].ldy; o.d_out = p.more[sl - 1].d_out;
            o.A_pool = p.more[sl - 1].A_pool; o.Bt_pool = p.more[sl - 1].Bt_pool;
        }
    }
    if constexpr (!DIREFT) asm volatile("" ::"s"(o.y), "s"(o.d_out), "s"(o.A_pool), "s"(o.Bt_pool), "s"(p.x), "s"(p.gtiles), "s"(p.chunks), "s"(p.shorts), "s"(p.rank));
    else asm volatile("" ::"s"(p.rank), "s"(p.d_out), "s"(p.col_split));
    if (!schedule_matches(p)) return;
    int n_chunk_units;
    const int n_units = tile_units<16>(p, &n_chunk_units);
    const int per_xcd = (n_units + 7) >> 3;
    for (int t = DIREFT ? blockIdx.x >> 3 : blockIdx.y; t < per_xcd; t += DIREFT ? gridDim.x >> 3 : gridDim.y) {
        const int unit = few_tiles_unit(p, n_chunk_units, per_xcd, t);
        if (unit < n_units) small_tile_one<NB, DIREFT, ODD, DEEP, WAVES, FEW, RK, false, LINES>(p, o, unit, n_chunk_units, area, red);
        __syncthreads();                                      // the next tile's sums go where this one's are still being read
    }
}

template <int NB, bool DIREFT, bool ODD, bool DEEP, int WAVES = SMALL_WAVES, bool FEW = true, int RK = 0, bool LINES = true>
__global__ __launch_bounds__(WAVES * 64, DEEP ? 2 : 4) void small_tile_kernel(ApplyArgs p, SmallLaunch l)
{
    small_tile_body<NB, DIREFT, ODD, DEEP, WAVES, FEW, RK, LINES>(p, l);
}

// the same for one of several residual streams (in-place calls): blockIdx.y is the layer
template <int NB, bool ODD, bool FEW, int RK = 0>
__global__ __launch_bounds__(SMALL_WAVES * 64, 2) void small_tile_layers_kernel(ApplyArgs p, SmallLaunch l)
{
    // beside the layer's pointers, not after them (8 layers, d = 512, 220 rows 7.7 us, now 7.3; 4 layers, d = 1024, 600 rows 7.4 / 7.1)
    // (above rank 32 there are no registers for that: 8 layers, rank 64, d = 1024, 400 rows 21.9 / 24.2)
    if constexpr (NB <= 2) asm volatile("" ::"s"(p.rank), "s"(p.d_out), "s"(p.col_split), "s"(p.header), "s"(p.T));
    select_layer(p);
    small_tile_body<NB, true, ODD, true, SMALL_WAVES, FEW, RK, true>(p, l);
}

// The shrink of a two-launch call of few tiles, rank 17 and up in multiples of 4: blockIdx.x = 8 part + XCD, a part being NB rank blocks of one of the
// outputs; blockIdx.y = the slot of a tile on that XCD.  Bound: a compute unit's texture path (64 bytes a cycle), through which a workgroup brings its tile's x and 32 to
// 64 ranks of A; two units on their way per wavefront.  Against the row-split kernel's 64-row tiles, whose wavefronts sweep all columns of their rows
// one unit after the other, whole calls, us: 1400 prompt rows, 4096 -> 4096, rank 32 30.2 / 17.0, 64 36.7 / 17.8; 8192 -> 8192, rank 64 64 / 26; 3600 rows, 4096 -> 4096, rank 32 57.8 /
// 32.4.  Against the small-batch kernel's single launch, 900 rows: rank 64, 4096 -> 4096 26.9 / 14.7, in place 42 / 16.5; rank 128 48 / 17.5, in place 137 (128-row tiles) / 19.6.
// WAVES: those of the single launch for the same batch (SmallShape), which sum z in that many groups: with and without room for z the bits are the same.
template <int NB, bool DIREFT, int RK = 0, int WAVES = SMALL_WAVES>
__global__ __launch_bounds__(WAVES * 64, 2) void small_shrink_kernel(ApplyArgs p, int slices)
{
    __shared__ u32x4_t area[WAVES][small_area<NB, DIREFT, false, false, RK>()];
    __shared__ float red[WAVES * NB * 4 * 64];
    const int parts = (p.rank + 16 * NB - 1) / (16 * NB), part = blockIdx.x >> 3, sl = part / parts;
    SmallOutput o = {nullptr, 0, 0, 0, p.A_pool, nullptr, sl, slices, (part - sl * parts) * 16 * NB};
    if constexpr (!DIREFT) {
        if (sl == 1) o.A_pool = p.more[0].A_pool;
        if (sl == 2) o.A_pool = p.more[1].A_pool;
    }
    asm volatile("" ::"s"(o.A_pool), "s"(p.x), "s"(p.gtiles), "s"(p.chunks), "s"(p.shorts), "s"(p.rank), "s"(p.zws));
    if (!schedule_matches(p)) return;
    int n_chunk_units;
    const int n_units = min((int64_t)tile_units<16>(p, &n_chunk_units), p.z_blocks);      // (only tables whose segments overlap list more tiles)
    const int per_xcd = (n_units + 7) >> 3;
    for (int t = blockIdx.y; t < per_xcd; t += gridDim.y) {
        const int unit = few_tiles_unit(p, n_chunk_units, per_xcd, t);
        if (unit < n_units) small_tile_one<NB, DIREFT, false, true, WAVES, true, RK, true, false>(p, o, unit, n_chunk_units, area, red);
        __syncthreads();                                      // the next tile's sums go where this one's are still being read
    }
}

}  // namespace preft
