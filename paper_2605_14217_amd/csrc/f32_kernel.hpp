// MFMA tile kernel for fp32 storage, every rank up to 128.
//
// One workgroup of WAVES wavefronts owns a tile of 16 rows of one adapter; the wavefronts split the columns in
// units of 64 (256 bytes per row, as in mfma_tile_kernel: 4 rows x 256 bytes per instruction, turned through a
// wavefront-private LDS buffer).  v_mfma_f32_16x16x4_f32, fp32 products and sums throughout:
//   shrink (Eq. 2: z = A x;  Eq. 3: z = A h + b): a lane (rank or row m, group g) holds the 16-byte piece 4s + g of
//       the unit, columns 16s + 4g .. + 3 of it; MFMA t of step s takes element t of both operands, so its four
//       k are columns 16s + 4g + t, g = 0..3.  A unit is summed in eight chains of two MFMAs, and the units of a
//       wavefront, the wavefronts after that: short chains keep the error of a sum of 4096 terms at or below that of
//       the per-row kernel, and the matrix pipe busy.
//   expand (Eq. 2: y += s B z;  Eq. 3: h += s B^T z): MFMA t of rank block b takes ranks 16b + 4g + t; the accumulator
//       of the shrink (lane (row, g): ranks 16b + 4g .. + 3) is its operand as it stands, the factor operand is the
//       16-byte piece of ranks 16b + 4g .. + 3 of a column (ranks that are not multiples of 4: element by element).
//       Lane (row, g) then owns columns 16s + 4g .. + 3: the piece it holds of the turned y.
// Widths are multiples of 4: pieces past the width alias the last one, are zeroed in the shrink and not stored.
//
// Bound: HBM in principle; in practice latency (fp32 batches are small).  Hence col_split workgroups share a tile of
// an out-of-place call, each running the whole shrink and expanding its share of the columns; where few tiles of wide rows wait for
// the chain of units all the same, the per-row kernel is taken (f32_rows_win).
// Per-row kernel (no matrix cores, factors streamed for every 4 rows) and this one: 4096 -> 4096, rank 16, 2304 rows 80 and
// 32 us (floor 19), 20 480 rows 508 and 205 (169); rank 64, 2304 rows 397 and 70; in place, d = 4096, rank 63 2730 and 88.  Above rank
// 64 the in-place form and the ranks that are no multiple of 4 spill (55-460 registers) and are still the faster ones: in place, d =
// 4096, 2304 rows, rank 127 5780 and 373, rank 100, 1024 -> 1024 960 and 35, 24 rows of d = 4832, rank 96 550 and 168.
// Relative error against 64 bits 1.5e-7 and 1.1e-7 (rank 16), 1.6e-7 and 1.2e-7 (rank 64).
#pragma once
#include "common.hpp"
#include "mfma_kernel.hpp"

#include <type_traits>

namespace preft {

constexpr int F32_WAVES = 8;
constexpr int f32_red_bytes(int NB) { return F32_WAVES * NB * 4 * 64 * 4; }
constexpr int f32_turn_bytes() { return F32_WAVES * 2 * 16 * MFMA_TRS * 16; }

// BY_LDS (ranks up to 32 that are no multiple of 4): the expand takes z as its first operand and whole units of factors through LDS, see below.
// HINT: y with the non-temporal hint (activations_stay has the rule).
template <int NB, bool DIREFT, bool ODD, bool BY_LDS, bool HINT>
__device__ __forceinline__ void f32_tile_body(const ApplyArgs &p)
{
    constexpr int WAVES = F32_WAVES;
    constexpr bool AHEAD = NB <= 2;                           // register budget: factors requested a unit ahead, or block by block
    static_assert(!BY_LDS || (ODD && NB <= 2), "ranks up to 32 that are no multiple of 4");
    static_assert(!BY_LDS || 64 * 16 * NB * 4 <= 2 * 16 * MFMA_TRS * 16, "a unit's factors fit the turn buffers");
    __shared__ __attribute__((aligned(16))) char lds[f32_red_bytes(NB) > f32_turn_bytes() ? f32_red_bytes(NB) : f32_turn_bytes()];

    if (!schedule_matches(p)) return;
    const int csplit = DIREFT ? 1 : p.col_split;
    int n_chunk_units;
    const int n_units = tile_units<16>(p, &n_chunk_units);
    // workgroups that share a tile sit side by side on one XCD (ids are dealt round-robin to the 8 XCDs)
    const int per_xcd = (n_units + 7) >> 3;
    const int t = (blockIdx.x >> 3) / csplit, cslice = (blockIdx.x >> 3) - t * csplit;
    const int unit = t < per_xcd ? few_tiles_unit(p, n_chunk_units, per_xcd, t) : n_units;
    if (unit >= n_units) return;
    TileRows tile;
    if (!tile_rows<16>(p, unit, n_chunk_units, tile)) return; // uniform over the workgroup

    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int rl = lane & 15, g = lane >> 4;                  // MFMA order
    const int q = lane >> 4, c16 = lane & 15;                 // unit load order
    const int r = p.rank;
    u32x4_t *tr = reinterpret_cast<u32x4_t *>(lds) + wave * (2 * 16 * MFMA_TRS);
    u32x4_t *tra = tr + 16 * MFMA_TRS;
    float *red = reinterpret_cast<float *>(lds);

    // row slots past the end of the tile alias its last row: same loads, same values; their stores are left out
    int64_t row_u[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) row_u[i] = tile.row(4 * i + q);
    gcptr_t A = as_global(as_const(p.A_pool)[tile.adapter]);
    gcptr_t Bt = as_global(as_const(p.Bt_pool)[tile.adapter]);
    gcptr_t xu[4];
    gptr_t yu[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        xu[i] = as_global(p.x) + row_u[i] * p.ldx * 4;
        yu[i] = as_global(p.y) + (BY_LDS ? tile.row(4 * q + i) : row_u[i]) * p.ldy * 4;
    }
    auto turned = [&](const u32x4_t (&raw)[4], u32x4_t (&op)[4], u32x4_t *buf) {
#pragma unroll
        for (int i = 0; i < 4; ++i) buf[(4 * i + q) * MFMA_TRS + c16] = raw[i];
#pragma unroll
        for (int s = 0; s < 4; ++s) op[s] = buf[rl * MFMA_TRS + 4 * s + g];
    };
    auto f = [](uint32_t v) { return __uint_as_float(v); };

    // ---------------------------------------------------------------- shrink
    f32x4_t acc[NB];
#pragma unroll
    for (int b = 0; b < NB; ++b) acc[b] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    {
        const int k_units = (p.d_in + 63) >> 6;
        const int last = p.d_in * 4 - 16;                     // byte offset of a row's last piece
        constexpr int NA = AHEAD ? NB : 1;
        auto load_a = [&](u32x4_t (&ar)[4], int b, int u) {
            const int off = min(u * 256 + c16 * 16, last);
#pragma unroll
            for (int i = 0; i < 4; ++i)                       // ranks past r alias the last one: their z is zeroed
                ar[i] = ld16(A + (uint32_t)(min(16 * b + 4 * i + q, r - 1) * (last + 16) + off));
        };
        auto load = [&](u32x4_t (&xr)[4], u32x4_t (&ar)[NA][4], int u) {
            const int off = min(u * 256 + c16 * 16, last);
#pragma unroll
            for (int i = 0; i < 4; ++i) xr[i] = ld16(xu[i] + off);      // read again by the workgroups that share the tile, or in place
            if constexpr (AHEAD) {
#pragma unroll
                for (int b = 0; b < NB; ++b) load_a(ar[b], b, u);
            }
        };
        auto use = [&](u32x4_t (&xr)[4], u32x4_t (&ar)[NA][4], int u) {
            const bool past = u * 256 + c16 * 16 > last;      // past the width: zero times zero
            if (past) {
#pragma unroll
                for (int i = 0; i < 4; ++i) xr[i] = u32x4_t{0u, 0u, 0u, 0u};
            }
            u32x4_t xo[4], ao[4];
            turned(xr, xo, tr);
#pragma unroll
            for (int b = 0; b < NB; ++b) {
                u32x4_t (&a)[4] = ar[AHEAD ? b : 0];
                if constexpr (!AHEAD) load_a(a, b, u);
                if (past) {
#pragma unroll
                    for (int i = 0; i < 4; ++i) a[i] = u32x4_t{0u, 0u, 0u, 0u};
                }
                turned(a, ao, tra);
                f32x4_t part[8];
#pragma unroll
                for (int c = 0; c < 8; ++c) {                 // chain c: half the elements of step c / 2
                    part[c] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                    for (int e = 2 * (c & 1); e < 2 * (c & 1) + 2; ++e)
                        part[c] = __builtin_amdgcn_mfma_f32_16x16x4f32(f(ao[c / 2][e]), f(xo[c / 2][e]), part[c], 0, 0, 0);
                }
                acc[b] += ((part[0] + part[1]) + (part[2] + part[3])) + ((part[4] + part[5]) + (part[6] + part[7]));
            }
        };
        u32x4_t x0[4], x1[4], a0[NA][4], a1[NA][4];
        int u = wave;
        if (u < k_units) load(x0, a0, u);
        while (u < k_units) {
            if (u + WAVES < k_units) load(x1, a1, u + WAVES);
            use(x0, a0, u);
            u += WAVES;
            if (u >= k_units) break;
            if (u + WAVES < k_units) load(x0, a0, u + WAVES);
            use(x1, a1, u);
            u += WAVES;
        }
    }

    // the wavefront's first unit of y and its factors are requested before z is summed
    const int c_units = (p.d_out + 63) >> 6;
    const int ubase = c_units * cslice / csplit, uend = c_units * (cslice + 1) / csplit;
    const int y_last = p.d_out * 4 - 16;
    constexpr int NW = AHEAD ? 4 : 1;
    u32x4_t y0[4], y1[4], w0[NW][NB], w1[NW][NB];
    auto load_w = [&](u32x4_t (&wr)[NB], int u, int s) {
        const int col = min(u * 64 + 16 * s + rl, p.d_out - 1);          // MFMA row m = rl of step s
        gcptr_t wc = Bt + (int64_t)col * r * 4;
#pragma unroll
        for (int b = 0; b < NB; ++b) {
            const int rank0 = 16 * b + 4 * g;
            // ranks past r: the load aliases one that exists, and the value is masked where it is used (zero times an
            // infinite factor would not be zero)
            if constexpr (ODD) {
#pragma unroll
                for (int e = 0; e < 4; ++e) wr[b][e] = ld4(wc + (b < NB / 2 ? rank0 + e : min(rank0 + e, r - 1)) * 4);     // the first half always exists
            } else {
                wr[b] = ld16(wc + (rank0 < r ? rank0 : 0) * 4);
            }
        }
    };
    auto load_yw = [&](u32x4_t (&yr)[4], u32x4_t (&wr)[NW][NB], int u) {
        const int off = min(u * 256 + c16 * 16, y_last);
#pragma unroll
        for (int i = 0; i < 4; ++i) yr[i] = ld16_hint<HINT>(yu[i] + off);
        if constexpr (BY_LDS) {                               // the unit's [64 columns][r] block, 16 r contiguous pieces
            gcptr_t block = Bt + (int64_t)u * 256 * r;
            const int last = min(16 * r, (p.d_out - u * 64) * r / 4) - 1;   // d_out % 4 == 0
#pragma unroll
            for (int j = 0; j < 4 * NB; ++j) wr[j / NB][j % NB] = ld16(block + min(lane + 64 * j, last) * 16);
        } else if constexpr (AHEAD) {
#pragma unroll
            for (int s = 0; s < 4; ++s) load_w(wr[s], u, s);
        }
    };

    // ---------------------------------------------------------------- sum over the wavefronts
    float z[NB][4];
    if (AHEAD && ubase + wave < uend) load_yw(y0, w0, ubase + wave);
    __syncthreads();                                          // the turn buffers become the sum's area
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
        for (int v = 0; v < 4; ++v)
            red[((wave * NB + b) * 4 + v) * 64 + lane] = acc[b][v];
    __syncthreads();                                          // also: every read of the tile precedes every write (in place)
#pragma unroll
    for (int b = 0; b < NB; ++b) {
        const int rank0 = 16 * b + 4 * g;
        gcptr_t bias = DIREFT ? bias_of(p, tile.adapter) : nullptr;
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            float s[WAVES];
#pragma unroll
            for (int w = 0; w < WAVES; ++w) s[w] = red[((w * NB + b) * 4 + v) * 64 + lane];
            const float sum = ((s[0] + s[1]) + (s[2] + s[3])) + ((s[4] + s[5]) + (s[6] + s[7]));
            float add = 0.f;
            if (DIREFT && bias && rank0 + v < r) add = Elem<float>::load1(bias, rank0 + v);
            z[b][v] = rank0 + v < r ? (sum + add) * p.scale : 0.f;
        }
    }
    __syncthreads();                                          // the area is the turn buffers again

    // ---------------------------------------------------------------- expand
    uint32_t last_mask[4];                                    // up to rank 32: which of the lane's factors of the last block exist
#pragma unroll
    for (int e = 0; e < 4; ++e) last_mask[e] = 16 * (NB - 1) + 4 * g + (ODD ? e : 0) < r ? 0xffffffffu : 0u;
    // Ranks that are no multiple of 4, up to 32: MFMA t of rank block b and column place k takes ranks 16b + 4g + t of the columns 4n + k; lane
    // (n, g) then owns the columns 4n .. 4n + 3 of the rows 4g .. 4g + 3, which it has loaded: y passes through registers only.
    // The factors of a unit are fetched in whole lines and lie in LDS as in memory.  (Fetched element by element as the operand
    // wants them, every lane is an access of its own: 4096 -> 4096, 2304 rows, rank 7 / 31 35.2 / 49.0 us, now 30.5 / 44.0; in place, rank 11,
    // 11 500 rows 120 and 104.  Multiples of 4 fetch 16 bytes a lane and gain nothing: rank 8 30.1 and 30.6, rank 16 31.9 and 31.2, rank 20 156 and 160.)
    char *fac = reinterpret_cast<char *>(tr);
    auto finish_by_lds = [&](u32x4_t (&y)[4], u32x4_t (&w)[NW][NB], int u) {
#pragma unroll
        for (int j = 0; j < 4 * NB; ++j)
            if (lane + 64 * j < 16 * r) *reinterpret_cast<u32x4_t *>(fac + (lane + 64 * j) * 16) = w[j / NB][j % NB];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            f32x4_t part[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) part[e] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int b = 0; b < NB; ++b)
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const int rank = 16 * b + 4 * g + e;      // past r: one that exists, masked (zero times an infinite factor would not be zero)
                    uint32_t v = *reinterpret_cast<const uint32_t *>(fac + ((4 * c16 + k) * r + min(rank, r - 1)) * 4);
                    if (b == NB - 1) v &= last_mask[e];
                    part[e] = __builtin_amdgcn_mfma_f32_16x16x4f32(z[b][e], f(v), part[e], 0, 0, 0);
                }
            const f32x4_t d = (part[0] + part[1]) + (part[2] + part[3]);
#pragma unroll
            for (int v = 0; v < 4; ++v) y[v][k] = __float_as_uint(f(y[v][k]) + d[v]);
        }
        const int off = u * 256 + c16 * 16;
#pragma unroll
        for (int v = 0; v < 4; ++v)
            if (off <= y_last && 4 * q + v < tile.n_rows) st16_stream(yu[v] + off, y[v]);
    };
    auto finish = [&](u32x4_t (&yr)[4], u32x4_t (&wr)[NW][NB], int u) {
        if constexpr (BY_LDS) { finish_by_lds(yr, wr, u); return; }
        u32x4_t yo[4];
        turned(yr, yo, tr);
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            u32x4_t (&w)[NB] = wr[AHEAD ? s : 0];
            if constexpr (!AHEAD) load_w(w, u, s);
            auto masked = [&](int b, int e) { return 16 * b + 4 * g + (ODD ? e : 0) < r ? w[b][e] : 0u; };
            if (NB < 8 && r != 16 * NB) {                     // (8 blocks: where they are used; a second copy of w would spill)
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    if constexpr (NB <= 2) {                  // only the last block can be partial
                        w[NB - 1][e] &= last_mask[e];
                    } else {
#pragma unroll
                        for (int b = 0; b < NB; ++b) w[b][e] = masked(b, e);
                    }
                }
            }
            f32x4_t part[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) part[e] = f32x4_t{0.f, 0.f, 0.f, 0.f};
            auto products = [&](auto blocks_tag, auto masked_tag) {
#pragma unroll
                for (int b = 0; b < decltype(blocks_tag)::value; ++b)
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        part[e] = __builtin_amdgcn_mfma_f32_16x16x4f32(f(decltype(masked_tag)::value ? masked(b, e) : w[b][e]), z[b][e], part[e], 0, 0, 0);
            };
            if constexpr (NB < 8) products(std::integral_constant<int, NB>{}, std::false_type{});
            else if (r == 128)    products(std::integral_constant<int, 8>{}, std::false_type{});
            else if (r == 96)     products(std::integral_constant<int, 6>{}, std::false_type{});
            else                  products(std::integral_constant<int, NB>{}, std::true_type{});
            const f32x4_t d = (part[0] + part[1]) + (part[2] + part[3]);
            u32x4_t o;
#pragma unroll
            for (int v = 0; v < 4; ++v) o[v] = __float_as_uint(f(yo[s][v]) + d[v]);
            tr[rl * MFMA_TRS + 4 * s + g] = o;
        }
        const int off = u * 256 + c16 * 16;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const u32x4_t o = tr[(4 * i + q) * MFMA_TRS + c16];
            if (off <= y_last && 4 * i + q < tile.n_rows) st16_stream(yu[i] + off, o);
        }
    };
    int u = ubase + wave;
    if (!AHEAD && u < uend) load_yw(y0, w0, u);
    while (u < uend) {
        if (u + WAVES < uend) load_yw(y1, w1, u + WAVES);
        finish(y0, w0, u);
        u += WAVES;
        if (u >= uend) break;
        if (u + WAVES < uend) load_yw(y0, w0, u + WAVES);
        finish(y1, w1, u);
        u += WAVES;
    }
}

template <int NB, bool DIREFT, bool ODD, bool BY_LDS, bool HINT = true>
__global__ __launch_bounds__(F32_WAVES * 64) void f32_tile_kernel(ApplyArgs p) { f32_tile_body<NB, DIREFT, ODD, BY_LDS, HINT>(p); }

// the same for one of several residual streams (in-place calls): blockIdx.y is the layer
template <int NB, bool ODD>
__global__ __launch_bounds__(F32_WAVES * 64) void f32_tile_layers_kernel(ApplyArgs p)
{
    select_layer(p);
    f32_tile_body<NB, true, ODD, ODD && NB <= 2, true>(p);
}

}  // namespace preft
