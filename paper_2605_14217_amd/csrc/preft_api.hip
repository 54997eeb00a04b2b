// C ABI of the adapter-apply library: argument validation, variant choice, launches.
// See include/preft.h for the contract of every entry point.
#include "../../include/preft.h"

#include "common.hpp"
#include "dispatch.hpp"
#include "expand_kernel.hpp"
#include "f32_kernel.hpp"
#include "mfma_kernel.hpp"
#include "mfma_wide_kernel.hpp"
#include "row_kernel.hpp"
#include "schedule.hpp"
#include "small_kernel.hpp"
#include "valu_kernel.hpp"
// most kernel instantiations are compiled in instances/group_*.hip (see gen_instances.py), in parallel
#ifndef PREFT_NO_EXTERN_KERNELS
#include "instances/extern_kernels.inc"
#endif

#include <mutex>

static_assert(preft::PREFT_MAX_RANK_DEV == PREFT_MAX_RANK, "device and public rank limits differ");

// Schedule area of preft_direft_apply_static: device memory that exists without any allocation call.
// Each GPU the library runs on holds its own copy at its own address until the process ends.  In
// host code the name below is only a stand-in for the symbol: the address a kernel can use comes
// from hipGetSymbolAddress (static_scratch_of), once per device.
static __device__ __align__(256) unsigned char scratch[PREFT_STATIC_SCRATCH_BYTES];

namespace {

using namespace preft;

constexpr int MODE_TEST_MASK = 0x7fff0000;
constexpr int MODE_MASK = PREFT_ALL_TOKENS | PREFT_SCHEDULE_READY | MODE_TEST_MASK;

inline Knobs knobs_of(int mode)
{
    Knobs k;
    k.variant   = (mode >> 16) & 7;
    k.waves     = (mode >> 19) & 15;
    k.rowblocks = (mode >> 23) & 3;
    k.colsplit  = (mode >> 25) & 15;
    k.resident  = (mode >> 29) & 3;
    return k;
}
inline bool knobs_valid(const Knobs &k)
{
    if (k.variant > 5) return false;
    if (k.waves != 0 && k.waves != 1 && k.waves != 2 && k.waves != 4 && k.waves != 8) return false;
    if (k.rowblocks > 2) return false;
    return true;
}

inline bool aligned16(const void *p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

size_t workspace_bytes(int64_t T, int64_t S)
{
    return (size_t)HEADER_INTS * 4 + (size_t)chunk_capacity(T, S) * sizeof(int4) +
           (size_t)short_capacity(T, S) * (sizeof(int4) + sizeof(int2));
}

// z area (LoRA calls whose sweeps run as two launches): after the schedule, the pieces of every 16-row block of a chunk
size_t z_offset(int64_t T, int64_t S) { return (workspace_bytes(T, S) + 255) & ~(size_t)255; }
size_t z_bytes(int64_t T, int64_t S, int rank, int n_proj)
{
    return (size_t)z_piece(chunk_capacity(T, S) * (CHUNK_ROWS / 16), n_proj, 0, z_rank_blocks(rank), 0) * 16;
}

ScheduleView view_of(void *workspace, int64_t T, int64_t S)
{
    ScheduleView v;
    char *base = reinterpret_cast<char *>(workspace);
    v.header = reinterpret_cast<int32_t *>(base);
    v.chunks = reinterpret_cast<int4 *>(base + HEADER_INTS * 4);
    v.chunk_cap = (int32_t)chunk_capacity(T, S);
    v.short_cap = (int32_t)short_capacity(T, S);
    char *after_chunks = base + HEADER_INTS * 4 + (size_t)v.chunk_cap * sizeof(int4);
    v.gtiles = reinterpret_cast<int4 *>(after_chunks);                  // 16-byte aligned
    v.shorts = reinterpret_cast<int2 *>(after_chunks + (size_t)v.short_cap * sizeof(int4));
    return v;
}

// Device address of this GPU's copy of `scratch` (looked up on the first call per device, with that
// device current; no allocation).
constexpr int MAX_DEVICES = 64;
std::mutex g_scratch_mutex;
void *g_scratch_ptr[MAX_DEVICES] = {};

int static_scratch_of(void **out)
{
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= MAX_DEVICES) return PREFT_EHIP;
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    if (!g_scratch_ptr[dev]) {
        void *ptr = nullptr;
        if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess || !ptr) return PREFT_EHIP;
        g_scratch_ptr[dev] = ptr;
    }
    *out = g_scratch_ptr[dev];
    return PREFT_OK;
}

int check_launch()
{
    return hipGetLastError() == hipSuccess ? PREFT_OK : PREFT_EHIP;
}

int check_tables(const void *workspace, size_t bytes, const int32_t *seg_start, const int32_t *seg_adapter,
                 const int32_t *seg_prefill_len, int32_t S, int32_t T, int32_t N, int mode)
{
    if (T < 0 || S < 0 || N < 0) return PREFT_EINVAL;
    if ((mode & ~MODE_MASK) != 0 || !knobs_valid(knobs_of(mode))) return PREFT_EINVAL;
    if (T == 0 || S == 0) return PREFT_OK;
    if (!seg_start || !seg_adapter || !seg_prefill_len) return PREFT_EINVAL;
    if (!workspace || !aligned16(workspace) || bytes < workspace_bytes(T, S)) return PREFT_EWORKSPACE;
    return PREFT_OK;
}

int launch_schedule(void *workspace, const int32_t *seg_start, const int32_t *seg_adapter,
                    const int32_t *seg_prefill_len, int32_t S, int32_t T, int32_t N, int mode,
                    hipStream_t stream)
{
    ScheduleView v = view_of(workspace, T, S);
    hipLaunchKernelGGL(schedule_kernel, dim3(1), dim3(sched_threads(S, N)), 0, stream, seg_start, seg_adapter,
                       seg_prefill_len, S, T, N, (mode & PREFT_ALL_TOKENS) ? 1 : 0, v);
    return check_launch();
}

// ------------------------------------------------------------------------------------
// tile-kernel dispatch
// ------------------------------------------------------------------------------------
template <int NB, bool DIREFT, bool ODD, int RK = 0>
void launch_small_shape(ApplyArgs a, int64_t S, int n_slices, const Knobs &k, hipStream_t stream)
{
    const unsigned tiles = likely_units(a, S);                // a multiple of 8 (col_split is 1 here)
    if constexpr (DIREFT) {
        const bool few = small_in_place_few(a, S);
        void (*kernel)(ApplyArgs, SmallLaunch) = few ? small_tile_kernel<NB, true, ODD, true, SMALL_WAVES, true, RK> : small_tile_kernel<NB, true, ODD, true, SMALL_WAVES, false, RK>;
        if (a.h_layers) kernel = few ? small_tile_layers_kernel<NB, ODD, true, RK> : small_tile_layers_kernel<NB, ODD, false, RK>;
        hipLaunchKernelGGL(kernel, dim3(tiles, a.n_layers), dim3(SMALL_WAVES * 64), 0, stream, a, SmallLaunch{1, 0});
    } else {
        const SmallShape shape = small_shape(a, S, n_slices, k);
        const int cols = 128 * shape.units;
        auto shares_of = [&](int d) { return (d + cols - 1) / cols; };
        const SmallLaunch l = {shares_of(a.d_out), n_slices > 1 ? shares_of(a.more[0].d_out) : 0};
        const int shares = l.shares0 + l.shares1 + (n_slices > 2 ? shares_of(a.more[1].d_out) : 0);     // small_shape: 1536 at most
        a.col_split = shape.units;
        auto pick = [&](auto few_tag) {
            constexpr bool FEW = decltype(few_tag)::value;
            void (*kernel)(ApplyArgs, SmallLaunch) = small_tile_kernel<NB, false, ODD, true, SMALL_WAVES, FEW, RK>;
            if constexpr (NB == 2 && !ODD && RK != 20 && RK != 28) { if (shape.units < SMALL_WAVES) kernel = small_tile_kernel<NB, false, ODD, true, SMALL_WAVES, FEW, RK, false>; }
            if constexpr (NB == 1) { if (!shape.deep) kernel = small_tile_kernel<NB, false, ODD, false, SMALL_WAVES, FEW, RK>; }
            if constexpr (NB > 2) { if (shape.waves == 4) kernel = small_tile_kernel<NB, false, ODD, true, 4, FEW>; }
            return kernel;
        };
        void (*kernel)(ApplyArgs, SmallLaunch) = small_few(a, S) ? pick(std::true_type{}) : pick(std::false_type{});
        const unsigned slots = tiles / 8 < 65535 ? tiles / 8 : 65535;
        hipLaunchKernelGGL(kernel, dim3((unsigned)shares * 8, slots), dim3(shape.waves * 64), 0, stream, a, l);
    }
}

// ranks 1..128, in place 1..64
template <bool DIREFT>
void launch_small(const ApplyArgs &a, int64_t S, int n_slices, const Knobs &k, hipStream_t stream)
{
    auto launch = [&](auto odd_tag) {
        constexpr bool ODD = decltype(odd_tag)::value;
        if (a.rank <= 8)       launch_small_shape<1, DIREFT, ODD, 8>(a, S, n_slices, k, stream);
        else if (a.rank <= 16) launch_small_shape<1, DIREFT, ODD>(a, S, n_slices, k, stream);
        else if (a.rank == 20) launch_small_shape<2, DIREFT, false, 20>(a, S, n_slices, k, stream);
        else if (a.rank == 24) launch_small_shape<2, DIREFT, false, 24>(a, S, n_slices, k, stream);
        else if (a.rank == 28) launch_small_shape<2, DIREFT, false, 28>(a, S, n_slices, k, stream);
        else if (a.rank <= 32) launch_small_shape<2, DIREFT, ODD>(a, S, n_slices, k, stream);
        else if (a.rank <= 64) launch_small_shape<4, DIREFT, ODD>(a, S, n_slices, k, stream);
        else                   launch_small_shape<8, DIREFT, ODD>(a, S, n_slices, k, stream);
    };
    if (a.rank == 1)       launch_small_shape<1, DIREFT, false, 1>(a, S, n_slices, k, stream);
    else if (a.rank == 2)  launch_small_shape<1, DIREFT, false, 2>(a, S, n_slices, k, stream);
    else if (a.rank == 3)  launch_small_shape<1, DIREFT, false, 3>(a, S, n_slices, k, stream);
    else if (a.rank == 4)  launch_small_shape<1, DIREFT, false, 4>(a, S, n_slices, k, stream);
    else if (a.rank % 4)   launch(std::integral_constant<bool, true>{});
    else                   launch(std::integral_constant<bool, false>{});
}

// the row-split kernel takes whole chunks only
inline unsigned chunk_grid(const ApplyArgs &a, int64_t S, int rows)
{
    const int64_t units = chunk_capacity(a.T, S) * (CHUNK_ROWS / rows);
    return (unsigned)(((units + 7) / 8) * 8);
}

// in place, part of the tile held in registers (HUNITS units of each wavefront), the rest streamed twice
template <int NB, int MB, int WAVES, int HUNITS>
void launch_mfma_partial(const ApplyArgs &a, int64_t S, hipStream_t stream)
{
    void (*kernel)(ApplyArgs) = mfma_tile_kernel<NB, MB, WAVES, HUNITS, true, 1, true>;
    if (a.h_layers) kernel = mfma_tile_layers_kernel<NB, MB, WAVES, HUNITS, true>;
    hipLaunchKernelGGL(kernel, dim3(tile_grid(a, S, 16 * MB), a.n_layers), dim3(WAVES * 64), 0, stream, a);
}

template <int NB, int MB, int WAVES, int HUNITS, bool DIREFT>
void launch_mfma(const ApplyArgs &a, int64_t S, hipStream_t stream)
{
    constexpr int R = 16 * MB;
    void (*kernel)(ApplyArgs) = mfma_tile_kernel<NB, MB, WAVES, HUNITS, DIREFT>;
    if constexpr (NB > 1 && !DIREFT) {
        if (activations_stay(a, S, a.d_out, 2, STAY_BF16)) kernel = mfma_tile_kernel<NB, MB, WAVES, HUNITS, DIREFT, 1, false, 0, false, false>;
    }
    if constexpr (DIREFT) {
        if (a.h_layers) kernel = mfma_tile_layers_kernel<NB, MB, WAVES, HUNITS>;
    }
    hipLaunchKernelGGL(kernel, dim3(tile_grid(a, S, R), a.n_layers), dim3(WAVES * 64), 0, stream, a);
}

// streaming variant (activations read in both sweeps): LoRA, and DiReFT rows too wide to hold
template <int NB, bool DIREFT>
void launch_mfma_stream(const ApplyArgs &a, int64_t S, int mb, int waves, hipStream_t stream)
{
    if constexpr (NB < 2) {                                // register budget
        if (waves == 8) {
            launch_mfma<NB, 1, 8, 0, DIREFT>(a, S, stream);
            return;
        }
    }
    if constexpr (NB < 8) {
        if (mb == 2) {
            launch_mfma<NB, 2, 4, 0, DIREFT>(a, S, stream);
            return;
        }
    }
    launch_mfma<NB, 1, 4, 0, DIREFT>(a, S, stream);
}

// DiReFT with the tile held in registers between the sweeps (rank <= 16): 8 wavefronts, HUNITS
// units of 128 columns each (register budget: 16 VGPRs per unit).  From rank 32 up the factor
// sweeps of a 16-row tile outweigh its activations and the register file has no room left to
// run them ahead, so those ranks take 32-row tiles (rank 32) or the row-split kernel (rank >= 64).
template <int NB>
bool launch_mfma_resident(const ApplyArgs &a, int64_t S, hipStream_t stream)
{
    if constexpr (NB > 1) {
        return false;
    } else {
        const int units = ((a.d_in >> 7) + 7) / 8;        // whole units per wavefront
        if (units <= 4) {
            launch_mfma<NB, 1, 8, 4, true>(a, S, stream);
            return true;
        }
        if (units <= 8) {
            launch_mfma<NB, 1, 8, 8, true>(a, S, stream);
            return true;
        }
        return false;
    }
}

// row-split kernel with the factors shared through LDS (rank >= 32, widths multiples of 128):
// `rw` row blocks of 16 `mb` rows x `cw` column groups of wavefronts per workgroup
template <int NB, int MB, int RW, int CW, bool DIREFT, bool ODD = false>
void launch_wide_shape(const ApplyArgs &a, int64_t S, hipStream_t stream)
{
    void (*kernel)(ApplyArgs) = mfma_wide_kernel<NB, MB, RW, CW, DIREFT, 1, false, ODD>;
    if constexpr (DIREFT) { if (a.h_layers) kernel = mfma_wide_layers_kernel<NB, MB, RW, CW, ODD>; }   // set on in-place calls only
    hipLaunchKernelGGL(kernel, dim3(chunk_grid(a, S, 16 * MB * RW), a.n_layers), dim3(RW * CW * 64), 0, stream, a);
}

// Columns of outputs whose rows do not start on 128-byte lines: neighbouring panels of those share lines.
int64_t columns_off_lines(const ApplyArgs &a, int n_slices)
{
    int64_t off = shares_lines(a.y, a.ldy * 2) ? a.d_out : 0;
    for (int i = 1; i < n_slices; ++i) off += shares_lines(a.more[i - 1].y, a.more[i - 1].ldy * 2) ? a.more[i - 1].d_out : 0;
    return off;
}
int64_t out_width(const ApplyArgs &a, int n_slices)
{
    int64_t width = a.d_out;
    for (int i = 1; i < n_slices; ++i) width += a.more[i - 1].d_out;
    return width;
}
bool rows_off_lines(const ApplyArgs &a, int n_slices) { return columns_off_lines(a, n_slices) > 0; }

// the row-split kernel's shrink launch, above rank 16, keeps byte offsets within a 64-row tile of x and within a factor in 32 bits
inline bool offsets_fit(const ApplyArgs &a) { return a.rank <= 16 || (a.ldx <= (1 << 22) && a.d_in <= (1 << 22)); }

// a workgroup of four wavefronts for every tile of `height` rows x `cols` columns
void launch_expand_kernel(void (*kernel)(ApplyArgs, int), ApplyArgs a, int64_t S, int n_slices, hipStream_t stream,
                          int height = 16 * EXPAND_MB, int cols = EXPAND_WAVES * 128, int threads = EXPAND_WAVES * 64)
{
    // Panels that share lines go to one XCD, from an eighth of the columns on (rank 8, 5000 rows, 1024 -> 5336, runs / memory order 26.3 / 29.4 us, 8192 on lines and
    // 2056 off 42.8 / 45.2, 8192 + 14336 on and 616 off 104 / 98, 2500 rows 58.5 / 52.0)
    int64_t all = a.d_out;
    for (int i = 1; i < n_slices; ++i) all += a.more[i - 1].d_out;
    a.xcd_runs = 8 * columns_off_lines(a, n_slices) >= all;
    // More tiles than the likely rows fill are likely to be empty, and an empty workgroup is not free (3584 decode rows, prompt
    // positions, 8192 -> 2 x 28672: 22 848 of them 23 us): the kernel strides over what exceeds the grid (and over what would
    // exceed the 2^32 work items of a launch)
    const int64_t rows = a.all_tokens && !a.chunks_only ? a.T : prompt_rows(a, S);
    const int64_t bound = tile_grid(a, S, height), likely = rows / height * 5 / 4 + (rows / 8 < 64 ? rows / 8 + 1 : 64) + (a.chunks_only ? 0 : likely_gathered(a, S));
    const int64_t grid = (bound < likely ? bound : likely) * expand_panels(a, n_slices, cols), most = (int64_t)1 << 23;
    hipLaunchKernelGGL(kernel, dim3((unsigned)(grid < most ? grid : most)), dim3(threads), 0, stream, a, n_slices);
}

template <int NB, bool ODD>
void launch_expand(const ApplyArgs &a, int64_t S, int n_slices, hipStream_t stream)
{
    const bool stay = a.x == a.y ? h_stays(a) : activations_stay(a, S, out_width(a, n_slices), 2, STAY_BF16);
    if constexpr (NB <= 2) {
        void (*kernel)(ApplyArgs, int) = mfma_expand_kernel<NB, EXPAND_MB, ODD, YHint::All>;
        if (stay) kernel = mfma_expand_kernel<NB, EXPAND_MB, ODD, YHint::None>;
        else if constexpr (NB == 1) {                              // (above rank 16 rows are off lines by their pitch only)
            int64_t on = a.d_out;
            for (int i = 1; i < n_slices; ++i) on += a.more[i - 1].d_out;
            const int64_t off = columns_off_lines(a, n_slices);
            on -= off;
            if (off > 0) kernel = on > 0 ? mfma_expand_kernel<NB, EXPAND_MB, ODD, YHint::ByOutput> : mfma_expand_kernel<NB, EXPAND_MB, ODD, YHint::None>;
        }
        launch_expand_kernel(kernel, a, S, n_slices, stream);
    } else {
        const int pu = panel_units(a, n_slices);
        void (*kernel)(ApplyArgs, int) = stay ? panel_expand_kernel<NB, PANEL_RW, 1, ODD, false, false> : panel_expand_kernel<NB, PANEL_RW, 1, ODD>;
        if constexpr (NB == 4) {
            if (pu == 2) kernel = stay ? panel_expand_kernel<NB, PANEL_RW, 2, ODD, false, false> : panel_expand_kernel<NB, PANEL_RW, 2, ODD>;
        }
        launch_expand_kernel(kernel, a, S, n_slices, stream, 16 * PANEL_RW, 128 * pu, 64 * PANEL_RW);
    }
}

// LoRA with a z area in the workspace: the shrink sweep leaves z there and the expand runs as a launch of its
// own (mfma_expand_kernel).  Measured on the same buffers, one launch -> two, prompts of about 700 rows:
//   rank 16, 4096 -> 2 x 14336: 1100 rows 67 -> 36 us, 8000 rows 247 -> 181, 37 000 rows 909 -> 789; 4096 -> 4096:
//     15.3 -> 15.5, 48.6 -> 46.2, 167 -> 159; 500 rows (against four workgroups per tile): 10.9 -> 13.2;
//     1024 -> 2728 (rows off 128-byte lines): 2000 rows 11.3 -> 13.6, 37 000 rows 114 -> 120; 2000 -> 3208:
//     15.0 -> 14.4, 154 -> 148.  Ranks 4-15 alike.
//   rank 1-3 (vector-ALU kernels), 4096 -> 4096: 1500 rows 13-15 -> 14-16, 11 300 rows 52 -> 52, 42 000 rows 190 -> 170;
//     4096 -> 2 x 14336: 1500 rows 62-82 -> 39-44, 42 000 rows 1030 -> 864; q+k+v of 8192, 350 000 rows 3556-3676 -> 3218-3407;
//     1024 -> 1024 + 2 x 512, 140 000 rows 258-265 -> 255-293; rows off 128-byte lines, 1024 -> 2728 10-11 -> 12-13,
//     2000 -> 3208, 11 200 rows 42-44 -> 50, but several outputs off lines, 4096 -> 9640 + 296, 1500 rows 26 -> 18.
//   rank 64, 8192 -> 8192: 1100 rows 167 -> 81 us, 8000 rows 182 -> 136, 37 000 rows 522 -> 387; rank 32 86 -> 48,
//     105 -> 97, 355 -> 372.
//   decode rows alone, 7 per adapter (gathered tiles), rank 16, 8192 -> 8192: 1200 rows 30 -> 35, 3584 rows 89 -> 89;
//     one per adapter 87 -> 109.
// Hence: above 1024 rows; up to rank 16 where the outputs are worth a second launch, and not for all-position
// batches of mostly single rows.  PREFT_TEST_RESIDENT(1) takes this form wherever it exists, PREFT_TEST_VARIANT(5) never.
bool wants_split(const ApplyArgs &a, int64_t S, int n_slices, const Knobs &k)
{
    if (!a.zws || (k.variant != 0 && k.variant != 4) || k.waves || k.rowblocks || k.colsplit) return false;
    if (!expand_ids_fit(a, S, n_slices) || !offsets_fit(a)) return false;
    if (k.resident == 1) return true;
    if (a.T <= 1024) return false;
    // hardly a prompt row, and none of the others counts, or the second launch does not take them: nothing to expand
    if ((!a.all_tokens || a.rank > 16) && prompt_rows(a, S) < 64) return false;
    int64_t width = a.d_out;
    for (int i = 1; i < n_slices; ++i) width += a.more[i - 1].d_out;
    // Rank 64, 89 740 rows, one launch -> two: 8192 -> 2 x 28672 4845 -> 4200, 8192 -> 8192 946 -> 845, q+k+v 1322 -> 1248, 28672 -> 8192 1716 ->
    // 1602, rank 63 q+k+v 1355 -> 1282; 352 814 rows, q+k+v 5100 -> 5000.  But 8192 -> 1024 376 -> 392: next to nothing to expand, and the single
    // launch has tiles enough.
    if (a.rank > 32 && a.T > 49152 && 4 * width <= a.d_in) return false;
    // Above rank 64 z is as many bytes as 256 columns of y, written once and read by every panel: that pays where the columns are many (the workgroups of the single launch, 128 rows each, leave the chip
    // idle and repeat nothing).  Two launches / one over random calls above 4096 rows, geometric mean by columns: up to 512 0.90 (22 of 107 slower, up to 1.9: rank 96, 128 -> 128, 9800 rows 20.4 /
    // 10.7), 513 to 1024 0.83 (11 of 48, up to 1.3; none of those of d_in >= 2048, up to 16384 rows and 64 rows a segment), 0.64, 0.54, 0.43 above.
    if (a.rank > 64 && width <= 1024) return a.d_in >= 2048 && width > 512 && a.T <= 16384 && a.T >= 64 * S;
    if (a.rank > 16) return true;
    if (a.all_tokens && a.T < 8 * S) return false;
    if (a.rank < 4) return a.T * width >= (n_slices > 1 ? 6000000 : 12000000) && width >= 3072 && (n_slices > 1 || !rows_off_lines(a, n_slices));
    return a.T * width >= 6000000 && (width >= 3072 || !rows_off_lines(a, n_slices));
}

// The in-place call above rank 32 as two launches of the row-split order.  The single launch reads h twice as well, in 64-row tiles that sweep all columns; narrow
// rows find part of the second read in the caches, as long as the batch fills the chip.  Rank 64, one launch -> two, us: 89 740 rows,
// d = 512 / 1024 / 2048 / 3072 / 4096 / 8192 / 14336: 56 -> 79, 110 -> 131, 234 -> 241, 338 -> 337, 447 -> 433, 878 -> 828, 1620 -> 1446; 23 000 rows, d = 2048
// 61 -> 69, 3072 90 -> 95, 4096 132 -> 115; 7000 rows, 512 14.8 -> 15.8, 1024 25 -> 23, 2048 45 -> 38, 4096 (10 prompts) 89 -> 56; 2500 rows, 1024 22 -> 18,
// 8192 155 -> 81.
bool wants_split_in_place(const ApplyArgs &a, int64_t S, const Knobs &k)
{
    if (!a.zws || a.h_layers || (k.variant != 0 && k.variant != 4) || k.waves || k.rowblocks || k.colsplit) return false;
    if (!expand_ids_fit(a, S, 1) || !offsets_fit(a)) return false;
    if (k.resident == 1) return true;
    if (a.T <= 1024 || prompt_rows(a, S) < 64) return false;
    // above rank 64, rank 96, one launch / two: 24 000 rows, d = 512 28.8 / 34, 2048 83 / 80, 4096 173 / 144; 26 600 rows, d = 1024 46 / 54; 12 000 rows, d = 512 27.0 / 25.0, 2048 79 / 51; rank 128,
    // d = 128, 4600 rows 11.1 / 14.2; in segments of 50 to 70 rows, 512, 8600 rows 42.5 / 47.8, 1024, 13 200 46.5 / 51.0
    if (a.rank > 64) return a.d_in >= 2048 || (a.d_in >= 512 && a.T <= 14336 && a.T >= 72 * S);
    return a.d_in >= 4096 || (a.d_in >= 1024 && a.T <= 8192);
}

// Whether the row-split kernel's single launch runs with two column groups at rank 17-32: every width a multiple of 256.
bool column_groups_fit(const ApplyArgs &a, int n_slices)
{
    bool fit = wide_widths_ok(a, 2);
    for (int i = 1; i < n_slices; ++i) fit = fit && (a.more[i - 1].d_out % 256) == 0;
    return fit;
}

// The row-split kernel's shrink launch, above rank 16: tiles of 64 rows, or, at rank 33-64 of several outputs or of the largest calls (above rank 64: see below), of 128, whose eight
// wavefronts share a step's factors: half the factor traffic, half as many workgroups (and with three outputs the four-wavefront form spills).
// 64 / 128 rows, whole calls, us: three outputs, 8192 -> 8192 + 2 x 1024, 89 740 rows 1270 / 1124, 4096 -> 4096 + 2 x 1024, 2500 rows 89 / 78, 9500
// rows 119 / 108; two, 8192 -> 2 x 28672, 89 740 rows 4120 / 4067, 4096 -> 2 x 14336, 23 000 rows 525 / 519, 9500 rows 223 / 233; one,
// 89 740 rows, 28672 -> 8192 1603 / 1503, 8192 -> 8192 836 / 835, in place 828 / 837, 37 000 rows, 4096 -> 4096 182 / 200.  Rank 32: 14336 -> 4096,
// 37 000 rows 307 / 332.
template <int NB, int SLICES, bool DIREFT>
void launch_wide_shrink(const ApplyArgs &a, int64_t S, hipStream_t stream)
{
    constexpr int RW = NB == 4 && SLICES == 3 ? 8 : 4;
    const bool stay = DIREFT && h_stays(a);
    void (*kernel)(ApplyArgs) = mfma_wide_kernel<NB, 1, RW, 1, DIREFT, SLICES, true>;
    if constexpr (NB <= 4) { if (a.rank % 4) kernel = mfma_wide_kernel<NB, 1, RW, 1, DIREFT, SLICES, true, true>; }
    if constexpr (DIREFT) {
        if (stay) kernel = mfma_wide_kernel<NB, 1, RW, 1, true, 1, true, false, false, false>;
        if constexpr (NB <= 4) { if (stay && a.rank % 4) kernel = mfma_wide_kernel<NB, 1, RW, 1, true, 1, true, true, false, false>; }
    }
    int waves = RW;
    if constexpr (NB <= 2) {                                // where the single launch sums in two column groups, so does this one
        if (a.rank % 4 == 0 && column_groups_fit(a, SLICES)) kernel = mfma_wide_kernel<NB, 1, 4, 1, DIREFT, SLICES, true, false, true>;
    } else if constexpr (NB == 4 && !DIREFT && SLICES < 3) {
        if (SLICES == 2 ? a.T > 16384 : a.T > 49152 && a.d_in > 8192) {
            kernel = (a.rank % 4) ? mfma_wide_kernel<NB, 1, 8, 1, DIREFT, SLICES, true, true> : mfma_wide_kernel<NB, 1, 8, 1, DIREFT, SLICES, true>;
            waves = 8;
        }
    }
    // Rank 65-128: one workgroup on a compute unit in either form, so 64 rows as long as those are no more than one for each.  One launch (128-row tiles, the expand in the same
    // workgroup) / 64 / 128, whole calls, us: rank 128, 4096 -> 4096, 3600 prompt rows 156 / 57 / 66, 12 000 167 / 89 / 96, 24 000 185 / 167 / 150; rank 96, 8192 -> 8192, 31 500 rows
    // 621 / 418 / 395; in place, d = 4096, 12 000 rows 154 / 91 / 97.
    if constexpr (NB == 8) {
        if (prompt_rows(a, S) / 64 + S / 4 > 256) {
            kernel = mfma_wide_kernel<NB, 1, 8, 1, DIREFT, SLICES, true>;
            if constexpr (DIREFT) { if (stay) kernel = mfma_wide_kernel<NB, 1, 8, 1, true, 1, true, false, false, false>; }
            waves = 8;
        }
    }
    hipLaunchKernelGGL(kernel, dim3(chunk_grid(a, S, 16 * waves)), dim3(64 * waves), 0, stream, a);
}

// above rank 16: the row-split kernel's shrink sweep of the chunks, then their expand launch
template <int NB, int SLICES, bool DIREFT = false>
bool launch_mfma_split(const ApplyArgs &a0, int64_t S, const Knobs &k, hipStream_t stream)
{
    if (!(DIREFT ? wants_split_in_place(a0, S, k) : wants_split(a0, S, SLICES, k)) || (a0.d_in % 128) != 0) return false;
    ApplyArgs a = a0;
    a.chunks_only = 1;
    launch_wide_shrink<NB, SLICES, DIREFT>(a, S, stream);
    if constexpr (NB <= 4) {
        if (a.rank % 4) { launch_expand<NB, true>(a, S, SLICES, stream); return true; }
    }
    launch_expand<NB, false>(a, S, SLICES, stream);
    return true;
}

// Rank 17 and up in multiples of 4, few tiles: the small-batch kernel's shrink sweep, then the expand launch; chunks and gathered tiles alike, any widths
template <bool DIREFT>
void launch_small_split(const ApplyArgs &a, int64_t S, int n_slices, const Knobs &k, hipStream_t stream)
{
    const unsigned tiles = likely_units(a, S), slots = tiles / 8 < 65535 ? tiles / 8 : 65535;
    // two rank blocks a workgroup while that makes no more workgroups than compute units, else up to four, which share the tile's x
    const int blocks = z_rank_blocks(a.rank), most = likely_tiles(a, S) * n_slices * ((blocks + 1) / 2) <= 256 ? 2 : 4, rank_parts = (blocks + most - 1) / most, nb = (blocks + rank_parts - 1) / rank_parts;
    void (*shrink)(ApplyArgs, int) = nb == 4 ? small_shrink_kernel<4, DIREFT> : nb == 3 ? small_shrink_kernel<3, DIREFT> : a.rank <= 24 ? small_shrink_kernel<2, DIREFT, 24> : small_shrink_kernel<2, DIREFT>;
    int waves = SMALL_WAVES;
    if constexpr (!DIREFT) {
        waves = small_shape(a, S, n_slices, k).waves;         // the single launch's: its sums of z are grouped by them
        if (waves == 4) shrink = nb == 4 ? small_shrink_kernel<4, false, 0, 4> : nb == 3 ? small_shrink_kernel<3, false, 0, 4> : small_shrink_kernel<2, false, 0, 4>;
    }
    const bool stay = DIREFT ? h_stays(a) : activations_stay(a, S, out_width(a, n_slices), 2, STAY_BF16);
    hipLaunchKernelGGL(shrink, dim3((unsigned)(n_slices * rank_parts) * 8, slots), dim3(waves * 64), 0, stream, a, n_slices);
    if (a.rank <= 32)
        launch_expand<2, false>(a, S, n_slices, stream);
    else if (a.rank <= 64)
        launch_expand_kernel(stay ? panel_expand_kernel<4, PANEL_RW, 2, false, true, false> : panel_expand_kernel<4, PANEL_RW, 2, false, true>, a, S, n_slices, stream, 16 * PANEL_RW, 256,
                             64 * PANEL_RW);
    else
        launch_expand_kernel(stay ? panel_expand_kernel<8, PANEL_RW, 1, false, true, false> : panel_expand_kernel<8, PANEL_RW, 1, false, true>, a, S, n_slices, stream, 16 * PANEL_RW, 128,
                             64 * PANEL_RW);
}

// A call that the small-batch kernel takes: in one launch, or in two where that is faster and the workspace has room for z; the same sums in the same
// order either way
template <bool DIREFT>
void launch_small_order(const ApplyArgs &a, int64_t S, int n_slices, const Knobs &k, hipStream_t stream)
{
    int64_t width = a.d_out;
    for (int i = 1; i < n_slices; ++i) width += a.more[i - 1].d_out;
    const int cols = a.rank <= 32 ? EXPAND_WAVES * 128 : a.rank <= 64 ? 256 : 128, height = a.rank <= 32 ? 16 * EXPAND_MB : 16 * PANEL_RW;
    const bool ids_fit = tile_grid(a, S, height) * expand_panels(a, n_slices, cols) < ((int64_t)1 << 31);
    if (a.zws && !a.h_layers && ids_fit && small_in_two(a, S, width, DIREFT, k)) launch_small_split<DIREFT>(a, S, n_slices, k, stream);
    else launch_small<DIREFT>(a, S, n_slices, k, stream);
}

// rank 4..16: the column-split kernel's shrink sweep, then the expand launch; chunks and gathered tiles alike
template <int SLICES>
bool launch_mfma_split16(const ApplyArgs &a, int64_t S, const Knobs &k, hipStream_t stream)
{
    constexpr int WAVES = SLICES == 3 ? 4 : 8;
    if (!wants_split(a, S, SLICES, k)) return false;
    if (a.rank % 4) {
        hipLaunchKernelGGL((mfma_tile_kernel<1, 1, WAVES, 0, false, SLICES, false, 2, true>), dim3(tile_grid(a, S, 16)),
                           dim3(WAVES * 64), 0, stream, a);
        launch_expand<1, true>(a, S, SLICES, stream);
        return true;
    }
    hipLaunchKernelGGL((mfma_tile_kernel<1, 1, WAVES, 0, false, SLICES, false, 0, true>), dim3(tile_grid(a, S, 16)),
                       dim3(WAVES * 64), 0, stream, a);
    launch_expand<1, false>(a, S, SLICES, stream);
    return true;
}

// rank 1..3: the vector-ALU kernel's shrink sweep and the expand launch that goes with it
template <int RANK, int SLICES>
void launch_valu_split_rank(const ApplyArgs &a, int64_t S, hipStream_t stream)
{
    hipLaunchKernelGGL((valu_tile_kernel<RANK, 4, 4, false, SLICES, 0, true>), dim3(tile_grid(a, S, 16)), dim3(256), 0, stream, a);
    launch_expand_kernel(thin_expand_kernel<RANK, EXPAND_MB>, a, S, SLICES, stream);
}

template <int SLICES>
bool launch_valu_split(const ApplyArgs &a, int64_t S, const Knobs &k, hipStream_t stream)
{
    if (k.variant != 0 || !wants_split(a, S, SLICES, k)) return false;
    if (a.rank == 1)      launch_valu_split_rank<1, SLICES>(a, S, stream);
    else if (a.rank == 2) launch_valu_split_rank<2, SLICES>(a, S, stream);
    else                  launch_valu_split_rank<3, SLICES>(a, S, stream);
    return true;
}

template <int NB, bool DIREFT>
bool launch_mfma_wide(const ApplyArgs &a, int64_t S, int mb, int waves, int cw, const Knobs &k, hipStream_t stream)
{
    if (NB < 2 && k.variant != 4) return false;               // rank <= 16: only on request
    if (!wide_widths_ok(a, 1)) return false;
    if constexpr (NB >= 4 || (NB == 2 && !DIREFT)) {
        if (launch_mfma_split<NB, 1, DIREFT>(a, S, k, stream)) return true;
    }
    if (!wide_widths_ok(a, cw)) cw = 1;
    if (mb != 1 && NB <= 4) {                                  // 4 wavefronts x 32 rows
        if constexpr (NB <= 4) launch_wide_shape<NB, 2, 4, 1, DIREFT>(a, S, stream);
        return true;
    }
    if (cw >= 2 && NB <= 4) {                                  // 2 column groups: 8 wavefronts on 64 rows
        if constexpr (NB <= 4) launch_wide_shape<NB, 1, 4, 2, DIREFT>(a, S, stream);
        return true;
    }
    if (waves == 8) launch_wide_shape<NB, 1, 8, 1, DIREFT>(a, S, stream);
    else            launch_wide_shape<NB, 1, 4, 1, DIREFT>(a, S, stream);
    return true;
}

// ranks above 16 that are no multiple of 4: the column-split kernel, 4 wavefronts on 16 rows (`mb` 2: 32, rank 17-32)
template <int NB, bool DIREFT>
void launch_mfma_odd_stream(const ApplyArgs &a, int64_t S, int mb, hipStream_t stream)
{
    const bool stay = !DIREFT && activations_stay(a, S, a.d_out, 2, STAY_BF16);
    void (*kernel)(ApplyArgs) = mfma_tile_kernel<NB, 1, 4, 0, DIREFT, 1, false, 1>;
    if constexpr (!DIREFT) { if (stay) kernel = mfma_tile_kernel<NB, 1, 4, 0, DIREFT, 1, false, 1, false, false>; }
    if constexpr (DIREFT) { if (a.h_layers) kernel = mfma_tile_layers_kernel<NB, 1, 4, 0, false, 1>; }
    int rows = 16;
    if constexpr (NB == 2) {
        if (mb == 2) {
            rows = 32;
            kernel = mfma_tile_kernel<NB, 2, 4, 0, DIREFT, 1, false, 1>;
            if constexpr (!DIREFT) { if (stay) kernel = mfma_tile_kernel<NB, 2, 4, 0, DIREFT, 1, false, 1, false, false>; }
            if constexpr (DIREFT) { if (a.h_layers) kernel = mfma_tile_layers_kernel<NB, 2, 4, 0, false, 1>; }
        }
    }
    hipLaunchKernelGGL(kernel, dim3(tile_grid(a, S, rows), a.n_layers), dim3(256), 0, stream, a);
}

template <typename E, bool DIREFT>
void launch_rows(const ApplyArgs &a, int64_t S, bool chunks_too, hipStream_t stream);

// The gathered tiles (16 rows of an adapter) of a call whose chunks the row-split kernel takes, which shares an adapter's factors among
// the 128 rows of a chunk.  A few of them go to the small-batch kernel, whose workgroups share a tile's columns (4096 -> 4096, rank 64, 7500 prompt rows
// beside 50 decode rows 98 -> 94 us; prompt positions only, an empty launch); many to 16-row tiles of the column-split kernel, an output in each plane of the grid, which
// run the shrink once (1024 -> 4096 + 2 x 1024, rank 48, 3000 decode rows of 200 adapters 59 us, 74 there); what neither reaches with 32-bit offsets to
// the per-row kernel.
template <int NB, bool DIREFT>
void launch_gathered(ApplyArgs a, int64_t S, int n_slices, hipStream_t stream)
{
    a.gathered_only = 1;
    int widest = a.d_out;
    for (int i = 1; i < n_slices; ++i) widest = a.more[i - 1].d_out > widest ? a.more[i - 1].d_out : widest;
    // In place the layers of a call multiply the tiles, and each has the bits of its one-layer call: a quarter as many (4 layers, rank 48, 1120 decode rows of 32 adapters, d = 512 / 1024 / 4096, column-split / this
    // 12.6 / 15.9, 17.9 / 20.9, 48.9 / 53.7 us).
    if (likely_gathered(a, S) <= (DIREFT ? 32 : 128) && a.d_in <= SMALL_WIDTH && widest <= SMALL_WIDTH) {
        launch_small<DIREFT>(a, S, n_slices, Knobs{}, stream);
        return;
    }
    auto output = [&](int i) {
        if (i > 0) {
            a.y = a.more[i - 1].y; a.ldy = a.more[i - 1].ldy; a.d_out = a.more[i - 1].d_out;
            a.A_pool = a.more[i - 1].A_pool; a.Bt_pool = a.more[i - 1].Bt_pool;
        }
    };
    if (!column_split_fits(a)) {
        for (int i = 0; i < n_slices; ++i) { output(i); launch_rows<bf16_tag, DIREFT>(a, S, false, stream); }
        return;
    }
    if constexpr (!DIREFT && (NB == 2 || NB == 4)) {
        if (n_slices > 1) {
            void (*kernel)(ApplyArgs) = a.rank % 4 ? mfma_tile_outputs_kernel<NB, 4, 1> : mfma_tile_outputs_kernel<NB, 4, 0>;
            hipLaunchKernelGGL(kernel, dim3(tile_grid(a, S, 16), n_slices), dim3(256), 0, stream, a);
            return;
        }
    }
    if constexpr (NB > 1) {
        if (a.rank % 4) { launch_mfma_odd_stream<NB, DIREFT>(a, S, 1, stream); return; }
    }
    launch_mfma_stream<NB, DIREFT>(a, S, 1, NB >= 2 ? 4 : 8, stream);
}

template <int NB, bool DIREFT>
void launch_mfma_nb(const ApplyArgs &a, int64_t S, const Knobs &k, hipStream_t stream)
{
    // rank >= 32: the factors outweigh a 16-row tile's activations, so more rows share them: the
    // row-split kernel.  Up to rank 64 with 4 wavefronts x 16 rows (two or three independent
    // workgroups per compute unit and twice the tiles: measured 3-10 points ahead of 8 wavefronts on
    // the 8B- and 70B-sized batches); above, 8 wavefronts (4 would leave one workgroup per unit)
    const int wide_mb = k.rowblocks ? k.rowblocks : 1;
    const int wide_waves = k.waves ? (k.waves == 8 ? 8 : 4) : (NB <= 4 ? 4 : 8);
    // Column groups (with test variant 4 the column-split knob names them: 1 or 2).  Two of them at
    // rank 32 (measured: 70B q,k,v,o 64 -> 70-76 % of peak, skewed batch 64-75 -> 78 %); at rank 48-64
    // the two factor units per step leave one workgroup per compute unit and that costs more than the
    // access pattern gains (o 62 -> 64.5 %, but gate+up 69 -> 62.5 %, down 64 -> 59 %).
    const int wide_cw = (k.variant == 4 && k.colsplit) ? k.colsplit : (NB <= 2 ? 2 : 1);
    // column-split kernel.  rank <= 16: 8 wavefronts per 16-row tile; rank 32 (widths the
    // row-split kernel does not take): 32-row tiles of 4 wavefronts
    const int mb = k.rowblocks ? k.rowblocks : (NB == 2 ? 2 : 1);
    const int waves = k.waves ? (k.waves == 8 ? 8 : 4) : (NB == 2 ? 4 : 8);
    if constexpr (DIREFT) {
        if (k.waves == 0 && k.variant != 4 && launch_mfma_resident<NB>(a, S, stream)) return;
        // rank 32: 32-row tiles of the column-split kernel (half the factor traffic per row of a
        // 16-row tile, and the tile's second read mostly still finds it in the memory-side cache)
        // measured ahead of the resident and row-split shapes at d = 4096 and d = 8192
        if constexpr (NB == 2) {
            if (k.waves == 0 && (k.variant == 0 || k.variant == 5) && k.rowblocks == 0 && column_split_fits(a)) {
                if (k.resident == 3 || keeps_units(a, S)) launch_mfma_partial<2, 2, 4, 8>(a, S, stream);
                else                                      launch_mfma<2, 2, 4, 0, true>(a, S, stream);
                return;
            }
        }
    }
    if constexpr (!DIREFT) {
        if constexpr (NB == 1) {
            if (k.variant == 0 && launch_mfma_split16<1>(a, S, k, stream)) return;
        }
    }
    if (k.variant != 3 && launch_mfma_wide<NB, DIREFT>(a, S, wide_mb, wide_waves, wide_cw, k, stream)) {
        launch_gathered<NB, DIREFT>(a, S, 1, stream);
        return;
    }
    launch_mfma_stream<NB, DIREFT>(a, S, mb, waves, stream);
}

// packed projections (LoRA, rank <= 16): one shrink sweep over x, one expand sweep per output.
// PIECES > 0: the any-rank shape (ranks that are not multiples of 4)
template <int SLICES, int PIECES = 0>
void launch_mfma_packed(const ApplyArgs &a, int64_t S, const Knobs &k, hipStream_t stream)
{
    if (k.variant == 0 && launch_mfma_split16<SLICES>(a, S, k, stream)) return;
    // three outputs: 4 wavefronts per tile leave room for two workgroups per compute unit (measured
    // better on small and large batches); two outputs: as for a single projection
    const int waves = k.waves ? (k.waves == 8 ? 8 : 4) : (SLICES == 2 ? 8 : 4);
    if (waves == 8)
        hipLaunchKernelGGL((mfma_tile_kernel<1, 1, 8, 0, false, SLICES, false, PIECES>), dim3(tile_grid(a, S, 16)),
                           dim3(512), 0, stream, a);
    else
        hipLaunchKernelGGL((mfma_tile_kernel<1, 1, 4, 0, false, SLICES, false, PIECES>), dim3(tile_grid(a, S, 16)),
                           dim3(256), 0, stream, a);
}

// packed projections at rank 17..64 (widths multiples of 128): the row-split kernel with one sweep
// over x for all outputs.  It takes the chunks; the gathered tiles (all-token mode: decode rows)
// go to one launch of the column-split kernel, an output in each plane of its grid.  (One launch per output cost 4.7 us each with
// nothing to do: rank 64, 4096 -> 4096 + 2 x 1024, 2500 rows 78 -> 74.5, with 900 decode rows in all-token mode 177 -> 141.)
template <int NB>
void launch_mfma_wide_packed(const ApplyArgs &a, int n_proj, int64_t S, const Knobs &k, hipStream_t stream)
{
    const bool split = n_proj == 2 ? launch_mfma_split<NB, 2>(a, S, k, stream) : launch_mfma_split<NB, 3>(a, S, k, stream);
    const bool odd = (a.rank % 4) != 0;
    // two column groups at rank 32 where every width allows it (see launch_mfma_nb); the any-rank form has the basic shape only
    const bool cw2 = NB <= 2 && !odd && column_groups_fit(a, n_proj);
    if (!split) {
        void (*kernel)(ApplyArgs) = n_proj == 2 ? mfma_wide_kernel<NB, 1, 4, 1, false, 2> : mfma_wide_kernel<NB, 1, 4, 1, false, 3>;
        if constexpr (NB <= 2) {
            if (cw2) kernel = n_proj == 2 ? mfma_wide_kernel<NB, 1, 4, 2, false, 2> : mfma_wide_kernel<NB, 1, 4, 2, false, 3>;
        }
        if (odd) kernel = n_proj == 2 ? mfma_wide_kernel<NB, 1, 4, 1, false, 2, false, true> : mfma_wide_kernel<NB, 1, 4, 1, false, 3, false, true>;
        hipLaunchKernelGGL(kernel, dim3(chunk_grid(a, S, 64)), dim3(cw2 ? 512 : 256), 0, stream, a);
    }
    launch_gathered<NB, false>(a, S, n_proj, stream);
}

// bf16 ranks up to 16 that are not multiples of 4 (5, 6, 7, 9, ...): the column-split kernel's any-rank
// shape, 8 wavefronts per 16-row tile; in place with the tile held in registers where it fits
template <bool DIREFT, int PIECES>
void launch_mfma_odd_pieces(const ApplyArgs &a, int64_t S, hipStream_t stream)
{
    void (*kernel)(ApplyArgs);
    int waves = 8;
    if constexpr (DIREFT) {
        // In place the tile stays in registers where it fits.  Up to 4096 columns: 4 wavefronts of 8
        // units each (the 8-wavefront shape of the other ranks has no registers left for the factor
        // block and spills; measured 58 against 55 % of peak at d = 4096), up to 8192: 8 wavefronts of 8
        const int units = (a.d_in >> 7) + ((a.d_in & 127) ? 1 : 0);
        const bool L = a.h_layers != nullptr;
        if (units <= 32) {
            kernel = L ? mfma_tile_layers_kernel<1, 1, 4, 8, false, PIECES> : mfma_tile_kernel<1, 1, 4, 8, true, 1, false, PIECES>;
            waves = 4;
        } else if (units <= 64) {
            kernel = L ? mfma_tile_layers_kernel<1, 1, 8, 8, false, PIECES> : mfma_tile_kernel<1, 1, 8, 8, true, 1, false, PIECES>;
        } else {
            kernel = L ? mfma_tile_layers_kernel<1, 1, 8, 0, false, PIECES> : mfma_tile_kernel<1, 1, 8, 0, true, 1, false, PIECES>;
        }
    } else {
        kernel = mfma_tile_kernel<1, 1, 8, 0, false, 1, false, PIECES>;
    }
    hipLaunchKernelGGL(kernel, dim3(tile_grid(a, S, 16), a.n_layers), dim3(waves * 64), 0, stream, a);
}

template <bool DIREFT>
void launch_mfma_odd(const ApplyArgs &a, int64_t S, const Knobs &k, hipStream_t stream)
{
    if constexpr (!DIREFT) {
        if (k.variant == 0 && launch_mfma_split16<1>(a, S, k, stream)) return;
    }
    // a unit's [128 columns][rank] block of the expand factor is 16 * rank pieces of 16 bytes: 2 per lane
    // up to rank 8, 4 up to rank 16
    if (a.rank <= 8) launch_mfma_odd_pieces<DIREFT, 2>(a, S, stream);
    else             launch_mfma_odd_pieces<DIREFT, 4>(a, S, stream);
}

// bf16 ranks above 16 that are not multiples of 4.  Widths multiples of 128: the row-split kernel's any-rank form takes the chunks (its
// basic shape: 4 wavefronts x 16 rows, above rank 64 8 x 16), the column-split kernel the gathered tiles (all-token mode: decode
// rows); other widths: the column-split kernel takes all.  (They took the per-row kernels: 30 to 300 times as long.)
template <int NB, bool DIREFT>
void launch_mfma_odd_wide(const ApplyArgs &a, int64_t S, const Knobs &k, hipStream_t stream)
{
    if (odd_streams(a, S, DIREFT, k)) {
        launch_mfma_odd_stream<NB, DIREFT>(a, S, 2, stream);
        return;
    }
    bool split = false;
    if constexpr (NB == 4 || (NB == 2 && !DIREFT)) split = launch_mfma_split<NB, 1, DIREFT>(a, S, k, stream);
    if (!split) launch_wide_shape<NB, 1, NB <= 4 ? 4 : 8, 1, DIREFT, true>(a, S, stream);
    launch_gathered<NB, DIREFT>(a, S, 1, stream);
}

template <bool DIREFT>
void launch_mfma_rank(const ApplyArgs &a, int64_t S, const Knobs &k, hipStream_t stream)
{
    const int nb = (a.rank + 15) / 16;
    if ((a.rank % 4) && a.rank > 16) {
        if (nb <= 2)      launch_mfma_odd_wide<2, DIREFT>(a, S, k, stream);
        else if (nb <= 4) launch_mfma_odd_wide<4, DIREFT>(a, S, k, stream);
        else              launch_mfma_odd_wide<8, DIREFT>(a, S, k, stream);
        return;
    }
    if (a.rank % 4) { launch_mfma_odd<DIREFT>(a, S, k, stream); return; }      // rank <= 16 (choose_path)
    if (nb <= 1)      launch_mfma_nb<1, DIREFT>(a, S, k, stream);
    else if (nb <= 2) launch_mfma_nb<2, DIREFT>(a, S, k, stream);
    else if (nb <= 4) launch_mfma_nb<4, DIREFT>(a, S, k, stream);
    else              launch_mfma_nb<8, DIREFT>(a, S, k, stream);
}

template <int RANK, bool DIREFT>
void launch_valu(const ApplyArgs &a, int64_t S, const Knobs &k, hipStream_t stream)
{
    // in place, rows of at most 4096 elements: 2 rows per wavefront stay in registers between the
    // sweeps, so h is read once (d = 4096: 56-59 -> 62-72 % of peak at rank 1-3).  Wider rows
    // would leave one row per wavefront, and the factors re-read for every row cost more than the
    // second read of h (d = 8192, rank 3: 42 % against 60 %).
    if constexpr (DIREFT) {
        if (k.waves == 0 && k.rowblocks == 0 && a.d_in <= 4096) {
            void (*resident)(ApplyArgs) = valu_tile_kernel<RANK, 2, 4, true, 1, 8>;
            if (a.h_layers) resident = valu_tile_layers_kernel<RANK, 2, 4, 8>;
            hipLaunchKernelGGL(resident, dim3(tile_grid(a, S, 8), a.n_layers), dim3(256), 0, stream, a);
            return;
        }
    }
    constexpr int RB = RANK <= 4 ? 4 : 2;
    int waves = k.waves ? k.waves : 4;
    void (*kernel)(ApplyArgs);
    if (waves == 4) {
        kernel = valu_tile_kernel<RANK, RB, 4, DIREFT>;
        if constexpr (DIREFT) { if (a.h_layers) kernel = valu_tile_layers_kernel<RANK, RB, 4>; }
    } else if (waves == 2) {
        kernel = valu_tile_kernel<RANK, RB, 2, DIREFT>;
        if constexpr (DIREFT) { if (a.h_layers) kernel = valu_tile_layers_kernel<RANK, RB, 2>; }
    } else {
        waves = 1;
        kernel = valu_tile_kernel<RANK, RB, 1, DIREFT>;
        if constexpr (DIREFT) { if (a.h_layers) kernel = valu_tile_layers_kernel<RANK, RB, 1>; }
    }
    hipLaunchKernelGGL(kernel, dim3(tile_grid(a, S, RB * waves), a.n_layers), dim3(64 * waves), 0, stream, a);
}

// packed projections at ranks 1..3 (vector-ALU kernel)
template <int SLICES>
void launch_valu_packed(const ApplyArgs &a, int64_t S, hipStream_t stream)
{
    constexpr int RB = 4;
    switch (a.rank) {
    case 1:  hipLaunchKernelGGL((valu_tile_kernel<1, RB, 4, false, SLICES>), dim3(tile_grid(a, S, RB * 4)), dim3(256), 0, stream, a); break;
    case 2:  hipLaunchKernelGGL((valu_tile_kernel<2, RB, 4, false, SLICES>), dim3(tile_grid(a, S, RB * 4)), dim3(256), 0, stream, a); break;
    default: hipLaunchKernelGGL((valu_tile_kernel<3, RB, 4, false, SLICES>), dim3(tile_grid(a, S, RB * 4)), dim3(256), 0, stream, a); break;
    }
}

template <bool DIREFT>
void launch_valu_rank(const ApplyArgs &a, int64_t S, const Knobs &k, hipStream_t stream)
{
    switch (a.rank) {
    case 1: launch_valu<1, DIREFT>(a, S, k, stream); break;
    case 2: launch_valu<2, DIREFT>(a, S, k, stream); break;
    case 3: launch_valu<3, DIREFT>(a, S, k, stream); break;
    case 4: launch_valu<4, DIREFT>(a, S, k, stream); break;
    case 5: launch_valu<5, DIREFT>(a, S, k, stream); break;
    case 6: launch_valu<6, DIREFT>(a, S, k, stream); break;
    case 7: launch_valu<7, DIREFT>(a, S, k, stream); break;
    default: launch_valu<8, DIREFT>(a, S, k, stream); break;
    }
}

template <typename E, bool DIREFT>
void launch_rows(const ApplyArgs &a, int64_t S, bool chunks_too, hipStream_t stream)
{
    void (*chunks_kernel)(ApplyArgs) = row_kernel_chunks<E, DIREFT>;
    void (*short_kernel)(ApplyArgs) = row_kernel_short<E, DIREFT>;
    if constexpr (DIREFT) {
        if (a.h_layers) {
            chunks_kernel = row_layers_kernel_chunks<E>;
            short_kernel = row_layers_kernel_short<E>;
        }
    }
    if (chunks_too) {
        hipLaunchKernelGGL(chunks_kernel,
                           dim3((unsigned)(chunk_capacity(a.T, S) * (CHUNK_ROWS / GROUP_ROWS)), a.n_layers),
                           dim3(ROW_THREADS), 0, stream, a);
    }
    int64_t g = ((gtile_capacity(a.T, S, a.N) * GTILE_ROWS + 7) / 8) * 8;     // a multiple of 8: one share per XCD
    if (g > 4096) g = 4096;
    hipLaunchKernelGGL(short_kernel, dim3((unsigned)g, a.n_layers), dim3(ROW_THREADS), 0, stream, a);
}

// Whether the per-row kernel is the faster one for an fp32 call.  A workgroup of the tile kernel walks its tile's columns 512 at a
// time, a trip to memory each, and in place does so alone: few tiles of wide rows wait for that chain (about 2 us per 1000 columns
// of each sweep).  The per-row kernel has a workgroup for every four rows, about 1 us per 1000 columns at rank 1, 1.8 at rank 4, and is
// left behind from rank 8 on, at ranks that are no power of two wherever its groups are full (prompts), by batches that fill the
// chip, and by mixed ones, where it takes its chunks and its gathered rows one after the other.  Measured on three sets of buffers in turn, per-row / tile kernel, us:
//   in place: rank 1, d = 4872, 65 decode rows 13 / 27, 300 prompt rows 15 / 28, 1080 23 / 31, d = 8192, 4000 78 / 64; 1000 decode rows
//     of 512 22 / 11, 4 rows of 1024 7 / 9; three prompts of 340 rows and three decode rows, d = 4096, rank 1 33 / 27; rank 4, d = 8192, 100 prompt rows 21 / 38, 500 decode rows 29 / 41; rank 3,
//     d = 4872, 65 decode rows 0.72 of the tile kernel's time, 300 prompt rows 1.23; rank 5, 16 decode rows 0.64, 65 rows of as many
//     adapters 0.94; rank 8 1.1 and more.
//   out of place: rank 1, 8192 -> 1024, 300 prompt rows 0.61, 2048 -> 8192 1.41, 65 decode rows 0.72, 2500 prompt rows 1.03; rank 4,
//     8192 -> 8192, 500 decode rows 0.86, 1000 1.09, 4872 -> 8192, 65 decode rows 1.1; rank 8, 14336 -> 1024, 16 rows 0.64,
//     8192 -> 8192 1.9.
bool f32_rows_win(const ApplyArgs &a, int64_t S, bool direft)
{
    const int r = a.rank;
    const int64_t T = a.T, tiles = likely_tiles(a, S), in = a.d_in, out = a.d_out;       // whatever n_layers: see takes_small
    const bool prompts = a.T >= 2 * S, mixed = prompts && a.all_tokens && S > 1 + a.T / 256;
    if (r > 8 || T > 2048 || mixed) return false;
    if (direft) {
        if (r <= 2) return in >= 1024;
        if (r == 4) return in >= 1536 && tiles <= 256 && tiles * 16 <= in;
        if (r == 3) return !prompts && in >= 1024 && T <= (in >= 4096 ? 512 : 128);
        return r < 8 && !prompts && in >= 1536 && tiles <= (r == 5 ? 60 : 32);
    }
    if (r <= 2 || r == 4) {
        if ((prompts || in < 1024) && tiles <= 48) return r == 4 ? out < in : out <= in;
        if (r == 4) return in >= 4096 && (prompts || T <= 768) && (T > 128 || in >= out);
        return in >= 2048 || out > 2048;
    }
    if (prompts) return tiles <= 32 && in >= (r == 3 ? 6 : r == 8 ? 7 : 12) * out;
    if (r == 3) return 2 * in >= 3 * out && in >= 4096 && tiles <= 200 && T <= 512;
    return in >= (r == 8 ? 6 : 4) * out && (tiles <= 60 || (r < 8 && in >= 8 * out && tiles <= 200));
}

// fp32: 8 wavefronts per 16-row tile; out of place, col_split workgroups per tile
template <int NB, bool DIREFT>
void launch_f32_nb(const ApplyArgs &a, int64_t S, hipStream_t stream)
{
    constexpr bool BY_LDS = NB <= 2;
    void (*kernel)(ApplyArgs);
    if constexpr (DIREFT) {
        if (a.h_layers) kernel = (a.rank % 4) ? f32_tile_layers_kernel<NB, true> : f32_tile_layers_kernel<NB, false>;
        else            kernel = (a.rank % 4) ? f32_tile_kernel<NB, true, true, BY_LDS> : f32_tile_kernel<NB, true, false, false>;
    } else {
        const bool stay = activations_stay(a, S, a.d_out, 4, STAY_F32);
        kernel = (a.rank % 4) ? f32_tile_kernel<NB, false, true, BY_LDS> : f32_tile_kernel<NB, false, false, false>;
        if (stay) kernel = (a.rank % 4) ? f32_tile_kernel<NB, false, true, BY_LDS, false> : f32_tile_kernel<NB, false, false, false, false>;
        // A workgroup of one or two units of 64 columns has one or two wavefronts at work on them, and LDS is only a further step on their way; at
        // rank 17-31, twice the factors, so is one unit for each of the eight.  Factors by LDS / lane by lane, 14 rows, us: rank 7, 512 -> 512 5.4 / 5.2, 1024 5.5 /
        // 5.2, 4096 (8 units a workgroup) 6.0 / 6.8; rank 31, 512 7.2 / 6.5, 1024 7.3 / 6.6, 2104 -> 4096 14.3 / 14.0, 512 -> 4096 8.5 / 8.9; 1200 rows, rank 31, 2104 ->
        // 512 15.0 / 14.7, 4096 (32 units) 25.4 / 26.6, rank 7 9.6 / 10.3, 17.7 / 20.2.
        if constexpr (BY_LDS) {
            const int units = (a.d_out + 63) / 64 / (a.col_split > 1 ? a.col_split : 1);
            if (a.rank % 4 && units < (NB == 1 ? F32_WAVES / 2 : 2 * F32_WAVES)) kernel = stay ? f32_tile_kernel<NB, false, true, false, false> : f32_tile_kernel<NB, false, true, false>;
        }
    }
    hipLaunchKernelGGL(kernel, dim3(tile_grid(a, S, 16), a.n_layers), dim3(F32_WAVES * 64), 0, stream, a);
}

// Workgroups per tile out of place, where few tiles leave the chip idle.  Each repeats the shrink; a workgroup takes about 8 us
// and 1 us for every 512 columns of x, 1.25 us for every 512 columns of its share of y; one fits a compute unit.  (rank 16, 4096 -> 4096, 1 / 2 / 4 / 8 workgroups: 300 rows
// 26 / 21 / 17 / 16 us, 2304 rows 34 / 40 / 47 / 75; rank 4, 2048 -> 8192, 500 decode rows of 64 adapters, 1 / 2 / 8: 31 / 21 / 29;
// 8192 -> 8192, 200 decode rows of 400 adapters, 1 / 8: 42 / 104.)
inline int f32_col_split(const ApplyArgs &a, int64_t S)
{
    const double tiles = (double)likely_tiles(a, S), in = a.d_in / 512.0, out = a.d_out / 512.0;
    int best = 1;
    double best_us = 0;
    for (int split = 1; split <= 8 && split * 64 <= a.d_out + 63; split *= 2) {
        const double rounds = tiles * split > 240 ? tiles * split / 240 : 1, us = rounds * (8 + in + 1.25 * out / split);
        // a first factor of megabytes is read from memory again by every further workgroup (rank 96, 8192 -> 14336, 1700 rows, 1 / 2 of them:
        // 391 / 473 us); and a gain within the estimate's error is none (rank 96, 680 -> 512: 25 / 30)
        if (split > 1 && tiles * split > 128 && (int64_t)a.d_in * a.rank > (1 << 19)) break;
        if (split == 1 || us < (tiles * split > 128 ? 0.9 : 1.0) * best_us) { best = split; best_us = us; }
    }
    return best;
}

template <bool DIREFT>
void launch_f32(ApplyArgs a, int64_t S, const Knobs &k, hipStream_t stream)
{
    if (!DIREFT) a.col_split = k.colsplit ? k.colsplit : f32_col_split(a, S);
    if (a.rank <= 16)      launch_f32_nb<1, DIREFT>(a, S, stream);
    else if (a.rank <= 32) launch_f32_nb<2, DIREFT>(a, S, stream);
    else if (a.rank <= 64) launch_f32_nb<4, DIREFT>(a, S, stream);
    else                   launch_f32_nb<8, DIREFT>(a, S, stream);
}

enum class Path { Rows, Valu, Mfma, F32 };

Path choose_path(const ApplyArgs &a, int64_t S, bool direft, int dtype, const Knobs &k)
{
    const int rank = a.rank;
    if (k.variant == 1) return Path::Rows;
    if (dtype != PREFT_BF16) {
        const bool narrow = a.d_in <= (1 << 22) && a.d_out <= (1 << 22);     // byte offsets within a factor fit 32 bits
        if (!narrow) return Path::Rows;
        if (k.variant == 0 && k.colsplit == 0 && f32_rows_win(a, S, direft)) return Path::Rows;
        return Path::F32;
    }
    const bool valu_ok = rank <= 8, mfma_ok = mfma_takes(a, k);
    if (k.variant == 2 && valu_ok) return Path::Valu;
    if ((k.variant == 3 || k.variant == 4) && mfma_ok) return Path::Mfma;
    if (rank <= 3) return Path::Valu;
    if (mfma_ok) return Path::Mfma;
    return Path::Rows;
}

template <bool DIREFT>
int launch_apply(const ApplyArgs &a, int64_t S, int dtype, const Knobs &k, hipStream_t stream)
{
    switch (choose_path(a, S, DIREFT, dtype, k)) {
    case Path::F32:
        launch_f32<DIREFT>(a, S, k, stream);
        break;
    case Path::Mfma: {                     // the tile kernels take chunks and gathered tiles alike
        if (takes_small(a, S, a.d_out, DIREFT, k)) launch_small_order<DIREFT>(a, S, 1, k, stream);
        else                           launch_mfma_rank<DIREFT>(a, S, k, stream);
        break;
    }
    case Path::Valu:
        if (takes_small(a, S, a.d_out, DIREFT, k)) { launch_small<DIREFT>(a, S, 1, k, stream); break; }
        if constexpr (!DIREFT) {
            if (a.rank <= 3 && launch_valu_split<1>(a, S, k, stream)) break;
        }
        launch_valu_rank<DIREFT>(a, S, k, stream);
        break;
    default:
        if (dtype == PREFT_BF16) launch_rows<bf16_tag, DIREFT>(a, S, true, stream);
        else                     launch_rows<float, DIREFT>(a, S, true, stream);
        break;
    }
    return check_launch();
}

// LoReFT derived factors of one adapter (App. C.2): D = W - R in the storage type, Rt = R^T.
template <typename E>
__global__ __launch_bounds__(256) void loreft_prepare_kernel(void *D, void *Rt, const void *W, const void *R,
                                                             int32_t d, int32_t rank)
{
    const int64_t n = (int64_t)d * rank;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
        const int64_t k = i / d, j = i - k * d;
        const float w = Elem<E>::load1(as_global(W), i), q = Elem<E>::load1(as_global(R), i);
        Elem<E>::store1(as_global(D), i, w - q);
        Elem<E>::store1(as_global(Rt), j * rank + k, q);
    }
}

// the fields of a launch that name the batch and its schedule
void bind_schedule(ApplyArgs &a, void *workspace, int32_t T, int32_t S, int32_t N, int mode)
{
    const ScheduleView v = view_of(workspace, T, S);
    a.T = T; a.S = S; a.N = N; a.all_tokens = (mode & PREFT_ALL_TOKENS) ? 1 : 0;
    a.header = v.header; a.chunks = v.chunks; a.shorts = v.shorts; a.gtiles = v.gtiles;
    a.gathered_only = 0; a.chunks_only = 0; a.xcd_runs = 0; a.col_split = 1; a.zws = nullptr; a.z_blocks = 0;
}

// a workspace with room for z lets LoRA calls run their sweeps as two launches
void bind_z(ApplyArgs &a, void *workspace, size_t bytes, int32_t T, int32_t S, int32_t rank, int32_t n_proj)
{
    if (bytes >= z_offset(T, S) + z_bytes(T, S, rank, n_proj)) {
        a.zws = reinterpret_cast<char *>(workspace) + z_offset(T, S);
        a.z_blocks = chunk_capacity(T, S) * (CHUNK_ROWS / 16);
    }
}

int check_matrix(const void *p, int64_t ld, int32_t width, int dtype)
{
    const int per16 = dtype == PREFT_BF16 ? 8 : 4;
    if (!p || width <= 0 || ld < width) return PREFT_EINVAL;
    if (!aligned16(p) || (width % per16) != 0 || (ld % per16) != 0) return PREFT_EALIGN;
    return PREFT_OK;
}

// the in-place launch shared by the one-layer and the many-layer DiReFT entry points; `a` names
// the residual stream(s) and the pools
int direft_launch(ApplyArgs a, int64_t ldh, int32_t T, int32_t d, const int32_t *seg_start,
                  const int32_t *seg_adapter, const int32_t *seg_prefill_len, int32_t S, int32_t N, int32_t rank,
                  float scale, int dtype, int mode, void *workspace, size_t bytes, void *stream)
{
    hipStream_t st = reinterpret_cast<hipStream_t>(stream);
    if (!(mode & PREFT_SCHEDULE_READY)) {
        const int rc = launch_schedule(workspace, seg_start, seg_adapter, seg_prefill_len, S, T, N, mode, st);
        if (rc != PREFT_OK) return rc;
    }
    bind_schedule(a, workspace, T, S, N, mode);
    bind_z(a, workspace, bytes, T, S, rank, 1);
    a.ldy = ldh; a.ldx = ldh; a.d_in = d; a.d_out = d;
    a.rank = rank; a.scale = scale;
    return launch_apply<true>(a, S, dtype, knobs_of(mode), st);
}

}  // namespace

extern "C" {

size_t preft_workspace_bytes(int32_t T, int32_t S)
{
    if (T < 0 || S < 0) return 0;
    return workspace_bytes(T, S);
}

size_t preft_workspace_bytes_z(int32_t T, int32_t S, int32_t rank, int32_t n_proj)
{
    if (T < 0 || S < 0 || rank < 1 || rank > PREFT_MAX_RANK || n_proj < 1 || n_proj > PREFT_MAX_PACKED) return 0;
    return z_offset(T, S) + z_bytes(T, S, rank, n_proj);
}

int preft_schedule(void *workspace, size_t bytes, const int32_t *seg_start, const int32_t *seg_adapter,
                   const int32_t *seg_prefill_len, int32_t S, int32_t T, int32_t N, int mode, void *stream)
{
    if (mode & PREFT_SCHEDULE_READY) return PREFT_EINVAL;
    int rc = check_tables(workspace, bytes, seg_start, seg_adapter, seg_prefill_len, S, T, N, mode);
    if (rc != PREFT_OK || T == 0 || S == 0) return rc;
    return launch_schedule(workspace, seg_start, seg_adapter, seg_prefill_len, S, T, N, mode,
                           reinterpret_cast<hipStream_t>(stream));
}

int preft_lora_apply(void *y, int64_t ldy, const void *x, int64_t ldx, int32_t T, int32_t d_in, int32_t d_out,
                     const int32_t *seg_start, const int32_t *seg_adapter, const int32_t *seg_prefill_len,
                     int32_t S, const void *const *A_pool, const void *const *B_pool, int32_t N, int32_t rank,
                     float scale, int dtype, int mode, void *workspace, size_t bytes, void *stream)
{
    if (dtype != PREFT_F32 && dtype != PREFT_BF16) return PREFT_EINVAL;
    int rc = check_tables(workspace, bytes, seg_start, seg_adapter, seg_prefill_len, S, T, N, mode);
    if (rc != PREFT_OK) return rc;
    if (rank < 1 || rank > PREFT_MAX_RANK) return PREFT_EUNSUPPORTED;
    if (T == 0 || S == 0) return PREFT_OK;
    if ((rc = check_matrix(y, ldy, d_out, dtype)) != PREFT_OK) return rc;
    if ((rc = check_matrix(x, ldx, d_in, dtype)) != PREFT_OK) return rc;
    if (!A_pool || !B_pool) return PREFT_EINVAL;
    {   // x and y must not overlap
        const size_t es = dtype == PREFT_BF16 ? 2 : 4;
        const char *y0 = reinterpret_cast<const char *>(y), *x0 = reinterpret_cast<const char *>(x);
        const char *y1 = y0 + ((size_t)(T - 1) * ldy + d_out) * es, *x1 = x0 + ((size_t)(T - 1) * ldx + d_in) * es;
        if (y0 < x1 && x0 < y1) return PREFT_EINVAL;
    }
    hipStream_t st = reinterpret_cast<hipStream_t>(stream);
    if (!(mode & PREFT_SCHEDULE_READY)) {
        rc = launch_schedule(workspace, seg_start, seg_adapter, seg_prefill_len, S, T, N, mode, st);
        if (rc != PREFT_OK) return rc;
    }
    ApplyArgs a;
    bind_schedule(a, workspace, T, S, N, mode);
    a.y = y; a.x = x; a.ldy = ldy; a.ldx = ldx; a.d_in = d_in; a.d_out = d_out;
    a.A_pool = A_pool; a.Bt_pool = B_pool; a.bias_pool = nullptr; a.rank = rank; a.scale = scale;
    bind_z(a, workspace, bytes, T, S, rank, 1);
    return launch_apply<false>(a, S, dtype, knobs_of(mode), st);
}

int preft_lora_apply_packed(int32_t n_proj, void *const *y, const int64_t *ldy, const int32_t *d_out, const void *x,
                            int64_t ldx, int32_t T, int32_t d_in, const int32_t *seg_start,
                            const int32_t *seg_adapter, const int32_t *seg_prefill_len, int32_t S,
                            const void *const *const *A_pools, const void *const *const *B_pools, int32_t N,
                            int32_t rank, float scale, int dtype, int mode, void *workspace, size_t bytes,
                            void *stream)
{
    if (n_proj < 1 || n_proj > PREFT_MAX_PACKED || !y || !ldy || !d_out || !A_pools || !B_pools) return PREFT_EINVAL;
    if (dtype != PREFT_F32 && dtype != PREFT_BF16) return PREFT_EINVAL;
    int rc = check_tables(workspace, bytes, seg_start, seg_adapter, seg_prefill_len, S, T, N, mode);
    if (rc != PREFT_OK) return rc;
    if (rank < 1 || rank > PREFT_MAX_RANK) return PREFT_EUNSUPPORTED;
    if (T == 0 || S == 0) return PREFT_OK;
    if ((rc = check_matrix(x, ldx, d_in, dtype)) != PREFT_OK) return rc;
    const size_t es = dtype == PREFT_BF16 ? 2 : 4;
    const char *x0 = reinterpret_cast<const char *>(x), *x1 = x0 + ((size_t)(T - 1) * ldx + d_in) * es;
    for (int32_t i = 0; i < n_proj; ++i) {
        if ((rc = check_matrix(y[i], ldy[i], d_out[i], dtype)) != PREFT_OK) return rc;
        if (!A_pools[i] || !B_pools[i]) return PREFT_EINVAL;
        const char *y0 = reinterpret_cast<const char *>(y[i]), *y1 = y0 + ((size_t)(T - 1) * ldy[i] + d_out[i]) * es;
        if (y0 < x1 && x0 < y1) return PREFT_EINVAL;                       // x and y must not overlap
        // outputs must not share an element: disjoint buffers, or disjoint column ranges of one
        // buffer (same row stride, both inside one row pitch); anything else that overlaps is refused
        for (int32_t j = 0; j < i; ++j) {
            const char *z0 = reinterpret_cast<const char *>(y[j]);
            const char *z1 = z0 + ((size_t)(T - 1) * ldy[j] + d_out[j]) * es;
            if (!(y0 < z1 && z0 < y1)) continue;
            if (ldy[i] != ldy[j]) return PREFT_EINVAL;
            const bool i_low = y0 < z0;
            const size_t w_lo = (size_t)(i_low ? d_out[i] : d_out[j]) * es, w_hi = (size_t)(i_low ? d_out[j] : d_out[i]) * es;
            const size_t delta = (size_t)(i_low ? z0 - y0 : y0 - z0), pitch = (size_t)ldy[i] * es;
            if (delta < w_lo || delta + w_hi > pitch) return PREFT_EINVAL;
        }
    }
    hipStream_t st = reinterpret_cast<hipStream_t>(stream);
    if (!(mode & PREFT_SCHEDULE_READY)) {
        rc = launch_schedule(workspace, seg_start, seg_adapter, seg_prefill_len, S, T, N, mode, st);
        if (rc != PREFT_OK) return rc;
    }
    const int ready = mode | PREFT_SCHEDULE_READY;
    const Knobs k = knobs_of(mode);
    const bool fused_valu = n_proj > 1 && dtype == PREFT_BF16 && rank <= 3 && (k.variant == 0 || k.variant == 2) &&
                            (k.waves == 0 || k.waves == 4);
    bool fused_wide = n_proj > 1 && dtype == PREFT_BF16 && rank > 16 && rank <= 64 &&
                      (k.variant == 0 || k.variant == 4 || k.variant == 5) && k.waves == 0 && k.rowblocks == 0 && (d_in % 128) == 0 &&
                      (k.colsplit ? k.colsplit == 1 || k.variant == 4 : T > SMALL_T);
    for (int32_t i = 0; i < n_proj && fused_wide; ++i) fused_wide = (d_out[i] % 128) == 0;
    ApplyArgs a;
    bind_schedule(a, workspace, T, S, N, mode);
    a.x = x; a.ldx = ldx; a.d_in = d_in; a.rank = rank;
    const bool fused_mfma = n_proj > 1 && dtype == PREFT_BF16 && rank >= 4 && rank <= 16 &&
                            (k.variant == 0 || k.variant == 3 || k.variant == 5) && column_split_fits(a);
    int32_t widest = 0;
    int64_t width = 0;
    for (int32_t i = 0; i < n_proj; ++i) { width += d_out[i]; if (d_out[i] > widest) widest = d_out[i]; }
    const bool fused_small = n_proj > 1 && dtype == PREFT_BF16 && takes_small(a, S, widest, width, false, k);
    const bool fused = fused_small || fused_mfma || fused_valu || fused_wide;
    if (!fused) {                                  // same result, one launch per projection
        for (int32_t i = 0; i < n_proj; ++i) {
            rc = preft_lora_apply(y[i], ldy[i], x, ldx, T, d_in, d_out[i], seg_start, seg_adapter, seg_prefill_len, S,
                                  A_pools[i], B_pools[i], N, rank, scale, dtype, ready, workspace, bytes, stream);
            if (rc != PREFT_OK) return rc;
        }
        return PREFT_OK;
    }
    a.y = y[0]; a.ldy = ldy[0]; a.d_out = d_out[0];
    a.A_pool = A_pools[0]; a.Bt_pool = B_pools[0]; a.bias_pool = nullptr; a.scale = scale;
    bind_z(a, workspace, bytes, T, S, rank, n_proj);
    for (int32_t i = 1; i < n_proj; ++i) {
        a.more[i - 1].y = y[i]; a.more[i - 1].ldy = ldy[i]; a.more[i - 1].d_out = d_out[i];
        a.more[i - 1].A_pool = A_pools[i]; a.more[i - 1].Bt_pool = B_pools[i];
    }
    if (fused_small) {
        launch_small_order<false>(a, S, n_proj, k, st);
    } else if (fused_wide) {
        if (rank <= 32) launch_mfma_wide_packed<2>(a, n_proj, S, k, st);
        else            launch_mfma_wide_packed<4>(a, n_proj, S, k, st);
    } else if (fused_mfma) {
        const int pieces = (rank % 4) == 0 ? 0 : rank < 8 ? 2 : 4;      // the any-rank shape's block pieces per lane
        if (n_proj == 2) {
            if (pieces == 0)      launch_mfma_packed<2>(a, S, k, st);
            else if (pieces == 2) launch_mfma_packed<2, 2>(a, S, k, st);
            else                  launch_mfma_packed<2, 4>(a, S, k, st);
        } else {
            if (pieces == 0)      launch_mfma_packed<3>(a, S, k, st);
            else if (pieces == 2) launch_mfma_packed<3, 2>(a, S, k, st);
            else                  launch_mfma_packed<3, 4>(a, S, k, st);
        }
    } else {
        if (n_proj == 2 ? launch_valu_split<2>(a, S, k, st) : launch_valu_split<3>(a, S, k, st)) return check_launch();
        if (n_proj == 2) launch_valu_packed<2>(a, S, st);
        else             launch_valu_packed<3>(a, S, st);
    }
    return check_launch();
}

int preft_loreft_prepare(void *D, void *Rt, const void *W, const void *R, int32_t d, int32_t rank, int dtype,
                         void *stream)
{
    if (dtype != PREFT_F32 && dtype != PREFT_BF16) return PREFT_EINVAL;
    if (!D || !Rt || !W || !R || d <= 0) return PREFT_EINVAL;
    if (rank < 1 || rank > PREFT_MAX_RANK) return PREFT_EUNSUPPORTED;
    if (!aligned16(D) || !aligned16(Rt) || !aligned16(W) || !aligned16(R)) return PREFT_EALIGN;
    {   // outputs must not overlap the inputs or each other
        const size_t bytes = (size_t)d * rank * (dtype == PREFT_BF16 ? 2 : 4);
        const char *p[4] = {reinterpret_cast<const char *>(D), reinterpret_cast<const char *>(Rt),
                            reinterpret_cast<const char *>(W), reinterpret_cast<const char *>(R)};
        for (int a = 0; a < 2; ++a)
            for (int b = a + 1; b < 4; ++b)
                if (p[a] < p[b] + bytes && p[b] < p[a] + bytes) return PREFT_EINVAL;
    }
    hipStream_t st = reinterpret_cast<hipStream_t>(stream);
    const int64_t n = (int64_t)d * rank;
    const unsigned grid = (unsigned)((n + 255) / 256 < 4096 ? (n + 255) / 256 : 4096);
    if (dtype == PREFT_BF16)
        hipLaunchKernelGGL((loreft_prepare_kernel<bf16_tag>), dim3(grid), dim3(256), 0, st, D, Rt, W, R, d, rank);
    else
        hipLaunchKernelGGL((loreft_prepare_kernel<float>), dim3(grid), dim3(256), 0, st, D, Rt, W, R, d, rank);
    return check_launch();
}

int preft_loreft_apply(void *h, int64_t ldh, int32_t T, int32_t d, const int32_t *seg_start,
                       const int32_t *seg_adapter, const int32_t *seg_prefill_len, int32_t S,
                       const void *const *D_pool, const void *const *Rt_pool, const void *const *b_pool,
                       int32_t N, int32_t rank, float scale, int dtype, int mode, void *workspace, size_t bytes,
                       void *stream)
{
    // h += s R^T (W h + b - R h) = s Rt (D h + b): the in-place kernels with the derived factors
    return preft_direft_apply(h, ldh, T, d, seg_start, seg_adapter, seg_prefill_len, S, D_pool, Rt_pool, b_pool, N,
                              rank, scale, dtype, mode, workspace, bytes, stream);
}

int preft_direft_apply(void *h, int64_t ldh, int32_t T, int32_t d, const int32_t *seg_start,
                       const int32_t *seg_adapter, const int32_t *seg_prefill_len, int32_t S,
                       const void *const *W1_pool, const void *const *W2t_pool, const void *const *b_pool,
                       int32_t N, int32_t rank, float scale, int dtype, int mode, void *workspace, size_t bytes,
                       void *stream)
{
    if (dtype != PREFT_F32 && dtype != PREFT_BF16) return PREFT_EINVAL;
    int rc = check_tables(workspace, bytes, seg_start, seg_adapter, seg_prefill_len, S, T, N, mode);
    if (rc != PREFT_OK) return rc;
    if (rank < 1 || rank > PREFT_MAX_RANK) return PREFT_EUNSUPPORTED;
    if (T == 0 || S == 0) return PREFT_OK;
    if ((rc = check_matrix(h, ldh, d, dtype)) != PREFT_OK) return rc;
    if (!W1_pool || !W2t_pool) return PREFT_EINVAL;
    ApplyArgs a;
    a.y = h; a.x = h; a.A_pool = W1_pool; a.Bt_pool = W2t_pool; a.bias_pool = b_pool;
    return direft_launch(a, ldh, T, d, seg_start, seg_adapter, seg_prefill_len, S, N, rank, scale, dtype, mode,
                         workspace, bytes, stream);
}

int preft_direft_apply_static(void *h, int64_t ldh, int32_t T, int32_t d, const int32_t *seg_start,
                              const int32_t *seg_adapter, const int32_t *seg_prefill_len, int32_t S,
                              const void *const *W1_pool, const void *const *W2t_pool, const void *const *b_pool,
                              int32_t N, int32_t rank, float scale, int dtype, int mode, void *stream)
{
    // sizes first (host arithmetic only): the schedule of this batch must fit the static area
    if (T < 0 || S < 0) return PREFT_EINVAL;
    if (workspace_bytes(T, S) > (size_t)PREFT_STATIC_SCRATCH_BYTES) return PREFT_ETOOLARGE;
    if (dtype != PREFT_F32 && dtype != PREFT_BF16) return PREFT_EINVAL;
    if (T == 0 || S == 0) {     // nothing to do: same answers as preft_direft_apply, without touching the device
        const int rc = check_tables(nullptr, 0, seg_start, seg_adapter, seg_prefill_len, S, T, N, mode);
        if (rc != PREFT_OK) return rc;
        return (rank < 1 || rank > PREFT_MAX_RANK) ? PREFT_EUNSUPPORTED : PREFT_OK;
    }
    void *area = nullptr;
    const int rc = static_scratch_of(&area);
    if (rc != PREFT_OK) return rc;
    return preft_direft_apply(h, ldh, T, d, seg_start, seg_adapter, seg_prefill_len, S, W1_pool, W2t_pool, b_pool, N,
                              rank, scale, dtype, mode, area, (size_t)PREFT_STATIC_SCRATCH_BYTES, stream);
}

int preft_direft_apply_layers(void *const *h_layers, int64_t ldh, int32_t n_layers, int32_t T, int32_t d,
                              const int32_t *seg_start, const int32_t *seg_adapter,
                              const int32_t *seg_prefill_len, int32_t S, const void *const *const *W1_pools,
                              const void *const *const *W2t_pools, const void *const *const *b_pools, int32_t N,
                              int32_t rank, float scale, int dtype, int mode, void *workspace, size_t bytes,
                              void *stream)
{
    if (dtype != PREFT_F32 && dtype != PREFT_BF16) return PREFT_EINVAL;
    if (n_layers < 0 || n_layers > PREFT_MAX_LAYERS) return PREFT_EINVAL;
    int rc = check_tables(workspace, bytes, seg_start, seg_adapter, seg_prefill_len, S, T, N, mode);
    if (rc != PREFT_OK) return rc;
    if (rank < 1 || rank > PREFT_MAX_RANK) return PREFT_EUNSUPPORTED;
    if (T == 0 || S == 0 || n_layers == 0) return PREFT_OK;
    if (!h_layers || !W1_pools || !W2t_pools) return PREFT_EINVAL;
    // the residual streams themselves are named on the device: only their common shape is checked
    const int per16 = dtype == PREFT_BF16 ? 8 : 4;
    if (d <= 0 || ldh < d) return PREFT_EINVAL;
    if ((d % per16) || (ldh % per16)) return PREFT_EALIGN;
    ApplyArgs a;
    a.y = nullptr; a.x = nullptr; a.A_pool = nullptr; a.Bt_pool = nullptr; a.bias_pool = nullptr;
    a.h_layers = h_layers; a.A_layers = W1_pools; a.Bt_layers = W2t_pools; a.bias_layers = b_pools;
    a.n_layers = n_layers;
    return direft_launch(a, ldh, T, d, seg_start, seg_adapter, seg_prefill_len, S, N, rank, scale, dtype, mode,
                         workspace, bytes, stream);
}

int preft_schedule_counts(const void *workspace, int32_t *counts, void *stream)
{
    if (!workspace || !counts) return PREFT_EINVAL;
    hipStream_t st = reinterpret_cast<hipStream_t>(stream);
    int32_t header[HEADER_INTS];
    if (hipMemcpyAsync(header, workspace, sizeof(header), hipMemcpyDeviceToHost, st) != hipSuccess)
        return PREFT_EHIP;
    if (hipStreamSynchronize(st) != hipSuccess) return PREFT_EHIP;
    counts[0] = header[HDR_CHUNKS]; counts[1] = header[HDR_SHORT_ROWS]; counts[2] = header[HDR_ACTIVE];
    return header[HDR_MISMATCH] ? PREFT_ESCHEDULE : PREFT_OK;
}

const char *preft_strerror(int code)
{
    switch (code) {
    case PREFT_OK:           return "ok";
    case PREFT_EINVAL:       return "invalid argument (null pointer, negative size, bad enum, overlapping x and y, or row stride below the width)";
    case PREFT_EUNSUPPORTED: return "unsupported rank (must be 1..128)";
    case PREFT_EALIGN:       return "pointer, width or row stride not a multiple of 16 bytes";
    case PREFT_EWORKSPACE:   return "workspace missing, misaligned or smaller than preft_workspace_bytes(T, S)";
    case PREFT_EHIP:         return "HIP runtime error (launch, copy or allocation)";
    case PREFT_ECAPACITY:    return "more distinct adapters in one batch than the slot manager has slots";
    case PREFT_ETOOLARGE:    return "batch too large for the static schedule area of preft_direft_apply_static (preft_workspace_bytes(T, S) exceeds PREFT_STATIC_SCRATCH_BYTES)";
    case PREFT_ESCHEDULE:    return "an apply call named another T, S, N or position set than the schedule in its workspace was built for; that call did nothing";
    default:                 return "unknown preft error code";
    }
}

int preft_version(void) { return 200; }

}  // extern "C"
