// Host side of the small-batch MFMA kernel: support check, launch plan, scratch sizing, dispatch.
#include "gptq_w4a16.h"
#include "skinny_kernel.h"

namespace gptq {

namespace {

constexpr int kMaxActivationLdsBytes = 64 * 1024;
constexpr size_t kCounterBytes = 256 * 1024;  // same fixed counter area as the vector kernel
constexpr int kMaxColumnTiles = (int)(kCounterBytes / sizeof(unsigned));

int ceil_div(int a, int b)
{
    return (a + b - 1) / b;
}

// Batches of more than 64 rows are processed 64 rows at a time (one launch each, same stream): the weights
// are streamed once per launch, the second time mostly from the memory-side cache.
constexpr int kRowsPerLaunch = 64;

int row_blocks(int M)
{
    return M <= 16 ? 1 : M <= 32 ? 2 : 4;
}

int rows_of_launch(int M)
{
    return M < kRowsPerLaunch ? M : kRowsPerLaunch;
}

// Wavefronts per workgroup: eight where the 64-column workgroups have a compute unit each, else four.
int waves_of(int tiles_n, int split_k, int wn, int tm)
{
    // (four row blocks do not fit the 256 registers that two wavefronts per SIMD leave each)
    return (wn == 1 && tm <= 2 && (long long)tiles_n * split_k <= 256) ? 8 : 4;
}

template <int TM, int WN, int WAVES, int GPU = 1, bool ACT = false, bool TAIL = false, bool STREAM = false,
          bool SERIAL = false>
hipError_t launch_tm(const skinny::Args &a, size_t lds, hipStream_t stream)
{
    auto kernel = skinny::skinny_kernel<TM, WN, WAVES, GPU, ACT, TAIL, STREAM, SERIAL>;
    if (lds > 48 * 1024) {
        hipError_t err = hipFuncSetAttribute(reinterpret_cast<const void *>(kernel),
                                             hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (err != hipSuccess)
            return err;
    }
    const unsigned grid = (unsigned)(a.tiles_n * a.row_tiles * (SERIAL ? 1 : a.split_k));
    hipLaunchKernelGGL(kernel, dim3(grid), dim3(64 * WAVES), lds, stream, a);
    return hipGetLastError();
}

// Groups of 128 / GPU k and a K that ends inside a unit.
template <int GPU, bool SERIAL>
hipError_t launch_tail(const skinny::Args &a, int tm, int waves, size_t lds, hipStream_t stream)
{
    if (tm == 1)
        return waves == 8 ? launch_tm<1, 1, 8, GPU, false, true, false, SERIAL>(a, lds, stream)
                          : launch_tm<1, 1, 4, GPU, false, true, false, SERIAL>(a, lds, stream);
    return waves == 8 ? launch_tm<2, 1, 8, GPU, false, true, false, SERIAL>(a, lds, stream)
                      : launch_tm<2, 1, 4, GPU, false, true, false, SERIAL>(a, lds, stream);
}

// Act-order with lookups.
template <bool TAIL, bool SERIAL>
hipError_t launch_lookup(const skinny::Args &a, int tm, int waves, size_t lds, hipStream_t stream)
{
    if (tm == 1)
        return waves == 8 ? launch_tm<1, 1, 8, 1, true, TAIL, false, SERIAL>(a, lds, stream)
                          : launch_tm<1, 1, 4, 1, true, TAIL, false, SERIAL>(a, lds, stream);
    if (tm == 2)
        return waves == 8 ? launch_tm<2, 1, 8, 1, true, TAIL, false, SERIAL>(a, lds, stream)
                          : launch_tm<2, 1, 4, 1, true, TAIL, false, SERIAL>(a, lds, stream);
    return launch_tm<4, 1, 4, 1, true, TAIL, false, SERIAL>(a, lds, stream);
}

// LDS that a workgroup of the act-order variant may use (the rest holds its static words).
constexpr size_t kActLdsBytes = 160 * 1024 - 512;

size_t act_table_bytes(const Problem &p)
{
    return (size_t)(p.K / p.group_size) * skinny::kActTableRow;
}

// Units whose table offsets fit the LDS behind the table (0: not even one unit's do).
int act_max_units(const Problem &p)
{
    const size_t table = act_table_bytes(p);
    return table >= kActLdsBytes ? 0 : (int)((kActLdsBytes - table) / (skinny::kUnitK * sizeof(uint32_t)));
}

}  // namespace

// K must be a multiple of 32; groups may be of any size, the table of all of them has to fit the LDS beside
// the offsets of a slice (K = 28672 with groups of 64 does, with groups of 32 does not and stays with the kernels of an
// explicit request).  Up to 606 groups slices have sixteen units or more; up to 630 they have four or more, and the
// table is laid out again for every few units: still faster than the general path up to 384 rows (20096x8192, 628 groups:
// M = 2 187 us against 1311, M = 256 686, 1372; 630 groups: M = 384 1186, 1401), but not at 512 and more (1581, 1440).
bool act_supported(const Problem &p)
{
    if (p.g_idx == nullptr || p.M < 2 || p.N < 8 || p.K % 32 != 0)
        return false;
    const long long tiles = (long long)ceil_div(p.N, skinny::kCols) * ceil_div(p.M, skinny::kActRows);
    return tiles <= kMaxColumnTiles && act_max_units(p) >= (p.M <= 384 ? 4 : 16);
}

void act_make_plan(const Problem &p, SkinnyPlan &plan)
{
    const int total_units = ceil_div(p.K, skinny::kUnitK);
    const int tm = row_blocks(p.M);
    const int tiles = ceil_div(p.N, skinny::kCols) * ceil_div(p.M, skinny::kActRows);
    plan.cols_per_wg = skinny::kCols;
    int split = plan.split_k;
    int quantum = 1;
    const bool automatic = split <= 0;
    if (!automatic) {
        // a request for the automatic plan's slices (a queried plan given back) is the automatic plan: its slices are
        // whole multiples of a quantum, which the number of slices alone does not tell
        SkinnyPlan own = {};
        act_make_plan(p, own);
        if (own.split_k == split) {
            plan = own;
            return;
        }
    }
    if (automatic) {
        // One workgroup per compute unit, as in the plain format: measured best of 1, 2, 3, 4, 6 and 8 slices on
        // 4096x11008 (M = 8: 12.7 us unsplit, 15.4 in two), 11008x4096 (25.9 unsplit, 13.7 in four, 15.2 in eight)
        // and 4096x4096 (12.1, 8.8 in four) for M = 2 ... 512.  Up to 64 rows the partial sums, written and read, stay
        // within the weight bytes (8 * split * M * N <= K * N / 2; 4096x4096 at M = 64, at that limit: 18.0 us in four
        // slices, 22.5 in two); above, their row tiles leave room for few slices anyway (at most K / 1024).
        split = (256 + tiles / 2) / tiles;
        const int max_split = p.K / (16 * (p.M < skinny::kActRows ? p.M : skinny::kActRows));
        if (split > max_split)
            split = max_split;
        // (and within the static scratch block, so that gptq_w4a16_gemm_static runs the same plan)
        const long long slice_bytes = (long long)p.M * p.N * sizeof(float);
        if (split * slice_bytes > (long long)(GPTQ_STATIC_SCRATCH_BYTES - kCounterBytes))
            split = (int)((GPTQ_STATIC_SCRATCH_BYTES - kCounterBytes) / slice_bytes);
        if (split < 1)
            split = 1;
        quantum = waves_of(tiles, split, 1, tm);
    }
    if (split > total_units)
        split = total_units;
    int ups = ceil_div(ceil_div(total_units, split), quantum) * quantum;
    if (ups > act_max_units(p))
        ups = act_max_units(p);
    if (ups > total_units)
        ups = total_units;
    plan.units_per_slice = ups;
    plan.split_k = ceil_div(total_units, ups);
    // Slices that only the room for their offsets calls for, with partial sums beyond the static block: the tiles alone fill
    // the chip then, and the workgroups walk the slices themselves (606 groups, ten slices: 2048x19392x8192 4485 us with
    // 671 MB of partial sums, 2929 without; 200x19392x8192 518, 356; 320x19392x4096 329, 340).
    plan.serial = plan.serial || (automatic && act_workspace_bytes(p, plan) > GPTQ_STATIC_SCRATCH_BYTES);
}

size_t act_workspace_bytes(const Problem &p, const SkinnyPlan &plan)
{
    return plan.split_k > 1 && !plan.serial ? kCounterBytes + (size_t)plan.split_k * p.M * p.N * sizeof(float) : 0;
}

hipError_t launch_act(const Problem &p, const SkinnyPlan &plan, void *workspace, hipStream_t stream)
{
    unsigned char *ws = static_cast<unsigned char *>(workspace);
    const int tm = row_blocks(p.M);
    skinny::Args a;
    a.x = p.x;
    a.qweight = p.qweight;
    a.qzeros = p.qzeros;
    a.scales = p.scales;
    a.g_idx = p.g_idx;
    a.out = p.out;
    a.counters = reinterpret_cast<unsigned *>(ws);
    a.partial = ws ? reinterpret_cast<float *>(ws + kCounterBytes) : nullptr;
    a.M = p.M;
    a.K = p.K;
    a.N = p.N;
    a.groups = p.K / p.group_size;
    a.row_tiles = ceil_div(p.M, skinny::kActRows);
    a.units_per_group = 1;
    a.unit_group_shift = 0;
    a.tiles_n = ceil_div(p.N, skinny::kCols);
    a.split_k = plan.split_k;
    a.units_per_slice = plan.units_per_slice;
    a.total_units = ceil_div(p.K, skinny::kUnitK);
    a.slots = nullptr;
    a.serial_slices = 0;
    const int waves = waves_of(a.tiles_n * a.row_tiles, a.split_k, 1, tm);
    const size_t table = act_table_bytes(p) + (size_t)plan.units_per_slice * skinny::kUnitK * sizeof(uint32_t);
    const size_t red = (size_t)waves * 16 * tm * skinny::kCols * sizeof(float);
    const size_t lds = table > red ? table : red;
    if (plan.serial)
        return p.K % skinny::kUnitK != 0 ? launch_lookup<true, true>(a, tm, waves, lds, stream)
                                         : launch_lookup<false, true>(a, tm, waves, lds, stream);
    return p.K % skinny::kUnitK != 0 ? launch_lookup<true, false>(a, tm, waves, lds, stream)
                                     : launch_lookup<false, false>(a, tm, waves, lds, stream);
}

bool skinny_supported(const Problem &p)
{
    if (p.g_idx != nullptr || p.M < 1 || p.M > kSkinnyMaxM || p.N < 8 || ceil_div(p.N, skinny::kCols) > kMaxColumnTiles)
        return false;
    // groups of 64 and 32 k: the 64-column kernel with up to two row blocks (K need not be whole 128-k units)
    if (p.group_size == 64 || p.group_size == 32)
        return p.M <= 32;
    return p.group_size % 128 == 0;
}

bool ring_supported(const Problem &p)
{
    if (p.K % skinny::kUnitK != 0)
        return false;
    if (p.M > 32 && p.M <= kRingMaxM && p.group_size == 64) {  // (from there on under the mid-batch kernel's id alone)
        Problem few = p;
        few.M = 32;
        return skinny_supported(few);
    }
    return skinny_supported(p) && p.M <= kRingMaxM;
}

bool ring_width(const Problem &p, int cols, int split_k)
{
    if (p.M > kRingWideMaxM && cols != 32)
        return false;
    // (skinny_supported leaves widths of 64 and more a counter for every tile; 32 columns have one up to N = 2097152)
    return (cols == 32 || cols == 64 || cols == 96 || (cols == 128 && p.M <= 32)) &&
           (split_k <= 1 || ceil_div(p.N, cols) <= kMaxColumnTiles);
}

namespace {

// Slots that two slices need: one for every pair of outputs.
size_t ring_slot_bytes(const Problem &p)
{
    return (size_t)p.M * p.N * sizeof(float);
}

// Microseconds that a launch of ring_kernel takes, fitted to 11 k measured plans of 160 random layers (K 1024-28672, N
// 1024-57344, groups of 128, 2-32 rows, weights from HBM).  A fixed part, the bytes at HBM speed, the units that one
// wavefront walks - more where workgroups share a compute unit -, the sum over the wavefronts, and the exchange: two
// slices swap their sums (exchange.h), more go through scratch, at a price for each of them.
// Checked, and that price set, on 33 k more plans of 590 layers with groups of 32, 64 and 128: the plan that it picks is
// 0.7 % behind the best one (0.97 % without the price, at worst 24: 9472x1792 at M = 2 in ten slices of 96 columns 8.5 us, in
// two of 32 7.3).  Factors on the units of groups of 64 and 32, 1.1 and 1.2, changed that by less than 0.1 % and are left out.
// 33-64 rows: the units alone, on 1100 plans of 245 layers with groups of 64 and 128.
float ring_estimate(const Problem &p, int cols, int split, int units_per_slice)
{
    static const float unit[4][8] = {{0.57f, 0.65f, 0.85f, 0.95f, 1.18f, 1.39f, 1.43f, 1.59f}, {0.90f, 0.92f, 1.20f, 1.24f, 1.71f, 1.93f},
                                     {1.27f, 1.29f, 1.72f, 1.80f, 2.34f, 2.64f}, {1.65f, 1.65f, 2.21f, 2.23f, 0.f, 0.f}};
    const int rows = p.M <= 48 ? (p.M - 1) / 8 : p.M <= 56 ? 6 : 7;
    const int tiles = ceil_div(p.N, cols);
    const int waves = skinny::ring_waves(tiles * split);
    const float rounds = (float)ceil_div(tiles * split, 256);
    const float m = (float)p.M, n = (float)p.N;
    float us = 2.8f + (float)p.K * n * 3.44e-8f;
    us += (float)ceil_div(units_per_slice, waves) * unit[cols / 32 - 1][rows] * (waves == 4 ? 0.52f : 1.f) * rounds;
    us += 3.3e-4f * (m < 4.f ? 4.f : m) * (float)cols * rounds;
    if (split == 2 && ring_slot_bytes(p) <= kSlotBytes)
        us += 0.7f + 0.004f * (float)tiles;
    else if (split > 1)
        us += 1.6f + 0.1f * (float)split + 4.5e-5f * m * (float)(cols * split) + 1.96e-6f * m * n * (float)split;
    return us;
}

// Fills what the plan leaves open: the width of a workgroup, the number of K slices, or both.
void ring_make_plan(const Problem &p, SkinnyPlan &plan)
{
    const int units = p.K / skinny::kUnitK;
    const bool any_width = plan.cols_per_wg == 0;
    const bool any_split = plan.split_k <= 0;
    float best = 0.f;
    SkinnyPlan choice = plan;
    choice.split_k = 0;
    for (int cols = any_width ? 32 : plan.cols_per_wg; cols <= (any_width ? 128 : plan.cols_per_wg); cols += 32) {
        const int tiles = ceil_div(p.N, cols);
        // Automatic slices: as long as every slice has a workgroup on a compute unit of its own and its wavefronts a unit
        // each; more never paid.  Their partial sums fit the static scratch block.
        for (int asked = any_split ? 1 : plan.split_k; asked <= (any_split ? 16 : plan.split_k); ++asked) {
            const int ups = ceil_div(units, asked < units ? asked : units);
            const int split = ceil_div(units, ups);
            if (!ring_width(p, cols, split))
                continue;
            if (any_split && asked > 1 &&
                (split != asked || tiles * split > 256 || ups < 8 ||
                 (long long)split * p.M * p.N * (long long)sizeof(float) > (long long)(GPTQ_STATIC_SCRATCH_BYTES - kCounterBytes)))
                continue;
            const float us = ring_estimate(p, cols, split, ups);
            if (choice.split_k == 0 || us < best) {
                best = us;
                choice.cols_per_wg = cols;
                choice.split_k = split;
                choice.units_per_slice = ups;
            }
        }
    }
    plan = choice;
}

}  // namespace

void skinny_make_plan(const Problem &p, SkinnyPlan &plan)
{
    const int launch_m = rows_of_launch(p.M);
    const int rows = 16 * row_blocks(launch_m);
    const int total_units = ceil_div(p.K, skinny::kUnitK);
    const int asked = plan.cols_per_wg;
    const bool any_width = !ring_width(p, asked, plan.split_k);
    // 256 columns, from groups of 128 k on: on request, above 32 rows, and up to 16 rows beyond 65536 columns.  The last as it
    // was before there was the ring, whose unsplit workgroups are ahead there as well (128 columns: 4096x98304 at M = 2 and 16
    // 44.8 us, 38.1 and 49.0, 39.3; 8192x131072 104, 106 and 126, 107; 96 columns: 4096x66560 30.9, 27.3 and 38.7, 30.5; behind
    // on 4096x131072 at M = 2 56.6, 62.4 and 1024x196608 at M = 16 23.4, 24.6): what gemm_static refuses for its partial sums
    // stays refused.  Up to 65536 columns the ring (8192x57344: M = 16 53 us, 48; level at two to four rows).
    const bool ring = ring_supported(p) && (!any_width || p.M <= kRingWideMaxM);
    const bool wide = p.group_size >= skinny::kUnitK &&
                      (asked == 256 ||
                       (any_width && (rows > 32 ? !ring && ceil_div(p.N, 256) >= 192 : rows == 16 && p.N > 65536)));
    if (ring && !wide) {
        if (any_width)
            plan.cols_per_wg = 0;
        ring_make_plan(p, plan);
        return;
    }
    plan.cols_per_wg = wide ? 256 : 64;
    // where the activations of a slice are staged in LDS (wide tiles, more than 32 rows) they must fit
    const bool direct = plan.cols_per_wg <= 128;
    int max_units = direct ? total_units : kMaxActivationLdsBytes / (rows * 2) / skinny::kUnitK;
    if (max_units < 1)
        max_units = 1;
    const int tiles_n = ceil_div(p.N, plan.cols_per_wg);
    int ups;
    if (plan.split_k > 0) {
        ups = ceil_div(total_units, plan.split_k < total_units ? plan.split_k : total_units);
    } else {
        // One workgroup per compute unit is the target (measured: 192..344 unsplit workgroups beat any split
        // of the same layer, and narrow layers want tiles * split = 256) - but the fp32 partial sums that the
        // slices exchange through scratch (8 bytes per slice and output: written once, read once) may not
        // exceed half of the packed weight bytes (K*N/2), or they, not the weights, set the time:
        // split * M * N * 8 <= K * N / 4 (measured on 4096x4096 at 24-32 rows: four slices 8.6-9.1 us, two
        // slices 9.7-10.5).  Slices are whole multiples of `quantum` units.
        int max_split = p.K / (32 * launch_m);
        if (max_split < 1)
            max_split = 1;
        int split = (256 + tiles_n / 2) / tiles_n;
        // A few workgroups more than compute units is the worst case (four-wavefront workgroups, some units with
        // two of them): 160 tiles x 2 slices on 8192x10240 measured 15.2 us at M = 2 against 13.4 unsplit.
        if (tiles_n > 128)
            split = 1;
        if (plan.cols_per_wg == 256) {
            // wide tiles (very wide layers): eight slices, within a quarter of the weight bytes for the partial
            // sums (8192x57344 at M = 2: 46.1 us with eight slices, 49.9 with four)
            split = 8;
            max_split = p.K / (64 * launch_m);
            if (max_split < 1)
                max_split = 1;
        }
        if (split > max_split)
            split = max_split;
        if (split < 1)
            split = 1;
        // narrow tiles: one unit per wavefront and turn
        const int quantum = plan.cols_per_wg == 64 ? waves_of(tiles_n, split, 1, row_blocks(launch_m)) : 1;
        ups = ceil_div(ceil_div(total_units, split), quantum) * quantum;
        if (ups > total_units)
            ups = total_units;
    }
    if (ups > max_units)
        ups = max_units;
    if (ups < 1)
        ups = 1;
    plan.units_per_slice = ups;
    plan.split_k = ceil_div(total_units, ups);
}

bool skinny_scratch_optional(const Problem &p, const SkinnyPlan &plan)
{
    return plan.cols_per_wg != 256 && (p.M <= 32 || (ring_supported(p) && ring_width(p, plan.cols_per_wg, plan.split_k)));
}

size_t skinny_workspace_bytes(const Problem &p, const SkinnyPlan &plan)
{
    if (plan.serial)
        return 0;
    size_t bytes = kCounterBytes;
    if (plan.split_k > 1)
        bytes += (size_t)plan.split_k * rows_of_launch(p.M) * p.N * sizeof(float);
    return bytes;
}

hipError_t launch_skinny(const Problem &p, const SkinnyPlan &plan, void *workspace, void *slots, hipStream_t stream)
{
    unsigned char *ws = static_cast<unsigned char *>(workspace);
    const int wn = plan.cols_per_wg / skinny::kCols;
    const bool ring = ring_supported(p) && ring_width(p, plan.cols_per_wg, plan.split_k);
    for (int m0 = 0; m0 < p.M; m0 += kRowsPerLaunch) {
        skinny::Args a;
        a.x = p.x + (size_t)m0 * p.K;
        a.qweight = p.qweight;
        a.qzeros = p.qzeros;
        a.scales = p.scales;
        a.g_idx = nullptr;
        a.groups = 0;
        a.row_tiles = 1;
        a.out = p.out + (size_t)m0 * p.N;
        a.counters = reinterpret_cast<unsigned *>(ws);
        a.partial = ws ? reinterpret_cast<float *>(ws + kCounterBytes) : nullptr;
        a.M = (p.M - m0) < kRowsPerLaunch ? (p.M - m0) : kRowsPerLaunch;
        a.K = p.K;
        a.N = p.N;
        a.units_per_group = p.group_size >= skinny::kUnitK ? p.group_size / skinny::kUnitK : 1;
        a.unit_group_shift = -1;
        for (int sh = 0; sh < 20; ++sh)
            if ((1 << sh) == a.units_per_group)
                a.unit_group_shift = sh;
        a.tiles_n = ceil_div(p.N, plan.cols_per_wg);
        a.split_k = plan.split_k;
        a.units_per_slice = plan.units_per_slice;
        a.total_units = ceil_div(p.K, skinny::kUnitK);
        a.slots = nullptr;
        a.serial_slices = 0;

        const int tm = row_blocks(a.M);
        const int rows = 16 * tm;
        const int gpu = p.group_size >= skinny::kUnitK ? 1 : skinny::kUnitK / p.group_size;
        const bool tail = p.K % skinny::kUnitK != 0;
        hipError_t err;
        if (ring || (wn != 4 && tm <= 2 && !tail)) {  // (or the rest of a batch of more than 64 rows)
            if (plan.serial && plan.split_k > 1) {  // (columns of its own whatever the sliced plan has)
                a.serial_slices = plan.split_k;
                a.split_k = 1;
                a.tiles_n = ceil_div(p.N, a.M > kRingWideMaxM ? 32 : skinny::kCols);
            } else if (plan.split_k == 2 && ring_slot_bytes(p) <= kSlotBytes) {
                a.slots = static_cast<unsigned long long *>(slots);
            }
            const bool streamed = tm == 1 && stream_weights(p);  // (more rows are not bound by the weights)
            err = gpu == 1   ? skinny::launch_ring<1>(a, plan.cols_per_wg, streamed, stream)
                  : gpu == 2 ? skinny::launch_ring<2>(a, plan.cols_per_wg, streamed, stream)
                             : skinny::launch_ring<4>(a, plan.cols_per_wg, streamed, stream);
            if (err != hipSuccess)
                return err;
            continue;
        }
        // 64-column workgroups read the activations straight from global memory
        const size_t xs = wn == 1 ? 0 : (size_t)rows * plan.units_per_slice * skinny::kUnitK * sizeof(half_t);
        const int waves = waves_of(a.tiles_n, a.split_k, wn, tm);
        const size_t red = (size_t)waves * rows * skinny::kCols * sizeof(float);  // [waves/wn][rows][64*wn]
        const size_t lds = xs > red ? xs : red;
        if (tail) {
            if (wn != 1 || tm > 2 || gpu == 1)
                return hipErrorInvalidValue;  // refused by skinny_supported / skinny_make_plan
            if (plan.serial)
                err = gpu == 2 ? launch_tail<2, true>(a, tm, waves, lds, stream)
                               : launch_tail<4, true>(a, tm, waves, lds, stream);
            else
                err = gpu == 2 ? launch_tail<2, false>(a, tm, waves, lds, stream)
                               : launch_tail<4, false>(a, tm, waves, lds, stream);
        } else if (gpu > 1 || (wn != 1 && wn != 4)) {
            return hipErrorInvalidValue;  // refused by skinny_supported / skinny_make_plan
        } else if (wn == 4) {
            err = tm == 2   ? launch_tm<2, 4, 4>(a, lds, stream)
                  : tm == 4 ? launch_tm<4, 4, 4>(a, lds, stream)
                  : stream_weights(p) ? launch_tm<1, 4, 4, 1, false, false, true>(a, lds, stream)
                                      : launch_tm<1, 4, 4>(a, lds, stream);
        } else {
            err = launch_tm<4, 1, 4>(a, lds, stream);
        }
        if (err != hipSuccess)
            return err;
    }
    return hipSuccess;
}

}  // namespace gptq
