// Host side of the MFMA kernel: tile selection and dispatch.
#include "gptq_w4a16.h"
#include "prefill_kernel.h"

namespace gptq {

namespace prefill {
template <int TILE>
hipError_t launch_tile(const Args &a, int mode, int kw, hipStream_t stream);
template <> hipError_t launch_tile<1>(const Args &, int, int, hipStream_t);
template <> hipError_t launch_tile<3>(const Args &, int, int, hipStream_t);
template <> hipError_t launch_tile<5>(const Args &, int, int, hipStream_t);
template <> hipError_t launch_tile<8>(const Args &, int, int, hipStream_t);
template <> hipError_t launch_tile<9>(const Args &, int, int, hipStream_t);
template <> hipError_t launch_tile<10>(const Args &, int, int, hipStream_t);
template <> hipError_t launch_tile<11>(const Args &, int, int, hipStream_t);
template <> hipError_t launch_tile<12>(const Args &, int, int, hipStream_t);
template <> hipError_t launch_tile<13>(const Args &, int, int, hipStream_t);
template <> hipError_t launch_tile<14>(const Args &, int, int, hipStream_t);
}  // namespace prefill

namespace {

struct TileShape {
    int bm, bn;
    bool may_split;  // K slices pay only where a thread holds few accumulators (the combine moves them all)
};
// by tile id (1, 3, 5, 8: see the plan documentation in the public header; the other ids up to 10 belonged to
// layouts that measurement retired - 2x2 wavefront grids, 32-k stages, a 32-row tile - and are refused; tiles 5 and 8 run
// with other rows where those fit the batch better, see row_choice)
constexpr TileShape kTiles[11] = {{0, 0, false},   {256, 256, false}, {0, 0, false}, {128, 128, true},
                                  {0, 0, false},   {64, 128, true},   {0, 0, false}, {0, 0, false},
                                  {128, 256, true}, {0, 0, false},    {0, 0, false}};
constexpr int kNumTiles = 10;
constexpr int kComputeUnits = 256;
constexpr size_t kCounterBytes = 256 * 1024;  // same fixed counter area as the other kernels
constexpr int kMaxSplit = 32;
// Rows that the workgroups of tiles 5 and 8 may have; the first is the tile's own.
constexpr int kRows[2][4] = {{64, 80, 96, 112}, {128, 112, 96, 80}};

int ceil_div_i(int a, int b)
{
    return (a + b - 1) / b;
}

// Rows of the batch, and those that only fill up the last workgroups.
int padded(const Problem &p, int rows)
{
    return ceil_div_i(p.M, rows) * rows;
}

// Rows number `i` of a workgroup of tile `t`, 0 if they are not for the problem: another number than the tile's own has to pad
// the batch less - or, on tile 5, as little, which makes fewer and larger tiles -, so that the scratch of slices is bounded by
// that of the tile's own rows.
// us, the tiles' own rows -> these: M = 77 8192x10240 30.1 -> 25.6 (80x128), 8192x57344 97.0 -> 92.0 (80x256), 28672x8192
// 61.7 -> 54.2 (80x128); 88x1664x25448 25.0 -> 18.4 (96x128); 100x4096x22016 39.5 -> 30.8 (112x128); 333x2752x6888 with groups
// of 32 31.9 -> 25.1 (96x128, unsplit; the others in two slices and more); 266x8448x28344 237 -> 175.
int row_choice(const Problem &p, int t, int i)
{
    const int own = kTiles[t].bm;
    if (t != 5 && t != 8)
        return i == 0 ? own : 0;
    const int rows = kRows[t == 8][i];
    return i == 0 || padded(p, rows) < padded(p, own) || (t == 5 && padded(p, rows) == padded(p, own)) ? rows : 0;
}

// What the estimate of rows that pad as little as the tile's own has to be multiplied with before it may choose them: the HALF
// variant on two of 96 rows (129-192 rows) is estimated about 10 % low against the 96x256 tile.  150 layers with groups of 32
// to 128 whose plan the 96 rows change at 129-192 rows: 41 are 8 % ahead by the estimate, all of them 7 % and more by the
// clock (174x2496x15488 with groups of 32 30.0 -> 24.7 us, 161x1984x13680 27.1 -> 20.6, 190x1344x13704 18.6 -> 15.4); 24 of the
// others lose 2-7 % (161x2912x48552 70.3, 75.7; 176x1024x47464 28.6, 30.3).  With the factor, 150 other layers whose plan the
// 96 rows change: 1.16 times as fast (geometric mean), 4 % at least.
double tie_factor(const Problem &p, int t, int rows, bool half)
{
    return half && p.M <= 192 && rows != kTiles[t].bm && padded(p, rows) == padded(p, kTiles[t].bm) ? 1.08 : 1.0;
}

// The output tiles of a tile shape, and how many of them the busiest XCD has (tile_of_workgroup).
struct Grid {
    int tiles, per_xcd;
};

Grid grid_of(const Problem &p, int t, int rows)
{
    const int tiles = ceil_div_i(p.M, rows) * ceil_div_i(p.N, kTiles[t].bn);
    return {tiles, ceil_div_i(tiles, 8)};
}

// K slices: how many, as whole stages make of `split`, and the stages of each.
struct Slices {
    int count, stages;
};

Slices slices_of(const Problem &p, int split)
{
    const int stages = ceil_div_i(p.K, 64);
    const int each = ceil_div_i(stages, split < 1 ? 1 : split);
    return {ceil_div_i(stages, each), each};
}

// Wavefront groups that share a tile of 128x256, each with half of the K slice: two where that gives every compute
// unit its two wavefronts per SIMD and otherwise it would have one (M = 512: 4096x12288 73.5 -> 58.0 us, 28672x8192
// in two slices 266 -> 226; M = 128, 8192x57344 152 -> 126).  With more workgroups than compute units two of them
// meet there anyway (4096x22016 at M = 512, 344 workgroups: 104 us with one group, 114 with two), and slices of a few
// stages do not earn the sum through LDS (4096x4096 at M = 256, eight stages: 34.2, 35.3).
int k_groups_of_tile8(const Grid &grid, const Slices &slices)
{
    return grid.tiles * slices.count <= kComputeUnits && slices.stages > 8 ? 2 : 1;
}

// The same for the 128x128 and 64x128 tiles, where no compute unit of the busiest XCD has more than one workgroup (the
// rings of two groups fill its LDS) and a slice has enough stages.  With one group against two: 64x128 tile, 4096x4096 at
// M = 512 32.9 -> 28.0 us, at M = 100 29.3 -> 24.9 (in four slices of 16 stages 16.1 -> 15.3), 28672x4096 at M = 100
// 183 -> 138; 128x128 tile, 4096x12288 at M = 256 61.2 -> 43.4, 11008x4096 at M = 512 147 -> 99.  Two groups fill the chip
// without the partial sums of two slices in scratch: 4096x4096 at M = 256 20.7 us in four slices -> 19.5 in two.
int k_groups_of_small_tile(const Grid &grid, const Slices &slices)
{
    return grid.per_xcd * slices.count <= kComputeUnits / 8 && slices.stages >= 16 ? 2 : 1;
}

int k_groups(int t, const Grid &grid, const Slices &slices)
{
    return t == 8 ? k_groups_of_tile8(grid, slices) : t == 3 || t == 5 ? k_groups_of_small_tile(grid, slices) : 1;
}

// Estimated duration (microseconds) of the pipelined kernel with tile `t`, the rows to a workgroup of `c`, and K slices.  A
// workgroup walks its stages at a pace set by instruction issue and latency: alone on a compute unit it leaves most of it
// idle, and co-resident workgroups slow each other down by less than their number.  What counts is the busiest compute unit of
// the busiest XCD: a tile's slices share an XCD and the tiles are dealt out in eight equal ranges (tile_of_workgroup), so 50
// tiles in five slices are 35 workgroups on 32 compute units there, not 250 on 256 (28160x2432 at M = 385: 136 us; 94 in
// six slices of fewer tiles).  The slices' exchange costs a fixed part, a part per slice that the last arriver of a tile
// reads, and the traffic of all partial tiles.  Constants: least squares over 2.0 k measured plans of 110 random problems (M
// 65-1100, K 1024-28672, N 1024-57344, a fifth of them with groups of 32; 4-8 % rms), whose picks are 0.6 % behind the best of
// every problem on average, 10 % at worst.  Tile 1 and the pairs of tile 8, whose pace is that of a full chip under sustained
// load, keep the ratio that 1.9 k problems of M 129-2048 had given (777x8192x57344 814 -> 744 us, 129x8192x57344 210 -> 187).
struct Pace {
    int tile, rows;
    double resident[3];  // one stage with that many workgroups of one wavefront group on a compute unit
    int most;            // workgroups that fit one
    double fixed;
    // Two wavefront groups: a pair of stages with up to half of the compute units busy, what it takes longer with all of them.
    double pair, pair_full, pair_fixed;
    double split, per_slice, per_mb;
};
constexpr Pace kPaces[] = {
    {1, 256, {}, 1, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0},  // (has a formula of its own)
    {5, 64, {0.385, 0.574, 0.860}, 3, 4.3, 0.567, 0.070, 4.25, 1.0, 0.60, 0.105},
    {5, 80, {0.414, 0.669, 0.0}, 2, 5.0, 0.664, 0.097, 5.1, 0.2, 0.83, 0.200},
    {5, 96, {0.412, 0.705, 0.0}, 2, 5.1, 0.698, 0.102, 5.2, 0.2, 0.90, 0.180},
    {5, 112, {0.397, 0.757, 0.0}, 2, 5.1, 0.761, 0.095, 5.4, 0.5, 0.93, 0.180},
    {3, 128, {0.580, 1.014, 0.0}, 2, 4.4, 1.019, 0.090, 4.4, 1.1, 1.00, 0.140},
    {8, 80, {0.650, 1.060, 0.0}, 2, 5.2, 1.057, 0.282, 5.9, 2.1, 1.38, 0.075},
    {8, 96, {0.800, 1.280, 0.0}, 2, 5.2, 1.162, 0.344, 5.4, 2.4, 1.64, 0.080},
    {8, 112, {0.840, 1.370, 0.0}, 2, 5.2, 1.229, 0.361, 6.0, 2.5, 1.82, 0.082},
    {8, 128, {0.920, 1.500, 0.0}, 2, 5.2, 1.267, 0.354, 6.5, 2.4, 1.79, 0.086}};

const Pace &pace_of(int t, int rows)
{
    const Pace *c = kPaces;
    while (c->tile != t || c->rows != rows)
        ++c;
    return *c;
}

double estimate_us(int t, const Pace &c, const Grid &grid, const Slices &slices, bool half)
{
    const int wgs = grid.tiles * slices.count;
    const int busiest = grid.per_xcd * slices.count;  // workgroups of the busiest XCD, which has 32 compute units
    if (t == 1)  // one workgroup per compute unit, whole rounds
        return ceil_div_i(busiest, 32) * (slices.stages * 1.30 * (half ? 1.16 : 1.0) + 9.9);
    // tile 8 in more workgroups than compute units and K slices: the exchange is not worth it
    if (t == 8 && slices.count > 1 && wgs > kComputeUnits)
        return 1e30;
    const double exchange =
        slices.count > 1 ? c.split + slices.count * c.per_slice + wgs * (double)c.rows * kTiles[t].bn * sizeof(float) / 1e6 * c.per_mb : 0.0;
    const int groups = k_groups(t, grid, slices);
    const double stage_scale = !half ? 1.0 : t == 5 ? (groups == 1 ? 1.25 : 1.22) : t == 3 ? 1.2 : 1.15;  // of the HALF variant
    if (groups == 2) {
        const double full = busiest <= 16 ? 0.0 : busiest >= 32 ? 1.0 : busiest / 16.0 - 1.0;
        return c.pair_fixed + ceil_div_i(slices.stages, 2) * (c.pair + c.pair_full * full) * stage_scale * (busiest > 32 ? 2.0 : 1.0) + exchange;
    }
    const int full = (busiest - 1) / (32 * c.most);  // times that a compute unit is filled up, then the rest
    const int rest = ceil_div_i(busiest - 32 * c.most * full, 32);
    const double stage = full * c.resident[c.most - 1] + (rest > 0 ? c.resident[rest - 1] : 0.0);
    return c.fixed + slices.stages * stage * stage_scale + (t == 8 ? 1.5 * full : 0.0) + exchange;
}

// Partial sums of one K slice, whatever the rows to a workgroup (other rows than the tile's own cover no more in all).
size_t partial_bytes(const Problem &p, int t)
{
    const TileShape &ts = kTiles[t];
    return (size_t)ceil_div_i(p.M, ts.bm) * ceil_div_i(p.N, ts.bn) * ts.bm * ts.bn * sizeof(float);
}

int mode_of(const Problem &p)
{
    if (p.g_idx)
        return prefill::kActOrder;
    // the pipelined kernel moves 16-byte chunks of every operand row: rows of packed zero points (N/8 words)
    // are 16-byte aligned only when N is a multiple of 32; its HALF variant moves them word by word
    if (p.group_size % 64 == 0 && p.N % 32 == 0)
        return prefill::kGroupPerStage;
    return (p.group_size % 32 == 0 && p.K >= 64) ? prefill::kGroupPerHalf : prefill::kGroupPerRow;
}

}  // namespace

bool prefill_pipelined(const Problem &p)
{
    return mode_of(p) == prefill::kGroupPerStage || mode_of(p) == prefill::kGroupPerHalf;
}

bool prefill_supported(const Problem &p)
{
    return p.M >= 1 && p.K % 8 == 0 && p.N % 8 == 0;
}

bool prefill_tile_exists(int tile)
{
    return tile >= 1 && tile <= kNumTiles && kTiles[tile].bm > 0;
}

void prefill_make_plan(const Problem &p, PrefillPlan &plan)
{
    if (!prefill_pipelined(p)) {
        plan.tile = 3;  // the general modes exist for one tile shape only, without a K split
        plan.split_k = 1;
        plan.rows = kTiles[3].bm;
        return;
    }
    const bool tile_given = prefill_tile_exists(plan.tile);
    const bool split_given = plan.split_k >= 1;
    // Few output tiles and a deep K leave most of the chip idle and every workgroup walking all of K: K slices
    // (combined through scratch in slice order) shorten the walk.  Cheapest (tile, split) by the estimate.
    const bool half = mode_of(p) == prefill::kGroupPerHalf;
    double best = 0.0;
    int best_tile = 3, best_split = 1, best_rows = kTiles[3].bm;
    const int stages = ceil_div_i(p.K, 64);
    Slices offered[kMaxSplit];
    int offers = 0;
    for (int split = 1; split <= kMaxSplit && split <= stages / 2 + (stages < 2); ++split) {
        if (split_given && split != (plan.split_k < stages ? plan.split_k : stages))
            continue;
        const Slices slices = slices_of(p, split);
        if (offers == 0 || slices.count != offered[offers - 1].count)
            offered[offers++] = slices;
    }
    for (int t = 1; t <= kNumTiles; ++t) {
        if (kTiles[t].bm == 0 || (tile_given && t != plan.tile))
            continue;
        // (up to 128 rows half of 256 and more are padding.  Slices that a plan asks for went to this tile, whose estimate knows no
        // exchange: 128x8192x8192 in eight 68 us, on the 64x128 tile 34; 113x2432x14080 in four 44, 26; 95x3072x632 in sixteen 74, 16)
        if (t == 1 && !tile_given && p.M <= 128)
            continue;
        const Pace *paces[4];
        Grid grids[4];
        double factors[4];
        int candidates = 0;
        for (int i = 0; i < 4; ++i) {
            const int rows = row_choice(p, t, i);
            if (rows == 0)
                continue;
            factors[candidates] = tie_factor(p, t, rows, half);
            paces[candidates] = &pace_of(t, rows);
            grids[candidates++] = grid_of(p, t, rows);
        }
        const size_t slice_bytes = partial_bytes(p, t);
        for (int o = 0; o < offers; ++o) {
            const Slices slices = offered[o];
            if (!split_given && slices.count > 1 && !kTiles[t].may_split)
                break;
            // (automatic slices stay within the static scratch block, so that gptq_w4a16_gemm_static runs the same plan)
            if (!split_given && slices.count > 1 && kCounterBytes + slices.count * slice_bytes > GPTQ_STATIC_SCRATCH_BYTES)
                break;
            for (int i = 0; i < candidates; ++i) {
                const double us = factors[i] * estimate_us(t, *paces[i], grids[i], slices, half);
                if (best == 0.0 || us < best - 1e-9) {
                    best = us;
                    best_tile = t;
                    best_split = slices.count;
                    best_rows = paces[i]->rows;
                }
            }
        }
    }
    if (best == 0.0) {  // a requested split beyond what the loop offers
        best_tile = tile_given ? plan.tile : 3;
        best_split = split_given ? plan.split_k : 1;
        best_rows = kTiles[best_tile].bm;
        for (int i = 1; i < 4; ++i) {
            const int rows = row_choice(p, best_tile, i);
            if (rows > 0 && padded(p, rows) < padded(p, best_rows))
                best_rows = rows;
        }
    }
    plan.rows = best_rows;
    plan.tile = best_tile;
    plan.split_k = best_split;
}

double prefill_estimate_us(const Problem &p, const PrefillPlan &plan)
{
    return estimate_us(plan.tile, pace_of(plan.tile, plan.rows), grid_of(p, plan.tile, plan.rows), slices_of(p, plan.split_k),
                       mode_of(p) == prefill::kGroupPerHalf);
}

size_t prefill_workspace_bytes(const Problem &p, const PrefillPlan &plan)
{
    if (plan.split_k <= 1 || plan.serial || !prefill_tile_exists(plan.tile))
        return 0;
    return kCounterBytes + plan.split_k * partial_bytes(p, plan.tile);
}

hipError_t launch_prefill(const Problem &p, const PrefillPlan &plan, void *workspace, hipStream_t stream)
{
    prefill::Args a;
    a.x = p.x;
    a.qweight = p.qweight;
    a.qzeros = p.qzeros;
    a.scales = p.scales;
    a.g_idx = p.g_idx;
    a.out = p.out;
    a.M = p.M;
    a.K = p.K;
    a.N = p.N;
    a.group_size = p.group_size;
    a.tiles_m = a.tiles_n = 0;
    a.split_k = (workspace && plan.split_k > 1) ? plan.split_k : 1;
    a.stages_per_slice = 0;
    a.serial_slices = 0;
    a.serial_kw = 1;
    a.counters = reinterpret_cast<unsigned *>(workspace);
    a.partial = workspace ? reinterpret_cast<float *>(static_cast<unsigned char *>(workspace) + kCounterBytes) : nullptr;
    if (a.split_k > 1 && (size_t)ceil_div_i(p.M, plan.rows) *
                               ceil_div_i(p.N, kTiles[plan.tile].bn) >
                             kCounterBytes / sizeof(unsigned))
        a.split_k = 1;  // more tiles than arrival counters: such a problem needs no split anyway
    const int mode = mode_of(p);
    if (plan.serial) {
        a.split_k = 1;
        a.serial_slices = plan.split_k;
        a.serial_kw = k_groups(plan.tile, grid_of(p, plan.tile, plan.rows), slices_of(p, plan.split_k));
        return prefill::launch_tile<5>(a, mode, 1, stream);
    }
    const bool pipelined = mode == prefill::kGroupPerStage || mode == prefill::kGroupPerHalf;
    const int kw = pipelined ? k_groups(plan.tile, grid_of(p, plan.tile, plan.rows), slices_of(p, plan.split_k)) : 1;
    switch (plan.tile) {
    case 1: return prefill::launch_tile<1>(a, mode, 1, stream);
    case 3: return prefill::launch_tile<3>(a, mode, kw, stream);
    case 5:
        return plan.rows == 112  ? prefill::launch_tile<14>(a, mode, kw, stream)
               : plan.rows == 96 ? prefill::launch_tile<13>(a, mode, kw, stream)
               : plan.rows == 80 ? prefill::launch_tile<12>(a, mode, kw, stream)
                                 : prefill::launch_tile<5>(a, mode, kw, stream);
    case 8:
        return plan.rows == 112  ? prefill::launch_tile<11>(a, mode, kw, stream)
               : plan.rows == 96 ? prefill::launch_tile<9>(a, mode, kw, stream)
               : plan.rows == 80 ? prefill::launch_tile<10>(a, mode, kw, stream)
                                 : prefill::launch_tile<8>(a, mode, kw, stream);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace gptq
