// Host side of the mid-batch streaming MFMA kernel: support check, launch plan, scratch sizing, dispatch.
#include "mid_kernel.h"

namespace gptq {

namespace {

constexpr size_t kCounterBytes = 256 * 1024;  // same fixed counter area as the other kernels
constexpr int kMaxColumnTiles = (int)(kCounterBytes / sizeof(unsigned));

int ceil_div(int a, int b)
{
    return (a + b - 1) / b;
}

// 32-row blocks of a workgroup's tile.
int row_blocks(int M)
{
    return M <= 32 ? 1 : M <= 64 ? 2 : M <= 96 ? 3 : 4;
}

template <int TMB, int NB, int WAVES, int DEPTH = 2>
hipError_t launch_one(const mid::Args &a, hipStream_t stream)
{
    auto kernel = mid::mid_kernel<TMB, NB, WAVES, DEPTH>;
    const size_t lds = (size_t)WAVES * DEPTH * (32 * TMB) * 128;
    if (lds > 48 * 1024) {
        hipError_t err = hipFuncSetAttribute(reinterpret_cast<const void *>(kernel),
                                             hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (err != hipSuccess)
            return err;
    }
    hipLaunchKernelGGL(kernel, dim3((unsigned)(a.tiles_n * a.split_k)), dim3(64 * WAVES), lds, stream, a);
    return hipGetLastError();
}

// 33-64 rows on 128-column tiles: whether four wavefronts on the pinned loop are faster than eight, two per SIMD, on the
// plain one.  They are on slices of up to 96 stages; deeper ones are bound by the load path, which eight keep fuller, and
// slices of less than 32 leave too little between the prologue and the exchange.  Eight wavefronts against four, unsplit,
// M = 33 / 48 / 64:  2048x28672 17.8 / 18.1 / 18.6 us, 16.3 / 16.7 / 17.3; 6144x57344 level; 8192x28672 43.8 / 44.8 / 46.3,
// 45.8 / 46.0 / 47.0; 8192x57344 87.1 / 88.2 / 90.5, 94.5 / 92.2 / 93.0.  In slices:  16 stages 28672x1024 26.3 / 32.4 / 38.6,
// 29.5 / 32.4 / 37.4 and 16384x2048 22.6 / 25.9 / 29.7, 24.9 / 27.6 / 31.1; 28 to 30 level; 64 stages 16384x8192
// 33.9 / 35.6 / 37.8, 32.8 / 34.6 / 37.4; 112 stages 28672x8192 2-5 % for eight.
bool pinned_on_wide_tiles(const MidPlan &plan)
{
    return plan.stages_per_slice <= 96 && (plan.split_k == 1 || plan.stages_per_slice >= 32);
}

}  // namespace

bool mid_supported(const Problem &p)
{
    if (p.g_idx != nullptr || p.M < 1 || p.M > kMidMaxM || p.N < 8 || p.K % mid::kStageK != 0 ||
        p.group_size % mid::kStageK != 0 || ceil_div(p.N, 64) > kMaxColumnTiles)
        return false;
    // the kernel divides stage numbers by the stages per group with one multiply-high, which is exact while
    // stages * stages per group stays below 2^32
    return (long long)(p.K / mid::kStageK) * (p.group_size / mid::kStageK) < (1ll << 31);
}

void mid_make_plan(const Problem &p, MidPlan &plan)
{
    const int tmb = row_blocks(p.M);
    const int total = p.K / mid::kStageK;
    // four row blocks leave registers for two n-blocks only; three have room for four, which gained on layers of 160-256
    // such tiles only (4096x22016 at M = 77 29.4 us; 34.6 with two, 33.7 on the big-tile kernel) and lost 40 % elsewhere
    if (tmb >= 3)
        plan.cols_per_wg = 64;
    if (plan.cols_per_wg != 64 && plan.cols_per_wg != 128) {
        // 128-column tiles where they alone give most compute units a workgroup, or where K is so deep that the
        // exchange of a few more slices is cheap next to the loop (28672x8192 at 64 rows: 50.1 us with 64 tiles
        // in four slices, 54.2 with 128 tiles in two); else 64
        const int tiles128 = ceil_div(p.N, 128);
        plan.cols_per_wg = (tiles128 >= 160 || (tiles128 <= 64 && p.K >= 16384)) ? 128 : 64;
    }
    const int tiles_n = ceil_div(p.N, plan.cols_per_wg);
    int split = plan.split_k;
    if (split <= 0) {
        // one workgroup per compute unit (their activation rings fill its LDS: workgroups beyond 256 wait for a
        // second round); a slice keeps at least eight stages, or sixteen up to 64 rows
        split = 256 / tiles_n;
        const int max_split = total / (tmb <= 2 ? 16 : 8);
        if (split > max_split)
            split = max_split;
        if (split < 1)
            split = 1;
    }
    if (split > total)
        split = total;
    const int sps = ceil_div(total, split);
    plan.stages_per_slice = sps;
    plan.split_k = ceil_div(total, sps);
}

// A fixed part, the stages that one wavefront walks in every round of workgroups, and the exchange: least squares over the
// automatic plans of 134 layers (K 1024-28672, N 1536-57344, groups of 128), 5-6 % rms.
double mid_estimate_us(const Problem &p, const MidPlan &plan)
{
    const double rounds = ceil_div(ceil_div(p.N, plan.cols_per_wg) * plan.split_k, 256);
    const double partial_mb = (double)plan.split_k * p.M * p.N * sizeof(float) / 1e6;
    const bool split = plan.split_k > 1;
    if (plan.cols_per_wg == 64)
        return 3.5 + 0.71 * ceil_div(plan.stages_per_slice, 4) * rounds + 2.7 * (rounds - 1.0) +
               (split ? 2.0 + 0.04 * plan.split_k + 1.1 * partial_mb : 0.0);
    if (pinned_on_wide_tiles(plan))
        return 7.1 + 1.09 * ceil_div(plan.stages_per_slice, 4) * rounds + 5.8 * (rounds - 1.0) +
               (split ? 0.8 * plan.split_k + 0.7 * partial_mb : 0.0);
    return 11.0 + 2.09 * ceil_div(plan.stages_per_slice, 8) * rounds + 8.9 * (rounds - 1.0) +
           (split ? 0.4 * plan.split_k + 1.2 * partial_mb : 0.0);
}

size_t mid_workspace_bytes(const Problem &p, const MidPlan &plan)
{
    size_t bytes = kCounterBytes;
    if (plan.split_k > 1)
        bytes += (size_t)plan.split_k * p.M * p.N * sizeof(float);
    return bytes;
}

hipError_t launch_mid(const Problem &p, const MidPlan &plan, void *workspace, hipStream_t stream)
{
    unsigned char *ws = static_cast<unsigned char *>(workspace);
    mid::Args a;
    a.x = p.x;
    a.qweight = p.qweight;
    a.qzeros = p.qzeros;
    a.scales = p.scales;
    a.out = p.out;
    a.counters = reinterpret_cast<unsigned *>(ws);
    a.partial = reinterpret_cast<float *>(ws + kCounterBytes);
    a.M = p.M;
    a.K = p.K;
    a.N = p.N;
    const uint32_t stages_per_group = (uint32_t)(p.group_size / mid::kStageK);
    a.group_mul = stages_per_group == 1 ? 0u : (uint32_t)(0x100000000ull / stages_per_group) + 1u;
    a.group_one = stages_per_group == 1 ? 1u : 0u;
    a.tiles_n = ceil_div(p.N, plan.cols_per_wg);
    a.split_k = plan.split_k;
    a.stages_per_slice = plan.stages_per_slice;
    a.total_stages = p.K / mid::kStageK;
    const int tmb = row_blocks(p.M);
    if (plan.cols_per_wg == 128) {
        if (tmb == 1)
            return launch_one<1, 4, 8>(a, stream);
        if (tmb == 2)
            return pinned_on_wide_tiles(plan) ? launch_one<2, 4, 4, 3>(a, stream) : launch_one<2, 4, 8>(a, stream);
        return hipErrorInvalidValue;  // refused by mid_make_plan
    }
    if (tmb == 1)
        return launch_one<1, 2, 8>(a, stream);
    // 33-64 rows: four wavefronts on the pinned loop against eight, two per SIMD, on the plain one.  M = 40 and 64:
    // 4096x12288 15.6 us -> 14.0, 15.9 -> 15.3; 11008x4096 15.9 -> 15.0, 18.1 -> 17.0; 8192x10240 23.7 -> 22.1, 26.5 -> 26.0.
    if (tmb == 2)
        return launch_one<2, 2, 4, 3>(a, stream);
    // 65-96 rows: three row blocks leave LDS for a third stage of activations.  With four blocks as above 96 rows:
    // 8192x10240 at M = 77 39.3 us -> 31.0, 8192x8192 31.3 -> 25.0.
    if (tmb == 3)
        return launch_one<3, 2, 4, 3>(a, stream);
    return launch_one<4, 2, 4>(a, stream);
}

}  // namespace gptq
