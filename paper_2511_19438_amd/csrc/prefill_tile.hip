// Instantiates the MFMA kernels for ONE tile configuration (GPTQ_PREFILL_TILE, set on the compiler
// command line) so that the configurations compile in parallel.
#include "prefill_kernel.h"

#ifndef GPTQ_PREFILL_TILE
#error "compile with -DGPTQ_PREFILL_TILE=<1|3|5|8|9|10|11|12|13|14>"
#endif

namespace gptq {
namespace prefill {

template <int TILE>
hipError_t launch_tile(const Args &a, int mode, int kw, hipStream_t stream);

namespace {

// rows x columns per workgroup, wavefront grid, k per stage, stage buffers in the LDS ring - of one wavefront group, and of
// each of two
#if GPTQ_PREFILL_TILE == 1
constexpr int BM = 256, BN = 256, WM = 1, WN = 4, BK = 64, NBUF = 3, NBUF2 = 0;
#elif GPTQ_PREFILL_TILE == 3
constexpr int BM = 128, BN = 128, WM = 2, WN = 2, BK = 64, NBUF = 3, NBUF2 = 3;
#elif GPTQ_PREFILL_TILE == 5
constexpr int BM = 64, BN = 128, WM = 1, WN = 4, BK = 64, NBUF = 4, NBUF2 = 4;
#elif GPTQ_PREFILL_TILE == 8
constexpr int BM = 128, BN = 256, WM = 1, WN = 4, BK = 64, NBUF = 3, NBUF2 = 3;
// tile 8 where other rows fit the batch better
#elif GPTQ_PREFILL_TILE == 9
constexpr int BM = 96, BN = 256, WM = 1, WN = 4, BK = 64, NBUF = 3, NBUF2 = 3;
#elif GPTQ_PREFILL_TILE == 10
constexpr int BM = 80, BN = 256, WM = 1, WN = 4, BK = 64, NBUF = 4, NBUF2 = 4;
#elif GPTQ_PREFILL_TILE == 11
constexpr int BM = 112, BN = 256, WM = 1, WN = 4, BK = 64, NBUF = 3, NBUF2 = 3;
// tile 5 where they do
#elif GPTQ_PREFILL_TILE == 12
constexpr int BM = 80, BN = 128, WM = 1, WN = 4, BK = 64, NBUF = 4, NBUF2 = 5;
#elif GPTQ_PREFILL_TILE == 13
constexpr int BM = 96, BN = 128, WM = 1, WN = 4, BK = 64, NBUF = 4, NBUF2 = 4;
#elif GPTQ_PREFILL_TILE == 14
constexpr int BM = 112, BN = 128, WM = 1, WN = 4, BK = 64, NBUF = 4, NBUF2 = 4;
#else
#error "unknown tile id"
#endif

template <typename Kernel>
hipError_t launch(Kernel kernel, Args a, size_t lds, bool may_split, hipStream_t stream, int kw = 1)
{
    a.tiles_m = (a.M + BM - 1) / BM;
    a.tiles_n = (a.N + BN - 1) / BN;
    const int total = a.tiles_m * a.tiles_n;
    // the requested split, in whole stages of this tile's BK
    const int all_stages = (a.K + BK - 1) / BK;
    int split = (may_split && a.split_k > 1) ? (a.split_k < all_stages ? a.split_k : all_stages) : 1;
    a.stages_per_slice = (all_stages + split - 1) / split;
    split = (all_stages + a.stages_per_slice - 1) / a.stages_per_slice;
    a.split_k = split;
    if (a.serial_slices > 1)
        a.stages_per_slice = (all_stages + a.serial_slices - 1) / a.serial_slices;  // of the workgroup's own slices
    const unsigned grid = 8u * (unsigned)((total + 7) / 8) * (unsigned)split;
    if (lds > 48 * 1024) {
        hipError_t err = hipFuncSetAttribute(reinterpret_cast<const void *>(kernel),
                                             hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (err != hipSuccess)
            return err;
    }
    hipLaunchKernelGGL(kernel, dim3(grid), dim3(kThreads * kw), lds, stream, a);
    return hipGetLastError();
}

}  // namespace

template <>
hipError_t launch_tile<GPTQ_PREFILL_TILE>(const Args &a, int mode, int kw, hipStream_t stream)
{
#if GPTQ_PREFILL_TILE != 1
    if (kw == 2 && mode == kGroupPerStage)
        return launch(prefill_pipelined_kernel<BM, BN, WM, WN, BK, NBUF2, false, 2>, a,
                      2 * (size_t)NBUF2 * StageLayout<BM, BN, BK, false>::BYTES, true, stream, 2);
    if (kw == 2 && mode == kGroupPerHalf)
        return launch(prefill_pipelined_kernel<BM, BN, WM, WN, BK, NBUF2, true, 2>, a,
                      2 * (size_t)NBUF2 * StageLayout<BM, BN, BK, true>::BYTES, true, stream, 2);
#endif
    if (kw != 1)
        return hipErrorInvalidValue;
#if GPTQ_PREFILL_TILE == 5
    if (a.serial_slices > 1 && mode == kGroupPerStage)
        return launch(prefill_pipelined_kernel<BM, BN, WM, WN, BK, NBUF, false, 1, true>, a,
                      (size_t)NBUF * StageLayout<BM, BN, BK, false>::BYTES, false, stream);
    if (a.serial_slices > 1 && mode == kGroupPerHalf)
        return launch(prefill_pipelined_kernel<BM, BN, WM, WN, BK, NBUF, true, 1, true>, a,
                      (size_t)NBUF * StageLayout<BM, BN, BK, true>::BYTES, false, stream);
#endif
    if (a.serial_slices > 1)
        return hipErrorInvalidValue;
    if (mode == kGroupPerStage)
        return launch(prefill_pipelined_kernel<BM, BN, WM, WN, BK, NBUF>, a,
                      (size_t)NBUF * StageLayout<BM, BN, BK, false>::BYTES, true, stream);
    if (mode == kGroupPerHalf)
        return launch(prefill_pipelined_kernel<BM, BN, WM, WN, BK, NBUF, true>, a,
                      (size_t)NBUF * StageLayout<BM, BN, BK, true>::BYTES, true, stream);
#if GPTQ_PREFILL_TILE == 3
    const size_t lds = 2 * (size_t)BM * 64 * sizeof(half_t);
    if (mode == kGroupPerRow)
        return launch(prefill_general_kernel<BM, BN, WM, WN, kGroupPerRow>, a, lds, false, stream);
    if (mode == kActOrder)
        return launch(prefill_general_kernel<BM, BN, WM, WN, kActOrder>, a, lds, false, stream);
#endif
    return hipErrorInvalidValue;
}

}  // namespace prefill
}  // namespace gptq
