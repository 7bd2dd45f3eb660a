// Launches of the small-batch kernel on a ring of LDS slots (ring_kernel.h), one translation unit per GPTQ_RING_GPU:
// quantisation groups per 128 k (1, 2 or 4).
#include "ring_kernel.h"

#ifndef GPTQ_RING_GPU
#error "compile with -DGPTQ_RING_GPU=<quantisation groups per 128-k unit>"
#endif

namespace gptq {
namespace skinny {

namespace {

constexpr int kGpu = GPTQ_RING_GPU;

template <int TM, int LX, int NF, int NH, int WAVES, bool STREAM, bool SERIAL = false>
hipError_t launch_one(const Args &a, hipStream_t stream)
{
    // Slots: what measured best.  32 columns three, 64 and more two (4096x22016 in 96 columns, M = 8: 11.7 us, 12.1 with three),
    // and two beyond 32 rows, whose eight rings would not fit the LDS otherwise.
    constexpr int COLS = 64 * NF + 32 * NH;
    constexpr int DEPTH = COLS == 32 && TM <= 2 ? 3 : 2;
    auto kernel = ring_kernel<TM, LX, NF, NH, WAVES, kGpu, DEPTH, STREAM, SERIAL>;
    constexpr size_t ring = (size_t)WAVES * DEPTH * RingSlot<COLS, LX, kGpu>::BYTES;
    constexpr size_t red = (size_t)WAVES * 16 * TM * COLS * sizeof(float);
    constexpr size_t lds = ring > red ? ring : red;
    static_assert(lds <= 160 * 1024 - 64, "one workgroup fits a compute unit");
    if (lds > 48 * 1024) {
        hipError_t err = hipFuncSetAttribute(reinterpret_cast<const void *>(kernel),
                                             hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (err != hipSuccess)
            return err;
    }
    hipLaunchKernelGGL(kernel, dim3((unsigned)(a.tiles_n * a.split_k)), dim3(64 * WAVES), lds, stream, a);
    return hipGetLastError();
}

template <int TM, int LX, int NF, int NH, bool STREAM>
hipError_t launch(const Args &a, hipStream_t stream)
{
    return ring_waves(a.tiles_n * a.split_k) == 8 ? launch_one<TM, LX, NF, NH, 8, STREAM>(a, stream)
                                                  : launch_one<TM, LX, NF, NH, 4, STREAM>(a, stream);
}

template <int NF, int NH>
hipError_t launch_rows(const Args &a, bool streamed, hipStream_t stream)
{
    if (a.M <= 8)
        return streamed ? launch<1, 1, NF, NH, true>(a, stream) : launch<1, 1, NF, NH, false>(a, stream);
    if (a.M <= 16)
        return streamed ? launch<1, 2, NF, NH, true>(a, stream) : launch<1, 2, NF, NH, false>(a, stream);
    if (a.M <= 24)
        return launch<2, 3, NF, NH, false>(a, stream);
    if (a.M <= 32)
        return launch<2, 4, NF, NH, false>(a, stream);
    if constexpr (NF < 2 && kGpu < 4) {
        if (a.M <= 40)
            return launch<3, 5, NF, NH, false>(a, stream);
        if (a.M <= 48)
            return launch<3, 6, NF, NH, false>(a, stream);
    }
    if constexpr (NF == 0 && kGpu < 4) {
        if (a.M <= 56)
            return launch<4, 7, NF, NH, false>(a, stream);
        if (a.M <= 64)
            return launch<4, 8, NF, NH, false>(a, stream);
    }
    return hipErrorInvalidValue;  // refused by ring_width
}

hipError_t launch_serial(const Args &a, hipStream_t stream)
{
    if (a.M <= 8)
        return launch_one<1, 1, 1, 0, 8, false, true>(a, stream);
    if (a.M <= 16)
        return launch_one<1, 2, 1, 0, 8, false, true>(a, stream);
    if (a.M <= 24)
        return launch_one<2, 3, 1, 0, 8, false, true>(a, stream);
    if (a.M <= 32)
        return launch_one<2, 4, 1, 0, 8, false, true>(a, stream);
    if constexpr (kGpu < 4) {
        if (a.M <= 40)
            return launch_one<3, 5, 1, 0, 8, false, true>(a, stream);
        if (a.M <= 48)
            return launch_one<3, 6, 1, 0, 8, false, true>(a, stream);
        if (a.M <= 56)
            return launch_one<4, 7, 0, 1, 8, false, true>(a, stream);
        if (a.M <= 64)
            return launch_one<4, 8, 0, 1, 8, false, true>(a, stream);
    }
    return hipErrorInvalidValue;  // refused by ring_supported
}

}  // namespace

template <>
hipError_t launch_ring<kGpu>(const Args &a, int cols, bool streamed, hipStream_t stream)
{
    if (a.serial_slices > 1)
        return launch_serial(a, stream);
    switch (cols) {
    case 32: return launch_rows<0, 1>(a, streamed, stream);
    case 64: return launch_rows<1, 0>(a, streamed, stream);
    case 96: return launch_rows<1, 1>(a, streamed, stream);
    case 128: return launch_rows<2, 0>(a, streamed, stream);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace skinny
}  // namespace gptq
