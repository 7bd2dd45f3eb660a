// Standalone int4 unpack and per-group dequantisation kernels for gfx950.
//
// These expose the first stages of the W4A16 GPTQ pipeline (the 4-bit field extraction and
// w = scale * (q - z)) as tensors so that they can be checked bit for bit.  Both are pure
// streaming kernels: one thread owns four (unpack) or eight (dequant) adjacent columns of one packed row
// (128-bit loads of qweight), i.e. 4 x 8 or 8 x 8 weights, and writes them row by row so that a wavefront
// stores 256 B (uint8) or 1 KB (fp16) of each output row contiguously.
#include "kernels.h"

namespace gptq {

namespace {

constexpr int kThreads = 256;

// q_out[k, n] = (qweight[k/8, n] >> 4*(k%8)) & 15
__global__ __launch_bounds__(kThreads) void unpack_qweight_kernel(const uint32_t *__restrict__ qweight,
                                                                   uint8_t *__restrict__ q_out, int rows, int N)
{
    const int quads = N >> 2;
    const long long idx = (long long)blockIdx.x * kThreads + threadIdx.x;
    if (idx >= (long long)rows * quads)
        return;
    const int row = (int)(idx / quads);
    const int n0 = (int)(idx % quads) * 4;
    const uint4 w = *reinterpret_cast<const uint4 *>(qweight + (size_t)row * N + n0);
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        const uint32_t packed = ((w.x >> (4 * j)) & 15u) | (((w.y >> (4 * j)) & 15u) << 8) |
                                (((w.z >> (4 * j)) & 15u) << 16) | (((w.w >> (4 * j)) & 15u) << 24);
        *reinterpret_cast<uint32_t *>(q_out + (size_t)(row * 8 + j) * N + n0) = packed;
    }
}

// z_out[r, n] = (qzeros[r, n/8] >> 4*(n%8)) & 15
__global__ __launch_bounds__(kThreads) void unpack_qzeros_kernel(const uint32_t *__restrict__ qzeros,
                                                                  uint8_t *__restrict__ z_out, long long words)
{
    const long long idx = (long long)blockIdx.x * kThreads + threadIdx.x;
    if (idx >= words)
        return;
    const uint32_t w = qzeros[idx];
    uint2 bytes;
    bytes.x = (w & 15u) | (((w >> 4) & 15u) << 8) | (((w >> 8) & 15u) << 16) | (((w >> 12) & 15u) << 24);
    bytes.y = ((w >> 16) & 15u) | (((w >> 20) & 15u) << 8) | (((w >> 24) & 15u) << 16) | (((w >> 28) & 15u) << 24);
    // word idx of row r covers columns 8*(idx % (N/8)) .. +7 of that row: the flat byte offset is simply 8*idx
    *reinterpret_cast<uint2 *>(z_out + 8 * idx) = bytes;
}

// How the dequantised rows are stored.
enum StorePolicy {
    kPlain = 0,         // through the L2
    kWriteThrough = 1,  // sc1: nothing is left dirty in the L2, the rows stay in the memory-side cache
    kBypass = 2         // non-temporal: past all caches
};
constexpr long long kBypassBytes = 224000000;

// w_out[k, n] = fp16( scales[r(k), n] * (q[k, n] - z[r(k), n]) ): exact integer difference, one fp16 multiply.
//
// Bound by HBM (2.5 bytes per weight, four fifths of them written), so what counts is how the rows are written: a thread
// owns EIGHT adjacent columns of one packed row (two 128-bit loads, one whole zero word), which makes every store 128
// bits and a wavefront's part of a row 1 KB contiguous.  The difference comes from the mantissa of 1024.0: (1024 + q) -
// (1024 + z) in packed halves is exact (and +0 for q = z, as the conversion of an integer 0 is).
//
// The written rows are 80 % of the traffic, and what counts next is whether their reader finds them in the memory-side
// cache (256 MB).  Outputs that hardly fit it go past all caches.  Smaller ones stay in it: bypassing it would make the
// dequantisation itself shorter there, too, but a product that follows longer by more.  Rows that are no whole pieces of
// 64 bytes (N % 32) share lines at their borders, which both other policies write twice: plain stores.  The weights
// alone, and with a product of 16 rows behind them, over a set of layers that exceeds the cache, us with plain /
// non-temporal / write-through stores:
//   4096x4096             9.8 /  7.5 /  8.8    25.8 /  30.4 /  24.8
//   11008x4096           23.1 / 17.8 / 22.4    71.5 /  87.8 /  70.9
//   8192x13312  218 MB   49.9 / 42.2 / 47.9    93.1 /  99.0 /  90.8
//   10368x11200 232 MB   53.0 / 45.0 / 52.0   107.0 / 106.8 / 107.0
//   8192x28672  470 MB  101.5 / 98.6 / 100.5  227.8 / 205.0 / 226.9
//   4096x4528            11.3 / 10.1 / 14.2    28.8 /  34.3 /  29.0
//   8192x28680          111.9 / 122.7 / 130.8 237.4 / 230.4 / 240.5
// (11008x4096 with four columns per thread and plain 64-bit stores: 24.0 alone.)
template <bool ACT_ORDER, int POLICY>
__global__ __launch_bounds__(kThreads) void dequant_kernel(const uint32_t *__restrict__ qweight,
                                                           const uint32_t *__restrict__ qzeros,
                                                           const half_t *__restrict__ scales,
                                                           const int32_t *__restrict__ g_idx,
                                                           half_t *__restrict__ w_out, int rows, int N,
                                                           int group_size)
{
    typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));
    constexpr int kSc1 = 16;  // cache policy of a buffer store
    // (kWriteThrough: the whole output is under 4 GB)
    const auto out_rsrc = __builtin_amdgcn_make_buffer_rsrc(w_out, 0, (uint32_t)rows * 16u * (uint32_t)N, 0x00020000);
    const int octs = N >> 3;
    const long long idx = (long long)blockIdx.x * kThreads + threadIdx.x;
    if (idx >= (long long)rows * octs)
        return;
    const int row = (int)(idx / octs);
    const int oct = (int)(idx - (long long)row * octs);
    const int n0 = oct * 8;
    const uint32_t *src = qweight + (size_t)row * N + n0;
    const uint4 wa = *reinterpret_cast<const uint4 *>(src), wb = *reinterpret_cast<const uint4 *>(src + 4);
    const uint32_t w[8] = {wa.x, wa.y, wa.z, wa.w, wb.x, wb.y, wb.z, wb.w};

    half8_t s, nz;  // scales and -(1024 + z) of the eight columns
    auto load_group = [&](int group) {
        s = *reinterpret_cast<const half8_t *>(scales + (size_t)group * N + n0);
        const uint32_t z = qzeros[(size_t)group * octs + oct];
#pragma unroll
        for (int c = 0; c < 8; ++c)
            nz[c] = __builtin_bit_cast(half_t, (uint16_t)(0xE400u | ((z >> (4 * c)) & 15u)));
    };
    if (!ACT_ORDER)
        load_group((row * 8) / group_size);  // group_size is a multiple of 8: one group per packed row
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        const int k = row * 8 + j;
        if (ACT_ORDER)
            load_group(g_idx[k]);
        half8_t o;
#pragma unroll
        for (int c = 0; c < 8; ++c)
            o[c] = __builtin_bit_cast(half_t, (uint16_t)(0x6400u | ((w[c] >> (4 * j)) & 15u)));
        o = (o + nz) * s;
        if (POLICY == kPlain)
            *reinterpret_cast<half8_t *>(w_out + (size_t)k * N + n0) = o;
        else if (POLICY == kBypass)
            __builtin_nontemporal_store(o, reinterpret_cast<half8_t *>(w_out + (size_t)k * N + n0));
        else
            __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4_t, o), out_rsrc,
                                                   ((uint32_t)k * (uint32_t)N + (uint32_t)n0) * 2u, 0, kSc1);
    }
}

inline unsigned blocks_for(long long items)
{
    return (unsigned)((items + kThreads - 1) / kThreads);
}

// z' = (z + delta) mod 16 for every nibble of every word (delta in 0..15; even and odd nibbles apart so that
// no carry crosses into a neighbour).
__global__ __launch_bounds__(kThreads) void shift_zeros_kernel(const uint32_t *__restrict__ in,
                                                               uint32_t *__restrict__ out, long long words,
                                                               uint32_t delta)
{
    const long long i = (long long)blockIdx.x * kThreads + threadIdx.x;
    if (i >= words)
        return;
    const uint32_t w = in[i];
    const uint32_t even = ((w & 0x0f0f0f0fu) + delta * 0x01010101u) & 0x0f0f0f0fu;
    const uint32_t odd = (((w >> 4) & 0x0f0f0f0fu) + delta * 0x01010101u) & 0x0f0f0f0fu;
    out[i] = even | (odd << 4);
}

}  // namespace

hipError_t launch_unpack(const uint32_t *qweight, uint8_t *q_out, const uint32_t *qzeros, uint8_t *z_out, int K,
                         int N, int group_size, hipStream_t stream)
{
    const int rows = K / 8;
    const long long items = (long long)rows * (N / 4);
    hipLaunchKernelGGL(unpack_qweight_kernel, dim3(blocks_for(items)), dim3(kThreads), 0, stream, qweight, q_out,
                       rows, N);
    hipError_t err = hipGetLastError();
    if (err != hipSuccess)
        return err;
    if (z_out) {
        const long long words = (long long)(K / group_size) * (N / 8);
        hipLaunchKernelGGL(unpack_qzeros_kernel, dim3(blocks_for(words)), dim3(kThreads), 0, stream, qzeros, z_out,
                           words);
        err = hipGetLastError();
    }
    return err;
}

hipError_t launch_shift_zeros(const uint32_t *in, uint32_t *out, long long words, int delta, hipStream_t stream)
{
    hipLaunchKernelGGL(shift_zeros_kernel, dim3(blocks_for(words)), dim3(kThreads), 0, stream, in, out, words,
                       (uint32_t)(delta & 15));
    return hipGetLastError();
}

hipError_t launch_dequant(const uint32_t *qweight, const uint32_t *qzeros, const half_t *scales,
                          const int32_t *g_idx, half_t *w_out, int K, int N, int group_size, hipStream_t stream)
{
    const int rows = K / 8;
    const long long items = (long long)rows * (N / 8);
    const int policy = N % 32 != 0 ? kPlain : 2ll * K * N > kBypassBytes ? kBypass : kWriteThrough;
    auto kernel = policy == kPlain    ? (g_idx ? dequant_kernel<true, kPlain> : dequant_kernel<false, kPlain>)
                  : policy == kBypass ? (g_idx ? dequant_kernel<true, kBypass> : dequant_kernel<false, kBypass>)
                                      : (g_idx ? dequant_kernel<true, kWriteThrough> : dequant_kernel<false, kWriteThrough>);
    hipLaunchKernelGGL(kernel, dim3(blocks_for(items)), dim3(kThreads), 0, stream, qweight, qzeros, scales, g_idx,
                       w_out, rows, N, group_size);
    return hipGetLastError();
}

}  // namespace gptq
