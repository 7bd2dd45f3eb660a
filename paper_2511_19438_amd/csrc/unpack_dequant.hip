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

constexpr long long kMemorySideCacheBytes = 256000000;

// w_out[k, n] = fp16( scales[r(k), n] * (q[k, n] - z[r(k), n]) ): exact integer difference, one fp16 multiply.
//
// Bound by HBM (2.5 bytes per weight, four fifths of them written), so what counts is how the rows are written: a thread
// owns EIGHT adjacent columns of one packed row (two 128-bit loads, one whole zero word), which makes every store 128
// bits and a wavefront's part of a row 1 KB contiguous.  The difference comes from the mantissa of 1024.0: (1024 + q) -
// (1024 + z) in packed halves is exact (and +0 for q = z, as the conversion of an integer 0 is).
//
// The written rows are 80 % of the traffic, and what counts next is whether their reader finds them in the memory-side
// cache (256 MB).  BYPASS, for outputs that do not fit it: non-temporal stores, past all caches.  Otherwise write-through
// stores (sc1): nothing is left dirty in the L2, and the rows stay in the memory-side cache.  Non-temporal stores would
// make the dequantisation itself shorter there, too, but a product that follows longer by more.  The weights alone, and
// with a product of 16 rows behind them, us with plain / non-temporal / write-through stores (the first three over a set of
// layers that exceeds the cache):
//   4096x4096    9.8 /  7.5 /  8.8    25.8 /  30.4 /  24.8
//   11008x4096  23.1 / 17.8 / 22.4    71.5 /  87.8 /  70.9
//   8192x12288  47.0 / 43.8 / 45.6    89.9 /  94.5 /  88.1
//   8192x16384  61.9 / 48.9 / 57.8   112.1 / 108.2 / 112.9   (268 MB)
//   8192x28672 102.5 / 86.4 / 101.4  230.6 / 205.3 / 230.6
// (11008x4096 with four columns per thread and plain 64-bit stores: 24.0 alone.)
template <bool ACT_ORDER, bool BYPASS>
__global__ __launch_bounds__(kThreads) void dequant_kernel(const uint32_t *__restrict__ qweight,
                                                           const uint32_t *__restrict__ qzeros,
                                                           const half_t *__restrict__ scales,
                                                           const int32_t *__restrict__ g_idx,
                                                           half_t *__restrict__ w_out, int rows, int N,
                                                           int group_size)
{
    typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));
    constexpr int kWriteThrough = 16;  // cache policy of a buffer store: sc1
    // (write-through: the whole output is under 4 GB)
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
        if (BYPASS)
            __builtin_nontemporal_store(o, reinterpret_cast<half8_t *>(w_out + (size_t)k * N + n0));
        else
            __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4_t, o), out_rsrc,
                                                   ((uint32_t)k * (uint32_t)N + (uint32_t)n0) * 2u, 0, kWriteThrough);
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
    const bool bypass = 2ll * K * N > kMemorySideCacheBytes;
    auto kernel = g_idx ? (bypass ? dequant_kernel<true, true> : dequant_kernel<true, false>)
                        : (bypass ? dequant_kernel<false, true> : dequant_kernel<false, false>);
    hipLaunchKernelGGL(kernel, dim3(blocks_for(items)), dim3(kThreads), 0, stream, qweight, qzeros, scales, g_idx,
                       w_out, rows, N, group_size);
    return hipGetLastError();
}

}  // namespace gptq
