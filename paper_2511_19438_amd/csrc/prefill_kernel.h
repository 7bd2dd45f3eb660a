// fp16 MFMA kernels for the W4A16 GPTQ matrix multiply at large batch (prefill), gfx950.
//
// This is the one place where the path is a real dense contraction, so it runs on the matrix
// cores (fp32 accumulation).  The paper's kernel (Opt4GPTQ, Section 3)
// uses one vector kernel for every batch size; what carries over is its pipeline order: stage the
// operands on chip with wide loads (Section 3.2), dequantise with packed half arithmetic
// (Section 3.3), accumulate on chip and commit each output once (Section 3.1).
//
// Design for CDNA4 (prefill_pipelined_kernel, the tuned path: no g_idx, group size a multiple of 64):
//   * Everything that comes from global memory - the activation tile, the packed weight words, the
//     scales and the packed zero points of a k stage - is copied global -> LDS by the DMA path
//     (global_load_lds_dwordx4), never through registers, into a ring of NBUF stage buffers that runs
//     NBUF-2 stages ahead of the MFMAs.  One s_waitcnt vmcnt(n) + s_barrier per stage publishes the
//     oldest batch in flight; loads complete in order, so "at most n outstanding" means "the batch
//     issued NBUF-2 stages ago has landed".
//   * v_mfma_f32_16x16x32_f16.  What bounds large products is the power that the matrix pipe draws (the clock falls to 1.65
//     GHz under it), and this form draws less for the same product than 32x32x16, whose accumulators pass twice as often: an
//     MFMA-only loop on N(0,1) activations and dequantised weights 1.92 PFLOP/s against 1.69, with two vector instructions
//     beside each 32 k operations 1.77 against 1.59 (a probe of both forms; probe.hip's has the 32x32x16 form alone).  Blocks of 16 rows also pad a ragged batch less.  One step with the
//     inline-assembly DMA and LDS reads below (through the builtin the compiler emptied the pipeline of loads once per
//     stage, in front of its first LDS read): 2048 rows through the four 8192-wide layers 2960 -> 2668 us, 512 rows through
//     the four 4096-wide ones 254 -> 230, 333x2752x6888 with groups of 32 31.5 -> 29.5.
//   * A operand (activations): 16-byte chunks are XOR-swizzled by row so that the 16-row operand
//     reads (ds_read_b128) are bank-conflict free on the 64-bank LDS.
//   * B operand (weights): a packed qweight word holds eight consecutive k of ONE column, which is
//     exactly what one lane of the MFMA's B operand holds.  Each lane reads its word(s) from
//     the LDS copy and dequantises them in registers into the four VGPRs of the operand:
//     v_perm_b32 + v_and_or_b32 build the pair (1024 + q_even, 64 + q_odd), a packed add of
//     (-(1024 + z), -(64 + z)) gives the exact integer differences and a packed multiply by the scale
//     gives the fp16 weight with one rounding.  The dequantised weights never touch LDS.
//   * Waves of a workgroup split the N extent of the tile where possible, so every weight is
//     dequantised by exactly one wave of the workgroup.
//   * The instruction order of a k step is pinned with scheduling barriers: every MFMA is followed by
//     a few instructions of the NEXT k step's LDS reads and dequantisation (one vector instruction per MFMA on a
//     256-row tile), which issue in the shadow of that MFMA (one wave per SIMD: nothing else would hide their latency or
//     keep the pipe fed).
//   * Lane j of an n-block owns TN adjacent columns (n-block t <-> column base + TN*j + t), so the
//     weight reads are TN dwords wide and the output stores are TN halves wide.
//   * Workgroup ids are remapped so that the tiles resident on one XCD (ids congruent mod 8) are
//     neighbours in the (m fastest) tile order and share their weight panel and activations in
//     that XCD's L2.
//
// Its HALF variant carries the scales and zero points of every 32-k half of a stage on their own, which serves group
// sizes that are odd multiples of 32, a K that ends half-way through a stage, and an N that is no multiple of 32.
//
// prefill_general_kernel serves the remaining cases (g_idx, group sizes that are not a multiple of
// 32) with 32x32x16 MFMAs and plain register staging; it is about correctness.
#pragma once

#include <type_traits>

#include "exchange.h"
#include "kernels.h"
#include "lds_dma.h"

namespace gptq {
namespace prefill {

constexpr int kThreads = 256;

enum Mode {
    kGroupPerStage = 0,  // group_size % 64 == 0, N % 32 == 0, no g_idx: pipelined kernel
    kGroupPerRow = 1,    // any group_size, no g_idx: looked up per packed row
    kActOrder = 2,       // g_idx: looked up per k
    kGroupPerHalf = 3    // group_size % 32 == 0, K >= 64, no g_idx: pipelined kernel, HALF variant
};

struct Args {
    const half_t *x;
    const uint32_t *qweight;
    const uint32_t *qzeros;
    const half_t *scales;
    const int32_t *g_idx;
    half_t *out;
    int M, K, N, group_size;
    int tiles_m, tiles_n;
    // K split of the pipelined kernel (few output tiles, deep K): slice s of a tile covers the stages
    // [s * stages_per_slice, ...); the slices meet in scratch, in slice order, as in the other kernels.
    int split_k;            // 1 = no split
    int stages_per_slice;
    float *partial;         // [split_k][tiles][accumulators per thread][256 threads] fp32 (see combine_slices)
    unsigned *counters;     // [tiles], zero between launches
    // SERIAL only: the slices that a workgroup walks (split_k is 1), and the wavefront groups that would have shared each
    int serial_slices, serial_kw;
};

typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));

__device__ __forceinline__ half2_t as_half2(uint32_t v)
{
    return __builtin_bit_cast(half2_t, v);
}

// (-(1024 + z), -(64 + z)) as packed fp16 bits
__device__ __forceinline__ uint32_t neg_bias(uint32_t z)
{
    return 0xD400E400u | z | (z << 20);
}

// Constants of the nibble -> fp16 conversion, kept in registers so that mask-and-bias is one v_and_or_b32
// (VOP3 on gfx9 takes no literals).  0x6400 = 1024.0 (ulp 1), 0x5400 = 64.0 (ulp 1/16).
struct PairMagic {
    uint32_t mask, bias;
    __device__ __forceinline__ PairMagic()
    {
        mask = 0x00f0000fu;
        bias = 0x54006400u;
        asm volatile("" : "+s"(mask), "+v"(bias));
    }
};

// Pair P (k = 2P, 2P+1) of one packed word -> two fp16 weights, as the bits of a half2.
// Byte P of w = q_{2P} | q_{2P+1} << 4 is spread to both halves, one nibble kept in each:
// low half 1024 + q_{2P}, high half 64 + q_{2P+1}; nz = (-(1024+z), -(64+z)), ss = (s, s).
template <int P>
__device__ __forceinline__ uint32_t dequant_pair(uint32_t w, const PairMagic &k, uint32_t nz, uint32_t ss)
{
    const uint32_t spread = __builtin_amdgcn_perm(0u, w, 0x0c000c00u | P | (P << 16));
    const half2_t v = (as_half2((spread & k.mask) | k.bias) + as_half2(nz)) * as_half2(ss);
    return __builtin_bit_cast(uint32_t, v);
}

// The first step of the same on its own: byte `pair` of w in the low byte of both halves.
__device__ __forceinline__ uint32_t spread_pair(uint32_t w, int pair)
{
    return __builtin_amdgcn_perm(0u, w, 0x0c000c00u | pair | (pair << 16));
}

__device__ __forceinline__ u32x4_t dequant_word(uint32_t w, const PairMagic &k, const uint32_t nz[4],
                                                const uint32_t ss[4])
{
    u32x4_t r;
    r[0] = dequant_pair<0>(w, k, nz[0], ss[0]);
    r[1] = dequant_pair<1>(w, k, nz[1], ss[1]);
    r[2] = dequant_pair<2>(w, k, nz[2], ss[2]);
    r[3] = dequant_pair<3>(w, k, nz[3], ss[3]);
    return r;
}

// body(integral_constant<int, 0>) ... body(integral_constant<int, COUNT - 1>): a loop whose counter is a constant in the body
// (longer ones than the compiler agrees to unroll would keep their register arrays in scratch memory).
template <int FIRST, int COUNT, typename Body>
__device__ __forceinline__ void static_for(Body &&body)
{
    if constexpr (COUNT == 1) {
        body(std::integral_constant<int, FIRST>());
    } else if constexpr (COUNT > 1) {
        static_for<FIRST, COUNT / 2>(body);
        static_for<FIRST + COUNT / 2, COUNT - COUNT / 2>(body);
    }
}

// XCD-aware tile order: workgroup ids congruent mod 8 run on one XCD; give each XCD a contiguous range
// of the (m fastest) tile order.  Returns false for the padding workgroups of the last range.
// With a K split the grid is `split_k` such ranges one after the other (the slices of a tile share an XCD).
__device__ __forceinline__ bool tile_of_workgroup(const Args &a, int &tile_m, int &tile_n, int &logical, int &slice)
{
    const int total = a.tiles_m * a.tiles_n;
    const int per_xcd = (total + 7) / 8;
    const int padded = per_xcd * 8;
    slice = blockIdx.x / padded;
    const int inner = blockIdx.x - slice * padded;
    logical = (inner & 7) * per_xcd + (inner >> 3);
    if (logical >= total)
        return false;
    tile_m = logical % a.tiles_m;
    tile_n = logical / a.tiles_m;
    return true;
}

// One fp16 rounding per output, TN adjacent columns per store.  Lane (lj, kh) holds, for 32-row block i and
// accumulator register r, row 8*(r/4) + 4*kh + r%4 of the block and column lj of n-block t.
template <int TM, int TN>
__device__ __forceinline__ void store_tile(const float16_t (&acc)[TM][TN], half_t *out, int row0, int col0,
                                           bool col_ok, int kh, int M, int N)
{
    if (!col_ok)
        return;
#pragma unroll
    for (int i = 0; i < TM; ++i) {
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const int m = row0 + i * 32 + 8 * (r >> 2) + 4 * kh + (r & 3);
            if (m < M) {
                half_t *dst = out + (size_t)m * N + col0;
                if (TN == 4) {
                    half4_t v = {(half_t)acc[i][0][r], (half_t)acc[i][1 % TN][r], (half_t)acc[i][2 % TN][r],
                                 (half_t)acc[i][3 % TN][r]};
                    *reinterpret_cast<half4_t *>(dst) = v;
                } else if (TN == 2) {
                    half2_t v = {(half_t)acc[i][0][r], (half_t)acc[i][1 % TN][r]};
                    *reinterpret_cast<half2_t *>(dst) = v;
                } else {
                    *dst = (half_t)acc[i][0][r];
                }
            }
        }
    }
}

// One fp16 rounding per output, TN adjacent columns per store.  Lane (lj, kg) holds, for 16-row block i and
// accumulator register r, row 4*kg + r of the block and column lj of n-block t.
template <int TM, int TN>
__device__ __forceinline__ void store_blocks(const float4_t (&acc)[TM][TN], half_t *out, int row0, int col0, bool col_ok, int kg,
                                             int M, int N)
{
    if (!col_ok)
        return;
#pragma unroll
    for (int i = 0; i < TM; ++i) {
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int m = row0 + i * 16 + 4 * kg + r;
            if (m < M) {
                half_t *dst = out + (size_t)m * N + col0;
                if (TN == 4)
                    *reinterpret_cast<half4_t *>(dst) = half4_t{(half_t)acc[i][0][r], (half_t)acc[i][1 % TN][r],
                                                                (half_t)acc[i][2 % TN][r], (half_t)acc[i][3 % TN][r]};
                else
                    *reinterpret_cast<half2_t *>(dst) = half2_t{(half_t)acc[i][0][r], (half_t)acc[i][1 % TN][r]};
            }
        }
    }
}

// K slices across workgroups (few output tiles, deep K).  Every slice leaves its results in scratch and the
// last workgroup of the tile to arrive adds them in slice order (deterministic), then goes on to store the
// tile.  The values travel in pairs - 64-bit accesses, pair p of thread t at [p][t]: coalesced - and the last
// arriver loads several slices before it uses any, so the combine costs a few scratch round trips instead of
// one per slice.  Device-scope accesses and an arrival counter with release / acquire at agent scope (exchange.h).
// Returns false in the workgroups that are not the last of their tile.  Partial layout:
// [split_k][tiles][ACC / 2 pairs][256 threads] x 8 bytes.
// `member`: whether this thread holds values (a workgroup of two K halves: only the first half's threads do; the
// others only pass the barriers).
template <int ACC>
__device__ __forceinline__ bool combine_slices(float (&v)[ACC], const Args &a, int slice, int tile_id, int tid,
                                               bool member)
{
    static_assert(ACC % 2 == 0, "values travel in pairs");
    typedef float f32x2_t __attribute__((ext_vector_type(2)));
    constexpr int PAIRS = ACC / 2;
    constexpr int CH = PAIRS < 64 ? PAIRS : 64;  // pairs of one slice loaded together
    constexpr int G = 64 / CH;                   // slices loaded together: up to 128 values in flight
    static_assert(PAIRS % CH == 0 && G <= 4, "whole batches");
    __shared__ int s_last;
    const size_t tiles = (size_t)a.tiles_m * a.tiles_n;
    unsigned long long *scratch = reinterpret_cast<unsigned long long *>(a.partial);
    unsigned long long *mine = scratch + ((size_t)slice * tiles + tile_id) * PAIRS * kThreads + tid;
    if (member) {
#pragma unroll
        for (int p = 0; p < PAIRS; ++p) {
            const f32x2_t pair = {v[2 * p], v[2 * p + 1]};
            __hip_atomic_store(mine + (size_t)p * kThreads, __builtin_bit_cast(unsigned long long, pair),
                               __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
    }
    __builtin_amdgcn_s_waitcnt(0);  // every partial store of this workgroup has been acknowledged (exchange.h)
    __syncthreads();
    if (threadIdx.x == 0)
        s_last = (slice_arrive(a.counters + tile_id) == (unsigned)(a.split_k - 1));
    __syncthreads();
    if (!s_last || !member)
        return false;
    slice_acquire();
#pragma unroll
    for (int e = 0; e < ACC; ++e)
        v[e] = 0.f;
#pragma unroll
    for (int c0 = 0; c0 < PAIRS; c0 += CH) {
        auto add = [&](int sl0, auto slices) {
            constexpr int S = decltype(slices)::value;
            unsigned long long part[S][CH];
#pragma unroll
            for (int u = 0; u < S; ++u) {
                const unsigned long long *theirs =
                    scratch + ((size_t)(sl0 + u) * tiles + tile_id) * PAIRS * kThreads + (size_t)c0 * kThreads + tid;
#pragma unroll
                for (int p = 0; p < CH; ++p)
                    part[u][p] =
                        __hip_atomic_load(theirs + (size_t)p * kThreads, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                // (half of a whole batch, all of a smaller one, is issued before the first add waits)
                if constexpr (G > 1)
                    if (u == (S == G ? S / 2 : S) - 1)
                        __builtin_amdgcn_sched_barrier(0);
            }
#pragma unroll
            for (int u = 0; u < S; ++u) {
#pragma unroll
                for (int p = 0; p < CH; ++p) {
                    const f32x2_t pair = __builtin_bit_cast(f32x2_t, part[u][p]);
                    v[2 * (c0 + p)] += pair[0];
                    v[2 * (c0 + p) + 1] += pair[1];
                }
            }
        };
        // Whole batches, then the rest in one of its own size: no slice is loaded twice.  (Left out by a factor of zero, a
        // repeated infinite sum became a NaN; by a select per value 142x2816x1600 in five slices took 13.6 us instead of
        // 13.1, and takes 12.2 now; 333x2752x6888 in three 32.0, 31.5, 30.4; 222x5632x608 in eight 15.2, 14.8, 15.2.)
        int sl0 = 0;
        for (; sl0 + G <= a.split_k; sl0 += G)
            add(sl0, std::integral_constant<int, G>());
        const int rest = a.split_k - sl0;
        if (G > 3 && rest == 3)
            add(sl0, std::integral_constant<int, (G > 3 ? 3 : 1)>());
        else if (G > 2 && rest == 2)
            add(sl0, std::integral_constant<int, (G > 2 ? 2 : 1)>());
        else if (G > 1 && rest == 1)
            add(sl0, std::integral_constant<int, 1>());
    }
    if (tid == 0)
        __hip_atomic_store(a.counters + tile_id, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);  // next launch
    return true;
}

// =====================================================================================================
// Tuned path
// =====================================================================================================

// LDS layout of one stage buffer of the pipelined kernel.
template <int BM, int BN, int BK, bool HALF>
struct StageLayout {
    static constexpr int A_BYTES = BM * BK * 2;        // [BM][BK] halves, 16-byte chunks swizzled
    static constexpr int B_BYTES = (BK / 8) * BN * 4;  // [BK/8][BN] packed words
    // scales [BN] halves, then zero words [BN/8], then padding; HALF: scales [2][BN], then zero words [2][BN/8],
    // padded to the 256 bytes of a wave-wide DMA of single words (any more padding and the 64x128 tile would fit a
    // compute unit twice only, not three times)
    static constexpr int SCALE_BYTES = 4 * BN;
    static constexpr int SZ_BYTES = HALF ? SCALE_BYTES + 256 : 1024;
    static constexpr int BYTES = A_BYTES + B_BYTES + SZ_BYTES;
};

// Tiles with up to 128 accumulator registers per lane are compiled to fit two workgroups on a compute unit
// (256 registers per lane each): one workgroup's dequantisation then runs under the other's MFMAs.
template <int BM, int BN>
constexpr int kWavesPerSimd = (BM * BN <= 128 * 256) ? 2 : 1;

// HALF: each 32-k half of a stage brings its own row of scales and of zero points, and both rows travel in DMA pieces
// that suit any N that is a multiple of 8: word by word (a row of zero points is only 4-byte aligned then), the
// wavefronts sharing the scales.  One DMA instruction and a few vector operations per stage more than the variant with
// one group per stage, which therefore stays where it applies (groups of 128 against groups of 32: 2048x4096x11008 on the
// 128x256 tile 194 us against 205, 512x4096x4096 on the 64x128 tile 33 against 39).  What it took over from the general
// path: 2048x4096x11008 582 -> 205 us, 333x2752x6888 107 -> 31 (groups of 32), 512x4096x4104 (groups of 128, a width of 8
// mod 32) 148 -> 44.
// A K that ends half-way through a stage (K % 64 == 32): the last stage covers the last 64 k, the first half of which
// the stage before has done already; its activations are cleared in LDS once they have landed, so nothing is read
// past a row's or the matrix' end and what is repeated contributes exact zeros.
//
// KW = 2: a workgroup of eight wavefronts, two per SIMD, in two groups of four that each walk half of the K slice for
// the SAME tile, with a ring of their own; only the stage barriers and the sum through LDS at the end are shared.  Two
// wavefronts per SIMD are what the matrix pipe needs to run under the other's dequantisation (128x256 tile: a 64-k
// stage takes 0.99 us alone on a compute unit, 1.31 us when two run), and where the tiles give every compute unit one
// workgroup at most, this is how they get there without partial sums in scratch.
// 4096x12288 at M = 512: 73.5 -> 58.0 us; 28672x8192 at M = 512, two slices: 266 -> 226.
//
// SERIAL: no scratch for the K slices.  A workgroup walks all slices of its tile one after the other - the halves of a
// slice that two wavefront groups would have shared, too - and adds their sums in the order of the sliced launch, so the
// bits are those of that launch whatever its tile was.  For the 64x128 tile only, whose accumulators leave room for
// the sums.  Slower than slices in parallel, and never chosen where scratch can be had.
template <int BM, int BN, int WM, int WN, int BK, int NBUF, bool HALF = false, int KW = 1, bool SERIAL = false>
__global__ __launch_bounds__(kThreads * KW, (kWavesPerSimd<BM, BN>)) void prefill_pipelined_kernel(const Args a)
{
    static_assert(KW == 1 || (KW == 2 && BM * BN <= 128 * 256), "two wavefronts per SIMD have 256 registers each");
    static_assert(!SERIAL || (KW == 1 && BM * BN <= 64 * 128), "32 accumulators, their sum and a half's");
    static_assert(WM * WN == 4, "four wavefronts per workgroup");
    static_assert(BK == 64, "stage of 64 k");
    static_assert(NBUF >= 3, "ring of at least three stage buffers");
    using L = StageLayout<BM, BN, BK, HALF>;
    constexpr int WAVE_M = BM / WM;
    constexpr int WAVE_N = BN / WN;
    constexpr int TM = WAVE_M / 16;
    constexpr int TN = WAVE_N / 16;
    static_assert(TM >= 4 && (TN == 2 || TN == 4), "wave tile: 16-row blocks by 32/64 columns");
    constexpr int KSTEPS = 2;                               // MFMA k steps per stage
    // A operands in registers, in use or on their way: a divisor of a stage's, enough of them to hide an LDS read
    constexpr int RING_A = TM < 5 || TM > 7 ? 8 : TM > 5 || TN == 4 ? TM : 2 * TM;
    static_assert(KSTEPS * TM % RING_A == 0, "an operand's register is the same in every stage");
    constexpr int CH = BK / 8;                              // 16-byte chunks per A row
    constexpr int RPB = 16 / CH;                            // A rows per 256-byte bank row
    // DMA instructions per thread for the A tile; in the last of 80 and 112 rows' two wavefronts repeat the other two's pieces
    constexpr int A_CHUNKS = (BM * CH + kThreads - 1) / kThreads;
    constexpr int A_REPEAT = A_CHUNKS * kThreads - BM * CH;
    static_assert(A_REPEAT == 0 || A_REPEAT == kThreads / 2, "whole wavefronts repeat");
    constexpr int B_CHUNKS = (BK / 8) * BN / 4 / kThreads;  // ... for the packed weights
    static_assert(A_CHUNKS >= 1 && B_CHUNKS >= 1, "tile too small for 256 threads");
    static_assert(BN / 8 + BN / 32 <= 64, "scales and zero points of a stage must fit one wave-wide DMA");
    constexpr int LOADS_PER_STAGE = A_CHUNKS + B_CHUNKS + (HALF ? 2 : 1);
    constexpr int MAX_IN_FLIGHT = (NBUF - 3) * LOADS_PER_STAGE;  // may stay outstanding when a stage is published
    static_assert(MAX_IN_FLIGHT < 64, "vmcnt is a 6-bit counter");

    extern __shared__ __align__(16) unsigned char smem_all[];

    const int kgroup = KW == 1 ? 0 : __builtin_amdgcn_readfirstlane(threadIdx.x / kThreads);
    const int tid = threadIdx.x % kThreads;  // within the four wavefronts that share a ring
    unsigned char *const smem = smem_all + (size_t)kgroup * NBUF * L::BYTES;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);  // wave-uniform: keep it in a scalar register
    const int wm = wave / WN;
    const int wn = wave % WN;
    const int lj = lane & 15;  // row of a 16-row block (A operand), column of a 16-column block (B operand, result)
    const int kg = lane >> 4;  // packed row inside a 32-k step

    int tile_m, tile_n, tile_id, slice;
    if (!tile_of_workgroup(a, tile_m, tile_n, tile_id, slice))
        return;
    const int m0 = tile_m * BM;
    const int n0 = tile_n * BN;
    const int N = a.N, K = a.K, M = a.M;
    // K is a multiple of the group size, which is a multiple of 64 (HALF: of 32, and K may end half-way)
    const int all_stages = HALF ? (K + BK - 1) / BK : K / BK;
    const int col_local = wn * WAVE_N + TN * lj;  // first of this lane's TN columns inside the tile
    const int col_raw = n0 + col_local;
    const bool col_ok = col_raw < N;
    float4_t acc[TM][TN];
    const int groups = SERIAL ? a.serial_kw : KW;
    float4_t total[SERIAL ? TM : 1][SERIAL ? TN : 1], half_sum[SERIAL ? TM : 1][SERIAL ? TN : 1];
    if (SERIAL) {
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int t = 0; t < TN; ++t)
                total[i][t] = half_sum[i][t] = float4_t{0.f, 0.f, 0.f, 0.f};
    }
    int group = kgroup;  // SERIAL: the groups of every slice, one after the other
    for (;;) {           // (a single pass unless SERIAL; the body, up to the sums, is not indented)
    // this workgroup's stages: [wg_first, wg_first + wg_stages); a group's: [first, first + stages), maybe none
    const int wg_first = slice * a.stages_per_slice;
    const int wg_stages = min(a.stages_per_slice, all_stages - wg_first);
    const int lead = groups == 1 ? wg_stages : (wg_stages + 1) / 2;  // stages of the first group: no group has more
    const int stages = group == 0 ? lead : wg_stages - lead;
    const int first = wg_first + (stages > 0 ? group * lead : 0);
    const int last = first + max(stages, 1) - 1;

#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int t = 0; t < TN; ++t)
            acc[i][t] = float4_t{0.f, 0.f, 0.f, 0.f};

    // ---- global sources of this thread's DMA slots, as 32-bit byte offsets from bases that are uniform over
    //      the workgroup (scalar registers).  Loads never branch: rows past M and columns past N are clamped
    //      to the last valid ones; what they produce lands in output rows / columns that are not stored.
    // A: slot p = tid + j*256 holds physical chunk p % CH of row p / CH = logical chunk (p % CH) ^ ((row / RPB) % CH).
    const char *a_base = reinterpret_cast<const char *>(a.x + (size_t)m0 * K);
    uint32_t a_off[A_CHUNKS];
#pragma unroll
    for (int j = 0; j < A_CHUNKS; ++j) {
        int slot = tid + j * kThreads;
        slot -= slot >= BM * CH ? A_REPEAT : 0;
        const int row = slot / CH;
        const int ch = (slot % CH) ^ ((row / RPB) & (CH - 1));
        a_off[j] = (uint32_t)((min(m0 + row, M - 1) - m0) * K + ch * 8) * 2u;
    }
    // B: slot p holds words 4*(p % (BN/4)) .. +3 of packed row p / (BN/4) of the stage.
    const char *b_base = reinterpret_cast<const char *>(a.qweight + n0);
    uint32_t b_off[B_CHUNKS];
#pragma unroll
    for (int j = 0; j < B_CHUNKS; ++j) {
        const int slot = tid + j * kThreads;
        const int row = slot / (BN / 4);
        const int c4 = slot % (BN / 4);
        b_off[j] = (uint32_t)(row * N + min(4 * c4, N - 4 - n0)) * 4u;
    }
    // scales / zero points: lanes 0 .. BN/8-1 fetch 8 scales each, the next BN/32 lanes 4 zero words each, the
    // rest refetch the last zero chunk into padding (every lane takes part: the DMA needs no exec mask).
    // (N is a multiple of 32 here, so a clamped chunk of four zero words still lies inside its row.)
    const int sz_lane = min(lane, BN / 8 + BN / 32 - 1);
    const bool sz_is_scale = sz_lane < BN / 8;
    const int sz_col = sz_is_scale ? min(n0 + 8 * sz_lane, N - 8) : min(n0 + 32 * (sz_lane - BN / 8), N - 32);
    const char *sz_src_plain = sz_is_scale ? reinterpret_cast<const char *>(a.scales + sz_col)
                                           : reinterpret_cast<const char *>(a.qzeros + (sz_col >> 3));
    // HALF, zero points: lane -> half lane / (BN/8) of the stage (lanes past the second one repeat it), one zero word
    // each; scales: two per lane, 128 per wavefront - wavefront -> half and part of the half's row.
    const int z_half = min(lane / (BN / 8), 1);
    const char *z_src = reinterpret_cast<const char *>(a.qzeros + (min(n0 + 8 * (lane % (BN / 8)), N - 8) >> 3));
    const uint32_t z_stride = (uint32_t)(N >> 3) * 4u;
    constexpr int S_PARTS = BN / 128;  // wavefronts per half's row of scales
    const int s_part = wave % (2 * S_PARTS);
    const int s_half = s_part / S_PARTS;
    const char *sz_src = HALF ? reinterpret_cast<const char *>(
                                    a.scales + min(n0 + 128 * (s_part % S_PARTS) + 2 * lane, N - 2))
                              : sz_src_plain;
    const uint32_t sz_stride = HALF || sz_is_scale ? (uint32_t)N * 2u : (uint32_t)(N >> 3) * 4u;  // bytes per group row
    const int stages_per_group = HALF ? a.group_size / 32 : a.group_size / BK;  // HALF: halves per group
    // the position of a stage in 32-k halves: twice its number, one less for a last stage that K ends half-way through
    const bool k_tail = HALF && (K & 32) != 0;
    const int first_half = 2 * first - (k_tail && first == all_stages - 1 ? 1 : 0);
    // the last stage within its group's stages (the barrier that goes with clearing it is everybody's), or none
    const bool wg_tail = k_tail && wg_first + wg_stages == all_stages;
    const int tail_group = groups == 1 || wg_stages == 1 ? 0 : 1;
    const int tail_stage = wg_tail ? (tail_group == 0 ? lead : wg_stages - lead) - 1 : -2;

    // The stage whose loads are issued next, as running source pointers (uniform for the activations and the
    // packed words, per lane for the scales / zero points) that advance by constants: no multiplication and no
    // division in the loop, and selects instead of branches - a branch would end the basic block, and the
    // dequantisation of a stage's last k step (pure arithmetic, first used in the next stage) would sink
    // across it, out of the MFMAs' shadow.
    int ld_stage = first;
    int ld_in_group = HALF ? (first_half + s_half) % stages_per_group : first % stages_per_group;
    int z_in_group = HALF ? (first_half + z_half) % stages_per_group : 0;
    const char *a_cur = uniform(a_base + (HALF ? (size_t)first_half * 64 : (size_t)first * BK * 2));
    const uint32_t b_step = (uint32_t)(BK / 8) * N * 4u;  // bytes between the packed rows of consecutive stages
    const char *b_cur = uniform(b_base + (HALF ? (size_t)first_half * (b_step / 2) : (size_t)first * b_step));
    const char *sz_cur = sz_src + (size_t)((HALF ? first_half + s_half : first) / stages_per_group) * sz_stride;
    const char *z_cur = z_src + (size_t)((first_half + z_half) / stages_per_group) * z_stride;  // HALF
    const uint32_t smem_base = __builtin_amdgcn_readfirstlane(
        (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char *)smem);
    // piece `p` (0 .. LOADS_PER_STAGE-1) of the loads of stage `ld_stage` into ring slot `ring`
    auto issue_piece = [&](int p, int ring) {
        const uint32_t base = smem_base + (uint32_t)ring * (uint32_t)L::BYTES;
        if (p < A_CHUNKS) {  // the wave's 64 lanes fill 64 consecutive 16-byte slots
            const int slot = p * kThreads + wave * 64;
            dma_16(base + (uint32_t)(slot - (slot >= BM * CH ? A_REPEAT : 0)) * 16u, a_off[p], a_cur);
        } else if (p < A_CHUNKS + B_CHUNKS)
            dma_16(base + L::A_BYTES + (uint32_t)((p - A_CHUNKS) * kThreads + wave * 64) * 16u, b_off[p - A_CHUNKS], b_cur);
        else if (HALF && p == LOADS_PER_STAGE - 1)
            dma_4(base + L::A_BYTES + L::B_BYTES + L::SCALE_BYTES, z_cur);
        else if (HALF)
            dma_4(base + L::A_BYTES + L::B_BYTES + s_part * 256u, sz_cur);
        else  // all four waves write the same bytes: keeps the per-wave count of outstanding loads identical
            dma_16(base + L::A_BYTES + L::B_BYTES, sz_cur);
    };
    auto advance_load_stage = [&]() {
        // past the end the last stage is refetched: uniform counts, no branch in the loads
        const int more = ld_stage < last ? 1 : 0;
        ld_stage += more;
        if (HALF) {
            // one half less into a last stage that K ends half-way through; a group may be a single half
            const bool into_tail = k_tail && ld_stage == all_stages - 1;
            a_cur += more ? (into_tail ? BK : BK * 2) : 0;
            b_cur = uniform(b_cur + (more ? (into_tail ? b_step / 2 : b_step) : 0u));
            ld_in_group += more ? (into_tail ? 1 : 2) : 0;
            z_in_group += more ? (into_tail ? 1 : 2) : 0;
#pragma unroll
            for (int w = 0; w < 2; ++w) {
                const bool s_wrap = ld_in_group >= stages_per_group;
                ld_in_group -= s_wrap ? stages_per_group : 0;
                sz_cur += s_wrap ? sz_stride : 0u;
                const bool z_wrap = z_in_group >= stages_per_group;
                z_in_group -= z_wrap ? stages_per_group : 0;
                z_cur += z_wrap ? z_stride : 0u;
            }
            return;
        }
        a_cur += more ? BK * 2 : 0;
        b_cur += more ? b_step : 0u;
        ld_in_group += more;
        const bool wrap = ld_in_group == stages_per_group;
        ld_in_group = wrap ? 0 : ld_in_group;
        sz_cur += wrap ? sz_stride : 0u;
    };
    // Publish the oldest batch in flight: every wave waits for its own part of it, the barrier does the rest.
    auto publish = [&]() {
        asm volatile("s_waitcnt vmcnt(%0)" ::"n"(MAX_IN_FLIGHT) : "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
    };

    // Clears the activations of the first half of the last stage (see above) once the stage is in LDS; the barrier
    // stands before any wavefront's first read of them.
    auto clear_repeated_half = [&](int ring) {
        for (int slot = tid; slot < (group == tail_group ? BM * 4 : 0); slot += kThreads) {
            const int row = slot >> 2;
            const int ch = (slot & 3) ^ ((row / RPB) & (CH - 1));
            *reinterpret_cast<uint4 *>(smem + (size_t)ring * L::BYTES + (size_t)(row * CH + ch) * 16) =
                make_uint4(0u, 0u, 0u, 0u);
        }
        __syncthreads();
    };

    // ---- operand registers ----
    half8_t afr[RING_A];            // A operands, one after the other: operand q of a stage (k step q / TM, block q % TM)
    u32x4_t bfr[2][TN];             // B operands (bits of 4 half2 each) of two consecutive k steps
    typedef uint32_t words_t __attribute__((ext_vector_type(TN)));
    typedef uint32_t words_half_t __attribute__((ext_vector_type(2)));
    typedef std::conditional_t<TN == 4, words_half_t, uint32_t> scales_t;  // two in each word
    words_t words[KSTEPS];          // packed words of this lane: of each k step, the ones to be dequantised next
    scales_t raw_s;                 // scales and zero word of the group to be used next
    uint32_t raw_z;
    uint32_t nz[TN], ss[TN];        // the same, of the group in use, as operands of the packed arithmetic
    const PairMagic magic;

    // A operand of 16-row block i at k step kk: row wm*WAVE_M + 16 i + lj, chunk (4 kk + kg) ^ swizzle(row).
    // The swizzle does not depend on i (16 rows are a whole number of swizzle periods), so the byte offset is
    // a per-lane value per k step plus i * 16 rows: the reads of one k step share ONE address register (the
    // stage buffer's base added once per k step) and differ in the instruction's immediate offset.
    static_assert(RPB == 2 && CH == 8, "sixteen rows, eight chunks: one period of the swizzle");
    uint32_t a_lane_off[KSTEPS];
#pragma unroll
    for (int kk = 0; kk < KSTEPS; ++kk) {
        const int row = wm * WAVE_M + lj;
        a_lane_off[kk] = smem_base + (uint32_t)(row * (BK * 2) + (((4 * kk + kg) ^ ((row / RPB) & (CH - 1))) * 16));
    }
    // The LDS reads of the loop are issued as inline asm and waited for by hand: the compiler's own counter
    // bookkeeping loses track of the order of LDS operations across the loop's back edge and falls back to
    // waiting for ALL outstanding LDS reads - including the one issued a few cycles earlier - before the first
    // use of every operand, which stalls the matrix pipe for an LDS round trip several times per k step.
    auto read_afrag = [&](int ring, auto operand, half8_t &dst) {  // operand (number in its stage) of the stage in `ring`
        constexpr int Q = decltype(operand)::value, KK = Q / TM, I = Q % TM;
        const uint32_t addr = a_lane_off[KK] + (uint32_t)ring * (uint32_t)L::BYTES;
        asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(dst) : "v"(addr), "n"(I * 16 * BK * 2));
    };
    // this lane's packed words of k step KK, and the scales and the zero word of the KK-th group of a stage
    const uint32_t w_lane_off = smem_base + (uint32_t)(kg * BN + col_local) * 4u;
    const uint32_t s_lane_off = smem_base + (uint32_t)col_local * 2u;
    const uint32_t z_lane_off = smem_base + (uint32_t)(col_local >> 3) * 4u;
    auto read_words = [&](int ring, auto step, words_t &dst) {
        const uint32_t addr = w_lane_off + (uint32_t)ring * (uint32_t)L::BYTES;
        constexpr int OFF = L::A_BYTES + decltype(step)::value * 4 * BN * 4;
        if (TN == 4)
            asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(dst) : "v"(addr), "n"(OFF));
        else
            asm volatile("ds_read_b64 %0, %1 offset:%2" : "=v"(dst) : "v"(addr), "n"(OFF));
    };
    auto read_group = [&](int ring, auto number, scales_t &scales, uint32_t &zeros) {
        constexpr int G = decltype(number)::value, SZ = L::A_BYTES + L::B_BYTES;
        const uint32_t s_addr = s_lane_off + (uint32_t)ring * (uint32_t)L::BYTES;
        const uint32_t z_addr = z_lane_off + (uint32_t)ring * (uint32_t)L::BYTES;
        if (TN == 4)
            asm volatile("ds_read_b64 %0, %1 offset:%2" : "=v"(scales) : "v"(s_addr), "n"(SZ + G * BN * 2));
        else
            asm volatile("ds_read_b32 %0, %1 offset:%2" : "=v"(scales) : "v"(s_addr), "n"(SZ + G * BN * 2));
        asm volatile("ds_read_b32 %0, %1 offset:%2"
                     : "=v"(zeros)
                     : "v"(z_addr), "n"(SZ + (HALF ? L::SCALE_BYTES + G * (BN / 8) * 4 : BN * 2)));
    };
    // When they are read: the A operand RING_A - 1 ahead with every operand's first MFMA, the words (and the group) that
    // are dequantised in the next k step after operand READ_AFTER of this one.
    constexpr int READ_AFTER = TM - 4;
    auto reads_words = [](int group) { return group % TM == READ_AFTER; };
    auto word_reads = [](int group) { return HALF || group < TM ? 3 : 1; };
    // The prologue issues the first RING_A - 1 operands in this order, too, but of the words in between those of k step 1 alone:
    // it has waited for the others before.
    auto in_prologue = [](int operand) { return operand + KSTEPS * TM - (RING_A - 1); };  // the group that issues it in the loop
    // LDS reads behind that of operand Q, in the first stage, where its wait stands
    auto behind_in_first_stage = [=](int operand) {
        int behind = -1;
        for (int q = 0; q < RING_A - 1 + operand; ++q) {
            const bool prologue = q < RING_A - 1;
            const int group = prologue ? in_prologue(q) : q - (RING_A - 1);
            behind = q == operand ? 0 : behind + (behind >= 0);
            if (behind >= 0 && reads_words(group) && (!prologue || group >= TM))
                behind += word_reads(group);
        }
        return behind;
    };
    // Before the first use of operand q of a stage: LDS reads return in order, so what may be outstanding is what has been
    // issued after its own read - the RING_A - 2 operands that follow and the words read in between, but for those that the
    // prologue leaves out (one wait serves the first stage and the others: on 80x128, whose ring is two k steps long,
    // operand 0 waits for the words and the group behind it as well).
    // (The operand is an in/out of the wait, so that the MFMA that consumes it cannot be moved above it.)
    auto wait_afrag = [&](auto operand, half8_t &frag) {
        constexpr int Q = decltype(operand)::value;
        constexpr int COUNT = [=] {
            int n = RING_A - 2;
            for (int g = Q - (RING_A - 1); g < Q; ++g) {
                const int group = (g + KSTEPS * TM) % (KSTEPS * TM);
                if (reads_words(group) && (g >= 0 || group >= TM))
                    n += word_reads(group);
            }
            return n;
        }();
        static_assert(COUNT <= behind_in_first_stage(Q), "a wait that the first stage meets with too few reads in flight is none");
        static_assert(COUNT < 16, "lgkmcnt is a 4-bit counter");
        asm volatile("s_waitcnt lgkmcnt(%1)" : "+v"(frag) : "n"(COUNT));
    };
    // The same for the words (and the group), behind the first MFMA of a k step: the operands read since may be outstanding.
    auto wait_words = [&](words_t &w) { asm volatile("s_waitcnt lgkmcnt(%1)" : "+v"(w) : "n"(TM - 1 - READ_AFTER)); };
    auto wait_group = [&](scales_t &scales, uint32_t &zeros) { asm volatile("" : "+v"(scales), "+v"(zeros)); };
    const int z_shift = 4 * (col_local & 7);
    auto unpack_scale = [&](int t) {
        uint32_t pair;
        if constexpr (TN == 4)
            pair = raw_s[t / 2];
        else
            pair = raw_s;
        ss[t] = __builtin_amdgcn_perm(0u, pair, t & 1 ? 0x03020302u : 0x01000100u);
    };
    auto unpack_zero = [&](int t) { nz[t] = neg_bias(raw_z >> (z_shift + 4 * t) & 15u); };

    // The vector work that prepares the B operands of a k step, as a list of small operations: `GROUP_OPS` that
    // unpack a new group's scales and zero points, then sixteen per packed word - spread, mask and bias, subtract the
    // zero point, scale, each for the four pairs of the word before the next, so that no operation follows the one it
    // depends on.
    constexpr int GROUP_OPS = 2 * TN;
    auto prepare_op = [&](int o, bool new_group, int kk, u32x4_t (&b)[TN]) {
        if (new_group && o < GROUP_OPS) {
            if (o & 1)
                unpack_zero(o / 2);
            else
                unpack_scale(o / 2);
            return;
        }
        const int d = o - (new_group ? GROUP_OPS : 0);
        const int t = d >> 4, pair = d & 3;
        switch (d >> 2 & 3) {
        case 0: b[t][pair] = spread_pair(words[kk][t], pair); break;
        case 1: b[t][pair] = (b[t][pair] & magic.mask) | magic.bias; break;
        case 2: b[t][pair] = __builtin_bit_cast(uint32_t, as_half2(b[t][pair]) + as_half2(nz[t])); break;
        default: b[t][pair] = __builtin_bit_cast(uint32_t, as_half2(b[t][pair]) * as_half2(ss[t])); break;
        }
    };

    // One k step, in exactly this instruction order (a scheduling barrier closes every slot): ONE MFMA, then
    // its share of the work for the NEXT k step - the LDS read of the A operand RING_A - 1 ahead (once per operand),
    // preparation of the B operands, and whatever `extra` adds (loads for a later stage).
    // An MFMA occupies the matrix pipe for 4 passes but the wave can issue other instructions right behind it,
    // so a handful of them per MFMA run in its shadow; several MFMAs back to back followed by a block of
    // vector work would leave the pipe idle during the block.
    constexpr int SLOTS = TM * TN;  // MFMAs per k step
    auto multiply = [&](float4_t &c, const half8_t &x, const u32x4_t &w) {
        // 256 accumulators fill one half of a wavefront's registers.  Left to itself the compiler keeps some of them in the
        // other half and swaps them in and out (288 moves per stage); the assembly says where they are.  It hides the MFMA
        // from the compiler's hazard checks: the B operands are complete three MFMAs before their use, the results are
        // first read after the wait states behind the loop.
        if constexpr (TM * TN == 64)
            asm volatile("v_mfma_f32_16x16x32_f16 %0, %1, %2, %0" : "+a"(c) : "v"(x), "v"(w));
        else
            c = __builtin_amdgcn_mfma_f32_16x16x32_f16(x, __builtin_bit_cast(half8_t, w), c, 0, 0, 0);
    };
    auto kstep = [&](auto step, int ring, int ring_next, auto &&extra) {
        constexpr int KK = decltype(step)::value, NXT = KK ^ 1;
        constexpr bool NEW_GROUP = HALF || NXT == 0;  // the k step being prepared brings a row of scales
        constexpr int OPS = 16 * TN + (NEW_GROUP ? GROUP_OPS : 0);
        static_for<0, SLOTS>([&](auto slot) {
            constexpr int m = decltype(slot)::value, i = m / TN, t = m % TN, q = KK * TM + i;
            if (t == 0)
                wait_afrag(std::integral_constant<int, q>(), afr[q % RING_A]);
            multiply(acc[i][t], afr[q % RING_A], bfr[KK][t]);
            if (m == 0) {
                wait_words(words[NXT]);
                if (NEW_GROUP)
                    wait_group(raw_s, raw_z);
            }
            if (t == 0) {
                constexpr int ahead = q + RING_A - 1;
                read_afrag(ahead < KSTEPS * TM ? ring : ring_next, std::integral_constant<int, ahead % (KSTEPS * TM)>(),
                           afr[ahead % RING_A]);
            }
#pragma unroll
            for (int o = m * OPS / SLOTS; o < (m + 1) * OPS / SLOTS; ++o)
                prepare_op(o, NEW_GROUP, NXT, bfr[NXT]);
            if (t == TN - 1 && reads_words(q)) {
                read_words(ring_next, step, words[KK]);
                if (HALF || KK == 0)
                    read_group(ring_next, step, raw_s, raw_z);
            }
            extra(m);
            __builtin_amdgcn_sched_barrier(0);
        });
    };
    using Step0 = std::integral_constant<int, 0>;
    using Step1 = std::integral_constant<int, 1>;
    auto nothing = [](int) {};

    // ---- prologue: put NBUF-1 stages in flight, publish the first two, load the first operands ----
#pragma unroll
    for (int s = 0; s < NBUF - 1; ++s) {
#pragma unroll
        for (int p = 0; p < LOADS_PER_STAGE; ++p)
            issue_piece(p, s);
        advance_load_stage();
    }
    publish();
    if (HALF && (tail_stage == 0 || tail_stage == 1))
        clear_repeated_half(tail_stage);
    read_words(0, Step0{}, words[0]);
    read_group(0, Step0{}, raw_s, raw_z);
    asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(words[0]), "+v"(raw_s), "+v"(raw_z));
#pragma unroll
    for (int o = 0; o < GROUP_OPS + 16 * TN; ++o)
        prepare_op(o, true, 0, bfr[0]);
    // (in the order of the loop: the waits count on it)
    static_for<0, RING_A - 1>([&](auto operand) {
        constexpr int q = decltype(operand)::value, issued_in = in_prologue(q);
        read_afrag(0, operand, afr[q]);
        if (issued_in >= TM && reads_words(issued_in)) {
            read_words(0, Step1{}, words[1]);
            if (HALF)
                read_group(0, Step1{}, raw_s, raw_z);
        }
    });
    static_assert(RING_A - 1 >= TM - READ_AFTER, "the words of k step 1 are read");

    // Invariant at the top of stage s: stages s and s+1 are in LDS and visible, every wave has left stage s-1,
    // the B operands of its k step 0 sit in bfr[0], the words of its k step 1 in words[1], and its first RING_A - 1 A
    // operands are on their way.
    int ring = 0;  // s % NBUF
    for (int s = 0; s < stages; ++s) {
        const int ring_next = ring + 1 == NBUF ? 0 : ring + 1;
        const int ring_free = ring == 0 ? NBUF - 1 : ring - 1;  // buffer of stage s-1
        // the loads of stage s+NBUF-1 (into the buffer stage s-1 has left) are spread over the slots of the
        // first k step, so that they issue in the shadow of MFMAs like everything else
        constexpr int PIECES_PER_SLOT = (LOADS_PER_STAGE + SLOTS - 1) / SLOTS;
        auto issue_loads = [&](int m) {
#pragma unroll
            for (int q = 0; q < PIECES_PER_SLOT; ++q)
                if (m * PIECES_PER_SLOT + q < LOADS_PER_STAGE)
                    issue_piece(m * PIECES_PER_SLOT + q, ring_free);
        };
        kstep(Step0{}, ring, ring_next, issue_loads);
        kstep(Step1{}, ring, ring_next, nothing);
        advance_load_stage();
        publish();  // stage s+2 has landed; everyone is done with stage s
        if (HALF && s + 2 == tail_stage)
            clear_repeated_half(ring_next + 1 == NBUF ? 0 : ring_next + 1);
        ring = ring_next;
    }
    if (KW > 1 && stages < lead)
        publish();  // the other group's last barrier
    // nothing may still be writing this workgroup's LDS when it retires; the LDS wait retires the operand reads
    // issued for the stage after the last one, whose destination registers stay reserved until here (named as
    // in/outs after the wait: the compiler knows nothing of the inline-asm reads in flight and could otherwise
    // reuse the registers of these dead values while a read is still due to land in them)
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_nop 15" ::: "memory");
#pragma unroll
    for (int q = 0; q < RING_A; ++q)
        asm volatile("" : "+v"(afr[q]));
    asm volatile("" : "+v"(words[0]), "+v"(words[1]), "+v"(raw_s), "+v"(raw_z));
    if constexpr (TM * TN == 64)  // (no sum is read before the wait states that end the asm above)
        static_for<0, TM * TN>([&](auto n) {
            float4_t &c = acc[decltype(n)::value / TN][decltype(n)::value % TN];
            asm volatile("" : "+a"(c));
        });

    if (SERIAL) {
        if (group + 1 < groups) {
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int t = 0; t < TN; ++t)
                    half_sum[i][t] = acc[i][t];
            ++group;
        } else {
            // (as the sliced launch: two halves to a slice, and the slices to zero)
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int t = 0; t < TN; ++t)
                    total[i][t] += groups > 1 ? half_sum[i][t] + acc[i][t] : acc[i][t];
            group = 0;
            ++slice;
        }
        if (slice < a.serial_slices) {
            __syncthreads();  // every wavefront has its operands: the next loads may overwrite the ring
            continue;
        }
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int t = 0; t < TN; ++t)
                acc[i][t] = total[i][t];
    }
    break;
    }

    if (KW > 1) {
        // the second group's sums go to the first through LDS (the rings are done with: every DMA has landed),
        // four values per access, [value / 4][thread]
        static_assert(KW == 1 || TM * TN * 4 * kThreads * 4 <= KW * NBUF * L::BYTES, "the sums fit the rings");
        __syncthreads();
        float4_t *sums = reinterpret_cast<float4_t *>(smem_all) + tid;
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int t = 0; t < TN; ++t)
                if (kgroup == 1)
                    sums[(i * TN + t) * kThreads] = acc[i][t];
        __syncthreads();
        if (kgroup == 0) {
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int t = 0; t < TN; ++t)
                    acc[i][t] += sums[(i * TN + t) * kThreads];
        }
    }
    if (!SERIAL && a.split_k > 1) {
        constexpr int ACC = TM * TN * 4;
        float flat[ACC];
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int t = 0; t < TN; ++t)
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    flat[(i * TN + t) * 4 + r] = acc[i][t][r];
        if (!combine_slices<ACC>(flat, a, slice, tile_id, tid, kgroup == 0))
            return;
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int t = 0; t < TN; ++t)
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    acc[i][t][r] = flat[(i * TN + t) * 4 + r];
    }
    if (kgroup == 0)
        store_blocks<TM, TN>(acc, a.out, m0 + wm * WAVE_M, col_raw, col_ok, kg, M, N);
}

// =====================================================================================================
// General path (g_idx, any group size, k tail): registers -> LDS, two buffers, one barrier per stage
// =====================================================================================================

template <int BM, int BN, int WM, int WN, int MODE>
__global__ __launch_bounds__(kThreads) void prefill_general_kernel(const Args a)
{
    static_assert(WM * WN == 4, "four wavefronts per workgroup");
    static_assert(MODE == kGroupPerRow || MODE == kActOrder, "the tuned modes use the pipelined kernel");
    constexpr int BK = 64;
    constexpr int WAVE_M = BM / WM;
    constexpr int WAVE_N = BN / WN;
    constexpr int TM = WAVE_M / 32;
    constexpr int TN = WAVE_N / 32;
    static_assert(TM >= 1 && (TN == 1 || TN == 2 || TN == 4), "wave tile: 32-row blocks by 32/64/128 columns");
    constexpr int A_CHUNKS = BM * (BK / 8) / kThreads;
    static_assert(A_CHUNKS >= 1, "tile too small for 256 threads");
    constexpr int KSTEPS = BK / 16;
    constexpr int STAGE_HALVES = BM * BK;

    extern __shared__ __align__(16) unsigned char smem[];
    half_t *lds_a = reinterpret_cast<half_t *>(smem);  // [2][BM][64] halves, chunk-swizzled

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = tid >> 6;
    const int wm = wave / WN;
    const int wn = wave % WN;
    const int lj = lane & 31;
    const int kh = lane >> 5;

    int tile_m, tile_n;
    int tile_id, slice;
    if (!tile_of_workgroup(a, tile_m, tile_n, tile_id, slice))
        return;
    const int m0 = tile_m * BM;
    const int n0 = tile_n * BN;
    const int N = a.N, K = a.K, M = a.M;
    const int rows = K >> 3;
    const int col_raw = n0 + wn * WAVE_N + TN * lj;
    const bool col_ok = col_raw < N;
    const int col0 = col_ok ? col_raw : N - TN;  // clamped: see the pipelined kernel
    const int zshift = 4 * (col0 & 7);
    const int stages = (K + BK - 1) / BK;

    float16_t acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int t = 0; t < TN; ++t)
#pragma unroll
            for (int r = 0; r < 16; ++r)
                acc[i][t][r] = 0.f;

    // slot p (16 bytes) holds chunk (p & 7) ^ ((row >> 1) & 7) of row p >> 3 (64 banks, 16 lanes per pass)
    const half_t *a_src[A_CHUNKS];
#pragma unroll
    for (int c = 0; c < A_CHUNKS; ++c) {
        const int slot = tid + c * kThreads;
        const int row = slot >> 3;
        const int ch = (slot & 7) ^ ((row >> 1) & 7);
        a_src[c] = a.x + (size_t)min(m0 + row, M - 1) * K + ch * 8;
    }
    uint4 a_next[A_CHUNKS];
    auto load_a = [&](int stage) {
        const int k0 = stage * BK;
#pragma unroll
        for (int c = 0; c < A_CHUNKS; ++c) {
            const int slot = tid + c * kThreads;
            const int ch = (slot & 7) ^ ((slot >> 4) & 7);
            const int k = k0 + ch * 8;
            const uint4 v = *reinterpret_cast<const uint4 *>(a_src[c] + min(k0, K - 8 - ch * 8));
            a_next[c] = k < K ? v : make_uint4(0, 0, 0, 0);  // the k tail must contribute exact zeros
        }
    };
    auto store_a = [&](int buf) {
#pragma unroll
        for (int c = 0; c < A_CHUNKS; ++c) {
            const int slot = tid + c * kThreads;
            *reinterpret_cast<uint4 *>(lds_a + (size_t)buf * STAGE_HALVES + (size_t)slot * 8) = a_next[c];
        }
    };
    uint32_t w_cur[KSTEPS][TN], w_nxt[KSTEPS][TN];
    auto load_b = [&](int stage, uint32_t (&w)[KSTEPS][TN]) {
        const int prow0 = stage * (BK / 8);
#pragma unroll
        for (int kk = 0; kk < KSTEPS; ++kk) {
            const int prow = min(prow0 + 2 * kk + kh, rows - 1);
            const uint32_t *src = a.qweight + (size_t)prow * N + col0;
            if (TN == 4) {
                const uint4 v = *reinterpret_cast<const uint4 *>(src);
                w[kk][0] = v.x;
                w[kk][1 % TN] = v.y;
                w[kk][2 % TN] = v.z;
                w[kk][3 % TN] = v.w;
            } else if (TN == 2) {
                const uint2 v = *reinterpret_cast<const uint2 *>(src);
                w[kk][0] = v.x;
                w[kk][1 % TN] = v.y;
            } else {
                w[kk][0] = *src;
            }
        }
    };
    const PairMagic magic;

    // B operands of k step `kk` of stage `s`, dequantised in registers
    auto make_bfrags = [&](int s, int kk, u32x4_t bfrag[TN]) {
        const int prow = s * (BK / 8) + 2 * kk + kh;  // this lane's packed row
#pragma unroll
        for (int t = 0; t < TN; ++t) {
            uint32_t nz[4] = {0, 0, 0, 0}, ss[4] = {0, 0, 0, 0};
            if (prow < rows) {  // past the k tail the scale stays zero: exact zero weights
                if (MODE == kGroupPerRow) {
                    const int g = (prow * 8) / a.group_size;
                    const uint32_t sb = __builtin_bit_cast(uint16_t, a.scales[(size_t)g * N + col0 + t]);
                    const uint32_t z = (a.qzeros[(size_t)g * (N >> 3) + (col0 >> 3)] >> (zshift + 4 * t)) & 15u;
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        nz[i] = neg_bias(z);
                        ss[i] = sb | (sb << 16);
                    }
                } else {
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const int g0 = a.g_idx[prow * 8 + 2 * i];
                        const int g1 = a.g_idx[prow * 8 + 2 * i + 1];
                        const uint32_t s0 = __builtin_bit_cast(uint16_t, a.scales[(size_t)g0 * N + col0 + t]);
                        const uint32_t s1 = __builtin_bit_cast(uint16_t, a.scales[(size_t)g1 * N + col0 + t]);
                        const uint32_t z0 = (a.qzeros[(size_t)g0 * (N >> 3) + (col0 >> 3)] >> (zshift + 4 * t)) & 15u;
                        const uint32_t z1 = (a.qzeros[(size_t)g1 * (N >> 3) + (col0 >> 3)] >> (zshift + 4 * t)) & 15u;
                        nz[i] = 0xD400E400u | z0 | (z1 << 20);
                        ss[i] = s0 | (s1 << 16);
                    }
                }
            }
            bfrag[t] = dequant_word(w_cur[kk][t], magic, nz, ss);
        }
    };
    auto read_afrags = [&](const half_t *base, int kk, half8_t af[TM]) {
#pragma unroll
        for (int i = 0; i < TM; ++i) {
            const int row = wm * WAVE_M + i * 32 + lj;
            const int ch = (2 * kk + kh) ^ ((row >> 1) & 7);
            af[i] = *reinterpret_cast<const half8_t *>(base + (size_t)row * BK + ch * 8);
        }
    };

    half8_t af[2][TM];
    u32x4_t bf[2][TN];
    load_a(0);
    load_b(0, w_cur);
    store_a(0);
    __syncthreads();
    for (int s = 0; s < stages; ++s) {
        const int buf = s & 1;
        const int sn = min(s + 1, stages - 1);  // the last iteration harmlessly refetches its own stage
        load_a(sn);
        load_b(sn, w_nxt);
        const half_t *base = lds_a + (size_t)buf * STAGE_HALVES;
        read_afrags(base, 0, af[0]);
        make_bfrags(s, 0, bf[0]);
#pragma unroll
        for (int kk = 0; kk < KSTEPS; ++kk) {
            if (kk + 1 < KSTEPS) {
                read_afrags(base, kk + 1, af[(kk + 1) & 1]);
                make_bfrags(s, kk + 1, bf[(kk + 1) & 1]);
            }
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int t = 0; t < TN; ++t)
                    acc[i][t] = __builtin_amdgcn_mfma_f32_32x32x16_f16(
                        af[kk & 1][i], __builtin_bit_cast(half8_t, bf[kk & 1][t]), acc[i][t], 0, 0, 0);
        }
        store_a(buf ^ 1);
#pragma unroll
        for (int kk = 0; kk < KSTEPS; ++kk)
#pragma unroll
            for (int t = 0; t < TN; ++t)
                w_cur[kk][t] = w_nxt[kk][t];
        __syncthreads();
    }

    store_tile<TM, TN>(acc, a.out, m0 + wm * WAVE_M, col_raw, col_ok, kh, M, N);
}

}  // namespace prefill
}  // namespace gptq
