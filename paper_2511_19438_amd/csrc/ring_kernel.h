// Small-batch MFMA kernel on a ring of LDS slots (2 <= M <= 48, on narrow layers 64; no g_idx, K a multiple of 128), gfx950.
//
// A layer of 4-25 MB takes 3-6 us to read, launch included; what a small batch costs above that is the price of everything
// around the packed words.  Measured on the variant that loads both operands straight into registers (skinny_kernel.h,
// which this one replaced for these formats; 4096x4096, 4096x12288, 4096x22016 and 11008x4096, M = 8 and 32, parts of
// the kernel taken out in copies of it):
//   * the activations, 64 bytes of each of 16 rows per load instruction: 0.5-2.5 us at 16 rows, 2-8 us at 32.  One
//     workgroup needs M * K * 2 bytes of them whatever its width, all through its compute unit's 64 bytes per clock;
//   * partial sums of K slices through scratch: 2.4 us of the 5.4 us that 4096x4096 spent in its workgroups;
//   * 172-192 busy compute units of 256 where the width did not divide well by 64 or 128.
// Hence:
//   * A workgroup owns 32, 64, 96 or 128 columns and, wherever the columns alone give enough workgroups, all of K: eight
//     wavefronts split it, their sums meet in LDS, and nothing goes through scratch.  (A plain read of 4096x4096 in 128
//     strips of 32 columns takes 3.5 us, of 4096x22016 in 230 strips of 96 9.5 us, in 344 of 64 11.)
//   * Packed words, activations, scales and zero points all travel global -> LDS by DMA, in whole pieces: 1 KB of
//     adjacent words, 8 rows x 128 bytes of x, one instruction for the scales and zero points of a group.  The loads of a
//     64-k stage are LW + LX + 1 instructions (3 for 32 columns and 8 rows) where registers took 16 per 128 k, and no
//     register waits for a load: a stage waits once for its loads, once for its LDS reads, and no barrier stands in the loop.
//   * The ring is short (two or three stages).  Longer ones measured slower at every size (4096x4096, M = 8, 32
//     columns: three stages 5.3 us, four 5.5, five 5.7, six 6.0).
// The arithmetic is skinny_kernel's: B operand = exact q - z, scaled per group in fp32.
//
// 33-48 rows: a third row block.  The mid-batch kernel, which served them, pads to 64 rows with one wavefront per SIMD; here
// two share it, and nothing but the rows' own activations is loaded or multiplied.  us at M = 40, mid-batch -> ring:
// 4096x12288 14.0 -> 12.7, 4096x4096 10.6 -> 7.4, 4096x22016 21.9 -> 17.2, 11008x4096 15.8 -> 14.2, 8192x10240 22.9 -> 20.0,
// 8192x8192 19.0 -> 16.9, 8192x57344 86.9 -> 76.4, 28672x8192 46.4 -> 40.8.  128 columns do not fit 256 registers then.  A
// fourth block (49-64 rows) leaves room in the LDS for eight wavefronts of 32 columns only and pays where those are one
// unsplit round (4096x4096 at M = 64: 12.0 -> 9.3); in 64 columns it was level with the mid-batch kernel or behind it.
#pragma once

#include "lds_dma.h"
#include "skinny_kernel.h"

namespace gptq {
namespace skinny {

typedef uint32_t u32x2_t __attribute__((ext_vector_type(2)));
typedef float f32x2_t __attribute__((ext_vector_type(2)));

constexpr int kStageK = 64;  // k per ring slot: two MFMA steps
constexpr int kUnitStages = kUnitK / kStageK;

// Layout of a slot.  LX: DMA instructions of its activations (8 rows each).  GPU: groups per 128-k unit (1: of 128 k and
// more, whose scales come with a unit's first stage only).
template <int COLS, int LX, int GPU>
struct RingSlot {
    static constexpr int W_BYTES = COLS * 32;                   // [8 packed rows][COLS] words
    static constexpr int X_BYTES = LX * 1024;                   // [8 LX rows][64] halves, 16-byte chunks swizzled
    static constexpr int SZ_LOADS = COLS <= 96 ? 1 : 2;         // of one group: COLS / 2 + COLS / 8 words
    static constexpr int SZ_BYTES = SZ_LOADS * 256;             // scales [COLS] halves, zero words [COLS / 8], padding
    static constexpr int GROUPS = GPU == 4 ? 2 : 1;             // groups of a stage
    static constexpr int BYTES = W_BYTES + X_BYTES + GROUPS * SZ_BYTES;
};

// TM: 16-row blocks.  LX: as above; rows that are not loaded repeat loaded ones, their outputs are not stored.
// NF, NH: a lane's columns, NF times four (64 columns of the tile each) and NH times two (32 columns).
// WAVES: eight wavefronts split the K slice, or four where there are more workgroups than compute units (ring_waves).
// Registers: two wavefronts share a SIMD, those of one workgroup or of two.  Unbounded, the compiler gave the instances of
// groups of 32, 17-32 rows and four wavefronts 280 (96 columns) and 356 (128), one workgroup to a compute unit; bounded it
// finds room for the same loop in 188 and 234 (8192x57344, groups of 32, 128 columns, M = 24: 106.5 us -> 72.7).
// SERIAL: no scratch for the K slices.  A workgroup walks all slices of its tile one after the other and adds their sums
// in registers, in slice order: the bits of the sliced launch, whose tile may be any (an output's sum does not depend on
// it).  For eight wavefronts of 64 columns, or 32 where the rows have no other width (kSerialCols).
template <int TM, int LX, int NF, int NH, int WAVES, int GPU, int DEPTH, bool STREAM,
          bool SERIAL = false>
__global__ __launch_bounds__(64 * WAVES, 2) void ring_kernel(const Args a)
{
    static_assert(DEPTH == 2 || DEPTH == 3, "the waits below");
    static_assert(!SERIAL || (WAVES == 8 && NF + NH == 1), "one serial width, see there");
    constexpr int kThreads = 64 * WAVES;
    constexpr int ROWS = 16 * TM;
    constexpr int NT = 4 * NF + 2 * NH;
    constexpr int COLS = 16 * NT;
    using Slot = RingSlot<COLS, LX, GPU>;
    constexpr int LW = Slot::W_BYTES / 1024;
    constexpr int LS = Slot::GROUPS * Slot::SZ_LOADS;
    // loads of a unit's first stage and of its second
    constexpr int LOADS0 = LW + LX + LS, LOADS1 = LW + LX + (GPU > 1 ? LS : 0);
    constexpr int XROWS = 8 * LX;
    constexpr int QUADS = COLS / 4;
    constexpr int PER_THREAD = (ROWS * QUADS + kThreads - 1) / kThreads;  // quads of the tile that a thread adds up
    static_assert(XROWS <= ROWS && XROWS > ROWS - 16, "every row block has rows of its own");

    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ int s_last;

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int cq = lane & 15;  // column group of the lane; A operand: row of a block
    const int kg = lane >> 4;  // packed row inside a 32-k step
    int tile = blockIdx.x, slice = 0;
    if (a.split_k > 1) {
        slice = tile / a.tiles_n;
        tile -= slice * a.tiles_n;
    }
    const int N = a.N;
    float4_t total[SERIAL ? PER_THREAD : 1];  // SERIAL: the thread's quads of the tile, over the slices so far
#pragma unroll
    for (float4_t &t : total)
        t = float4_t{0.f, 0.f, 0.f, 0.f};
    for (;;) {  // (a single pass unless SERIAL; the body, up to the sums over the wavefronts, is not indented)
    const int u0 = slice * a.units_per_slice;
    const int u1 = min(u0 + a.units_per_slice, a.total_units);
    const int per_wave = (u1 - u0 + WAVES - 1) / WAVES;
    const int wu0 = min(u0 + wave * per_wave, u1);
    const int wu1 = min(wu0 + per_wave, u1);

    // ---- DMA sources: a wavefront-uniform base that advances from stage to stage and a byte offset per lane ----
    uint32_t off_w[LW];
#pragma unroll
    for (int q = 0; q < LW; ++q) {
        const int chunk = q * 64 + lane;  // of the stage's 8 packed rows, COLS / 4 chunks each
        const int row = chunk / (COLS / 4);
        off_w[q] = ((uint32_t)row * N + min(tile * COLS + 4 * (chunk % (COLS / 4)), N - 4)) * 4u;  // (past N: not stored)
    }
    uint32_t off_x[LX];
#pragma unroll
    for (int q = 0; q < LX; ++q) {
        const int row = 8 * q + (lane >> 3);
        off_x[q] = ((uint32_t)min(row, a.M - 1) * a.K + (uint32_t)((lane & 7) ^ (row >> 1 & 7)) * 8) * 2u;
    }
    const char *w_next = reinterpret_cast<const char *>(a.qweight + (size_t)wu0 * 16 * N);
    const char *x_next = reinterpret_cast<const char *>(a.x + (size_t)wu0 * kUnitK);
    const size_t w_step = (size_t)N * 32;
    int group, in_group = 0;
    if (GPU > 1) {
        group = wu0 * GPU;
    } else {
        group = a.unit_group_shift >= 0 ? wu0 >> a.unit_group_shift : wu0 / a.units_per_group;
        in_group = wu0 - group * a.units_per_group;
    }
    const char *sz_next[Slot::SZ_LOADS];  // per lane: two scales, or a zero word
    uint32_t sz_step[Slot::SZ_LOADS];
#pragma unroll
    for (int j = 0; j < Slot::SZ_LOADS; ++j) {
        const int i = 64 * j + lane;
        const bool scales = i < COLS / 2;
        const int n = scales ? min(tile * COLS + 2 * i, N - 2)
                             : min(tile * COLS + 8 * min(i - COLS / 2, COLS / 8 - 1), N - 8);
        sz_next[j] = scales ? reinterpret_cast<const char *>(a.scales + (size_t)group * N + n)
                            : reinterpret_cast<const char *>(a.qzeros + ((size_t)group * N + n) / 8);
        sz_step[j] = scales ? (uint32_t)N * 2u : (uint32_t)N / 2u;
    }

    const unsigned char *const ring = smem + (size_t)wave * (DEPTH * Slot::BYTES);
    const uint32_t ring_lds = __builtin_amdgcn_readfirstlane(
        (uint32_t)(uintptr_t)(__attribute__((address_space(3))) const unsigned char *)ring);
    int left = (wu1 - wu0) * kUnitStages;  // stages whose loads have not been issued
    uint32_t put = ring_lds;               // the slot that is filled next
    auto issue = [&](bool first_of_unit) {
#pragma unroll
        for (int q = 0; q < LW; ++q)
            dma_16<STREAM>(put + q * 1024, off_w[q], w_next);
        if (GPU > 1 || first_of_unit) {
#pragma unroll
            for (int g = 0; g < Slot::GROUPS; ++g) {
                bool step = true;
                if (GPU == 1) {
                    step = ++in_group == a.units_per_group;
                    in_group = step ? 0 : in_group;
                }
#pragma unroll
                for (int j = 0; j < Slot::SZ_LOADS; ++j) {
                    dma_4(put + Slot::W_BYTES + Slot::X_BYTES + g * Slot::SZ_BYTES + j * 256, sz_next[j]);
                    sz_next[j] += step ? sz_step[j] : 0u;
                }
            }
        }
#pragma unroll
        for (int q = 0; q < LX; ++q)
            dma_16(put + Slot::W_BYTES + q * 1024, off_x[q], x_next);
        w_next += w_step;
        x_next += kStageK * 2;
        put += Slot::BYTES;
        put = put == ring_lds + DEPTH * Slot::BYTES ? ring_lds : put;
        --left;
    };

    // ---- operand addresses inside a slot ----
    uint32_t a_off[TM];  // row of block i, chunk kg; a step further is chunk kg + 4: a flipped bit, swizzled or not
#pragma unroll
    for (int i = 0; i < TM; ++i) {
        const int row = 16 * i + cq < XROWS ? 16 * i + cq : cq % (XROWS < 16 ? XROWS : 16);
        a_off[i] = (uint32_t)Slot::W_BYTES + row * 128u + ((uint32_t)(kg ^ (row >> 1 & 7)) << 4);
    }
    struct Words {
        u32x4_t f[NF > 0 ? NF : 1];
        u32x2_t h;
    };
    auto read_step = [&](const unsigned char *slot, int st, Words &w, u32x4_t (&x)[TM]) {
        const unsigned char *row = slot + (4 * st + kg) * (COLS * 4);
#pragma unroll
        for (int b = 0; b < NF; ++b)
            w.f[b] = *reinterpret_cast<const u32x4_t *>(row + b * 256 + cq * 16);
        if (NH)
            w.h = *reinterpret_cast<const u32x2_t *>(row + NF * 256 + cq * 8);
#pragma unroll
        for (int i = 0; i < TM; ++i)
            x[i] = *reinterpret_cast<const u32x4_t *>(slot + (a_off[i] ^ (uint32_t)(st << 6)));
    };

    float4_t acc[TM][NT];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int t = 0; t < NT; ++t)
            acc[i][t] = float4_t{0.f, 0.f, 0.f, 0.f};
    const NibbleMagic magic;
    constexpr int SPG = 4 / GPU;  // 32-k steps per quantisation group

    if (wu0 < wu1) {
#pragma unroll
        for (int i = 0; i < DEPTH - 1; ++i)  // (two stages at least: a unit has two)
            issue(i == 0);
        uint32_t get = 0;
        for (int u = wu0; u < wu1; ++u) {
            float4_t d[TM][NT];
            half2_t neg_lo[NT], neg_hi[NT];
            float sf[NT];
#pragma unroll
            for (int s = 0; s < kUnitStages; ++s) {
                // The stage has arrived once no more than the loads of the DEPTH - 1 stages after it are outstanding, or
                // of as many as there still are.
                constexpr int kBoth = LOADS0 + LOADS1;
                if (left > 0) {
                    issue((s + DEPTH - 1) % kUnitStages == 0);
                    if (DEPTH == 3)
                        wait_loads<kBoth>();
                    else if (s == 0)
                        wait_loads<LOADS1>();
                    else
                        wait_loads<LOADS0>();
                } else if (DEPTH == 3 && s == 0) {
                    wait_loads<LOADS1>();
                } else {  // the last stage (a ring of three is past its last load one stage before)
                    wait_loads<0>();
                }
                const unsigned char *slot = ring + get;
                Words w[2];
                u32x4_t x[2][TM];
                read_step(slot, 0, w[0], x[0]);
#pragma unroll
                for (int st = 0; st < 2; ++st) {
                    const int step = 2 * s + st;  // of the unit
                    if (step % SPG == 0) {        // a group begins: its zero points and scales
                        const unsigned char *sz =
                            slot + Slot::W_BYTES + Slot::X_BYTES + (GPU == 4 ? st : 0) * Slot::SZ_BYTES;
#pragma unroll
                        for (int b = 0; b < NF + NH; ++b) {
                            const int col = b < NF ? b * kCols + 4 * cq : NF * kCols + 2 * cq;
                            const uint32_t zeros =
                                *reinterpret_cast<const uint32_t *>(sz + COLS * 2 + (col >> 3) * 4) >> (4 * (col & 7));
                            uint32_t pair[2];
                            pair[0] = *reinterpret_cast<const uint32_t *>(sz + col * 2);
                            pair[1] = b < NF ? *reinterpret_cast<const uint32_t *>(sz + col * 2 + 4) : 0u;
#pragma unroll
                            for (int j = 0; j < (b < NF ? 4 : 2); ++j) {
                                const uint32_t z = zeros >> (4 * j) & 15u;
                                const uint32_t zz = z | (z << 16);
                                neg_lo[4 * b + j] = as_half2(zz | 0xE400E400u);         // (-(1024 + z)) x2
                                neg_hi[4 * b + j] = as_half2((zz << 4) | 0xD400D400u);  // (-(64 + z)) x2
                                const uint16_t bits = (uint16_t)((j & 1) ? pair[j / 2] >> 16 : pair[j / 2] & 0xffffu);
                                sf[4 * b + j] = (float)__builtin_bit_cast(half_t, bits);
                            }
                        }
                    }
                    if (st == 0) {
                        read_step(slot, 1, w[1], x[1]);  // in flight under this step's arithmetic
                        __builtin_amdgcn_sched_barrier(0);
                    }
                    half8_t av[TM];
#pragma unroll
                    for (int i = 0; i < TM; ++i) {  // the k order of the weights: halves (0,4) (1,5) (2,6) (3,7)
                        const u32x4_t xv = x[st][i];
                        const u32x4_t xp = {__builtin_amdgcn_perm(xv[2], xv[0], 0x05040100u),
                                            __builtin_amdgcn_perm(xv[2], xv[0], 0x07060302u),
                                            __builtin_amdgcn_perm(xv[3], xv[1], 0x05040100u),
                                            __builtin_amdgcn_perm(xv[3], xv[1], 0x07060302u)};
                        av[i] = __builtin_bit_cast(half8_t, xp);
                    }
#pragma unroll
                    for (int t = 0; t < NT; ++t) {
                        const uint32_t word = t < 4 * NF ? w[st].f[t < 4 * NF ? t / 4 : 0][t % 4] : w[st].h[t % 2];
                        const uint32_t w8 = word >> 8;
                        const half2_t c0 = as_half2((word & magic.mask_lo) | magic.bias_lo) + neg_lo[t];
                        const half2_t c1 = as_half2((word & magic.mask_hi) | magic.bias_hi) + neg_hi[t];
                        const half2_t c2 = as_half2((w8 & magic.mask_lo) | magic.bias_lo) + neg_lo[t];
                        const half2_t c3 = as_half2((w8 & magic.mask_hi) | magic.bias_hi) + neg_hi[t];
                        const half8_t b = half8_t{c0[0], c0[1], c1[0], c1[1], c2[0], c2[1], c3[0], c3[1]};
                        const float4_t zero = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                        for (int i = 0; i < TM; ++i)
                            d[i][t] = __builtin_amdgcn_mfma_f32_16x16x32_f16(av[i], b, step % SPG == 0 ? zero : d[i][t], 0,
                                                                             0, 0);
                    }
                    if (step % SPG == SPG - 1) {  // the group is complete: scale its sum
#pragma unroll
                        for (int t = 0; t < NT; ++t)
#pragma unroll
                            for (int i = 0; i < TM; ++i)
#pragma unroll
                                for (int r = 0; r < 4; ++r)
                                    acc[i][t][r] = __builtin_fmaf(sf[t], d[i][t][r], acc[i][t][r]);
                    }
                }
                get += Slot::BYTES;
                get = get == (uint32_t)(DEPTH * Slot::BYTES) ? 0u : get;
                // The next turn fills this slot again: its reads have to be done.  Not all of them have been used: with
                // groups of 32 the scales of the last step belong to multiply-adds that the compiler moves behind this point.
                asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
                __builtin_amdgcn_sched_barrier(0);
            }
        }
    }

    // ---- the wavefronts meet in LDS (the rings are reused: every DMA has landed), fixed order ----
    __syncthreads();
    float *red = reinterpret_cast<float *>(smem);  // [WAVES][ROWS][COLS]
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            float *row = red + ((size_t)wave * ROWS + 16 * i + 4 * kg + r) * COLS;
#pragma unroll
            for (int b = 0; b < NF; ++b)
                *reinterpret_cast<float4_t *>(row + b * kCols + 4 * cq) =
                    float4_t{acc[i][4 * b][r], acc[i][4 * b + 1][r], acc[i][4 * b + 2][r], acc[i][4 * b + 3][r]};
            if (NH)
                *reinterpret_cast<f32x2_t *>(row + NF * kCols + 2 * cq) = f32x2_t{acc[i][4 * NF][r], acc[i][4 * NF + 1][r]};
        }
    __syncthreads();
    auto add_up = [&](int e, float4_t &sum) {
        const int m = e / QUADS;
        const int col = (e - m * QUADS) * 4;
        const int n = tile * COLS + col;
        float4_t s = *reinterpret_cast<const float4_t *>(red + (size_t)m * COLS + col);
#pragma unroll
        for (int w = 1; w < WAVES; ++w)
            s += *reinterpret_cast<const float4_t *>(red + ((size_t)w * ROWS + m) * COLS + col);
        if (SERIAL) {
            sum += s;
            s = sum;
        }
        if (n >= N || (SERIAL && slice + 1 < a.serial_slices))
            return;
        if (a.split_k == 1) {
            *reinterpret_cast<half4_t *>(a.out + (size_t)m * N + n) =
                half4_t{(half_t)s[0], (half_t)s[1], (half_t)s[2], (half_t)s[3]};
        } else if (a.slots) {
            unsigned long long *slot = a.slots + ((size_t)m * N + n) / 2;
            f32x2_t lo = {s[0], s[1]}, hi = {s[2], s[3]};
            const unsigned long long found_lo = slot_swap(slot, lo), found_hi = slot_swap(slot + 1, hi);
            if (slot_collect(slot, found_lo, lo))
                *reinterpret_cast<half2_t *>(a.out + (size_t)m * N + n) = half2_t{(half_t)lo[0], (half_t)lo[1]};
            if (slot_collect(slot + 1, found_hi, hi))
                *reinterpret_cast<half2_t *>(a.out + (size_t)m * N + n + 2) = half2_t{(half_t)hi[0], (half_t)hi[1]};
        } else {
            unsigned long long *dst =
                reinterpret_cast<unsigned long long *>(a.partial + ((size_t)slice * a.M + m) * N + n);
            __hip_atomic_store(dst, __builtin_bit_cast(unsigned long long, f32x2_t{s[0], s[1]}), __ATOMIC_RELAXED,
                               __HIP_MEMORY_SCOPE_AGENT);
            __hip_atomic_store(dst + 1, __builtin_bit_cast(unsigned long long, f32x2_t{s[2], s[3]}), __ATOMIC_RELAXED,
                               __HIP_MEMORY_SCOPE_AGENT);
        }
    };
    if constexpr (SERIAL) {
#pragma unroll
        for (int j = 0; j < PER_THREAD; ++j)
            if (tid + j * kThreads < a.M * QUADS)
                add_up(tid + j * kThreads, total[j]);
    } else {
        for (int e = tid; e < a.M * QUADS; e += kThreads)
            add_up(e, total[0]);
    }

    if (!SERIAL || ++slice >= a.serial_slices)
        break;
    __syncthreads();  // the sums have been read: the next slice's stages may take their place
    }

    // ---- K slices across workgroups: the last one of this column tile to arrive adds them in slice order ----
    if (a.split_k > 1 && !a.slots) {
        __builtin_amdgcn_s_waitcnt(0);  // every partial store of this workgroup has been acknowledged (exchange.h)
        __syncthreads();
        if (tid == 0)
            s_last = (slice_arrive(a.counters + tile) == (unsigned)(a.split_k - 1));
        __syncthreads();
        if (s_last) {
            slice_acquire();
            for (int e = tid; e < a.M * QUADS; e += kThreads) {
                const int m = e / QUADS;
                const int n = tile * COLS + (e - m * QUADS) * 4;
                if (n >= N)
                    continue;
                const size_t off = (size_t)m * N + n;
                float4_t s = {0.f, 0.f, 0.f, 0.f};
                for (int sl0 = 0; sl0 < a.split_k; sl0 += 8) {  // eight slices are requested before the first is used
                    unsigned long long v[8][2];
#pragma unroll
                    for (int j = 0; j < 8; ++j) {
                        const int sl = min(sl0 + j, a.split_k - 1);
                        const unsigned long long *src =
                            reinterpret_cast<const unsigned long long *>(a.partial + (size_t)sl * a.M * N + off);
                        v[j][0] = __hip_atomic_load(src, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                        v[j][1] = __hip_atomic_load(src + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    }
#pragma unroll
                    for (int j = 0; j < 8; ++j) {
                        const bool keep = sl0 + j < a.split_k;  // (a select: 0 * infinity would be a NaN)
                        const f32x2_t lo = __builtin_bit_cast(f32x2_t, v[j][0]);
                        const f32x2_t hi = __builtin_bit_cast(f32x2_t, v[j][1]);
                        s[0] += keep ? lo[0] : 0.f;
                        s[1] += keep ? lo[1] : 0.f;
                        s[2] += keep ? hi[0] : 0.f;
                        s[3] += keep ? hi[1] : 0.f;
                    }
                }
                *reinterpret_cast<half4_t *>(a.out + off) =
                    half4_t{(half_t)s[0], (half_t)s[1], (half_t)s[2], (half_t)s[3]};
            }
            if (tid == 0)
                __hip_atomic_store(a.counters + tile, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
    }
}

}  // namespace skinny
}  // namespace gptq
