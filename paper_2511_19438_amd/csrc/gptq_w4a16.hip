// C-ABI entry points of the W4A16 GPTQ library: argument validation, kernel choice, scratch.
// The contract of every function is stated in include/gptq_w4a16.h.
#include "gptq_w4a16.h"

#include <mutex>
#include <vector>

#include "kernels.h"

namespace {

using namespace gptq;

constexpr int kVersion = 100;  // 0.1.0
constexpr int kMaxDevices = 16;
constexpr int kDecodeMaxM = 16;

struct Workspace {
    void *ptr = nullptr;
    size_t bytes = 0;  // without the slots
    bool owned = false;
};

// Scratch of a launch: the block, and the slots of two-slice exchanges (exchange.h) behind it where the library owns it.
// A caller's workspace has none: the same launches then exchange through partial sums, with the same result.
struct Scratch {
    void *ws = nullptr;
    void *slots = nullptr;
};

std::mutex g_mutex;
Workspace g_ws[kMaxDevices];
std::vector<void *> g_retired[kMaxDevices];  // outgrown library-owned blocks, still referenced by earlier work

// Scratch of gptq_w4a16_gemm_static(): a fixed block in every device's copy of the code object, for callers
// that may not allocate.  The array's name is only a host-side handle; its device address is looked up once
// per device (static_scratch_ptr) and that pointer is what kernels and fills receive.
constexpr size_t kStaticScratchBytes = GPTQ_STATIC_SCRATCH_BYTES;
void *g_static_ptr[kMaxDevices] = {};

}  // namespace

static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes + kSlotBytes];

namespace {

// The current device's static scratch; the first call on a device looks its address up.  No allocation, and nothing to
// clear: the array has static storage, so that the arrival counters at its front and the slots at its end are zero when the
// code object is loaded, and every launch leaves them zero.
int static_scratch_ptr(Scratch *out)
{
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices)
        return GPTQ_HIP_ERROR;
    std::lock_guard<std::mutex> lock(g_mutex);
    if (!g_static_ptr[dev]) {
        void *ptr = nullptr;
        if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess || !ptr)
            return GPTQ_HIP_ERROR;
        g_static_ptr[dev] = ptr;
    }
    out->ws = g_static_ptr[dev];
    out->slots = static_cast<unsigned char *>(g_static_ptr[dev]) + kStaticScratchBytes;
    return GPTQ_OK;
}

bool aligned16(const void *p)
{
    return (reinterpret_cast<uintptr_t>(p) & 15u) == 0;
}

int check_shape(int K, int N, int group_size)
{
    if (K <= 0 || N <= 0 || group_size <= 0)
        return GPTQ_INVALID_ARG;
    if (K % 8 || N % 8 || group_size % 8 || K % group_size)
        return GPTQ_UNSUPPORTED_SHAPE;
    // The kernels address with 32-bit byte offsets from 64-bit bases: the packed weights (K*N/2 bytes) must
    // stay under 4 GiB, a tile's rows of x (256 * K * 2 bytes) too, and row / column numbers under 2^24
    // (24-bit multiplies).  Real layers are three orders of magnitude below these limits.
    if (K >= (1 << 23) || N >= (1 << 24) || (long long)K * N >= (1LL << 33))
        return GPTQ_UNSUPPORTED_SHAPE;
    return GPTQ_OK;
}

// Clears device memory and returns when that has happened: a memset of device memory may return before it is done, and
// the streams that use the memory next need not wait for the null stream it runs on (hipStreamNonBlocking).
bool clear_now(void *p, size_t bytes)
{
    return hipMemset(p, 0, bytes) == hipSuccess && hipStreamSynchronize(nullptr) == hipSuccess;
}

// Makes sure the current device has scratch of at least `bytes`; returns it in *out.
//
// Library-owned scratch only ever grows, and a block that has been handed to a launch is never freed while the
// library keeps its own scratch: launches still in flight and HIP graphs captured earlier hold its address (partial
// sums, arrival counters, gathered activations).  A block that became too small is retired instead and stays
// valid; retired blocks are released by gptq_w4a16_set_workspace().  Growth allocates and clears memory, which is
// not allowed while `stream` is being captured: such a call is refused.
int acquire_workspace(size_t bytes, hipStream_t stream, Scratch *out)
{
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices)
        return GPTQ_HIP_ERROR;
    std::lock_guard<std::mutex> lock(g_mutex);
    Workspace &ws = g_ws[dev];
    if (ws.ptr && ws.bytes >= bytes) {
        out->ws = ws.ptr;
        out->slots = ws.owned ? static_cast<unsigned char *>(ws.ptr) + ws.bytes : nullptr;
        return GPTQ_OK;
    }
    if (ws.ptr && !ws.owned)
        return GPTQ_WORKSPACE_TOO_SMALL;
    hipStreamCaptureStatus capturing = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(stream, &capturing) != hipSuccess) {
        (void)hipGetLastError();
        return GPTQ_HIP_ERROR;
    }
    if (capturing != hipStreamCaptureStatusNone)
        return GPTQ_WORKSPACE_TOO_SMALL;
    size_t want = bytes + bytes / 2;
    if (want < (size_t)(8u << 20))
        want = (size_t)(8u << 20);
    want = (want + 255) & ~(size_t)255;
    void *p = nullptr;
    if (hipMalloc(&p, want + kSlotBytes) != hipSuccess)
        return GPTQ_HIP_ERROR;
    // the arrival counters at the front and the slots at the end must start at zero; clear everything once
    if (!clear_now(p, want + kSlotBytes)) {
        (void)hipFree(p);
        return GPTQ_HIP_ERROR;
    }
    if (ws.ptr)
        g_retired[dev].push_back(ws.ptr);
    ws.ptr = p;
    ws.bytes = want;
    ws.owned = true;
    out->ws = p;
    out->slots = static_cast<unsigned char *>(p) + want;
    return GPTQ_OK;
}

// Default kernel by batch size, from measurement on Llama-shaped layers.  A single row is streamed fastest
// by the vector kernel.  From two rows on the small-batch MFMA kernel wins: its time is nearly flat up to 16
// rows and grows slowly to 32, where the vector kernel pays for every weight once per batch row.  The mid-batch
// streaming kernel's id stands for 33 to 64 rows, 17-32 rows on wide or very deep layers, and 65-128 rows where its
// 64-column tiles give between half and all of the compute units one workgroup each, or K is deep; where the
// small-batch or the big-tile kernel has overtaken it since, that one runs under the id (ring_in_place_of_mid,
// big_in_place_of_mid).
constexpr int kVectorMaxM = 1;
constexpr int kSmallBatchAutoMaxM = 32;
// Formats that the small-batch kernel does not take (groups of 96, ...): the vector kernel up to eight rows, then the
// pipelined big-tile kernel with K slices (4128x4096, groups of 96: M = 8 15.9 us against 16.1, M = 9 29.7 against 16.0;
// 2784x6888: M = 4 9.1 against 14.8, M = 16 32.3 against 14.6).
// Up to 16 rows deep narrow layers stay with the vector kernel, too: the big-tile kernel has few tiles there and many slices
// (groups of 96, M = 9 and 16: 8064x512 15.9 us against 18.8, 16.1, 18.6; 16128x256 16.4, 22.5; 8064x1024 16.9, 19.1; but
// 8064x1536 20.0, 19.8 and 12096x768 21.6, 20.1, 25.7, 20.1; 4032x512 15.2, 13.9).
constexpr int kVectorFallbackMaxM = 8;

bool vector_fallback(const Problem &p)
{
    if (p.M <= kVectorFallbackMaxM)
        return true;
    return p.M <= kDecodeMaxM && (!prefill_pipelined(p) || (p.K >= 6144 && (long long)p.K * p.N < (1ll << 23)));
}

// Small groups with a K that ends inside a 128-k unit, up to four rows: whether the vector kernel is the better one.  At
// two rows it is on half of the shapes (3776x34176 18.4 us against 22.9).  At three and four the small-batch kernel is
// ahead (2-90 %) where its 64-column workgroups fill whole rounds of the chip, and behind where a deep K meets a last
// round that is half empty, because the vector kernel has wider tiles to choose from.  Sweep of 17 widths and 6 depths,
// groups of 32 and 64, vector against small-batch at three rows:
//   a round less than four fifths full, K from 6144, 50 M weights:  12320x18432 29.5 us, 46.4; 8224x9216 14.5, 17.8
//     (groups of 64 13.8, 15.9); in smaller matrices the small-batch kernel stays ahead (8224x2056 10.3, 8.4), and below
//     that depth, too (4128x12288 11.8, 10.7);
//   beyond 16384 columns a round less than 70 % full, K from 2048 (groups of 64: 3072):  4128x20480 15.0, 19.5; 2080x18432
//     10.4, 11.4 (1120x18432 8.7, 8.0); groups of 64 3136x18432 10.7, 12.2 (2112x18432 10.1, 9.6);
//   groups of 32, K from 8192, N from 14336: level at best (28704x28672 89.6, 107.6; 16416x16384 33.9, 33.9).
// Layers so small that the launch dominates (1344x1536 4.9, 5.4) and very wide ones (8256x38256 41, 51; 2112x57344 17, 22;
// but 4160x45056 36, 29) stay with the vector kernel as well.
bool tail_prefers_vector(const Problem &p)
{
    if (p.M <= 2)
        return true;
    if (p.M > 4)
        return false;
    if ((long long)p.K * p.N < (1ll << 22) || p.N > 32768)
        return true;
    SkinnyPlan plan = {};
    skinny_make_plan(p, plan);
    const int workgroups = (p.N + 63) / 64 * plan.split_k;
    const double full = workgroups / (256.0 * ((workgroups + 255) / 256));
    if (full < 0.8 && p.K >= 6144 && (long long)p.K * p.N >= (3ll << 24))
        return true;
    if (full < 0.7 && p.N > 16384 && p.K >= (p.group_size == 32 ? 2048 : 3072))
        return true;
    return p.group_size == 32 && p.K >= 8192 && p.N >= 14336;
}

bool small_batch_by_default(const Problem &p)
{
    if (!skinny_supported(p))
        return false;
    if (p.K % 128 != 0 && tail_prefers_vector(p))
        return false;
    return p.M <= kSmallBatchAutoMaxM;
}

bool mid_batch_by_default(const Problem &p)
{
    if (!mid_supported(p) || p.M <= 16)
        return false;
    const long long tiles64 = (p.N + 63) / 64;
    if (p.M <= 32)
        return tiles64 >= 160 || (long long)p.K * p.N >= (1ll << 27);
    if (p.M <= 64)
        return true;
    // Up to 96 rows of a deep and wide layer: K slices of the big-tile kernel's 96x256 tile, which pads the batch less
    // and has two wavefronts per SIMD.  Mid-batch against big-tile at 65, 80 and 96 rows over K 12288-28672 and N
    // 2048-16384: from 128 column tiles and K = 16384 on level at worst and up to 51 % ahead (16384x8192 48.6 us, 48.4;
    // 20480x12288 87.1, 64.9; 28672x8192 78.5, 66.4), from 96 tiles on at K = 20480 (20480x6144 49.4, 48.3; 28672x7168
    // 73.1, 64.4).  Narrower layers lose with it, their tiles being too few (28672x4096 43.3, 51.6; 16384x2048 19.9, 24.8;
    // 24576x5120 45.0, 53.5) - down to a few hundred columns, where the mid-batch kernel has to make more slices than its
    // exchange is worth (16384x512 25.1, 21.2; 96 rows of 20480x896 26.9, 24.1, but 65 rows 23.7, 24.1).
    if (p.M <= 96 && p.K >= 16384 &&
        (tiles64 >= 128 || (tiles64 >= 96 && p.K >= 20480) || tiles64 <= 8 || (tiles64 <= 14 && p.M > 80)))
        return false;
    return tiles64 <= 256 && (tiles64 >= 128 || p.K >= 8192);
}

// Whether a plan settles which of the kernels under the mid-batch kernel's id runs: by the id, or by a tile that one of them has
// at these rows.
bool names_kernel_of_mid(const Problem &p, const gptq_w4a16_plan_t *plan)
{
    if (!plan || plan->kernel == 4)
        return plan != nullptr;
    const int t = plan->tile;
    return t == 64 || (t == 128 && p.M <= 64) || (ring_supported(p) && ring_width(p, t, plan->split_k)) ||
           (p.M > 48 && prefill_pipelined(p) && (t == 3 || t == 5 || t == 8));
}

// Whether the small-batch kernel on its ring of LDS slots, which has overtaken the mid-batch kernel on small batches, runs in
// its place, with widths and slices of its own where a plan leaves them open.
bool ring_in_place_of_mid(const Problem &p, const gptq_w4a16_plan_t *plan)
{
    if (!ring_supported(p))
        return false;
    // Up to 32 rows: 170 random layers at 17-32 rows 1-35 % faster, 2 % slower on one; 4096x22016 at M = 32 19.6 us -> 15.7,
    // 28672x8192 40.5 -> 34.1.
    if (p.M <= 32)
        return true;
    // 33-48 rows: 145 random layers 1.31 times as fast on average, 4-7 % slower on four (shallow ones and 11904x2104).
    // (A plan that names one of the kernels gets the ring with a width that automatic plans have there, else the mid-batch kernel.)
    if (names_kernel_of_mid(p, plan))
        return ring_width(p, plan->tile, plan->split_k);
    if (p.M <= kRingWideMaxM)
        return true;
    // 49-64 rows, in 32 columns: ahead on every layer of one round of workgroups up to this depth and on narrow ones of any
    // (100 random layers: 5-79 %, K 2048-4096 30 % and more; 5632x7552 at M = 64 17.6 us -> 16.7, 13312x1280 at M = 56
    // 16.1 -> 11.2), level or behind on deeper ones (6144x4576 14.4, 15.8; 8960x4864 17.2, 21.3) and with more tiles
    // (1792x8832 7.8, 9.0; 3456x10256 14.8, 19.9).
    return p.N <= 2048 || (p.N <= 8192 && p.K <= 5632);
}

// Whether the big-tile kernel, which has overtaken the mid-batch kernel beyond 64 rows on most layers since its workgroups may
// have 80, 96 and 112 rows, runs in its place: a plan under the mid-batch kernel's id with a tile of the other's.  Mid-batch
// against big-tile on 150 layers that mid_batch_by_default names: mid-batch ahead on shallow ones with a round of unsplit
// workgroups (80x2176x8320 10.7 us, 13.8; 96x4096x12288 19.2, 20.8; but 104x1792x14912 13.9, 13.0 and 65x4992x8832 20.5, 18.7)
// and, by 1 % on average, up to 80 rows on narrow ones in slices (72x25984x1984 23.1, 26.4; 80x28544x3520 35.8, 33.0); behind
// by 5-60 % elsewhere (77x8192x10240 30.1, 25.6; 100x28672x8192 72, 60; 112x11008x4096 26.2, 22.7; 128x8192x8192 32.4, 27.9).
// 49-64 rows, where the ring does not serve: as the estimates of both have it, that of the big-tile kernel 3 % ahead, or 8 % of
// 128-column tiles, whose estimate is high on one round of shallow ones (134 layers: 8 % faster on average, 64x8192x10240 26.8,
// 23.1; 60x1280x35968 23.2, 15.9; 56x25856x8320 69.8, 50.2).
// (`big`: its plan, with what `plan` leaves open filled in)
bool big_in_place_of_mid(const Problem &p, const MidPlan &mid, const gptq_w4a16_plan_t *plan, PrefillPlan &big)
{
    if (p.M <= 48 || !prefill_pipelined(p))
        return false;
    big.tile = 0;
    big.split_k = plan ? plan->split_k : 0;
    if (names_kernel_of_mid(p, plan)) {
        big.tile = plan->tile;
        if (plan->tile != 3 && plan->tile != 5 && plan->tile != 8)
            return false;
    } else if (p.M > 64) {
        const int tiles64 = (p.N + 63) / 64;
        if ((tiles64 > 128 && p.K <= 4736 && p.M <= 96) || (tiles64 <= 64 && tiles64 > 16 && p.M <= 80))
            return false;
    } else {
        prefill_make_plan(p, big);
        return prefill_estimate_us(p, big) < (mid.cols_per_wg == 64 ? 0.97 : 0.92) * mid_estimate_us(p, mid);
    }
    prefill_make_plan(p, big);
    return true;
}

// Act-order as stored: whether the lookup variant (64x64 tiles, each with its own table) is the better one against the
// kernels without it.  It is everywhere but where a shallow K leaves many tiles little to do, against the big-tile kernel's
// general path: 256x256x4096 9 us against 20, 512x256x4096 15, 20, but 1024x256x4096 26, 21 and 2048x256x40960 458, 272;
// 512x544x4096 18, 39, but 2048x544x40960 614, 568.  From K = 768 on it is ahead at every size (2048x768x16384 278, 318).
bool act_by_default(const Problem &p)
{
    if (!act_supported(p))
        return false;
    const long long tiles = (long long)((p.N + 63) / 64) * ((p.M + 63) / 64);
    return !(p.M > 64 && p.K < 384 && tiles > 640) && !(p.M > 256 && p.K < 640 && tiles > 2048);
}

// What a call resolves to: the kernel and its decomposition, after the automatic choices.
struct Resolved {
    int kernel;  // 1 vector, 2 big-tile MFMA, 3 small-batch MFMA, 4 mid-batch streaming MFMA
    bool act;    // the act-order lookup variant of the small-batch kernel (plan in `skinny`) runs in its place
    bool ring;   // the small-batch kernel (plan in `skinny`) runs in the mid-batch kernel's place
    bool big;    // the big-tile kernel (plan in `prefill`) does
    DecodePlan decode;
    SkinnyPlan skinny;
    MidPlan mid;
    PrefillPlan prefill;
    size_t least;  // bytes of scratch that are asked for even if the launch needs less
};

Resolved resolve(const Problem &p, const gptq_w4a16_plan_t *plan)
{
    Resolved r = {};
    int kernel = plan ? plan->kernel : 0;
    const bool lookup = plan && (plan->flags & GPTQ_ACT_LOOKUP) != 0;  // (check_flags: the problem has the variant)
    if (lookup || (kernel == 0 && act_by_default(p))) {
        // act-order as stored: the lookup variant for every batch of two rows and more.  Reported under the ids of
        // the kernels that serve an explicit request there (the vector kernel up to 16 rows, the big-tile kernel's
        // general path above), with a flag that tells it from them.
        r.kernel = lookup ? kernel : (p.M <= kDecodeMaxM) ? 1 : 2;
        r.act = true;
        r.skinny.split_k = plan ? plan->split_k : 0;
        act_make_plan(p, r.skinny);
        return r;
    }
    if (kernel == 0) {
        if (p.M <= kVectorMaxM)
            kernel = 1;
        else if (mid_batch_by_default(p))
            kernel = 4;
        else if (small_batch_by_default(p))
            kernel = 3;
        else
            kernel = vector_fallback(p) ? 1 : 2;
    }
    if (kernel == 3 && !skinny_supported(p))
        kernel = (p.M <= kDecodeMaxM) ? 1 : 2;
    if (kernel == 4 && !mid_supported(p))
        kernel = (p.M <= kDecodeMaxM) ? 1 : 2;
    if (kernel == 2 && !prefill_supported(p))
        kernel = 1;
    r.kernel = kernel;
    if (kernel == 1) {
        r.decode.cols_per_wg = plan ? plan->tile : 0;
        r.decode.split_k = plan ? plan->split_k : 0;
        r.decode.flags = plan ? plan->flags : 0;
        decode_make_plan(p, r.decode);
        if (!decode_plan_fits(p, r.decode)) {
            // the big-tile kernel's general path takes any format at any M
            r.kernel = kernel = 2;
            r.prefill.tile = 0;
            r.prefill.split_k = 0;
            prefill_make_plan(p, r.prefill);
        }
    } else if (kernel == 3) {
        r.skinny.cols_per_wg = plan ? plan->tile : 0;
        r.skinny.split_k = plan ? plan->split_k : 0;
        skinny_make_plan(p, r.skinny);
    } else if (kernel == 4) {
        r.mid.cols_per_wg = plan ? plan->tile : 0;
        r.mid.split_k = plan ? plan->split_k : 0;
        mid_make_plan(p, r.mid);
        if (ring_in_place_of_mid(p, plan)) {
            r.ring = true;
            if (plan) {
                const bool named = plan->kernel == 4;
                r.skinny.cols_per_wg = ring_width(p, plan->tile, r.mid.split_k) ? plan->tile : named ? r.mid.cols_per_wg : 0;
                // (slices of the mid-batch kernel's own choice are made for its own widths)
                r.skinny.split_k = plan->split_k > 0 || (named && r.skinny.cols_per_wg == r.mid.cols_per_wg) ? r.mid.split_k : 0;
            }
            if (p.M > kRingWideMaxM)
                r.skinny.cols_per_wg = 32;
            skinny_make_plan(p, r.skinny);
        } else {
            r.big = big_in_place_of_mid(p, r.mid, plan, r.prefill);
        }
    } else {
        r.prefill.tile = plan ? plan->tile : 0;
        r.prefill.split_k = plan ? plan->split_k : 0;
        prefill_make_plan(p, r.prefill);
    }
    return r;
}

size_t scratch_bytes(const Problem &p, const Resolved &r)
{
    size_t bytes;
    if (r.act)
        bytes = act_workspace_bytes(p, r.skinny);
    else if (r.kernel == 1)
        bytes = decode_workspace_bytes(p, r.decode);
    else if (r.kernel == 3 || r.ring)
        bytes = skinny_workspace_bytes(p, r.skinny);
    else if (r.kernel == 4 && !r.big)
        bytes = mid_workspace_bytes(p, r.mid);
    else
        bytes = prefill_workspace_bytes(p, r.prefill);  // 0 unless K is split
    return bytes > r.least ? bytes : r.least;
}

int launch_resolved(const Problem &p, const Resolved &r, const Scratch &scratch, hipStream_t stream)
{
    hipError_t err;
    void *const ws = scratch.ws;
    if (r.act)
        err = launch_act(p, r.skinny, ws, stream);
    else if (r.kernel == 1)
        err = launch_decode(p, r.decode, ws, stream);
    else if (r.kernel == 3 || r.ring)
        err = launch_skinny(p, r.skinny, ws, scratch.slots, stream);
    else if (r.kernel == 4 && !r.big)
        err = launch_mid(p, r.mid, ws, stream);
    else
        err = launch_prefill(p, r.prefill, ws, stream);
    return err == hipSuccess ? GPTQ_OK : GPTQ_HIP_ERROR;
}

// Scratch that a call may rely on the caller for, whatever its plan would like: what the vector kernel takes for up to 16
// rows, nothing above and nothing for the big-tile kernel.
size_t required_scratch(const Problem &p, const gptq_w4a16_plan_t *request)
{
    if (p.M > kDecodeMaxM || (request && request->kernel == 2))
        return 0;
    gptq_w4a16_plan_t vector = {};
    vector.kernel = 1;
    return scratch_bytes(p, resolve(p, &vector));
}

// Act-order problems, the big-tile kernel and the small-batch kernel (all widths but 256 where it runs on its ring, and up to 32 rows else) do not fail where the
// scratch of their K slices cannot be had - a workspace of the caller's that is too small, growth under capture, the
// static block: every workgroup then walks the slices itself, in the same order, so that the result does not depend on
// the scratch.  (How many slices pay is a matter of measurement and may change; which calls a workspace serves may
// not.)  A number of slices that the caller asked for is never given up.  False: the call needs what it needs.
bool fall_back(const Problem &p, const gptq_w4a16_plan_t *request, Resolved &r)
{
    if (r.skinny.serial || r.prefill.serial || (request && request->split_k > 0))
        return false;
    if (r.act || ((r.kernel == 3 || r.ring) && skinny_scratch_optional(p, r.skinny)))
        r.skinny.serial = true;
    else if ((r.kernel == 2 || r.big) && r.prefill.split_k > 1)
        r.prefill.serial = true;
    else
        return false;
    r.least = required_scratch(p, request);
    return true;
}

int run_gemm(const Problem &p, hipStream_t stream, const gptq_w4a16_plan_t *plan)
{
    Resolved r = resolve(p, plan);
    Scratch scratch;
    for (;;) {
        const size_t bytes = scratch_bytes(p, r);
        const int rc = bytes > 0 ? acquire_workspace(bytes, stream, &scratch) : GPTQ_OK;
        if (rc == GPTQ_OK)
            return launch_resolved(p, r, scratch, stream);
        if (rc != GPTQ_WORKSPACE_TOO_SMALL || !fall_back(p, plan, r))
            return rc;
    }
}

size_t align256(size_t v)
{
    return (v + 255) & ~(size_t)255;
}

int check_plan(const gptq_w4a16_plan_t *plan)
{
    if (!plan)
        return GPTQ_OK;
    if (plan->kernel < 0 || plan->kernel > 4 || plan->split_k < 0 || plan->tile < 0)
        return GPTQ_INVALID_ARG;
    for (int i = 0; i < 4; ++i)
        if (plan->reserved[i] != 0)
            return GPTQ_INVALID_ARG;
    if (plan->flags == GPTQ_ACT_LOOKUP)
        return (plan->kernel == 1 || plan->kernel == 2) && (plan->tile == 0 || plan->tile == 64) ? GPTQ_OK
                                                                                                  : GPTQ_INVALID_ARG;
    // the ablation switches belong to the vector kernel
    if (plan->flags < 0 || plan->flags > 15 || (plan->flags != 0 && plan->kernel != 1))
        return GPTQ_INVALID_ARG;
    if (plan->kernel == 2 && plan->tile != 0 && !prefill_tile_exists(plan->tile))
        return GPTQ_INVALID_ARG;
    return GPTQ_OK;
}

// Whether the problem has the variants that a plan's flags ask for.
int check_flags(const Problem &p, const gptq_w4a16_plan_t *plan)
{
    if (!plan)
        return GPTQ_OK;
    if (plan->flags == GPTQ_ACT_LOOKUP)
        return !p.g_idx ? GPTQ_INVALID_ARG : act_supported(p) ? GPTQ_OK : GPTQ_UNSUPPORTED_SHAPE;
    return (plan->flags & 7) != 0 && !decode_ablation_supported(p) ? GPTQ_UNSUPPORTED_SHAPE : GPTQ_OK;
}

// Validates the arguments of a GEMM call and fills `p`.
int make_problem(const void *x, const void *qweight, const void *qzeros, const void *scales, const void *g_idx,
                 void *out, int M, int K, int N, int group_size, const gptq_w4a16_plan_t *plan, Problem &p)
{
    if (!x || !qweight || !qzeros || !scales || !out || M <= 0)
        return GPTQ_INVALID_ARG;
    const int rc = check_shape(K, N, group_size);
    if (rc != GPTQ_OK)
        return rc;
    if (check_plan(plan) != GPTQ_OK)
        return GPTQ_INVALID_ARG;
    if (!aligned16(x) || !aligned16(qweight) || !aligned16(qzeros) || !aligned16(scales) || !aligned16(out) ||
        (g_idx && !aligned16(g_idx)))
        return GPTQ_MISALIGNED;
    p.x = static_cast<const half_t *>(x);
    p.qweight = static_cast<const uint32_t *>(qweight);
    p.qzeros = static_cast<const uint32_t *>(qzeros);
    p.scales = static_cast<const half_t *>(scales);
    p.g_idx = static_cast<const int32_t *>(g_idx);
    p.out = static_cast<half_t *>(out);
    p.M = M;
    p.K = K;
    p.N = N;
    p.group_size = group_size;
    return check_flags(p, plan);
}

}  // namespace

extern "C" {

int gptq_w4a16_gemm_plan(const void *x, const void *qweight, const void *qzeros, const void *scales,
                         const void *g_idx, void *out, int M, int K, int N, int group_size,
                         gptq_stream_t stream, const gptq_w4a16_plan_t *plan)
{
    Problem p;
    const int rc = make_problem(x, qweight, qzeros, scales, g_idx, out, M, K, N, group_size, plan, p);
    if (rc != GPTQ_OK)
        return rc;
    return run_gemm(p, static_cast<hipStream_t>(stream), plan);
}

int gptq_w4a16_gemm_static(const void *x, const void *qweight, const void *qzeros, const void *scales,
                           const void *g_idx, void *out, int M, int K, int N, int group_size,
                           gptq_stream_t stream)
{
    Problem p;
    const int rc = make_problem(x, qweight, qzeros, scales, g_idx, out, M, K, N, group_size, nullptr, p);
    if (rc != GPTQ_OK)
        return rc;
    Resolved r = resolve(p, nullptr);
    while (scratch_bytes(p, r) > kStaticScratchBytes)
        if (!fall_back(p, nullptr, r))
            return GPTQ_STATIC_SCRATCH_EXCEEDED;
    hipStream_t st = static_cast<hipStream_t>(stream);
    Scratch scratch;
    const int wrc = static_scratch_ptr(&scratch);
    if (wrc != GPTQ_OK)
        return wrc;
    return launch_resolved(p, r, scratch, st);
}

int gptq_w4a16_gemm(const void *x, const void *qweight, const void *qzeros, const void *scales,
                    const void *g_idx, void *out, int M, int K, int N, int group_size, gptq_stream_t stream)
{
    return gptq_w4a16_gemm_plan(x, qweight, qzeros, scales, g_idx, out, M, K, N, group_size, stream, nullptr);
}

int gptq_w4a16_plan_query(int M, int K, int N, int group_size, int act_order, const gptq_w4a16_plan_t *request,
                          gptq_w4a16_plan_t *resolved)
{
    if (!resolved || M <= 0)
        return GPTQ_INVALID_ARG;
    const int rc = check_shape(K, N, group_size);
    if (rc != GPTQ_OK)
        return rc;
    if (check_plan(request) != GPTQ_OK)
        return GPTQ_INVALID_ARG;
    static const int32_t some_g_idx = 0;  // only its presence matters to the plan
    Problem p = {};
    p.g_idx = act_order ? &some_g_idx : nullptr;
    p.M = M;
    p.K = K;
    p.N = N;
    p.group_size = group_size;
    const int frc = check_flags(p, request);
    if (frc != GPTQ_OK)
        return frc;
    const Resolved r = resolve(p, request);
    gptq_w4a16_plan_t out = {};
    out.kernel = r.kernel;
    if (r.act) {
        out.split_k = r.skinny.split_k;
        out.tile = r.skinny.cols_per_wg;
        out.flags = GPTQ_ACT_LOOKUP;
    } else if (r.kernel == 1) {
        out.split_k = r.decode.split_k;
        out.tile = r.decode.cols_per_wg;
        out.flags = r.decode.flags;
    } else if (r.kernel == 3 || r.ring) {
        out.split_k = r.skinny.split_k;
        out.tile = r.skinny.cols_per_wg;
    } else if (r.kernel == 4 && !r.big) {
        out.split_k = r.mid.split_k;
        out.tile = r.mid.cols_per_wg;
    } else {
        out.split_k = r.prefill.split_k;
        out.tile = r.prefill.tile;
    }
    *resolved = out;
    return GPTQ_OK;
}

int gptq_w4a16_act_order_prepare(const void *qweight, const void *g_idx, void *qweight_sorted, void *perm, int K,
                                 int N, int group_size, gptq_stream_t stream)
{
    if (!qweight || !g_idx || !qweight_sorted || !perm)
        return GPTQ_INVALID_ARG;
    const int rc = check_shape(K, N, group_size);
    if (rc != GPTQ_OK)
        return rc;
    if (!aligned16(qweight) || !aligned16(g_idx) || !aligned16(qweight_sorted) || !aligned16(perm))
        return GPTQ_MISALIGNED;
    if (qweight == qweight_sorted)
        return GPTQ_INVALID_ARG;  // the gather is not in place
    hipStream_t st = static_cast<hipStream_t>(stream);
    int *status = nullptr;
    if (hipMalloc(reinterpret_cast<void **>(&status), sizeof(int)) != hipSuccess)
        return GPTQ_HIP_ERROR;
    int host_status = 0;
    bool ok = hipMemsetAsync(status, 0, sizeof(int), st) == hipSuccess;
    ok = ok && launch_rank_rows(static_cast<const int32_t *>(g_idx), static_cast<int32_t *>(perm), K, group_size,
                                status, st) == hipSuccess;
    ok = ok && hipMemcpyAsync(&host_status, status, sizeof(int), hipMemcpyDeviceToHost, st) == hipSuccess;
    ok = ok && hipStreamSynchronize(st) == hipSuccess;
    (void)hipFree(status);
    if (!ok)
        return GPTQ_HIP_ERROR;
    if (host_status & 1)
        return GPTQ_INVALID_ARG;  // g_idx entry outside [0, K / group_size)
    if (host_status & 2)
        return GPTQ_UNSUPPORTED_SHAPE;  // a group owns more (so another fewer) than group_size rows
    if (launch_sort_rows(static_cast<const uint32_t *>(qweight), static_cast<const int32_t *>(perm),
                         static_cast<uint32_t *>(qweight_sorted), K, N, st) != hipSuccess)
        return GPTQ_HIP_ERROR;
    return hipStreamSynchronize(st) == hipSuccess ? GPTQ_OK : GPTQ_HIP_ERROR;
}

int gptq_w4a16_gemm_prepared(const void *x, const void *qweight_sorted, const void *qzeros, const void *scales,
                             const void *perm, void *out, int M, int K, int N, int group_size,
                             gptq_stream_t stream)
{
    if (!x || !qweight_sorted || !qzeros || !scales || !perm || !out || M <= 0)
        return GPTQ_INVALID_ARG;
    const int rc = check_shape(K, N, group_size);
    if (rc != GPTQ_OK)
        return rc;
    if (!aligned16(x) || !aligned16(qweight_sorted) || !aligned16(qzeros) || !aligned16(scales) || !aligned16(out) ||
        !aligned16(perm))
        return GPTQ_MISALIGNED;
    Problem p;
    p.x = nullptr;  // the gathered copy, below
    p.qweight = static_cast<const uint32_t *>(qweight_sorted);
    p.qzeros = static_cast<const uint32_t *>(qzeros);
    p.scales = static_cast<const half_t *>(scales);
    p.g_idx = nullptr;
    p.out = static_cast<half_t *>(out);
    p.M = M;
    p.K = K;
    p.N = N;
    p.group_size = group_size;
    Resolved r = resolve(p, nullptr);
    hipStream_t st = static_cast<hipStream_t>(stream);
    if (r.kernel == 1 && M == 1 && r.decode.chunk_rows == 4 && r.decode.flags == 0) {
        // the vector kernel gathers the activations itself while it stages them: one launch
        p.x = static_cast<const half_t *>(x);
        p.x_perm = static_cast<const int32_t *>(perm);
        Scratch scratch;
        const size_t bytes = scratch_bytes(p, r);
        if (bytes > 0) {
            const int wrc = acquire_workspace(bytes, st, &scratch);
            if (wrc != GPTQ_OK)
                return wrc;
        }
        return launch_resolved(p, r, scratch, st);
    }
    // scratch: what the kernel needs, then the gathered activations
    // (the counter area at the front stays reserved even if this launch needs none: it must remain zero)
    size_t kernel_bytes;
    Scratch scratch;
    for (;;) {
        kernel_bytes = align256(scratch_bytes(p, r));
        if (kernel_bytes < decode_counter_bytes(N))
            kernel_bytes = decode_counter_bytes(N);
        const int wrc = acquire_workspace(kernel_bytes + (size_t)M * K * sizeof(half_t), st, &scratch);
        if (wrc == GPTQ_OK)
            break;
        if (wrc != GPTQ_WORKSPACE_TOO_SMALL || !fall_back(p, nullptr, r))
            return wrc;
    }
    half_t *xp = reinterpret_cast<half_t *>(static_cast<unsigned char *>(scratch.ws) + kernel_bytes);
    if (launch_gather_activations(static_cast<const half_t *>(x), static_cast<const int32_t *>(perm), xp, M, K, st) !=
        hipSuccess)
        return GPTQ_HIP_ERROR;
    p.x = xp;
    return launch_resolved(p, r, scratch, st);
}

int gptq_w4a16_shift_zeros(const void *qzeros_in, void *qzeros_out, int delta, int K, int N, int group_size,
                           gptq_stream_t stream)
{
    if (!qzeros_in || !qzeros_out)
        return GPTQ_INVALID_ARG;
    const int rc = check_shape(K, N, group_size);
    if (rc != GPTQ_OK)
        return rc;
    if (!aligned16(qzeros_in) || !aligned16(qzeros_out))
        return GPTQ_MISALIGNED;
    const long long words = (long long)(K / group_size) * (N / 8);
    const hipError_t err = launch_shift_zeros(static_cast<const uint32_t *>(qzeros_in),
                                              static_cast<uint32_t *>(qzeros_out), words, ((delta % 16) + 16) % 16,
                                              static_cast<hipStream_t>(stream));
    return err == hipSuccess ? GPTQ_OK : GPTQ_HIP_ERROR;
}

int gptq_w4a16_dequant(const void *qweight, const void *qzeros, const void *scales, const void *g_idx,
                       void *w_out, int K, int N, int group_size, gptq_stream_t stream)
{
    if (!qweight || !qzeros || !scales || !w_out)
        return GPTQ_INVALID_ARG;
    const int rc = check_shape(K, N, group_size);
    if (rc != GPTQ_OK)
        return rc;
    if (!aligned16(qweight) || !aligned16(qzeros) || !aligned16(scales) || !aligned16(w_out) ||
        (g_idx && !aligned16(g_idx)))
        return GPTQ_MISALIGNED;
    const hipError_t err = launch_dequant(static_cast<const uint32_t *>(qweight), static_cast<const uint32_t *>(qzeros),
                                          static_cast<const half_t *>(scales), static_cast<const int32_t *>(g_idx),
                                          static_cast<half_t *>(w_out), K, N, group_size,
                                          static_cast<hipStream_t>(stream));
    return err == hipSuccess ? GPTQ_OK : GPTQ_HIP_ERROR;
}

int gptq_w4a16_unpack(const void *qweight, void *q_out, const void *qzeros, void *z_out, int K, int N,
                      int group_size, gptq_stream_t stream)
{
    if (!qweight || !q_out || (z_out && !qzeros))
        return GPTQ_INVALID_ARG;
    const int rc = check_shape(K, N, group_size);
    if (rc != GPTQ_OK)
        return rc;
    if (!aligned16(qweight) || !aligned16(q_out) || (z_out && (!aligned16(qzeros) || !aligned16(z_out))))
        return GPTQ_MISALIGNED;
    const hipError_t err =
        launch_unpack(static_cast<const uint32_t *>(qweight), static_cast<uint8_t *>(q_out),
                      static_cast<const uint32_t *>(qzeros), static_cast<uint8_t *>(z_out), K, N, group_size,
                      static_cast<hipStream_t>(stream));
    return err == hipSuccess ? GPTQ_OK : GPTQ_HIP_ERROR;
}

size_t gptq_w4a16_workspace_bytes(int M, int K, int N, int group_size)
{
    if (M <= 0 || check_shape(K, N, group_size) != GPTQ_OK)
        return 0;
    // The automatic plan never uses more slices than this bound; explicit plans are checked at launch.
    Problem p = {};
    p.M = M;
    p.K = K;
    p.N = N;
    p.group_size = group_size;
    DecodePlan dp = {};
    decode_make_plan(p, dp);
    size_t bytes = decode_workspace_bytes(p, dp);
    // act-order problems may be planned with a different slice count
    int dummy = 0;
    p.g_idx = &dummy;
    DecodePlan da = {};
    decode_make_plan(p, da);
    const size_t act = decode_workspace_bytes(p, da);
    if (act > bytes)
        bytes = act;
    p.g_idx = nullptr;
    if (skinny_supported(p)) {
        SkinnyPlan sp = {};
        skinny_make_plan(p, sp);
        const size_t sk = skinny_workspace_bytes(p, sp);
        if (sk > bytes)
            bytes = sk;
    }
    // the big-tile and mid-batch kernels split K on few-tile shapes; counted where the default dispatch picks them
    for (int act = 0; act < 2; ++act) {
        p.g_idx = act ? &dummy : nullptr;
        const Resolved r = resolve(p, nullptr);
        if (r.act || r.kernel == 2 || r.kernel == 4) {
            const size_t pf = scratch_bytes(p, r);
            if (pf > bytes)
                bytes = pf;
        }
    }
    return bytes;
}

int gptq_w4a16_set_workspace(void *dev_ptr, size_t bytes)
{
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices)
        return GPTQ_HIP_ERROR;
    if (dev_ptr && (reinterpret_cast<uintptr_t>(dev_ptr) & 255u) != 0)
        return GPTQ_MISALIGNED;
    if (dev_ptr && bytes < decode_counter_bytes(0))
        return GPTQ_WORKSPACE_TOO_SMALL;  // not even room for the arrival counters
    std::lock_guard<std::mutex> lock(g_mutex);
    Workspace &ws = g_ws[dev];
    // the library's own blocks, current and retired, go now: drain the device first
    if ((ws.ptr && ws.owned) || !g_retired[dev].empty()) {
        if (hipDeviceSynchronize() != hipSuccess)
            return GPTQ_HIP_ERROR;
        if (ws.ptr && ws.owned)
            (void)hipFree(ws.ptr);
        for (void *old : g_retired[dev])
            (void)hipFree(old);
        g_retired[dev].clear();
    }
    ws = Workspace();
    if (dev_ptr) {
        if (hipDeviceSynchronize() != hipSuccess)
            return GPTQ_HIP_ERROR;
        if (!clear_now(dev_ptr, bytes))
            return GPTQ_HIP_ERROR;
        ws.ptr = dev_ptr;
        ws.bytes = bytes;
        ws.owned = false;
    }
    return GPTQ_OK;
}

const char *gptq_w4a16_strerror(int code)
{
    switch (code) {
    case GPTQ_OK: return "ok";
    case GPTQ_INVALID_ARG: return "invalid argument (null pointer, non-positive size or bad plan)";
    case GPTQ_UNSUPPORTED_SHAPE: return "unsupported shape (K, N, group_size must be multiples of 8; group_size must divide K)";
    case GPTQ_MISALIGNED: return "a base pointer is not 16-byte aligned";
    case GPTQ_HIP_ERROR: return "a HIP call or kernel launch failed";
    case GPTQ_WORKSPACE_TOO_SMALL: return "caller-set workspace is too small for this problem";
    case GPTQ_STATIC_SCRATCH_EXCEEDED:
        return "problem needs more split-K scratch than the 48 MiB static block of gptq_w4a16_gemm_static";
    default: return "unknown status code";
    }
}

int gptq_w4a16_version(void)
{
    return kVersion;
}

}  // extern "C"
