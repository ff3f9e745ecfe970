// C-ABI entry points of libfscnn.so (declared and documented in include/fscnn.h):
// argument validation, handle management, plan caching, kernel dispatch.  No arithmetic of
// the method happens on the host.
#include <limits.h>
#include <string.h>

#include <algorithm>
#include <atomic>
#include <new>

#include "host_word.h"
#include "internal.h"

using namespace fscnn;

namespace {

#define FSCNN_HIP(expr)                            \
    do {                                           \
        hipError_t e_ = (expr);                    \
        if (e_ != hipSuccess) {                    \
            (void)hipGetLastError();               \
            return e_ == hipErrorOutOfMemory ? FSCNN_ERR_ALLOC : FSCNN_ERR_DEVICE; \
        }                                          \
    } while (0)

fscnn_status_t out_shape(int H, int W, int R, int S, int sh, int sw, int ph, int pw, int *Ho, int *Wo)
{
    if (H <= 0 || W <= 0 || R <= 0 || S <= 0 || sh <= 0 || sw <= 0 || ph < 0 || pw < 0)
        return FSCNN_ERR_SHAPE;
    const long long spanh = (long long)H + 2LL * ph - R;
    const long long spanw = (long long)W + 2LL * pw - S;
    if (spanh < 0 || spanw < 0) return FSCNN_ERR_SHAPE;
    const long long ho = spanh / sh + 1, wo = spanw / sw + 1;
    if (ho > INT_MAX || wo > INT_MAX) return FSCNN_ERR_SHAPE;
    *Ho = (int)ho;
    *Wo = (int)wo;
    return FSCNN_OK;
}

bool fits_int(long long v) { return v > 0 && v < (1LL << 31); }

fscnn_status_t have_device(int *dev)
{
    int n = 0;
    if (hipGetDeviceCount(&n) != hipSuccess || n <= 0) {
        (void)hipGetLastError();
        return FSCNN_ERR_DEVICE;
    }
    if (hipGetDevice(dev) != hipSuccess) {
        (void)hipGetLastError();
        return FSCNN_ERR_DEVICE;
    }
    return FSCNN_OK;
}

bool live(const fscnn_filter_t *f) { return f && f->magic == kFilterMagic; }
bool live(const fscnn_input_t *i) { return i && i->magic == kInputMagic; }
bool live(const fscnn_dense_t *d) { return d && d->magic == kDenseMagic; }

// Share of a bank's entries that are stored (1 exactly for a bank without zeros).
double density(const fscnn_filter_t *f) { return (double)f->nnz / ((double)f->K * f->C * f->R * f->S); }

// Large device blocks that destroyed handles leave behind, for the next handles: releasing an allocation of some MB takes the
// runtime 20 to 290 us (it waits for the device as well) and making one 10 to 40; smaller ones than kPoolLeast take 1 us and are not
// kept.  A program that compresses its banks for one pass makes a dozen scratch buffers of the channel split (13-layer stack,
// N = 1, a load and a pass: at 224x224 2.99 ms with all of them released, 1.42 with 64 MB kept, 1.25 now); one that compresses an
// activation per pass makes one of 40 MB (512 channels at 28x28, N = 8, with the convolution: 235 us released, 186 kept).  What
// is held is bounded per pool; a full pool drops what nobody took while kPoolAge blocks came in, or refuses; all of it is given
// back when an allocation of the library fails, and by fscnn_pool_trim.
//
// A handle whose calls all ran on the default stream gives its blocks back in that stream's order, without a wait, and only calls
// on the default stream of the same device take them (that stream lives as long as the process and is never captured, so a later
// taker's work is behind the earlier one's).  The streams that have used any other handle may be gone, and nothing orders a new one
// behind them: its destruction waits for the device, as hipFree does, and its blocks are idle then and serve any stream
// (compress + convolve on a stream of the caller's, 512 channels at 28x28, N = 16: 718 us released, 324 kept).
constexpr size_t kPoolLeast = 2u << 20, kPoolBuffers = 64, kPoolAge = 256;
struct DevicePool {
    struct Entry {
        int device;
        void *buf;
        size_t bytes;
        bool idle;
        size_t since;                    // `given` when it came
    };
    const size_t max_bytes;
    std::mutex mu;
    std::vector<Entry> free;             // in the order they came
    size_t held = 0, given = 0;

    explicit DevicePool(size_t bytes) : max_bytes(bytes) {}
    // the smallest that is large enough, up to four times what is needed
    bool take(int device, hipStream_t st, size_t bytes, void **buf, size_t *got)
    {
        std::lock_guard<std::mutex> lock(mu);
        size_t best = free.size();
        for (size_t i = 0; i < free.size(); ++i)
            if (free[i].device == device && (free[i].idle || !st) && free[i].bytes >= bytes && free[i].bytes / 4 <= bytes &&
                (best == free.size() || free[i].bytes < free[best].bytes))
                best = i;
        if (best == free.size()) return false;
        *buf = free[best].buf;
        *got = free[best].bytes;
        held -= free[best].bytes;
        free.erase(free.begin() + best);
        return true;
    }
    bool give(int device, void *buf, size_t bytes, bool idle)
    {
        if (bytes < kPoolLeast || bytes > max_bytes) return false;
        std::lock_guard<std::mutex> lock(mu);
        ++given;
        auto full = [&] { return free.size() >= kPoolBuffers || held + bytes > max_bytes; };
        while (full() && !free.empty() && given - free.front().since > kPoolAge) {
            held -= free.front().bytes;
            (void)hipFree(free.front().buf);
            free.erase(free.begin());
        }
        if (full()) return false;
        free.push_back({device, buf, bytes, idle, given});
        held += bytes;
        return true;
    }
    void trim()
    {
        std::lock_guard<std::mutex> lock(mu);
        for (auto &q : free) (void)hipFree(q.buf);
        free.clear();
        held = 0;
    }
};
// (never destroyed: handles may outlive static objects)
// banks, plans, and scratch of the channel split; blocks of 8 MB and more have a pool of their own, so that a few of them do not
// keep the many smaller ones out (the 13-layer stack at N = 1 leaves 50 MB of the former and 47 of the latter)
DevicePool &filter_pool(size_t bytes)
{
    static DevicePool *small = new DevicePool(64u << 20), *large = new DevicePool(64u << 20);
    return bytes < (8u << 20) ? *small : *large;
}
DevicePool &input_pool()    // compressed activations
{
    static DevicePool *pool = new DevicePool(512u << 20);
    return *pool;
}

// hipMalloc that gives the pools back before it fails
hipError_t device_alloc(void **p, size_t bytes)
{
    hipError_t e = hipMalloc(p, bytes);
    if (e != hipErrorOutOfMemory) return e;
    (void)hipGetLastError();
    filter_pool(0).trim();
    filter_pool(~(size_t)0).trim();
    input_pool().trim();
    return hipMalloc(p, bytes);
}

// a block for work on `st`; *got: its size
hipError_t block_alloc(DevicePool &pool, int device, hipStream_t st, void **p, size_t bytes, size_t *got)
{
    if (pool.take(device, st, bytes, p, got)) return hipSuccess;
    *got = bytes;
    return device_alloc(p, bytes);
}

// How a handle leaves its blocks: with uses queued on the default stream and on no other, idle, or neither is known.
enum class Left { kInOrder, kIdle, kUnknown };

// in_order: all uses are on the default stream; largest: of the blocks, in bytes (nothing is waited for where none will be kept)
Left blocks_left(int device, bool in_order, size_t largest)
{
    if (in_order) return Left::kInOrder;
    if (largest < kPoolLeast) return Left::kUnknown;
    // hipFree waits for the device.  (So does hipDeviceSynchronize, but that ends a capture in relaxed mode.)
    int dev = -1;
    void *p = nullptr;
    if (hipGetDevice(&dev) == hipSuccess && dev == device && hipMalloc(&p, 256) == hipSuccess && hipFree(p) == hipSuccess) return Left::kIdle;
    (void)hipGetLastError();
    return Left::kUnknown;
}

// (hipFree waits for the device)
void block_free(DevicePool &pool, int device, void *p, size_t bytes, Left left)
{
    if (p && (left == Left::kUnknown || !pool.give(device, p, bytes, left == Left::kIdle))) (void)hipFree(p);
}

// the same for filter handles
hipError_t filter_alloc(int device, hipStream_t st, void **p, size_t bytes, size_t *got)
{
    return block_alloc(filter_pool(bytes), device, st, p, bytes, got);
}

void filter_free(int device, void *p, size_t bytes, Left left) { block_free(filter_pool(bytes), device, p, bytes, left); }

bool capturing(hipStream_t st)
{
    hipStreamCaptureStatus c = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(st, &c) != hipSuccess) {
        (void)hipGetLastError();
        return false;
    }
    return c != hipStreamCaptureStatusNone;
}

// 0: st is not capturing; else the number of the capture, which no other has
unsigned long long capture_id(hipStream_t st)
{
    hipStreamCaptureStatus c = hipStreamCaptureStatusNone;
    unsigned long long id = 0;
    if (!capturing(st)) return 0;
    if (hipStreamGetCaptureInfo(st, &c, &id) == hipSuccess && id) return id;
    (void)hipGetLastError();
    return ~0ull;
}

// f(block, bytes) for every device block of a plan (the records' one holds the pointers as well)
template <class F> void for_blocks(const SfPlan *p, F f)
{
    f(p->recs, p->recs_bytes);
    f(p->packed, p->packed_bytes);
    f(p->parts, p->parts_bytes);
    for (auto *list : {&p->split, &p->outgrown})
        for (auto &sc : *list) f(sc.buf, sc.bytes);
}

// device: where the plan's buffers live
void free_plan(SfPlan *p, int device, Left left)
{
    if (!p) return;
    for_blocks(p, [&](void *buf, size_t bytes) { filter_free(device, buf, bytes, left); });
    delete p;
}

// Scratch of the channel-split mode for a call on `st`: the buffer this stream used before if it is
// large enough, else a new one (the first such call of a plan on a stream allocates).  One buffer per
// stream: calls that share a handle on different streams never share scratch.
fscnn_status_t split_scratch(fscnn_filter_t *f, SfPlan *p, hipStream_t st, size_t bytes, float **out)
{
    std::lock_guard<std::mutex> lock(f->mu);
    SfPlan::SplitScratch *sc = nullptr;
    for (auto &q : p->split)
        if (q.stream == st) sc = &q;
    if (sc && sc->bytes >= bytes) {
        *out = sc->buf;
        return FSCNN_OK;
    }
    float *nb = nullptr;
    hipError_t e = hipSuccess;
    if (capturing(st)) {
        // (a capture in relaxed mode; in the others the allocation is refused.)  The clear must run now: recorded, it
        // would leave the counters as they are for calls that come before the first replay
        hipStream_t own = nullptr;
        e = device_alloc(reinterpret_cast<void **>(&nb), bytes);
        if (e == hipSuccess) e = hipStreamCreateWithFlags(&own, hipStreamNonBlocking);
        if (e == hipSuccess) e = launch_split_clear(nb, own);
        if (e == hipSuccess) e = hipStreamSynchronize(own);
        if (own) (void)hipStreamDestroy(own);
    } else {
        e = filter_alloc(f->device, st, reinterpret_cast<void **>(&nb), bytes, &bytes);
        if (e == hipSuccess) e = launch_split_clear(nb, st);
    }
    if (e != hipSuccess) {
        (void)hipGetLastError();
        if (nb) (void)hipFree(nb);
        return FSCNN_ERR_ALLOC;
    }
    if (sc) {
        // launches in flight and graphs captured so far use the smaller one: it stays with the plan
        p->outgrown.push_back({sc->stream, sc->buf, sc->bytes});
        sc->buf = nb;
        sc->bytes = bytes;
    } else {
        p->split.push_back({st, nb, bytes});
    }
    *out = nb;
    return FSCNN_OK;
}

// Room for the sums of a divided contraction's parts, behind the counters; NULL where there is none and none can be made now (no
// room, or `st` is capturing): then one work-group per tile takes all channels.
float *split_sums(fscnn_filter_t *f, SfPlan *p, hipStream_t st, size_t bytes)
{
    bool have = false;
    if (capturing(st)) {
        std::lock_guard<std::mutex> lock(f->mu);
        for (auto &q : p->split) have |= q.stream == st && q.bytes >= bytes;
        if (!have) return nullptr;
    }
    float *buf;
    return split_scratch(f, p, st, bytes, &buf) == FSCNN_OK ? buf + 256 : nullptr;
}

// Returns the plan of `variant` (>= 1) for this handle, building it on `st` when absent.
// kDirectPlan stands for the direct kernel (no device data besides the canonical CSR), kContractPlan
// for the contraction on the matrix cores (the bank as a dense array).
fscnn_status_t get_plan(fscnn_filter_t *f, int variant, hipStream_t st, SfPlan **out)
{
    std::lock_guard<std::mutex> lock(f->mu);
    for (SfPlan *p : f->plans)
        if (p->variant == variant) {
            *out = p;
            return FSCNN_OK;
        }
    SfPlan *p = new (std::nothrow) SfPlan();
    if (!p) return FSCNN_ERR_ALLOC;
    p->variant = variant;
    if (variant == kDirectPlan) {
        p->direct = true;
        f->plans.push_back(p);
        *out = p;
        return FSCNN_OK;
    }
    if (variant == kContractPlan || variant == kSplitPlan) {
        int dev;
        fscnn_status_t ds = have_device(&dev);
        if (ds == FSCNN_OK && dev != f->device) ds = FSCNN_ERR_MISMATCH;
        if (ds != FSCNN_OK) {
            delete p;
            return ds;
        }
        hipError_t e;
        if (variant == kSplitPlan) {
            e = filter_alloc(dev, st, &p->parts, (size_t)split_packed_bytes(f->K, f->C, f->R * f->S), &p->parts_bytes);
            if (e == hipSuccess) e = launch_split_rows(f->rowptr, f->idx, f->val, f->K, f->C, f->R * f->S, p->parts, st);
        } else {
            e = filter_alloc(dev, st, reinterpret_cast<void **>(&p->packed),
                            sizeof(float) * (size_t)(contract_packed_elems(f->K, f->C, f->R * f->S) + 4), &p->packed_bytes);
            if (e == hipSuccess) e = launch_pack_rows(f->rowptr, f->idx, f->val, f->K, f->C, f->R * f->S, p->packed, st);
        }
        if (e == hipSuccess) e = hipStreamSynchronize(st);   // the plan may be used from other streams
        if (e != hipSuccess) {
            (void)hipGetLastError();
            free_plan(p, f->device, Left::kUnknown);
            return e == hipErrorOutOfMemory ? FSCNN_ERR_ALLOC : FSCNN_ERR_DEVICE;
        }
        f->plans.push_back(p);
        *out = p;
        return FSCNN_OK;
    }
    // the configuration (validated against the call's stride by resolve_variant) fixes the stride
    if (!sf_variant_geom(variant, f->R, f->S, 1, 1, &p->g) && !sf_variant_geom(variant, f->R, f->S, 2, 2, &p->g)) {
        delete p;
        return FSCNN_ERR_UNSUPPORTED;
    }
    const SfGeom &g = p->g;
    p->NCH = (f->C + g.CC - 1) / g.CC;
    p->NG = (f->K + g.KG - 1) / g.KG;
    const long long nb = (long long)p->NG * p->NCH * g.KG;
    // records: one per stored value; the taps-outer form lists every tap of every chunk instead
    const long long cap = g.DENSE ? (long long)p->NG * g.WAVES * p->NCH * g.CC * f->R * f->S * g.SLOTS : f->nnz;
    if (!fits_int(nb + 1) || cap + kPlanSpare >= (1LL << 31)) {
        delete p;
        return FSCNN_ERR_UNSUPPORTED;
    }
    // the plan is built next to the handle's arrays
    int dev;
    fscnn_status_t ds = have_device(&dev);
    if (ds == FSCNN_OK && dev != f->device) ds = FSCNN_ERR_MISMATCH;
    if (ds != FSCNN_OK) {
        delete p;
        return ds;
    }
    // one allocation: the records, the pointers, and scratch of the launch that writes them
    const size_t nrecs = (size_t)(cap + kPlanSpare);
    hipError_t e = filter_alloc(dev, st, reinterpret_cast<void **>(&p->recs),
                               sizeof(Rec) * nrecs + sizeof(int) * (size_t)(nb + 1 + plan_scratch_elems(g, p->NCH, p->NG)), &p->recs_bytes);
    HostWord word;
    if (e == hipSuccess) {
        p->segptr = reinterpret_cast<int *>(p->recs + nrecs);
        e = launch_plan(f->rowptr, f->idx, f->val, f->K, f->R, f->S, g, p->NCH, p->NG, p->segptr + (nb + 1), p->segptr,
                        g.DENSE ? nullptr : p->recs, g.DENSE ? -1 : word.slot(), g.DENSE ? nullptr : word.hand_out(), st);
    }
    if (e == hipSuccess && g.DENSE)
        e = launch_plan_fill_dense(f->rowptr, f->idx, f->val, f->K, f->C, f->R, f->S, g, p->NCH, p->NG, cap, p->recs, st);
    // The plan may be used from other streams: wait for the build.
    int built = 0;
    if (e == hipSuccess) e = g.DENSE ? hipStreamSynchronize(st) : word.wait(nullptr, st, &built);
    if (e != hipSuccess) {
        (void)hipGetLastError();
        free_plan(p, f->device, Left::kUnknown);
        return e == hipErrorOutOfMemory ? FSCNN_ERR_ALLOC : FSCNN_ERR_DEVICE;
    }
    p->nrec = cap;
    f->plans.push_back(p);
    *out = p;
    return FSCNN_OK;
}

// Which variant serves this geometry: `variant` > 0 is taken as is (checked), 0 = automatic,
// anything the tiled kernel cannot do goes to the direct kernel (-1).
fscnn_status_t resolve_variant(const fscnn_filter_t *f, int N, int H, int W, int sh, int sw,
                               int variant, int *resolved, bool n4 = false, bool pool = false,
                               bool emit = false)
{
    // the tiled kernel serves strides 1 and 2 (equal on both axes) and addresses up to four
    // images' channels with 32-bit byte offsets
    const bool tiled_ok = sh == sw && (sh == 1 || sh == 2) && (long long)f->C * H * W * 16 < 0x7ffffff0LL;
    if (variant < 0 || variant > sf_variant_count()) return FSCNN_ERR_UNSUPPORTED;
    if (variant > 0) {
        SfGeom g;
        if (!tiled_ok || !sf_variant_geom(variant, f->R, f->S, sh, sw, &g)) return FSCNN_ERR_UNSUPPORTED;
        *resolved = variant;
        return FSCNN_OK;
    }
    // N4 tensors need four images per lane whatever the batch size; the choice goes by the
    // output's extent (about the input's divided by the stride)
    // one or two images through NCHW tensors: the four-image forms, their image slots filled with
    // bands of the image (sf_choose_bands), so the choice sees four slots of a quarter (half) the height
    int slots = n4 && N < 4 ? 4 : N, rows = (H + sh - 1) / sh;
    const bool banded = !n4 && N <= 2;
    if (banded) {
        rows = (rows + 4 / N - 1) / (4 / N);
        slots = 4;
    }
    int v = tiled_ok ? sf_choose_variant(slots, f->C, f->K, rows, (W + sw - 1) / sw, f->R, f->S, sh, pool, n4,
                                         density(f), banded, emit)
                     : 0;
    *resolved = v > 0 ? v : -1;
    return FSCNN_OK;
}

// What the direct kernel takes, for the choice between it and the contractions.  Up to 12 entries a filter, and below 16 where up to 8 channels
// leave the contraction in fp32 one chain as well, its sums are as exact as that one's (2-norm against 64 bits 0.95 to 1.02 times, the mean of
// each of a dozen groups of 105 random layers of 3x3 to 7x7) and its time decides (1 -> 300 at 14x9, stride 3, N = 2: 9.2 us contracted, 6.8
// direct; 40 -> 300 5x5 at 16x16, N = 1, 1 % stored: 13.8, 10.1), a quarter ahead for what the estimate is off (12 -> 192 5x5 at 12x12, N = 24,
// 1.5 % stored: estimated 22 us, 30 measured, 22.8 contracted).  Beyond, its chains of roundings show (1.05 to 1.9 times the error of the contraction in
// fp32, 2 to 4 times that of the one in parts): there the contractions serve what was faster so than with one row a thread, though four
// rows a thread take about half of that (21 -> 38 5x5 at 184x189, N = 30, 3 %: estimated 500 us, 640 in parts).
double direct_us(const fscnn_filter_t *f, int N, int Ho, int Wo)
{
    const double waves = (double)N * f->K * ((Wo + 63) / 64) * ((Ho + 3) / 4) * 4, one_row = 9.7 + (double)f->nnz / f->K * (0.132 + 7.48e-5 * waves);
    const bool exact = f->R * f->S >= 9 && f->nnz <= (f->C <= 8 ? 16LL * f->K - 1 : 12LL * f->K);
    return exact ? std::min(1.25 * sf_direct_us(N, f->K, Ho, Wo, f->nnz), one_row) : one_row;
}

// Whether an automatic call is served by the contraction on the matrix cores instead of the resolved
// gather configuration (or the direct kernel), which takes gather_us: by their estimated times (512 -> 512 at
// 28x28, N = 8, measured: 126 / 217 / 320 / 500 us at 10 / 20 / 30 / 50 % stored against 250 us contracted).
// Fewer than 16 input channels leave most of a slice idle (an RGB layer at 224x224, N = 1: 23 us gathered,
// 50 contracted).  Plain NCHW calls only.
bool contracts(const fscnn_filter_t *f, int N, int H, int W, int sh, int sw, int Ho, int Wo, int resolved, double gather_us,
               ContractPick *pick)
{
    const double dense = (double)f->K * f->C * f->R * f->S * Ho * Wo * N, gather = 1e-6 * gather_us;
    if (2 * dense / 150e12 + 4e-6 > gather || (resolved > 0 && f->C < 16)) return false;
    *pick = contract_pick(kContractDense, N, f->C, f->K, H, W, f->R, f->S, Ho, Wo, sh, sw);
    return pick->cfg >= 0 && pick->seconds < gather;
}

// Whether such a call is served by the contraction in bfloat16 parts, where what it would go to otherwise takes
// `other` seconds (512 -> 512 at 28x28, N = 8, any share stored: 250 us contracted in fp32, 132 in parts; gathered 126
// at 10 % stored; 96 -> 256 5x5 at 27x27, N = 8: 82 and 37).  A tenth ahead, for what two estimates are off.  An emitting call's
// results are then counted in a pass of their own (4 us).  Through N4 tensors and with the merged pool another microsecond ahead:
// where the gather takes 8 to 10 us its estimate is 1 to 2 above (47 -> 503 at 6x6, N = 3, pooled: 10.5 us, estimated 11.9; 10.9 in
// parts, estimated 9.2).  NCHW into N4 tensors stays gathered.  Not for filters of fewer than 16 stored entries on average: there
// the rounding of the single products shows (2-norm against 64 bits up to 1.15 times the gather's; from 16 on it was 0.5 times
// that of what served the call before, over 2112 random layers of zero-mean weights, and never more; 0.2 to 0.8 times where
// activations and weights have one sign, over 40 layers).  Nor where one filter stores fewer than 4: a product of six parts is off by
// up to 2^-24 before it is rounded, and the results of such a filter are the less exact ones (rows of 1, 2, 3, 4, 5, 8, 16 entries in banks of
// 150 on average, 2-norm as multiples of the gather's: 1.03, 1.05, 1.01, 0.97, 0.95, 0.88, 0.7; largest error of a single entry 1.5 times).
bool splits(const fscnn_filter_t *f, int N, int H, int W, int sh, int sw, int Ho, int Wo, int pw, bool in4, bool out4, bool pool, double other,
            bool emit, ContractPick *pick)
{
    if (out4 && !in4) return false;
    const double dense = (double)f->K * f->C * f->R * f->S * Ho * Wo * N;
    if (f->nnz < 16LL * f->K || f->fewest < 4 || 2 * dense / 350e12 + 3e-6 > other) return false;
    *pick = split_pick(N, f->C, f->K, H, W, f->R, f->S, Ho, Wo, sh, sw, pw, true, in4, pool);
    return pick->cfg >= 0 && pick->seconds + (emit ? 4e-6 : in4 || pool ? 1e-6 : 0) < 0.9 * other;
}

// Whether a 1x1 call at stride 1 without padding is served by the kernel for these, where what it would go to otherwise takes other_us: by its
// estimated time, a tenth ahead (130 random layers and those of the 52-layer stack: 1.5 times as fast, none slower; 256 -> 128 at 44x44, N = 1, 5 %
// stored, 11.4 us contracted in fp32, 5.4 so; at 52x52, N = 32, through N4 tensors 33 gathered, 60 so).  Its sums are as exact as those of
// the gather kernels or more; the contraction in fp32 is the more exact one, by up to a tenth, from some 150 entries a filter on.
bool pointwise(const fscnn_filter_t *f, int N, int H, int W, bool n4, bool contracted, double other_us)
{
    return f->R == 1 && f->S == 1 && (!contracted || f->nnz <= 128LL * f->K) && pointwise_serves(N, f->C, H, W, f->K, n4) &&
           pointwise_us(N, f->C, H, W, f->K, n4, f->nnz) < 0.9 * other_us;
}

// The plan of `variant` if it is there
SfPlan *made_plan(fscnn_filter_t *f, int variant)
{
    std::lock_guard<std::mutex> lock(f->mu);
    for (SfPlan *p : f->plans)
        if (p->variant == variant) return p;
    return nullptr;
}

// The plan of a contraction (kContractPlan, kSplitPlan) that is to serve an automatic call, NULL where it cannot be made now: no room for
// the bank as a dense array, or a capture on the stream (building it allocates and waits).  The call then goes to
// the gather configuration or the direct kernel, which need none of that or fail for reasons of their own.
fscnn_status_t contract_plan(fscnn_filter_t *f, int variant, hipStream_t st, SfPlan **out)
{
    *out = made_plan(f, variant);
    if (*out) return FSCNN_OK;
    if (capturing(st)) return FSCNN_OK;
    const fscnn_status_t s = get_plan(f, variant, st, out);
    if (s != FSCNN_OK) *out = nullptr;
    return s == FSCNN_ERR_ALLOC ? FSCNN_OK : s;
}

// How a call is served.  An explicitly selected configuration runs as it is; the automatic choice is
// remembered for the geometry (evaluating the models takes up to 3 us).  Call with the handle's lock not held.
fscnn_status_t route_call(fscnn_filter_t *f, int N, int H, int W, int sh, int sw, int pw, int Ho, int Wo, int in4, int out4, int pool,
                          int variant, bool emit, SfRoute *r)
{
    const int key[9] = {N, H, W, sh, sw, pw, Ho, Wo, (in4 ? 1 : 0) | (out4 ? 2 : 0) | (pool ? 4 : 0) | (emit ? 8 : 0)};
    if (variant == 0) {
        std::lock_guard<std::mutex> lock(f->mu);
        for (const auto &c : f->routes)
            if (memcmp(c.key, key, sizeof key) == 0) {
                *r = c;
                return FSCNN_OK;
            }
    }
    *r = SfRoute();
    fscnn_status_t s = resolve_variant(f, N, H, W, sh, sw, variant, &r->variant, in4 || out4, pool != 0, emit);
    if (s != FSCNN_OK) return s;
    sf_choose_bands(r->variant, N, Ho, in4 || out4, pool != 0, &r->band_shift, &r->band_h);
    if (variant != 0) return FSCNN_OK;
    memcpy(r->key, key, sizeof key);
    double us = direct_us(f, N, Ho, Wo);
    if (r->variant > 0)
        r->csplit = sf_choose_csplit(r->variant, N << r->band_shift, f->C, f->K, r->band_h, Wo, density(f), in4, emit, &us);
    r->contract = !in4 && !out4 && !pool && contracts(f, N, H, W, sh, sw, Ho, Wo, r->variant, us, &r->pick);
    r->split = splits(f, N, H, W, sh, sw, Ho, Wo, pw, in4, out4, pool, r->contract ? r->pick.seconds : 1e-6 * us, emit, &r->spick);
    r->pointwise = r->variant != 0 && sh == 1 && sw == 1 && Ho == H && Wo == W && (in4 != 0) == (out4 != 0) && !pool && !emit &&
                   pointwise(f, N, H, W, in4, r->contract, r->contract ? 1e6 * r->pick.seconds : us);
    std::lock_guard<std::mutex> lock(f->mu);
    if (f->routes.size() < 8) {
        f->routes.push_back(*r);
    } else {
        f->routes[f->next_route] = *r;
        f->next_route = (f->next_route + 1) % 8;
    }
    return FSCNN_OK;
}

// Number of stored values of a compressed activation.  A handle made without a host synchronisation
// (sparse output emission) learns it here: wait for the pass that filled it, read the pointer array's
// last element.  Returns -1 on a runtime error.
long long input_nnz(const fscnn_input_t *in)
{
    if (in->nnz >= 0) return in->nnz;
    int total = 0;
    const size_t last = (size_t)in->N * in->H * in->W * (size_t)in->NCH;
    if (hipEventSynchronize(in->filled) != hipSuccess ||
        hipMemcpy(&total, in->cptr + last, sizeof(int), hipMemcpyDeviceToHost) != hipSuccess) {
        (void)hipGetLastError();
        return -1;
    }
    const_cast<fscnn_input_t *>(in)->nnz = total;   // a cache of what the device holds
    return total;
}

// Room for a bank in bfloat16 parts on `st`: the buffer this stream used before on the handle if it is large enough, else a
// new one; NULL where there is none and none can be made (no room, or `st` is capturing).  One per stream: calls that share a
// handle on different streams never share it.  A capture takes over the stream's buffer: its graph may be replayed on any stream,
// beside later calls on this one, which make another.  Call with in->mu held, and hold it until the launches that write and read the room are
// made: calls of two threads on one stream share it in stream order, launches of one must not come between the other's.
void *bank_scratch(const fscnn_input *in, hipStream_t st, size_t bytes)
{
    constexpr int kGraphs = 16;                       // that have a buffer of the handle
    const unsigned long long graph = capture_id(st);
    fscnn_input::Bank *own = nullptr;                 // not in a graph
    int graphs = 0;
    for (auto &b : in->banks) {
        graphs += b.graph != 0;
        if (b.stream != st || b.bytes < bytes) continue;
        if (b.graph == graph) return b.buf;
        if (!b.graph) own = &b;
    }
    if (st) in->in_order = false;
    if (graph) {
        if (!own || graphs >= kGraphs) return nullptr;
        own->graph = graph;
        return own->buf;
    }
    void *p = nullptr;
    size_t room = 1 << 20;                            // (powers of two: what outgrown buffers hold is bounded by the largest)
    while (room < bytes) room *= 2;
    if (block_alloc(input_pool(), in->device, st, &p, room, &bytes) != hipSuccess) {
        (void)hipGetLastError();
        return nullptr;
    }
    // (a smaller one stays with the handle: launches in flight and graphs captured so far use it)
    in->banks.push_back({st, p, bytes, 0});
    return p;
}

// Orders work on `st` behind the pass that fills a compressed-activation handle (it runs on the
// stream the handle was made on and may still be in flight).
hipError_t after_fill(const fscnn_input_t *in, hipStream_t st)
{
    if (st) in->in_order = false;
    return st == in->made_on ? hipSuccess : hipStreamWaitEvent(st, in->filled, 0);
}

fscnn_status_t check_conv_args(const fscnn_filter_t *f, const float *x, int N, int C, int H, int W,
                               int sh, int sw, int ph, int pw, const float *y, int *Ho, int *Wo)
{
    if (!f || !x || !y) return FSCNN_ERR_NULL;
    if (!live(f)) return FSCNN_ERR_HANDLE;
    if (N <= 0 || C <= 0) return FSCNN_ERR_SHAPE;
    fscnn_status_t s = out_shape(H, W, f->R, f->S, sh, sw, ph, pw, Ho, Wo);
    if (s != FSCNN_OK) return s;
    if (C != f->C) return FSCNN_ERR_MISMATCH;
    // one image's tensors are indexed with ints; images are addressed with 64-bit offsets, so the
    // batch is bounded only by the number of work-groups a launch can have (checked there)
    if (!fits_int((long long)C * H * W) || !fits_int((long long)f->K * *Ho * *Wo)) return FSCNN_ERR_UNSUPPORTED;
    if (x == y) return FSCNN_ERR_UNSUPPORTED;
    return FSCNN_OK;
}

}  // namespace

extern "C" {

const char *fscnn_status_string(fscnn_status_t s)
{
    switch (s) {
        case FSCNN_OK: return "ok";
        case FSCNN_ERR_NULL: return "null pointer argument";
        case FSCNN_ERR_SHAPE: return "invalid shape (non-positive size, negative pad or empty output)";
        case FSCNN_ERR_MISMATCH: return "tensor dimensions do not match the handle";
        case FSCNN_ERR_UNSUPPORTED: return "request outside what the kernels cover";
        case FSCNN_ERR_ALLOC: return "allocation failed";
        case FSCNN_ERR_DEVICE: return "HIP runtime error or no device";
        case FSCNN_ERR_HANDLE: return "not a live handle";
    }
    return "unknown status";
}

fscnn_status_t fscnn_conv2d_out_shape(int H, int W, int R, int S, int sh, int sw, int ph, int pw,
                                      int *Ho, int *Wo)
{
    if (!Ho || !Wo) return FSCNN_ERR_NULL;
    return out_shape(H, W, R, S, sh, sw, ph, pw, Ho, Wo);
}

fscnn_status_t fscnn_filter_compress(const float *w_dev, int K, int C, int R, int S, void *stream,
                                     fscnn_filter_t **out)
{
    if (!w_dev || !out) return FSCNN_ERR_NULL;
    if (K <= 0 || C <= 0 || R <= 0 || S <= 0) return FSCNN_ERR_SHAPE;
    const long long row = (long long)C * R * S;
    if (!fits_int(row) || !fits_int(row * K)) return FSCNN_ERR_SHAPE;
    int dev;
    fscnn_status_t s = have_device(&dev);
    if (s != FSCNN_OK) return s;
    hipStream_t st = (hipStream_t)stream;

    fscnn_filter_t *f = new (std::nothrow) fscnn_filter();
    if (!f) return FSCNN_ERR_ALLOC;
    f->magic = kFilterMagic;
    f->device = dev;
    f->K = K; f->C = C; f->R = R; f->S = S;
    f->nnz = 0;
    f->rowptr = nullptr; f->idx = nullptr; f->val = nullptr;
    f->in_order = !st;
    int *cnt = nullptr;
    int total = 0;
    HostWord word, packed;
    // two allocations: the pointers with the counts they are scanned from, and the nodes
    hipError_t e = filter_alloc(dev, st, reinterpret_cast<void **>(&f->rowptr),
                               sizeof(int) * (size_t)(K + 2 + K + scan_tmp_elems(K)), &f->rowptr_bytes);
    if (e == hipSuccess) cnt = f->rowptr + (K + 2);
    if (e == hipSuccess) e = launch_filter_count(w_dev, K, row, cnt, f->rowptr, word.slot(), word.hand_out(), st);
    if (e == hipSuccess) e = word.wait(f->rowptr + K, st, &total, &f->fewest);
    if (e == hipSuccess && total < 0) e = hipErrorUnknown;
    if (e == hipSuccess) {
        f->nnz = total;
        const size_t n = total > 0 ? (size_t)total : 1;
        e = filter_alloc(dev, st, reinterpret_cast<void **>(&f->idx), (sizeof(uint32_t) + sizeof(float)) * n, &f->idx_bytes);
        if (e == hipSuccess) f->val = reinterpret_cast<float *>(f->idx + n);
    }
    if (e == hipSuccess) e = launch_filter_pack(w_dev, K, row, f->rowptr, f->idx, f->val, packed.slot(), packed.hand_out(), st);
    if (e == hipSuccess) e = packed.wait(nullptr, st, &total);   // (w may be another's from here on, and any stream use the handle)
    if (e != hipSuccess) {
        (void)hipGetLastError();
        if (f->rowptr) (void)hipFree(f->rowptr);
        if (f->idx) (void)hipFree(f->idx);   // with the values behind the indices
        f->magic = 0;
        delete f;
        return e == hipErrorOutOfMemory ? FSCNN_ERR_ALLOC : FSCNN_ERR_DEVICE;
    }
    *out = f;
    return FSCNN_OK;
}

fscnn_status_t fscnn_filter_info(const fscnn_filter_t *f, int *K, int *C, int *R, int *S,
                                 long long *nnz)
{
    if (!f) return FSCNN_ERR_NULL;
    if (!live(f)) return FSCNN_ERR_HANDLE;
    if (K) *K = f->K;
    if (C) *C = f->C;
    if (R) *R = f->R;
    if (S) *S = f->S;
    if (nnz) *nnz = f->nnz;
    return FSCNN_OK;
}

fscnn_status_t fscnn_filter_export(const fscnn_filter_t *f, int *rowptr_host, unsigned *idx_host,
                                   float *val_host)
{
    if (!f || !rowptr_host) return FSCNN_ERR_NULL;
    if (!live(f)) return FSCNN_ERR_HANDLE;
    if (f->nnz > 0 && (!idx_host || !val_host)) return FSCNN_ERR_NULL;
    FSCNN_HIP(hipMemcpy(rowptr_host, f->rowptr, sizeof(int) * (size_t)(f->K + 1), hipMemcpyDeviceToHost));
    if (f->nnz > 0) {
        FSCNN_HIP(hipMemcpy(idx_host, f->idx, sizeof(uint32_t) * (size_t)f->nnz, hipMemcpyDeviceToHost));
        FSCNN_HIP(hipMemcpy(val_host, f->val, sizeof(float) * (size_t)f->nnz, hipMemcpyDeviceToHost));
    }
    return FSCNN_OK;
}

fscnn_status_t fscnn_filter_prepare_ex(fscnn_filter_t *f, int N, int H, int W, int sh, int sw, int ph,
                                       int pw, fscnn_layout_t x_layout, fscnn_layout_t y_layout, int pool,
                                       int variant, void *stream)
{
    if (!f) return FSCNN_ERR_NULL;
    if (!live(f)) return FSCNN_ERR_HANDLE;
    if (N <= 0) return FSCNN_ERR_SHAPE;
    if ((x_layout != FSCNN_LAYOUT_NCHW && x_layout != FSCNN_LAYOUT_N4) ||
        (y_layout != FSCNN_LAYOUT_NCHW && y_layout != FSCNN_LAYOUT_N4))
        return FSCNN_ERR_UNSUPPORTED;
    int Ho, Wo;
    fscnn_status_t s = out_shape(H, W, f->R, f->S, sh, sw, ph, pw, &Ho, &Wo);
    if (s != FSCNN_OK) return s;
    const int in4 = x_layout == FSCNN_LAYOUT_N4, out4 = y_layout == FSCNN_LAYOUT_N4;
    SfRoute r;
    s = route_call(f, N, H, W, sh, sw, pw, Ho, Wo, in4, out4, pool, variant, false, &r);
    if (s != FSCNN_OK) return s;
    if ((in4 || out4 || pool) && r.variant < 0) return FSCNN_ERR_UNSUPPORTED;
    if (r.variant > 0 && !sf_variant_has_layout(r.variant, in4, out4, pool)) return FSCNN_ERR_UNSUPPORTED;
    if (r.pointwise) {
        int dev;
        s = have_device(&dev);
        return s == FSCNN_OK && dev != f->device ? FSCNN_ERR_MISMATCH : s;
    }
    if (stream) f->in_order = false;
    SfPlan *p = nullptr;
    if (r.split) s = contract_plan(f, kSplitPlan, (hipStream_t)stream, &p);
    if (p && r.spick.parts > 1) (void)split_sums(f, p, (hipStream_t)stream, split_sums_bytes(r.spick, N, f->K, Ho, Wo, in4));
    if (s != FSCNN_OK || p) return s;
    if (r.contract) s = contract_plan(f, kContractPlan, (hipStream_t)stream, &p);
    if (s != FSCNN_OK || p) return s;
    s = get_plan(f, r.variant, (hipStream_t)stream, &p);
    if (s != FSCNN_OK || p->direct) return s;
    if (r.csplit > 1) {
        float *parts;
        s = split_scratch(f, p, (hipStream_t)stream, sf_split_bytes(p->g, r.csplit, N << r.band_shift, f->K, r.band_h, Wo), &parts);
    }
    return s;
}

fscnn_status_t fscnn_filter_prepare(fscnn_filter_t *f, int N, int H, int W, int sh, int sw, int ph,
                                    int pw, int variant, void *stream)
{
    return fscnn_filter_prepare_ex(f, N, H, W, sh, sw, ph, pw, FSCNN_LAYOUT_NCHW, FSCNN_LAYOUT_NCHW, 0, variant,
                                   stream);
}

fscnn_status_t fscnn_filter_plan_export(fscnn_filter_t *f, int N, int H, int W, int sh, int sw,
                                        int ph, int pw, int variant, int *params_host,
                                        int *segptr_host, unsigned *rec_off_host,
                                        float *rec_val_host)
{
    if (!f || !params_host) return FSCNN_ERR_NULL;
    if (!live(f)) return FSCNN_ERR_HANDLE;
    if (N <= 0) return FSCNN_ERR_SHAPE;
    int Ho, Wo;
    fscnn_status_t s = out_shape(H, W, f->R, f->S, sh, sw, ph, pw, &Ho, &Wo);
    if (s != FSCNN_OK) return s;
    int v;
    s = resolve_variant(f, N, H, W, sh, sw, variant, &v);
    if (s != FSCNN_OK) return s;
    SfPlan *p;
    s = get_plan(f, v, nullptr, &p);
    if (s != FSCNN_OK) return s;
    for (int i = 0; i < 16; ++i) params_host[i] = 0;
    params_host[0] = p->variant;
    params_host[9] = p->direct ? 1 : 0;
    if (p->direct) return FSCNN_OK;
    params_host[1] = p->g.CC;
    params_host[2] = p->g.KG;
    params_host[3] = p->NCH;
    params_host[4] = p->NG;
    params_host[5] = p->g.IN_ROWS;
    params_host[6] = p->g.PITCH;
    params_host[7] = p->g.BV;
    params_host[8] = (int)p->nrec;
    params_host[10] = p->g.SLOTS;
    params_host[11] = p->g.WAVES;
    params_host[12] = p->g.DENSE;
    const long long nb = (long long)p->NG * p->NCH * p->g.KG;
    if (segptr_host)
        FSCNN_HIP(hipMemcpy(segptr_host, p->segptr, sizeof(int) * (size_t)(nb + 1), hipMemcpyDeviceToHost));
    if ((rec_off_host || rec_val_host) && p->nrec > 0) {
        if (!rec_off_host || !rec_val_host) return FSCNN_ERR_NULL;
        Rec *tmp = new (std::nothrow) Rec[(size_t)p->nrec];
        if (!tmp) return FSCNN_ERR_ALLOC;
        hipError_t e = hipMemcpy(tmp, p->recs, sizeof(Rec) * (size_t)p->nrec, hipMemcpyDeviceToHost);
        if (e == hipSuccess)
            for (long long i = 0; i < p->nrec; ++i) {
                rec_off_host[i] = tmp[i].off;
                rec_val_host[i] = tmp[i].val;
            }
        delete[] tmp;
        FSCNN_HIP(e);
    }
    return FSCNN_OK;
}

fscnn_status_t fscnn_filter_destroy(fscnn_filter_t *f)
{
    if (!f) return FSCNN_ERR_NULL;
    if (!live(f)) return FSCNN_ERR_HANDLE;
    f->magic = 0;
    size_t largest = std::max(f->rowptr_bytes, f->idx_bytes);
    for (const SfPlan *p : f->plans)
        for_blocks(p, [&](void *, size_t bytes) { largest = std::max(largest, bytes); });
    const Left left = blocks_left(f->device, f->in_order, largest);
    for (SfPlan *p : f->plans) free_plan(p, f->device, left);
    f->plans.clear();
    filter_free(f->device, f->rowptr, f->rowptr_bytes, left);
    filter_free(f->device, f->idx, f->idx_bytes, left);
    delete f;
    return FSCNN_OK;
}

fscnn_status_t fscnn_pool_trim(void)
{
    filter_pool(0).trim();
    filter_pool(~(size_t)0).trim();
    input_pool().trim();
    return FSCNN_OK;
}

int fscnn_sf_variant_count(void) { return sf_variant_count(); }
const char *fscnn_sf_variant_name(int variant) { return sf_variant_name(variant); }

fscnn_status_t fscnn_sf_variant_choice(const fscnn_filter_t *f, int N, int H, int W, int sh, int sw,
                                       int n4, int pool, int *variant_out)
{
    if (!f || !variant_out) return FSCNN_ERR_NULL;
    if (!live(f)) return FSCNN_ERR_HANDLE;
    if (N <= 0 || H <= 0 || W <= 0 || sh <= 0 || sw <= 0) return FSCNN_ERR_SHAPE;
    return resolve_variant(f, N, H, W, sh, sw, 0, variant_out, n4 != 0, pool != 0);
}

fscnn_status_t fscnn_sf_band_choice(int variant, int N, int Ho, int n4, int pool, int *bands_out,
                                    int *band_rows_out)
{
    if (!bands_out || !band_rows_out) return FSCNN_ERR_NULL;
    if (N <= 0 || Ho <= 0) return FSCNN_ERR_SHAPE;
    if (variant < 1 || variant > sf_variant_count()) return FSCNN_ERR_UNSUPPORTED;
    int shift;
    sf_choose_bands(variant, N, Ho, n4 != 0, pool != 0, &shift, band_rows_out);
    *bands_out = 1 << shift;
    return FSCNN_OK;
}

fscnn_status_t fscnn_sf_contract_choice(fscnn_filter_t *f, int N, int H, int W, int sh, int sw, int ph, int pw,
                                        int *tile_out, int *panels_out)
{
    if (!f || !tile_out || !panels_out) return FSCNN_ERR_NULL;
    if (!live(f)) return FSCNN_ERR_HANDLE;
    if (N <= 0) return FSCNN_ERR_SHAPE;
    int Ho, Wo;
    fscnn_status_t s = out_shape(H, W, f->R, f->S, sh, sw, ph, pw, &Ho, &Wo);
    if (s != FSCNN_OK) return s;
    SfRoute r;
    s = route_call(f, N, H, W, sh, sw, pw, Ho, Wo, 0, 0, 0, 0, false, &r);
    if (s != FSCNN_OK) return s;
    const bool served = r.contract && !r.pointwise;
    *tile_out = served ? r.pick.cfg : -1;
    *panels_out = served ? r.pick.npan : 0;
    return FSCNN_OK;
}

fscnn_status_t fscnn_sf_split_choice(fscnn_filter_t *f, int N, int H, int W, int sh, int sw, int ph, int pw,
                                     int *tile_out, int *panels_out, int *parts_out)
{
    if (!f || !tile_out || !panels_out) return FSCNN_ERR_NULL;
    if (!live(f)) return FSCNN_ERR_HANDLE;
    if (N <= 0) return FSCNN_ERR_SHAPE;
    int Ho, Wo;
    fscnn_status_t s = out_shape(H, W, f->R, f->S, sh, sw, ph, pw, &Ho, &Wo);
    if (s != FSCNN_OK) return s;
    SfRoute r;
    s = route_call(f, N, H, W, sh, sw, pw, Ho, Wo, 0, 0, 0, 0, false, &r);
    if (s != FSCNN_OK) return s;
    if (parts_out) *parts_out = r.split ? r.spick.parts : 0;
    *tile_out = r.split ? r.spick.cfg : -1;
    *panels_out = r.split ? r.spick.npan : 0;
    return FSCNN_OK;
}

fscnn_status_t fscnn_sf_serves(fscnn_filter_t *f, int N, int H, int W, int sh, int sw, int ph, int pw, fscnn_layout_t x_layout,
                               fscnn_layout_t y_layout, int pool, int *serves_out)
{
    if (!f || !serves_out) return FSCNN_ERR_NULL;
    if (!live(f)) return FSCNN_ERR_HANDLE;
    if (N <= 0) return FSCNN_ERR_SHAPE;
    if ((x_layout != FSCNN_LAYOUT_NCHW && x_layout != FSCNN_LAYOUT_N4) || (y_layout != FSCNN_LAYOUT_NCHW && y_layout != FSCNN_LAYOUT_N4))
        return FSCNN_ERR_UNSUPPORTED;
    int Ho, Wo;
    fscnn_status_t s = out_shape(H, W, f->R, f->S, sh, sw, ph, pw, &Ho, &Wo);
    if (s != FSCNN_OK) return s;
    if (pool && (Ho < 2 || Wo < 2)) return FSCNN_ERR_SHAPE;
    const int in4 = x_layout == FSCNN_LAYOUT_N4, out4 = y_layout == FSCNN_LAYOUT_N4;
    SfRoute r;
    s = route_call(f, N, H, W, sh, sw, pw, Ho, Wo, in4, out4, pool, 0, false, &r);
    if (s != FSCNN_OK) return s;
    if ((in4 || out4 || pool) && r.variant < 0) return FSCNN_ERR_UNSUPPORTED;
    if (r.variant > 0 && !sf_variant_has_layout(r.variant, in4, out4, pool)) return FSCNN_ERR_UNSUPPORTED;
    *serves_out = r.pointwise ? FSCNN_SERVES_POINTWISE : r.split ? FSCNN_SERVES_SPLIT : r.contract ? FSCNN_SERVES_CONTRACT
                  : r.variant > 0 ? FSCNN_SERVES_GATHER : FSCNN_SERVES_DIRECT;
    return FSCNN_OK;
}

fscnn_status_t fscnn_si_contract_choice(int N, int C, int H, int W, int K, int ph, int pw, int prepared, long long *from_out,
                                        int *tile_out, int *panels_out)
{
    if (!from_out || !tile_out || !panels_out) return FSCNN_ERR_NULL;
    if (N <= 0 || C <= 0 || K <= 0) return FSCNN_ERR_SHAPE;
    int Ho, Wo;
    fscnn_status_t s = out_shape(H, W, 3, 3, 1, 1, ph, pw, &Ho, &Wo);
    if (s != FSCNN_OK) return s;
    if (!fits_int((long long)N * C * H * W) || !fits_int((long long)N * K * Ho * Wo) || !fits_int((long long)K * C * 9))
        return FSCNN_ERR_UNSUPPORTED;
    const SiChoice c = si_choose(N, C, H, W, K, Ho, Wo, pw, prepared != 0);
    *from_out = c.from;
    *tile_out = c.pick.cfg;
    *panels_out = c.pick.cfg < 0 ? 0 : c.pick.npan;
    return FSCNN_OK;
}

fscnn_status_t fscnn_si_split_choice(int N, int C, int H, int W, int K, int ph, int pw, int prepared, long long *from_out,
                                     int *tile_out, int *panels_out)
{
    if (!from_out || !tile_out || !panels_out) return FSCNN_ERR_NULL;
    if (N <= 0 || C <= 0 || K <= 0) return FSCNN_ERR_SHAPE;
    int Ho, Wo;
    fscnn_status_t s = out_shape(H, W, 3, 3, 1, 1, ph, pw, &Ho, &Wo);
    if (s != FSCNN_OK) return s;
    if (!fits_int((long long)N * C * H * W) || !fits_int((long long)N * K * Ho * Wo) || !fits_int((long long)K * C * 9))
        return FSCNN_ERR_UNSUPPORTED;
    const SiChoice c = si_choose(N, C, H, W, K, Ho, Wo, pw, prepared != 0);
    *from_out = c.split_from;
    *tile_out = c.spick.cfg;
    *panels_out = c.spick.cfg >= 0 ? c.spick.npan : 0;
    return FSCNN_OK;
}

// emit_cnt / counted: sparse output emission.  When the launch that serves the call can count the
// non-zero results per (pixel, step of 8 channels) in its epilogue it writes them to emit_cnt and
// sets *counted; otherwise the caller counts in a pass of its own.
static fscnn_status_t conv_sf_common(fscnn_filter_t *f, const float *x_dev, int N, int C, int H,
                                     int W, int sh, int sw, int ph, int pw, const float *bias_dev,
                                     int relu, float *y_dev, fscnn_layout_t x_layout,
                                     fscnn_layout_t y_layout, int variant, int pool, void *stream,
                                     int *emit_cnt = nullptr, bool *counted = nullptr)
{
    if (counted) *counted = false;
    int Ho, Wo;
    fscnn_status_t s = check_conv_args(f, x_dev, N, C, H, W, sh, sw, ph, pw, y_dev, &Ho, &Wo);
    if (s != FSCNN_OK) return s;
    if ((x_layout != FSCNN_LAYOUT_NCHW && x_layout != FSCNN_LAYOUT_N4) ||
        (y_layout != FSCNN_LAYOUT_NCHW && y_layout != FSCNN_LAYOUT_N4))
        return FSCNN_ERR_UNSUPPORTED;
    const int in4 = x_layout == FSCNN_LAYOUT_N4, out4 = y_layout == FSCNN_LAYOUT_N4;
    if ((in4 && ((uintptr_t)x_dev & 15)) || (out4 && ((uintptr_t)y_dev & 15))) return FSCNN_ERR_UNSUPPORTED;
    // (a group of four interleaved images is indexed with ints, the groups with 64-bit offsets)
    if ((in4 && !fits_int(4LL * C * H * W)) || (out4 && !fits_int(4LL * f->K * Ho * Wo)))
        return FSCNN_ERR_UNSUPPORTED;
    if (pool && (Ho < 2 || Wo < 2)) return FSCNN_ERR_SHAPE;   // empty pooled output
    SfRoute r;
    s = route_call(f, N, H, W, sh, sw, pw, Ho, Wo, in4, out4, pool, variant, emit_cnt != nullptr, &r);
    if (s != FSCNN_OK) return s;
    if ((in4 || out4 || pool) && r.variant < 0) return FSCNN_ERR_UNSUPPORTED;   // the direct kernel: NCHW, no pool
    if (r.variant > 0 && !sf_variant_has_layout(r.variant, in4, out4, pool)) return FSCNN_ERR_UNSUPPORTED;
    int dev;
    s = have_device(&dev);
    if (s != FSCNN_OK) return s;
    if (dev != f->device) return FSCNN_ERR_MISMATCH;   // the handle's buffers live on another GPU
    hipStream_t st = (hipStream_t)stream;
    if (st) f->in_order = false;
    if (r.pointwise) {
        FSCNN_HIP(launch_pointwise(f->rowptr, f->idx, f->val, x_dev, N, C, H, W, f->K, in4 != 0, bias_dev, relu, y_dev, st));
        return FSCNN_OK;
    }
    SfPlan *p = nullptr;
    if (r.split) s = contract_plan(f, kSplitPlan, st, &p);
    if (s != FSCNN_OK) return s;
    // from the choice of scratch to the last launch that uses it: threads that share a handle share a stream's scratch in
    // stream order, and a launch of one must not come between the two of another
    std::unique_lock<std::mutex> launching(f->launching, std::defer_lock);
    if (p) {
        if (r.spick.parts > 1) launching.lock();
        float *sums = r.spick.parts > 1 ? split_sums(f, p, st, split_sums_bytes(r.spick, N, f->K, Ho, Wo, in4)) : nullptr;
        FSCNN_HIP(launch_split_dense(x_dev, p->parts, f->rowptr, f->idx, f->val, N, C, H, W, f->K, f->R, Ho, Wo, sh, sw, ph, pw,
                                     bias_dev, relu, y_dev, in4, out4, pool, r.spick, sums, st));
        return FSCNN_OK;
    }
    if (r.contract) s = contract_plan(f, kContractPlan, st, &p);
    if (s != FSCNN_OK) return s;
    if (p) {
        // (the tiled gather kernels multiply entries outside the image by zeros as well)
        const int *wflag = r.variant < 0 ? reinterpret_cast<const int *>(p->packed + contract_packed_elems(f->K, f->C, f->R * f->S)) : nullptr;
        FSCNN_HIP(launch_contract_dense(x_dev, p->packed, wflag, f->rowptr, f->idx, f->val, N, C, H, W, f->K, f->R, f->S,
                                        Ho, Wo, sh, sw, ph, pw, bias_dev, relu, y_dev, r.pick, st));
        return FSCNN_OK;
    }
    // (the 1x1 kernel is what prepares nothing for the geometry, so an emitting call may find no plan in a capture, which cannot make one)
    if (emit_cnt && f->R == 1 && f->S == 1 && sh == 1 && sw == 1 && Ho == H && Wo == W && pointwise_serves(N, C, H, W, f->K, false) &&
        !made_plan(f, r.variant) && capturing(st)) {
        FSCNN_HIP(launch_pointwise(f->rowptr, f->idx, f->val, x_dev, N, C, H, W, f->K, false, bias_dev, relu, y_dev, st));
        return FSCNN_OK;
    }
    s = get_plan(f, r.variant, st, &p);
    if (s != FSCNN_OK) return s;
    if (p->direct) {
        FSCNN_HIP(launch_conv_sf_direct(f->rowptr, f->idx, f->val, x_dev, N, C, H, W, f->K, f->R,
                                        f->S, Ho, Wo, sh, sw, ph, pw, bias_dev, relu, y_dev, st));
    } else {
        float *parts = nullptr;
        if (r.csplit > 1) {
            launching.lock();
            s = split_scratch(f, p, st, sf_split_bytes(p->g, r.csplit, N << r.band_shift, f->K, r.band_h, Wo), &parts);
            if (s != FSCNN_OK) return s;
        }
        int *cnt = (emit_cnt && !out4 && !pool) ? emit_cnt : nullptr;
        FSCNN_HIP(launch_conv_sf_tiled(*p, x_dev, N, C, H, W, f->K, Ho, Wo, ph, pw, bias_dev, relu,
                                       y_dev, in4, out4, pool, r.csplit, parts, cnt, r.band_shift, r.band_h, st));
        if (counted) *counted = cnt != nullptr;
    }
    return FSCNN_OK;
}

fscnn_status_t fscnn_conv2d_sparse_filter_ex(fscnn_filter_t *f, const float *x_dev, int N, int C,
                                             int H, int W, int sh, int sw, int ph, int pw,
                                             const float *bias_dev, int relu, float *y_dev,
                                             fscnn_layout_t x_layout, fscnn_layout_t y_layout,
                                             int variant, void *stream)
{
    return conv_sf_common(f, x_dev, N, C, H, W, sh, sw, ph, pw, bias_dev, relu, y_dev, x_layout,
                          y_layout, variant, 0, stream);
}

fscnn_status_t fscnn_conv2d_sparse_filter_leaky(fscnn_filter_t *f, const float *x_dev, int N, int C,
                                                int H, int W, int sh, int sw, int ph, int pw,
                                                const float *bias_dev, float negative_slope,
                                                float *y_dev, fscnn_layout_t x_layout,
                                                fscnn_layout_t y_layout, int variant, void *stream)
{
    if (!(negative_slope >= 0.0f && negative_slope <= 1.0f)) return FSCNN_ERR_SHAPE;   // also rejects NaN
    return conv_sf_common(f, x_dev, N, C, H, W, sh, sw, ph, pw, bias_dev, act_code(negative_slope),
                          y_dev, x_layout, y_layout, variant, 0, stream);
}

fscnn_status_t fscnn_conv2d_sparse_filter_pool2x2(fscnn_filter_t *f, const float *x_dev, int N,
                                                  int C, int H, int W, int sh, int sw, int ph,
                                                  int pw, const float *bias_dev, int relu,
                                                  float *y_dev, fscnn_layout_t x_layout,
                                                  fscnn_layout_t y_layout, int variant,
                                                  void *stream)
{
    return conv_sf_common(f, x_dev, N, C, H, W, sh, sw, ph, pw, bias_dev, relu, y_dev, x_layout,
                          y_layout, variant, 1, stream);
}

fscnn_status_t fscnn_conv2d_sparse_filter_v(fscnn_filter_t *f, const float *x_dev, int N, int C,
                                            int H, int W, int sh, int sw, int ph, int pw,
                                            const float *bias_dev, int relu, float *y_dev,
                                            int variant, void *stream)
{
    return fscnn_conv2d_sparse_filter_ex(f, x_dev, N, C, H, W, sh, sw, ph, pw, bias_dev, relu, y_dev,
                                         FSCNN_LAYOUT_NCHW, FSCNN_LAYOUT_NCHW, variant, stream);
}

fscnn_status_t fscnn_layout_convert(const float *src_dev, int N, int C, int H, int W,
                                    fscnn_layout_t src_layout, float *dst_dev,
                                    fscnn_layout_t dst_layout, void *stream)
{
    if (!src_dev || !dst_dev) return FSCNN_ERR_NULL;
    if (N <= 0 || C <= 0 || H <= 0 || W <= 0) return FSCNN_ERR_SHAPE;
    const bool s4 = src_layout == FSCNN_LAYOUT_N4, d4 = dst_layout == FSCNN_LAYOUT_N4;
    if ((!s4 && src_layout != FSCNN_LAYOUT_NCHW) || (!d4 && dst_layout != FSCNN_LAYOUT_NCHW) ||
        s4 == d4 || src_dev == dst_dev)
        return FSCNN_ERR_UNSUPPORTED;
    if (!fits_int(((long long)N + 3) / 4 * 4 * C * H * W)) return FSCNN_ERR_UNSUPPORTED;
    if ((uintptr_t)(s4 ? src_dev : dst_dev) & 15) return FSCNN_ERR_UNSUPPORTED;
    int dev;
    fscnn_status_t s = have_device(&dev);
    if (s != FSCNN_OK) return s;
    FSCNN_HIP(launch_layout_convert(src_dev, N, C, H, W, s4 ? 1 : 0, dst_dev, (hipStream_t)stream));
    return FSCNN_OK;
}

fscnn_status_t fscnn_conv2d_sparse_filter(fscnn_filter_t *f, const float *x_dev, int N, int C, int H,
                                          int W, int sh, int sw, int ph, int pw,
                                          const float *bias_dev, int relu, float *y_dev,
                                          void *stream)
{
    return fscnn_conv2d_sparse_filter_v(f, x_dev, N, C, H, W, sh, sw, ph, pw, bias_dev, relu, y_dev,
                                        0, stream);
}

// Dense N x C x H x W activations -> compressed handle.  Waits once, for the number of stored
// values.  Up to kWholeBytes of indices and values, were every value stored, are allocated with the
// pointers before anything runs (and as much again for the dense form, input_dense_from()), and the passes follow each other without the host; beyond that the
// number of stored values sizes a second allocation (making and releasing one takes 50 us, more than
// the passes of a 28x28 layer), and also where the live handles already hold kUnusedBytes more than they store
// or the allocation fails.  The pass that fills the handle may still be running on st when this
// returns, and reads x.
constexpr long long kWholeBytes = 256LL << 20, kUnusedBytes = 1LL << 30;
std::atomic<long long> unused_bytes{0};
static fscnn_status_t compress_activations(const float *x_dev, int N, int C, int H, int W,
                                           hipStream_t st, fscnn_input_t **out)
{
    if (N <= 0 || C <= 0 || H <= 0 || W <= 0) return FSCNN_ERR_SHAPE;
    const long long npix = (long long)N * H * W;
    if (!fits_int(npix + 1) || !fits_int(npix * C)) return FSCNN_ERR_SHAPE;
    const int CC = kSiCC, NCH = (C + CC - 1) / CC;
    // the packing pass keeps a pixel's whole list in LDS: up to 8192 channels
    if (!fits_int(npix * NCH + 1) || NCH > 8192 / kSiCC) return FSCNN_ERR_UNSUPPORTED;
    int dev;
    fscnn_status_t s = have_device(&dev);
    if (s != FSCNN_OK) return s;
    fscnn_input_t *in = new (std::nothrow) fscnn_input();
    if (!in) return FSCNN_ERR_ALLOC;
    in->magic = kInputMagic;
    in->device = dev;
    in->N = N; in->C = C; in->H = H; in->W = W;
    in->nnz = 0; in->CC = CC; in->NCH = NCH;
    in->cidx = nullptr; in->xval = nullptr; in->cptr = nullptr;
    in->ptr_block = nullptr; in->node_block = nullptr;
    in->made_on = st; in->filled = nullptr;
    in->in_order = !st;
    int total = 0;
    HostWord word;
    const long long nstep = npix * NCH;   // (pixel, channel step) pairs
    auto up = [](size_t v) { return (v + 255) / 256 * 256; };
    // first allocation: the pointer array, the scratch of the passes (it stays with the handle, so nothing
    // is freed here), and the nodes if they are allocated for the worst case.  Spare entries: the
    // sparse-input kernels fetch the next (channel, value) pairs of a pixel's list ahead, up to kSiSpare
    // positions past the one in use
    const size_t scratch_at = up((size_t)(nstep + 1) * sizeof(int));
    const size_t nodes_at = scratch_at + up(sizeof(int) * (size_t)input_scratch_elems(npix, NCH));
    auto val_at = [&](size_t n) { return up(n * sizeof(uint32_t)); };
    const size_t most = (size_t)(npix * C) + kSiSpare;
    const size_t dense_at = up(nodes_at + val_at(most) + most * sizeof(float));
    bool whole = npix * C * 8 <= kWholeBytes && unused_bytes.load() + npix * C * 12 <= kUnusedBytes;
    hipError_t e = hipErrorOutOfMemory;
    if (whole) {
        e = block_alloc(input_pool(), dev, st, &in->ptr_block, dense_at + sizeof(float) * (size_t)(npix * C), &in->ptr_bytes);
        if (e == hipErrorOutOfMemory) {
            (void)hipGetLastError();
            whole = false;
        }
    }
    if (!whole) e = block_alloc(input_pool(), dev, st, &in->ptr_block, nodes_at, &in->ptr_bytes);
    int *scratch = nullptr, *host = nullptr;
    const bool scanned = !whole || input_scans(npix, NCH);   // (the number sizes the second allocation)
    auto fill = [&](void *nodes, size_t n) {
        in->cidx = static_cast<uint32_t *>(nodes);
        in->xval = reinterpret_cast<float *>(static_cast<char *>(nodes) + val_at(n));
        float *dense = whole ? reinterpret_cast<float *>(static_cast<char *>(in->ptr_block) + dense_at) : nullptr;
        return launch_input_fill(x_dev, N, C, H, W, NCH, scratch, scanned, in->cptr, in->cidx, in->xval, kSiSpare, dense, input_dense_from(npix, C),
                                 scanned ? nullptr : host, st);
    };
    if (e == hipSuccess) {
        char *base = static_cast<char *>(in->ptr_block);
        in->cptr = reinterpret_cast<int *>(base);
        scratch = reinterpret_cast<int *>(base + scratch_at);
        host = word.hand_out();
        e = launch_input_sums(x_dev, nullptr, N, C, H, W, NCH, scratch, scanned, scanned ? host : nullptr, st);
        if (e == hipSuccess && whole) e = fill(base + nodes_at, most);
    }
    if (e == hipSuccess) e = word.wait(scratch + input_groups(npix, NCH), st, &total);
    if (e == hipSuccess && total < 0) e = hipErrorUnknown;
    if (e == hipSuccess) {
        in->nnz = total;
        if (whole) {
            in->unused = 8 * (npix * C - total);
            if (total >= input_dense_from(npix, C)) in->dense = reinterpret_cast<float *>(static_cast<char *>(in->ptr_block) + dense_at);
            else in->unused += 4 * npix * C;
            unused_bytes += in->unused;
        } else {
            const size_t n = (size_t)total + kSiSpare;
            e = block_alloc(input_pool(), dev, st, &in->node_block, val_at(n) + n * sizeof(float), &in->node_bytes);
            if (e == hipSuccess) e = fill(in->node_block, n);
        }
    }
    if (e == hipSuccess) e = hipEventCreateWithFlags(&in->filled, hipEventDisableTiming);
    if (e == hipSuccess) e = hipEventRecord(in->filled, st);
    if (e != hipSuccess) {
        (void)hipGetLastError();
        (void)hipStreamSynchronize(st);   // nothing may still write into what is freed next
        if (in->filled) (void)hipEventDestroy(in->filled);
        if (in->ptr_block) (void)hipFree(in->ptr_block);
        if (in->node_block) (void)hipFree(in->node_block);
        unused_bytes -= in->unused;
        in->magic = 0;
        delete in;
        return e == hipErrorOutOfMemory ? FSCNN_ERR_ALLOC : FSCNN_ERR_DEVICE;
    }
    *out = in;
    return FSCNN_OK;
}

fscnn_status_t fscnn_input_compress(const float *x_dev, int N, int C, int H, int W, void *stream,
                                    fscnn_input_t **out)
{
    if (!x_dev || !out) return FSCNN_ERR_NULL;
    return compress_activations(x_dev, N, C, H, W, (hipStream_t)stream, out);
}

namespace {

// Where the parts of an emitted handle's one allocation start (256-byte aligned parts): pointer
// array | counts | scratch of the passes | indices | values | the dense result when the caller takes none.
struct EmitLayout {
    long long nstep, dense;
    size_t cnt_at, sum_at, idx_at, val_at, y_at;
    size_t bytes(bool with_y) const { return y_at + (with_y ? sizeof(float) * (size_t)dense : 0); }
};

EmitLayout emit_layout(long long npix, int K, int NCH)
{
    EmitLayout L;
    L.nstep = npix * NCH;
    L.dense = npix * K;
    auto up = [](size_t v) { return (v + 255) / 256 * 256; };
    L.cnt_at = up((size_t)(L.nstep + 1) * sizeof(int));
    L.sum_at = L.cnt_at + up(sizeof(int) * (size_t)L.nstep);
    L.idx_at = L.sum_at + up(sizeof(int) * (size_t)input_scratch_elems(npix, NCH));
    L.val_at = L.idx_at + up(sizeof(uint32_t) * (size_t)(L.dense + kSiSpare));
    L.y_at = L.val_at + up(sizeof(float) * (size_t)(L.dense + kSiSpare));
    return L;
}

// Argument checks shared by the two emitting calls; fills the result's shape.
fscnn_status_t emit_check(fscnn_filter_t *f, int N, int C, int H, int W, int sh, int sw, int ph,
                          int pw, int *Ho, int *Wo, int *NCH)
{
    if (!live(f)) return FSCNN_ERR_HANDLE;
    if (N <= 0 || C <= 0) return FSCNN_ERR_SHAPE;
    fscnn_status_t s = out_shape(H, W, f->R, f->S, sh, sw, ph, pw, Ho, Wo);
    if (s != FSCNN_OK) return s;
    const long long npix = (long long)N * *Ho * *Wo, dense = npix * f->K;
    if (!fits_int(dense) || !fits_int(dense + kSiSpare)) return FSCNN_ERR_UNSUPPORTED;
    *NCH = (f->K + kSiCC - 1) / kSiCC;
    if (!fits_int(npix * *NCH + 1) || *NCH > 8192 / kSiCC) return FSCNN_ERR_UNSUPPORTED;
    return FSCNN_OK;
}

// The work of an emitting call on a handle whose allocation is in place: the convolution with its
// bias / activation epilogue (which, where the launch can, counts the non-zero results per pixel
// and step of 8 channels itself), else a count pass, one scan, one pass that writes the pairs.
fscnn_status_t emit_run(fscnn_filter_t *f, const float *x_dev, int N, int C, int H, int W, int sh,
                        int sw, int ph, int pw, const float *bias_dev, int relu, float *y_dev,
                        void *stream, fscnn_input_t *in)
{
    hipStream_t st = (hipStream_t)stream;
    if (st) in->in_order = false;
    const int K = f->K, Ho = in->H, Wo = in->W;
    const EmitLayout L = emit_layout((long long)N * Ho * Wo, K, in->NCH);
    char *base = static_cast<char *>(in->ptr_block);
    int *cnt = reinterpret_cast<int *>(base + L.cnt_at);
    float *own = in->emit_has_y ? reinterpret_cast<float *>(base + L.y_at) : nullptr, *y = y_dev ? y_dev : own;
    bool counted = false;
    fscnn_status_t s = conv_sf_common(f, x_dev, N, C, H, W, sh, sw, ph, pw, bias_dev, relu, y,
                                      FSCNN_LAYOUT_NCHW, FSCNN_LAYOUT_NCHW, 0, 0, stream, cnt, &counted);
    if (s != FSCNN_OK) return s;
    hipError_t e = hipSuccess;
    int *scratch = reinterpret_cast<int *>(base + L.sum_at);
    const bool scanned = input_scans((long long)N * Ho * Wo, in->NCH);
    e = launch_input_sums(y, counted ? cnt : nullptr, N, K, Ho, Wo, in->NCH, scratch, scanned, nullptr, st);
    if (e == hipSuccess) e = launch_input_fill(y, N, K, Ho, Wo, in->NCH, scratch, scanned, in->cptr, in->cidx, in->xval, kSiSpare,
                                               y_dev ? own : nullptr, 0, nullptr, st);   // (the count may not be looked at: a replay brings another)
    if (e == hipSuccess) e = hipEventRecord(in->filled, st);
    if (e != hipSuccess) {
        (void)hipGetLastError();
        return e == hipErrorOutOfMemory ? FSCNN_ERR_ALLOC : FSCNN_ERR_DEVICE;
    }
    in->nnz = -1;
    in->dense = own;   // stays as it is until the next fill
    in->made_on = st;
    return FSCNN_OK;
}

}  // namespace

fscnn_status_t fscnn_conv2d_sparse_filter_emit(fscnn_filter_t *f, const float *x_dev, int N, int C,
                                               int H, int W, int sh, int sw, int ph, int pw,
                                               const float *bias_dev, int relu, float *y_dev,
                                               void *stream, fscnn_input_t **out)
{
    if (!f || !x_dev || !out) return FSCNN_ERR_NULL;
    int Ho, Wo, NCH;
    fscnn_status_t s = emit_check(f, N, C, H, W, sh, sw, ph, pw, &Ho, &Wo, &NCH);
    if (s != FSCNN_OK) return s;
    int dev;
    s = have_device(&dev);
    if (s != FSCNN_OK) return s;
    fscnn_input_t *in = new (std::nothrow) fscnn_input();
    if (!in) return FSCNN_ERR_ALLOC;
    in->magic = kInputMagic;
    in->device = dev;
    in->N = N; in->C = f->K; in->H = Ho; in->W = Wo;
    in->nnz = -1; in->CC = kSiCC; in->NCH = NCH;
    in->ptr_block = nullptr; in->node_block = nullptr;
    in->made_on = (hipStream_t)stream; in->filled = nullptr;
    // ONE allocation, sized for the worst case (every result non-zero), so that nothing here waits
    // for the device
    const EmitLayout L = emit_layout((long long)N * Ho * Wo, f->K, NCH);
    in->emit_bytes = L.bytes(y_dev == nullptr);
    in->emit_has_y = y_dev == nullptr;
    hipError_t e = block_alloc(input_pool(), dev, (hipStream_t)stream, &in->ptr_block, in->emit_bytes, &in->ptr_bytes);
    if (e == hipSuccess) e = hipEventCreateWithFlags(&in->filled, hipEventDisableTiming);
    if (e != hipSuccess) {
        (void)hipGetLastError();
        if (in->ptr_block) (void)hipFree(in->ptr_block);
        delete in;
        return FSCNN_ERR_ALLOC;
    }
    char *base = static_cast<char *>(in->ptr_block);
    in->cptr = reinterpret_cast<int *>(base);
    in->cidx = reinterpret_cast<uint32_t *>(base + L.idx_at);
    in->xval = reinterpret_cast<float *>(base + L.val_at);
    s = emit_run(f, x_dev, N, C, H, W, sh, sw, ph, pw, bias_dev, relu, y_dev, stream, in);
    if (s != FSCNN_OK) {
        (void)hipStreamSynchronize((hipStream_t)stream);   // nothing may still write into what is freed next
        (void)hipEventDestroy(in->filled);
        (void)hipFree(in->ptr_block);
        in->magic = 0;
        delete in;
        return s;
    }
    *out = in;
    return FSCNN_OK;
}

fscnn_status_t fscnn_conv2d_sparse_filter_emit_into(fscnn_filter_t *f, const float *x_dev, int N,
                                                    int C, int H, int W, int sh, int sw, int ph,
                                                    int pw, const float *bias_dev, int relu,
                                                    float *y_dev, void *stream, fscnn_input_t *into)
{
    if (!f || !x_dev || !into) return FSCNN_ERR_NULL;
    if (!live(into)) return FSCNN_ERR_HANDLE;
    int Ho, Wo, NCH;
    fscnn_status_t s = emit_check(f, N, C, H, W, sh, sw, ph, pw, &Ho, &Wo, &NCH);
    if (s != FSCNN_OK) return s;
    int dev;
    s = have_device(&dev);
    if (s != FSCNN_OK) return s;
    if (into->device != dev) return FSCNN_ERR_MISMATCH;
    // only a handle that an emitting call made, for a result of this very shape, has the room
    if (into->emit_bytes == 0) return FSCNN_ERR_UNSUPPORTED;
    if (into->N != N || into->C != f->K || into->H != Ho || into->W != Wo) return FSCNN_ERR_MISMATCH;
    if (!y_dev && !into->emit_has_y) return FSCNN_ERR_NULL;
    return emit_run(f, x_dev, N, C, H, W, sh, sw, ph, pw, bias_dev, relu, y_dev, stream, into);
}

fscnn_status_t fscnn_input_info(const fscnn_input_t *in, int *N, int *C, int *H, int *W,
                                long long *nnz)
{
    if (!in) return FSCNN_ERR_NULL;
    if (!live(in)) return FSCNN_ERR_HANDLE;
    if (N) *N = in->N;
    if (C) *C = in->C;
    if (H) *H = in->H;
    if (W) *W = in->W;
    if (nnz) {
        *nnz = input_nnz(in);
        if (*nnz < 0) return FSCNN_ERR_DEVICE;
    }
    return FSCNN_OK;
}

fscnn_status_t fscnn_input_export(const fscnn_input_t *in, int *prow_host, unsigned *cidx_host,
                                  float *val_host)
{
    if (!in || !prow_host) return FSCNN_ERR_NULL;
    if (!live(in)) return FSCNN_ERR_HANDLE;
    const long long stored = input_nnz(in);
    if (stored < 0) return FSCNN_ERR_DEVICE;
    if (stored > 0 && (!cidx_host || !val_host)) return FSCNN_ERR_NULL;
    FSCNN_HIP(hipEventSynchronize(in->filled));
    // the row pointers are every NCH-th chunk pointer
    const size_t npix = (size_t)in->N * in->H * in->W;
    FSCNN_HIP(hipMemcpy2D(prow_host, sizeof(int), in->cptr, sizeof(int) * (size_t)in->NCH, sizeof(int), npix,
                          hipMemcpyDeviceToHost));
    FSCNN_HIP(hipMemcpy(prow_host + npix, in->cptr + npix * (size_t)in->NCH, sizeof(int), hipMemcpyDeviceToHost));
    if (stored > 0) {
        FSCNN_HIP(hipMemcpy(cidx_host, in->cidx, sizeof(uint32_t) * (size_t)stored, hipMemcpyDeviceToHost));
        FSCNN_HIP(hipMemcpy(val_host, in->xval, sizeof(float) * (size_t)stored, hipMemcpyDeviceToHost));
    }
    return FSCNN_OK;
}

fscnn_status_t fscnn_input_destroy(fscnn_input_t *in)
{
    if (!in) return FSCNN_ERR_NULL;
    if (!live(in)) return FSCNN_ERR_HANDLE;
    in->magic = 0;
    const bool in_order = in->in_order;
    if (!in_order) (void)hipEventSynchronize(in->filled);
    (void)hipEventDestroy(in->filled);
    size_t largest = std::max(in->ptr_bytes, in->node_bytes);
    for (auto &b : in->banks) largest = std::max(largest, b.bytes);
    const Left left = blocks_left(in->device, in_order, largest);
    block_free(input_pool(), in->device, in->ptr_block, in->ptr_bytes, left);
    block_free(input_pool(), in->device, in->node_block, in->node_bytes, left);
    for (auto &b : in->banks) block_free(input_pool(), in->device, b.buf, b.bytes, left);
    unused_bytes -= in->unused;
    delete in;
    return FSCNN_OK;
}

fscnn_status_t fscnn_conv2d_sparse_input(const fscnn_input_t *in, const float *w_dev, int K, int R,
                                         int S, int sh, int sw, int ph, int pw,
                                         const float *bias_dev, int relu, float *y_dev, void *stream)
{
    if (!in || !w_dev || !y_dev) return FSCNN_ERR_NULL;
    if (!live(in)) return FSCNN_ERR_HANDLE;
    if (K <= 0) return FSCNN_ERR_SHAPE;
    int Ho, Wo;
    fscnn_status_t s = out_shape(in->H, in->W, R, S, sh, sw, ph, pw, &Ho, &Wo);
    if (s != FSCNN_OK) return s;
    if (!fits_int((long long)K * in->C * R * S) || !fits_int((long long)in->N * K * Ho * Wo))
        return FSCNN_ERR_UNSUPPORTED;
    int dev;
    s = have_device(&dev);
    if (s != FSCNN_OK) return s;
    if (dev != in->device) return FSCNN_ERR_MISMATCH;
    hipStream_t st = (hipStream_t)stream;
    SiChoice c;
    void *bank = nullptr;
    std::unique_lock<std::mutex> launching(in->mu, std::defer_lock);
    const bool chosen = si_tiled_supported(K, in->C, R, S, sh, sw);
    if (chosen) {
        c = si_choose(in->N, in->C, in->H, in->W, K, Ho, Wo, pw, false);
        if (in->dense && (in->nnz < 0 ? c.split_from <= (long long)in->N * in->C * in->H * in->W : in->nnz >= c.split_from)) {
            launching.lock();
            bank = bank_scratch(in, st, (size_t)split_packed_bytes(K, in->C, 9));
        }
    }
    FSCNN_HIP(after_fill(in, st));
    FSCNN_HIP(launch_conv_si(in, w_dev, K, R, S, Ho, Wo, sh, sw, ph, pw, bias_dev, relu, y_dev, chosen ? &c : nullptr, bank, st));
    return FSCNN_OK;
}

fscnn_status_t fscnn_dense_filter_prepare(const float *w_dev, int K, int C, int R, int S, void *stream,
                                          fscnn_dense_t **out)
{
    if (!w_dev || !out) return FSCNN_ERR_NULL;
    if (K <= 0 || C <= 0 || R <= 0 || S <= 0) return FSCNN_ERR_SHAPE;
    const int Kpad = (K + 255) / 256 * 256;
    if (!fits_int((long long)K * C * R * S) || !fits_int((long long)Kpad * C * R * S)) return FSCNN_ERR_SHAPE;
    int dev;
    fscnn_status_t s = have_device(&dev);
    if (s != FSCNN_OK) return s;
    fscnn_dense_t *d = new (std::nothrow) fscnn_dense();
    if (!d) return FSCNN_ERR_ALLOC;
    d->magic = kDenseMagic;
    d->device = dev;
    d->K = K; d->C = C; d->R = R; d->S = S; d->Kpad = Kpad;
    d->wT = nullptr;
    const size_t words = (size_t)Kpad * C * R * S;
    bool pack = R == 3 && S == 3;   // what the prepared calls serve
    const size_t packed = pack ? (size_t)Kpad * ((C + 15) / 16 * 16) * 9 : 0;
    const size_t two = (sizeof(float) * (words + packed) + 256 + 255) / 256 * 256;
    bool parts = pack;
    hipError_t e = device_alloc(reinterpret_cast<void **>(&d->wT), parts ? two + (size_t)split_packed_bytes(K, C, 9) : two);
    if (e == hipErrorOutOfMemory && parts) {   // without the third copy
        (void)hipGetLastError();
        parts = false;
        e = device_alloc(reinterpret_cast<void **>(&d->wT), two);
    }
    if (e == hipErrorOutOfMemory && pack) {   // without the second copy: the gather kernels serve every call
        (void)hipGetLastError();
        pack = false;
        e = device_alloc(reinterpret_cast<void **>(&d->wT), sizeof(float) * words);
    }
    d->packed = pack ? d->wT + words : nullptr;
    d->flag = pack ? reinterpret_cast<int *>(d->packed + packed) : nullptr;
    d->parts = parts ? reinterpret_cast<char *>(d->wT) + two : nullptr;
    if (e == hipSuccess)
        e = pack ? launch_pack_dense(w_dev, K, C, Kpad, d->packed, d->wT, d->flag, (hipStream_t)stream)
                 : launch_dense_transpose(w_dev, K, C, R * S, Kpad, d->wT, (hipStream_t)stream);
    if (e == hipSuccess && parts) e = launch_split_bank(w_dev, K, C, d->parts, (hipStream_t)stream);
    if (e != hipSuccess) {
        (void)hipGetLastError();
        if (d->wT) (void)hipFree(d->wT);
        d->magic = 0;
        delete d;
        return e == hipErrorOutOfMemory ? FSCNN_ERR_ALLOC : FSCNN_ERR_DEVICE;
    }
    *out = d;
    return FSCNN_OK;
}

fscnn_status_t fscnn_dense_filter_destroy(fscnn_dense_t *d)
{
    if (!d) return FSCNN_ERR_NULL;
    if (!live(d)) return FSCNN_ERR_HANDLE;
    d->magic = 0;
    if (d->wT) (void)hipFree(d->wT);
    delete d;
    return FSCNN_OK;
}

int fscnn_si_variant_count(void) { return si_variant_count(); }

fscnn_status_t fscnn_conv2d_sparse_input_prepared(const fscnn_input_t *in, const fscnn_dense_t *d,
                                                  int sh, int sw, int ph, int pw,
                                                  const float *bias_dev, int relu, float *y_dev,
                                                  int variant, void *stream)
{
    if (!in || !d || !y_dev) return FSCNN_ERR_NULL;
    if (!live(in) || !live(d)) return FSCNN_ERR_HANDLE;
    if (d->C != in->C) return FSCNN_ERR_MISMATCH;
    int Ho, Wo;
    fscnn_status_t s = out_shape(in->H, in->W, d->R, d->S, sh, sw, ph, pw, &Ho, &Wo);
    if (s != FSCNN_OK) return s;
    if (variant < 0 || variant > si_variant_count()) return FSCNN_ERR_UNSUPPORTED;
    // the prepared form serves 3x3 / stride 1; other geometries take fscnn_conv2d_sparse_input
    if (d->R != 3 || d->S != 3 || sh != 1 || sw != 1) return FSCNN_ERR_UNSUPPORTED;
    if (!fits_int((long long)in->N * d->K * Ho * Wo)) return FSCNN_ERR_UNSUPPORTED;
    int dev;
    s = have_device(&dev);
    if (s != FSCNN_OK) return s;
    if (dev != in->device || dev != d->device) return FSCNN_ERR_MISMATCH;
    FSCNN_HIP(after_fill(in, (hipStream_t)stream));
    FSCNN_HIP(launch_conv_si_prepared(in, d, Ho, Wo, ph, pw, bias_dev, relu, y_dev, variant,
                                      (hipStream_t)stream));
    return FSCNN_OK;
}

long long fscnn_sparse_transpose_workspace(long long new_rows, long long nnz)
{
    return reorder_workspace_bytes(new_rows, nnz);
}

static fscnn_status_t reorder_common(bool tensor, const int *rowptr, const unsigned *idx,
                                     const float *val, int n_rows, int n_cols, int H,
                                     long long n_buckets, long long nnz, int *tptr,
                                     unsigned *tidx, float *tval, void *ws, long long ws_bytes,
                                     void *stream)
{
    if (!rowptr || !tptr || !ws) return FSCNN_ERR_NULL;
    if (nnz < 0 || nnz >= (1LL << 31)) return FSCNN_ERR_SHAPE;
    if (nnz > 0 && (!idx || !val || !tidx || !tval)) return FSCNN_ERR_NULL;
    if (!fits_int(n_buckets + 1)) return FSCNN_ERR_UNSUPPORTED;
    const long long need = reorder_workspace_bytes(n_buckets, nnz);
    if (need < 0 || ws_bytes < need || ((uintptr_t)ws & 3)) return FSCNN_ERR_UNSUPPORTED;
    int dev;
    fscnn_status_t s = have_device(&dev);
    if (s != FSCNN_OK) return s;
    FSCNN_HIP(launch_reorder(tensor, rowptr, idx, val, n_rows, n_cols, H, n_buckets, nnz, tptr, tidx,
                             tval, ws, (hipStream_t)stream));
    return FSCNN_OK;
}

fscnn_status_t fscnn_sparse_transpose(const int *rowptr_dev, const unsigned *idx_dev,
                                      const float *val_dev, int n_rows, int n_cols, long long nnz,
                                      int *tptr_dev, unsigned *tidx_dev, float *tval_dev,
                                      void *workspace_dev, long long workspace_bytes, void *stream)
{
    if (n_rows <= 0 || n_cols <= 0) return FSCNN_ERR_SHAPE;
    return reorder_common(false, rowptr_dev, idx_dev, val_dev, n_rows, n_cols, 1, n_cols, nnz,
                          tptr_dev, tidx_dev, tval_dev, workspace_dev, workspace_bytes, stream);
}

fscnn_status_t fscnn_sparse_transpose_noalloc(const int *rowptr_dev, const unsigned *idx_dev,
                                              const float *val_dev, int n_rows, int n_cols,
                                              long long nnz, int *tptr_dev, unsigned *tidx_dev,
                                              float *tval_dev, void *stream)
{
    if (n_rows <= 0 || n_cols <= 0) return FSCNN_ERR_SHAPE;
    if (!rowptr_dev || !tptr_dev) return FSCNN_ERR_NULL;
    if (nnz < 0 || nnz >= (1LL << 31)) return FSCNN_ERR_SHAPE;
    const long long need = reorder_workspace_bytes(n_cols, nnz);
    if (need < 0 || need > kStaticScratchBytes) return FSCNN_ERR_UNSUPPORTED;   // beyond the static scratch
    int dev;
    fscnn_status_t s = have_device(&dev);
    if (s != FSCNN_OK) return s;
    void *ws = nullptr;
    FSCNN_HIP(static_scratch(&ws));
    return reorder_common(false, rowptr_dev, idx_dev, val_dev, n_rows, n_cols, 1, n_cols, nnz, tptr_dev,
                          tidx_dev, tval_dev, ws, kStaticScratchBytes, stream);
}

fscnn_status_t fscnn_sparse_tensor_transpose(const int *rowptr_dev, const unsigned *widx_dev,
                                             const float *val_dev, int W, int H, int C,
                                             long long nnz, int *tptr_dev, unsigned *cidx_dev,
                                             float *tval_dev, void *workspace_dev,
                                             long long workspace_bytes, void *stream)
{
    if (W <= 0 || H <= 0 || C <= 0) return FSCNN_ERR_SHAPE;
    if (!fits_int((long long)C * H + 1) || !fits_int((long long)W * H + 1)) return FSCNN_ERR_SHAPE;
    return reorder_common(true, rowptr_dev, widx_dev, val_dev, C * H, W, H, (long long)W * H, nnz,
                          tptr_dev, cidx_dev, tval_dev, workspace_dev, workspace_bytes, stream);
}

fscnn_status_t fscnn_maxpool2x2_ex(const float *x_dev, int N, int C, int H, int W, float *y_dev,
                                   fscnn_layout_t layout, void *stream)
{
    if (!x_dev || !y_dev) return FSCNN_ERR_NULL;
    if (N <= 0 || C <= 0 || H < 2 || W < 2) return FSCNN_ERR_SHAPE;
    if (layout != FSCNN_LAYOUT_NCHW && layout != FSCNN_LAYOUT_N4) return FSCNN_ERR_UNSUPPORTED;
    const int n4 = layout == FSCNN_LAYOUT_N4;
    if (!fits_int(((long long)N + 3) / 4 * 4 * C * H * W)) return FSCNN_ERR_UNSUPPORTED;
    if (n4 && (((uintptr_t)x_dev | (uintptr_t)y_dev) & 15)) return FSCNN_ERR_UNSUPPORTED;
    int dev;
    fscnn_status_t s = have_device(&dev);
    if (s != FSCNN_OK) return s;
    FSCNN_HIP(launch_maxpool2x2(x_dev, N, C, H, W, y_dev, n4, (hipStream_t)stream));
    return FSCNN_OK;
}

fscnn_status_t fscnn_maxpool2x2(const float *x_dev, int N, int C, int H, int W, float *y_dev,
                                void *stream)
{
    return fscnn_maxpool2x2_ex(x_dev, N, C, H, W, y_dev, FSCNN_LAYOUT_NCHW, stream);
}

}  // extern "C"
